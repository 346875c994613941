// Sweeps of narrow trees (nx + nu <= 32) in bands of stages: Algorithms 3 and
// 4 of arXiv 2107.01745, Sec. III-D, with the recursion of sweep.hip, for the
// stages whose cost is latency and not bandwidth.
//
// A band is a run of consecutive stages; one workgroup takes one subtree of
// the band (the nodes below one node of its first stage) through all of the
// band's stages in one launch, so a tree of a dozen stages takes a handful of
// launches instead of one per stage and direction.  The first band of every
// instance is one subtree (the root's): its workgroup does the backward and
// then the forward pass in the same launch.  Between bands the launches pass
// qhat (backward) and x (forward) through memory; inside a band they stay in
// LDS.
//
// A lane group of G = 8 or 16 lanes per node (2G >= nx + nu), a column
// pair per lane, 64 / G nodes per wavefront, dealt to the wavefronts in a fixed
// order (deterministic).  The per-edge product is formed on the child's side:
// node i turns its children's vectors p_j and its own terms into qhat_i and
// sends p_i = [A_i B_i]' qhat_i up, so a node's work does not grow with its
// children and every product of a stage runs in parallel.
//
// What bounds it: the chain of dependent steps, one per stage, and the
// instructions in it (a wavefront has its SIMD to itself).  What a wavefront's
// next nodes need (their matrices' first rows, their own vector entries) is
// requested before the barrier in front of them.  A stage takes about 1.1 us in
// each direction (nx=4, nu=2: 12 steps in 16 us, 24 with barriers that wait for
// the loads in flight and a select per row), where a launch per stage took 6.
#include <algorithm>

#include "sweep_common.h"

namespace stotree {

namespace {

using namespace dev;

constexpr int kBandWidth = 32;       // largest padded nx + nu
constexpr int kBandWaves = 8;        // most wavefronts of a workgroup
constexpr int kBandLdsDoubles = 5120;  // LDS of the node vectors of two stages, two right-hand sides (doubles)
constexpr int kBandSlack = 16;       // doubles past the last vector that a product's last batch may read
constexpr int kBandMaxNodes = 64;    // most nodes of one stage of a subtree

// An LDS-only barrier: the wavefronts meet with their LDS accesses done, but
// the loads requested for their next nodes stay in flight (__syncthreads
// waits for those too, a memory latency per stage).
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);           // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// The product of the nodes' matrices (n rows of ldb bytes at a
// wavefront-uniform base plus this lane's byte offset) with vectors in LDS, in
// batches of RB rows: open requests the first batch, ready the second (when
// the product's input is about to be formed), run the later ones while earlier
// ones are multiplied.  Loads past the end re-read the last row, so no load and
// no LDS read sits under a branch.
template <int RB>
struct Rows {
    const char *M;
    unsigned off;
    int ldb, n;
    double2 m0[RB], m1[RB];

    __device__ __forceinline__ void load(double2 (&m)[RB], int b) const
    {
#pragma unroll
        for (int u = 0; u < RB; ++u) {
            const int r = b * RB + u;
            m[u] = *reinterpret_cast<const double2 *>(M + (off + (unsigned)((r < n ? r : n - 1) * ldb)));
        }
    }
    __device__ __forceinline__ void open(const double *base, unsigned off_, int ld, int n_)
    {
        M = reinterpret_cast<const char *>(base);
        off = off_;
        ldb = ld * (int)sizeof(double);
        n = n_;
        load(m0, 0);
    }
    __device__ __forceinline__ void ready()
    {
        if (n > RB) load(m1, 1);
    }
    template <int NRHS>
    __device__ __forceinline__ void mul(const double2 (&m)[RB], int b, const double *v, int ldv,
                                        double (&acc)[NRHS][2]) const
    {
        double w[NRHS][RB];
#pragma unroll
        for (int k = 0; k < NRHS; ++k)
#pragma unroll
            for (int u = 0; u < RB; ++u) w[k][u] = v[k * ldv + b * RB + u];
        auto add = [&](int u) {
#pragma unroll
            for (int k = 0; k < NRHS; ++k) {
                acc[k][0] = fma(m[u].x, w[k][u], acc[k][0]);
                acc[k][1] = fma(m[u].y, w[k][u], acc[k][1]);
            }
        };
        // only the rows there are, from the last one down (a jump, no select per row)
        static_assert(RB == 4 || RB == 6, "cases below");
        const int left = n - b * RB;
        switch (left < RB ? left : RB) {
        case 6: add(RB - 1); [[fallthrough]];
        case 5: add(RB == 6 ? 4 : 0); [[fallthrough]];
        case 4: add(3); [[fallthrough]];
        case 3: add(2); [[fallthrough]];
        case 2: add(1); [[fallthrough]];
        default: add(0);
        }
    }
    template <int NRHS>
    __device__ __forceinline__ void run(const double *v, int ldv, double (&acc)[NRHS][2])
    {
#pragma unroll
        for (int k = 0; k < NRHS; ++k) acc[k][0] = acc[k][1] = 0.0;
        const int nb = (n + RB - 1) / RB;
        for (int b = 0; b < nb; b += 2) {
            mul<NRHS>(m0, b, v, ldv, acc);
            if (b + 2 < nb) load(m0, b + 2);
            if (b + 1 < nb) {
                mul<NRHS>(m1, b + 1, v, ldv, acc);
                if (b + 3 < nb) load(m1, b + 3);
            }
        }
    }
};

constexpr int kRowsM = 6;            // rows per batch: [A B] (backward), [A B]' and K' (forward)
constexpr int kRowsK = 4;            // K and R~^{-1}

// One subtree's table: its stages lev = 0 .. nlev-1 (0: its root; nlev-1: the
// children of the band's last stage), stage lev holding the nodes [lo(lev),
// lo(lev) + cnt(lev)), and its chunks: a stage's nodes by 64 / G, one chunk a
// wavefront's work, listed from the deepest stage up (first node within the
// stage, times 64, plus the stage).  Chunks are dealt to the wavefronts in
// turn, so that a wavefront's next chunk is a workgroup's worth of chunks away
// and its loads, requested when the chunk before it is done, have that long to
// arrive.  Lane lev holds stage lev's pair and lane c the wavefront's c-th
// chunk of the next 64, so the table is read once.  (Nothing a node needs
// from memory goes through scalar loads: a wait for one of those waits for all
// that are outstanding, the next node's included.)
struct Subtree {
    const int *chunks;
    int vlo, vcnt, nlev, t0, nchunks;
    int task, vtask;                 // the wavefront's current chunk, its chunks by lane
    __device__ __forceinline__ Subtree(const int *tab, int lane)
    {
        const int v = tab[lane & 3];
        nlev = __builtin_amdgcn_readlane(v, 0);
        t0 = __builtin_amdgcn_readlane(v, 1);
        nchunks = __builtin_amdgcn_readlane(v, 2);
        const int lev = lane < nlev ? lane : nlev - 1;
        vlo = tab[4 + 2 * lev];
        vcnt = tab[5 + 2 * lev];
        chunks = tab + 4 + 2 * nlev;
    }
    __device__ __forceinline__ int lo(int lev) const { return __builtin_amdgcn_readlane(vlo, lev); }
    __device__ __forceinline__ int cnt(int lev) const { return __builtin_amdgcn_readlane(vcnt, lev); }
    // chunk `task` of the wavefront (down: in the order listed, else from the end): its stage and first
    // node; stage -1 past the last one
    template <bool UP>
    __device__ __forceinline__ void next(int wave, int lane, int &lev, int &k)
    {
        if ((task & (kWave - 1)) == 0) {
            const int q = wave + (task + lane) * (int)(blockDim.x / kWave);
            vtask = q < nchunks ? chunks[UP ? q : nchunks - 1 - q] : -1;
        }
        const int c = __builtin_amdgcn_readlane(vtask, task & (kWave - 1));
        ++task;
        lev = c < 0 ? -1 : c & 63;
        k = c >> 6;
    }
};

template <int NRHS, int G>
__device__ __forceinline__ void band_bwd(const SweepArgs &a, const InstDesc &I, Subtree &s, double *buf, int half,
                                         double *vec, int wave, int lane)
{
    const int nx = I.nx, nu = I.nu, W = nx + nu, ldM = I.ldM;
    const int edge = s.nlev - 1, c0 = 2 * (lane & (G - 1)), grp = lane / G;
    const bool leaf_edge = s.t0 + edge == I.N;    // the edge stage holds leaves
    const double *pM = a.Mb + I.Mb, *pK = a.Kb + I.Kb, *pR = a.Rn + I.Rn, *pch = a.chat + I.chat, *psg = a.sig + I.sig;
    const double *py = a.y + I.y, *psc = a.sc ? a.sc + I.sc : nullptr;
    // duals of leaf j: at Vnl nu + j nx
    const double *pe = leaf_edge ? py + (long long)I.Vnl * nu : a.qhat + I.x;
    const long long pe_rs = leaf_edge ? a.y_rs : a.qhat_rs;
    double *pk = a.kbuf + I.u, *pq = a.qhat + I.x;
    const int *pc = a.cp + I.cp;
    // column pairs this lane loads: lanes past the row re-read its first columns
    const unsigned cM = (c0 < W ? c0 : 0) * 8u, cX = (c0 < nx ? c0 : 0) * 8u, cU = (c0 < nu ? c0 : 0) * 8u;
    const unsigned e0 = c0 < W ? c0 : W - 1, e1 = c0 + 1 < W ? c0 + 1 : W - 1;     // this lane's entries of a node
    const unsigned x0 = c0 < nx ? c0 : nx - 1, x1 = c0 + 1 < nx ? c0 + 1 : nx - 1; // and of an edge node
    double *v = vec + grp * ldM;                  // [sum p ; own terms], its first nx entries then qhat
    const int ldv = kWave / G * ldM;
    Rows<kRowsM> m;
    Rows<kRowsK> kb, rn;
    double yv[NRHS][2], hv[2], sv;
    int ch0 = 0, ch1 = 0;
    int lev, k, i = 0, cnt = 0;
    // this group's node of the next chunk (the stage's last one past the end) and its loads
    auto fetch = [&]() {
        if (lev < 0) return;
        cnt = s.cnt(lev);
        i = s.lo(lev) + (k + grp < cnt ? k + grp : cnt - 1);
        sv = psc ? psc[(unsigned)i] : 1.0;
        if (lev == edge) {
            const unsigned o = (unsigned)i * nx;
            hv[0] = pch[o + x0];
            hv[1] = pch[o + x1];
#pragma unroll
            for (int r = 0; r < NRHS; ++r) {
                yv[r][0] = (pe + r * pe_rs)[o + x0];
                yv[r][1] = (pe + r * pe_rs)[o + x1];
            }
        } else {
            const unsigned ox = (unsigned)i * nx, ou = (unsigned)i * nu - nx, ow = (unsigned)i * W;
            hv[0] = *(e0 < (unsigned)nx ? pch + (ox + e0) : psg + (ou + e0));
            hv[1] = *(e1 < (unsigned)nx ? pch + (ox + e1) : psg + (ou + e1));
#pragma unroll
            for (int r = 0; r < NRHS; ++r) {
                yv[r][0] = (py + r * a.y_rs)[ow + e0];
                yv[r][1] = (py + r * a.y_rs)[ow + e1];
            }
            ch0 = pc[(unsigned)i];
            ch1 = pc[(unsigned)i + 1];
            rn.open(pR, (unsigned)i * (unsigned)(nu * I.ldu * 8) + cU, I.ldu, nu);
            kb.open(pK, (unsigned)i * (unsigned)(nu * I.ldx * 8) + cX, I.ldx, nu);
        }
        if (lev > 0) m.open(pM, (unsigned)i * (unsigned)(nx * ldM * 8) + cM, ldM, nx);
    };
    // -R~^{-1} g of the node just done: only the forward pass needs it, so it is
    // formed after the barrier, while the stage above is on its way, unless this
    // wavefront has a chunk of that stage (4,095-node two-mode tree 54 -> 49 us a
    // sweep)
    int ki = 0;
    bool kown = false;
    auto store_k = [&]() {
        double ra[NRHS][2];
        rn.template run<NRHS>(v + nx, ldv, ra);
        const unsigned ou = (unsigned)ki * nu + c0;
#pragma unroll
        for (int r = 0; r < NRHS; ++r)
#pragma unroll
            for (int e = 0; e < 2; ++e)
                if (c0 + e < nu && kown) (pk + r * a.kbuf_rs)[ou + e] = ra[r][e];
    };
    s.task = 0;
    s.next<true>(wave, lane, lev, k);
    fetch();
    for (int t = edge; t >= 0; --t) {
        bool behind = false;                       // k and the next chunk's loads are still to do
        const double *pb = buf + ((t + 1) & 1) * half + (c0 < ldM ? c0 : 0);
        double *pw = buf + (t & 1) * half + c0;
        const int lo1 = t < edge ? s.lo(t + 1) : 0;
        while (lev == t) {
            const int j = k + grp;
            const bool own = j < cnt;              // not a repeat of the stage's last node
            if (t > 0) m.ready();
            double w[NRHS][2];
            const bool lin = t < edge || leaf_edge;
            const double ws = lin ? sv : 1.0, wh0 = lin && a.affine ? hv[0] : 0.0, wh1 = lin && a.affine ? hv[1] : 0.0;
#pragma unroll
            for (int r = 0; r < NRHS; ++r) {
                w[r][0] = ws * yv[r][0] + wh0;
                w[r][1] = ws * yv[r][1] + wh1;
            }
            if (t < edge) {
                rn.ready();
                kb.ready();
                const double *pj = pb + (ch0 - lo1) * NRHS * ldM;
                for (int c = ch0; c < ch1; ++c, pj += NRHS * ldM)
#pragma unroll
                    for (int r = 0; r < NRHS; ++r) {
                        const double2 p = *reinterpret_cast<const double2 *>(pj + r * ldM);
                        w[r][0] += p.x;
                        w[r][1] += p.y;
                    }
            }
            if (c0 < ldM)
#pragma unroll
                for (int r = 0; r < NRHS; ++r)
                    *reinterpret_cast<double2 *>(v + r * ldv + c0) = make_double2(w[r][0], w[r][1]);
            wave_sync();
            if (t < edge) {
                double ka[NRHS][2];
                kb.template run<NRHS>(v + nx, ldv, ka);
                const unsigned ox = (unsigned)i * nx + c0;
                const bool out = t == 0 && i > 0 && own;
                ki = i;
                kown = own;
#pragma unroll
                for (int r = 0; r < NRHS; ++r)
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        if (c0 + e < nx) {
                            const double q = w[r][e] + ka[r][e];
                            v[r * ldv + c0 + e] = q;
                            if (out) (pq + r * a.qhat_rs)[ox + e] = q;
                        }
                    }
                wave_sync();
            }
            if (t > 0) {
                double pa[NRHS][2];
                m.template run<NRHS>(v, ldv, pa);
                if (c0 < ldM && own)
#pragma unroll
                    for (int r = 0; r < NRHS; ++r)
                        *reinterpret_cast<double2 *>(pw + (j * NRHS + r) * ldM) = make_double2(pa[r][0], pa[r][1]);
            }
            s.next<true>(wave, lane, lev, k);
            // (a chunk of the very next stage needs its loads now)
            behind = lev < t - 1;
            if (behind) break;
            if (t < edge) store_k();
            wave_sync();         // the next chunk overwrites v
            fetch();
        }
        if (t > 0) lds_barrier();
        if (behind) {
            if (t < edge) store_k();
            wave_sync();
            fetch();
        }
    }
}

template <int NRHS, int G>
__device__ __forceinline__ void band_fwd(const SweepArgs &a, const InstDesc &I, Subtree &s, double *buf, int half,
                                         int wave, int lane)
{
    const int nx = I.nx, nu = I.nu, W = nx + nu, ldM = I.ldM;
    const int edge = s.nlev - 1, c0 = 2 * (lane & (G - 1)), grp = lane / G;
    const bool leaf_edge = s.t0 + edge == I.N;
    const double *pM = a.Mf + I.Mf, *pK = a.Kf + I.Kf, *pc = a.cvec + I.c, *pk = a.kbuf + I.u;
    const int *pa = a.anc + I.sc;
    const unsigned cX = (c0 < nx ? c0 : 0) * 8u, cU = (c0 < nu ? c0 : 0) * 8u;
    const unsigned x0 = c0 < nx ? c0 : nx - 1, x1 = c0 + 1 < nx ? c0 + 1 : nx - 1;
    const unsigned u0 = c0 < nu ? c0 : nu - 1, u1 = c0 + 1 < nu ? c0 + 1 : nu - 1;
    // outputs: the dual layout (W rows per node, nx per leaf), or x and u
    double *px = a.xo + (a.dual_out ? I.y : I.x), *pu = a.dual_out ? a.xo + I.y + nx : a.uo + I.u;
    const int xs = a.dual_out ? W : nx, us = a.dual_out ? W : nu;
    const long long us_rs = a.dual_out ? a.xo_rs : a.uo_rs;
    double *pe = leaf_edge && a.dual_out ? px + (long long)I.Vnl * nu : px;     // the edge stage's x
    const int es = leaf_edge ? nx : xs;
    Rows<kRowsM> m, kf;
    double cv[2], kv[NRHS][2];       // entries added to the products
    double xr[NRHS][2];              // the subtree's root: x itself
    int par = 0;
    int lev, k, i = 0, cnt = 0;
    auto fetch = [&]() {
        if (lev < 0) return;
        cnt = s.cnt(lev);
        i = s.lo(lev) + (k + grp < cnt ? k + grp : cnt - 1);
        if (lev > 0) {
            const unsigned o = (unsigned)i * nx;
            cv[0] = pc[o + x0];
            cv[1] = pc[o + x1];
            par = pa[(unsigned)i];
            m.open(pM, (unsigned)i * (unsigned)(W * I.ldx * 8) + cX, I.ldx, W);
        } else {
            const double *src = i > 0 ? px + (unsigned)i * xs : a.x0 + I.x0;
            const long long rs = i > 0 ? a.xo_rs : a.x0_rs;
            const bool have = i > 0 || a.affine;
#pragma unroll
            for (int r = 0; r < NRHS; ++r) {
                xr[r][0] = have ? src[r * rs + x0] : 0.0;
                xr[r][1] = have ? src[r * rs + x1] : 0.0;
            }
        }
        if (lev < edge) {
            const unsigned o = (unsigned)i * nu;
#pragma unroll
            for (int r = 0; r < NRHS; ++r) {
                kv[r][0] = (pk + r * a.kbuf_rs)[o + u0];
                kv[r][1] = (pk + r * a.kbuf_rs)[o + u1];
            }
            kf.open(pK, (unsigned)i * (unsigned)(nx * I.ldu * 8) + cU, I.ldu, nx);
        }
    };
    s.task = 0;
    s.next<false>(wave, lane, lev, k);
    fetch();
    for (int t = 0; t <= edge; ++t) {
        const int lo1 = t > 0 ? s.lo(t - 1) : 0;
        while (lev == t) {
            const int j = k + grp;
            const bool own = j < cnt;
            // a repeat of the stage's last node writes the same values to the same place in LDS
            double *xu = buf + (t & 1) * half + (own ? j : cnt - 1) * NRHS * ldM;
            double x[NRHS][2];
            if (t == 0) {
#pragma unroll
                for (int r = 0; r < NRHS; ++r) { x[r][0] = xr[r][0]; x[r][1] = xr[r][1]; }
            } else {
                m.ready();
                const double *xp = buf + ((t - 1) & 1) * half + (par - lo1) * NRHS * ldM;
                m.template run<NRHS>(xp, ldM, x);
                const double h0 = a.affine ? cv[0] : 0.0, h1 = a.affine ? cv[1] : 0.0;
#pragma unroll
                for (int r = 0; r < NRHS; ++r) { x[r][0] += h0; x[r][1] += h1; }
            }
            if (t < edge) kf.ready();
            const bool store_x = own && (t > 0 || i == 0);
            double *po = t == edge ? pe : px;
            const unsigned ox = (unsigned)i * (t == edge ? es : xs) + c0, ou = (unsigned)i * us + c0;
#pragma unroll
            for (int r = 0; r < NRHS; ++r)
#pragma unroll
                for (int e = 0; e < 2; ++e)
                    if (c0 + e < nx) {
                        if (store_x) (po + r * a.xo_rs)[ox + e] = x[r][e];
                        if (t < edge) xu[r * ldM + c0 + e] = x[r][e];
                    }
            if (t < edge) {
                wave_sync();
                double ua[NRHS][2];
                kf.template run<NRHS>(xu, ldM, ua);
#pragma unroll
                for (int r = 0; r < NRHS; ++r)
#pragma unroll
                    for (int e = 0; e < 2; ++e)
                        if (c0 + e < nu) {
                            const double u = ua[r][e] + kv[r][e];
                            if (own) (pu + r * us_rs)[ou + e] = u;
                            xu[r * ldM + nx + c0 + e] = u;
                        }
            }
            s.next<false>(wave, lane, lev, k);
            fetch();
        }
        if (t < edge) lds_barrier();
    }
}

// Lists of one band's subtrees, by lane-group width (consecutive block ranges).
struct BandLists {
    int n;
    int G[2], half[2], ldM[2], first_block[3];
    const Item *items[2];       // (instance, offset of the subtree's table)
    const int *tabs;
};

// PASS 0: backward, 1: forward, 2: both (the first band: the subtree is the
// whole band, so the forward pass only needs this workgroup's results).
template <int NRHS, int G, int PASS>
__device__ __forceinline__ void band_body(const SweepArgs &a, const BandLists &bl, int c, double *lds)
{
    const Item it = bl.items[c][blockIdx.x - bl.first_block[c]];
    if (skipped(a, it.inst)) return;
    const InstDesc I = a.inst[it.inst];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x & (kWave - 1);
    Subtree s(bl.tabs + it.idx, lane);
    const int half = bl.half[c] * NRHS;
    double *vec = lds + 2 * half + wave * NRHS * (kWave / G) * bl.ldM[c];
    if (PASS != 1) band_bwd<NRHS, G>(a, I, s, lds, half, vec, wave, lane);
    if (PASS == 2) __syncthreads();      // the forward pass reads the k other wavefronts stored
    if (PASS != 0) band_fwd<NRHS, G>(a, I, s, lds, half, wave, lane);
}

template <int NRHS, int PASS>
__global__ void __launch_bounds__(kWave *kBandWaves, 1) band_kernel(SweepArgs a, BandLists bl)
{
    extern __shared__ double lds[];
    int c = 0;
    while (c + 1 < bl.n && (int)blockIdx.x >= bl.first_block[c + 1]) ++c;
    if (bl.G[c] == 8) band_body<NRHS, 8, PASS>(a, bl, c, lds);
    else band_body<NRHS, 16, PASS>(a, bl, c, lds);
}

// Nodes of a stage of a subtree whose vectors fit the LDS.
int band_nodes(const InstDesc &I)
{
    return std::min(kBandMaxNodes, kBandLdsDoubles / (4 * I.ldM));
}

}  // namespace

// Cuts of instance I into bands down to stage last: band b covers the stages
// [cut[b], cut[b+1]), as many as keep every stage of its subtrees within
// band_nodes.  Empty if the instance is too wide or a node has too many
// children for a band.
std::vector<int> band_cuts(const InstDesc &I, const int *sp, const int *cp, int last)
{
    std::vector<int> cut;
    if (I.ldM > kBandWidth || last < 1) return cut;
    // a node's offset in each matrix pool is a 32-bit byte offset
    const long long per = std::max({(long long)I.nx * I.ldM, (long long)(I.nx + I.nu) * I.ldx, (long long)I.nu * I.ldu,
                                    (long long)I.nu * I.ldx, (long long)I.nx * I.ldu});
    if (8LL * I.V * per >= 1LL << 32) return cut;
    const int most = band_nodes(I);
    cut.push_back(0);
    for (int t = 0; t < last;) {
        // the subtrees' node ranges, stage by stage: first node of each root's range
        std::vector<int> at(sp[t + 1] - sp[t] + 1);
        for (size_t r = 0; r < at.size(); ++r) at[r] = sp[t] + (int)r;
        int e = t;
        while (e < last) {
            std::vector<int> nx(at.size());
            int widest = 0;
            for (size_t r = 0; r < at.size(); ++r) nx[r] = cp[at[r]];
            for (size_t r = 0; r + 1 < at.size(); ++r) widest = std::max(widest, nx[r + 1] - nx[r]);
            if (widest > most || e - t >= kWave - 1) break;
            at.swap(nx);
            ++e;
        }
        if (e == t) return {};       // one node's children alone are too many
        cut.push_back(e);
        t = e;
    }
    return cut;
}

// Work lists of the bands; cuts[b] is instance b's cut list (empty: the
// instance runs per stage).  cp: host child pointers.
void build_bands(tree_factors *f, const std::vector<std::vector<int>> &cuts, ListArena &arena)
{
    f->bands.clear();
    f->band_tabs = nullptr;
    size_t nb = 0;
    for (const auto &c : cuts) nb = std::max(nb, c.size());
    if (nb < 2) return;
    std::vector<int> tabs;
    std::vector<std::vector<Item>> items((nb - 1) * 2);
    f->bands.resize(nb - 1);
    for (int b = 0; b < f->ninst; ++b) {
        const InstDesc &I = f->inst[b];
        const int *sp = f->sp_pool.data() + I.sp, *cp = f->cp_pool.data() + I.cp;
        const int cls = I.ldM <= 16 ? 0 : 1;
        for (size_t k = 0; k + 1 < cuts[b].size(); ++k) {
            BandPlan &bp = f->bands[k];
            const int t0 = cuts[b][k], t1 = cuts[b][k + 1];
            bp.ldM[cls] = std::max(bp.ldM[cls], I.ldM);
            for (int r = sp[t0]; r < sp[t0 + 1]; ++r) {
                items[2 * k + cls].push_back({b, (int)tabs.size()});
                const size_t head = tabs.size();
                tabs.insert(tabs.end(), {t1 - t0 + 1, t0, 0, 0});
                int lo = r, hi = r + 1;
                for (int t = t0; t <= t1; ++t) {
                    tabs.push_back(lo);
                    tabs.push_back(hi - lo);
                    bp.half[cls] = std::max(bp.half[cls], (hi - lo) * I.ldM);
                    if (t < t1) { lo = cp[lo]; hi = cp[hi]; }
                }
                const int per = kWave / (8 << cls);
                for (int lev = t1 - t0; lev >= 0; --lev)
                    for (int q = 0; q < tabs[head + 5 + 2 * lev]; q += per, ++tabs[head + 2]) {
                        tabs.push_back(q * 64 + lev);
                        // a wavefront for each chunk of the widest stage
                        while (bp.nw < kBandWaves && bp.nw * per <= q) bp.nw *= 2;
                    }
            }
        }
    }
    f->band_tabs = arena.put(tabs);
    for (size_t k = 0; k + 1 < nb; ++k)
        for (int c = 0; c < 2; ++c) {
            f->bands[k].count[c] = (int)items[2 * k + c].size();
            f->bands[k].items[c] = arena.put(items[2 * k + c]);
        }
}

template <int NRHS>
static void launch_band_n(const tree_factors *f, const SweepArgs &a, int band, int pass, hipStream_t st)
{
    const BandPlan &b = f->bands[band];
    BandLists bl{};
    size_t lds = 0;
    for (int c = 0; c < 2; ++c) {
        if (!b.count[c]) continue;
        bl.G[bl.n] = 8 << c;
        bl.half[bl.n] = b.half[c];
        bl.ldM[bl.n] = b.ldM[c];
        bl.items[bl.n] = b.items[c];
        bl.first_block[bl.n + 1] = bl.first_block[bl.n] + b.count[c];
        ++bl.n;
        lds = std::max(lds, sizeof(double) * NRHS * (2 * (size_t)b.half[c] + (size_t)b.nw * (kWave / (8 << c)) * b.ldM[c]) +
                                kBandSlack * sizeof(double));
    }
    bl.tabs = f->band_tabs;
    const dim3 grid(bl.first_block[bl.n]), blk(kWave * b.nw);
    if (pass == 0) hipLaunchKernelGGL((band_kernel<NRHS, 0>), grid, blk, lds, st, a, bl);
    else if (pass == 1) hipLaunchKernelGGL((band_kernel<NRHS, 1>), grid, blk, lds, st, a, bl);
    else hipLaunchKernelGGL((band_kernel<NRHS, 2>), grid, blk, lds, st, a, bl);
}

void launch_band(const tree_factors *f, const SweepArgs &a, int nrhs, int band, int pass, hipStream_t st)
{
    if (nrhs == 1) launch_band_n<1>(f, a, band, pass, st);
    else launch_band_n<2>(f, a, band, pass, st);
}

}  // namespace stotree
