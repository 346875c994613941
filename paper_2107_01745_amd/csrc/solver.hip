// Device-resident dual MINFBE (Algorithm 1) and NAMA (Algorithm 2) of
// arXiv 2107.01745, Sec. III-B/III-C, in the preconditioned dual variables of
// Sec. III-E when the handle asks for it.  A batched handle runs every
// instance in the same launches: each block of a vector pass belongs to one
// instance, each instance has its own control block (step, L-BFGS memory,
// stop flag), and finished instances are skipped by every kernel.
//
// Every iteration is a fixed sequence of kernels on the caller's stream; all
// scalars (residual norms, curvature test, L-BFGS coefficients, the accepted
// step) are reduced and decided on the device by single-block "finalize"
// kernels, so the host only reads a stop flag every check_every iterations,
// while the device works on.
// Once the flag is set every remaining kernel returns immediately.
//
// Vector passes (grid-stride over the m dual rows, row r of node i scaled by
// s_i = sqrt(pi_i)):
//   resid   z = proj_[s lo, s hi](y/lambda + s Hx), R = z - s Hx (Sec. II-D);
//           for NAMA also the L-BFGS pair s = y - y_prev, q = R - R_prev and
//           every inner product the compact L-BFGS form needs (one pass).
//   grad    (MINFBE) grad phi = R + lambda s H xhat(s R) (Sec. III-A), the
//           pair with the previous gradient, and the same inner products.
//   combine d = -B g in the compact representation of the L-BFGS inverse
//           Hessian (Byrd, Nocedal and Schnabel 1994), which equals the
//           two-loop recursion but needs one pass over the stored pairs.
//   ls      all trial steps tau = 2^-nu, nu = 0..nu_max, in one pass: since
//           x(.) is affine, H x(w) = s Hx + s H xhat(w - y) is formed from the
//           homogeneous sweeps already done, and the change of the FBE
//           phi(w) - phi(y) is accumulated row by row (Sec. III-B, the
//           tau-independent quantities of the line-search reformulation).
//   update  y+ = T_lambda(w) = w - lambda R(w).
//
// Also here: the accelerated dual proximal gradient GPAD (the warm start of
// Sec. III-F and the comparison method of Sec. IV-A), the two lambda
// backtracking tests of Sec. III-B, a primal-infeasibility test, soft rows
// (a weighted Huber function of the distance to the row's interval in
// place of the hard bound, Sec. II-B), and the constraint map z = [F G] (x, u)
// around the sweeps (cmap.hip).
#include <algorithm>
#include <cfloat>
#include <cmath>
#include <cstring>
#include <mutex>
#include <vector>

#include "internal.h"

namespace stotree {

namespace {

constexpr int kMemMax = 16;   // L-BFGS memory supported on the device
constexpr int kNuCap = 30;    // largest nu_max
constexpr int kNuDefault = 10; // default nu_max
constexpr int kVB = 256;      // threads per block of the vector kernels
constexpr int kFin = 512;     // threads per block of the finalize kernels

constexpr int kBtMax = 50;     // halvings of lambda before an instance gives up
constexpr int kTraceCols = 40; // trace row: lambda, res, accepted nu, nu_max, pairs, dphi[nu]...
constexpr int kTracePhi = 5;
constexpr double kEpsDiv = 1e-3;   // null-space tolerance of the infeasibility test
constexpr double kEpsObj = 1e-4;   // its bound on the objective's fall along d (see fin_div_kernel)
constexpr double kEpsNullGpad = 1e-4;  // its null-space part for GPAD (see fin_div_kernel)
constexpr int kDivHits = 2;        // consecutive windows that must pass it

// reduction slots
constexpr int R_MAX = 0, R_MAXU = 1, R_MAX3 = 2, R_SS = 3, R_BAD = 4, PB = 5;
constexpr int kNMax = 3;  // slots [0, kNMax) are max-reduced, the rest summed
constexpr int nv_pair(int memcap) { return PB + 6 + 5 * memcap; }
constexpr int kNVMax = nv_pair(kMemMax) > kNuCap + 3 + kNMax ? nv_pair(kMemMax) : kNuCap + 3 + kNMax;

struct Ctl {
    int done, status, iter, have_pair;
    int first_blk, nblk, skip, redo;      // skip: update undone by test 1; redo: see update_kernel
    int cnt, free_slot, pushes, skips;
    int ls_trials, sweeps_aff, sweeps_hom, accepted_nu;
    int max_iter, mem, nu_max, method;
    int buf, bt_pending, backtracks, backtrack;
    int ck_set, div_now, div_store, nodiv;
    int div_hits;                         // consecutive windows that passed the infeasibility test
    int order[kMemMax];
    double lam, eps, eps_curv, tau, cr;
    double res, resu, rr, gg_prev, gamma;
    double L, inv_norm, bt_param, hh;
    double theta, beta;                   // GPAD: theta_k and the next extrapolation weight
    double SY[kMemMax + 1][kMemMax + 1];  // s_a . q_b by slot
    double QQ[kMemMax + 1][kMemMax + 1];  // q_a . q_b by slot
    double coefS[kMemMax], coefQ[kMemMax];
    double ls_val[kNuCap + 1];
};
constexpr int kCtlInts = (int)(sizeof(Ctl) / sizeof(int));

struct VecArgs {
    const InstDesc *inst;
    const int *blk;  // per block: instance, block within the instance, blocks of the instance
    const double *sc, *lo, *hi;
    const double *pw, *hub;  // soft rows (pi * weight, Huber threshold) or null: all hard
    Ctl *ctl;
    int *ndone;
    long long m_tot;
    double *part;
    int nblocks, method;
    const double *y, *yp, *hx, *rp, *gp, *hr, *hd, *d;
    double *r, *g, *S, *Q, *yn;
    double *Rw, *hw;         // backtracking test 1: R(w), s H x(w) of the update (null: not kept)
    double *yck;             // infeasibility test: iterate at the last test, then the change since
};

// The rows a block visits: rows lb*kVB + tid + n*nblk*kVB of its instance.
struct BlockRows {
    int b, lb, nb;
    InstDesc I;
    unsigned nlr;  // rows owned by non-leaf nodes
};

__device__ __forceinline__ BlockRows block_rows(const VecArgs &a)
{
    BlockRows br;
    br.b = a.blk[3 * blockIdx.x];
    br.lb = a.blk[3 * blockIdx.x + 1];
    br.nb = a.blk[3 * blockIdx.x + 2];
    br.I = a.inst[br.b];
    br.nlr = (unsigned)((long long)br.I.Vnl * br.I.nc);
    return br;
}

// sqrt(pi) of the node owning local row k (1 without preconditioning); the
// dual layout has nc rows per non-leaf node and ncN per leaf.
__device__ __forceinline__ double row_scale(const VecArgs &a, const BlockRows &br, long long k)
{
    if (!a.sc) return 1.0;
    const unsigned kk = (unsigned)k;
    const unsigned node = kk < br.nlr ? kk / (unsigned)br.I.nc
                                      : (unsigned)br.I.Vnl + (kk - br.nlr) / (unsigned)br.I.ncN;
    return a.sc[br.I.sc + node];
}

// Bounds and penalty of local row kl in the scaled variables of Sec. III-E:
// the row function pi w psi_d(dist(z / s, [lo, hi])) equals
// w' psi_d'(dist(zb, [s lo, s hi])) with w' = pi w / s and d' = s d.
struct RowG {
    double lo, hi, w, d;   // w = +inf: hard row
};
__device__ __forceinline__ RowG row_g(const VecArgs &a, const BlockRows &br, long long kl, double s)
{
    RowG g;
    g.lo = s * a.lo[br.I.box + kl];
    g.hi = s * a.hi[br.I.box + kl];
    g.w = INFINITY;
    g.d = 0.0;
    if (a.pw) {
        const double pw = a.pw[br.I.box + kl];
        if (pw < INFINITY) {
            g.w = pw / s;
            g.d = s * a.hub[br.I.box + kl];
        }
    }
    return g;
}

// Row prox of Sec. II-D, z = argmin g(z) + (lambda/2)(z - v)^2: the
// projection on [lo, hi] for a hard row; for a soft row the distance t to
// the interval shrinks to t / (1 + w / (lambda d)) on the quadratic part of
// the Huber function (shrunk distance <= d) and to max(t - w/lambda, 0)
// beyond it.  gz receives g(z) (0 for a hard row).
__device__ __forceinline__ double row_prox(double v, const RowG &g, double lam, double &gz)
{
    gz = 0.0;
    if (!(g.w < INFINITY)) return v < g.lo ? g.lo : (v > g.hi ? g.hi : v);
    const bool above = v > g.hi;
    if (!above && !(v < g.lo)) return v;
    const double t = above ? v - g.hi : g.lo - v;
    const double wl = g.w / lam;
    double sh;
    if (g.d > 0.0 && t <= g.d + wl) {
        sh = t / (1.0 + wl / g.d);
        gz = g.w * sh * sh / (2.0 * g.d);
    } else {
        sh = t - wl > 0.0 ? t - wl : 0.0;
        gz = g.w * (sh - 0.5 * g.d);
    }
    return above ? g.hi + sh : g.lo - sh;
}

#define FOR_BLOCK_ROWS(br, kl, k)                                                             \
    for (long long kl = (long long)(br).lb * kVB + threadIdx.x, k = (br).I.y + kl; kl < (br).I.m; \
         kl += (long long)(br).nb * kVB, k = (br).I.y + kl)

__device__ __forceinline__ double clampd(double v, double lo, double hi)
{
    return v < lo ? lo : (v > hi ? hi : v);
}

__device__ __forceinline__ double wave_red(double x, bool is_max)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const double o = __shfl_xor(x, off, 64);
        x = is_max ? fmax(x, o) : x + o;
    }
    return x;
}

// Sums over the wavefront of v[0..N), value idx left in the lanes that return
// idx (ok): at each exchange a lane keeps half of the values and hands the
// other half to its partner, so N values take about N exchanges instead of
// 6 N (the same pairs are added as by one butterfly per value).
template <int N, int OFF, int M>
__device__ __forceinline__ int fold_sums(double (&v)[M], int lane, bool &ok)
{
    constexpr int H = (N + 1) / 2;
    const bool hi = (lane & OFF) != 0;
#pragma unroll
    for (int j = 0; j < H; ++j) {
        const double a = v[j], b = j + H < N ? v[j + H] : 0.0;
        v[j] = (hi ? b : a) + __shfl_xor(hi ? a : b, OFF, 64);
    }
    int idx = 0;
    if constexpr (OFF > 1) idx = fold_sums<H, OFF / 2>(v, lane, ok);
    idx += hi ? H : 0;
    ok = ok && idx < N;
    return idx;
}

// Block-reduce acc and store slot v < NV of this block at part[v*nblocks+b]:
// slots [0, kNMax) are maxima (with MAXES; otherwise nothing reads them), the
// rest sums.
template <int NV, bool MAXES = true>
__device__ void block_store(double (&acc)[NV], double *part, int nblocks)
{
    constexpr int NS = NV - kNMax;
    static_assert(NS <= 128, "two folds");
    __shared__ double red[kVB / 64][NV];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (MAXES)
#pragma unroll
        for (int v = 0; v < kNMax; ++v) {
            const double x = wave_red(acc[v], true);
            if (lane == 0) red[w][v] = x;
        }
    constexpr int N0 = NS < 64 ? NS : 64;
    double s0[N0];
#pragma unroll
    for (int v = 0; v < N0; ++v) s0[v] = acc[kNMax + v];
    bool ok = true;
    const int i0 = fold_sums<N0, 32>(s0, lane, ok);
    if (ok) red[w][kNMax + i0] = s0[0];
    if constexpr (NS > 64) {
        double s1[NS - 64];
#pragma unroll
        for (int v = 64; v < NS; ++v) s1[v - 64] = acc[kNMax + v];
        ok = true;
        const int i1 = fold_sums<NS - 64, 32>(s1, lane, ok);
        if (ok) red[w][kNMax + 64 + i1] = s1[0];
    }
    __syncthreads();
    for (int v = threadIdx.x + (MAXES ? 0 : kNMax); v < NV; v += blockDim.x) {
        double x = red[0][v];
        for (int k = 1; k < kVB / 64; ++k) x = (v < kNMax) ? fmax(x, red[k][v]) : x + red[k][v];
        part[(long long)v * nblocks + blockIdx.x] = x;
    }
}

// Finalize-side reduction of nv slots over blocks [first, first+count) (fixed
// order) into out; a wavefront per slot.
__device__ void reduce_partials(const double *part, int nblocks, int first, int count, int nv, double *out)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    for (int v = w; v < nv; v += nw) {
        const bool mx = v < kNMax;
        const double *p = part + (long long)v * nblocks + first;
        double x = 0.0;
        // four loads in flight (blocks past the end re-read the first one and are not added)
        for (int b = lane; b < count; b += 256) {
            double q[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) q[u] = p[b + 64 * u < count ? b + 64 * u : b];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (b + 64 * u < count) x = mx ? fmax(x, q[u]) : x + q[u];
        }
        x = wave_red(x, mx);
        if (lane == 0) out[v] = x;
    }
    __syncthreads();
}

// The finalize kernels take their decisions on a copy of the control block in
// LDS (one thread's chain of dependent accesses: from memory and with its small
// arrays in scratch it took 15 us on the smallest problems) and write it back
// whole.
__device__ __forceinline__ void ctl_copy(Ctl *dst, const Ctl *src)
{
    static_assert(sizeof(Ctl) % 8 == 0, "copied in doubles");
    double *d = reinterpret_cast<double *>(dst);
    const double *s = reinterpret_cast<const double *>(src);
    for (int k = threadIdx.x; k < (int)(sizeof(Ctl) / 8); k += blockDim.x) d[k] = s[k];
    __syncthreads();
}

template <int MEMCAP>
__device__ __forceinline__ void pair_dots(const VecArgs &a, long long k, double s, double q, double g,
                                          bool have_pair, int cnt, int fslot, const int *order,
                                          double (&acc)[nv_pair(MEMCAP)])
{
    if (have_pair) {
        a.S[(long long)fslot * a.m_tot + k] = s;
        a.Q[(long long)fslot * a.m_tot + k] = q;
        acc[PB + 0] += s * q;
        acc[PB + 1] += s * s;
        acc[PB + 2] += q * q;
        acc[PB + 3] += s * g;
        acc[PB + 4] += q * g;
    }
    acc[PB + 5] += g * g;
#pragma unroll
    for (int j = 0; j < MEMCAP; ++j) {
        if (j < cnt) {
            const double sj = a.S[(long long)order[j] * a.m_tot + k];
            const double qj = a.Q[(long long)order[j] * a.m_tot + k];
            if (have_pair) {
                acc[PB + 6 + 5 * j + 0] += s * qj;
                acc[PB + 6 + 5 * j + 1] += sj * q;
                acc[PB + 6 + 5 * j + 2] += q * qj;
            }
            acc[PB + 6 + 5 * j + 3] += sj * g;
            acc[PB + 6 + 5 * j + 4] += qj * g;
        }
    }
}

__device__ __forceinline__ bool idle(const Ctl *c) { return c->done || c->skip; }

// Residual pass.  PAIR (NAMA): g = R and the L-BFGS pair/dots.
template <bool PAIR, int MEMCAP>
__global__ void __launch_bounds__(kVB) resid_kernel(VecArgs a)
{
    const BlockRows br = block_rows(a);
    const Ctl *c = a.ctl + br.b;
    if (idle(c)) return;
    constexpr int NV = PAIR ? nv_pair(MEMCAP) : PB;
    double acc[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) acc[v] = 0.0;
    const double lam = c->lam;
    const bool have_pair = PAIR && c->have_pair;
    const int cnt = c->cnt, fslot = c->free_slot;
    int order[MEMCAP > 0 ? MEMCAP : 1];
#pragma unroll
    for (int j = 0; j < MEMCAP; ++j) order[j] = c->order[j];
    FOR_BLOCK_ROWS(br, kl, k) {
        const double s = row_scale(a, br, kl);
        const double h = s * a.hx[k];
        const double yk = a.y[k];
        double gz;
        const double z = row_prox(yk / lam + h, row_g(a, br, kl, s), lam, gz);
        const double R = z - h;
        a.r[k] = R;
        const double aR = fabs(R);
        acc[R_MAX] = fmax(acc[R_MAX], aR);
        acc[R_MAXU] = fmax(acc[R_MAXU], aR / s);
        acc[R_SS] += R * R;
        acc[R_BAD] += isfinite(R) ? 0.0 : 1.0;
        if constexpr (PAIR) {
            const double sv = have_pair ? yk - a.yp[k] : 0.0;
            const double qv = have_pair ? R - a.rp[k] : 0.0;
            pair_dots<MEMCAP>(a, k, sv, qv, R, have_pair, cnt, fslot, order, acc);
        }
    }
    block_store(acc, a.part, a.nblocks);
}

// MINFBE gradient of the FBE and the L-BFGS pair/dots; slot R_SS collects
// ||s H xhat(s R)||^2 for backtracking test 2.
template <int MEMCAP>
__global__ void __launch_bounds__(kVB) grad_kernel(VecArgs a)
{
    const BlockRows br = block_rows(a);
    const Ctl *c = a.ctl + br.b;
    if (idle(c)) return;
    double acc[nv_pair(MEMCAP)];
#pragma unroll
    for (int v = 0; v < nv_pair(MEMCAP); ++v) acc[v] = 0.0;
    const double lam = c->lam;
    const bool have_pair = c->have_pair;
    const int cnt = c->cnt, fslot = c->free_slot;
    int order[MEMCAP > 0 ? MEMCAP : 1];
#pragma unroll
    for (int j = 0; j < MEMCAP; ++j) order[j] = c->order[j];
    FOR_BLOCK_ROWS(br, kl, k) {
        const double s = row_scale(a, br, kl);
        const double shr = s * a.hr[k];
        const double g = a.r[k] + lam * shr;
        a.g[k] = g;
        acc[R_SS] += shr * shr;
        const double sv = have_pair ? a.y[k] - a.yp[k] : 0.0;
        const double qv = have_pair ? g - a.gp[k] : 0.0;
        pair_dots<MEMCAP>(a, k, sv, qv, g, have_pair, cnt, fslot, order, acc);
    }
    block_store(acc, a.part, a.nblocks);
}

template <int MEMCAP>
__global__ void __launch_bounds__(kVB) combine_kernel(VecArgs a)
{
    const BlockRows br = block_rows(a);
    const Ctl *c = a.ctl + br.b;
    if (idle(c)) return;
    const int cnt = c->cnt;
    const double gam = c->gamma;
    int order[MEMCAP > 0 ? MEMCAP : 1];
    double cs[MEMCAP > 0 ? MEMCAP : 1], cq[MEMCAP > 0 ? MEMCAP : 1];
#pragma unroll
    for (int j = 0; j < MEMCAP; ++j) { order[j] = c->order[j]; cs[j] = c->coefS[j]; cq[j] = c->coefQ[j]; }
    FOR_BLOCK_ROWS(br, kl, k) {
        double v = gam * a.g[k];
#pragma unroll
        for (int j = 0; j < MEMCAP; ++j)
            if (j < cnt)
                v += cs[j] * a.S[(long long)order[j] * a.m_tot + k] + cq[j] * a.Q[(long long)order[j] * a.m_tot + k];
        a.r[k] = -v;  // a.r points at the direction buffer here
    }
}

// The row prox of a line search, where one row is tried at many points: the
// quotients that do not depend on the point, formed once.  Where w / (2 d)
// overflows (a Huber threshold near the smallest doubles), h is the largest
// double: the shrunk distance there is zero or some 1e-308 of the distance, and
// infinity times it would be NaN.
struct RowTrial {
    double lo, hi, w, d, wl, q, h;   // wl = w / lambda, q = 1 + wl / d, h = w / (2 d)
};
__device__ __forceinline__ RowTrial row_trial(const RowG &g, double lam)
{
    RowTrial t{g.lo, g.hi, g.w, g.d, 0.0, 1.0, 0.0};
    if (g.w < INFINITY) {
        t.wl = g.w / lam;
        if (g.d > 0.0) {
            t.q = 1.0 + t.wl / g.d;
            t.h = fmin(g.w / (2.0 * g.d), DBL_MAX);
        }
    }
    return t;
}
__device__ __forceinline__ double row_prox(double v, const RowTrial &g, double &gz)
{
    gz = 0.0;
    const double in = v < g.lo ? g.lo : (v > g.hi ? g.hi : v);
    if (!(g.w < INFINITY) || in == v || v != v) return in;
    const bool above = v > g.hi;
    const double t = above ? v - g.hi : g.lo - v;
    double sh;
    if (g.d > 0.0 && t <= g.d + g.wl) {
        sh = t / g.q;
        gz = g.h * sh * sh;
    } else {
        sh = t - g.wl > 0.0 ? t - g.wl : 0.0;
        gz = g.w * (sh - 0.5 * g.d);
    }
    return above ? g.hi + sh : g.lo - sh;
}

// All trial steps in one pass; slot nu holds sum over rows of the change of
// the FBE at w(tau_nu) relative to y, with phi = f-hat + <y, z> -
// (lambda/2) ||R||^2 - g(z).  NUC: the largest nu_max the variant serves
// (its accumulators, and so its register demand, scale with it).  For NAMA
// the slot after the last trial collects ||s H xhat(s r)||^2 (backtracking
// test 2).
// Everything a trial needs is linear in tau: w = y + d0 + tau d1,
// s H x(w) = h0 + tau h1 and w / lambda + s H x(w) = v0 + tau v1, so a row
// divides twice (y / lambda, d / lambda) and not once per trial: FP64
// arithmetic bounds this pass, the divisions were half of it.
template <int NUC>
__global__ void __launch_bounds__(kVB) ls_kernel(VecArgs a)
{
    const BlockRows br = block_rows(a);
    const Ctl *c = a.ctl + br.b;
    if (idle(c)) return;
    const double lam = c->lam;
    const int numax = c->nu_max;
    const bool nama = a.method == 1;
    double acc[NUC + 1];
    double hh = 0.0;
#pragma unroll
    for (int v = 0; v < NUC + 1; ++v) acc[v] = 0.0;
    FOR_BLOCK_ROWS(br, kl, k) {
        const double s = row_scale(a, br, kl);
        const RowTrial rg = row_trial(row_g(a, br, kl, s), lam);
        const double yk = a.y[k], rk = a.rp[k], dk = a.d[k];
        const double ah = s * a.hx[k];
        const double brk = nama ? s * a.hr[k] : 0.0;
        hh += brk * brk;
        const double bd = s * a.hd[k];
        const double yl = yk / lam, lr = nama ? lam * rk : 0.0, lb = lam * brk;
        double gy;
        (void)row_prox(yl + ah, rg, gy);   // g at z(y) = R + s H x
        const double ey = yk * (rk + ah) - 0.5 * lam * rk * rk - gy;
        const double d0 = -lr, d1 = dk + lr, g1 = bd + lb;       // w - y, s H xhat(w - y) = -lb + tau g1
        const double h0 = ah - lb;
        const double v0 = (yl - (nama ? rk : 0.0)) + h0, v1 = (dk / lam + (nama ? rk : 0.0)) + g1;
        double tau = 1.0;
#pragma unroll
        for (int nu = 0; nu <= NUC; ++nu) {
            if (nu <= numax) {
                const double dl = fma(tau, d1, d0);
                const double hd = fma(tau, g1, -lb);
                const double hw = fma(tau, g1, h0);
                double gw;
                const double zw = row_prox(fma(tau, v1, v0), rg, gw);
                const double Rw = zw - hw;
                acc[nu] += (yk + dl) * zw - dl * fma(0.5, hd, ah) - 0.5 * lam * Rw * Rw - gw - ey;
            }
            tau *= 0.5;
        }
    }
    // the sums follow the (unused) max slots, then hh
    double packed[kNMax + NUC + 2];
#pragma unroll
    for (int v = 0; v < NUC + 2; ++v)
        packed[kNMax + v] = v <= numax ? (v < NUC + 1 ? acc[v] : 0.0) : (v == numax + 1 ? hh : 0.0);
    block_store<kNMax + NUC + 2, false>(packed, a.part, a.nblocks);
}

// y+ = T(w) at the accepted step (tau = c->tau); with a.Rw kept, R(w) and
// s H x(w) for backtracking test 1.  A redone update (redo = 1: lambda
// halved by test 2) copies y; a skipped one (redo = 2: test 1 undid the
// previous update) leaves y+ as it is, since it already holds the iterate
// the next update starts from.
__global__ void __launch_bounds__(kVB) update_kernel(VecArgs a)
{
    const BlockRows br = block_rows(a);
    const Ctl *c = a.ctl + br.b;
    if (idle(c) || c->redo == 2) return;
    if (c->redo == 1) {
        FOR_BLOCK_ROWS(br, kl, k) a.yn[k] = a.y[k];
        return;
    }
    const double lam = c->lam, tau = c->tau, cr = c->cr;
    const bool nama = a.method == 1;
    FOR_BLOCK_ROWS(br, kl, k) {
        const double s = row_scale(a, br, kl);
        const double dl = cr * a.rp[k] + tau * a.d[k];
        const double hd = (nama ? cr * s * a.hr[k] : 0.0) + tau * s * a.hd[k];
        const double w = a.y[k] + dl, hw = s * a.hx[k] + hd;
        double gw;
        const double zw = row_prox(w / lam + hw, row_g(a, br, kl, s), lam, gw);
        a.yn[k] = w - lam * (zw - hw);
        if (a.Rw) {
            a.Rw[k] = zw - hw;
            a.hw[k] = hw;
        }
    }
}

// Backtracking test 1 at the start of the update after y+ = T(w): with
// H x(y+) from this update's affine sweep, sums <R(w), s H x(y+) - s H x(w)>
// and ||R(w)||^2 (f-hat is quadratic, so f-hat(y+) - f-hat(w) minus the
// linear term of the test is -(1/2) <y+ - w, s H xhat(y+ - w)>, and
// s H xhat(y+ - w) = s H x(y+) - s H x(w) with y+ - w = -lambda R(w)).
__global__ void __launch_bounds__(kVB) bt_kernel(VecArgs a)
{
    const BlockRows br = block_rows(a);
    const Ctl *c = a.ctl + br.b;
    if (c->done || !c->bt_pending) return;
    double acc[kNMax + 2] = {};
    FOR_BLOCK_ROWS(br, kl, k) {
        const double s = row_scale(a, br, kl);
        const double Rw = a.Rw[k];
        acc[kNMax + 0] += Rw * (s * a.hx[k] - a.hw[k]);
        acc[kNMax + 1] += Rw * Rw;
    }
    block_store<kNMax + 2, false>(acc, a.part, a.nblocks);
}

// Infeasibility test, first pass: yck becomes y - yck (the change since the
// last test), or y itself at the first test.
__global__ void __launch_bounds__(kVB) div_prep_kernel(VecArgs a)
{
    const BlockRows br = block_rows(a);
    const Ctl *c = a.ctl + br.b;
    if (idle(c) || !c->div_store) return;
    if (c->div_now) {
        FOR_BLOCK_ROWS(br, kl, k) a.yck[k] = a.y[k] - a.yck[k];
    } else {
        FOR_BLOCK_ROWS(br, kl, k) a.yck[k] = a.y[k];
    }
}

// Second pass, after the homogeneous sweep of the change d (in a.hd): max |d|,
// max |s H xhat(s d)|, max |d| on rows whose g* is +inf along d (an infinite
// bound on the side d points to, or a soft row), and sigma(d) - <d, s H x(y)>;
// then yck = y.
__global__ void __launch_bounds__(kVB) div_kernel(VecArgs a)
{
    const BlockRows br = block_rows(a);
    const Ctl *c = a.ctl + br.b;
    if (idle(c) || !c->div_now) return;
    double acc[kNMax + 1] = {};
    FOR_BLOCK_ROWS(br, kl, k) {
        const double s = row_scale(a, br, kl);
        const double d = a.yck[k];
        const double ad = fabs(d);
        acc[0] = fmax(acc[0], ad);
        acc[1] = fmax(acc[1], fabs(s * a.hd[k]));
        if (d != 0.0) {
            const RowG rg = row_g(a, br, kl, s);
            const double bound = d > 0.0 ? rg.hi : rg.lo;
            if (rg.w < INFINITY || !isfinite(bound)) acc[2] = fmax(acc[2], ad);
            else acc[kNMax] += bound * d;
            acc[kNMax] -= d * s * a.hx[k];
        }
        a.yck[k] = a.y[k];
    }
    block_store(acc, a.part, a.nblocks);
}

// GPAD update: y^{k+1} = T(w^k) = w^k - lambda R(w^k) into y (the main
// sequence, a.yn), w^{k+1} = y^{k+1} + beta (y^{k+1} - y^k) into w (a.r is
// R, a.g the evaluation point w, updated in place).
__global__ void __launch_bounds__(kVB) gpad_update_kernel(VecArgs a)
{
    const BlockRows br = block_rows(a);
    const Ctl *c = a.ctl + br.b;
    if (c->done) return;
    const double lam = c->lam, beta = c->beta;
    FOR_BLOCK_ROWS(br, kl, k) {
        const double yold = a.yn[k];
        const double ynew = a.g[k] - lam * a.r[k];
        a.yn[k] = ynew;
        a.g[k] = ynew + beta * (ynew - yold);
    }
}

__global__ void __launch_bounds__(kVB) copy_kernel(VecArgs a)
{
    const BlockRows br = block_rows(a);
    FOR_BLOCK_ROWS(br, kl, k) a.yn[k] = a.y[k];
}

// ---------------------------- finalize kernels ---------------------------
// One block of kFin threads per instance; thread 0 takes the scalar decisions.
// div_due: this update runs the infeasibility test (which then takes the
// max_iter decision after it, as the test comes first).
__device__ void finish_residual(Ctl *c, const double *red, int *ndone, int div_due)
{
    c->sweeps_aff++;
    c->res = red[R_MAX];
    c->resu = red[R_MAXU];
    c->rr = red[R_SS];
    if (red[R_BAD] > 0.0 || !isfinite(red[R_SS])) { c->done = 1; c->status = STOTREE_ERR_NUMERIC; }
    else if (red[R_MAX] <= c->eps) { c->done = 1; c->status = STOTREE_OK; }
    else if (c->iter >= c->max_iter && !(div_due && c->ck_set)) { c->done = 1; c->status = STOTREE_NOT_CONVERGED; }
    if (c->done) atomicAdd(ndone, 1);
    c->div_store = div_due && !c->done;
    c->div_now = c->div_store && c->ck_set;
    c->nodiv = !c->div_now;
}
// Cautious push of the candidate pair (Li and Fukushima: push when
// <s,q> > eps' ||s||^2 ||g_prev||^2) and the compact-form coefficients of
// d = -B g = -(gamma g + S p1 + gamma Q p2).
__device__ void lbfgs_update(Ctl *c, const double *red)
{
    int cnt = c->cnt, fs = c->free_slot;
    const int mem = c->mem;
    __shared__ double sg[kMemMax + 1], qg[kMemMax + 1];
    for (int j = 0; j < cnt; ++j) {
        sg[c->order[j]] = red[PB + 6 + 5 * j + 3];
        qg[c->order[j]] = red[PB + 6 + 5 * j + 4];
    }
    if (c->have_pair) {
        const double sq = red[PB + 0], ss = red[PB + 1], qq = red[PB + 2];
        if (sq > c->eps_curv * ss * c->gg_prev && isfinite(sq) && qq > 0.0) {
            c->SY[fs][fs] = sq;
            c->QQ[fs][fs] = qq;
            for (int j = 0; j < cnt; ++j) {
                const int oj = c->order[j];
                c->SY[fs][oj] = red[PB + 6 + 5 * j + 0];
                c->SY[oj][fs] = red[PB + 6 + 5 * j + 1];
                c->QQ[fs][oj] = c->QQ[oj][fs] = red[PB + 6 + 5 * j + 2];
            }
            sg[fs] = red[PB + 3];
            qg[fs] = red[PB + 4];
            int evicted = -1;
            if (cnt == mem) {
                evicted = c->order[0];
                for (int j = 1; j < cnt; ++j) c->order[j - 1] = c->order[j];
                --cnt;
            }
            c->order[cnt++] = fs;
            if (evicted >= 0) {
                fs = evicted;
            } else {
                for (int sl = 0; sl <= mem; ++sl) {
                    bool used = false;
                    for (int j = 0; j < cnt; ++j) used |= (c->order[j] == sl);
                    if (!used) { fs = sl; break; }
                }
            }
            c->pushes++;
        } else {
            c->skips++;
        }
    }
    c->cnt = cnt;
    c->free_slot = fs;
    c->have_pair = 1;
    c->gg_prev = red[PB + 5];
    if (cnt == 0) {
        c->gamma = 1.0;
        return;
    }
    const int n = c->order[cnt - 1];
    const double gam = c->SY[n][n] / c->QQ[n][n];
    __shared__ double u1[kMemMax], u2[kMemMax], p1[kMemMax], p2[kMemMax], t[kMemMax];
    for (int i = 0; i < cnt; ++i) {
        u1[i] = sg[c->order[i]];
        u2[i] = gam * qg[c->order[i]];
    }
    auto Rm = [&](int i, int j) { return c->SY[c->order[i]][c->order[j]]; };
    for (int i = cnt - 1; i >= 0; --i) {          // p2 = -R^{-1} u1
        double v = -u1[i];
        for (int j = i + 1; j < cnt; ++j) v -= Rm(i, j) * p2[j];
        p2[i] = v / Rm(i, i);
    }
    for (int i = 0; i < cnt; ++i) {               // t = (D + gamma Q'Q)(-p2) - u2
        double v = -Rm(i, i) * p2[i];
        for (int j = 0; j < cnt; ++j) v -= gam * c->QQ[c->order[i]][c->order[j]] * p2[j];
        t[i] = v - u2[i];
    }
    for (int i = 0; i < cnt; ++i) {               // p1 = R^{-T} t
        double v = t[i];
        for (int j = 0; j < i; ++j) v -= Rm(j, i) * p1[j];
        p1[i] = v / Rm(i, i);
    }
    for (int i = 0; i < cnt; ++i) {
        c->coefS[i] = p1[i];
        c->coefQ[i] = gam * p2[i];
    }
    c->gamma = gam;
}

// Empties the L-BFGS memory (lambda changed); the next pass forms no pair.
__device__ void lbfgs_clear(Ctl *c)
{
    c->cnt = 0;
    c->free_slot = 0;
    c->have_pair = 0;
    c->gamma = 1.0;
}

// Halving of lambda by a backtracking test; false (and the instance stops
// with ERR_NUMERIC) after kBtMax halvings.
__device__ bool halve_lambda(Ctl *c, int *ndone)
{
    if (++c->backtracks > kBtMax) {
        c->done = 1;
        c->status = STOTREE_ERR_NUMERIC;
        atomicAdd(ndone, 1);
        return false;
    }
    c->lam *= 0.5;
    lbfgs_clear(c);
    return true;
}

__global__ void __launch_bounds__(kFin) fin_resid_kernel(Ctl *ctl, const double *part, int nblocks,
                                                        int with_pair, int *ndone, int div_due)
{
    __shared__ Ctl cs;
    ctl_copy(&cs, ctl + blockIdx.x);
    if (idle(&cs)) return;
    __shared__ double red[kNVMax];
    reduce_partials(part, nblocks, cs.first_blk, cs.nblk, with_pair ? PB + 6 + 5 * cs.cnt : PB, red);
    if (threadIdx.x == 0) {
        finish_residual(&cs, red, ndone, div_due);
        if (!cs.done && with_pair) lbfgs_update(&cs, red);
    }
    __syncthreads();
    ctl_copy(ctl + blockIdx.x, &cs);
}

__global__ void __launch_bounds__(kFin) fin_grad_kernel(Ctl *ctl, const double *part, int nblocks)
{
    __shared__ Ctl cs;
    ctl_copy(&cs, ctl + blockIdx.x);
    if (idle(&cs)) return;
    __shared__ double red[kNVMax];
    reduce_partials(part, nblocks, cs.first_blk, cs.nblk, PB + 6 + 5 * cs.cnt, red);
    if (threadIdx.x == 0) {
        cs.sweeps_hom++;
        cs.hh = red[R_SS];
        lbfgs_update(&cs, red);
    }
    __syncthreads();
    ctl_copy(ctl + blockIdx.x, &cs);
}

// Line-search decision (the largest tau = 2^-nu with phi(w) <= phi(y), else
// tau = 0), the trace row, backtracking test 2, and the end of the update:
// the iteration counter, the buffer that holds the next iterate, and the
// flag that arms test 1 for the next update.  A skipped update (test 1
// undid the previous one) only moves to the other buffer.
__device__ void finish_line_search(Ctl *c, const double *red, int b, int *ndone, double *trace, int trace_iters)
{
    int acc = -1;
    for (int nu = 0; nu <= c->nu_max; ++nu) {
        const double dphi = red[kNMax + nu];
        c->ls_val[nu] = dphi;
        if (acc < 0 && isfinite(dphi) && dphi <= 0.0) acc = nu;
    }
    if (trace && c->iter < trace_iters) {
        double *row = trace + ((long long)b * trace_iters + c->iter) * kTraceCols;
        for (int k = 0; k < kTraceCols; ++k) row[k] = NAN;
        row[0] = c->lam;
        row[1] = c->res;
        row[2] = acc;
        row[3] = c->nu_max;
        row[4] = c->cnt;
        for (int nu = 0; nu <= c->nu_max && kTracePhi + nu < kTraceCols; ++nu) row[kTracePhi + nu] = c->ls_val[nu];
    }
    c->sweeps_hom += c->method == 1 ? 2 : 1;
    c->buf ^= 1;
    c->redo = 0;
    if (c->backtrack == 2) {
        // test 2: lambda ||s H xhat(s R)|| > eps'' ||R|| (the gradients of
        // f-hat at T(y) and y differ by lambda s H xhat(s R), T(y) - y = -lambda R)
        const double hh = c->method == 1 ? red[kNMax + c->nu_max + 1] : c->hh;
        if (c->lam * sqrt(hh) > c->bt_param * sqrt(c->rr)) {
            if (halve_lambda(c, ndone)) c->redo = 1;
            c->bt_pending = 0;
            return;
        }
    }
    c->accepted_nu = acc;
    c->tau = acc >= 0 ? ldexp(1.0, -acc) : 0.0;
    c->cr = c->method == 1 ? -(1.0 - c->tau) * c->lam : 0.0;
    c->ls_trials += acc >= 0 ? acc + 1 : c->nu_max + 1;
    c->bt_pending = c->backtrack == 1;
    c->iter++;
}

__global__ void __launch_bounds__(kFin) fin_ls_kernel(Ctl *ctl, const double *part, int nblocks, int *ndone,
                                                     double *trace, int trace_iters)
{
    __shared__ Ctl cs;
    ctl_copy(&cs, ctl + blockIdx.x);
    if (cs.done) return;
    if (cs.skip) {
        // redo = 2: the update kernel leaves y+ as it is
        if (threadIdx.x == 0) {
            Ctl *c = ctl + blockIdx.x;
            c->skip = 0;
            c->buf = cs.buf ^ 1;
            c->redo = 2;
        }
        return;
    }
    __shared__ double red[kNVMax];
    // the max slots hold nothing here
    reduce_partials(part, nblocks, cs.first_blk, cs.nblk, kNMax + cs.nu_max + 2, red);
    if (threadIdx.x == 0) finish_line_search(&cs, red, blockIdx.x, ndone, trace, trace_iters);
    __syncthreads();
    ctl_copy(ctl + blockIdx.x, &cs);
}

// Test 1: halve lambda when <R(w), s H x(y+) - s H x(w)> > (1 - beta) ||R(w)||^2;
// the update that produced y+ is then undone (this update is skipped and
// the next one starts again from y^k, which the buffer of y+ of this update
// still holds).
__global__ void __launch_bounds__(kVB) fin_bt_kernel(Ctl *ctl, const double *part, int nblocks, int *ndone)
{
    Ctl *c = ctl + blockIdx.x;
    if (c->done || !c->bt_pending) return;
    __shared__ double red[kNVMax];
    reduce_partials(part, nblocks, c->first_blk, c->nblk, kNMax + 2, red);
    if (threadIdx.x != 0) return;
    c->bt_pending = 0;
    if (red[kNMax + 0] > (1.0 - c->bt_param) * red[kNMax + 1]) {
        c->sweeps_aff++;
        if (halve_lambda(c, ndone)) {
            c->skip = 1;
            c->iter--;
        }
    }
}

// Infeasibility decision (see div_kernel), then the max_iter test it deferred.
__global__ void __launch_bounds__(kVB) fin_div_kernel(Ctl *ctl, const double *part, int nblocks, int *ndone)
{
    Ctl *c = ctl + blockIdx.x;
    if (idle(c) || !c->div_store) return;
    __shared__ double red[kNVMax];
    if (c->div_now) reduce_partials(part, nblocks, c->first_blk, c->nblk, kNMax + 1, red);
    if (threadIdx.x != 0) return;
    c->div_store = 0;
    if (!c->div_now) {
        c->ck_set = 1;
        return;
    }
    c->div_now = 0;
    c->nodiv = 1;
    c->sweeps_hom++;
    const double dn = red[0], hn = red[1], dbad = red[2], lin = red[kNMax];
    // GPAD's momentum carries a feasible but slowly converging problem along
    // a nearly null direction for many windows (ratios of 2e-4 to 6e-4):
    // its null-space part is held to a tighter tolerance.  The objective
    // bound is looser: along a true null direction (first ratio 1e-9 and
    // below) the objective ratio of infeasible problems settles at 5e-4 to
    // 9e-4 in these norms; the null-space ratio is what separates feasible
    // paths, whose objective ratios can exceed 1e-3
    const double eps_null = c->method == 2 ? kEpsNullGpad : kEpsDiv;
    const bool pass = dn > 0.0 && dbad <= 1e-9 * dn && c->lam * hn <= eps_null * dn && lin <= -kEpsObj * dn * c->res;
    c->div_hits = pass ? c->div_hits + 1 : 0;
    if (c->div_hits >= kDivHits) {
        c->done = 1;
        c->status = STOTREE_ERR_DIVERGED;
    } else if (c->iter >= c->max_iter) {
        c->done = 1;
        c->status = STOTREE_NOT_CONVERGED;
    }
    if (c->done) atomicAdd(ndone, 1);
}

// GPAD end of update: theta_{k+1} = (sqrt(theta^4 + 4 theta^2) - theta^2)/2
// and the extrapolation weight theta_{k+1} (1/theta_k - 1) of w^{k+1}.
__global__ void __launch_bounds__(kVB) fin_gpad_kernel(Ctl *ctl)
{
    Ctl *c = ctl + blockIdx.x;
    if (c->done || threadIdx.x != 0) return;
    const double th = c->theta;
    const double tn = 0.5 * (sqrt(th * th * th * th + 4.0 * th * th) - th * th);
    c->beta = tn * (1.0 / th - 1.0);
    c->theta = tn;
    c->iter++;
}

// Final dual of every instance into the caller's buffer (buffer 0): the
// instances whose last iterate sits in buffer 1 are copied.
__global__ void __launch_bounds__(kVB) gather_final_kernel(VecArgs a)
{
    const BlockRows br = block_rows(a);
    if (!a.ctl[br.b].buf) return;
    FOR_BLOCK_ROWS(br, kl, k) a.yn[k] = a.y[k];
}

// ----------------------------- power iteration ---------------------------
__global__ void __launch_bounds__(kVB) power_init_kernel(VecArgs a)
{
    const BlockRows br = block_rows(a);
    const double v = 1.0 / sqrt((double)br.I.m);
    FOR_BLOCK_ROWS(br, kl, k) a.yn[k] = v;
}

__global__ void __launch_bounds__(kVB) power_step_kernel(VecArgs a)
{
    // w = -s H xhat(s v) (the dual Hessian applied to v), slots: <v,w>, ||w||^2
    const BlockRows br = block_rows(a);
    double acc[kNMax + 2] = {0.0, 0.0, 0.0, 0.0};
    FOR_BLOCK_ROWS(br, kl, k) {
        const double s = row_scale(a, br, kl);
        const double w = -s * a.hx[k];
        acc[kNMax + 0] += a.y[k] * w;
        acc[kNMax + 1] += w * w;
        a.r[k] = w;
    }
    block_store<kNMax + 2, false>(acc, a.part, a.nblocks);
}

__global__ void __launch_bounds__(kVB) power_fin_kernel(Ctl *ctl, const double *part, int nblocks)
{
    Ctl *c = ctl + blockIdx.x;
    __shared__ double red[kNVMax];
    reduce_partials(part, nblocks, c->first_blk, c->nblk, kNMax + 2, red);
    if (threadIdx.x != 0) return;
    c->L = red[kNMax + 0];
    const double nw = sqrt(red[kNMax + 1]);
    c->inv_norm = nw > 0.0 ? 1.0 / nw : 0.0;
}

__global__ void __launch_bounds__(kVB) power_scale_kernel(VecArgs a)
{
    const BlockRows br = block_rows(a);
    const double inv = a.ctl[br.b].inv_norm;
    FOR_BLOCK_ROWS(br, kl, k) a.yn[k] = a.r[k] * inv;
}

// ------------------------------- host side -------------------------------
struct WsNeed {
    int mem;
    bool g, div, bt;
};

// need.g: the two FBE-gradient vectors (MINFBE only); need.div: the iterate
// of the infeasibility test; need.bt: R(w), H x(w) for backtracking test 1.
int ensure_solver_ws(tree_factors *f, WsNeed need)
{
    SolverWS &w = f->sws;
    if (w.buf && w.mem >= need.mem && (w.has_g || !need.g) && (w.has_div || !need.div) && (w.has_bt || !need.bt))
        return STOTREE_OK;
    if (w.buf) {
        // keep what the old workspace offered
        need.mem = std::max(need.mem, w.mem);
        need.g |= w.has_g;
        need.div |= w.has_div;
        need.bt |= w.has_bt;
        (void)hipFree(w.buf);
        w.buf = nullptr;
        w.bytes = 0;
    }
    // blocks per instance: one per 1024 rows, at most 1024; one per 256 rows (a
    // row per thread) on handles of few rows.  20 iterations of NAMA by the second
    // / by the first: 30,700 rows 6.86 / 7.15 ms, 107,500 7.36 / 7.53, 174,460 6.82 /
    // 6.87, 245,740 7.62 / 7.37, 488,080 12.10 / 11.91.
    const int per = f->m_tot <= 768LL * kVB ? kVB : 4 * kVB;
    std::vector<int> blk;
    w.blk_first.assign(f->ninst, 0);
    for (int b = 0; b < f->ninst; ++b) {
        const long long m = f->inst[b].m;
        const int nb = (int)std::max<long long>(1, std::min<long long>(1024, (m + per - 1) / per));
        w.blk_first[b] = (int)(blk.size() / 3);
        for (int l = 0; l < nb; ++l) { blk.push_back(b); blk.push_back(l); blk.push_back(nb); }
    }
    const int nblocks = (int)(blk.size() / 3);
    const long long m = f->m_tot;
    const long long nvec = (need.g ? 9 : 7) + 2LL * (need.mem + 1) + (need.div ? 1 : 0) + (need.bt ? 2 : 0);
    const long long nxu = f->cmap ? 4 * f->mxu_tot : 0;
    const size_t vec_bytes = sizeof(double) * ((size_t)nvec * m + (size_t)nxu + (size_t)kNVMax * nblocks);
    const size_t ctl_bytes = sizeof(Ctl) * (size_t)f->ninst;
    const size_t bytes = vec_bytes + ctl_bytes + sizeof(int) * (blk.size() + 1) + 512;
    STOTREE_HIP(hipMalloc(&w.buf, bytes));
    w.bytes = bytes;
    w.mem = need.mem;
    w.nblocks = nblocks;
    double *p = w.buf;
    w.y[1] = p; p += m;
    w.r[0] = p; p += m;
    w.r[1] = p; p += m;
    w.has_g = need.g;
    w.g[0] = w.g[1] = nullptr;
    if (need.g) {
        w.g[0] = p; p += m;
        w.g[1] = p; p += m;
    }
    w.hx = p; p += m;
    w.hr2 = p; p += 2 * m;  // hr, hd
    w.d = p; p += m;
    w.S = p; p += (long long)(need.mem + 1) * m;
    w.Qv = p; p += (long long)(need.mem + 1) * m;
    w.has_div = need.div;
    w.yck = nullptr;
    if (need.div) { w.yck = p; p += m; }
    w.has_bt = need.bt;
    w.Rw = w.hw = nullptr;
    if (need.bt) {
        w.Rw = p; p += m;
        w.hw = p; p += m;
    }
    w.xu = nullptr;
    if (nxu) { w.xu = p; p += nxu; }
    w.partials = p; p += (size_t)kNVMax * nblocks;
    w.ctl = p;
    char *q = reinterpret_cast<char *>(p) + ctl_bytes;
    w.blk = reinterpret_cast<int *>(q);
    w.ndone = w.blk + blk.size();
    STOTREE_HIP(hipMemcpy(w.blk, blk.data(), sizeof(int) * blk.size(), hipMemcpyHostToDevice));
    return STOTREE_OK;
}

VecArgs vec_args(const tree_factors *f)
{
    VecArgs a{};
    a.inst = f->d_inst;
    a.blk = f->sws.blk;
    a.sc = f->precondition ? f->sc : nullptr;
    a.lo = f->lo;
    a.hi = f->hi;
    a.pw = f->pw;
    a.hub = f->hub;
    a.ctl = reinterpret_cast<Ctl *>(f->sws.ctl);
    a.ndone = f->sws.ndone;
    a.m_tot = f->m_tot;
    a.part = f->sws.partials;
    a.nblocks = f->sws.nblocks;
    a.yck = f->sws.yck;
    return a;
}

// A sweep of nrhs in {1, 2} right-hand sides whose duals are at (y, y + y_rs)
// in the dual layout, writing H x there at (out, out + o_rs); instances whose
// flag (an int of each control block, flag_of(ctl)) is set are skipped.  With
// a constraint map the duals go through to_xu and the sweep's (x, u) output
// through from_xu.
hipError_t dual_sweep(const tree_factors *f, int affine, const double *x0, const double *y, long long y_rs,
                      double *out, long long o_rs, const int *flags, int nrhs, hipStream_t st, int active = -1)
{
    SweepArgs a = sweep_args(f, affine);
    a.x0 = x0; a.x0_rs = 0;
    a.dual_out = 1;
    a.done = flags;
    a.done_stride = kCtlInts;
    if (!f->cmap) {
        a.y = y; a.y_rs = y_rs;
        a.xo = out; a.xo_rs = o_rs;
        return launch_sweep_any(f, a, nrhs, st, active);
    }
    double *vin = f->sws.xu, *vout = f->sws.xu + 2 * f->mxu_tot;
    hipError_t e = map_to_xu(f, y, y_rs, vin, nrhs, st);
    if (e != hipSuccess) return e;
    a.y = vin; a.y_rs = f->mxu_tot;
    a.xo = vout; a.xo_rs = f->mxu_tot;
    if ((e = launch_sweep_any(f, a, nrhs, st, active)) != hipSuccess) return e;
    return map_from_xu(f, vout, out, o_rs, nrhs, st);
}

const int *done_flags(const Ctl *ctl) { return ctl ? &ctl->done : nullptr; }
const int *div_flags(const Ctl *ctl) { return &ctl->nodiv; }

struct IterArgs {
    const double *x0;
    double *ybuf[2];
    int k, method, active;
    int div_due, backtrack;
    double *trace;
    int trace_iters;
    const struct Poll *poll;  // the host waits for this iteration's count of finished instances (or null)
};

// Where a solve's host loop receives the count of finished instances: pinned
// memory and an event, taken from a pool for the length of a call (a new pair
// costs two allocations, and a controller that linearises its model again makes
// a new handle for every solve).  The pool keeps at most kPollKept pairs for the
// process and may be used by several threads at once; pairs belong to a device.
struct Poll {
    int dev = -1;
    int *count = nullptr;
    hipEvent_t ev = nullptr;
    mutable bool pending = false;        // a copy into count may be on its way
};
constexpr size_t kPollKept = 16;
struct PollPool {
    std::mutex mu;
    std::vector<Poll> kept;
};
PollPool &poll_pool()
{
    static PollPool *p = new PollPool;   // not torn down: the runtime may be gone by then
    return *p;
}
struct PollLease : Poll {
    int take()
    {
        STOTREE_HIP(hipGetDevice(&dev));
        PollPool &p = poll_pool();
        {
            std::lock_guard<std::mutex> lock(p.mu);
            for (size_t k = p.kept.size(); k-- > 0;)
                if (p.kept[k].dev == dev) {
                    static_cast<Poll &>(*this) = p.kept[k];
                    p.kept.erase(p.kept.begin() + (long)k);
                    return STOTREE_OK;
                }
        }
        STOTREE_HIP(hipHostMalloc(reinterpret_cast<void **>(&count), sizeof(int), 0));
        STOTREE_HIP(hipEventCreateWithFlags(&ev, hipEventDisableTiming));
        return STOTREE_OK;
    }
    hipError_t wait()
    {
        const hipError_t e = hipEventSynchronize(ev);
        if (e == hipSuccess) pending = false;
        return e;
    }
    ~PollLease()
    {
        // (a solve that failed may leave a copy on its way)
        if (pending && wait() != hipSuccess) return;
        if (count && ev) {
            PollPool &p = poll_pool();
            std::lock_guard<std::mutex> lock(p.mu);
            if (p.kept.size() < kPollKept) {
                p.kept.push_back(*this);
                return;
            }
        }
        if (count) (void)hipHostFree(count);
        if (ev) (void)hipEventDestroy(ev);
    }
};

// Requests the count for the host, which waits for the event.
hipError_t enqueue_poll(const Poll &p, const SolverWS &w, hipStream_t st)
{
    const hipError_t e = hipMemcpyAsync(p.count, w.ndone, sizeof(int), hipMemcpyDeviceToHost, st);
    if (e != hipSuccess) return e;
    p.pending = true;
    return hipEventRecord(p.ev, st);
}

// Infeasibility test of the iterate y (after fin_resid): the change since
// the last test, its homogeneous sweep into hd, the reductions and the
// decision.  first: no instance has an earlier iterate yet, this one is only
// kept (no change to sweep).
hipError_t enqueue_div_test(const tree_factors *f, const double *y, bool first, hipStream_t st)
{
    const SolverWS &w = f->sws;
    VecArgs a = vec_args(f);
    Ctl *ctl = a.ctl;
    const dim3 grid(a.nblocks), blk(kVB), fgrid(f->ninst);
    double *hd = w.hr2 + f->m_tot;
    a.y = y; a.hx = w.hx; a.hd = hd;
    hipLaunchKernelGGL(div_prep_kernel, grid, blk, 0, st, a);
    if (!first) {
        hipError_t e = dual_sweep(f, 0, nullptr, w.yck, 0, hd, 0, div_flags(ctl), 1, st);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(div_kernel, grid, blk, 0, st, a);
    }
    hipLaunchKernelGGL(fin_div_kernel, fgrid, blk, 0, st, ctl, a.part, a.nblocks, a.ndone);
    return hipGetLastError();
}

template <int MEMCAP, int NUC>
hipError_t enqueue_iteration(const tree_factors *f, const IterArgs &it, hipStream_t st)
{
    const SolverWS &w = f->sws;
    VecArgs a = vec_args(f);
    a.method = it.method;
    Ctl *ctl = a.ctl;
    const int k = it.k, method = it.method, active = it.active;
    const dim3 grid(a.nblocks), blk(kVB), fgrid(f->ninst);
    double *y = it.ybuf[k & 1], *yn = it.ybuf[(k + 1) & 1];
    double *r = w.r[k & 1], *rp = w.r[(k + 1) & 1];
    double *g = w.g[k & 1], *gp = w.g[(k + 1) & 1];
    double *hr = w.hr2, *hd = w.hr2 + f->m_tot;
    hipError_t e;
    // x(y) -> H x
    if ((e = dual_sweep(f, 1, it.x0, y, 0, w.hx, 0, done_flags(ctl), 1, st, active))) return e;
    if (it.backtrack == 1) {
        VecArgs ba = a;
        ba.hx = w.hx; ba.Rw = w.Rw; ba.hw = w.hw;
        hipLaunchKernelGGL(bt_kernel, grid, blk, 0, st, ba);
        hipLaunchKernelGGL(fin_bt_kernel, fgrid, blk, 0, st, ctl, a.part, a.nblocks, a.ndone);
    }
    a.y = y; a.yp = yn; a.hx = w.hx; a.rp = rp; a.r = r;
    a.S = w.S; a.Q = w.Qv;
    if (method == 1) {
        hipLaunchKernelGGL((resid_kernel<true, MEMCAP>), grid, blk, 0, st, a);
        hipLaunchKernelGGL(fin_resid_kernel, fgrid, dim3(kFin), 0, st, ctl, a.part, a.nblocks, 1, a.ndone, it.div_due);
        if (it.div_due && (e = enqueue_div_test(f, y, k == 0, st))) return e;
        if (it.poll && (e = enqueue_poll(*it.poll, w, st))) return e;
        VecArgs cb = a;
        cb.g = r;           // g = R
        cb.r = w.d;         // output direction
        hipLaunchKernelGGL((combine_kernel<MEMCAP>), grid, blk, 0, st, cb);
        // x-hat(r) and x-hat(d) in one two-right-hand-side sweep (p-NAMA)
        if ((e = dual_sweep(f, 0, nullptr, r, w.d - r, hr, hd - hr, done_flags(ctl), 2, st, active))) return e;
    } else {
        hipLaunchKernelGGL((resid_kernel<false, 0>), grid, blk, 0, st, a);
        hipLaunchKernelGGL(fin_resid_kernel, fgrid, dim3(kFin), 0, st, ctl, a.part, a.nblocks, 0, a.ndone, it.div_due);
        if (it.div_due && (e = enqueue_div_test(f, y, k == 0, st))) return e;
        if (it.poll && (e = enqueue_poll(*it.poll, w, st))) return e;
        // grad phi = R + lambda s H xhat(s R)
        if ((e = dual_sweep(f, 0, nullptr, r, 0, hr, 0, done_flags(ctl), 1, st, active))) return e;
        VecArgs ga = a;
        ga.hr = hr; ga.g = g; ga.gp = gp;
        hipLaunchKernelGGL((grad_kernel<MEMCAP>), grid, blk, 0, st, ga);
        hipLaunchKernelGGL(fin_grad_kernel, fgrid, dim3(kFin), 0, st, ctl, a.part, a.nblocks);
        VecArgs cb = a;
        cb.g = g; cb.r = w.d;
        hipLaunchKernelGGL((combine_kernel<MEMCAP>), grid, blk, 0, st, cb);
        if ((e = dual_sweep(f, 0, nullptr, w.d, 0, hd, 0, done_flags(ctl), 1, st, active))) return e;
    }
    VecArgs la = vec_args(f);
    la.method = method;
    la.y = y; la.rp = r; la.d = w.d; la.hx = w.hx; la.hr = hr; la.hd = hd; la.yn = yn;
    hipLaunchKernelGGL(ls_kernel<NUC>, grid, blk, 0, st, la);
    hipLaunchKernelGGL(fin_ls_kernel, fgrid, dim3(kFin), 0, st, ctl, a.part, a.nblocks, a.ndone, it.trace, it.trace_iters);
    if (it.backtrack == 1) { la.Rw = w.Rw; la.hw = w.hw; }
    hipLaunchKernelGGL(update_kernel, grid, blk, 0, st, la);
    return hipGetLastError();
}

// One GPAD update at the point w (kept in ybuf[0], the caller's buffer), with
// the main sequence y^k in ybuf[1].
hipError_t enqueue_gpad(const tree_factors *f, const IterArgs &it, hipStream_t st)
{
    const SolverWS &w = f->sws;
    VecArgs a = vec_args(f);
    a.method = 2;
    Ctl *ctl = a.ctl;
    const dim3 grid(a.nblocks), blk(kVB), fgrid(f->ninst);
    double *wv = it.ybuf[0], *ym = it.ybuf[1], *r = w.r[0];
    hipError_t e;
    if ((e = dual_sweep(f, 1, it.x0, wv, 0, w.hx, 0, done_flags(ctl), 1, st, it.active))) return e;
    a.y = wv; a.hx = w.hx; a.r = r;
    hipLaunchKernelGGL((resid_kernel<false, 0>), grid, blk, 0, st, a);
    hipLaunchKernelGGL(fin_resid_kernel, fgrid, dim3(kFin), 0, st, ctl, a.part, a.nblocks, 0, a.ndone, it.div_due);
    if (it.div_due && (e = enqueue_div_test(f, wv, it.k == 0, st))) return e;
    if (it.poll && (e = enqueue_poll(*it.poll, w, st))) return e;
    hipLaunchKernelGGL(fin_gpad_kernel, fgrid, dim3(64), 0, st, ctl);
    VecArgs ua = a;
    ua.g = wv; ua.r = r; ua.yn = ym;
    hipLaunchKernelGGL(gpad_update_kernel, grid, blk, 0, st, ua);
    return hipGetLastError();
}

using IterFn = hipError_t (*)(const tree_factors *, const IterArgs &, hipStream_t);

// Variant for the L-BFGS memory (accumulators per pair slot) and the number
// of line-search trials; the default options (mem 5, nu_max 10) have their own.
template <int NUC>
IterFn pick_iter_mem(int mem)
{
    if (mem <= 4) return enqueue_iteration<4, NUC>;
    if (mem == 5) return enqueue_iteration<5, NUC>;
    if (mem <= 8) return enqueue_iteration<8, NUC>;
    return enqueue_iteration<16, NUC>;
}

IterFn pick_iter(int mem, int nu_max)
{
    return nu_max <= kNuDefault ? pick_iter_mem<kNuDefault>(mem) : pick_iter_mem<kNuCap>(mem);
}

// Power iteration on every instance (per-instance normalisation); leaves
// L_b in the control blocks.
int power_iterations(tree_factors *f, int iters, hipStream_t st)
{
    const SolverWS &w = f->sws;
    VecArgs a = vec_args(f);
    const dim3 grid(a.nblocks), blk(kVB), fgrid(f->ninst);
    double *v = w.r[0], *wv = w.r[1], *hv = w.hx;
    VecArgs pa = a;
    pa.yn = v;
    hipLaunchKernelGGL(power_init_kernel, grid, blk, 0, st, pa);
    for (int it = 0; it < iters; ++it) {
        hipError_t e = dual_sweep(f, 0, nullptr, v, 0, hv, 0, nullptr, 1, st);
        if (e != hipSuccess) { set_error(std::string("dual_lipschitz: ") + hipGetErrorString(e)); return STOTREE_ERR_DEVICE; }
        pa.y = v; pa.hx = hv; pa.r = wv; pa.yn = v;
        hipLaunchKernelGGL(power_step_kernel, grid, blk, 0, st, pa);
        hipLaunchKernelGGL(power_fin_kernel, fgrid, blk, 0, st, a.ctl, a.part, a.nblocks);
        hipLaunchKernelGGL(power_scale_kernel, grid, blk, 0, st, pa);
    }
    STOTREE_HIP(hipGetLastError());
    return STOTREE_OK;
}

// Host copy of the control blocks with the block ranges filled in.
std::vector<Ctl> fresh_ctl(const tree_factors *f)
{
    std::vector<Ctl> h(f->ninst);
    for (int b = 0; b < f->ninst; ++b) {
        Ctl &c = h[b];
        std::memset(&c, 0, sizeof(Ctl));
        c.first_blk = f->sws.blk_first[b];
        const int next = b + 1 < f->ninst ? f->sws.blk_first[b + 1] : f->sws.nblocks;
        c.nblk = next - c.first_blk;
        c.gamma = 1.0;
        c.theta = 1.0;
        c.nodiv = 1;
        c.status = STOTREE_NOT_CONVERGED;
    }
    return h;
}

}  // namespace

int lipschitz(const tree_factors *fc, int iters, double *L, hipStream_t st)
{
    tree_factors *f = const_cast<tree_factors *>(fc);
    const SolverWS &w = f->sws;
    int rc = ensure_solver_ws(f, WsNeed{w.buf ? w.mem : 1, w.has_g, w.has_div, w.has_bt});
    if (rc) return rc;
    if ((rc = ensure_sweep_ws(f, 2))) return rc;
    std::vector<Ctl> h = fresh_ctl(f);
    Ctl *dctl = reinterpret_cast<Ctl *>(f->sws.ctl);
    STOTREE_HIP(hipMemcpyAsync(dctl, h.data(), sizeof(Ctl) * h.size(), hipMemcpyHostToDevice, st));
    if ((rc = power_iterations(f, iters, st))) return rc;
    STOTREE_HIP(hipMemcpyAsync(h.data(), dctl, sizeof(Ctl) * h.size(), hipMemcpyDeviceToHost, st));
    STOTREE_HIP(hipStreamSynchronize(st));
    for (int b = 0; b < f->ninst; ++b) L[b] = h[b].L;
    return STOTREE_OK;
}

int solve(const tree_factors *fc, const double *x0, const solver_opts *opts_in, double *y_io, double *x,
          double *u, solver_info *info, hipStream_t st, int method)
{
    tree_factors *f = const_cast<tree_factors *>(fc);
    solver_opts o{};
    o.eps = 1e-6; o.eps_curv = 1e-12; o.mem = 5; o.nu_max = 10; o.max_iter = 1000; o.check_every = 1;
    if (opts_in) o = *opts_in;
    if (o.mem < 1 || o.mem > kMemMax || o.nu_max < 0 || o.nu_max > kNuCap || o.max_iter < 0 ||
        o.check_every < 1 || !(o.eps >= 0.0) || !(o.lambda >= 0.0) || !(o.eps_curv >= 0.0) ||
        o.backtrack < 0 || o.backtrack > 2 || o.trace_iters < 0 || (o.trace_iters > 0 && !o.trace)) {
        set_error("solve: options out of range (mem 1..16, nu_max 0..30, check_every >= 1, backtrack 0..2)");
        return STOTREE_ERR_ARG;
    }
    const int backtrack = method == 2 ? 0 : o.backtrack;
    if ((backtrack == 1 && !(o.bt_param >= 0.0 && o.bt_param < 1.0)) ||
        (backtrack == 2 && !(o.bt_param > 0.0 && o.bt_param < 0.5))) {
        set_error("solve: bt_param must lie in [0, 1) for backtracking test 1 and in (0, 1/2) for test 2");
        return STOTREE_ERR_ARG;
    }
    const int div_window = o.div_window == 0 ? 50 : (o.div_window < 0 ? 0 : o.div_window);
    int rc = ensure_solver_ws(f, WsNeed{o.mem, method == 0, div_window > 0, backtrack == 1});
    if (rc) return rc;
    if ((rc = ensure_sweep_ws(f, 2))) return rc;
    PollLease poll;
    if ((rc = poll.take())) return rc;
    const SolverWS &w = f->sws;
    Ctl *dctl = reinterpret_cast<Ctl *>(w.ctl);
    std::vector<Ctl> h = fresh_ctl(f);
    std::vector<double> lam(f->ninst, o.lambda);
    if (o.lambda == 0.0) {
        // with backtracking a short power iteration suffices: its Rayleigh
        // quotient is at most L, so the start 1/L-hat is at least 1/L and the
        // tests bring it down
        std::vector<double> L(f->ninst);
        if ((rc = lipschitz(f, backtrack ? 5 : 100, L.data(), st))) return rc;
        for (int b = 0; b < f->ninst; ++b) {
            if (!(L[b] > 0.0) || !std::isfinite(L[b])) {
                set_error("solve: could not estimate L of instance " + std::to_string(b));
                return STOTREE_ERR_NUMERIC;
            }
            lam[b] = backtrack ? 1.0 / L[b] : 1.0 / (1.1 * L[b]);
        }
    }
    for (int b = 0; b < f->ninst; ++b) {
        Ctl &c = h[b];
        c.max_iter = o.max_iter; c.mem = o.mem; c.nu_max = o.nu_max; c.method = method;
        c.lam = lam[b]; c.eps = o.eps; c.eps_curv = o.eps_curv;
        c.backtrack = backtrack; c.bt_param = o.bt_param;
    }
    STOTREE_HIP(hipMemcpyAsync(dctl, h.data(), sizeof(Ctl) * h.size(), hipMemcpyHostToDevice, st));
    STOTREE_HIP(hipMemsetAsync(w.ndone, 0, sizeof(int), st));
    double *ybuf[2] = {y_io, w.y[1]};
    if (method == 2) {
        // GPAD: y^0 = y^{-1} = the initial dual (w^0 = y^0 in the caller's buffer)
        VecArgs ca = vec_args(f);
        ca.y = y_io; ca.yn = w.y[1];
        hipLaunchKernelGGL(copy_kernel, dim3(ca.nblocks), dim3(kVB), 0, st, ca);
    }
    IterFn iter = method == 2 ? enqueue_gpad : pick_iter(o.mem, o.nu_max);
    // each halving of lambda costs one update that does not count
    const int last = o.max_iter + (backtrack ? kBtMax + 1 : 0);
    int k = 0, ndone = 0, ahead = 0, polls = 0;
    // instances finished by the last check are skipped by the sweeps (the
    // count may lag behind by check_every iterations, in GPAD by one more; it
    // only grows)
    auto enqueue = [&](bool polled) -> hipError_t {
        IterArgs it{x0, {ybuf[0], ybuf[1]}, k, method, f->ninst - ndone,
                    div_window > 0 && k % div_window == 0, backtrack, o.trace, o.trace_iters, polled ? &poll : nullptr};
        ++k;
        return iter(f, it, st);
    };
    // The host reads the count while the device has work (36 us an iteration
    // otherwise).  Instances finish at the residual, in the middle of an
    // iteration, so the count is requested there and the host waits with the rest
    // of the iteration queued behind it; a solve that ends has queued no launch for
    // the poll.  One whole iteration more goes in before the host waits where that
    // cannot be in vain, in a solve without a residual to stop at (eps = 0: it runs
    // to max_iter; 0.5 to 3% on trees swept in bands), and for GPAD, which has only
    // two short kernels behind its residual, from the second poll on (if the count
    // then ends the solve, those kernels find every instance finished).
    // Accepted at the first residual, against always queueing one more: MINFBE on
    // the 6,485-node tree with nx=50, nu=30 588 us (660), on the 4,095-node
    // two-mode tree 197 (237), GPAD there 183 (195); 20 iterations of NAMA on an
    // 8-scenario tree with nx=4, nu=2 and eps > 0 1,612 (1,559), elsewhere the same.
    while (ndone < f->ninst && k <= last) {
        const bool inside = o.eps > 0.0 && (method != 2 || polls == 0);
        hipError_t e = hipSuccess;
        for (int c = ahead; c < o.check_every && k <= last && e == hipSuccess; ++c)
            e = enqueue(inside && (c + 1 == o.check_every || k == last));
        if (e == hipSuccess && !inside) e = enqueue_poll(poll, w, st);
        ahead = 0;
        ++polls;
        if (e == hipSuccess && !inside && k <= last) {
            e = enqueue(false);
            ahead = 1;
        }
        if (e != hipSuccess) {
            (void)hipStreamSynchronize(st);    // what is queued writes the caller's buffers
            set_error(std::string("solve: ") + hipGetErrorString(e));
            return STOTREE_ERR_DEVICE;
        }
        STOTREE_HIP(poll.wait());
        ndone = *poll.count;
    }
    if (method != 2) {
        // last iterate of every instance into y_io (GPAD keeps it there)
        VecArgs ga = vec_args(f);
        ga.y = w.y[1]; ga.yn = y_io;
        hipLaunchKernelGGL(gather_final_kernel, dim3(ga.nblocks), dim3(kVB), 0, st, ga);
    }
    // x(y) in the caller's layout
    SweepArgs a = sweep_args(f, 1);
    a.x0 = x0;
    a.y = y_io;
    if (f->cmap) {
        hipError_t e = map_to_xu(f, y_io, f->m_tot, w.xu, 1, st);
        if (e != hipSuccess) { set_error(std::string("solve: ") + hipGetErrorString(e)); return STOTREE_ERR_DEVICE; }
        a.y = w.xu;
    }
    a.xo = x; a.uo = u; a.dual_out = 0;
    hipError_t e = launch_sweep_any(f, a, 1, st);
    if (e != hipSuccess) { set_error(std::string("solve: ") + hipGetErrorString(e)); return STOTREE_ERR_DEVICE; }
    STOTREE_HIP(hipMemcpyAsync(h.data(), dctl, sizeof(Ctl) * h.size(), hipMemcpyDeviceToHost, st));
    STOTREE_HIP(hipStreamSynchronize(st));
    solver_info agg{};
    agg.status = STOTREE_OK;
    for (int b = 0; b < f->ninst; ++b) {
        const Ctl &c = h[b];
        solver_info &in = f->last_info[b];
        in = solver_info{};
        in.iters = c.iter;
        in.sweeps_affine = c.sweeps_aff + 1;
        in.sweeps_hom = c.sweeps_hom;
        in.ls_trials = c.ls_trials;
        in.lbfgs_push = c.pushes;
        in.lbfgs_skip = c.skips;
        in.status = c.status;
        in.res_scaled_inf = c.res;
        in.res_unscaled_inf = c.resu;
        in.lambda = c.lam;
        in.backtracks = c.backtracks;
        agg.iters = std::max(agg.iters, in.iters);
        agg.sweeps_affine = std::max(agg.sweeps_affine, in.sweeps_affine);
        agg.sweeps_hom = std::max(agg.sweeps_hom, in.sweeps_hom);
        agg.ls_trials += in.ls_trials;
        agg.lbfgs_push += in.lbfgs_push;
        agg.lbfgs_skip += in.lbfgs_skip;
        agg.backtracks = std::max(agg.backtracks, in.backtracks);
        agg.res_scaled_inf = std::max(agg.res_scaled_inf, in.res_scaled_inf);
        agg.res_unscaled_inf = std::max(agg.res_unscaled_inf, in.res_unscaled_inf);
        if (in.status < 0) agg.status = std::min(agg.status, in.status);
        else if (agg.status >= 0 && in.status == STOTREE_NOT_CONVERGED) agg.status = STOTREE_NOT_CONVERGED;
    }
    agg.lambda = h[0].lam;
    *info = agg;
    if (agg.status == STOTREE_ERR_NUMERIC) set_error("solve: non-finite values in the iterates (or lambda halved too often)");
    if (agg.status == STOTREE_ERR_DIVERGED) set_error("solve: the infeasibility test fired (no point meets the constraints)");
    return agg.status;
}

}  // namespace stotree
