"""Schedules of a handle, host side (no GPU: kernel launches are logged and not run)."""
import hostsim


def test_failed_rebuild_keeps_the_schedule():
    """sweep_schedule and sweep_autotune that run out of memory leave the lists, the knobs and the
    recorded graphs of the handle as they were: the next sweep launches what it launched before."""
    hostsim.run("""
        for prob in (problem([2, 2, 1, 1, 1, 1, 1], 4, 2), problem([3, 3, 1, 1], 40, 20)):
            tf = factor(prob)
            rc, before = sweep(tf)
            assert rc == 0 and before
            knobs = st.sweep_schedule_get(tf)
            for at in range(3):
                fake.fake_fail_mallocs_from(at)
                try:
                    st.sweep_schedule(tf, (16, 0, 4, 3, 5))
                    ok = True
                except st.StotreeError as e:
                    assert e.code == -8, e
                    ok = False
                fake.fake_fail_mallocs_from(-1)
                if ok:
                    break
                assert st.sweep_schedule_get(tf) == knobs
                calls()
                assert sweep(tf) == (0, before)
            assert at > 0                       # at least one failure was seen
            st.sweep_schedule(tf, knobs)
            # the autotuner: its scratch, then a candidate's lists
            for at in (0, 3, 6, 12):
                fake.fake_fail_mallocs_from(at)
                try:
                    st.sweep_autotune(tf, stream=0)
                    assert False
                except st.StotreeError as e:
                    assert e.code == -8, e
                fake.fake_fail_mallocs_from(-1)
                assert st.sweep_schedule_get(tf)[4] == knobs[4]
                calls()
                rc, now = sweep(tf)
                assert rc == 0 and now
            tf.free()
    """)


def test_sweep_in_place_on_a_batch():
    """x or u in the memory of y: on a batch swept in bands no instance's results may be written while
    another's duals are still to be read, so no launch does both directions; one tree alone may."""
    hostsim.run("""
        prob = problem([2, 2, 2], 4, 2)
        both = lambda names: any("ELi2EE" in n for n in names if n.startswith("band_kernel"))
        for tf, apart in ((factor(prob), False), (factor(prob, prob, prob), True)):
            for nrhs in (1, 2):
                y = buf(nrhs * tf.m)
                for kw in (dict(x=y), dict(u=y), dict(x=y + 8 * (nrhs * tf.m - 1))):
                    rc, names = sweep(tf, nrhs, y=y, **kw)
                    assert rc == 0 and names and all(n.startswith("band_kernel") for n in names), names
                    assert both(names) != apart, (names, nrhs)
                assert both(sweep(tf, nrhs)[1])
            tf.free()
    """)


def test_which_chains_go_with_the_bands():
    """Chains below s* run in the bands where they are short, and in the chain kernels where those are
    the faster: at 16 lanes a node, many instances of one scenario, or long rows read in pairs.  An
    instance without a stage above s* does not send the others back to a launch per stage."""
    hostsim.run("""
        def kinds(*probs):
            tf = factor(*probs)
            rc, names = sweep(tf)
            tf.free()
            assert rc == 0
            return sorted({re.match("band|narrow_chain|[a-z]+_chain|[a-z]+_trunk|narrow_level", n).group(0) for n in names})

        one = lambda nx, nu, N: problem([1] * N, nx, nu)
        assert kinds(*[one(4, 2, 3)] * 500) == ["band"]
        assert kinds(*[one(20, 10, 3)] * 400) == ["band"]
        assert kinds(*[one(20, 10, 3)] * 401) == ["narrow_chain"]
        assert kinds(*[one(16, 16, 2)] * 256) == ["band"]
        assert kinds(*[one(16, 16, 2)] * 257) == ["narrow_chain"]
        assert kinds(one(16, 16, 3)) == ["narrow_chain"]
        for nx, nu, tail, with_bands in ((16, 16, 3, False), (16, 16, 2, True), (16, 9, 3, True), (16, 10, 3, False),
                                         (17, 15, 3, True), (17, 15, 4, False), (8, 8, 3, True), (8, 8, 4, False)):
            got = kinds(problem([2, 2] + [1] * tail, nx, nu))
            assert got == (["band"] if with_bands else ["band", "narrow_chain"]), (nx, nu, tail, got)
        # a mixed handle
        assert kinds(problem([3, 3], 4, 2), one(4, 2, 9)) == ["band", "narrow_chain"]
        assert kinds(problem([3, 3], 4, 2), problem([2, 1], 40, 20)) == ["bwd_trunk", "fwd_trunk", "narrow_chain"]
    """)


def test_autotune_leaves_knobs_without_effect():
    """Lane group, chain order and wavefront cap change nothing where stages and chains run in bands: the
    autotuner must not pick them on timing noise (here every later timing of the same work is a little
    shorter), and a cached schedule from before the bands is not applied."""
    hostsim.run("""
        import json, os, tempfile
        n = [0]

        @C.CFUNCTYPE(C.c_float)
        def elapsed():
            names = launches()
            n[0] += 1
            bands = names and all(k.startswith(("band_kernel", "narrow_chain_kernel")) for k in names)
            return (10.0 if bands else 1000.0) - 1e-3 * n[0]

        fake.fake_on_elapsed(elapsed)
        tf = factor(problem([2, 2, 1], 4, 2))                   # all in bands
        assert st.sweep_autotune(tf, stream=0)["knobs"] == [8, 1, 16, 0, 16]
        tf = factor(problem([2, 2] + [1] * 6, 4, 2))            # chains of their own: group and order count
        k = st.sweep_autotune(tf, stream=0)["knobs"]
        assert k[2:] == [16, 0, 16], k
        tf = factor(problem([3, 3, 1, 1], 40, 20))              # no bands: every knob counts
        k = st.sweep_autotune(tf, stream=0)["knobs"]
        assert k[2] == 2 and k[3] != 0, k
        # a cache written when launch form 0 was one launch per stage
        tf = factor(problem([2, 2, 1], 4, 2))
        cache = os.path.join(tempfile.mkdtemp(), "tune.json")
        old_key = re.sub(r":k5.*", ":k5", st.forest_signature(tf, 1))
        json.dump({old_key: {"knobs": [64, 0, 2, 0, 16], "ms": 1.0}}, open(cache, "w"))
        rec = st.sweep_autotune(tf, cache=cache, stream=0)
        assert not rec["cached"] and rec["knobs"] == [8, 1, 16, 0, 16], rec
        assert st.sweep_autotune(tf, cache=cache, stream=0)["cached"]
    """)


def test_stage_lists_are_uploaded_once_and_only_where_read():
    """Bytes of a schedule's lists (8 a pair, each list rounded to 64)."""
    hostsim.run("""
        def bytes_of(tf, knobs=(8, 1, 16, 0, 16)):
            calls()
            st.sweep_schedule(tf, knobs)
            return [int(ln.split()[1]) for ln in calls() if ln.startswith("malloc")]

        p = problem([4] * 5 + [1, 1], 20, 14)           # 341 nodes above 1,024 chains, two to a wavefront
        tf = factor(p)
        need = 8 * (341 + 1024 + 512)                   # stages; the panels' chains; the chain wavefronts
        (got,) = bytes_of(tf)
        assert need <= got <= need + 64 * 10, (got, need)
        (got,) = bytes_of(tf, (8, 1, 16, 2, 16))        # form 2: one list for panels, lane groups beside it
        assert need <= got <= need + 8 * 341 + 64 * 10, (got, need)
        got, counters = bytes_of(tf, (8, 1, 16, 1, 16))  # form 1: its entry nodes and counters
        assert need + 8 * 256 <= got <= need + 8 * 256 + 64 * 10 and counters == 4 * (tf.V + 1), (got, counters)
        # 8 copies in bands: nothing per stage but the panels' list of the first copy
        q = problem([4] * 5, 4, 2)
        tf = st.tree_factor_shared(q, 8, stream=0)
        tf1 = factor(q)
        (one,), (eight,) = bytes_of(tf1), bytes_of(tf)
        assert eight <= 8 * (one - 8 * 341) + 8 * 341 + 64 * 80, (one, eight)
    """)


def test_band_shapes_run_in_bands():
    """The shapes of the GPU tests of banded sweeps take the route those tests are about."""
    hostsim.run("""
        from test_gpu_bands import SHAPES, _prob
        for s in SHAPES:
            nx, nu, N, S, b0 = s
            tf = factor(_prob(s))
            for nrhs in (1, 2):
                rc, names = sweep(tf, nrhs)
                banded = nx + nu <= 32 and s[3:] not in ((65, 65), (41, 41))     # too wide; one child too many
                assert rc == 0 and any(n.startswith("band_kernel") for n in names) == banded, (s, names)
            tf.free()
    """)


def test_right_hand_sides_per_panel_workgroup():
    """Launches of 416 nodes or chains and more take all 64 copies in a workgroup, smaller ones 16."""
    hostsim.run("""
        for scen in (415, 416):
            p = treegen.draw_problem(treegen.capped_tree(4, scen, 21), 4, 2, np.random.default_rng(1))
            tf = st.tree_factor_shared(p, 64, stream=0)
            calls()
            rc, names = sweep(tf)
            got = {n for n in names if "chain64" in n}
            want = 64 if scen == 416 else 16
            assert rc == 0 and got == {f"bwd_chain64_kernelILi1ELi{want}EE", f"fwd_chain64_kernelILi1ELi{want}EE"}, names
            assert {n for n in names if "trunk64" in n} == {"bwd_trunk64_kernelILi1ELi16EE", "fwd_trunk64_kernelILi1ELi16EE"}
    """)
