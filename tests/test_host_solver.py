"""The solvers' host loop (no GPU: kernel launches are logged and not run; the test plays the device's
part of counting finished instances)."""
import hostsim

SETUP = """
    # the residual's decision number `stop` ends the solve: it counts every instance as finished
    state = dict(seen=0, stop=0, ninst=1)

    @C.CFUNCTYPE(None, C.c_char_p, C.POINTER(C.c_void_p))
    def on_launch(name, args):
        if b"fin_resid_kernel" in name:
            if state["seen"] == state["stop"]:
                ndone = C.cast(args[4], C.POINTER(C.c_void_p))[0]      # fin_resid_kernel(ctl, part, nblocks, with_pair, ndone, div_due)
                C.cast(ndone, C.POINTER(C.c_int))[0] = state["ninst"]
            state["seen"] += 1

    fake.fake_on_launch(on_launch)
    SOLVERS = dict(nama=L.nama_solve, minfbe=L.minfbe_solve, gpad=L.gpad_solve)

    def solve(tf, method, stop, check_every=1, max_iter=1000, eps=1e-6):
        state.update(seen=0, stop=stop, ninst=tf.ninst)
        info = st.SolverInfo()
        opts = st.make_opts(lam=0.1, eps=eps, max_iter=max_iter, check_every=check_every, div_window=-1)
        calls()
        rc = SOLVERS[method](tf.handle, buf(tf.x0_len), C.byref(opts), buf(tf.m), buf(tf.x_len), buf(tf.u_len),
                             C.byref(info), None)
        assert rc >= 0, (rc, st.stotree_last_error())
        return calls()
"""


def _run(body):
    import textwrap
    hostsim.run(textwrap.dedent(SETUP) + textwrap.dedent(body))


def test_a_solve_that_stops_queues_no_further_iteration():
    """The residual of iteration `stop` ends the solve: NAMA and MINFBE queue the iterations up to that
    one and nothing of the next; GPAD at most one more, and none at the first residual.  The number of
    residuals seen is the number of iterations queued."""
    _run("""
        for prob in (problem([2, 2, 2], 4, 2), problem([2, 2, 1, 1], 40, 20)):
            tf = factor(prob)
            for method in SOLVERS:
                for stop in (0, 1, 2, 5):
                    solve(tf, method, stop)
                    queued = stop + 1 + (method == "gpad" and stop > 0)
                    assert state["seen"] == queued, (method, stop, state["seen"])
                solve(tf, method, stop=4, check_every=3)
                assert state["seen"] == (7 if method == "gpad" else 6), (method, state)
                # never stopped by the device: max_iter + 1 residuals
                solve(tf, method, stop=10 ** 9, max_iter=7)
                assert state["seen"] == 8, (method, state)
            tf.free()
    """)


def test_the_host_waits_with_work_queued_behind_the_count():
    """NAMA and MINFBE: between the request of the count and the host's wait lies the second half of the
    iteration."""
    _run("""
        tf = factor(problem([2, 2, 2], 4, 2))
        for method in ("nama", "minfbe"):
            log = solve(tf, method, 3)
            waits = [k for k, ln in enumerate(log) if ln == "event sync"]
            assert len(waits) == 4
            for w in waits:
                r = max(k for k in range(w) if log[k] == "event record")
                between = launches(log[r:w])
                assert any(n.startswith("ls_kernel") for n in between) and "update_kernel" in between, between
    """)


def test_new_handles_need_no_new_pinned_memory():
    """A controller that factors and solves again at every instant: pinned memory and events are
    allocated for the first solve only; concurrent solves get their own, and no more than 16 are kept."""
    _run("""
        import threading
        count = lambda log: sum(ln.startswith(("hostmalloc", "event create")) for ln in log)
        total = 0
        for _ in range(20):
            tf = factor(problem([2, 2], 3, 1))
            total += count(solve(tf, "nama", 1))
            tf.free()
        assert total == 2, total
        # 40 threads inside a solve at once
        inside = threading.Barrier(40)

        @C.CFUNCTYPE(None, C.c_char_p, C.POINTER(C.c_void_p))
        def meet(name, args):
            if b"gather_final" in name:
                inside.wait(60)

        fake.fake_on_launch(meet)
        tfs = [factor(problem([2, 2], 3, 1)) for _ in range(40)]
        opts = st.make_opts(lam=0.1, max_iter=0, div_window=-1)
        args = [[C.c_void_p(v) for v in (buf(t.x0_len), buf(t.m), buf(t.x_len), buf(t.u_len))] for t in tfs]
        def go(t, a):
            info = st.SolverInfo()
            assert L.nama_solve(t.handle, a[0], C.byref(opts), a[1], a[2], a[3], C.byref(info), None) == 1
        def round_():
            th = [threading.Thread(target=go, args=ta) for ta in zip(tfs, args)]
            for t in th: t.start()
            for t in th: t.join()
        calls()
        round_()
        assert count(calls()) == 2 * 39
        round_()
        assert count(calls()) == 2 * 24          # 16 kept
    """)


def test_blocks_of_the_vector_passes():
    """A thread per row up to 196,608 rows in all, then 1,024 rows a block, 1,024 blocks an instance at most."""
    _run("""
        for branching, nx, nu, copies in (([2, 2, 2], 4, 2, 1), ([64, 64], 40, 7, 1), ([64, 64], 40, 12, 1), ([16, 16], 20, 10, 40)):
            p = problem(branching, nx, nu)
            tf = factor(p) if copies == 1 else factor(*[p] * copies)
            m = p.m
            per = 256 if tf.m <= 196608 else 1024
            log = solve(tf, "nama", 0)
            grid = {int(ln.split()[3]) for ln in log if "12resid_kernel" in ln}
            assert grid == {copies * min(1024, -(-m // per))}, (m, grid)
            tf.free()
        assert per == 1024 and 256 * 768 == 196608
    """)


def test_a_solve_without_a_residual_to_stop_at_keeps_one_iteration_ahead():
    """eps = 0: the host waits for the count of one iteration with the whole next one queued, and never
    queues more than max_iter asks for."""
    _run("""
        tf = factor(problem([2, 2, 2], 4, 2))
        for method in SOLVERS:
            log = solve(tf, method, 10 ** 9, max_iter=6, eps=0.0)
            assert state["seen"] == 7
            waits = [k for k, ln in enumerate(log) if ln == "event sync"]
            resid = lambda part: sum("fin_resid_kernel" in ln for ln in part)
            assert [resid(log[:w]) for w in waits] == [2, 3, 4, 5, 6, 7], method
    """)
