"""What the library's host code asks of the HIP runtime, and what it leaves
behind when the runtime refuses, on a stub runtime (no GPU, kernels do
nothing)."""
import pytest

import hip_stub


def test_batch_keeps_its_tables_when_new_ones_are_refused(tmp_path):
    """A choice whose tables cannot be allocated leaves the batch with the
    choice and the tables it had: the next step launches what it did before."""
    hip_stub.run(tmp_path, """
        b = batch([((300,), 2), ((2000, 300), 0), ((90, 90), 1)])
        b.set_depth(1)
        b.set_graphs(False)
        log()
        b.step(8)
        before = log()
        assert sum("k_batch_regions" in x for x in before) == 8
        stub.stub_refuse_from(ctypes.c_uint64(1))
        for change in (lambda: b.set_region(32), lambda: b.set_depth(8), lambda: b.set_region(0),
                       lambda: b.set_resident_limit(0), lambda: b.autotune(2)):
            try:
                change()
                raise SystemExit("a refused allocation went unnoticed")
            except ace.AceError as e:
                assert e.code == ace.ACE_E_NOMEM, e.code
            log()
            b.step(8)
            assert log() == before
            b.monitor()
            assert not any("(nil)" in x.split("args")[1] for x in log() if "args" in x)
        stub.stub_refuse_from(ctypes.c_uint64(2 ** 64 - 1))
        b.set_depth(4)
        log()
        b.step(8)
        assert sum("k_batch_regions" in x for x in log()) == 2
        b.close()
    """)


def test_leaving_a_capturing_stream_does_not_wait_for_it(tmp_path):
    """Switching a handle away from, or to, a stream under capture issues no
    synchronisation (one on the old stream would break its capture); between
    streams that do not capture it waits for the old one."""
    hip_stub.run(tmp_path, """
        A, B = 0x1000, 0x2000
        s = solver(2, (300, 200), 0)
        b = batch([((300,), 2), ((200, 300), 0)])
        p = ace.Pop(2, [64, 64], [0.0, 0.0], [64.0, 64.0], 7.0, 1e-3, 2)
        for h in (s, b, p):
            h.set_stream(A)
            log()
            h.set_stream(B)
            assert log() == ["sync 0x1000"]
            stub.stub_set_capturing(ctypes.c_void_p(A), 1)
            h.set_stream(A)
            if h is s:
                h.step(3)
            h.set_stream(B)
            assert not [x for x in log() if "sync" in x or "broken" in x]
            stub.stub_set_capturing(ctypes.c_void_p(A), 0)
            h.set_stream(None)
            h.close()
    """)


def test_population_step_that_fails_on_the_way(tmp_path):
    """A launch refused in the middle of a call whose inner steps write phi alone
    leaves the handle at the state the call began with: its step count, and phi
    from its populations at the next step."""
    hip_stub.run(tmp_path, """
        import numpy as np
        p = ace.Pop(2, [64, 64], [0.0, 0.0], [64.0, 64.0], 7.0, 1e-3, 2)
        p.set_phi0(np.zeros((64, 64)))
        p.step(2)
        log()
        stub.stub_fail_launch(ctypes.c_int64(3))
        try:
            p.step(6)
            raise SystemExit("a refused launch went unnoticed")
        except ace.AceError as e:
            assert e.code == ace.ACE_E_HIP
        stub.stub_fail_launch(ctypes.c_int64(-1))
        assert L.ace_pop_step_count(p._h) == 2
        log()
        p.step(1)
        assert ["k_pop_moment" in x for x in log()] == [True, False]
        assert L.ace_pop_step_count(p._h) == 3
        p.close()
    """)


def test_checkpointed_forward_replays_graphs(tmp_path):
    """Segments of many launches are replayed between the launches that read and
    write checkpoints; a launch refused on the way leaves the step count of the
    field the handle holds."""
    hip_stub.run(tmp_path, """
        import numpy as np
        s = solver(3, (24, 20, 28), 0)
        s.set_kernel(ace.ACE_KERNEL_DIRECT)  # one step per launch
        phi = np.zeros(s.shape)
        s.set_graph_launches(32)
        log()
        s.forward_ckpt(phi, 450, 150)
        lines = log()
        steps = [x for x in lines if x.startswith("launch")]
        assert sum(x == "instantiate" for x in lines) <= 2  # (one per buffer the segments begin in)
        assert sum(x == "replay" for x in lines) == 9  # 3 of 32 steps a segment
        captured = 32 * sum(x == "instantiate" for x in lines)
        assert len(steps) - captured == 450 - 9 * 32
        assert s.step_count == 450
        s.set_graph_launches(0)
        for after in (1, 3, 4, 5):
            stub.stub_fail_launch(ctypes.c_int64(after))
            try:
                s.forward_ckpt(phi, 12, 4)
                raise SystemExit("a refused launch went unnoticed")
            except ace.AceError:
                pass
            # (launch 4 writes the second checkpoint, not the handle's field)
            assert s.step_count == (3 if after == 4 else after)
        stub.stub_fail_launch(ctypes.c_int64(-1))
        s.close()
    """)


@pytest.mark.parametrize("M,kernel", [((60_000_000, 1), "k_tb"), ((1, 300_000_000), "k_tb"), ((500_000_000, 1), "k_step_direct"),
                                      ((2 ** 30, 1), "k_step_direct"), ((200_000_000, 1, 1), "k_t"), ((1, 1, 2 ** 28 - 1), "k_col3d"),
                                      ((8, 20000, 20000), "k_tblock3d"), ((1000, 1000), "k_tb2"), ((200, 200, 200), "k_tb3")])
def test_default_launches_hold_thin_fields(tmp_path, M, kernel):
    """Fields with an axis of a few nodes, whose regions would be more workgroups of
    1024 threads than one launch holds (2^32 work items): the default run, its
    monitors and a reverse sweep launch nothing that is refused."""
    hip_stub.run(tmp_path, f"""
        M = {M!r}
        s = solver(len(M), M, 1)
        for n in (23, 3, 2, 1):
            log()
            s.step(n)
            lines = log()
            assert lines and all(x.startswith("launch") for x in lines), lines
            if n == 23:
                assert all({kernel!r} in x for x in lines[:1]), lines
        E = np.zeros(16)
        e, m = E.ctypes.data_as(ctypes.POINTER(ctypes.c_double)), E.ctypes.data_as(ctypes.POINTER(ctypes.c_double))
        assert L.ace_run_monitored(s._h, 23, 10, e, m) in (0, 3, 4)
        assert not [x for x in log() if x.startswith("refused")]
        phi = ctypes.c_void_p(L.ace_field_ptr(s._h))
        if s.total < 2 ** 30:
            assert L.ace_forward_ckpt(s._h, phi, ace.ACE_DEVICE, 7, 4) == 0
            g = ctypes.c_double()
            assert L.ace_backward(s._h, phi, phi, ctypes.byref(g), ace.ACE_DEVICE) == 0
        assert not [x for x in log() if x.startswith("refused")]
        s.close()
    """)


def test_batch_splits_launches_of_many_pieces(tmp_path):
    """A launch of a batch with more pieces than one launch holds is split."""
    hip_stub.run(tmp_path, """
        b = batch([((500_000_000, 1), 1), ((300,), 2)])
        b.set_region(64)
        for call in (lambda: b.step(8), b.monitor, lambda: L.ace_batch_get_all(b._h, ctypes.c_void_p(4096), ace.ACE_DEVICE)):
            log()
            call()
            lines = [x for x in log() if "launch" in x or "refused" in x]
            assert lines and all(x.startswith("launch") for x in lines), lines
        b.set_graphs(False)
        b.step(8)
        regions = [x for x in log() if "k_batch_regions" in x]
        grids = [int(x.split("grid ")[1].split()[0]) for x in regions]
        tables = [int(x.split()[-1], 16) for x in regions]
        assert len(grids) > 2 and max(grids) * 1024 < 2 ** 32
        per = len(grids) // 2  # (two rounds)
        assert sum(grids[:per]) >= 500_000_000 // 62
        assert all(t1 - t0 == 12 * g for t0, t1, g in zip(tables[:per], tables[1:per], grids))
        b.close()
    """)


def test_batch_captures_one_graph(tmp_path):
    """Calls of many different step counts share one graph of 64 rounds, captured
    by the first call it fits into; no call leaves an odd round to copy back."""
    hip_stub.run(tmp_path, """
        b = batch([((300,), 2), ((200, 300), 0), ((90, 90), 1)])
        b.set_depth(5)
        log()
        b.step(319)
        assert not [x for x in log() if x in ("instantiate", "replay")]
        seen = []
        for n in list(range(320, 360)) + [641, 1000, 2100, 5000]:
            b.step(n)
            lines = log()
            seen += lines
            replays = sum(x == "replay" for x in lines)
            assert replays == n // 320 - (n % 320 == 1)
            assert not [x for x in lines if "k_batch_copy" in x]
            direct = sum("k_batch_regions" in x for x in lines) - 64 * ("instantiate" in lines)
            assert direct <= 66
        assert sum(x == "instantiate" for x in seen) == 1
        b.set_depth(4)
        b.step(256)
        assert sum(x == "instantiate" for x in log()) == 1
        b.close()
    """)


def test_batch_autotuner_trials(tmp_path):
    """The batch autotuner times the depth the batch chose by itself, and resident
    limits only where whole instances per workgroup are the fastest."""
    hip_stub.run(tmp_path, """
        import json
        def tune(first, step, fixed=0):
            b = batch([((200, 300), 0), ((90, 90), 1)])  # few regions: the rule takes depth 8
            if fixed:
                b.set_depth(fixed)
            stub.stub_elapsed(ctypes.c_float(first), ctypes.c_float(step))
            rec = json.loads(b.autotune(2))
            b.close()
            return [(c["region"], c["depth"]) for c in rec["candidates"]], rec["choice"]
        trials, choice = tune(100.0, -1.0)  # the last shape is the fastest
        assert trials[-1] == (64, 8) and len(trials) == 12
        assert (choice["region"], choice["depth"], choice["resident_limit"]) == (64, 8, 8000)
        trials, choice = tune(100.0, -1.0, fixed=8)
        assert trials[-1] == (64, 6) and len(trials) == 11 and choice["depth"] == 6
        trials, choice = tune(1.0, 1.0)  # the first one is
        assert trials[12:] == [(0, 4)] * 4 and choice["region"] == 0
    """)
