"""Context calls and static calls on two streams at once: every call gives the
bits it gives alone.  The context's selections here need the device to
themselves (rows held in registers, one and several problems), so they and the
static calls, launched eagerly or replayed from a graph, take turns."""
import threading
import time

import pytest

from paper_2608_02134_amd import binding, synth
from paper_2608_02134_amd.binding import make_pruner, to_device

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

CALLS = 12


def _tensors(prob):
    w = prob.workload
    return (to_device(prob.hidden, w.dtype, torch), to_device(prob.text_q, w.dtype, torch),
            to_device(prob.vis_k, w.dtype, torch), torch.from_numpy(prob.pos3d).cuda())


def _static_call(prob, cfg, x):
    """A call on the current stream into new outputs, as a function without allocations."""
    w = prob.workload
    kr = binding.gmc_realized_k(w.n, prob.k)
    out = (torch.zeros((w.batch, kr, w.d), dtype=x[0].dtype, device="cuda"),
           torch.zeros((w.batch, kr, 3), dtype=torch.int32, device="cuda"),
           torch.zeros((w.batch, kr), dtype=torch.int32, device="cuda"))

    def go():
        code = binding.gmc_prune_static(cfg, w.batch, *(t.data_ptr() for t in x), w.n, w.t, prob.k,
                                        *(o.data_ptr() for o in out), None, torch.cuda.current_stream().cuda_stream)
        assert code == binding.GMC_OK, binding.gmc_last_error()
    return go, out


def _same(got, want):
    return all(torch.equal(a, b) for a, b in zip(got, want))


@pytest.mark.parametrize("replayed", [False, True], ids=["eager", "graph"])
@pytest.mark.parametrize("batch,grid,t", [(1, (1, 16, 24), 560), (8, (1, 15, 20), 200), (16, (1, 19, 21), 16),
                                          (16, (1, 19, 21), 0)])
def test_context_and_static_calls_side_by_side(batch, grid, t, replayed):
    ctx = synth.make_problem("tiny", batch=batch, grid=grid, t=t, k=60)
    sta = synth.make_problem("tiny", grid=(1, 24, 25), t=24, k=120)
    print(f"\n[case] side by side: context B={batch} N={ctx.workload.n} T={t}, static N={sta.workload.n}, "
          f"replayed={replayed}", flush=True)
    pr = make_pruner(ctx, torch)
    try:
        xc, xs = _tensors(ctx), _tensors(sta)
        cfg = binding.GmcConfig.from_buffer_copy(pr.cfg)
        probe = to_device(sta.probe, sta.workload.dtype, torch)
        cfg.value_probe = probe.data_ptr()
        # alone
        want_c = [o.clone() for o in pr.prune(*xc, ctx.k)[:3]]
        go, out = _static_call(sta, cfg, xs)
        go()
        torch.cuda.synchronize()
        want_s = [o.clone() for o in out]
        streams = [torch.cuda.Stream(), torch.cuda.Stream()]
        graphs = []
        if replayed:
            for o in out:
                o.zero_()
            torch.cuda.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=streams[1]):
                go()
            torch.cuda.synchronize()
            graphs.append(g)
        torch.cuda.synchronize()
        got_c, got_s, errors = [], [], []

        def context_calls():
            try:
                with torch.cuda.stream(streams[0]):
                    for _ in range(CALLS):
                        got_c.append([o.clone() for o in pr.prune(*xc, ctx.k)[:3]])
            except BaseException as e:   # noqa: B036 - reported by the main thread
                errors.append(e)

        def static_calls():
            try:
                with torch.cuda.stream(streams[1]):
                    for _ in range(CALLS):
                        for o in out:
                            o.zero_()
                        graphs[0].replay() if replayed else go()
                        got_s.append([o.clone() for o in out])
            except BaseException as e:   # noqa: B036
                errors.append(e)

        threads = [threading.Thread(target=f) for f in (context_calls, static_calls)]
        for th in threads:
            th.start()
        for th in threads:
            th.join()
        torch.cuda.synchronize()
        assert not errors, errors
        code, diag = binding.gmc_get_diag(0)
        assert code == binding.GMC_OK, binding.gmc_last_error()
        assert len(got_c) == len(got_s) == CALLS
        assert all(_same(g, want_c) for g in got_c)
        assert all(_same(g, want_s) for g in got_s)
    finally:
        pr.close()


@pytest.mark.parametrize("batch,grid,t", [(1, (1, 24, 25), 24), (1, (1, 46, 47), 64), (1, (1, 16, 24), 560),
                                          (1, (1, 9, 11), 2400), (1, (1, 9, 11), 3200), (300, (1, 8, 8), 8)],
                         ids=["split", "streamed", "streamed_rows", "weights_in_memory", "rounds", "rounds_many"])
def test_static_routes_leave_their_turn(batch, grid, t):
    """Every way a static call selects gives what the context does, and a context
    call that needs the device to itself does not wait after it."""
    prob = synth.make_problem("tiny", batch=batch, grid=grid, t=t, k=40)
    wide = synth.make_problem("tiny", batch=1, grid=(1, 16, 24), t=560, k=40)
    print(f"\n[case] static route: B={batch} N={prob.workload.n} T={t}", flush=True)
    pr = make_pruner(prob, torch)
    try:
        x = _tensors(prob)
        want = [o.clone() for o in pr.prune(*x, prob.k)[:3]]
        cfg = binding.GmcConfig.from_buffer_copy(pr.cfg)
        probe = to_device(prob.probe, prob.workload.dtype, torch)   # (outlives pr, which the last calls follow)
        cfg.value_probe = probe.data_ptr()
        go, out = _static_call(prob, cfg, x)
        for o in out:
            o.zero_()
        go()
        torch.cuda.synchronize()
        assert torch.equal(out[2], want[2]) and torch.equal(out[1], want[1])
        # the same members and fp32 sums in one order: only the assignment's
        # gate could differ in its last bits
        torch.testing.assert_close(out[0], want[0], rtol=1e-5, atol=1e-5)
    finally:
        pr.close()
    pr = make_pruner(wide, torch)
    try:
        x = _tensors(wide)
        pr.prune(*x, wide.k)
        torch.cuda.synchronize()
        go()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        pr.prune(*x, wide.k)
        torch.cuda.synchronize()
        assert time.perf_counter() - t0 < 1.0   # (a turn that was not left costs 2 s)
        code, _ = binding.gmc_get_diag(0)
        assert code == binding.GMC_OK, binding.gmc_last_error()
    finally:
        pr.close()
