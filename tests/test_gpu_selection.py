"""GPU parity of the persistent selection's variants against the fp64 oracle
in follow mode (tolerances of tests/parity.py): rows in registers, streamed
rows, streamed rows with the weights in memory, at the edges of their ranges
(client rows at and beside multiples of 256, blocks with a partial share of
tokens, tokens beyond the held ones)."""
import pytest

from oracle import gmc_oracle as O
from paper_2608_02134_amd import synth

from .gpu_run import run
from .parity import check_problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

# batch, grid (frames, h, w), queries, budget; 8 query heads, so M = 8 T + N + 256
CASES = {
    "rows_1024": (40, (1, 8, 13), 3, 40),            # M = 384, J = 4, 6 blocks a problem
    "rows_2048_streams_rest": (16, (1, 19, 21), 16, 40),   # M = 783, J = 4, 25 tokens a block: 20 held
    "rows_3584_three": (8, (1, 15, 20), 200, 40),    # J = 14, R = 3
    "rows_3584_five": (12, (1, 15, 20), 200, 40),    # J = 14, R = 5
    "rows_5120_exact": (1, (1, 16, 24), 560, 60),    # J = 20, M = 5120
    "rows_5121": (1, (1, 5, 77), 560, 60),           # J = 24, M = 5121, odd
    "rows_many_tokens": (1, (1, 42, 50), 200, 48),   # J = 20, R = 3, N = 2100
    "rows_6144_below": (1, (1, 1, 287), 700, 33),    # J = 24, M = 6143
    "rows_7168": (1, (1, 16, 17), 830, 33),          # J = 28, M = 7168
    "rows_8192": (1, (1, 9, 9), 980, 33),            # J = 32, fewer tokens than two a wave
    "rows_9216": (1, (1, 10, 14), 1100, 33),         # J = 36, M = 9196
    "rows_12288": (2, (1, 10, 13), 1480, 33),        # J = 48
    "streamed": (2, (1, 11, 12), 1600, 33),          # M = 13188: weights and coverage in LDS
    "streamed_weights_in_memory": (2, (1, 9, 11), 2400, 33),   # M = 19555
    "rows_1376_five": (16, (1, 16, 20), 100, 40),    # J = 8, every token held
    # tokens beyond the held ones streamed
    "rows_1497_and_streamed": (16, (1, 21, 21), 100, 40),   # J = 8, 28 tokens a block: 20 held
    "rows_2297_and_streamed": (12, (1, 21, 21), 200, 40),   # J = 14, 21: 20
    "rows_4676_and_streamed": (6, (1, 30, 34), 425, 40),    # J = 20, 25: 12
    "rows_5456_and_streamed": (8, (1, 20, 20), 600, 40),    # J = 24, 13: 12
    "rows_7056_and_streamed": (8, (1, 20, 20), 800, 40),    # J = 28, 13: 8
    "rows_7856_and_streamed": (8, (1, 20, 20), 900, 40),    # J = 32, 13: 8
    "rows_9056_and_streamed": (8, (1, 20, 20), 1050, 40),   # J = 36, 13: 8
    "rows_11056_and_streamed": (2, (1, 20, 20), 1300, 40),  # J = 48, 8: 4
    # all streamed: too few of the tokens would be held, too many problems
    "few_held": (16, (1, 30, 30), 16, 40),           # M = 1284, 57 tokens a block
    "seventeen_problems": (17, (1, 19, 21), 16, 40),
}


@pytest.mark.parametrize("case", list(CASES))
def test_selection_variants(case):
    batch, grid, t, k = CASES[case]
    prob = synth.make_problem("tiny", batch=batch, grid=grid, t=t, k=k)
    w = prob.workload
    print(f"\n[case] selection {case}: B={batch} N={w.n} T={t} K={k} M={8 * t + w.n + 256}", flush=True)
    outs, pr = run(prob, torch)
    pr.close()
    for b in sorted({0, batch // 2, batch - 1}):
        rep = check_problem(prob.hidden[b], prob.text_q[b], prob.vis_k[b], prob.pos3d[b], prob.probe, k, outs[b],
                            w.dtype, O.GmcParams())
        print(f"  problem {b}: {rep}", flush=True)


def test_batches_above_sixteen():
    """Batches of b = 32 from pools of 64: the batch's tokens reach the blocks
    that own no row chunk."""
    prob = synth.make_problem("tiny", grid=(1, 20, 20), t=3, k=100)
    print(f"\n[case] selection b=32: N={prob.workload.n} K={prob.k}", flush=True)
    outs, pr = run(prob, torch, batch_b=32, pool_mult=2)
    pr.close()
    check_problem(prob.hidden[0], prob.text_q[0], prob.vis_k[0], prob.pos3d[0], prob.probe, prob.k, outs[0],
                  prob.workload.dtype, O.GmcParams(batch_b=32, pool_mult=2))


# batch, grid, queries, budget, overrides: shapes whose blocks stream tokens,
# where a call that traces its gains forms all of them and a plain one leaves
# out those that cannot enter the pool
LEFT_OUT = {
    "held_and_streamed": (16, (1, 19, 21), 16, 120, {}),
    "held_and_streamed_wide_rows": (8, (1, 20, 25), 700, 200, {}),
    "streamed": (2, (1, 11, 12), 1600, 100, {}),
    "weights_in_memory": (2, (1, 9, 11), 2400, 90, {}),
    "page": (1, (1, 64, 64), 40, 700, {}),
    "keys_in_memory": (1, (2, 50, 50), 24, 300, {"batch_b_bounded": 16}),
    "batch_of_62": (16, (1, 19, 21), 16, 200, {"batch_b": 62, "pool_mult": 1}),
    "batch_of_64": (16, (1, 19, 21), 16, 200, {"batch_b": 64, "pool_mult": 1}),
    "batch_of_1": (16, (1, 19, 21), 16, 60, {"batch_b": 1}),
}


@pytest.mark.parametrize("same", [False, True], ids=["drawn", "equal_tokens"])
@pytest.mark.parametrize("case", list(LEFT_OUT))
def test_gains_left_out(case, same):
    """A plain call selects what the traced one does: bit for bit, as the
    gains that both form are the same sums."""
    batch, grid, t, k, over = LEFT_OUT[case]
    prob = synth.make_problem("tiny", batch=batch, grid=grid, t=t, k=k)
    if same:   # every gain but those of a few tokens vanishes after the first picks
        prob.hidden[:, 3:] = prob.hidden[:, 3:4]
        prob.vis_k[:, 3:] = prob.vis_k[:, 3:4]
    print(f"\n[case] gains left out {case}: N={prob.workload.n} K={k} equal={same}", flush=True)
    full, pr = run(prob, torch, **over)
    plain, _ = run(prob, torch, trace=False, pruner=pr)
    pr.close()
    for b in range(batch):
        for key in ("out_idx", "out_pos", "out_hidden"):
            assert (full[b][key] == plain[b][key]).all(), (case, b, key)


@pytest.mark.parametrize("b,mult,k", [(17, 4, 60), (64, 4, 300), (65, 4, 200), (100, 3, 250), (512, 4, 3000),
                                      (1000, 2, 2100)])
def test_large_pools(b, mult, k):
    """Pools above 64: segments of one to eight positions per thread, partial
    ones, and a last round with fewer tokens left than the pool holds."""
    prob = synth.make_problem("tiny", grid=(1, 17, 242), t=3, k=k)
    print(f"\n[case] large pools: N={prob.workload.n} b={b} pool={b * mult} K={k}", flush=True)
    outs, pr = run(prob, torch, batch_b_bounded=b, pool_mult=mult)
    pr.close()
    check_problem(prob.hidden[0], prob.text_q[0], prob.vis_k[0], prob.pos3d[0], prob.probe, prob.k, outs[0],
                  prob.workload.dtype, O.GmcParams(batch_b_bounded=b, pool_mult=mult), app_proj=prob.app_proj)
