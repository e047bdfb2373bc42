"""GPU parity against the fp64 oracle (tolerances of tests/parity.py) around
the token count from which the separability gate has its own launch."""
import pytest

from oracle import gmc_oracle as O
from paper_2608_02134_amd import synth

from .gpu_run import run
from .parity import check_problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)


@pytest.mark.parametrize("grid", [(1, 89, 92), (2, 64, 64), (1, 1, 8193)], ids=["8188", "8192", "8193"])
def test_gate_once(grid):
    prob = synth.make_problem("tiny", grid=grid, t=5, k=70)
    print(f"\n[case] gate once: N={prob.workload.n}", flush=True)
    outs, pr = run(prob, torch)
    pr.close()
    check_problem(prob.hidden[0], prob.text_q[0], prob.vis_k[0], prob.pos3d[0], prob.probe, prob.k, outs[0],
                  prob.workload.dtype, O.GmcParams(), app_proj=prob.app_proj)
