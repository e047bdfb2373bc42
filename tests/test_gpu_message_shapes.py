"""GPU parity of the grounded bank's head statistics against the fp64 oracle
(tolerances of tests/parity.py) at the edges of their load paths: query rows
that are and are not a multiple of four, at and beside the 64-column chunk,
and probe ranks from 1 to 8."""
import dataclasses

import numpy as np
import pytest

from oracle import gmc_oracle as O
from paper_2608_02134_amd import synth

from .gpu_run import run
from .parity import check_problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)


@pytest.mark.parametrize("t,r", [(1, 4), (3, 4), (4, 4), (5, 3), (63, 4), (64, 4), (65, 4), (66, 2), (68, 4), (68, 3),
                                 (127, 4), (129, 1), (132, 4), (68, 5), (66, 5), (64, 6), (132, 7), (63, 7), (68, 8),
                                 (65, 8)])
def test_head_statistics(t, r):
    prob = synth.make_problem("tiny", batch=2, grid=(1, 11, 13), t=t, k=40)
    hq, own, d = prob.probe.shape
    more = np.random.default_rng(7).standard_normal((hq, max(r - own, 0), d)).astype(np.float32) / np.sqrt(d)
    probe = np.concatenate([prob.probe, more.astype(prob.probe.dtype)], 1)[:, :r]
    prob = dataclasses.replace(prob, probe=np.ascontiguousarray(probe))
    w = prob.workload
    print(f"\n[case] head statistics: B={w.batch} N={w.n} T={t} r={r}", flush=True)
    outs, pr = run(prob, torch)
    pr.close()
    for b in range(w.batch):
        check_problem(prob.hidden[b], prob.text_q[b], prob.vis_k[b], prob.pos3d[b], prob.probe, prob.k, outs[b],
                      w.dtype, O.GmcParams())
