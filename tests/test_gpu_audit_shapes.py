"""GPU parity of the realisation audit at the edges of its tiles: head
dimensions off the common ones, fewer keys than a tile, one carrier, one
query, more client rows than a mass block, carriers without members, tensors
that start at any element."""
import numpy as np
import pytest

from oracle import gmc_oracle as O
from paper_2608_02134_amd.binding import Pruner, to_device

from .test_gpu_audit import REL_TOL, VEC_TOL, _inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

CASES = {
    "one_carrier": dict(dtype="bf16", n=5, k=1, t=1, hq=4, hkv=2, dh=96),
    "tile_edges": dict(dtype="bf16", n=128, k=16, t=16, hq=2, hkv=2, dh=160),
    "past_tile_edges": dict(dtype="bf16", n=129, k=17, t=17, hq=3, hkv=1, dh=192),
    "wide_fp32": dict(dtype="f32", n=70, k=33, t=5, hq=2, hkv=1, dh=256),
    "wide_bf16": dict(dtype="bf16", n=70, k=33, t=5, hq=2, hkv=1, dh=224),
    "two_list_passes": dict(dtype="bf16", n=2100, k=9, t=3, hq=2, hkv=1, dh=32),
    "many_rows": dict(dtype="f32", n=40, k=8, t=90, hq=16, hkv=4, dh=32),   # 1440 client rows
}


def _offset(a):
    """The same values in a tensor that starts one element past an allocation."""
    buf = torch.empty(a.numel() + 1, dtype=a.dtype, device=a.device)
    out = buf[1:].view(a.shape)
    out.copy_(a)
    return out


@pytest.mark.parametrize("case", list(CASES))
@pytest.mark.parametrize("shift", [False, True], ids=["aligned", "any_element"])
def test_audit_shapes(case, shift):
    c = CASES[case]
    print(f"\n[case] audit {case} shift={shift}: {c}", flush=True)
    q, kf, vf, kc, vc, carrier, w, nv = _inputs(11, **c, nonvis=True, weights=True)
    tdt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    probe = torch.zeros((c["hq"], 4, 64), dtype=tdt, device="cuda")
    # the scratch is the client matrices' room: three problems' worth
    pr = Pruner(d=64, n_q_heads=c["hq"], n_kv_heads=c["hkv"], head_dim=c["dh"], probe=probe, dtype=tdt,
                max_batch=3, max_n=c["n"], max_t=c["t"])
    try:
        dev = lambda a: (_offset if shift else (lambda x: x))(to_device(a, c["dtype"], torch))
        out, rows, vec = pr.audit(dev(q), dev(kf), dev(vf), dev(kc), dev(vc), torch.from_numpy(carrier).cuda(),
                                  torch.from_numpy(w).cuda(), torch.from_numpy(nv).cuda(), rows=True, vectors=True)
        torch.cuda.synchronize()
        out, rows, vec = out.cpu().numpy()[0], rows.cpu().numpy()[0], vec.cpu().numpy()[0]
    finally:
        pr.close()
    ref = O.message_audit(q[0], kf[0], vf[0], kc[0], vc[0], carrier[0], w[0], nv[0])
    r = ref["rows"]
    scale = np.max(np.abs(r["y"]), axis=2, keepdims=True)
    for i, key in enumerate(("y", "yc", "term1", "term2")):
        assert np.max(np.abs(vec[:, :, i, :] - r[key]) / scale) <= VEC_TOL, key
    np.testing.assert_allclose(rows[:, :, 6], r["l1"], rtol=REL_TOL, atol=1e-6)
    np.testing.assert_allclose(rows[:, :, 7], r["bound"], rtol=REL_TOL, atol=1e-5)
    for i, key in enumerate(("e_m", "alpha", "kappa", "norm_y", "norm_yc", "norm_diff")):
        assert out[i] == pytest.approx(ref[key], rel=REL_TOL, abs=1e-6), key


def test_carrier_without_members():
    """Its grouped mass is 0 and its clients' bound infinite; nothing else changes."""
    c = dict(dtype="bf16", n=60, k=12, t=4, hq=2, hkv=1, dh=64)
    q, kf, vf, kc, vc, carrier, w, nv = _inputs(3, **c, nonvis=False, weights=False)
    carrier[carrier == 7] = 3
    probe = torch.zeros((2, 4, 64), dtype=torch.bfloat16, device="cuda")
    pr = Pruner(d=64, n_q_heads=2, n_kv_heads=1, head_dim=64, probe=probe, dtype=torch.bfloat16, max_batch=3, max_n=60,
                max_t=4)
    try:
        dev = lambda a: to_device(a, "bf16", torch)
        out, rows, _ = pr.audit(dev(q), dev(kf), dev(vf), dev(kc), dev(vc), torch.from_numpy(carrier).cuda(), rows=True)
        rows, out = rows.cpu().numpy()[0], out.cpu().numpy()[0]
    finally:
        pr.close()
    ref = O.message_audit(q[0], kf[0], vf[0], kc[0], vc[0], carrier[0], None, None)
    assert np.all(np.isinf(rows[:, :, 7])) and np.all(np.isinf(ref["rows"]["bound"]))
    np.testing.assert_allclose(rows[:, :, 6], ref["rows"]["l1"], rtol=REL_TOL, atol=1e-6)
    assert out[0] == pytest.approx(ref["e_m"], rel=REL_TOL)
