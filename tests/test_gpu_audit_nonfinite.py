"""Non-finite values in the realisation audit stay where they are: an infinity in
the last value row (tiles past it load nothing in its place) and NaN keys in the
first tile."""
import numpy as np
import pytest

from oracle import gmc_oracle as O
from paper_2608_02134_amd.binding import Pruner, to_device

from .test_gpu_audit import REL_TOL, VEC_TOL, _inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)


def _audit(c, q, kf, vf, kc, vc, carrier, nv):
    tdt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    probe = torch.zeros((c["hq"], 4, 64), dtype=tdt, device="cuda")
    pr = Pruner(d=64, n_q_heads=c["hq"], n_kv_heads=c["hkv"], head_dim=c["dh"], probe=probe, dtype=tdt, max_batch=3,
                max_n=c["n"], max_t=c["t"])
    try:
        dev = lambda a: to_device(a, c["dtype"], torch)
        _, rows, vec = pr.audit(dev(q), dev(kf), dev(vf), dev(kc), dev(vc), torch.from_numpy(carrier).cuda(), None,
                                None if nv is None else torch.from_numpy(nv).cuda(), rows=True, vectors=True)
        torch.cuda.synchronize()
        return rows.cpu().numpy()[0], vec.cpu().numpy()[0]
    finally:
        pr.close()


CASES = [dict(dtype="bf16", n=70, k=33, t=5, hq=2, hkv=1, dh=64), dict(dtype="bf16", n=35, k=17, t=3, hq=2, hkv=1, dh=224),
         dict(dtype="f32", n=70, k=33, t=5, hq=2, hkv=1, dh=128), dict(dtype="f32", n=50, k=20, t=5, hq=2, hkv=1, dh=256)]
IDS = [f"{c['dtype']}_{c['dh']}" for c in CASES]


@pytest.mark.parametrize("c", CASES, ids=IDS)
def test_infinite_value_in_the_last_row(c):
    print(f"\n[case] audit, infinite last values: {c}", flush=True)
    q, kf, vf, kc, vc, carrier, _, nv = _inputs(5, **c, nonvis=True, weights=False)
    ref = O.message_audit(q[0], kf[0], vf[0], kc[0], vc[0], carrier[0], None, nv[0])["rows"]
    vf[0, -1, :, 0], vc[0, -1, :, 0] = np.inf, -np.inf
    rows, vec = _audit(c, q, kf, vf, kc, vc, carrier, nv)
    assert np.all(np.isposinf(vec[:, :, 0, 0])) and np.all(np.isneginf(vec[:, :, 1, 0]))
    for i, key in enumerate(("y", "yc")):
        scale = np.max(np.abs(ref["y"]), axis=2, keepdims=True)
        assert np.max(np.abs(vec[:, :, i, 1:] - ref[key][:, :, 1:]) / scale) <= VEC_TOL, key
    assert np.all(np.isposinf(rows[:, :, 0])) and np.all(np.isposinf(rows[:, :, 1]))
    np.testing.assert_allclose(rows[:, :, 6], ref["l1"], rtol=REL_TOL, atol=1e-6)


@pytest.mark.parametrize("c", CASES, ids=IDS)
def test_nan_keys_in_the_first_tile(c):
    """They make the Full log-sum-exp NaN, and with it every Full message; no
    carrier's logarithm counts towards the bound."""
    print(f"\n[case] audit, NaN keys: {c}", flush=True)
    q, kf, vf, kc, vc, carrier, _, nv = _inputs(6, **c, nonvis=False, weights=False)
    kf[0, :4] = np.nan
    rows, vec = _audit(c, q, kf, vf, kc, vc, carrier, nv)
    assert np.all(np.isnan(vec[:, :, 0])) and np.all(np.isfinite(vec[:, :, 1]))
    assert np.all(np.isnan(rows[:, :, 6])) and np.all(rows[:, :, 7] == 0.0)
