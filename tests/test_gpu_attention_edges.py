"""The attention kernels of bf16 heads of 32 and of fp32 storage at the sizes where their tiles can
go wrong, through sr_cross_attention_fwd / _bwd: one row, one past a 32-row unit, a 64-row tile and
a 128-row workgroup, ragged on both sides; against the oracle's attention in fp64.  A non-finite
sample leaves its neighbours' bits alone (ragged tiles read past a sample's rows)."""
import numpy as np
import pytest

from oracle import block as oblk
from oracle.numerics import storage_to_f64
from test_gpu_cross_attention import _data, _gpu

pytestmark = pytest.mark.gpu

SIZES = [(1, 1, 1), (2, 33, 65), (2, 65, 33), (3, 129, 64), (1, 64, 129), (2, 128, 300), (2, 200, 1)]
# bf16: one rounding of each result, half a unit in the last of 8 bits: 2^-8 = 3.9e-3 of its value; dq
# and dk once more through Delta = rowsum(dO O) of the rounded O; fp32: sums of a few hundred products
TOL = {"bf16": {"O": 4e-3, "lse": 1e-5, "dq": 8e-3, "dk": 8e-3, "dv": 4e-3},
       "f32": {"O": 2e-6, "lse": 2e-6, "dq": 5e-6, "dk": 5e-6, "dv": 2e-6}}


@pytest.mark.parametrize("dtype,H", [("bf16", 8), ("f32", 8), ("f32", 4), ("f32", 2)])
@pytest.mark.parametrize("B,Sq,Skv", SIZES)
def test_attention_edges(B, Sq, Skv, H, dtype):
    D = 256
    print(f"[edges] B={B} Sq={Sq} Skv={Skv} H={H} {dtype}", flush=True)
    q, kv, dO = _data(B, Sq, Skv, D, dtype, 5)
    O, lse, dq, dkv = _gpu(B, Sq, Skv, D, H, dtype, q, kv, dO)
    q64, kv64, dO64 = storage_to_f64(q), storage_to_f64(kv), storage_to_f64(dO)
    qh, kh, vh = (oblk.split_heads(t, H) for t in (q64, kv64[..., :D], kv64[..., D:]))
    s = np.einsum("bhid,bhjd->bhij", qh, kh) / np.sqrt(D // H)
    m = s.max(-1)
    ref = {"O": oblk.merge_heads(oblk.attention_fwd(qh, kh, vh)),
           "lse": (m + np.log(np.exp(s - m[..., None]).sum(-1))) / np.log(2.0)}
    ref["dq"], ref["dk"], ref["dv"] = (oblk.merge_heads(t) for t in
                                       oblk.attention_bwd(qh, kh, vh, oblk.split_heads(dO64, H)))
    got = {"O": storage_to_f64(O), "lse": lse, "dq": storage_to_f64(dq), "dk": storage_to_f64(dkv)[..., :D],
           "dv": storage_to_f64(dkv)[..., D:]}
    # one key: P = 1, so dq = dk = 0 exactly and Delta - dP is rounding alone; scale by dO . v
    scale = {k: max(np.abs(r).max(), np.abs(dO64).max() if k in ("dq", "dk") and Skv == 1 else 0.0)
             for k, r in ref.items()}
    errs = {k: float(np.abs(got[k] - ref[k]).max() / scale[k]) for k in ref}
    print(f"[edges] errors {errs}", flush=True)
    bad = {k: v for k, v in errs.items() if not v <= TOL[dtype][k]}
    assert not bad, bad


@pytest.mark.parametrize("dtype,H", [("bf16", 8), ("f32", 8), ("f32", 4), ("f32", 2)])
def test_attention_neighbour_not_finite(dtype, H):
    B, Sq, Skv, D = 3, 45, 77, 256
    q, kv, dO = _data(B, Sq, Skv, D, dtype, 6)
    clean = _gpu(B, Sq, Skv, D, H, dtype, q, kv, dO)
    nan = np.float32(np.nan) if dtype == "f32" else np.uint16(0x7FC0)
    q2, kv2, dO2 = q.copy(), kv.copy(), dO.copy()
    for t in (q2, kv2, dO2):
        t[1] = nan
    got = _gpu(B, Sq, Skv, D, H, dtype, q2, kv2, dO2)
    for a, b in zip(clean, got):
        assert np.array_equal(a[[0, 2]], b[[0, 2]])
