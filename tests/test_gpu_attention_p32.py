"""At head dim 32 (bf16 storage) the probabilities P and the score gradients dS enter their products with all 24
bits of fp32.  Each result below is a sum of two nearly cancelling parts, sixteen terms of weight P_A against
sixteen of weight w P_B, so that it is 2^-11 of its parts and a relative error of 2^-18 in P shows as 2^-7."""
import numpy as np
import pytest

from oracle.numerics import storage_to_f64
from paper_2607_02829_amd import inputs
from test_gpu_cross_attention import _gpu

pytestmark = pytest.mark.gpu

HD = 32
B = 48
# One rounding of the result to 8 bits, 2^-9; and the fp32 errors of the two parts: each exponential's argument (up to
# 2.6) rounds by 2^-23 ln 2, its scale factor by 2^-24 of it, the exponential by 2^-23, the part's sum by 2^-24:
# 2.7 x 2^-23 a part, 5.4 x 2^-23 of both, magnified by at most 2^11.5: 2^-9.
TOL = 2.0 ** -8


def _bf16(x):
    return storage_to_f64(inputs.to_storage(np.asarray(x, np.float32), "bf16"))


def _pairs(weight):
    """B triples (a, b, w) of bf16 values whose weight(a) - w weight(b) is 2^-11.5 .. 2^-10.5 of weight(a)."""
    rng = np.random.default_rng(3)
    out = []
    while len(out) < B:
        a, b = _bf16(rng.uniform(-10.0, -2.0, 2))
        w = float(_bf16([weight(a) / weight(b)])[0])
        d = abs(1.0 - w * weight(b) / weight(a))
        if 2.0 ** -11.5 <= d <= 2.0 ** -10.5:
            out.append((a, b, w))
    return out


def _check(name, got, ref):
    err = np.abs(got - ref) / np.abs(ref)
    print(f"[p32] {name}: largest relative error {err.max():.2e}", flush=True)
    assert err.max() <= TOL, (name, err)


def test_sums_over_keys():
    # one query, keys: two of score 0, sixteen of score a, sixteen of score b
    pairs = _pairs(lambda a: np.exp(a / np.sqrt(HD)))
    q, kv, dO = np.zeros((B, 1, 64)), np.zeros((B, 34, 128)), np.zeros((B, 1, 64))
    sign = np.where(np.arange(34) % 2, -1.0, 1.0)
    for i, (a, b, w) in enumerate(pairs):
        q[i, 0, 0] = 1.0
        kv[i, 2:18, 0], kv[i, 18:, 0] = a, b
        v = kv[i, :, 64:]
        v[2:18, 0], v[18:, 0] = 1.0, -w            # O[0] = sum of P over A - w times that over B
        v[:, 1], dO[i, 0, 1] = sign, 1.0           # dP = +-1, Delta = 0 but for rounding: dS = +-P
        kv[i, 2:18, 2], kv[i, 18:, 2] = sign[2:18], -w * sign[18:]   # dq[2] likewise, q[2] being 0
    st = [inputs.to_storage(t.astype(np.float32), "bf16") for t in (q, kv, dO)]
    O, lse, dq, _ = (storage_to_f64(t) if t.dtype == np.uint16 else t.astype(np.float64)
                     for t in _gpu(B, 1, 34, 64, 2, "bf16", *st))
    s = np.einsum("bid,bjd->bij", q[..., :HD], kv[..., :HD])[:, 0] / np.sqrt(HD)
    P = np.exp(s) / np.exp(s).sum(-1, keepdims=True)
    _check("O", O[:, 0, 0], np.einsum("bj,bj->b", P, kv[..., 64]))
    ds = P * (sign[None] - O[:, 0, 1][:, None])
    _check("dq", dq[:, 0, 2], np.einsum("bj,bj->b", ds, kv[..., 2]) / np.sqrt(HD))
    err = np.abs(lse[:, 0, 0] - np.log2(np.exp(s).sum(-1)))
    print(f"[p32] lse: largest error {err.max():.2e}", flush=True)
    # the denominator's sum and logarithm in fp32, values below 8: a few units of 2^-22
    assert err.max() <= 8e-7


def test_sums_over_queries():
    # keys: two of score a or b by the query, two of score 0; sixteen queries of each score
    pairs = _pairs(lambda a: 1.0 / (2.0 + 2.0 * np.exp(-a / np.sqrt(HD))))
    q, kv, dO = np.zeros((B, 32, 64)), np.zeros((B, 4, 128)), np.zeros((B, 32, 64))
    sign = np.array([1.0, -1.0, 1.0, -1.0])
    for i, (a, b, w) in enumerate(pairs):
        kv[i, :2, 0] = 1.0
        kv[i, :, 65] = sign
        q[i, :16, 0], q[i, 16:, 0] = a, b
        q[i, :16, 2], q[i, 16:, 2] = 1.0, -w       # dk[2], k[2] being 0
        dO[i, :16, 0], dO[i, 16:, 0] = 1.0, -w     # dv[0], v[0] being 0
        dO[i, :, 1] = 1.0
    st = [inputs.to_storage(t.astype(np.float32), "bf16") for t in (q, kv, dO)]
    O, _, _, dkv = (storage_to_f64(t) if t.dtype == np.uint16 else t for t in _gpu(B, 32, 4, 64, 2, "bf16", *st))
    s = np.einsum("bid,bjd->bij", q[..., :HD], kv[..., :HD]) / np.sqrt(HD)
    P = np.exp(s) / np.exp(s).sum(-1, keepdims=True)
    _check("dv", dkv[:, 0, 64], np.einsum("bi,bi->b", P[:, :, 0], dO[..., 0]))
    ds = P * (sign[None, None] - O[..., 1][..., None])
    _check("dk", dkv[:, 0, 2], np.einsum("bi,bi->b", ds[:, :, 0], q[..., 2]) / np.sqrt(HD))
