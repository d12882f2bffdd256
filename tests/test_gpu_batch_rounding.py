"""A sample in a batch against the same sample alone.  The tiles that share a k range and the runs of a cut attention are
chosen by the rows and heads of the whole call, so below the sizes at which one sample fills the GPU the sums are grouped
differently: the results agree to the rounding of the stored activations.  From those sizes on they agree bit for bit."""
import numpy as np
import pytest

from gpu_helpers import gpu_blocks, host_inputs
from oracle.numerics import storage_to_f64
from paper_2607_02829_amd import inputs

pytestmark = pytest.mark.gpu


def _both(B, S, D, H, F, dtype, kind):
    w = inputs.small(name="batch", dtype=dtype, B=B, Hg=1, Wg=S, D=D, H=H, F=F, kind=kind)
    h, params, cond, dh = host_inputs(w, 1, S=S)
    batch = gpu_blocks(w, S, h, params, cond, dh)
    one = lambda b: gpu_blocks(w.with_(B=1), S, h[b:b + 1], params, None if cond is None else cond[b:b + 1], dh[b:b + 1])
    return batch, [one(b) for b in (0, B - 1)]


@pytest.mark.parametrize("B,S,D,H,F,dtype,kind", [
    (8, 128, 1024, 16, 4096, "bf16", "preln"),    # 32 x 32 tiles in eight groups alone, 64 x 64 in two in the batch
    (6, 200, 256, 4, 1024, "bf16", "adaln"),
    (4, 1030, 128, 2, 512, "bf16", "preln"),      # two runs in both, other tiles
    (8, 2100, 128, 4, 512, "bf16", "preln"),      # head dim 32, four runs alone, none in the batch
    (6, 2050, 256, 4, 1024, "bf16", "preln"),     # head dim 64, four runs alone, none in the batch
    (8, 120, 256, 4, 1024, "f32", "preln"),
])
def test_to_rounding(B, S, D, H, F, dtype, kind):
    print(f"[batch] B={B} S={S} D={D} H={H} {dtype} {kind}", flush=True)
    batch, alone = _both(B, S, D, H, F, dtype, kind)
    # each side rounds the block's stored activations to 2^-9 (bf16), in norm 2^-9 / sqrt(3) a time, some eight times on
    # the way to an output; the two sides' roundings are independent at worst.  fp32: sums of up to 4096 products, as
    # against the oracle
    tol = 2.0 ** -9 * np.sqrt(2 * 8 / 3) if dtype == "bf16" else 4e-6
    for got, b in zip(alone, (0, B - 1)):
        for n in ("h_out", "dh_in"):
            x, y = storage_to_f64(batch[n][b]), storage_to_f64(got[n][0])
            err = np.linalg.norm(x - y) / np.linalg.norm(y)
            print(f"[batch] sample {b} {n}: {err:.1e}", flush=True)
            assert err <= tol, (b, n, err)


@pytest.mark.parametrize("B,S,D,H", [
    (2, 2049, 1024, 16),   # more than 256 tiles of 64 x 64 and more than 128 workgroups of 256 rows in one sample
    (3, 1089, 1024, 8),    # head dim 128: never cut
    (2, 4161, 256, 8),     # head dim 32, more than 256 workgroups of 128 rows
])
def test_bit_for_bit(B, S, D, H):
    print(f"[batch] bits B={B} S={S} D={D} H={H}", flush=True)
    batch, alone = _both(B, S, D, H, 4 * D, "bf16", "preln")
    for got, b in zip(alone, (0, B - 1)):
        for n in ("h_out", "dh_in"):
            assert np.array_equal(batch[n][b], got[n][0]), (b, n)
