"""A non-finite sample leaves the bits of the samples before and after it alone, at every head dim: the last,
ragged tile of a sample reaches past its rows, into those of the next one.  Through the asymmetric attention, and
through blocks forward and backward, with attention whole and cut into runs."""
import numpy as np
import pytest

from gpu_helpers import gpu_blocks, host_inputs
from paper_2607_02829_amd import abi, device, inputs
from test_gpu_cross_attention import _data, _gpu

pytestmark = pytest.mark.gpu


def _bad(dtype, what):
    if dtype == "f32":
        return np.float32(np.nan if what == "nan" else np.inf)
    return np.uint16(0x7FC0 if what == "nan" else 0x7F80)


@pytest.mark.parametrize("what", ["nan", "inf"])
@pytest.mark.parametrize("H", [8, 4, 2])   # head dims 32, 64, 128
def test_cross_attention(H, what):
    B, Sq, Skv, D = 3, 45, 77, 256
    print(f"[isolation] cross H={H} {what}", flush=True)
    q, kv, dO = _data(B, Sq, Skv, D, "bf16", 6)
    clean = _gpu(B, Sq, Skv, D, H, "bf16", q, kv, dO)
    q2, kv2, dO2 = q.copy(), kv.copy(), dO.copy()
    for t in (q2, kv2, dO2):
        t[1] = _bad("bf16", what)
    got = _gpu(B, Sq, Skv, D, H, "bf16", q2, kv2, dO2)
    for n, a, b in zip(("O", "lse", "dq", "dkv"), clean, got):
        assert np.array_equal(a[0], b[0]), f"{n} of the sample before"
        assert np.array_equal(a[2], b[2]), f"{n} of the sample after"


@pytest.mark.parametrize("S,D,H,dtype,kind", [
    (45, 128, 4, "bf16", "preln"), (45, 128, 2, "bf16", "preln"), (45, 256, 2, "bf16", "preln"),
    (300, 128, 2, "bf16", "adaln"), (77, 128, 2, "f32", "preln"),
    (1030, 64, 1, "bf16", "preln"),    # head dim 64, two runs
    (1030, 64, 2, "bf16", "preln"),    # head dim 32, two runs
])
def test_blocks(S, D, H, dtype, kind):
    print(f"[isolation] blocks S={S} D={D} H={H} {dtype} {kind}", flush=True)
    w = inputs.small(name="iso", dtype=dtype, B=3, Hg=1, Wg=S, D=D, H=H, F=2 * D, kind=kind)
    h, params, cond, dh = host_inputs(w, 2, S=S)
    clean = gpu_blocks(w, S, h, params, cond, dh)
    bad = h.copy()
    bad[1, 0] = _bad(dtype, "nan")   # one token: attention spreads it over the sample
    got = gpu_blocks(w, S, bad, params, cond, dh)
    for n in ("h_out", "dh_in"):
        for b in (0, 2):
            assert np.array_equal(clean[n][b], got[n][b]), f"{n} of sample {b}"
    if clean["dcond"] is not None:
        assert np.array_equal(clean["dcond"][[0, 2]], got["dcond"][[0, 2]])


@pytest.mark.parametrize("S,D,H,dtype", [(45, 128, 2, "bf16"), (300, 128, 2, "bf16"), (45, 128, 4, "bf16"), (45, 128, 1, "f32")])
def test_column_sums(S, D, H, dtype):
    import torch
    print(f"[isolation] column sums S={S} D={D} H={H} {dtype}", flush=True)
    w = inputs.small(name="iso", dtype=dtype, B=3, Hg=1, Wg=S, D=D, H=H, F=2 * D, n_blocks=1)
    h, params, _, _ = host_inputs(w, 1, S=S)
    cfg = device.config_for(w, n_blocks=1)
    dp = device.DeviceParams(params, w.kind)

    def sums(x):
        saved, scratch = device.workspace(cfg, S)
        xd = device.to_device(x)
        out = torch.empty((3, H, S), dtype=torch.float32, device="cuda")
        abi.sr_dense_blocks_fwd(cfg, dp.array, None, xd, torch.empty_like(xd), saved, scratch)
        abi.sr_attention_colsums(cfg, S, saved, 0, out)
        torch.cuda.synchronize()
        return out.cpu().numpy()

    bad = h.copy()
    bad[1, 0] = _bad(dtype, "nan")
    clean, got = sums(h), sums(bad)
    assert np.isfinite(clean).all() and np.array_equal(clean[[0, 2]], got[[0, 2]])
