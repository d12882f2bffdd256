"""Blocks at every row length the LayerNorm kernels treat differently (one, two and four columns per lane
group; an exact and an open number of groups per lane), with row counts that leave a workgroup's last rows
out; outputs and every gradient against the fp64 oracle."""
import pytest

from gpu_helpers import check_pairs, gpu_blocks, host_inputs, oracle_blocks, pairs
from paper_2607_02829_amd import inputs

pytestmark = pytest.mark.gpu


WIDTHS = [64, 128, 192, 256, 320, 384, 512, 640, 768, 1280, 2048]


def _run(D, B, S, kind, dtype):
    print(f"[ln widths] D={D} {kind} {dtype}", flush=True)
    w = inputs.small(name="widths", dtype=dtype, B=B, Hg=1, Wg=S, D=D, H=D // 64, F=2 * D, kind=kind)
    h, params, cond, dh = host_inputs(w, 1, S=S)
    return pairs(gpu_blocks(w, S, h, params, cond, dh), oracle_blocks(w, h, params, cond, dh), kind)


@pytest.mark.parametrize("kind", ["preln", "adaln"])
@pytest.mark.parametrize("D", WIDTHS)
def test_block_widths_f32(D, kind):
    check_pairs(_run(D, 1 if kind == "preln" else 2, 21 if kind == "preln" else 9, kind, "f32"), "f32", "[ln widths]")


@pytest.mark.parametrize("D", WIDTHS)
def test_block_widths_bf16(D):
    # ln1's gradients are left to fp32: over 21 tokens attention is nearly uniform, so du1 is nearly one
    # vector v for all rows and dW_ln1 = sum_s du1 * xhat ~ v * sum_s xhat cancels (the rows' mean is zero);
    # rounding du1 to 2^-9 per row is then up to 2^-9 * sum|xhat| / |sum xhat| of the result
    items = [p for p in _run(D, 1, 21, "preln", "bf16") if not p[0].endswith(("ln1_w", "ln1_b"))]
    check_pairs(items, "bf16", "[ln widths]")
