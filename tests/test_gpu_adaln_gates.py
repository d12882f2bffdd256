"""adaLN blocks at the edges of the conditioning kernels: more samples than one pass over a weight takes,
token counts around the 64-row chunks of the gate gradients, widths that leave lanes of a 256-column block
idle; outputs and every gradient against the fp64 oracle."""
import pytest

from gpu_helpers import check_pairs, gpu_blocks, host_inputs, oracle_blocks, pairs
from paper_2607_02829_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,S,D", [(1, 64, 64), (9, 65, 192), (17, 3, 320), (8, 129, 256)])
def test_adaln_edges(B, S, D, dtype):
    print(f"[adaln] B={B} S={S} D={D} {dtype}", flush=True)
    w = inputs.small(name="gates", dtype=dtype, B=B, Hg=1, Wg=S, D=D, H=D // 64, F=2 * D, kind="adaln")
    h, params, cond, dh = host_inputs(w, 1, S=S)
    got = gpu_blocks(w, S, h, params, cond, dh)
    check_pairs(pairs(got, oracle_blocks(w, h, params, cond, dh), "adaln"), dtype, "[adaln]")
