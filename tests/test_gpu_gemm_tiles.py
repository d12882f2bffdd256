"""bf16 blocks at the sizes where the GEMMs change their tile: 32 x 32 tiles with the k loop shared by
eight groups, 32 x 64 with four, 64 x 64 with two, 64 x 128, and 128 x 128 at one and two workgroups per
CU, ragged in the token count, with k ranges that the groups do not share evenly; outputs and every
gradient against the fp64 oracle, pre-LN and adaLN."""
import pytest

from gpu_helpers import check_pairs, gpu_blocks, host_inputs, oracle_blocks, pairs
from paper_2607_02829_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,S,D,H,F,kind", [
    (1, 1, 64, 1, 64, "preln"),        # one k-tile for eight groups
    (1, 33, 192, 3, 768, "adaln"),     # three and twelve k-tiles, a second tile row of one row
    (3, 43, 320, 5, 1280, "preln"),    # five k-tiles; 32 x 32 and 32 x 64
    (1, 257, 1024, 16, 4096, "preln"),   # 32 x 64 and 64 x 128
    (2, 507, 1024, 16, 4096, "adaln"),   # 64 x 64 and 128 x 128 at one per CU
    (1, 2049, 640, 10, 2560, "preln"),   # 64 x 128, 128 x 128 at one and at two per CU
])
def test_blocks_across_tile_shapes(B, S, D, H, F, kind):
    print(f"[gemm tiles] B={B} S={S} D={D} F={F} {kind}", flush=True)
    w = inputs.small(name="tiles", B=B, Hg=1, Wg=S, D=D, H=H, F=F, kind=kind)
    h, params, cond, dh = host_inputs(w, 1, S=S)
    got = gpu_blocks(w, S, h, params, cond, dh)
    check_pairs(pairs(got, oracle_blocks(w, h, params, cond, dh), kind), "bf16", "[gemm tiles]")
