"""fp32 blocks at the sizes where the fp32 GEMMs change their tile: 32 x 32 tiles with the k loop shared
by eight waves (few outputs), 64 x 64, and 128 x 128 tiles, each ragged in the token count; outputs and
every gradient against the fp64 oracle, pre-LN and adaLN."""
import pytest

from gpu_helpers import compare, gpu_blocks, host_inputs, oracle_blocks
from paper_2607_02829_amd import inputs

pytestmark = pytest.mark.gpu

# (B, S, D, H, F, kind): rows B*S; the widest output F decides whether 64 x 64 or 128 x 128 tiles are used
CASES = [(1, 1, 64, 1, 64, "preln"), (1, 33, 64, 2, 256, "preln"), (3, 65, 192, 3, 768, "adaln"),
         (2, 513, 256, 4, 1024, "preln"), (1, 1031, 320, 5, 1024, "preln"), (2, 1000, 1024, 16, 4096, "preln")]


@pytest.mark.parametrize("B,S,D,H,F,kind", CASES)
def test_f32_blocks_across_tile_shapes(B, S, D, H, F, kind):
    print(f"[f32 blocks] B={B} S={S} D={D} F={F} {kind}", flush=True)
    w = inputs.small(name="f32t", dtype="f32", B=B, Hg=1, Wg=S, D=D, H=H, F=F, kind=kind)
    h, params, cond, dh = host_inputs(w, 1, S=S)
    errs = compare(gpu_blocks(w, S, h, params, cond, dh), oracle_blocks(w, h, params, cond, dh), "f32", kind)
    print(f"[f32 blocks] worst {max(errs.values()):.2e} ({max(errs, key=errs.get)})", flush=True)
    # sums of up to 4096 fp32 products, errors growing with the square root of the count: 64 x 6e-8
    bad = {k: v for k, v in errs.items() if not v <= 4e-6}
    assert not bad, bad
