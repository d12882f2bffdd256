"""Self-attention whose streamed dimension is cut into runs (few heads): head dims 32 and 64, two, three
and four runs, token counts that leave the last run short and ragged, and the largest that stays uncut;
one block forward and backward against the fp64 oracle, and bitwise repeatable."""
import numpy as np
import pytest

from gpu_helpers import check_pairs, gpu_blocks, host_inputs, oracle_blocks, pairs
from paper_2607_02829_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,S,D,H", [
    (1, 1023, 64, 1),    # 16 tiles, just under: two runs
    (1, 1025, 128, 2),   # a 17th tile of one row
    (2, 1700, 64, 2),    # head dim 32, 27 tiles in three runs
    (1, 2100, 128, 4),   # head dim 32, four runs, the last one short
    (1, 2050, 256, 4),   # four runs, the last tile of two rows
    (1, 960, 128, 2),    # 15 tiles: uncut
])
def test_split_attention_block(B, S, D, H):
    print(f"[split] B={B} S={S} D={D} H={H}", flush=True)
    w = inputs.small(name="split", B=B, Hg=1, Wg=S, D=D, H=H, F=4 * D)
    h, params, cond, dh = host_inputs(w, 1, S=S)
    a = gpu_blocks(w, S, h, params, cond, dh)
    check_pairs(pairs(a, oracle_blocks(w, h, params, cond, dh)), "bf16", "[split]")
    b = gpu_blocks(w, S, h, params, cond, dh)
    assert np.array_equal(a["h_out"], b["h_out"]) and np.array_equal(a["dh_in"], b["dh_in"])
    assert all(np.array_equal(x[k], y[k], equal_nan=True) for x, y in zip(a["grads"], b["grads"]) for k in x)


# The forward's planes lie in the buffers of h1, z and GELU(z), so the MLP width decides how many runs it may have:
# one (uncut) at F = D, three at 2 D, four from 3 D; at F = 5 D / 4 and 11 D / 4 the plane that does not fit whole is
# left out.  The backward has four runs throughout.
@pytest.mark.parametrize("S,D,H", [(2050, 256, 4), (2100, 128, 4)])
@pytest.mark.parametrize("quarters", [4, 5, 8, 11, 12])
def test_split_by_mlp_width(S, D, H, quarters):
    F = D * quarters // 4 // 64 * 64
    print(f"[split] S={S} D={D} H={H} F={F}", flush=True)
    w = inputs.small(name="split", B=1, Hg=1, Wg=S, D=D, H=H, F=F)
    h, params, cond, dh = host_inputs(w, 1, S=S)
    a = gpu_blocks(w, S, h, params, cond, dh)
    check_pairs(pairs(a, oracle_blocks(w, h, params, cond, dh)), "bf16", "[split]")
