"""Weight and bias gradients at the sizes where their tile and their split over tokens change: 64 x 128 tiles
in several runs, one round of 128 x 128 where 64 x 128 would need two, and, over many tokens, 128 x 128 tiles in
runs at one and two workgroups per CU, the last run short and ragged; against the fp64 oracle and
against the gradients of each sample alone, and bitwise repeatable."""
import numpy as np
import pytest
import torch

from gpu_helpers import check_pairs, gpu_blocks, host_inputs, oracle_blocks, pairs
from paper_2607_02829_amd import abi, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,D,F", [(700, 768, 3072), (8191, 64, 128), (8200, 128, 256)])
def test_block_against_oracle(S, D, F):
    print(f"[dW] S={S} D={D} F={F}", flush=True)
    w = inputs.small(name="dw", B=1, Hg=1, Wg=S, D=D, H=D // 64, F=F)
    h, params, cond, dh = host_inputs(w, 1, S=S)
    check_pairs(pairs(gpu_blocks(w, S, h, params, cond, dh), oracle_blocks(w, h, params, cond, dh)), "bf16", "[dW]")


@pytest.mark.parametrize("B,S,D,F", [(4, 2081, 1024, 4096), (3, 2731, 768, 3072), (5, 2100, 1024, 2048)])
def test_many_tokens(B, S, D, F):
    # attention stays within a sample, so the batch's gradients are the sums of those of its samples run alone:
    # fp32 sums of the same bf16 products, grouped differently, 2^-24 sqrt(tokens) of the norm, times 8.  The
    # activations are the same bit for bit as long as one sample's products sum their k range in the order of the
    # batch's (S > 2048 at these widths: no tile with groups).
    print(f"[dW] B={B} S={S} D={D} F={F}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(5)

    def normal(*shape, std=1.0):
        return (torch.randn(shape, generator=gen, device="cuda") * std).to(torch.bfloat16)

    shapes = {"ln1_w": (D,), "ln1_b": (D,), "w_qkv": (3 * D, D), "b_qkv": (3 * D,), "w_o": (D, D), "b_o": (D,),
              "ln2_w": (D,), "ln2_b": (D,), "w_fc1": (F, D), "b_fc1": (F,), "w_fc2": (D, F), "b_fc2": (D,)}
    params = {n: normal(*s, std=0.02 if n.startswith("w") else 0.5) for n, s in shapes.items()}
    x, dh = normal(B, S, D), normal(B, S, D)
    p = (abi.SrBlockParams * 1)()
    for n in abi.PARAM_FIELDS:
        setattr(p[0], n, params[n].data_ptr() if n in params else None)

    def step(b0, nb):
        cfg = abi.SrConfig(B=nb, L=S, D=D, H=D // 64, F=F, n_blocks=1, dtype=abi.SR_BF16, kind=abi.SR_BLOCK_PRELN,
                           ln_eps=1e-6, idx_shared=0)
        sb, cb = abi.sr_workspace_bytes(cfg, S)
        saved, scratch = (torch.empty(n, dtype=torch.uint8, device="cuda") for n in (sb, cb))
        grads = {n: torch.full(s, float("nan"), device="cuda") for n, s in shapes.items()}
        gr = (abi.SrBlockGrads * 1)()
        for n in abi.PARAM_FIELDS:
            setattr(gr[0], n, grads[n].data_ptr() if n in grads else None)
        h, dx = torch.empty((nb, S, D), dtype=torch.bfloat16, device="cuda"), torch.empty_like(dh[b0:b0 + nb])
        abi.sr_sparse_blocks_fwd(cfg, S, p, None, x[b0:b0 + nb], h, saved)
        abi.sr_sparse_blocks_bwd(cfg, S, p, None, saved, dh[b0:b0 + nb], dx, gr, None, scratch)
        torch.cuda.synchronize()
        return grads

    got, again = step(0, B), step(0, B)
    parts = [step(b, 1) for b in range(B)]
    for n in shapes:
        assert torch.equal(got[n], again[n]), n
        want = sum(q[n].double() for q in parts)
        err = float((got[n].double() - want).norm() / want.norm())
        print(f"[dW] {n} {err:.1e}", flush=True)
        assert err <= 8 * 2.0 ** -24 * np.sqrt(B * S), n
