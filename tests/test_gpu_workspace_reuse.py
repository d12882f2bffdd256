"""One workspace, sized for the largest keep ratio, serves every smaller token count: forward and backward in
buffers sized for S = 8193 give the bits of the same call in buffers of its own size."""
import pytest
import torch

from paper_2607_02829_amd import abi, device, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S", [8192, 4050])
def test_smaller_call_in_a_larger_workspace(S):
    print(f"[workspace] S={S}", flush=True)
    w = inputs.small(name="ws", B=1, Hg=1, Wg=8193, D=256, H=4, F=1024, n_blocks=1)
    cfg = device.config_for(w)
    params = device.DeviceParams(inputs.params_to_storage(inputs.block_params(w), w.dtype), w.kind)
    gen = torch.Generator(device="cuda").manual_seed(1)
    x, dy = (torch.randn((1, S, w.D), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(2))

    def step(rows):
        saved, scratch = device.workspace(cfg, rows)
        h, dx, g = torch.empty_like(x), torch.empty_like(x), device.DeviceGrads(w, 1)
        abi.sr_sparse_blocks_fwd(cfg, S, params.array, None, x, h, saved, scratch)
        abi.sr_sparse_blocks_bwd(cfg, S, params.array, None, saved, dy, dx, g.array, None, scratch)
        torch.cuda.synchronize()
        return [h, dx, *g.tensors[0].values()]

    for a, b in zip(step(8193), step(S)):
        assert torch.equal(a, b)
