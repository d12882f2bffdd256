"""Token selection at the sizes where a wave's run of tokens, a 64-token group or the cached keys end, and
top-k with scores that share their leading bits, tie in masses or are all equal; against the oracle, bit for
bit."""
import numpy as np
import pytest
import torch

from oracle import select as osel
from paper_2607_02829_amd import abi

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (63, 63), (64, 1), (65, 64), (1023, 500), (1024, 1024), (1025, 7), (2047, 1024), (16200, 4050),
         (19968, 5000), (19969, 19969)]


def _cfg(L, B=2):
    return abi.SrConfig(B=B, L=L, D=64, H=1, F=64, n_blocks=1, dtype=abi.SR_F32, kind=abi.SR_BLOCK_PRELN, ln_eps=1e-6,
                        idx_shared=0)


@pytest.mark.parametrize("L,K", SIZES)
def test_random(L, K):
    print(f"[select random] L={L} K={K}", flush=True)
    cfg = _cfg(L)
    idx = torch.empty((2, K), dtype=torch.int32, device="cuda")
    abi.sr_select_indices(cfg, K, abi.SR_SEL_RANDOM, 42, 3, None, None, idx, None)
    torch.cuda.synchronize()
    assert np.array_equal(idx.cpu().numpy(), osel.select_random(2, L, K, 42, 3))


@pytest.mark.parametrize("L,K", SIZES + [(32768, 8192), (32769, 100)])
@pytest.mark.parametrize("kind", ["equal", "few", "close", "extremes"])
def test_topk_planes(L, K, kind):
    print(f"[select topk] L={L} K={K} {kind}", flush=True)
    rng = np.random.default_rng(L + K)
    score = {"equal": np.full((2, 1, L), 3.0), "few": rng.integers(0, 3, (2, 1, L)),
             "close": 1.0 + rng.random((2, 1, L)) * 1e-3,
             "extremes": np.where(rng.random((2, 1, L)) < 0.5, 0.0, np.finfo(np.float32).max)}[kind].astype(np.float32)
    planes = torch.from_numpy(score).cuda()
    idx = torch.empty((2, K), dtype=torch.int32, device="cuda")
    abi.sr_select_topk_scores(_cfg(L), K, planes, 1, idx)
    torch.cuda.synchronize()
    assert np.array_equal(idx.cpu().numpy(), osel.select_topk_planes(score, K))


@pytest.mark.parametrize("L,K", [(638976, 159744), (638977, 160000), (1300001, 1299999)])
def test_random_in_segments(L, K):
    # keys not kept in LDS: their classes are, for 638976 tokens at a time
    test_random(L, K)


@pytest.mark.parametrize("L,K", [(32769, 8192), (524288, 131072), (524289, 400000), (1100003, 550000)])
@pytest.mark.parametrize("parts", [1, 5])
@pytest.mark.parametrize("kind", ["equal", "few", "random"])
def test_topk_planes_in_segments(L, K, parts, kind):
    # 524288 tokens at a time; ties on both sides of a segment's end
    print(f"[select topk segments] L={L} K={K} parts={parts} {kind}", flush=True)
    rng = np.random.default_rng(L + K)
    shape = (2, parts, L)
    score = {"equal": np.full(shape, 3.0, np.float32), "few": rng.integers(0, 3, shape).astype(np.float32),
             "random": rng.random(shape, dtype=np.float32)}[kind]
    planes = torch.from_numpy(score).cuda()
    idx = torch.empty((2, K), dtype=torch.int32, device="cuda")
    abi.sr_select_topk_scores(_cfg(L), K, planes, parts, idx)
    torch.cuda.synchronize()
    assert np.array_equal(idx.cpu().numpy(), osel.select_topk_planes(score, K))
