"""Token positions of the blocks that survive the cross-document filter, around the 16 blocks of a workgroup and the 1024 of
one scan: every block of one document, and a share of two documents' blocks, with a short last block; bit for bit."""
import numpy as np
import pytest

from oracle import samkv_oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("blocks,p", [([1], 1.0), ([16], 1.0), ([17], 1.0), ([1023], 1.0), ([1024], 1.0), ([1025], 1.0),
                                      ([3700], 1.0), ([40, 3], 0.5), ([2100, 2047], 0.9)])
def test_positions(blocks, p):
    import torch
    from paper_2508_11661_amd import samkv as S
    block, n_init, n_local, hkv = 4, 1, 1, 2
    lens = [block * n - n % 3 for n in blocks]
    rng = np.random.default_rng(sum(blocks))
    b32 = [rng.standard_normal((hkv, n)).astype(np.float32) for n in blocks]
    k = [torch.zeros((hkv, n, 64), dtype=torch.bfloat16, device="cuda") for n in lens]
    caches = S.Caches(k, None, hkv)
    share = [p] * len(lens)
    want = O.block_filter([b.astype(np.float64) for b in b32], lens, block, share, n_init, n_local)
    gidx = torch.full(want.shape, -1, dtype=torch.int32, device="cuda")
    ws = torch.empty(S.samkv_block_workspace_bytes(caches, block), dtype=torch.uint8, device="cuda")
    S.samkv_block_select_filter(torch.from_numpy(np.concatenate(b32, axis=1)).cuda(), caches, block, share, n_init, n_local,
                                gidx, ws)
    assert np.array_equal(gidx.cpu().numpy(), want)
