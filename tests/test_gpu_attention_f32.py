"""Float32 attention at the sizes where its kernels change shape: one and several steps of 64 or 128 keys, ragged last
steps and row tiles, both row-tile sizes of the causal problem (64 rows x two key groups from 512 row tiles on, 32 rows x
four below), query problems of up to 32 rows and more, key chunks with a merge, both head dimensions."""
import pytest

from tests import test_gpu_attention_edges as E

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,hq,hkv,m", [
    (128, 8, 8, 1), (128, 8, 2, 33), (64, 8, 2, 128), (128, 6, 3, 129), (64, 24, 24, 257),   # 32 rows x 4 key groups
    (128, 512, 8, 64), (128, 256, 16, 65), (64, 512, 8, 1), (64, 64, 8, 513), (128, 104, 13, 300),  # 64 rows x 2
])
def test_recompute(d, hq, hkv, m):
    E.test_recompute_attention_shapes("f32", d, hq, hkv, m)


@pytest.mark.parametrize("d,hq,hkv,lq,m", [
    (128, 8, 8, 1, 1), (64, 8, 1, 4, 127), (128, 16, 2, 4, 513), (128, 7, 1, 5, 2049),   # rows <= 32 and one beyond
    (64, 16, 4, 16, 64), (128, 8, 2, 16, 257), (64, 32, 8, 33, 1300),                   # 64-row tiles
])
def test_query(d, hq, hkv, lq, m):
    E.test_query_attention_shapes("f32", d, hq, hkv, lq, m)


@pytest.mark.parametrize("d,hq,hkv,lq,m", [
    (64, 8, 2, 3, 97), (128, 8, 2, 8, 600), (128, 16, 16, 40, 700),      # 32-row causal tiles, both query shapes
    (64, 96, 8, 2, 400), (128, 80, 8, 6, 450),                           # 64-row causal tiles, both query shapes
])
def test_both_in_one_call(d, hq, hkv, lq, m):
    E.test_both_attentions_in_one_call("f32", d, hq, hkv, lq, m)


@pytest.mark.parametrize("d,m", [(64, 5), (128, 100), (128, 200)])
def test_row_without_mass(d, m):
    """Every score of the row is -inf (a product beyond float32): its log-sum-exp is -inf, whichever waves hold keys."""
    import torch
    from paper_2508_11661_amd import samkv as S
    q, k, v = E._data(d, "f32", 1, 1, 1, m, d)
    q[..., 0], k[..., 0] = 4.0, -2.0 ** 127
    out, lse = torch.zeros((1, 1, d), device="cuda"), torch.zeros((1, 1), device="cuda")
    ws = torch.empty((S.samkv_workspace_bytes(1, 1, 1, d, 1, m),), dtype=torch.uint8, device="cuda")
    S.samkv_query_attn(E.H.to_dev(q, "f32"), E.H.to_dev(k, "f32"), E.H.to_dev(v, "f32"), d ** -0.5, out, lse, ws)
    assert torch.isneginf(lse).all()
