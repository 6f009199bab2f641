"""Float32 attention at the edges of its one kernel: a workgroup holds 32 query rows and four waves, wave w takes the key
tiles w, w + 4, ... of 32 keys, so the edges are 32 keys (a wave's tile), 128 (one step of all four; waves beyond the keys
hold none), 256 (the shortest key chunk of a query problem; a last chunk may hold one key) and 32 rows."""
import pytest

from tests import test_gpu_attention_edges as E

pytestmark = pytest.mark.gpu

EDGES = [31, 32, 33, 95, 96, 97, 127, 128, 129, 255, 256, 257]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("m", EDGES)
def test_recompute_edges(d, m):
    """Causal: m rows against m keys, so the rows leave the same remainders (31, none and 1 of a tile) as the keys."""
    E.test_recompute_attention_shapes("f32", d, 4, 2, m)


@pytest.mark.parametrize("d,hq,hkv,m", [
    (128, 8, 8, 1), (128, 8, 2, 33), (64, 8, 2, 128), (128, 6, 3, 129), (64, 24, 24, 257),              # few row tiles
    (128, 512, 8, 64), (128, 256, 16, 65), (64, 512, 8, 1), (64, 64, 8, 513), (128, 104, 13, 300),      # many
])
def test_recompute(d, hq, hkv, m):
    E.test_recompute_attention_shapes("f32", d, hq, hkv, m)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("rows", [1, 31, 33])
@pytest.mark.parametrize("m", EDGES + [289, 512, 513, 545])
def test_query_edges(d, rows, m):
    """One head, so the keys are cut into chunks of 256: 257, 289, 513 and 545 keys leave last chunks of 1 and 33."""
    E.test_query_attention_shapes("f32", d, 1, 1, rows, m)


@pytest.mark.parametrize("d,hq,hkv,lq,m", [
    (128, 8, 8, 1, 1), (64, 8, 1, 4, 127), (128, 16, 2, 4, 513), (128, 7, 1, 5, 2049),   # one row tile, full or not; two
    (64, 16, 4, 16, 64), (128, 8, 2, 16, 257), (64, 32, 8, 33, 1300),                    # two and more row tiles per KV head
])
def test_query(d, hq, hkv, lq, m):
    E.test_query_attention_shapes("f32", d, hq, hkv, lq, m)


@pytest.mark.parametrize("d,hq,hkv,lq,m", [
    (64, 8, 2, 3, 97), (128, 8, 2, 8, 600), (128, 16, 16, 40, 700),      # query keys in one chunk, and in several
    (64, 96, 8, 2, 400), (128, 80, 8, 6, 450),                           # more causal workgroups than are resident
    (64, 4, 2, 16, 129), (128, 4, 2, 15, 257),                           # a last key tile, and a last chunk, of one key
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
