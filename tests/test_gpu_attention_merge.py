"""Merge of the query attention's key chunks on both sides of every count at which it takes more groups of threads or
requests (2, 4, 8, 16, 32 and 64 chunks), a ragged last chunk, fewer rows than a workgroup holds, both head dimensions;
chunks with infinite outputs and without mass."""
import numpy as np
import pytest

from tests import test_gpu_attention_edges as E

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,hq,hkv,lq,m", [
    ("bf16", 128, 8, 1, 1, 2048), ("bf16", 128, 8, 1, 1, 2049), ("bf16", 128, 8, 1, 1, 16384), ("bf16", 128, 3, 1, 1, 5000),
    ("bf16", 128, 8, 1, 1, 512), ("f32", 64, 8, 1, 1, 513), ("bf16", 64, 8, 1, 1, 1024), ("bf16", 128, 8, 1, 1, 1025),
    ("bf16", 128, 8, 1, 1, 4096), ("f32", 128, 8, 1, 1, 4097), ("bf16", 64, 8, 1, 1, 8192), ("bf16", 128, 8, 1, 1, 8193),
    ("bf16", 64, 8, 2, 3, 2100), ("bf16", 64, 1, 1, 1, 16001), ("f32", 128, 2, 1, 1, 9000), ("f32", 64, 5, 5, 1, 2400),
])
def test_many_key_chunks(dtype, d, hq, hkv, lq, m):
    E.test_query_attention_shapes(dtype, d, hq, hkv, lq, m)


@pytest.mark.parametrize("d,hq,m", [(64, 1, 2400), (128, 2, 9100), (128, 1, 700)])
def test_infinite_value(d, hq, m):
    """float32, one value of the last, ragged chunk is infinite: its channel comes out infinite, every other one as ever."""
    import torch
    from paper_2508_11661_amd import samkv as S
    q, k, v = E._data(m, "f32", hq, 1, 1, m, d)
    v[0, m - 70, 5] = np.inf
    out = torch.full((hq, 1, d), float("nan"), device="cuda")
    lse = torch.full((hq, 1), float("nan"), device="cuda")
    ws = torch.empty((S.samkv_workspace_bytes(1, hq, 1, d, 1, m),), dtype=torch.uint8, device="cuda")
    S.samkv_query_attn(E.H.to_dev(q, "f32"), E.H.to_dev(k, "f32"), E.H.to_dev(v, "f32"), d ** -0.5, out, lse, ws)
    assert torch.isposinf(out[:, :, 5]).all()
    v[0, m - 70, 5] = 0
    o_ref, l_ref = E.O.attention(q, k, v, d ** -0.5, False)
    o_ref[:, :, 5] = 0
    out[:, :, 5] = 0
    E.H.check_attention(out.cpu().numpy(), lse.cpu().numpy(), o_ref, l_ref, "f32", "infinite value")


@pytest.mark.parametrize("dtype,d,chunks", [("f32", 64, (0, 2, 4, 6, 8)), ("f32", 128, (3,)), ("f32", 128, range(1, 10)),
                                            ("bf16", 128, (0, 2, 4, 6, 8)), ("bf16", 64, range(0, 9))])
def test_chunks_without_mass(dtype, d, chunks):
    """Every score of some of the ten chunks of 256 keys is -inf (a product beyond float32): they do not count, in the
    output and in the log-sum-exp, whichever group of threads they belong to."""
    import torch
    from paper_2508_11661_amd import samkv as S
    m = 2400
    q, k, v = E._data(d, dtype, 1, 1, 1, m, d)
    q[..., 0], k[..., 0] = 4.0, 0.0
    for c in chunks:
        k[0, 256 * c:256 * (c + 1), 0] = np.float32(-2.0 ** 127)
    out = torch.full((1, 1, d), float("nan"), device="cuda")
    lse = torch.full((1, 1), float("nan"), device="cuda")
    ws = torch.empty((S.samkv_workspace_bytes(1, 1, 1, d, 1, m),), dtype=torch.uint8, device="cuda")
    S.samkv_query_attn(E.H.to_dev(q, dtype), E.H.to_dev(k, dtype), E.H.to_dev(v, dtype), d ** -0.5, out, lse, ws)
    o_ref, l_ref = E.O.attention(q, k, v, d ** -0.5, False)
    E.H.check_attention(out.cpu().numpy(), lse.cpu().numpy(), o_ref, l_ref, dtype, "chunks without mass")
