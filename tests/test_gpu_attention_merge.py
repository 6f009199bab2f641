"""Merge of the query attention's key chunks: 8 chunks (the last count that one thread per four channels walks alone), 9,
one batch of requests per group (64), a ragged last chunk, fewer rows than a workgroup holds, both head dimensions."""
import pytest

from tests import test_gpu_attention_edges as E

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,hq,hkv,lq,m", [
    ("bf16", 128, 8, 1, 1, 2048), ("bf16", 128, 8, 1, 1, 2049), ("bf16", 128, 8, 1, 1, 16384), ("bf16", 128, 3, 1, 1, 5000),
    ("bf16", 64, 8, 2, 3, 2100), ("bf16", 64, 1, 1, 1, 16001), ("f32", 128, 2, 1, 1, 9000), ("f32", 64, 5, 5, 1, 2400),
])
def test_many_key_chunks(dtype, d, hq, hkv, lq, m):
    E.test_query_attention_shapes(dtype, d, hq, hkv, lq, m)
