"""Query attention with the query tokens' own keys where its parts change shape: one token, own keys around one and two
64-key tiles, a row tile of 128 that cuts a head's tokens, one key in the cache, one chunk and several with and without a
ragged last one, as many as there can be, 512 rows per KV head and more, and the sizes beyond which the own keys run as a
launch of their own."""
import pytest

from tests import test_gpu_attention_edges as E

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,hq,hkv,lq,m", [
    ("bf16", 128, 8, 8, 1, 1), ("bf16", 64, 8, 1, 1, 64), ("bf16", 128, 8, 2, 63, 65), ("bf16", 128, 8, 2, 64, 256),
    ("bf16", 64, 12, 4, 65, 257), ("bf16", 128, 7, 1, 43, 511), ("bf16", 64, 14, 2, 37, 4099), ("bf16", 128, 16, 16, 127, 1000),
    ("bf16", 128, 4, 1, 128, 700), ("bf16", 64, 16, 2, 129, 2050), ("bf16", 128, 4, 4, 600, 333),
    ("bf16", 128, 64, 8, 256, 6100), ("f32", 128, 8, 2, 33, 40), ("f32", 64, 14, 2, 5, 2100),
    # own keys bounded by the largest token of a row tile: tiles inside a head's tokens, across two heads and across several
    ("bf16", 64, 8, 2, 300, 100), ("bf16", 128, 6, 2, 200, 70), ("bf16", 64, 12, 2, 100, 5), ("bf16", 128, 16, 2, 33, 300),
    ("bf16", 128, 2, 2, 1024, 300), ("bf16", 64, 2, 2, 1025, 300), ("bf16", 64, 8, 2, 512, 1),
    ("bf16", 128, 8, 1, 1, 16384), ("bf16", 64, 4, 2, 1, 20000), ("f32", 128, 8, 1, 1, 16384),  # the most chunks there are
])
def test_parts(dtype, d, hq, hkv, lq, m):
    E.test_query_attention_with_self_tail(dtype, d, hq, hkv, lq, m)
