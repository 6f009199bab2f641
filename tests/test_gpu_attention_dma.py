"""The asynchronous-load attention kernels where their tiling can go wrong: row counts around the remainder that sets
where the causal row tiles start (0, 1, 63 .. 65, 192 .. 255 rows beyond a multiple of 256), one to four key tiles,
one and two key groups, both head dimensions, the pair launch, and query problems of 256-row tiles with and without
key chunks."""
import pytest

from tests import test_gpu_attention_edges as E

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,hq,hkv,m", [
    (64, 1024, 8, 1), (64, 1024, 8, 63), (64, 1024, 8, 64), (64, 1024, 8, 65), (64, 1040, 8, 129), (64, 1024, 8, 193),
    (64, 1024, 8, 255), (64, 1024, 8, 256), (64, 515, 5, 320), (64, 512, 8, 321), (64, 344, 8, 577),
    (64, 120, 8, 2049), (64, 120, 8, 2303),
    (128, 384, 8, 192), (128, 384, 8, 193), (128, 192, 8, 257), (128, 192, 8, 320), (128, 195, 5, 321),
    (128, 48, 8, 2049), (128, 48, 8, 2303), (64, 80, 8, 3329), (64, 512, 8, 257),
    (128, 128, 8, 140), (64, 130, 10, 300), (128, 136, 8, 512), (128, 127, 127, 300),  # many heads, few rows
    # two key groups: one key, one and both groups' first tiles, remainders of 128
    (128, 8, 2, 1), (128, 8, 2, 32), (128, 8, 2, 33), (128, 7, 1, 64), (128, 8, 2, 65), (128, 6, 2, 127), (128, 8, 8, 128),
    (128, 8, 2, 129), (128, 5, 5, 192), (128, 8, 2, 193), (128, 8, 2, 256), (128, 4, 2, 257), (128, 8, 2, 1000),
    (64, 8, 2, 1), (64, 8, 2, 64), (64, 8, 2, 65), (64, 7, 1, 129), (64, 8, 2, 193), (64, 8, 2, 385), (64, 16, 2, 1030),
])
def test_recompute(d, hq, hkv, m):
    E.test_recompute_attention_shapes("bf16", d, hq, hkv, m)


@pytest.mark.parametrize("d,hq,hkv,lq,m", [
    (64, 16, 2, 64, 1), (64, 16, 2, 64, 64), (64, 16, 2, 65, 130), (64, 16, 2, 100, 1000), (64, 24, 8, 256, 3001),
])
def test_query(d, hq, hkv, lq, m):
    E.test_query_attention_shapes("bf16", d, hq, hkv, lq, m)


@pytest.mark.parametrize("d,hq,hkv,lq,m", [(64, 512, 8, 3, 321), (64, 120, 8, 45, 2100), (128, 200, 8, 3, 321),
                                           (64, 8, 2, 3, 321), (128, 8, 2, 40, 130), (128, 8, 2, 1, 1), (64, 8, 2, 70, 65)])
def test_both_in_one_call(d, hq, hkv, lq, m):
    E.test_both_attentions_in_one_call("bf16", d, hq, hkv, lq, m)
