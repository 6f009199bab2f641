"""Row selection at the lengths where its kernel changes (keys per thread, threads per row, bit passes or histograms),
with the score patterns that take the threshold search to its ends: distinct scores, many exact ties, one value only, two
values, negative zero, and forced positions.  Whole numbers: exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

LENGTHS = [1, 63, 64, 65, 1023, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 8193, 16384, 16385, 32768, 32769, 65535, 65536]


def _rows(pattern, n, rng):
    if pattern == "distinct":
        return rng.standard_normal(n).astype(np.float32) * 30
    if pattern == "ties":
        return (rng.integers(-6, 6, size=n) * 0.5).astype(np.float32) * np.where(rng.random(n) < 0.5, 1, -1).astype(np.float32)
    if pattern == "equal":
        return np.full(n, -3.25, np.float32)
    return np.where(rng.random(n) < 0.3, np.float32(1.0), np.float32(1.0) + np.float32(2.0 ** -23))   # last bit decides


def _want(x, k, n_sink, n_local):
    n = len(x)
    s = x.astype(np.float64) + 0.0
    forced = (np.arange(n) < n_sink) | (np.arange(n) >= n - n_local)
    order = np.lexsort((np.arange(n), -s, ~forced))
    return np.sort(order[:k])


@pytest.mark.parametrize("length", LENGTHS)
@pytest.mark.parametrize("pattern", ["distinct", "ties", "equal", "last_bit"])
def test_rows(length, pattern):
    import torch
    from paper_2508_11661_amd import samkv as S
    rng = np.random.default_rng(length)
    heads, lens = 2, [length, max(1, length // 3)]
    scores = np.stack([np.concatenate([_rows(pattern, n, rng) for n in lens]) for _ in range(heads)])
    caches = S.Caches([torch.zeros((heads, n, 64), dtype=torch.bfloat16, device="cuda") for n in lens], None, heads)
    dev = torch.from_numpy(scores).cuda()
    for ratio, n_sink, n_local in ((0.15, 0, 0), (1.0, 0, 0), (0.4, min(3, length // 9), min(5, length // 9))):
        ks = [S.samkv_kept_count(n, ratio) for n in lens]
        if min(ks) < n_sink + n_local:
            continue
        idx = torch.full((heads, sum(ks)), -1, dtype=torch.int32, device="cuda")
        S.samkv_topk_select(dev, caches, ratio, n_sink, n_local, idx, None)
        got = idx.cpu().numpy()
        for g in range(heads):
            for i, n in enumerate(lens):
                a, o = sum(lens[:i]), sum(ks[:i])
                assert np.array_equal(got[g, o:o + ks[i]], _want(scores[g, a:a + n], ks[i], n_sink, n_local)), (g, i, ratio)


@pytest.mark.parametrize("length,docs,heads", [(1025, 32, 8), (1500, 16, 16), (2048, 20, 13), (2049, 32, 32), (3001, 59, 13),
                                              (4096, 77, 10)])
@pytest.mark.parametrize("pattern", ["distinct", "ties", "equal", "last_bit"])
def test_many_rows(length, docs, heads, pattern):
    """Row counts from which the threshold comes from bit passes again (256 rows of up to 2048 keys, 768 of up to 4096)."""
    import torch
    from paper_2508_11661_amd import samkv as S
    rng = np.random.default_rng(length)
    lens = [length - 3 * (i % 7) for i in range(docs)]
    scores = np.stack([np.concatenate([_rows(pattern, n, rng) for n in lens]) for _ in range(heads)])
    caches = S.Caches([torch.zeros((heads, n, 64), dtype=torch.bfloat16, device="cuda") for n in lens], None, heads)
    ks = [S.samkv_kept_count(n, 0.2) for n in lens]
    idx = torch.full((heads, sum(ks)), -1, dtype=torch.int32, device="cuda")
    S.samkv_topk_select(torch.from_numpy(scores).cuda(), caches, 0.2, 2, 3, idx, None)
    got = idx.cpu().numpy()
    for g in range(heads):
        for i, n in enumerate(lens):
            a, o = sum(lens[:i]), sum(ks[:i])
            assert np.array_equal(got[g, o:o + ks[i]], _want(scores[g, a:a + n], ks[i], 2, 3)), (g, i)


@pytest.mark.parametrize("dtype,d,length", [("bf16", 128, 1024), ("bf16", 64, 1025), ("bf16", 128, 2048), ("f32", 64, 2049),
                                            ("bf16", 128, 4096), ("bf16", 64, 4097), ("f32", 128, 8192)])
def test_fused_rows(dtype, d, length):
    """score + select + gather in one call against the separate calls: the same positions, the same rows."""
    import torch
    from paper_2508_11661_amd import samkv as S
    gen = torch.Generator(device="cuda").manual_seed(length)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    rnd = lambda *s: torch.randn(s, device="cuda", generator=gen).to(dt)
    hq, hkv, lens = 4, 2, [length, length // 2 + 1, 7]
    caches = S.Caches([rnd(hkv, n, d) for n in lens], [rnd(hkv, n, d) for n in lens], hq)
    q_tok, q_loc = rnd(hq, 9, d), rnd(len(lens), hq, 5, d)
    a, b = S.alloc_layer_buffers(caches, 9, 0.2), S.alloc_layer_buffers(caches, 9, 0.2)
    S.samkv_score_select_gather(caches, q_tok, q_loc, 0.2, 1, 1, None, a.idx, a.cu_k_dev, a.k_c, a.v_c, a.ws)
    S.samkv_score(caches, q_tok, q_loc, b.scores, b.ws)
    S.samkv_topk_select(b.scores, caches, 0.2, 1, 1, b.idx, b.cu_k_dev, b.ws)
    S.samkv_gather(caches, b.idx, 0.2, b.k_c, b.v_c)
    for x in ("idx", "cu_k_dev", "k_c", "v_c"):
        assert torch.equal(getattr(a, x), getattr(b, x)), x


WAVE_EDGES = [2, 127, 128, 129, 255, 256, 257, 511, 512, 513]


@pytest.mark.parametrize("length", WAVE_EDGES)
@pytest.mark.parametrize("pattern", ["distinct", "ties", "equal", "last_bit"])
def test_rows_of_one_wave(length, pattern):
    """Rows of up to 512 scores are selected by one wave: the edges of its keys per lane (2, 4, 8)."""
    test_rows(length, pattern)


@pytest.mark.parametrize("length", WAVE_EDGES)
def test_shares_of_short_rows(length):
    """Shares from nothing at all to everything, forced positions among them: a document may keep no position."""
    import torch
    from paper_2508_11661_amd import samkv as S
    rng = np.random.default_rng(7 * length)
    heads, lens = 3, [length] * 4
    scores = np.stack([np.concatenate([_rows(p, length, rng) for p in ("distinct", "ties", "equal", "last_bit")]) for _ in range(heads)])
    caches = S.Caches([torch.zeros((heads, n, 64), dtype=torch.bfloat16, device="cuda") for n in lens], None, heads)
    dev = torch.from_numpy(scores).cuda()
    for shares, n_sink, n_local in (([0.0, 0.5, 0.0, 1.0], 0, 0), ([0.3, 0.0, 1.0, 0.01], 1, 1)):
        ks = [S.samkv_kept_count_mid(n, p, n_sink, n_local) for n, p in zip(lens, shares)]
        idx = torch.full((heads, sum(ks)), -1, dtype=torch.int32, device="cuda")
        S.samkv_topk_select_v(dev, caches, shares, n_sink, n_local, idx, None)
        got = idx.cpu().numpy()
        for g in range(heads):
            for i, n in enumerate(lens):
                o = sum(ks[:i])
                assert np.array_equal(got[g, o:o + ks[i]], _want(scores[g, i * n:(i + 1) * n], ks[i], n_sink, n_local)), (g, i)


@pytest.mark.parametrize("length", [64, 255, 256, 257, 511, 512, 513, 8192])
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f32", 64)])
def test_fused_short_rows(length, dtype, d):
    """Score, selection and compaction in one call at the edges of its selections, everything kept among the shares: the same
    as the separate calls bit for bit."""
    import torch
    from paper_2508_11661_amd import samkv as S
    dt = {"f32": torch.float32, "bf16": torch.bfloat16}[dtype]
    gen = torch.Generator(device="cuda").manual_seed(length)
    R = lambda *s: torch.randn(s, device="cuda", generator=gen).to(dt)
    hkv, group, lens = 2, 2, [length, max(1, length - 3), max(1, length // 3)]
    k, v = [R(hkv, n, d) for n in lens], [R(hkv, n, d) for n in lens]
    k[0][:, length // 2:] = k[0][:, :1]                       # many equal scores
    caches = S.Caches(k, v, hkv * group)
    q_tok, q_loc = R(hkv * group, 5, d), R(len(lens), hkv * group, 7, d)
    for ratio, n_sink, n_local in ((0.2, 0, 0), (1.0, 0, 0), (0.5, 4, 6)):
        a, b = S.alloc_layer_buffers(caches, 5, ratio), S.alloc_layer_buffers(caches, 5, ratio)
        S.samkv_score_select_gather(caches, q_tok, q_loc, ratio, n_sink, n_local, a.scores, a.idx, a.cu_k_dev, a.k_c, a.v_c, a.ws)
        S.samkv_score(caches, q_tok, q_loc, b.scores, b.ws)
        S.samkv_topk_select(b.scores, caches, ratio, n_sink, n_local, b.idx, b.cu_k_dev, b.ws)
        S.samkv_gather(caches, b.idx, ratio, b.k_c, b.v_c)
        for x in ("scores", "idx", "cu_k_dev", "k_c", "v_c"):
            assert torch.equal(getattr(a, x), getattr(b, x)), (ratio, x)
