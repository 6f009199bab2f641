"""Float32 attention on products of bf16 terms, at the edges of its kernels: eight waves of 32 query rows, as 256
rows of a workgroup (one stream of keys, 32 a step) or as 128 rows whose keys two groups of waves share (64 a step).  The
sizes are beyond those that `attn_f32_shape` leaves to the float32 products.  The inputs that terms do not hold (infinities,
NaN, magnitudes past 2^60, in V past 2^48) must come out as exactly as with float32 products, and so must all others."""
import math

import pytest

from tests import test_gpu_attention_edges as E

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("m", [319, 320, 321, 351, 352, 353, 383, 384, 385])
def test_recompute_keys2_edges(d, m):
    """128 rows per workgroup: last row tiles and last steps of 1, 31, 32, 33, 63 and 64 keys."""
    E.test_recompute_attention_shapes("f32", d, 72, 8, m)


@pytest.mark.parametrize("d,hq,hkv,m", [
    (128, 136, 8, 129), (64, 200, 8, 129), (128, 136, 17, 161), (128, 136, 8, 255), (128, 136, 8, 256),  # one tile of 256
    (128, 400, 8, 65), (64, 400, 8, 96),                                                                # 128 rows, not full
    (128, 200, 8, 257), (128, 192, 24, 289), (64, 256, 8, 321), (128, 128, 8, 513), (64, 96, 8, 1000),  # 128 rows
    (128, 8, 8, 1700), (64, 6, 3, 2700),                                                 # few heads: float32 products
])
def test_recompute(d, hq, hkv, m):
    E.test_recompute_attention_shapes("f32", d, hq, hkv, m)


@pytest.mark.parametrize("d,hq,hkv,lq,m", [
    (128, 16, 2, 16, 8800), (128, 8, 2, 33, 9001), (64, 8, 1, 5, 75001), (64, 16, 4, 50, 4033),       # float32 products
    (128, 64, 16, 40, 3001), (64, 64, 16, 40, 3021), (128, 256, 256, 150, 70),            # 128 rows, the last one as above
])
def test_query(d, hq, hkv, lq, m):
    E.test_query_attention_shapes("f32", d, hq, hkv, lq, m)


@pytest.mark.parametrize("d,hq,hkv,lq,m", [
    (128, 64, 8, 4, 321), (64, 72, 8, 7, 385),       # query on float32 products: an odd number of units, and an even one
    (128, 64, 8, 64, 600), (64, 64, 8, 96, 700),     # the same, of several row tiles
    (128, 128, 8, 8, 700), (64, 128, 8, 40, 1100),   # the same, and 128 rows for both
])
def test_both_in_one_call(d, hq, hkv, lq, m):
    E.test_both_attentions_in_one_call("f32", d, hq, hkv, lq, m)


KINDS = ["k_inf", "k_past", "v_inf", "v_nan", "q_past", "k_rows", "k_chunks", "k_inside", "v_rows", "v_chunks", "v_far", "v_tiny",
         "products", "zero"]


@pytest.mark.parametrize("hq,m", [(72, 330), (136, 200)])  # 128 rows per workgroup, and 256
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("kind", KINDS)
def test_odd_inputs(kind, d, hq, m):
    import torch
    from paper_2508_11661_amd import samkv as S
    gen = torch.Generator(device="cuda").manual_seed(7)
    normal = lambda *s: torch.randn(s, device="cuda", generator=gen)
    power = lambda lo, hi, *s: torch.exp2(torch.randint(lo, hi, s, device="cuda", generator=gen).float())
    q, k, v = normal(hq, m, d), normal(1, m, d), normal(1, m, d)
    bad = None  # a row and channel of V that is no number
    if kind == "k_inf":
        q[..., 5] = -q[..., 5].abs() - 0.1
        k[0, 150, 5] = math.inf                               # a score of -inf for the rows behind it
    if kind == "k_past":
        q[..., 0], k[0, 100:140, 0] = 4.0, -2.0 ** 127        # -inf by overflow
    if kind in ("v_inf", "v_nan"):
        bad = (120, 7)
        v[0, 120, 7] = -math.inf if kind == "v_inf" else math.nan
    if kind == "q_past":
        # its scores stay of order 10: at 2^70 x 2^-60 they reach 2^13, whose float32 rounding alone, 2^13 x 2^-24 = 5e-4,
        # is past the bar
        q[:, 170] *= 2.0 ** 70
        k[0, :, :] *= 2.0 ** -70
    if kind == "k_rows":
        k *= power(-20, 3, 1, m, 1)
    if kind == "k_chunks":
        k *= power(-20, 3, 1, 1, d // 4).repeat_interleave(4, 2)
    if kind == "k_inside":                                    # within what the terms hold
        k *= power(-11, 0, 1, 1, d // 4).repeat_interleave(4, 2)
        q *= power(-5, 5, 1, m, 1)
    if kind == "v_rows":
        v *= power(-30, 30, 1, m, 1)
    if kind == "v_chunks":
        v *= power(-24, 0, 1, 1, d // 4).repeat_interleave(4, 2)
    if kind == "v_far":                                       # every four rows alike, far from the others
        v *= power(-30, 0, 1, (m + 3) // 4, 1).repeat_interleave(4, 1)[:, :m]
    if kind == "v_tiny":
        v *= 2.0 ** -100
    if kind == "products":
        q *= 2.0 ** 55
        k *= 2.0 ** -55
    if kind == "zero":
        v.zero_()
    scale = d ** -0.5
    s = (q.double() @ k[0].double().T)
    s = torch.where(s < -3.4e38, -math.inf, s) * scale        # what float32 products overflow to
    s.masked_fill_(torch.ones((m, m), device="cuda", dtype=torch.bool).triu(1), -math.inf)
    lse_ref = torch.logsumexp(s, 2)
    p = torch.exp(s - lse_ref[..., None])
    vv = v[0].double()
    if bad is not None:
        vv[bad] = 0.0
    ref = p @ vv
    out, lse = torch.full((hq, m, d), 7.0, device="cuda"), torch.zeros((hq, m), device="cuda")
    S.samkv_recompute_attn(q, k, v, scale, out, lse, None)
    torch.cuda.synchronize()
    got = out.double()
    if bad is not None:
        col = got[:, bad[0]:, bad[1]]                          # every row that sees it
        assert (torch.isneginf(col) if kind == "v_inf" else torch.isnan(col)).all()
        got[..., bad[1]] = ref[..., bad[1]]
    # per row: the output's error against its largest value, 1e-4 as in the repository's float32 bar; channels that differ in
    # magnitude are held to their own
    per = d // 4 if kind == "v_chunks" else 1
    err = (got - ref).abs().reshape(hq, m, per, -1).amax(3)
    top = ref.abs().reshape(hq, m, per, -1).amax(3)
    assert (err <= 1e-4 * top).all(), (err / top.clamp_min(1e-300)).max().item()
    assert ((lse.double() - lse_ref).abs() <= 1e-4 * lse_ref.abs().clamp_min(1.0)).all()


def _reference(q, k, v, scale, causal):
    """float64, every head of one KV head: outputs and log-sum-exp"""
    import torch
    s = (q.double() @ k[0].double().T) * scale
    if causal:
        s.masked_fill_(torch.ones(s.shape[1:], device="cuda", dtype=torch.bool).triu(1), -math.inf)
    lse = torch.logsumexp(s, 2)
    return torch.exp(s - lse[..., None]) @ v[0].double(), lse


def _run(q, k, v, scale, causal):
    import torch
    from paper_2508_11661_amd import samkv as S
    out, lse = torch.full_like(q, math.nan), torch.full(q.shape[:2], math.nan, device="cuda")
    if causal:
        S.samkv_recompute_attn(q, k, v, scale, out, lse, None)
    else:
        ws = torch.empty((S.samkv_workspace_bytes(1, q.shape[0], 1, q.shape[2], q.shape[1], k.shape[1]),), dtype=torch.uint8,
                         device="cuda")
        S.samkv_query_attn(q, k, v, scale, out, lse, ws)
    torch.cuda.synchronize()
    return out, lse


# heads, rows, keys of a problem on 128 and on 256 rows per workgroup, the last step and row tile ragged
SHAPES = {"causal128": (72, 330, 330), "causal256": (136, 200, 200), "query128": (8, 45, 14001), "query256": (136, 300, 3001)}


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("kind", ["zero", "zero_rows", "zero_rows_zero_keys", "tiny"])
def test_scores_that_vanish(kind, d, shape):
    """Products so small that the factor which undoes the operands' scales passes below float32: uniform weights, as the masked
    scores of a diagonal or ragged tile must not meet a factor of zero.  Outputs of float32 rounding: 2^-24 per weight and sum."""
    import torch
    hq, rows, m = SHAPES[shape]
    gen = torch.Generator(device="cuda").manual_seed(11)
    normal = lambda *s: torch.randn(s, device="cuda", generator=gen)
    q, k, v = normal(hq, rows, d), normal(1, m, d), normal(1, m, d)
    if kind == "zero":
        q.zero_(), k.zero_()
    if kind in ("zero_rows", "zero_rows_zero_keys"):
        q[:, ::3] = 0.0
        k *= 1e-4
    if kind == "zero_rows_zero_keys":
        k[:, :70] = 0.0
    if kind == "tiny":
        q *= 2.0 ** -70
        k *= 2.0 ** -70
    out, lse = _run(q, k, v, d ** -0.5, shape.startswith("causal"))
    ref, lse_ref = _reference(q, k, v, d ** -0.5, shape.startswith("causal"))
    assert ((out.double() - ref).norm() <= 4e-6 * ref.norm()).item()
    assert ((lse.double() - lse_ref).abs().max() <= 4e-6).item()


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("value", [math.inf, -math.inf, math.nan])
def test_infinity_behind_a_large_value(value, d, shape):
    """An infinity or NaN of V that follows, in the rows that a wave stages, a number of 2^126, so that no larger scale exists: it
    comes out as itself.  (The other numbers are small enough for a sum of 3000 and within reach of that scale.)"""
    import torch
    hq, rows, m = SHAPES[shape]
    gen = torch.Generator(device="cuda").manual_seed(12)
    normal = lambda *s: torch.randn(s, device="cuda", generator=gen)
    q, k, v = normal(hq, rows, d), normal(1, m, d), normal(1, m, d)
    v *= 2.0 ** 119
    v[0, 20, 3] = 2.0 ** 126
    v[0, 150, 7] = value
    causal = shape.startswith("causal")
    out, lse = _run(q, k, v, d ** -0.5, causal)
    col = out[:, 150 if causal else 0:, 7]
    assert (torch.isnan(col) if math.isnan(value) else col == value).all()
    assert torch.isfinite(lse).all()


SINKS = [f"sink {nats} nats, V x {v}" for nats in (8, 12, 16, 20, 40) for v in (0.0, 0.01)]
CHANNELS = [f"channel of {x} x 2^-{e}" for x in ("V", "K") for e in (12, 20, 24)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("kind", ["normal", "channel scales", "leading zeros of V", "v x 2^-130"] + SINKS + CHANNELS)
def test_precision_of_float32(kind, d, shape):
    """No more error against float64 than float32 products make, which is what the same heads get in a call of their own, too
    small for the terms: over all outputs and, as a channel far below the others shows in its own outputs only, over each
    channel.  A sink is a key that takes nearly all of the weight and has little or no V, so that the outputs are sums of small
    weights."""
    import torch
    hq, rows, m = SHAPES[shape]
    gen = torch.Generator(device="cuda").manual_seed(13)
    normal = lambda *s: torch.randn(s, device="cuda", generator=gen)
    q, k, v = normal(hq, rows, d), normal(1, m, d), normal(1, m, d)
    if kind == "channel scales":
        scales = torch.exp2(2 * normal(d).clamp(-1, 1))
        q, k, v = q * scales, k * scales, v * scales
    if kind == "leading zeros of V":
        v[0, :70] = 0.0
    if kind == "v x 2^-130":
        v *= 2.0 ** -130
    if kind in SINKS:
        nats, x = float(kind.split()[1]), float(kind.split()[-1])
        q += 1.0                                              # the direction of the sink's key
        k[0, 0] = nats * d ** -0.5
        v[0, 0] *= x
    if kind in CHANNELS:
        e = int(kind.split("-")[1])
        if "V" in kind:
            v[..., 5] *= 2.0 ** -e
        else:
            k[..., ::8] *= 2.0 ** -e
            q[..., ::8] *= 2.0 ** e
    causal, scale = shape.startswith("causal"), d ** -0.5
    out, lse = _run(q, k, v, scale, causal)
    heads = [0, hq // 2, hq - 1]
    ref, lse_ref = _reference(q[heads], k, v, scale, causal)
    if causal:
        plain, lse_plain = _run(q[heads], k, v, scale, True)
    else:
        parts = [_run(q[h:h + 1, n:n + 50].contiguous(), k, v, scale, False) for h in heads for n in range(0, rows, 50)]
        plain = torch.cat([x[0] for x in parts], 1).view(3, rows, d)
        lse_plain = torch.cat([x[1] for x in parts], 1).view(3, rows)
    per = lambda x, r: (x.double() - r).flatten(0, 1).norm(dim=0)
    ours, theirs = per(out[heads], ref), per(plain, ref)
    # Half as much again, as the roundings of a sink's score move whole rows; and outputs that one key holds nearly alone are
    # rounded once in each step of 32 keys, by 2^-25 of them, where a call of fewer keys has fewer steps.
    own = 2.0 ** -25 * math.sqrt(m / 32) * ref.norm()
    assert (ours.norm() <= 1.5 * theirs.norm() + own).item(), (ours.norm() / theirs.norm()).item()
    if kind in CHANNELS:
        assert (ours <= 2 * theirs).all(), (ours / theirs).max().item()
    assert ((lse[heads].double() - lse_ref).norm() <= 1.5 * (lse_plain.double() - lse_ref).norm()).item()


@pytest.mark.parametrize("d,hq,hkv,m", [
    (128, 16, 16, 2300), (64, 40, 8, 1300),                           # few heads, 128 rows per workgroup
    (128, 400, 8, 300), (64, 400, 8, 290), (128, 200, 8, 900),        # 256 rows, several row tiles
])
def test_recompute_long(d, hq, hkv, m):
    E.test_recompute_attention_shapes("f32", d, hq, hkv, m)


@pytest.mark.parametrize("d,hq,hkv,lq,m", [
    (128, 8, 2, 50, 9001), (64, 8, 1, 33, 18001), (64, 64, 64, 129, 600),   # 128 rows, one chunk and several
    (128, 16, 4, 50, 60001), (128, 256, 256, 150, 140), (64, 192, 24, 200, 130),  # 256 rows
])
def test_query_long(d, hq, hkv, lq, m):
    E.test_query_attention_shapes("f32", d, hq, hkv, lq, m)


@pytest.mark.parametrize("d,hq,hkv,lq,m", [
    (128, 72, 8, 4, 341), (64, 72, 8, 7, 385),          # causal on 128 rows, the query on float32 products
    (128, 64, 8, 128, 600), (64, 64, 8, 130, 700),      # 128 rows for both
    (128, 192, 24, 250, 300),                           # the query on 256 rows
    (128, 400, 8, 1, 300), (64, 400, 8, 1, 290),        # causal on 256 rows, the query on each
    (128, 400, 8, 50, 300), (128, 408, 24, 110, 300), (64, 408, 24, 110, 290),
])
def test_both_in_one_call_shapes(d, hq, hkv, lq, m):
    E.test_both_attentions_in_one_call("f32", d, hq, hkv, lq, m)


@pytest.mark.parametrize("d,hq,hkv,lq,m", [(128, 16, 16, 1024, 600), (64, 32, 16, 512, 900)])
def test_no_workspace_where_float32_products_need_none(d, hq, hkv, lq, m):
    """Problems whose row tiles fill the chip with float32 products take one chunk of keys and no workspace, as ever; the terms'
    larger workgroups would cut the keys in two.  One byte less than those chunks take counts as no workspace, too."""
    import torch
    from paper_2508_11661_amd import samkv as S
    gen = torch.Generator(device="cuda").manual_seed(17)
    normal = lambda *s: torch.randn(s, device="cuda", generator=gen)
    q, qt, k, v, scale = normal(hq, m, d), normal(hq, lq, d), normal(hkv, m, d), normal(hkv, m, d), d ** -0.5
    ref, lse_ref = _reference(qt[:1], k[:1], v[:1], scale, False)
    for ws in (None, torch.empty((hq * lq * (d + 1) * 8 - 1,), dtype=torch.uint8, device="cuda")):
        for both in (False, True):
            out, lse = torch.full_like(qt, math.nan), torch.full((hq, lq), math.nan, device="cuda")
            if both:
                rec, rec_lse = torch.empty_like(q), torch.empty((hq, m), device="cuda")
                S.samkv_recompute_query_attn(q, qt, k, v, scale, rec, rec_lse, out, lse, ws)
            else:
                S.samkv_query_attn(qt, k, v, scale, out, lse, ws)
            torch.cuda.synchronize()
            assert ((out[:1].double() - ref).norm() <= 4e-6 * ref.norm()).item()
            assert ((lse[:1].double() - lse_ref).abs().max() <= 4e-6).item()
            assert torch.isfinite(out).all() and torch.isfinite(lse).all()
