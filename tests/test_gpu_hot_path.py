"""The whole path in one call of the library (samkv_hot_path) against its two calls, samkv_score_select_gather and
samkv_recompute_query_attn: every output the same bits, because the heads' largest V magnitudes that the compaction finds are
those that the attentions would look for.  Shapes reach both compactions (in the row's workgroup, and the streaming kernel's two
step counts), both prologues and rows beyond the fused kernel; V's magnitudes differ from head to head by powers of two, with a
head of zeros, so that a wrong maximum would show in every output."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,lens,hkv,group,lq,ratio,n_sink,n_local", [
    ("bf16", 128, [40, 1, 97], 8, 4, 5, 0.3, 0, 0),
    ("bf16", 64, [300, 513, 129], 4, 2, 9, 0.2, 4, 6),
    ("bf16", 128, [1024] * 10, 8, 4, 32, 0.15, 0, 0),
    ("bf16", 128, [700, 9001], 4, 3, 16, 0.1, 0, 0),          # rows beyond the fused kernel
    ("bf16", 64, [60] * 66, 32, 1, 3, 0.5, 0, 0),             # more than 2048 rows, the prologue in two launches
    ("bf16", 128, [260] * 40, 64, 1, 3, 0.45, 0, 0),          # the same with eight steps per wave
    ("f32", 64, [256] * 4, 2, 4, 16, 0.15, 0, 0),
])
def test_one_call(dtype, d, lens, hkv, group, lq, ratio, n_sink, n_local):
    import torch
    from paper_2508_11661_amd import samkv as S
    dt = {"f32": torch.float32, "bf16": torch.bfloat16}[dtype]
    gen = torch.Generator(device="cuda").manual_seed(len(lens) + d)
    R = lambda *s: torch.randn(s, device="cuda", generator=gen).to(dt)
    hq = hkv * group
    mag = torch.exp2((torch.arange(hkv, device="cuda") % 7 - 3).float() * 6).to(dt).view(hkv, 1, 1)
    mag[hkv // 2] = 0.0
    k, v = [R(hkv, n, d) for n in lens], [R(hkv, n, d) * mag for n in lens]
    caches = S.Caches(k, v, hq)
    q_tok, q_loc = R(hq, lq, d), R(len(lens), hq, 6, d)
    m = sum(S.samkv_kept_count(n, ratio) for n in lens)
    q_rec = R(hq, m, d)
    names = ("scores", "idx", "cu_k_dev", "k_c", "v_c", "rec_out", "rec_lse", "q_out", "q_lse")
    two = S.alloc_layer_buffers(caches, lq, ratio)
    S.samkv_score_select_gather(caches, q_tok, q_loc, ratio, n_sink, n_local, two.scores, two.idx, two.cu_k_dev, two.k_c,
                                two.v_c, two.ws)
    S.samkv_recompute_query_attn(q_rec, q_tok, two.k_c, two.v_c, d ** -0.5, two.rec_out, two.rec_lse, two.q_out, two.q_lse, two.ws)
    one = S.alloc_layer_buffers(caches, lq, ratio)
    one.ws.fill_(0xFF)                                        # nothing in the workspace is taken for granted
    for rep in range(2):                                      # and nothing is left over from the call before
        S.hot_path(caches, q_tok, q_loc, q_rec, ratio, d ** -0.5, one, n_sink, n_local)
        for x in names:
            assert torch.equal(getattr(one, x), getattr(two, x)), (rep, x)
    # a workspace that holds the two calls' scratch and nothing behind it
    need = S.samkv_workspace_bytes(len(lens), hq, hkv, d, lq, m) - (hkv * (m // 16 + 8 * len(lens)) * 4 + 255) // 256 * 256 - 256
    small = S.alloc_layer_buffers(caches, lq, ratio)
    small.ws = small.ws[:need]
    S.hot_path(caches, q_tok, q_loc, q_rec, ratio, d ** -0.5, small, n_sink, n_local)
    for x in names:
        assert torch.equal(getattr(small, x), getattr(two, x)), x


def test_other_heads_take_the_two_calls():
    """Caches made for fewer query heads than the states have: accepted, scored with the first heads."""
    import torch
    from paper_2508_11661_amd import samkv as S
    R = lambda *s: torch.randn(s, device="cuda").to(torch.bfloat16)
    lens, hkv, d, lq = [80, 50], 2, 64, 4
    caches = S.Caches([R(hkv, n, d) for n in lens], [R(hkv, n, d) for n in lens], 2)
    m = sum(S.samkv_kept_count(n, 0.5) for n in lens)
    q_tok, q_loc, q_rec = R(4, lq, d), R(2, 2, 3, d), R(4, m, d)
    b = S.alloc_layer_buffers(S.Caches(caches.k, caches.v, 4), lq, 0.5)
    S.hot_path(caches, q_tok, q_loc, q_rec, 0.5, 0.125, b)
    out, lse = torch.empty_like(b.rec_out), torch.empty_like(b.rec_lse)
    S.samkv_recompute_attn(q_rec, b.k_c, b.v_c, 0.125, out, lse, b.ws)
    assert torch.equal(out, b.rec_out) and torch.equal(lse, b.rec_lse)


@pytest.mark.parametrize("d,lens,hkv,group,ratio", [
    (128, [9001] + [20, 64, 128, 1] * 8, 4, 2, 0.5),          # one document much longer than the others
    (128, [128] * 66, 32, 1, 0.5), (64, [256] * 66, 32, 1, 0.5),  # every document fills its workgroups
    (128, [127, 129] * 33, 32, 1, 0.5), (64, [9000, 1], 2, 1, 1.0),
])
def test_one_call_of_uneven_documents(d, lens, hkv, group, ratio):
    """The words of the V magnitudes lie one behind the other, by the documents' prefix sums: none is missed or left as it was."""
    test_one_call("bf16", d, lens, hkv, group, 3, ratio, 0, 0)
