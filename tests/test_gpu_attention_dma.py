"""The bf16 attention kernels where their tiling can go wrong, each at the sizes that its dispatch rule gives it: row counts
around the remainder that sets where the causal row tiles of the asynchronous kernels start, one to several key tiles, one
and two key groups, both head dimensions, the pair launch, query problems of 256-row tiles with and without key chunks, and
the row and workgroup counts at which one kernel gives way to the next."""
import pytest

from tests import test_gpu_attention_edges as E

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,hq,hkv,m", [
    # register-staged: one to three key tiles, remainders of 128, many heads, the largest row counts of its rules
    (64, 1024, 8, 1), (64, 1024, 8, 63), (64, 1024, 8, 64), (64, 1024, 8, 65), (64, 1040, 8, 129), (64, 1024, 8, 193),
    (64, 1024, 8, 255), (64, 1024, 8, 256), (64, 515, 5, 320), (64, 512, 8, 321), (64, 512, 8, 257), (64, 130, 10, 300),
    (128, 384, 8, 192), (128, 384, 8, 193), (128, 192, 8, 257), (128, 192, 8, 320), (128, 195, 5, 321), (128, 128, 8, 140),
    (128, 136, 8, 512), (128, 127, 127, 300), (128, 127, 127, 512), (64, 130, 10, 513), (128, 128, 8, 640), (64, 160, 32, 640), (64, 112, 112, 640),
    (128, 8, 2, 1), (128, 8, 2, 32), (128, 8, 2, 33), (128, 7, 1, 64), (128, 8, 2, 65), (128, 6, 2, 127), (128, 8, 8, 128),
    (128, 8, 2, 129), (128, 5, 5, 192), (128, 8, 2, 256), (128, 4, 2, 257), (128, 8, 2, 320), (64, 8, 2, 320),
    (64, 8, 2, 1), (64, 8, 2, 64), (64, 8, 2, 65), (64, 7, 1, 129), (64, 8, 2, 193),
    (128, 96, 12, 768), (128, 48, 8, 1536), (64, 76, 19, 384), (128, 75, 15, 400),
    # 256 rows per workgroup: 0, 1, 63, 64, 65, 192, 193 and 255 rows beyond a multiple of 256
    (128, 112, 8, 704), (128, 112, 16, 768), (128, 115, 5, 769), (128, 112, 8, 831), (128, 112, 8, 832), (128, 112, 16, 833),
    (128, 112, 8, 960), (128, 115, 5, 961), (128, 112, 8, 1023), (128, 128, 8, 641), (128, 48, 8, 2049), (128, 48, 8, 2303),
    (64, 130, 130, 768), (64, 256, 8, 769), (64, 100, 100, 831), (64, 256, 8, 832), (64, 100, 100, 833), (64, 256, 8, 960),
    (64, 100, 100, 961), (64, 256, 8, 1023), (64, 120, 8, 2049), (64, 120, 8, 2303), (64, 80, 8, 3329),
    # two key groups, one workgroup per compute unit: remainders of 128, both groups' first and last tiles
    (128, 8, 2, 321), (128, 7, 1, 384), (128, 8, 2, 385), (128, 5, 5, 449), (128, 2, 2, 640), (128, 6, 2, 767), (128, 8, 2, 1000),
    (64, 8, 2, 321), (64, 7, 1, 384), (64, 8, 2, 385), (64, 5, 5, 449), (64, 8, 8, 512), (64, 4, 4, 895), (64, 16, 2, 1030),
    (128, 28, 7, 2433), (64, 60, 5, 1024),
    # the same, two workgroups per compute unit
    (64, 100, 10, 700), (64, 64, 8, 899), (64, 96, 12, 640), (64, 61, 61, 1000), (64, 60, 4, 1025), (64, 60, 5, 1087), (64, 24, 8, 2753), (64, 24, 8, 2815),
])
def test_recompute(d, hq, hkv, m):
    E.test_recompute_attention_shapes("bf16", d, hq, hkv, m)


@pytest.mark.parametrize("d,hq,hkv,lq,m", [
    # register-staged: up to 511 rows per KV head, and more of them with few keys
    (64, 16, 2, 64, 1), (64, 16, 2, 64, 64), (64, 16, 2, 65, 130), (64, 16, 2, 100, 1000), (64, 24, 8, 256, 3001),
    (128, 16, 2, 200, 1), (128, 16, 2, 65, 64), (128, 24, 8, 171, 1300), (128, 64, 8, 100, 3661), (64, 64, 8, 256, 3814),
    # 256 rows per workgroup beyond: several chunks with a ragged last one, one chunk of two and three key tiles
    (128, 64, 8, 100, 3663), (64, 64, 8, 256, 3816), (64, 64, 8, 257, 4001), (128, 256, 64, 1500, 65), (64, 256, 64, 1500, 164),
])
def test_query(d, hq, hkv, lq, m):
    E.test_query_attention_shapes("bf16", d, hq, hkv, lq, m)


@pytest.mark.parametrize("d,hq,hkv,lq,m", [
    (64, 512, 8, 3, 321), (128, 200, 8, 3, 321), (128, 8, 2, 40, 130), (128, 8, 2, 1, 1), (64, 8, 2, 70, 65),  # register-staged
    (64, 120, 8, 45, 2100), (128, 112, 8, 3, 769),                                                          # 256 rows
    (64, 8, 2, 3, 321), (128, 8, 2, 40, 400), (64, 16, 4, 100, 900), (64, 60, 4, 5, 1025),                  # two key groups
])
def test_both_in_one_call(d, hq, hkv, lq, m):
    E.test_both_attentions_in_one_call("bf16", d, hq, hkv, lq, m)


@pytest.mark.parametrize("d,hq,hkv,m", [(128, 8, 2, 400), (64, 8, 2, 400), (128, 64, 8, 1600), (64, 256, 8, 1200)])
def test_rows_without_mass_in_the_first_tile(d, hq, hkv, m):
    """Odd rows have only scores of -inf (products beyond float32) in the first 64 keys, even rows of the same wave do not:
    from key 64 on the odd rows are ordinary ones."""
    import numpy as np
    import torch
    from paper_2508_11661_amd import samkv as S
    q, k, v = E._data(m, "bf16", hq, hkv, m, m, d)
    q[:, ::2, 0], q[:, 1::2, 0] = 0.0, 4.0
    k[..., 0] = 0.0
    k[:, :64, 0] = np.float32(-2.0 ** 127)
    out, lse = torch.full((hq, m, d), float("nan"), device="cuda"), torch.full((hq, m), float("nan"), device="cuda")
    ws = torch.empty((S.samkv_workspace_bytes(1, hq, hkv, d, 1, m),), dtype=torch.uint8, device="cuda")
    S.samkv_recompute_attn(E.H.to_dev(q, "bf16"), E.H.to_dev(k, "bf16"), E.H.to_dev(v, "bf16"), d ** -0.5, out, lse, ws)
    rows = np.array([0, 30, 62, 64, 65, 67, 95, 96, 127, 128, 129, 200, 321, 399, m - 2, m - 1])
    for h in (0, hq // 2 + 1, hq - 1):
        g = h // (hq // hkv)
        o_ref, l_ref = E.O.attention(q[h:h + 1], k[g:g + 1], v[g:g + 1], d ** -0.5, True, rows=rows)
        E.H.check_attention(out[h:h + 1, rows].cpu().numpy(), lse[h:h + 1, rows].cpu().numpy(), o_ref, l_ref, "bf16", f"head {h}")


@pytest.mark.parametrize("causal,d,hq,hkv,lq,m", [
    (True, 128, 16, 16, 0, 700), (True, 128, 9, 9, 0, 700), (True, 64, 8, 8, 0, 3000), (True, 64, 5, 5, 0, 4200),
    (False, 128, 64, 8, 1300, 300), (False, 128, 56, 7, 1500, 300), (False, 128, 64, 8, 200, 2100), (False, 64, 56, 7, 600, 4200),
])
def test_value_scales(causal, d, hq, hkv, lq, m):
    """The half-precision copy of V in every order in which its preparation walks heads and chunks (one or two launches, a
    head count that is a multiple of 8 or not, causal or not): heads of very different magnitude, each with its own scale."""
    import numpy as np
    import torch
    from paper_2508_11661_amd import samkv as S
    rows = m if causal else lq
    q, k, v = E._data(m + hkv, "bf16", hq, hkv, rows, m, d)
    mag = np.array([2.0 ** (7 * (g % 5) - 14) for g in range(hkv)], np.float32)
    v = v * mag[:, None, None]
    out, lse = torch.full((hq, rows, d), float("nan"), device="cuda"), torch.full((hq, rows), float("nan"), device="cuda")
    ws = torch.empty((S.samkv_workspace_bytes(1, hq, hkv, d, rows, m),), dtype=torch.uint8, device="cuda")
    args = (E.H.to_dev(q, "bf16"), E.H.to_dev(k, "bf16"), E.H.to_dev(v, "bf16"), d ** -0.5, out, lse, ws)
    S.samkv_recompute_attn(*args) if causal else S.samkv_query_attn(*args)
    pick = np.array([0, 63, 64, rows // 2, rows - 1])
    for g in range(hkv):
        h = g * (hq // hkv)
        o_ref, l_ref = E.O.attention(q[h:h + 1], k[g:g + 1], v[g:g + 1], d ** -0.5, causal, rows=pick)
        got = out[h:h + 1, pick].cpu().numpy() / mag[g]
        E.H.check_attention(got, lse[h:h + 1, pick].cpu().numpy(), o_ref / mag[g], l_ref, "bf16", f"KV head {g}")
