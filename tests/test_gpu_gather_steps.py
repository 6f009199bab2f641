"""Gathers of the kept rows on both sides of the rule for the rows per workgroup: half a large workgroup and one row more,
7/8 of it and one row more, all of it and one row more, 120 to 272 (document, head) pairs, three large workgroups per
document the last of which is half full or one row more, 504 and 512 large workgroups in all, and documents of mixed
counts, some of which keep nothing.  Copies: exact."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 128), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("docs,group", [(32, 1), (15, 2), (17, 2), (21, 1), (64, 1)])
@pytest.mark.parametrize("fill", ["half", "half+1", "most", "most+1", "full", "full+1", "three", "three+1", "mixed"])
def test_gather_steps(dtype, d, docs, group, fill):
    import torch
    from paper_2508_11661_amd import samkv as S
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    rows = 64 // (d * dt.itemsize // 16) * 8 * 4
    hkv, length = 8, 3 * rows + 40
    n = {"half": rows // 2, "most": rows * 7 // 8, "full": rows, "three": rows * 5 // 2}.get(fill.split("+")[0], 0) + ("+" in fill)
    ks = [n] * docs if fill != "mixed" else [(0, 1, rows, 5, rows // 2 + 1)[i % 5] for i in range(docs)]
    gen = torch.Generator("cuda").manual_seed(docs)
    def rand(*shape):
        return torch.randn(shape, device="cuda", generator=gen).to(dt)
    k, v = ([rand(hkv, length, d) for _ in range(docs)] for _ in "kv")
    q = [rand(hkv * group, length, d) for _ in range(docs)]
    caches = S.Caches(k, v, hkv * group)
    cu = [sum(ks[:i]) for i in range(docs + 1)]
    idx = torch.cat([torch.stack([torch.randperm(length, device="cuda", generator=gen)[:c].sort().values for _ in range(hkv)])
                     for c in ks], dim=1).to(torch.int32)
    kc, vc = (torch.zeros((hkv, cu[-1], d), dtype=dt, device="cuda") for _ in "kv")
    qr = torch.zeros((hkv * group, cu[-1], d), dtype=dt, device="cuda")
    S.samkv_gather_v(caches, idx, cu, kc, vc)
    S.samkv_gather_q_v(caches, q, idx, cu, qr)
    for i in range(docs):
        at = idx[:, cu[i]:cu[i + 1]].long()
        for h in range(hkv * group):
            g = h // group
            assert torch.equal(qr[h, cu[i]:cu[i + 1]], q[i][h, at[g]]), (i, h)
            if h % group == 0:
                assert torch.equal(kc[g, cu[i]:cu[i + 1]], k[i][g, at[g]]), (i, g)
                assert torch.equal(vc[g, cu[i]:cu[i + 1]], v[i][g, at[g]]), (i, g)
