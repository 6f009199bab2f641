"""bf16 attention whose query rows reach the registers by way of LDS (two key groups, one workgroup per compute unit): both
attentions in one call, every row, at the edges of the 128-row tiles and of their 64-key steps, with fewer and more query
rows than a tile."""
import math

import numpy as np
import pytest

from oracle import samkv_oracle as O
from paper_2508_11661_amd import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("m,lq", [(321, 1), (383, 127), (385, 128), (448, 129), (511, 5), (513, 300), (640, 64)])
def test_query_rows_at_tile_edges(d, m, lq):
    import torch
    from paper_2508_11661_amd import samkv as S
    hq, hkv, scale = 4, 2, 1.0 / math.sqrt(d)
    rng = np.random.default_rng(m + d)
    draw = lambda h, n, s: synth.round_to_dtype(rng.standard_normal((h, n, d), dtype=np.float32) * s, "bf16")
    q, qt, k, v = draw(hq, m, 1.5), draw(hq, lq, 1.5), draw(hkv, m, 1.5), draw(hkv, m, 2.0)
    nan = lambda *shape: torch.full(shape, float("nan"), device="cuda")
    ro, rl, qo, ql = nan(hq, m, d), nan(hq, m), nan(hq, lq, d), nan(hq, lq)
    ws = torch.empty((S.samkv_workspace_bytes(1, hq, hkv, d, lq, m),), dtype=torch.uint8, device="cuda")
    S.samkv_recompute_query_attn(*(H.to_dev(x, "bf16") for x in (q, qt, k, v)), scale, ro, rl, qo, ql, ws)
    for name, o, l, x, causal in (("recompute", ro, rl, q, True), ("query", qo, ql, qt, False)):
        o_ref, l_ref = O.attention(x, k, v, scale, causal)
        H.check_attention(o.cpu().numpy(), l.cpu().numpy(), o_ref, l_ref, "bf16", f"{name} d={d} m={m} lq={lq}")
