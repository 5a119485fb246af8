"""headkv_assign_budgets where the layout's tables, and the budgets with the
labels, are on either side of what the pinned buffers hold: the attention after
an update of heads that keep their newest tokens, against fp64 torch."""
import math

import pytest
import torch

from paper_2605_20600_amd import binding as B, workloads as W
from paper_2605_20600_amd.session import Session, make_config

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,heads", [
    (3276, 10),    # 32,760 heads: 24 bytes of tables and 8 of budgets each, below 1 MiB
    (3277, 10),    # 32,770: the tables by copies
    (13108, 10)])  # 131,080: the budgets and labels by copies as well
def test_tables_in_pinned_and_plain_memory(batch, heads):
    d, thr, P, last = 64, 4, 4, 11
    wl = W.LUMINA768.with_(batch=batch, heads=heads, layers=1, head_dim=d, prefix_len=0, period=P,
                           grid_rows=4, grid_cols=4, row_end=False, group_threshold=thr,
                           budget_mode=B.HEADKV_BUDGET_OVERRIDE, override=None)
    BH, N = batch * heads, wl.num_visual
    gen = torch.Generator(device="cuda").manual_seed(3)
    q, k, v = (torch.randn((last + 1, BH, d), generator=gen, device="cuda").bfloat16()
               for _ in range(3))
    budget = torch.randint(1, N + 1, (BH,), generator=gen, device="cuda", dtype=torch.int32)
    sess = Session(make_config(wl))
    sess.prefill(0, None, None)
    for t in range(last + 1):
        sess.append_and_evict(0, t, q[t], k[t], v[t])
        if t == thr - 1:
            local = torch.ones(BH, dtype=torch.uint8, device="cuda")
            assert torch.equal(sess.assign_budgets(0, is_local=local, override=budget), budget)
    out = sess.decode_attn(0, q[last])
    # the last step is an update's (thr - 1 + 2 P): a local head holds its newest
    age = last - torch.arange(last + 1, device="cuda")
    s = (k.double() * q[last].double()).sum(-1) / math.sqrt(d)
    s = s.masked_fill(age[:, None] >= budget[None], -math.inf)
    ref = (torch.softmax(s, 0)[..., None] * v.double()).sum(0)
    # fp32 logits, weights and sums of up to 12 terms
    assert float((out - ref).abs().max()) <= 2e-5 * float(v.abs().max())
