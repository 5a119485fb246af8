"""Attention-sum eviction scores at the edges of their query groups: windows of
one query, of just less and just as many as a group needs, of one and of
several groups with a short last one, and a single query per pass where a
group's weights do not fit; with fewer and with more heads than compute units.
Retained sets bit-exact against the oracle."""
import pytest
import torch

import oracle
from paper_2605_20600_amd import binding as B, workloads as W
from paper_2605_20600_amd.runner import DeviceInputs, new_session, run_generation

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,batch,heads,d,C,thr", [
    (1, 1, 4, 64, 32, 64), (7, 1, 4, 64, 32, 64), (8, 1, 4, 64, 0, 64), (15, 1, 4, 128, 32, 64),
    (16, 1, 4, 64, 32, 65), (17, 1, 4, 128, 3, 64), (33, 1, 4, 64, 32, 64), (49, 2, 8, 128, 32, 70),
    (9, 65, 4, 64, 16, 64), (20, 9, 32, 128, 32, 64),
    (16, 1, 4, 64, 2048, 390)])
def test_attention_sum_groups(P, batch, heads, d, C, thr):
    grid = 24
    wl = W.TINY.with_(batch=batch, heads=heads, head_dim=d, prefix_len=C, period=P,
                      grid_rows=grid, grid_cols=grid, group_threshold=thr, rho=(1, 8),
                      amp_mode="lumina", v_positional=False, score_mode=B.HEADKV_SCORE_ATTN_SUM)
    t_g = thr - 1
    steps = [t_g, t_g + P, t_g + 2 * P, t_g + 2 * P + 1]
    inp = DeviceInputs(wl)
    sess = new_session(wl)
    res = run_generation(sess, inp, snap_steps=steps, steps=steps[-1] + 1)
    torch.cuda.synchronize()
    for b in sorted({0, batch - 1}):
        ref = oracle.simulate(wl, 0, b, snap_steps=steps)
        assert (res["budgets"][0].view(batch, heads)[b].cpu().numpy() == ref["budgets"]).all()
        for i, t in enumerate(steps):
            mask = res["snap"][(t, 0)][0].view(batch, heads, -1)[b].cpu().numpy()
            for h in range(heads):
                assert (mask[h] == ref["snaps"][h][i]).all(), (b, h, t)
