"""The merge of a head's chunks in the decode attention: the chunks' shares where
the log2 of their sums is large (as a float it would have steps of 2^-18 to
2^-17), against the exact average, and chunks on both sides of the sums that a
float holds, +-100 in log2, and far beyond."""
import pytest
import torch

from paper_2605_20600_amd import binding as B, workloads as W
from paper_2605_20600_amd.session import Session, make_config

pytestmark = pytest.mark.gpu


def _outputs(d, score, tokens, turn, first):
    """Attention over t + 1 tokens of equal weight, t = first .. tokens - 1: the
    first `turn` values are 1, the others -1.  score: the logit in log2 units."""
    heads = 2
    wl = W.LUMINA768.with_(batch=1, heads=heads, layers=1, head_dim=d, prefix_len=0, period=tokens,
                           grid_rows=tokens // 20, grid_cols=20, row_end=False, group_threshold=8,
                           budget_mode=B.HEADKV_BUDGET_OVERRIDE, override=None)
    sess = Session(make_config(wl))
    q = torch.full((1, heads, d), score / (d ** 0.5 * 1.4427), device="cuda").bfloat16()
    q[:, :, 0] += score * d ** 0.5 / 1.4427 - q.float().sum(-1)  # to a step of q / d
    one = torch.ones_like(q)
    budget = torch.full((heads,), wl.num_visual, dtype=torch.int32, device="cuda")
    outs = []
    sess.prefill(0, None, None)
    for t in range(tokens):
        sess.append_and_evict(0, t, q, one, one if t < turn else -one)
        if t == 7:
            sess.score_heads(0, q)
            sess.assign_budgets(0, override=budget)
        if t >= first:
            outs.append(sess.decode_attn(0, q))
    n = torch.arange(first + 1, tokens + 1, device="cuda", dtype=torch.float64)
    exact = (2 * n.clamp(max=turn) - n) / n
    return torch.stack(outs).double() - exact[:, None, None, None]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("score", [-90, 12, 90])
def test_shares_of_chunks(score, d):
    err = _outputs(d, score, 1600, 700, 800)
    # at most 4 levels (13 chunks of 128 tokens) of 5 roundings of 2^-24 of
    # values up to 1, each 2^-24 / sqrt(3) in the mean square at most, and the
    # chunk's own normalisation; the log2 of a sum as a float of 90 to 100 alone
    # has 2^-18 ln 2 / 2 / sqrt(3) a level
    assert float(err.pow(2).mean().sqrt()) <= 2.0 ** -24 * 25 ** 0.5 / 3 ** 0.5


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("score", [-4000, -127.5, -108, 92.05, 93.06, 127.5, 4000])
def test_large_sums(score, d):
    # half a step of the log2 as a float (2^-13 at 4000, less below) is an error
    # in the share of a subtree at each of the levels
    err = _outputs(d, score, 1600, 700, 1200)
    assert float(err.abs().max()) <= 4 * 0.5 * 2.0 ** -13
