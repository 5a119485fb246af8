"""The order in which an fp64 matrix step adds its four products, which the
attention-sum scores of a group of queries rely on (csrc/cache_kernels.hip:
v_mfma_f64_16x16x4 rounds like four fused multiply-adds in order of the dims).
Keys hold a huge value, its negative and small values around them, so that what
is left of the small ones, and with it the retained set, depends on the order:
bit-exact against the oracle, which adds the dims one by one."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_20600_amd import binding as B, workloads as W
from paper_2605_20600_amd.runner import DeviceInputs, new_session, run_generation
from test_gpu_ties import _Inputs, _slice

HUGE = 2.0 ** 60
# where the huge value and its negative lie, from the first dim of a step
PLACES = [(0, 1), (0, 2), (0, 3), (1, 2), (1, 3), (2, 3), (1, 0), (2, 0), (3, 1), (3, 4), (2, 5),
          (-1, 0), (-1, 1), (-1, 3)]


def _inputs(wl):
    inp = DeviceInputs(wl, layers=[0], device="cpu")
    k, q = inp.k[0], inp.q[0]
    N, _, H, d = k.shape
    for t in range(N):
        for h in range(H):
            first, second = PLACES[(t + 5 * h) % len(PLACES)]
            step = 4 + 4 * ((t // len(PLACES) + 3 * h) % (d // 4 - 3))
            k[t, 0, h, step + first], k[t, 0, h, step + second] = HUGE, -HUGE
    # the huge products cancel: one value in all dims of a query
    scale = (1 + torch.arange(N) % 8)[:, None, None, None] / 8
    q.copy_((scale * torch.ones_like(q, dtype=torch.float32)).to(q.dtype))
    return inp


def _logits(k, order):
    """Sums of the dims of k [..., d], each step's four by `order`."""
    acc = np.zeros(k.shape[:-1])
    for i in range(0, k.shape[-1], 4):
        acc = order(acc, *(k[..., i + j] for j in range(4)))
    return acc


def test_the_keys_tell_orders_apart():
    k = _inputs(W.TINY)
    k = k.k[0].double().numpy()
    in_order = _logits(k, lambda s, a, b, c, d: (((s + a) + b) + c) + d)
    for other in (lambda s, a, b, c, d: (((s + d) + c) + b) + a,
                  lambda s, a, b, c, d: s + (((a + b) + c) + d),
                  lambda s, a, b, c, d: s + ((a + b) + (c + d)),
                  lambda s, a, b, c, d: s + ((a + c) + (b + d)),
                  lambda s, a, b, c, d: (s + (a + b)) + (c + d),
                  lambda s, a, b, c, d: (s + (a + c)) + (b + d)):
        assert (_logits(k, other) != in_order).mean() > 0.1


@pytest.mark.gpu
@pytest.mark.parametrize("P,d", [(16, 64), (16, 128), (11, 64), (4, 128)])
def test_retained_sets_by_sums_in_order(P, d):
    # groups of 16 and of 11 queries on the matrix cores, and one at a time
    wl = W.TINY.with_(head_dim=d, period=P, rho=(1, 4), v_positional=False,
                      score_mode=B.HEADKV_SCORE_ATTN_SUM)
    H, t_g = wl.heads, wl.group_threshold - 1
    steps = [t_g + u * P for u in range(5)]
    cpu = _inputs(wl)
    glob = torch.zeros(H, dtype=torch.uint8)
    res = run_generation(new_session(wl), _Inputs(cpu, "cuda"), snap_steps=steps,
                         steps=steps[-1] + 1, label_override={0: glob.cuda()})
    torch.cuda.synchronize()
    ref = oracle.simulate(wl, 0, 0, snap_steps=steps, inputs=_slice(cpu, 0),
                          label_override=glob.numpy())
    for i, t in enumerate(steps):
        mask = res["snap"][(t, 0)][0].cpu().numpy()
        for h in range(H):
            assert ref["stats"][h]["evicted"] > 0 and ref["stats"][h]["min_gap"] > 1e-9
            assert (mask[h] == ref["snaps"][h][i]).all(), (h, t)
