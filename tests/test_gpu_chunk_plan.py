"""Attention over chunk tables on both sides of the block-size rule: tables with
at most one chunk per compute unit (256) at 256, 512 and 1024 threads and with
the wide pass, and one chunk more; the last step of
a generation that keeps every token, against fp64 attention over all of them."""
import math

import pytest
import torch

from paper_2605_20600_amd import binding as B, workloads as W
from paper_2605_20600_amd.runner import DeviceInputs, new_session, run_generation

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,long_heads,d", [
    (64, 0, 128),    # 4 chunks of 128 tokens a head: 256 chunks, 256 threads
    (64, 1, 128),    # 257 of them: 512 threads
    (127, 1, 128),   # 2 of 256 tokens, one head of 3: 255, 512 threads
    (128, 1, 128),   # 257: 1024 threads
    (250, 20, 128),  # 270 of 512 tokens, 250 of 576: 1024 threads, wide pass
    (250, 20, 64),   # the same at d = 64: 270 of 512, 250 of 1024 tokens
    (128, 0, 64),    # 2 of 256 tokens: 256 threads
    (128, 1, 64),    # 257: 512 threads
    (3, 1, 64)])
def test_chunk_block_sizes(heads, long_heads, d):
    C, P, short = 100, 7, 403
    wl = W.LUMINA768.with_(batch=1, heads=heads, layers=1, head_dim=d, prefix_len=C, period=P,
                           grid_rows=26, grid_cols=20, row_end=False, group_threshold=50,
                           budget_mode=B.HEADKV_BUDGET_OVERRIDE, override=None)
    inp = DeviceInputs(wl)
    # tables are cut for prefix + budget + P + 1 tokens: 511 (short), 520
    # (long); no step has more tokens than the budget
    bud = torch.full((heads,), short, dtype=torch.int32, device="cuda")
    bud[:long_heads] += 9
    inp.override[0] = bud
    steps = short
    sess = new_session(wl)
    res = run_generation(sess, inp, out_steps=[steps - 1], snap_steps=[steps - 1], steps=steps)
    got = res["out"][(steps - 1, 0)].double()
    assert int(res["snap"][(steps - 1, 0)][1].min()) == steps
    q = inp.q[0][steps - 1].double()
    k = torch.cat((inp.kc[0], inp.k[0][:steps].permute(1, 2, 0, 3)), 2).double()
    v = torch.cat((inp.vc[0], inp.v[0][:steps].permute(1, 2, 0, 3)), 2).double()
    w = torch.softmax((k * q[:, :, None]).sum(-1) / math.sqrt(d), -1)
    ref = (w[..., None] * v).sum(2)
    # fp32 logits of up to 2^6 in log2 units (ulp 2^-18), weights and sums
    assert float((got - ref).abs().max()) <= 2.0 ** -16 * float(v.abs().max())


@pytest.mark.parametrize("heads,C,steps,d", [
    (200, 100, 460, 128),  # one wide chunk of 560 tokens
    (110, 100, 1000, 128),  # two wide chunks of 550
    (110, 100, 2050, 64),  # two wide chunks of 1075
    (4, 128, 4540, 128),   # 37 chunks of 128 tokens a head
    (1, 2048, 4540, 64)])  # 26 chunks of 256
def test_wide_chunks_and_many_chunks(heads, C, steps, d):
    wl = W.LUMINA768.with_(batch=1, heads=heads, layers=1, head_dim=d, prefix_len=C, period=7,
                           grid_rows=steps // 20 + 1, grid_cols=20, row_end=False,
                           group_threshold=50, budget_mode=B.HEADKV_BUDGET_OVERRIDE, override=None)
    inp = DeviceInputs(wl)
    inp.override[0] = torch.full((heads,), steps, dtype=torch.int32, device="cuda")
    sess = new_session(wl)
    res = run_generation(sess, inp, out_steps=[steps - 1], steps=steps)
    got = res["out"][(steps - 1, 0)]
    last = inp.q[0][steps - 1]
    # the allocation-free entry point runs the same chunks without the append
    assert torch.equal(sess.decode_attn(0, last), sess.decode_attn_noalloc(0, last))
    q = last.double()
    k = torch.cat((inp.kc[0], inp.k[0][:steps].permute(1, 2, 0, 3)), 2).double()
    v = torch.cat((inp.vc[0], inp.v[0][:steps].permute(1, 2, 0, 3)), 2).double()
    w = torch.softmax((k * q[:, :, None]).sum(-1) / math.sqrt(d), -1)
    ref = (w[..., None] * v).sum(2)
    # as above; every level of the merge adds a few ulp of fp32
    bound = 2.0 ** -16 * float(v.abs().max())
    assert float((got.double() - ref).abs().max()) <= bound
    assert float((sess.decode_attn(0, last).double() - ref).abs().max()) <= bound
