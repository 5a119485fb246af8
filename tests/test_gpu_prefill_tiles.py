"""Prefix prefill attention at the edges of its tiles: 32-query wavefronts, key
tiles of 32 and 64, blocks of one, two and four wavefronts (the last two, and
how the output is written, also depend on the number of heads), ragged last
tiles, against fp64 torch on the
same inputs; and the prefix rows it stores, through the attention of the first
decode step."""
import math

import pytest
import torch

from paper_2605_20600_amd import workloads as W
from paper_2605_20600_amd.runner import DeviceInputs, new_session

pytestmark = pytest.mark.gpu


def _causal(q, k, v):
    C, d = q.shape[-2:]
    s = torch.matmul(q, k.transpose(-1, -2).contiguous()) / math.sqrt(d)
    s = s.masked_fill(~torch.ones((C, C), dtype=torch.bool, device=q.device).tril(), -math.inf)
    return torch.matmul(torch.softmax(s, -1), v)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("C,batch,heads", [
    (2, 1, 3), (31, 2, 4), (32, 1, 5), (33, 1, 5), (63, 1, 3), (64, 3, 4), (65, 1, 3),
    (96, 1, 3), (127, 1, 8), (128, 1, 3), (129, 1, 3), (192, 1, 2), (257, 1, 3),
    (100, 8, 32), (100, 257, 1), (128, 9, 32), (70, 513, 1)])
def test_prefill_tiles(C, batch, heads, d):
    wl = W.LUMINA768.with_(batch=batch, heads=heads, layers=1, head_dim=d, prefix_len=C,
                           grid_rows=2, grid_cols=4, period=5, group_threshold=5,
                           amp_mode="lumina")
    inp = DeviceInputs(wl)
    sess = new_session(wl)
    out = sess.prefill_attn(0, inp.qc[0], inp.kc[0], inp.vc[0])
    q, k, v = (x[0].double() for x in (inp.qc, inp.kc, inp.vc))
    ref = _causal(q, k, v)
    # each weight is rounded to bf16 (relative error up to 2^-9) in the sum and
    # in its normaliser: |o - ref| <= 2^-9 sum p |v - ref| / (1 - 2^-9) <= 2^-8
    # max |v| and its second order; fp32 sums and exp2 add less than 1e-4
    bound = 2.0 ** -8 * 1.01 * v.abs().amax(dim=(-1, -2), keepdim=True) + 1e-4
    assert bool(((out.double() - ref).abs() <= bound).all())
    # every prefix row is in the cache: the first step attends over all of them
    dec = sess.decode_step(0, 0, inp.q[0][0], inp.k[0][0], inp.v[0][0]).double()
    q1 = inp.q[0][0].double()
    k1 = torch.cat((k, inp.k[0][0].double()[:, :, None]), 2)
    v1 = torch.cat((v, inp.v[0][0].double()[:, :, None]), 2)
    w = torch.softmax((k1 * q1[:, :, None]).sum(-1) / math.sqrt(d), -1)
    # fp32 logits, weights and sums of up to C + 1 terms
    assert float((dec - (w[..., None] * v1).sum(2)).abs().max()) <= 2e-5 * float(v1.abs().max())


@pytest.mark.parametrize("d", [64, 128])
def test_prefill_later_infinities(d):
    # infinite values and NaN keys at token 40 and from 96 on stay out of the
    # rows of earlier groups of 32 queries, wherever the key tiles of 64 end
    C, heads = 130, 3
    wl = W.LUMINA768.with_(batch=1, heads=heads, layers=1, head_dim=d, prefix_len=C, grid_rows=2,
                           grid_cols=4, period=5, group_threshold=5)
    inp = DeviceInputs(wl)
    sess = new_session(wl)
    ref = sess.prefill_attn(0, inp.qc[0], inp.kc[0], inp.vc[0])
    for first in (40, 96, 129):
        kc, vc = inp.kc[0].clone(), inp.vc[0].clone()
        vc[:, :, first:] = math.inf
        kc[:, :, first:] = math.nan
        out = sess.prefill_attn(0, inp.qc[0], kc, vc)
        clean = first // 32 * 32
        assert torch.equal(out[:, :, :clean], ref[:, :, :clean])
        assert not bool(torch.isfinite(out[:, :, first:]).any())


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("sign", [1, -1])
@pytest.mark.parametrize("log2q", [4, 12, 20, 40])
def test_prefill_large_scores(log2q, sign, d):
    # scores of 2^15 to 2^51 in log2 units: a last place of the larger ones is
    # worth more than exp2's whole range.  The dot products are exact in fp32
    # (8-bit keys times a power of two), and two keys' scores are at least 184
    # apart, so each row takes one value, that of its largest key so far.
    C, heads = 120, 3
    wl = W.LUMINA768.with_(batch=1, heads=heads, layers=1, head_dim=d, prefix_len=C, grid_rows=2,
                           grid_cols=4, period=5, group_threshold=5)
    gen = torch.Generator().manual_seed(7)
    c = torch.stack([torch.randperm(C, generator=gen) for _ in range(heads)])
    c = (sign * (128 + c).float()).cuda()
    kc = c[None, :, :, None].expand(1, heads, C, d).bfloat16().contiguous()
    qc = torch.full((1, heads, C, d), 2.0 ** log2q, device="cuda").bfloat16()
    vc = torch.randn((1, heads, C, d), generator=gen).cuda().bfloat16()
    out = new_session(wl).prefill_attn(0, qc, kc, vc)
    first = c.cummax(1).indices[None, :, :, None].expand(1, heads, C, d)
    ref = torch.gather(vc.float(), 2, first)
    # one weight w, and its inverse: w v exact, 1 / w and the product rounded
    assert float((out - ref).abs().max()) <= 2.0 ** -22 * float(vc.abs().max())
