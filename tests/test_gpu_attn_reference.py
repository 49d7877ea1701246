"""Attention whose softmax reference follows the maximum lazily: scores that climb by less and by more than the slack per block of
32 keys, all keys of a block alike or one of them alone, and scores that fall; the three forms of the kernel.  Importance scores whose
running maximum moves.  Needs a GPU."""
import numpy as np
import pytest
import torch

import oracle
import paper_2603_00198_amd as strd
from paper_2603_00198_amd import synth
from util import TOL, assert_close

pytestmark = pytest.mark.gpu
f = synth.np64


@pytest.mark.parametrize("T,Hq,d", [(250, 2, 128), (700, 2, 64), (700, 4, 128), (3100, 32, 128)])   # one group, two groups, 8 waves
@pytest.mark.parametrize("rise", [0.5, 6.0, 9.0, -6.0])     # log2 of the probability's growth from block to block
@pytest.mark.parametrize("alone", [False, True])
def test_attention_scores_that_climb(T, Hq, d, rise, alone):
    print("[case] attn climb T=%d Hq=%d d=%d rise=%s alone=%s" % (T, Hq, d, rise, alone), flush=True)
    Hkv = 2 if Hq < 8 else 8
    g = torch.Generator().manual_seed(T + d)
    q, k, v = (torch.randn(T, h, d, generator=g) for h in (Hq, Hkv, Hkv))
    q[:, :, 0] = 8.0            # the first channel carries the climb: score = 8 k0 / sqrt(d) + noise
    blocks = torch.arange(T) // 32 % 12
    climb = blocks.float() * rise / 1.4426950408889634 * d ** 0.5 / 8.0
    k[:, :, 0] = torch.where(torch.arange(T) % 32 == 7, climb, torch.zeros(T))[:, None] if alone else climb[:, None]
    q, k, v = (t.to(torch.bfloat16) for t in (q, k, v))
    o = strd.attn_prefill(q.cuda(), k.cuda(), v.cuda())
    heads = [0, Hq - 1]
    kv = [0, Hkv - 1]
    ref = oracle.attn(f(q[:, heads]), f(k[:, kv]), f(v[:, kv]))
    assert_close(f(o[:, heads]), ref, TOL[torch.bfloat16], "o", units=(0, 1))


@pytest.mark.parametrize("N,M,Hq,Hkv,d", [(1500, 20, 4, 2, 128), (1500, 70, 8, 2, 64), (40000, 33, 8, 8, 128)])
@pytest.mark.parametrize("jump", [30.0, 58.0, 75.0, 200.0, -75.0])   # log2 of what later keys have over the first
def test_importance_scores_of_keys_far_above_the_first(N, M, Hq, Hkv, d, jump):
    print("[case] score climb N=%d M=%d d=%d jump=%s" % (N, M, d, jump), flush=True)
    g = torch.Generator().manual_seed(N + d)
    q, k = torch.randn(M, Hq, d, generator=g), torch.randn(N, Hkv, d, generator=g)
    q[:, :, 0] = 16.0
    up = torch.zeros(N)
    up[N // 3:] = jump / 2          # a step within a slice, and lone keys above it
    up[N // 2::97] = jump
    k[:, :, 0] = (up / 1.4426950408889634 * d ** 0.5 / 16.0)[:, None]
    q, k = q.to(torch.bfloat16), k.to(torch.bfloat16)
    s = strd.score_attn(q.cuda(), k.cuda())
    assert_close(s.cpu().numpy(), oracle.score_attn(f(q), f(k)), 1e-4, "scores", units=(0,))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("jump", [30.0, 58.0, 75.0, 200.0, -75.0])
def test_packed_scores_of_keys_far_above_the_first(d, jump):
    """Two tiles of rows per wave and six slices of two chunks of keys, the step in the second chunk of one."""
    N, M, Hq, Hkv, nseq = 1500, 70, 8, 2, 48
    print("[case] packed score climb d=%d jump=%s" % (d, jump), flush=True)
    g = torch.Generator().manual_seed(d)
    q, k = torch.randn(M, Hq, d, generator=g), torch.randn(N, Hkv, d, generator=g)
    q[:, :, 0] = 16.0
    up = torch.zeros(N)
    up[N // 3 + 150:] = jump / 2
    up[N // 2::97] = jump
    k[:, :, 0] = (up / 1.4426950408889634 * d ** 0.5 / 16.0)[:, None]
    q, k = q.to(torch.bfloat16), k.to(torch.bfloat16)
    k_all = torch.cat([k, torch.zeros(M, Hkv, d, dtype=k.dtype)]).cuda().repeat(nseq, 1, 1)
    q_all = torch.cat([torch.zeros(N, Hq, d, dtype=q.dtype), q]).cuda().repeat(nseq, 1, 1)
    s = strd.score_attn_varlen(q_all, k_all, [(N, M, 1)] * nseq)[:, :N]
    assert (s == s[0]).all()
    assert_close(s[0].cpu().numpy(), oracle.score_attn(f(q), f(k)), 1e-4, "scores", units=(0,))


@pytest.mark.parametrize("N,M,Hq,Hkv,d,packed,cut", [(40000, 70, 32, 8, 128, 0, 1280), (65536, 40, 28, 4, 64, 0, 1024),
                                                    (4000, 128, 32, 8, 128, 8, 768)])     # cut: keys per slice of pass 1
@pytest.mark.parametrize("low", [-20.0, -21.5, -23.0, -24.25, -26.0])
def test_importance_scores_lose_no_bits_where_a_few_late_keys_matter(N, M, Hq, Hkv, d, packed, cut, low):
    """The first keys of every slice score 2^-40 to 2^-54 of a few late ones; two tiles of rows per wave.  All rows are
    alike, so that the log-sum-exp's error does not average out, and all products are exact.  In units of log2 a late key's
    weight is off by the rounding of s * scale - lse (< 8: 2^-22) and of lse (< 4: 2^-23, its logarithm an ulp, 2^-22, the scale 2^-23): 2.6e-7
    with ln 2, in quadrature; the sums of up to 16 equal terms per lane add 2e-7.  Half as much again as the two give."""
    print("[case] late keys N=%d M=%d d=%d packed=%d low=%s" % (N, M, d, packed, low), flush=True)
    late = torch.tensor([cut + 300, cut + 450, 3 * cut + 200, 3 * cut + 500, 4 * cut + 700])      # none in the first 128 of a slice
    q, k = torch.zeros(M, Hq, d), torch.zeros(N, Hkv, d)
    q[:, :, 0] = 16.0
    k[:, :, 0] = low * (d / 128) ** 0.5
    k[late, :, 0] = torch.tensor([0.25, -0.5, 0.75, 0.125, -0.3125])[:, None] * (d / 128) ** 0.5
    q, k = q.bfloat16(), k.bfloat16()
    z = f(k[:, 0, 0]) * 16.0 / d ** 0.5
    want = np.exp(z - z.max()) / np.exp(z - z.max()).sum()
    if packed:
        rows = lambda t, n: torch.cat([t.cuda(), torch.zeros(n, *t.shape[1:], dtype=t.dtype, device="cuda")])
        k_all = torch.cat([rows(k, M)] * packed)
        q_all = torch.cat([torch.cat([torch.zeros(N, Hq, d, dtype=q.dtype, device="cuda"), q.cuda()])] * packed)
        s = strd.score_attn_varlen(q_all, k_all, [(N, M, 1)] * packed)
    else:
        s = strd.score_attn(q.cuda(), k.cuda())[None]
    got = f(s[:, :N])[:, late.numpy()]
    assert np.abs(got / want[late.numpy()] - 1).max() <= 5e-7, np.abs(got / want[late.numpy()] - 1).max()
