"""Attention whose softmax reference follows the maximum lazily: scores that climb by less and by more than the slack per block of
32 keys, all keys of a block alike or one of them alone, and scores that fall; the three forms of the kernel.  Needs a GPU."""
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
@pytest.mark.parametrize("jump", [30.0, 58.0, 75.0, 200.0, -75.0])   # log2 of what later keys have over the first: the sums' limit is 2^60
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
