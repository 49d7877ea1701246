"""The general kernels (fp32 arithmetic, any shape) at the edges of their tiles: one token, a tile, a
chunk and one more; rows of exactly 16, 64, 128 elements, rows with a padded end, rows read element by
element; several key slices and row tiles; with and without a carried state.  Against the fp64 oracle at
a tenth of the fp32 tolerance: sums of at most a few hundred products of 24-bit numbers stay within
1e-5 of the largest result.  Needs a GPU."""
import numpy as np
import pytest
import torch

import oracle
import paper_2603_00198_amd as strd
from paper_2603_00198_amd import synth
from util import TOL, assert_close

pytestmark = pytest.mark.gpu
DEV = "cuda"
f = synth.np64
F32, BF16 = torch.float32, torch.bfloat16
BOUND = {F32: 1e-5, BF16: TOL[BF16]}


def _say(msg):
    print("[case] " + msg, flush=True)


def _draw(seed, dtype):
    g = torch.Generator().manual_seed(seed)
    return lambda *shape: torch.randn(*shape, generator=g).to(dtype)


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("T,d", [(1, 64), (16, 64), (17, 20), (33, 7), (257, 64), (130, 128), (95, 80), (70, 130), (49, 256)])
def test_attention(T, d, dtype):
    if dtype == BF16 and d in (64, 128):
        d += 4   # the bf16 matrix-core kernel owns 64 and 128
    _say("general attn T=%d d=%d %s" % (T, d, dtype))
    rn = _draw(T + d, dtype)
    q, k, v = rn(T, 6, d), rn(T, 3, d), rn(T, 3, d)
    assert_close(f(strd.attn_prefill(q.to(DEV), k.to(DEV), v.to(DEV))), oracle.attn(f(q), f(k), f(v)), BOUND[dtype], "o",
                 units=(0, 1))


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("N,M,Hq,Hkv,d", [(1, 1, 1, 1, 16), (17, 5, 6, 2, 64), (300, 23, 4, 4, 12), (2100, 40, 8, 2, 128),
                                          (129, 9, 3, 1, 130), (65, 700, 8, 2, 33)])
def test_score_attn(N, M, Hq, Hkv, d, dtype):
    if dtype == BF16 and d in (64, 128):
        d += 4
    _say("general score_attn N=%d M=%d Hq=%d Hkv=%d d=%d %s" % (N, M, Hq, Hkv, d, dtype))
    rn = _draw(N + M, dtype)
    q, k = rn(M, Hq, d), rn(N, Hkv, d)
    assert_close(f(strd.score_attn(q.to(DEV), k.to(DEV))), oracle.score_attn(f(q), f(k)), BOUND[dtype], "s", units=(0,))


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("N,M,G,H,n", [(1, 1, 1, 1, 1), (33, 16, 1, 8, 16), (100, 37, 3, 6, 20), (47, 200, 2, 10, 128),
                                       (260, 5, 8, 8, 130)])
def test_score_mamba(N, M, G, H, n, dtype):
    if dtype == BF16 and n in (64, 128):
        n -= 4
    _say("general score_mamba N=%d M=%d G=%d H=%d n=%d %s" % (N, M, G, H, n, dtype))
    rn = _draw(N + M, dtype)
    B, C, dt = rn(N, G, n), rn(M, G, n), torch.nn.functional.softplus(_draw(N, F32)(N, H))
    assert_close(f(strd.score_mamba(B.to(DEV), C.to(DEV), dt.to(DEV))), oracle.score_mamba(f(B), f(C), f(dt)), BOUND[dtype],
                 "s", units=(0,))


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("carry", [True, False])
@pytest.mark.parametrize("T,H,P,G,n", [(0, 2, 32, 1, 16), (1, 2, 32, 1, 16), (64, 4, 64, 2, 64), (65, 3, 20, 1, 40),
                                       (200, 2, 80, 1, 128), (130, 2, 33, 2, 7), (577, 8, 32, 1, 16), (129, 1, 64, 1, 200)])
def test_scan(T, H, P, G, n, carry, dtype):
    if dtype == BF16 and n in (64, 128):
        n -= 4
    _say("general scan T=%d H=%d P=%d G=%d n=%d carry=%s %s" % (T, H, P, G, n, carry, dtype))
    rn, r32 = _draw(T + P, dtype), _draw(T + n, F32)
    x, B, C = rn(T, H, P), rn(T, G, n), rn(T, G, n)
    dt = torch.nn.functional.softplus(r32(T, H))
    A = -torch.exp(2 * torch.rand(H, generator=torch.Generator().manual_seed(T)))
    D, S_in = (r32(H), r32(H, P, n)) if carry else (None, None)
    dev = lambda t: None if t is None else t.to(DEV)
    y, S = strd.ssd_prefill(dev(x), dev(dt), dev(A), dev(B), dev(C), dev(D), dev(S_in))
    if T == 0:
        assert torch.equal(S.cpu(), S_in if carry else torch.zeros(H, P, n))
        return
    y_ref, S_ref = oracle.ssd_seq(f(x), f(dt), f(A), f(B), f(C), None if D is None else f(D), None if S_in is None else f(S_in))
    assert_close(f(y), y_ref, BOUND[dtype], "y", units=(1,))
    assert_close(f(S), S_ref, 1e-5 if dtype == F32 else BOUND[dtype], "S", units=(0,))
    y2, none = strd.ssd_prefill(dev(x), dev(dt), dev(A), dev(B), dev(C), dev(D), dev(S_in), want_state=False)
    assert none is None and torch.equal(y2, y)


@pytest.mark.parametrize("H,P,G,n,carry", [(8, 32, 1, 16, False), (8, 64, 2, 64, True), (4, 48, 1, 128, True), (4, 40, 2, 256, True),
                                           (4, 33, 1, 30, True)])
def test_scan_in_single_precision_is_as_exact_as_the_recurrence(H, P, G, n, carry):
    """The distance from 64 bits over all outputs (2-norm): a few roundings of 2^-24 that do not grow with the row
    length.  The token-by-token recurrence is 0.9 to 1.05e-7 off here; a weight in one chain of n products 1.1 to 2.9e-7."""
    _say("scan, distance from 64 bits, H=%d P=%d n=%d" % (H, P, n))
    T = 300
    g = torch.Generator().manual_seed(n)
    rn = lambda *shape: torch.randn(*shape, generator=g)
    x, B, C = rn(T, H, P), rn(T, G, n), rn(T, G, n)
    dt, A = torch.nn.functional.softplus(rn(T, H)), -torch.exp(2 * torch.rand(H, generator=g))
    D, S_in = (rn(H), rn(H, P, n)) if carry else (None, None)
    dev = lambda t: None if t is None else t.to(DEV)
    y, S = strd.ssd_prefill(dev(x), dev(dt), dev(A), dev(B), dev(C), dev(D), dev(S_in))
    y_ref, S_ref = oracle.ssd_seq(f(x), f(dt), f(A), f(B), f(C), f(D) if carry else None, f(S_in) if carry else None)
    assert np.linalg.norm(f(y) - y_ref) < 1.05e-7 * np.linalg.norm(y_ref)
    assert np.linalg.norm(f(S) - S_ref) < 6e-8 * np.linalg.norm(S_ref)


@pytest.mark.parametrize("T", [2368, 2369, 2432, 2433, 4100, 7936, 7937, 8200])
def test_scan_around_the_switch_to_segments(T):
    """128 heads of 64 channels: up to 124 steps of 64 tokens run in one piece (no workspace), 125 and more in four
    segments of 32 and more (the last one shorter).  The first and the last group's heads against the recurrence, the
    gather form bit for bit."""
    _say("scan, 128 heads, T=%d" % T)
    H, P, G, n, M = 128, 64, 8, 128, 33
    assert (strd.lib().strd_ssd_prefill_workspace(T, H, P, G, n, 256, 1) > 0) == (T > 124 * 64)
    g = torch.Generator().manual_seed(T)
    rows = T + 57
    x = torch.randn(rows, H, P, generator=g).to(BF16)
    B, C = (torch.randn(rows, G, n, generator=g) / n ** 0.5).to(BF16), torch.randn(rows, G, n, generator=g).to(BF16)
    dt = torch.nn.functional.softplus(torch.randn(rows, H, generator=g))
    A, D, S_in = -torch.exp(2 * torch.rand(H, generator=g)), torch.randn(H, generator=g), torch.randn(H, P, n, generator=g)
    N, K = rows - M, T - M
    idx = torch.sort(torch.randperm(N, generator=g)[:K]).values.int()
    keep = torch.cat([idx.long(), torch.arange(N, rows)])
    dev = lambda t: t.to(DEV)
    y, S = strd.ssd_prefill(*(dev(t[keep].contiguous()) for t in (x, dt)), dev(A), *(dev(t[keep].contiguous()) for t in (B, C)),
                            dev(D), dev(S_in))
    yg, Sg = strd.ssd_prefill_gather(dev(x), dev(dt), dev(A), dev(B), dev(C), dev(idx), N, M, dev(D), dev(S_in))
    assert torch.equal(yg, y) and torch.equal(Sg, S)
    for h0, grp in ((0, 0), (126, 7)):
        hs = slice(h0, h0 + 2)
        y_ref, S_ref = oracle.ssd_seq(f(x[keep][:, hs]), f(dt[keep][:, hs]), f(A[hs]), f(B[keep][:, grp:grp + 1]),
                                      f(C[keep][:, grp:grp + 1]), f(D[hs]), f(S_in[hs]))
        assert_close(f(y[:, hs]), y_ref, TOL[BF16], "y", units=(1,))
        assert_close(f(S[hs]), S_ref, TOL[BF16], "S", units=(0,))


WHOLE, HALVES, QUARTERS = 0, 1, 2   # strd_linear_mfma_cut


# token rows x columns whose last round of 256 tiles is cut into quarters: one tile; an edge row of one token; a row of
# tiles; edge row, edge column and corner; a column just over half full (not an edge); 155 tiles, left whole; 48 tiles of an
# edge row; an edge column of 8
@pytest.mark.parametrize("T,Nd", [(256, 256), (4097, 4096), (4096 + 256, 4096), (4096 + 100, 4096 + 64), (4096, 4096 + 136),
                                  (5 * 256, 31 * 256), (9 * 256 + 5, 56 * 256), (12 * 256, 44 * 256 + 8)])
def test_projection_with_a_cut_last_round(T, Nd):
    """Every element against the fp32 product of the same bf16 operands: one bf16 step of the result plus the
    rounding of 64 sums of products of standard normals (under 1e-5)."""
    _say("projection T=%d Nd=%d" % (T, Nd))
    Kd = 64
    g = torch.Generator(device=DEV).manual_seed(T + Nd)
    x = torch.randn(T, Kd, generator=g, device=DEV).to(BF16)
    w = torch.randn(Kd, Nd, generator=g, device=DEV).to(BF16)
    res = torch.randn(T, Nd, generator=g, device=DEV).to(BF16)
    out = torch.full((T + 1, Nd), 7.0, device=DEV, dtype=BF16)
    strd.linear_mfma(x, w, residual=res, out=out[:T])
    ref = x.float() @ w.float() + res.float()
    err = (out[:T].float() - ref).abs()
    assert bool((err <= ref.abs() * 2.0 ** -8 + 1e-4).all()), float(err.max())
    assert bool((out[T] == 7.0).all()), "wrote past the last row"


@pytest.mark.parametrize("Kd", [64, 128, 192, 1088])
@pytest.mark.parametrize("T,Nd,cut", [(1280, 4096, HALVES), (1273, 4096 - 8, HALVES), (3000, 8192, HALVES), (2176, 10368, HALVES),
                                      (2049, 10248, HALVES), (1280 - 7, 7936 - 24, WHOLE), (4096 - 3, 4096 - 40, WHOLE),
                                      (4096 + 100, 4096 + 64, QUARTERS), (300, 1000, QUARTERS)])
def test_projection_by_kind_of_cut_and_depth(T, Nd, cut, Kd):
    """Whole tiles, halves (alone, ragged, with an edge row and an edge column of tiles) and quarters; two, four and six
    stages of the copy ring, and many.  Every element against 64 bits: half a bf16 step of the result (and of the sum
    without the residual) and Kd roundings of 2^-24 of the sum of magnitudes, 0.64 Kd."""
    _say("projection T=%d Nd=%d Kd=%d cut=%d" % (T, Nd, Kd, cut))
    assert strd.lib().strd_linear_mfma_cut(T, Nd) == cut
    g = torch.Generator(device=DEV).manual_seed(T + Nd + Kd)
    x = torch.randn(T, Kd, generator=g, device=DEV).to(BF16)
    w = torch.randn(Kd, Nd, generator=g, device=DEV).to(BF16)
    res = torch.randn(T, Nd, generator=g, device=DEV).to(BF16)
    out = torch.full((T + 1, Nd), 7.0, device=DEV, dtype=BF16)
    out[:T] = res
    strd.linear_mfma(x, w, residual=out[:T], out=out[:T])
    ref = x.double() @ w.double() + res.double()
    err = (out[:T].double() - ref).abs() - (ref.abs() * 2.0 ** -8 + Kd * 2.0 ** -24 * Kd)
    assert bool((err <= 0).all()), float(err.max())
    assert bool((out[T] == 7.0).all()), "wrote past the last row"


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("T", [256, 257, 288, 320, 321, 385, 448, 515, 1021])
def test_attention_with_two_key_groups(T, d):
    """Sequences of a few 64-key chunks: one group of waves up to 256 tokens, two from there on (an even and an odd
    number of chunks, a last chunk of one key, query tiles that see no key of the second group)."""
    _say("attn, key groups, T=%d d=%d" % (T, d))
    rn = _draw(T + d, BF16)
    q, k, v = rn(T, 4, d), rn(T, 2, d), rn(T, 2, d)
    assert_close(f(strd.attn_prefill(q.to(DEV), k.to(DEV), v.to(DEV))), oracle.attn(f(q), f(k), f(v)), TOL[BF16], "o",
                 units=(0, 1))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("T,Hq", [(300, 170), (300, 184), (641, 84), (641, 96)])
def test_attention_past_two_rounds_of_workgroups(T, Hq, d):
    """More than 512 blocks of 128 queries, one group of waves per workgroup again; fewer, two."""
    _say("attn, rounds, T=%d Hq=%d d=%d" % (T, Hq, d))
    rn = _draw(T + d, BF16)
    q, k, v = rn(T, Hq, d), rn(T, 2, d), rn(T, 2, d)
    assert_close(f(strd.attn_prefill(q.to(DEV), k.to(DEV), v.to(DEV))), oracle.attn(f(q), f(k), f(v)), TOL[BF16], "o",
                 units=(0, 1))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("N,M,Hq,Hkv", [(1, 1, 2, 2), (127, 3, 4, 2), (1024, 65, 4, 2), (1025, 17, 6, 2), (2048, 128, 8, 4),
                                        (2048, 129, 8, 4), (16384, 5, 4, 2), (16385, 5, 4, 2), (16385, 40, 4, 2)])
def test_score_attn_narrow_and_fused(N, M, Hq, Hkv, d):
    """Column sums with 128 and with 256 keys per workgroup (the line is at 128 workgroups of 256), and with the
    slices of a row combined there (up to 4096 pairs per kv head, eight in flight) or in a launch of their own."""
    _say("score_attn N=%d M=%d Hq=%d Hkv=%d d=%d" % (N, M, Hq, Hkv, d))
    rn = _draw(N + M + d, BF16)
    q, k = rn(M, Hq, d), rn(N, Hkv, d)
    assert_close(f(strd.score_attn(q.to(DEV), k.to(DEV))), oracle.score_attn(f(q), f(k)), TOL[BF16], "s", units=(0,))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("rep", [1, 2, 4, 8])
def test_decode_attention_trips(rep, d):
    """bf16 cache, trips of 16 tokens by four waves: one token, a trip and one more, a round of the waves and one
    more, slices longer than a round whose last wave has a trip less, an even and an odd number of trips."""
    for T, Hkv in ((1, 2), (16, 2), (17, 1), (64, 2), (65, 2), (16 * 256 * 5 + 3, 1), (16 * 64 * 9, 8), (16 * 64 * 9 + 1, 8)):
        _say("attn_decode_step T=%d Hkv=%d rep=%d d=%d" % (T, Hkv, rep, d))
        rn = _draw(T + rep + d, BF16)
        q, k, v = rn(Hkv * rep, d), rn(T, Hkv, d), rn(T, Hkv, d)
        k[T // 2] = (3 * q.float().view(Hkv, rep, d)[:, 0]).to(BF16)   # the first head of each group: a peaked row
        assert_close(f(strd.attn_decode_step(q.to(DEV), k.to(DEV), v.to(DEV))), oracle.attn_decode_step(f(q), f(k), f(v)),
                     TOL[BF16], "o", units=(0,))


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("T,d", [(20, 20), (33, 64), (64, 7), (77, 128), (300, 48), (70, 130), (35, 256)])
def test_attention_keeps_non_finite_rows_to_themselves(T, d, dtype):
    """One inf or NaN in v at token s is no business of the tokens before s, of the other channels or of the other kv
    head: they have the same bits as with 0 in its place (its probability does not change).  From s on its channel
    is not finite.  The same for the whole row of k at s, which makes rows from s on NaN."""
    if dtype == BF16 and d in (64, 128):
        d += 4
    rn = _draw(T + d, dtype)
    q, k, v = rn(T, 4, d).to(DEV), rn(T, 2, d).to(DEV), rn(T, 2, d).to(DEV)
    c = d // 2 - 1
    for s in sorted({1, 15, 16, 17, T // 2, T - 2, T - 1}):
        for bad in (float("inf"), float("nan")):
            _say("attn T=%d d=%d %s, %f at %d" % (T, d, dtype, bad, s))
            clean, dirty = v.clone(), v.clone()
            clean[s, 1, c], dirty[s, 1, c] = 0.0, bad
            want, got = strd.attn_prefill(q, k, clean), strd.attn_prefill(q, k, dirty)
            assert not bool(torch.isfinite(got[s:, 2:, c]).any())
            got[s:, 2:, c] = want[s:, 2:, c]
            assert torch.equal(got, want)
        kd = k.clone()
        kd[s, 1] = float("nan")
        want, got = strd.attn_prefill(q, k, v), strd.attn_prefill(q, kd, v)
        assert bool(torch.isnan(got[s:, 2:]).all())
        got[s:, 2:] = want[s:, 2:]
        assert torch.equal(got, want)


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("T,H,P,G,n", [(20, 2, 32, 1, 16), (64, 2, 64, 1, 64), (100, 2, 20, 1, 40), (130, 2, 33, 2, 7),
                                       (145, 2, 80, 1, 128)])
def test_scan_keeps_non_finite_rows_to_themselves(T, H, P, G, n, dtype):
    """One inf or NaN in x at token s is no business of the tokens before s, of the other channels or of the other
    head: they have the same bits as with 0 in its place; from s on its channel is not finite, nor is its state.  The
    last token's inf leaves an infinite state (no row past the end is added to it)."""
    if dtype == BF16 and n in (64, 128):
        n -= 4
    rn, r32 = _draw(T + P, dtype), _draw(T + n, F32)
    x, B, C = rn(T, H, P).to(DEV), rn(T, G, n).to(DEV), rn(T, G, n).to(DEV)
    dt, A, D = torch.nn.functional.softplus(r32(T, H)).to(DEV), -0.1 * torch.ones(H, device=DEV), r32(H).to(DEV)
    p = P // 2 - 1
    for s in sorted({1, 15, 16, 17, T // 2, T - 2, T - 1}):
        for bad in (float("inf"), float("nan")):
            _say("scan T=%d P=%d n=%d %s, %f at %d" % (T, P, n, dtype, bad, s))
            clean, dirty = x.clone(), x.clone()
            clean[s, 1, p], dirty[s, 1, p] = 0.0, bad
            (want, Sw), (got, Sg) = (strd.ssd_prefill(t, dt, A, B, C, D) for t in (clean, dirty))
            assert not bool(torch.isfinite(got[s:, 1, p]).any()) and not bool(torch.isfinite(Sg[1, p]).any())
            if s == T - 1 and bad == float("inf"):
                assert bool((Sg[1, p] == torch.sign(B[s, G - 1].float()) * bad).all())
            got[s:, 1, p], Sg[1, p] = want[s:, 1, p], Sw[1, p]
            assert torch.equal(got, want) and torch.equal(Sg, Sw)


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("T", [1, 63, 64, 65, 200])
def test_scan_without_memory(T, dtype):
    """A = -inf: every decay is exp(-inf) = 0, a token sees only itself.  Beside it a head whose decays are below every
    number (the same result), a usual one, and an incoming state that goes at once."""
    _say("scan, A = -inf, T=%d %s" % (T, dtype))
    H, P, n = 3, 20, 12
    rn, r32 = _draw(T, dtype), _draw(T + 1, F32)
    x, B, C = rn(T, H, P), rn(T, 1, n), rn(T, 1, n)
    dt, D, S_in = 0.1 + torch.nn.functional.softplus(r32(T, H)), r32(H), r32(H, P, n)
    A = torch.tensor([float("-inf"), -1e30, -1.0])
    dev = lambda t: t.to(DEV)
    for carry in (False, True):
        y, S = strd.ssd_prefill(*(dev(t) for t in (x, dt, A, B, C, D)), dev(S_in) if carry else None)
        y_ref, S_ref = oracle.ssd_seq(f(x), f(dt), np.maximum(f(A), -1e30), f(B), f(C), f(D), f(S_in) if carry else None)
        assert_close(f(y), y_ref, BOUND[dtype], "y", units=(1,))
        assert_close(f(S), S_ref, BOUND[dtype], "S", units=(0,))


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("dead", [100, 1024, 1150, 2047])
@pytest.mark.parametrize("M", [16, 300])
def test_score_attn_with_keys_no_query_can_see(M, dead, dtype):
    """The first `dead` keys score -inf with every query: whole slices of the keys (128 of them in the bf16 kernel,
    eight combined at a time up to 4096 pairs, in a launch of their own beyond) have neither maximum nor sum."""
    _say("score_attn, %d keys at -inf, M=%d %s" % (dead, M, dtype))
    rn = _draw(M + dead, dtype)
    q, k = rn(M, 2, 64).abs() + 0.1, rn(2048, 2, 64)
    k[:dead] = float("-inf")
    got = f(strd.score_attn(q.to(DEV), k.to(DEV)))
    want = oracle.score_attn(f(q), np.where(np.isfinite(f(k)), f(k), -1e30))
    assert (got[:dead] == 0.0).all()
    assert_close(got, want, BOUND[dtype], "s", units=(0,))


def _scan_inputs(T, H, P, G, n, dtype, seed):
    rn, r32 = _draw(seed, dtype), _draw(seed + 1, F32)
    x, B, C = rn(T, H, P), rn(T, G, n), rn(T, G, n)
    return x, torch.nn.functional.softplus(r32(T, H)), -torch.exp(2 * torch.rand(H, generator=torch.Generator().manual_seed(T))), \
        B, C, r32(H), r32(H, P, n)


@pytest.mark.parametrize("T", [1024, 1025, 2048, 2118])
def test_scan_in_rounds_of_chunks(T):
    """64 heads of 64 x 1024: 16 chunks of 64 tokens make a round.  One round, one and a token, two, two and a part;
    the first and the last head against the recurrence."""
    _say("general scan in rounds, T=%d" % T)
    t = _scan_inputs(T, 64, 64, 1, 1024, F32, T)
    x, dt, A, B, C, D, S_in = (v.to(DEV) for v in t)
    y, S = strd.ssd_prefill(x, dt, A, B, C, D, S_in)
    y0, _ = strd.ssd_prefill(x, dt, A, B, C, D, None, want_state=False)
    for h in (0, 63):
        hs = slice(h, h + 1)
        rows = (f(t[0][:, hs]), f(t[1][:, hs]), f(t[2][hs]), f(t[3]), f(t[4]), f(t[5][hs]))
        y_ref, S_ref = oracle.ssd_seq(*rows, f(t[6][hs]))
        assert_close(f(y[:, hs]), y_ref, BOUND[F32], "y", units=(1,))
        assert_close(f(S[hs]), S_ref, BOUND[F32], "S", units=(0,))
        assert_close(f(y0[:, hs]), oracle.ssd_seq(*rows, None)[0], BOUND[F32], "y from zero", units=(1,))


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("T,H,P,G,n", [(1, 2, 32, 1, 16), (65, 3, 20, 1, 40), (200, 2, 80, 1, 130), (577, 8, 32, 1, 16)])
def test_scan_without_a_workspace(T, H, P, G, n, dtype):
    """A caller that brings none, or too little, gets the recurrence."""
    _say("general scan without a workspace, T=%d P=%d n=%d %s" % (T, P, n, dtype))
    t = _scan_inputs(T, H, P, G, n, dtype, T + n)
    dev = [v.to(DEV) for v in t]
    y_ref, S_ref = oracle.ssd_seq(*(f(v) for v in t))
    y, S = strd.ssd_prefill(*dev, ws=torch.empty(16, dtype=torch.uint8, device=DEV))
    y2, S2 = torch.empty_like(y), torch.empty_like(S)
    ptr = [v.data_ptr() for v in dev]
    assert strd.lib().strd_ssd_prefill(*ptr, y2.data_ptr(), S2.data_ptr(), T, H, P, G, n, 256,
                                       0 if dtype == F32 else 1, None, 0, torch.cuda.current_stream().cuda_stream) == 0
    assert torch.equal(y, y2) and torch.equal(S, S2)
    assert_close(f(y), y_ref, BOUND[dtype], "y", units=(1,))
    assert_close(f(S), S_ref, BOUND[dtype], "S", units=(0,))


@pytest.mark.parametrize("d,dtype,Hq,T", [(33, F32, 16, 22), (33, BF16, 16, 116), (72, F32, 16, 65), (128, F32, 16, 32),
                                          (65, F32, 16, 150), (127, BF16, 16, 291), (200, F32, 16, 187), (136, BF16, 16, 206),
                                          (256, F32, 16, 76), (256, BF16, 16, 129), (130, F32, 16, 206), (255, BF16, 16, 412),
                                          (130, F32, 2, 600), (250, BF16, 1, 1025)])
def test_attention_by_rows_and_by_tiles(d, dtype, Hq, T):
    """The longest sequence that goes row by row, and one token more, in tiles.  One NaN in v stays with its own and
    later queries, its channel and its kv head: the rest has the same bits as with 0 in its place."""
    for n in (T, T + 1):
        _say("attn, rows and tiles, d=%d %s Hq=%d T=%d" % (d, dtype, Hq, n))
        rn, Hkv = _draw(n + d, dtype), 1 if Hq == 1 else 2
        q, k, v = rn(n, Hq, d), rn(n, Hkv, d), rn(n, Hkv, d)
        q, k, v, v_host = q.to(DEV), k.to(DEV), v.to(DEV), v
        o = strd.attn_prefill(q, k, v)
        assert_close(f(o), oracle.attn(f(q), f(k), f(v_host)), BOUND[dtype], "o", units=(0, 1))
        for s in (n // 2, n - 2):
            clean, dirty = v.clone(), v.clone()
            clean[s, -1, d - 1], dirty[s, -1, d - 1] = 0.0, float("nan")
            want, got = strd.attn_prefill(q, k, clean), strd.attn_prefill(q, k, dirty)
            mine = slice(Hq - Hq // Hkv, Hq)
            assert bool(torch.isnan(got[s:, mine, d - 1]).all())
            got[s:, mine, d - 1] = want[s:, mine, d - 1]
            assert torch.equal(got, want)


def test_attention_with_rows_of_16_megabytes():
    """65536 heads of 64: rows past what a 24-bit product reaches (and one head less: rows just below it)."""
    T, d = 35, 64
    for H in (65535, 65536):
        _say("attn, %d heads" % H)
        q, k, v = (torch.randn(T, H, d, device=DEV, generator=torch.Generator(device=DEV).manual_seed(H + i)) for i in range(3))
        o = strd.attn_prefill(q, k, v)
        for h in (0, H // 2, H - 1):
            hs = slice(h, h + 1)
            assert_close(f(o[:, hs]), oracle.attn(f(q[:, hs]), f(k[:, hs]), f(v[:, hs])), BOUND[F32], "o", units=(0,))


def test_scan_with_a_state_of_a_gigabyte():
    """4097 heads of 64 x 1024, one more than the chunks' launches take: the recurrence, with or without a workspace."""
    _say("general scan, 4097 heads of 64 x 1024")
    t = _scan_inputs(3, 4097, 64, 1, 1024, F32, 5)[:-1]
    y, S = strd.ssd_prefill(*(v.to(DEV) for v in t))
    for h in (0, 4096):
        hs = slice(h, h + 1)
        y_ref, S_ref = oracle.ssd_seq(f(t[0][:, hs]), f(t[1][:, hs]), f(t[2][hs]), f(t[3]), f(t[4]), f(t[5][hs]), None)
        assert_close(f(y[:, hs]), y_ref, BOUND[F32], "y", units=(1,))
        assert_close(f(S[hs]), S_ref, BOUND[F32], "S", units=(0,))


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("H,P,G,n,last", [(8, 32, 1, 16, 5), (3, 33, 1, 7, 5), (8, 64, 1, 130, 4), (256, 20, 1, 40, 8), (128, 64, 8, 256, 2),
                                          (2, 20, 1, 512, 6), (2, 20, 1, 1024, 8)])
def test_scan_of_a_few_tokens(H, P, G, n, last, dtype):
    """Token by token up to `last` (no workspace), in chunks from one more."""
    for T in (1, last, last + 1):
        _say("general scan, T=%d H=%d P=%d n=%d %s" % (T, H, P, n, dtype))
        ws = strd.lib().strd_ssd_prefill_workspace(T, H, P, G, n, 256, 0 if dtype == F32 else 1)
        assert (ws == 0) == (T <= last)
        t = _scan_inputs(T, H, P, G, n, dtype, T + n)
        y, S = strd.ssd_prefill(*(v.to(DEV) for v in t))
        y_ref, S_ref = oracle.ssd_seq(*(f(v) for v in t))
        assert_close(f(y), y_ref, BOUND[dtype], "y", units=(1,))
        assert_close(f(S), S_ref, BOUND[dtype], "S", units=(0,))


@pytest.mark.parametrize("H,P,G,n,T", [(8, 64, 1, 128, 1000), (24, 64, 1, 128, 1990), (24, 64, 1, 64, 4000), (30, 128, 2, 128, 3001),
                                       (60, 64, 2, 128, 3000), (60, 64, 2, 64, 5999), (4, 32, 1, 64, 1100)])
def test_scan_with_few_heads_and_slow_decays(H, P, G, n, T):
    """The incoming state lives through every tile of its segment; one, two or four workgroups repair it.  The first and
    the last head against the recurrence, through the index list bit for bit."""
    _say("scan, seams, H=%d P=%d n=%d T=%d" % (H, P, n, T))
    assert strd.lib().strd_ssd_prefill_workspace(T, H, P, G, n, 256, 1) > 0
    g = torch.Generator().manual_seed(T)
    x = torch.randn(T, H, P, generator=g).to(BF16)
    B, C = (torch.randn(T, G, n, generator=g) / n ** 0.5).to(BF16), torch.randn(T, G, n, generator=g).to(BF16)
    dt, A = torch.rand(T, H, generator=g), -0.002 * (0.5 + torch.rand(H, generator=g))
    D, S_in = torch.randn(H, generator=g), torch.randn(H, P, n, generator=g)
    dev = [t.to(DEV) for t in (x, dt, A, B, C)]
    y, S = strd.ssd_prefill(*dev, D.to(DEV), S_in.to(DEV))
    N = T - 40
    yg, Sg = strd.ssd_prefill_gather(*dev, torch.arange(N, dtype=torch.int32, device=DEV), N, 40, D.to(DEV), S_in.to(DEV))
    assert torch.equal(yg, y) and torch.equal(Sg, S)
    for h in (0, H - 1):
        hs, gs = slice(h, h + 1), slice(h * G // H, h * G // H + 1)
        y_ref, S_ref = oracle.ssd_seq(f(x[:, hs]), f(dt[:, hs]), f(A[hs]), f(B[:, gs]), f(C[:, gs]), f(D[hs]), f(S_in[hs]))
        assert_close(f(y[:, hs]), y_ref, TOL[BF16], "y", units=(1,))
        assert_close(f(S[hs]), S_ref, TOL[BF16], "S", units=(0,))


@pytest.mark.parametrize("M,Hq,Hkv,d", [(1, 1, 1, 64), (4, 8, 2, 128), (85, 1, 1, 64), (86, 1, 1, 64)])
@pytest.mark.parametrize("N", [5888, 6016, 6144, 6145, 6300])
def test_score_attn_around_the_rule_for_combined_slices(N, M, Hq, Hkv, d):
    """Up to 48 slices of 128 keys (and 4096 pairs of a slice and a row) combined in pass 2, more in a launch."""
    _say("score_attn, slices, M=%d N=%d" % (M, N))
    rn = _draw(N + M, BF16)
    q, k = rn(M, Hq, d), rn(N, Hkv, d)
    assert_close(f(strd.score_attn(q.to(DEV), k.to(DEV))), oracle.score_attn(f(q), f(k)), BOUND[BF16], "s", units=(0,))


# ------------------------------------------------------------------ selection --------------
@pytest.mark.parametrize("in_bin", [4095, 4096, 4097, 30000])
@pytest.mark.parametrize("N,low_bits", [(65536, 11), (65537, 12), (131072, 13), (131072 + 5, 21), (1 << 20, 21)])
def test_select_topk_many_candidates_after_two_digits(N, low_bits, in_bin):
    """Scores built from their bit patterns so that the first two 11-bit digits of key - min(key) leave `in_bin` keys
    (the list holds 4096) that differ in the bits below, none to ten: threshold values in and around them."""
    _say("topk, two digits, N=%d low_bits=%d in_bin=%d" % (N, low_bits, in_bin))
    r = np.random.default_rng(in_bin + low_bits)
    third = max(low_bits - 11, 0)
    off = r.integers(0, 1 << (11 + low_bits), N)
    off[off >> low_bits == 700] += 1 << low_bits
    where = r.choice(np.arange(2, N), in_bin + N // 8, replace=False)
    # an eighth more keys share the first digit only
    off[where] = (700 << low_bits) + r.integers(0, 1 << low_bits, len(where))
    same = where[:in_bin]
    off[same] = (700 << low_bits) + (5 << third) + r.integers(0, 1 << third, in_bin)
    off[0], off[1] = 0, (1 << (11 + low_bits)) - 1
    off = np.minimum(off, 0xFF7FFFFF - 0x00800001)    # at 32 bits: the finite floats
    key = (np.uint64(0x00800001) + off.astype(np.uint64)).astype(np.uint32)
    s = np.where(key & np.uint32(0x80000000), key ^ np.uint32(0x80000000), ~key).astype(np.uint32).view(np.float32)
    above = int((off >= (700 << low_bits) + (6 << third)).sum())
    for K in (above, above + 1, above + in_bin // 2, above + in_bin, above + in_bin + 1):
        got = strd.select_topk(torch.from_numpy(s).to(DEV), K).cpu().numpy()
        np.testing.assert_array_equal(got, oracle.select_topk(s.astype(np.float64), K))


@pytest.mark.parametrize("N", [49152, 65536, 131072, 1 << 20])
def test_selection_time_does_not_hang_on_the_values(N):
    """Close scores beside a zero, and two values: right, and not several times slower than scores that spread out
    (measured 1.3 times at most; workgroups that read one another's scores, or a list of one value, made it 3 to 12)."""
    _say("topk, time by values, N=%d" % N)
    g = torch.Generator().manual_seed(N)
    u = torch.rand(N, generator=g)
    close, two = 1e-5 * (1.0 + 1e-4 * u), torch.full((N,), 1e-5)
    close[7] = 0.0
    two[::2] = 0.0

    def micros(s):
        best = float("inf")
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                strd.select_topk(s, N // 4)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) * 50.0)
        return best

    base = micros(u.to(DEV))
    for s in (close, two):
        got = strd.select_topk(s.to(DEV), N // 4).cpu().numpy()
        np.testing.assert_array_equal(got, oracle.select_topk(s.numpy().astype(np.float64), N // 4))
        assert micros(s.to(DEV)) < 2.0 * base


# ------------------------------------------------------------------ binding ----------------
def test_numbers_that_are_not_whole_or_do_not_fit_are_refused():
    """The binding takes what has __index__ and fits 32 bits, as torch and ctypes do: nothing is cut to size."""
    _say("binding, numbers")
    s, idx = torch.rand(64, device=DEV), torch.arange(4, dtype=torch.int32, device=DEV)
    t, x = torch.zeros(8, 2, device=DEV), torch.zeros(8, 2, 4, device=DEV)
    dt, A, bc = torch.zeros(8, 2, device=DEV), torch.zeros(2, device=DEV), torch.zeros(8, 1, 4, device=DEV)
    for K in (2.7, "2", 2 ** 32 + 5, 2 ** 70, None):
        with pytest.raises((strd.StrdError, TypeError)):
            strd.select_topk(s, K)
        with pytest.raises((strd.StrdError, TypeError)):
            strd.compact_batch([t], idx, K, 4)
        with pytest.raises((strd.StrdError, TypeError)):
            strd.ssd_prefill(x, dt, A, bc, bc, chunk=K)
    with pytest.raises((strd.StrdError, TypeError)):
        strd.compact_batch([t], idx, 2 ** 32 + 4, 4)
    with pytest.raises((strd.StrdError, TypeError)):
        strd.select_topk_varlen(torch.rand(1, 8, device=DEV), [(2 ** 32 + 8, 1, 2)])
    assert strd.select_topk(s, np.int64(3)).shape == (3,) and strd.select_topk(s, torch.tensor(3)).shape == (3,)
    assert strd.select_topk_varlen(s[None], [(64.0, 1, np.float64(3))]).shape == (3,)   # descriptors go through int()


def test_compaction_takes_tensors_of_any_number_of_dimensions():
    """Rows of nine and ten dimensions, an index column, and more outputs than tensors (all of them come back)."""
    _say("binding, dimensions")
    idx = torch.tensor([1, 4], dtype=torch.int32, device=DEV)
    keep = torch.tensor([1, 4, 6, 7], device=DEV)
    a = torch.randn(8, *[1, 2] * 4, device=DEV)
    b = torch.randn(8, *[2, 1, 1] * 3, device=DEV).to(BF16)
    for index in (idx, idx[:, None]):
        (ca, cb), none = strd.compact_batch([a, b], index, 6, 2)
        assert none is None and torch.equal(ca, a[keep]) and torch.equal(cb, b[keep])
        (ca,), _ = strd.compact_varlen([a], index, [(6, 2, 2)])
        assert torch.equal(ca, a[keep])
    outs = [torch.empty(4, *a.shape[1:], device=DEV), torch.zeros(3, device=DEV)]
    got, _ = strd.compact_batch([a], idx, 6, 2, outs=outs)
    assert len(got) == 2 and got[0] is outs[0] and got[1] is outs[1] and torch.equal(got[0], a[keep])


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("T,H,P,G,n", [(9, 8, 32, 1, 16), (64 * 16, 8, 32, 1, 16), (64 * 16 + 1, 8, 32, 1, 16), (64 * 9 - 5, 32, 32, 4, 16),
                                       (64 * 8, 8, 64, 2, 16), (130, 6, 20, 3, 4), (64 * 5 + 3, 3, 40, 1, 12)])
@pytest.mark.parametrize("carry", [False, True])
def test_scan_of_a_few_chunks_in_one_launch(T, H, P, G, n, carry, dtype):
    """The same bits as the first tokens of a scan too long for one launch (outputs depend on earlier tokens alone), the state
    against the oracle; with and without a state output."""
    long = 64 * 40
    g = torch.Generator().manual_seed(T + H)
    x, B, C = (torch.randn(long, *s, generator=g).to(dtype).to(DEV) for s in ((H, P), (G, n), (G, n)))
    dt = torch.nn.functional.softplus(torch.randn(long, H, generator=g)).to(DEV)
    A = (-0.3 * torch.exp(2 * torch.rand(H, generator=g))).to(DEV)
    D, S_in = (torch.randn(H, generator=g).to(DEV), torch.randn(H, P, n, generator=g).to(DEV)) if carry else (None, None)
    y_long, _ = strd.ssd_prefill(x, dt, A, B, C, D=D, S_in=S_in)
    short = [t[:T].contiguous() for t in (x, dt, B, C)]
    y, S = strd.ssd_prefill(short[0], short[1], A, short[2], short[3], D=D, S_in=S_in)
    assert torch.equal(y, y_long[:T])
    y2, none = strd.ssd_prefill(short[0], short[1], A, short[2], short[3], D=D, S_in=S_in, want_state=False)
    assert none is None and torch.equal(y2, y)
    f = synth.np64
    opt = lambda t: None if t is None else f(t)
    y_ref, S_ref = oracle.ssd_seq(f(short[0]), f(short[1]), f(A), f(short[2]), f(short[3]), opt(D), opt(S_in))
    assert_close(f(y), y_ref, TOL[dtype], "y", units=(1,))
    assert_close(f(S), S_ref, TOL[torch.float32], "state", units=(0,))


@pytest.mark.parametrize("N", [700, 4096 + 33])
@pytest.mark.parametrize("M,Hq,Hkv,d", [(1, 1, 1, 64), (8, 8, 2, 128), (33, 2, 2, 64), (97, 4, 4, 128), (32, 8, 2, 128), (43, 3, 1, 64),
                                        (129, 1, 1, 128), (65, 4, 1, 128), (100, 3, 1, 64)])
def test_score_attn_rows_that_leave_waves_without_a_tile(N, M, Hq, Hkv, d):
    """1 to 300 query rows of a kv head: none, one or two tiles of 32 rows in a wave of pass 1, one to three chunks of 128 in
    pass 2 (the log-sum-exps of the first two at once), keys that end inside a chunk."""
    _say("score_attn rows N=%d M=%d Hq=%d Hkv=%d d=%d" % (N, M, Hq, Hkv, d))
    rn = _draw(N + M, BF16)
    q, k = rn(M, Hq, d), rn(N, Hkv, d)
    assert_close(f(strd.score_attn(q.to(DEV), k.to(DEV))), oracle.score_attn(f(q), f(k)), BOUND[BF16], "s", units=(0,))


@pytest.mark.parametrize("M,Hq,Hkv", [(8213, 8, 1), (600, 24, 2), (1280, 2, 2)])
def test_score_attn_of_many_rows(M, Hq, Hkv):
    """257, 58 and 10 workgroups per slice of keys: no whole number of the chip's rounds, nearly one, and one of more than its slices;
    chunks of 128 rows copied whole and, in the first two, a last one of 40 and 32 rows."""
    _say("score_attn many rows M=%d Hq=%d Hkv=%d" % (M, Hq, Hkv))
    rn = _draw(M + Hq, BF16)
    q, k = rn(M, Hq, 64), rn(700, Hkv, 64)
    assert_close(f(strd.score_attn(q.to(DEV), k.to(DEV))), oracle.score_attn(f(q), f(k)), BOUND[BF16], "s", units=(0,))


@pytest.mark.parametrize("M,Hq,Hkv,d,N", [(1280, 1, 1, 64, 300), (1281, 1, 1, 64, 300), (2049, 1, 1, 128, 300), (683, 3, 1, 128, 300),
                                          (683, 3, 1, 128, 100), (1281, 8, 8, 64, 4400), (37, 8, 8, 64, 4400)])
def test_score_attn_rows_copied_with_and_without_branches(M, Hq, Hkv, d, N):
    """Pass 2 on both sides of its lines, 1280 rows per kv head of 64 elements and 2048 of 128 (more of them where the query heads per kv
    head are a power of two), with one and two key tiles per wave and with the slices combined in it."""
    _say("score_attn copies M=%d Hq=%d Hkv=%d d=%d N=%d" % (M, Hq, Hkv, d, N))
    rn = _draw(M + N, BF16)
    q, k = rn(M, Hq, d), rn(N, Hkv, d)
    assert_close(f(strd.score_attn(q.to(DEV), k.to(DEV))), oracle.score_attn(f(q), f(k)), BOUND[BF16], "s", units=(0,))


@pytest.mark.parametrize("H,G,n", [(64, 1, 128), (8, 1, 64), (48, 2, 128), (80, 1, 64), (20, 1, 128), (70, 1, 64), (32, 2, 64)])
def test_score_mamba_heads_of_a_group(H, G, n):
    """dt of 8 to 80 heads of a group, added up by 16 lanes per token: fewer heads than lanes, as many, several times as many with and
    without a rest, rows of dt that start anywhere in a 64-byte line."""
    _say("score_mamba heads H=%d G=%d n=%d" % (H, G, n))
    rn = _draw(H + n, BF16)
    B, C, dt = rn(300, G, n), rn(37, G, n), rn(300, H).float().abs()
    got = strd.score_mamba(B.to(DEV), C.to(DEV), dt.to(DEV))
    assert_close(f(got), oracle.score_mamba(f(B), f(C), f(dt)), BOUND[BF16], "s", units=(0,))


@pytest.mark.parametrize("T,H,P", [(40, 2, 192), (33, 2, 256), (40, 1, 260), (9, 2, 512), (64, 2, 1024), (30, 3, 4096), (12, 3100, 4)])
@pytest.mark.parametrize("carry", [False, True])
def test_scan_of_one_chunk_without_an_end_state(T, H, P, carry):
    """16 state entries, up to more channels than a launch has LDS for and more heads than one launch is for."""
    g = torch.Generator().manual_seed(T + P)
    x, B, C = (torch.randn(T, *s, generator=g).to(DEV) for s in ((H, P), (1, 16), (1, 16)))
    dt = torch.nn.functional.softplus(torch.randn(T, H, generator=g)).to(DEV)
    A = (-0.3 * torch.exp(2 * torch.rand(H, generator=g))).to(DEV)
    S_in = torch.randn(H, P, 16, generator=g).to(DEV) if carry else None
    y, none = strd.ssd_prefill(x, dt, A, B, C, S_in=S_in, want_state=False)
    f = synth.np64
    y_ref, _ = oracle.ssd_seq(f(x), f(dt), f(A), f(B), f(C), None, f(S_in) if carry else None)
    assert none is None
    assert_close(f(y), y_ref, TOL[torch.float32], "y", units=(1,))


def _scan_in_place(x, dt, A, B, C, S, chunk=64):
    """The C call with one buffer for the state carried in and the state at the end; the outputs."""
    T, H, P = x.shape
    G, n = B.shape[1:]
    io = strd.binding.STRD_F32 if x.dtype == F32 else strd.binding.STRD_BF16
    L = strd.lib()
    size = L.strd_ssd_prefill_workspace(T, H, P, G, n, chunk, io)
    ws = torch.empty(max(size, 16), dtype=torch.uint8, device=DEV)
    y = torch.empty_like(x)
    rc = L.strd_ssd_prefill(x.data_ptr(), dt.data_ptr(), A.data_ptr(), B.data_ptr(), C.data_ptr(), None, S.data_ptr(), y.data_ptr(),
                            S.data_ptr(), T, H, P, G, n, chunk, io, ws.data_ptr(), size, torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    return y


@pytest.mark.parametrize("dtype,T,H,P,G,n", [(F32, 9, 8, 32, 1, 16), (F32, 64 * 16 + 1, 8, 32, 1, 16), (BF16, 500, 6, 20, 3, 4),
                                            (F32, 3000, 8, 32, 1, 16), (F32, 3, 8, 32, 1, 16), (BF16, 700, 8, 64, 2, 128)])
def test_scan_with_its_state_in_place(dtype, T, H, P, G, n):
    """Token by token, in one launch's range, in chunks and in one walk: the same bits as with two buffers."""
    rn = _draw(T + n, dtype)
    x, B, C = rn(T, H, P).to(DEV), rn(T, G, n).to(DEV), rn(T, G, n).to(DEV)
    dt = torch.nn.functional.softplus(rn(T, H).float()).to(DEV)
    A = -(0.3 + rn(H).float().abs()).to(DEV)
    S = rn(H, P, n).float().to(DEV)
    y_ref, S_ref = strd.ssd_prefill(x, dt, A, B, C, S_in=S)
    y = _scan_in_place(x, dt, A, B, C, S)
    assert torch.equal(y, y_ref) and torch.equal(S, S_ref)


@pytest.mark.parametrize("T,H,G,n", [(64 * 32 - 5, 32, 2, 128), (64 * 17, 15, 1, 64)])
def test_long_scan_with_its_state_in_place(T, H, G, n):
    """Sequences that are cut into segments (of two heads per workgroup and of one) otherwise: against the call with two buffers and the
    oracle, a second call going on from the state of the first."""
    P, first = 64, T - 64 * 9
    rn = _draw(T + n, BF16)
    x, B, C = rn(T, H, P).to(DEV), (rn(T, G, n) / n ** 0.5).to(DEV), rn(T, G, n).to(DEV)
    dt = torch.nn.functional.softplus(rn(T, H).float()).to(DEV)
    A = -(0.05 + rn(H).float().abs()).to(DEV)
    S0 = rn(H, P, n).float().to(DEV)
    y_ref, S_ref = strd.ssd_prefill(x, dt, A, B, C, S_in=S0)
    S = S0.clone()
    y = torch.cat([_scan_in_place(*(t[a:b].contiguous() if t is not A else A for t in (x, dt, A, B, C)), S)
                   for a, b in ((0, first), (first, T))])
    assert_close(f(y), f(y_ref), BOUND[BF16], "y of one buffer and of two", units=(1,))
    assert_close(f(S), f(S_ref), BOUND[BF16], "state of one buffer and of two", units=(0,))
    for h in (0, H - 1):
        q = h // (H // G)
        y_o, S_o = oracle.ssd_seq(f(x[:, h:h + 1]), f(dt[:, h:h + 1]), f(A[h:h + 1]), f(B[:, q:q + 1]), f(C[:, q:q + 1]), None,
                                  f(S0[h:h + 1]))
        assert_close(f(y[:, h:h + 1]), y_o, BOUND[BF16], "y of head %d" % h, units=(1,))
        assert_close(f(S[h:h + 1]), S_o, BOUND[BF16], "state of head %d" % h, units=(0,))


@pytest.mark.parametrize("K", [64 * 20 + 7, 0])
def test_gathering_scan_with_its_state_in_place(K):
    """The bits of the dense call in place, for a sequence that is cut into segments otherwise; and with nothing kept but the text."""
    N, M, H, P, G, n = 1500, 64 * 17 - 3, 16, 64, 2, 128
    rn = _draw(K + 1, BF16)
    x, B, C = rn(N + M, H, P).to(DEV), rn(N + M, G, n).to(DEV), rn(N + M, G, n).to(DEV)
    dt = torch.nn.functional.softplus(rn(N + M, H).float()).to(DEV)
    A = -(0.3 + rn(H).float().abs()).to(DEV)
    S = rn(H, P, n).float().to(DEV)
    idx = torch.sort(torch.randperm(N, generator=torch.Generator().manual_seed(K))[:K]).values
    keep = torch.cat([idx, torch.arange(N, N + M)]).to(DEV)
    S_ref = S.clone()
    y_ref = _scan_in_place(x[keep], dt[keep], A, B[keep], C[keep], S_ref)
    idx, y, L = idx.to(torch.int32).to(DEV), torch.empty(K + M, H, P, dtype=BF16, device=DEV), strd.lib()
    size = L.strd_ssd_prefill_workspace(K + M, H, P, G, n, 64, strd.binding.STRD_BF16)
    ws = torch.empty(size, dtype=torch.uint8, device=DEV)
    assert size > 0      # the segments' scratch
    rc = L.strd_ssd_prefill_gather(x.data_ptr(), dt.data_ptr(), A.data_ptr(), B.data_ptr(), C.data_ptr(), None, S.data_ptr(),
                                   idx.data_ptr() if K else None, y.data_ptr(), S.data_ptr(), N, M, K, H, P, G, n, 64,
                                   strd.binding.STRD_BF16, ws.data_ptr(), size, torch.cuda.current_stream().cuda_stream)
    assert rc == 0 and torch.equal(y, y_ref) and torch.equal(S, S_ref)
