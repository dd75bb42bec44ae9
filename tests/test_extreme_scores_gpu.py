"""Scores at the far ends of fp32: attention over rows that all score near -2^105 is still the softmax of their differences,
and a query that sees nothing but its own token gets that token's value whatever the score is -- also one that overflowed."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2410_12876_amd as ag
import workloads as W
from gpu_util import DEV, attn_error, attn_tolerance, cache_from_host, dev, ensure_built, host_f32, make_ctx
from test_parity_configs_gpu import _prefill_recent

pytestmark = pytest.mark.gpu

# scale * log2(e) is 2^-3 exactly in fp32, and q, k have one feature that is not 0, a power of two: every score is exact
SCALE = float(np.float32(0.0866434))
while np.float32(SCALE) * np.float32(1.4426950408889634) != np.float32(0.125):
    SCALE = float(np.nextafter(np.float32(SCALE), np.float32(1)))
Q0 = 2.0 ** 54                     # a key of -x scores -x 2^51 in log2 units
LOW = 2.0 ** 54                    # 2^105 = 4e31


@pytest.fixture(scope="module", autouse=True)
def _lib():
    ensure_built()


def _one_feature(shape, value):
    x = np.zeros(shape, dtype=np.float32)
    x[..., 0] = value
    return x


@pytest.mark.parametrize("dtype,D,G", [("bf16", 128, 1), ("bf16", 64, 4), ("f32", 64, 2), ("f32", 128, 1)])
@pytest.mark.parametrize("own", [1.0, 2.0, 0.5])       # the new token's score against the cached rows': as low, lower, higher
def test_decode_of_scores_far_below_zero(dtype, D, G, own):
    lens = np.array([0, 1, 40, 300, 2000, 5000], dtype=np.int32)
    U = len(lens)
    wl = W.decode_batch(70, "low", dtype, 1, U * G, U, D, lens, 1, pos0=int(lens.max()) + 1)
    k = W.store(_one_feature(wl.k_cache.f32.shape, -LOW), dtype)
    ctx = make_ctx(1, 1, U * G, U, D, ag.AG_BF16 if dtype == "bf16" else ag.AG_F32, cache_rows=int(wl.row_off[-1]))
    cache = cache_from_host(1, U, D, k, wl.v_cache, wl.idx, wl.row_off, wl.len0)
    ref = oracle.Cache(k.f32.copy(), wl.v_cache.f32.copy(), wl.idx.copy(), wl.row_off.copy(), wl.len0.copy())
    _, _, vn, _ = wl.step_inputs(0, 0.5)
    q, kn = W.store(_one_feature((1, U * G, D), Q0), dtype), W.store(_one_feature((1, U, D), -LOW * own), dtype)
    out = torch.empty_like(dev(q))
    ag.ag_decode_attn(ctx, dev(q), dev(kn), dev(vn), None, wl.pos0, SCALE, cache, out)
    want, _ = oracle.decode_step(q.f32, kn.f32, vn.f32, None, wl.pos0, ref, SCALE)
    got = host_f32(out)
    assert np.isfinite(got).all() and attn_error(dtype, got, want) <= attn_tolerance(dtype, want)
    ctx.close()


@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("bf16", 64), ("f32", 128)])
@pytest.mark.parametrize("ring", [False, True])
def test_decode_of_an_empty_cache_is_the_new_value_whatever_the_score(dtype, D, ring):
    """Eight units without a row and one with some beside them; the ring, where there is one, holds kept tokens only."""
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    U, n = 9, 70
    ro = torch.arange(U + 1, device=DEV) * 80
    cache = ag.KVCache(torch.randn(U * 80, D, device=DEV).to(td), torch.randn(U * 80, D, device=DEV).to(td),
                       torch.zeros(U * 80, dtype=torch.int32, device=DEV), ro,
                       torch.tensor([0] * 8 + [n], dtype=torch.int32, device=DEV), 1, U, D)
    rr = None
    if ring:
        rr = ag.RecentRing(torch.full((U, 40, D), float("nan"), dtype=td, device=DEV), torch.full((U, 40, D), float("nan"), dtype=td, device=DEV),
                           torch.ones(U, 40, dtype=torch.uint8, device=DEV), torch.arange(40, dtype=torch.int32, device=DEV).repeat(U, 1), 40)
    ctx = make_ctx(1, 1, U, U, D, ag.AG_BF16 if dtype == "bf16" else ag.AG_F32, cache_rows=U * 80)
    q = torch.zeros(1, U, D, dtype=td, device=DEV)
    k = torch.zeros(1, U, D, dtype=td, device=DEV)
    v = torch.randn(1, U, D, device=DEV).to(td)
    big = 2.0 ** 100
    for u, (a, b) in enumerate([(big, big), (big, -big), (float("nan"), 1.0), (float("inf"), 1.0), (-float("inf"), 1.0),
                                (2.0 ** 60, -2.0 ** 60), (2.0 ** 60, 2.0 ** 60), (1.0, 1.0)]):
        q[0, u, 0], k[0, u, 0] = a, b
    out = torch.empty_like(q)
    ag.ag_decode_attn_recent(ctx, q, k, v, torch.zeros(1, U, dtype=torch.uint8, device=DEV), 40, 0.125, cache, rr, out)
    assert torch.equal(out[:, :8], v[:, :8]) and torch.isfinite(out[:, 8].float()).all()
    ctx.close()


@pytest.mark.parametrize("dtype,Hq,Hkv,D,L", [("f32", 2, 2, 64, 70), ("f32", 4, 1, 128, 33), ("bf16", 2, 2, 128, 300),
                                              ("bf16", 4, 1, 64, 200), ("bf16", 8, 2, 128, 70)])
@pytest.mark.parametrize("n_recent", [1, 5])
@pytest.mark.parametrize("keep", [0.0, 0.4])
def test_prefill_of_scores_far_below_zero(dtype, Hq, Hkv, D, L, n_recent, keep):
    """Every fourth key scores half as low as the others: the visible ones of them share the weight (evicted ones too, as a
    query's own token or inside the window); a query that sees none averages what it sees."""
    g = np.random.default_rng(71)
    kk = _one_feature((1, Hkv, L, D), -LOW)
    kk[:, :, ::4, 0] *= 0.5
    q, k, v = W.store(_one_feature((1, Hq, L, D), Q0), dtype), W.store(kk, dtype), W.store(g.standard_normal((1, Hkv, L, D)).astype(np.float32), dtype)
    flags = (g.random((1, Hkv, L)) < keep).astype(np.uint8)
    got = host_f32(_prefill_recent(q, k, v, flags, SCALE, n_recent))
    want = oracle.prefill_attn(q.f32, k.f32, v.f32, flags, SCALE, n_recent=n_recent)
    assert np.isfinite(got).all() and attn_error(dtype, got, want) <= attn_tolerance(dtype, want)
    if keep == 0.0 and n_recent == 1:
        assert np.array_equal(got, np.repeat(v.f32, Hq // Hkv, axis=1))


@pytest.mark.parametrize("dtype,D", [("f32", 64), ("f32", 256), ("bf16", 128), ("bf16", 64)])
def test_prefill_of_a_fully_evicted_head_is_the_own_value_whatever_the_score(dtype, D):
    B, H, L = 1, 2, 150
    g = np.random.default_rng(72)
    q, k, v = (g.standard_normal((B, H, L, D)).astype(np.float32) for _ in range(3))
    big = np.float32(2.0 ** 100)
    for t, (a, b) in enumerate([(big, big), (big, -big), (np.nan, 1.0), (np.inf, 1.0), (-np.inf, 1.0), (1.0, np.nan)]):
        q[:, :, 10 * t], k[:, :, 10 * t] = 0.0, 0.0
        q[:, :, 10 * t, 0], k[:, :, 10 * t, 0] = a, b
    flags = np.zeros((B, H, L), dtype=np.uint8)
    tv = W.store(v, dtype)
    for n_recent in (1, 2):
        got = host_f32(_prefill_recent(W.store(q, dtype), W.store(k, dtype), tv, flags, 1.0 / math.sqrt(D), n_recent))
        assert np.array_equal(got[:, :, 0], tv.f32[:, :, 0])
        if n_recent == 1:
            assert np.array_equal(got, tv.f32)


@pytest.mark.parametrize("D", [128, 64])
def test_prefill_bf16_own_score_that_overflowed_takes_all_the_weight(D):
    """An evicted query whose own score is +infinity, beside kept ones that it sees."""
    B, H, L = 1, 2, 200
    g = np.random.default_rng(73)
    q, k, v = (g.standard_normal((B, H, L, D)).astype(np.float32) for _ in range(3))
    flags = (g.random((B, H, L)) < 0.5).astype(np.uint8)
    flags[:, :, :60], flags[:, :, 60::20] = 1, 0
    q[:, :, 60::20], k[:, :, 60::20] = 0.0, 0.0
    q[:, :, 60::20, 0], k[:, :, 60::20, 0] = np.float32(2.0 ** 100), np.float32(2.0 ** 100)
    k[:, :, :, 0] = np.where(flags != 0, 0.0, k[:, :, :, 0])
    tv = W.store(v, "bf16")
    got = host_f32(_prefill_recent(W.store(q, "bf16"), W.store(k, "bf16"), tv, flags, 1.0 / math.sqrt(D), 1))
    assert np.array_equal(got[:, :, 60::20], tv.f32[:, :, 60::20])
