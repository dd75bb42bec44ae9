"""How the decode launch cuts its work: whole units, pieces of long ones, equal ranges over many; tile edges; arguments
that are not 16-byte aligned.  All against the oracle."""
import threading

import numpy as np
import pytest
import torch

import oracle
import paper_2410_12876_amd as ag
import workloads as W
from gpu_util import DEV, attn_error, attn_tolerance, cache_from_host, dev, ensure_built, host_f32, make_ctx
from test_parity_gpu import check_decode

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    ensure_built()


@pytest.mark.parametrize("dtype,B,Hq,Hkv,D,lens", [
    ("bf16", 1, 4, 4, 128, [31, 32, 33, 0]),                    # one tile, its edges
    ("bf16", 1, 8, 8, 64, [1, 63, 64, 65, 1023, 1024, 1025, 2]),   # a unit of 32 tiles stays whole, 33 are cut (8 waves)
    ("bf16", 1, 8, 2, 128, [9000, 1025]),                       # few units, many pieces
    ("bf16", 2, 32, 8, 128, [7000] * 15 + [3]),                 # more than one round of the launch: pieces of two rounds
    # 65 to 128 units of more than two rounds: equal ranges, 8 waves
    ("bf16", 24, 16, 4, 128, [1500, 2900, 3000, 1700]),
    ("bf16", 32, 8, 4, 64, [2500, 3000, 1600]),
    ("f32", 25, 8, 4, 64, [3000, 2000]),
    ("f32", 25, 4, 4, 128, [3000, 2000]),
    # more than 128 units: 4 waves, a team of them per unit, or equal ranges where one unit is long for that
    ("bf16", 43, 3, 3, 128, [5, 170, 40, 480]),
    ("bf16", 65, 4, 4, 128, [5, 170, 40, 480]),
    ("bf16", 66, 4, 4, 128, [900, 40, 1000]),                   # 264 units: 8 of 256 CUs would have two, so equal ranges from 6 rounds on
    ("bf16", 50, 4, 4, 128, [3000, 1500, 2, 700, 2222]),
    ("bf16", 65, 8, 4, 128, [5, 1170, 40, 2480]),
    ("bf16", 100, 16, 4, 64, [600, 30, 2000, 0]),
    ("f32", 68, 4, 4, 128, [40, 1500]),
    ("bf16", 1, 8, 1, 128, [12345]),                            # one unit, eight heads
    ("f32", 1, 4, 4, 64, [33, 992, 2500, 0]),
    ("f32", 70, 8, 4, 128, [7, 100, 31, 250]),
    # fp32: tiles of 16 rows (32 of D = 64 with one or two heads), whole up to one round, teams up to 8 (4 at eight heads of 128); 192 units are few
    ("f32", 1, 64, 8, 128, [15, 16, 17, 0, 128, 129, 145, 500]),
    ("f32", 1, 16, 8, 64, [256, 257, 1, 33, 16, 255, 2000, 31]),
    ("f32", 24, 32, 8, 128, [186, 60, 0, 17]),
    ("f32", 193, 4, 1, 128, [512, 30, 511]),
    ("f32", 193, 4, 1, 128, [513, 0, 511]),
    ("f32", 65, 32, 4, 128, [256, 30, 241, 16]),
    ("f32", 65, 32, 4, 128, [257, 15]),
    ("f32", 130, 16, 4, 64, [250, 241, 1]),                     # two waves a unit
])
def test_decode_work_split(dtype, B, Hq, Hkv, D, lens):
    U = B * Hkv
    len0 = np.resize(np.asarray(lens, dtype=np.int32), U)
    g = np.random.default_rng(U + D)
    len0 = np.where(len0 > 100, len0 - g.integers(0, 3, size=U) * (U > 16), len0).astype(np.int32)
    wl = W.decode_batch(60, "split", dtype, B, Hq, Hkv, D, len0, 2, pos0=int(len0.max()) + 1)
    print("decode split", dtype, B, Hq, Hkv, D, int(len0.sum()), flush=True)
    check_decode(wl, 2, 0.5, dtype)


def test_decode_takes_new_rows_at_any_even_address():
    B, Hq, Hkv, D = 2, 8, 2, 128
    wl = W.decode_batch(61, "loose", "bf16", B, Hq, Hkv, D, np.array([40, 0, 700, 1300], dtype=np.int32), 1, pos0=1400)
    ctx = make_ctx(B, 1, Hq, Hkv, D, ag.AG_BF16, cache_rows=int(wl.row_off[-1]))
    cache = cache_from_host(B, Hkv, D, wl.k_cache, wl.v_cache, wl.idx, wl.row_off, wl.len0)
    ref = oracle.Cache(wl.k_cache.f32.copy(), wl.v_cache.f32.copy(), wl.idx.copy(), wl.row_off.copy(), wl.len0.copy())
    q, kn, vn, _ = wl.step_inputs(0, 0.5)

    def shifted(t, by):
        x = torch.zeros(t.numel() + 8, dtype=t.dtype, device=DEV)[by:by + t.numel()].view(t.shape)
        return x.copy_(t)
    out = shifted(dev(q), 3)
    ag.ag_decode_attn(ctx, dev(q), shifted(dev(kn), 1), shifted(dev(vn), 5), None, wl.pos0, wl.scale, cache, out)
    want, dropped = oracle.decode_step(q.f32, kn.f32, vn.f32, None, wl.pos0, ref, wl.scale)
    assert dropped == 0
    assert attn_error("bf16", host_f32(out), want) <= attn_tolerance("bf16", want)
    gk = host_f32(cache.k)
    for u in range(B * Hkv):
        a, n = int(wl.row_off[u]), int(ref.len[u])
        assert np.array_equal(gk[a:a + n], ref.k[a:a + n])
    ctx.poll_error()
    ctx.close()


def test_decode_unit_of_more_than_four_gib():
    """A unit whose K (and V) rows span more than 32 bits of bytes: the only keys that matter lie past that point.  Every
    cached key is 0 except two that draw all the weight, so the output is the mean of their values (to the n exp(-60) of the rest)."""
    n, D = (1 << 24) + 70, 128
    ctx = make_ctx(1, 1, 1, 1, D, ag.AG_BF16, cache_rows=n + 1)
    k, v = (torch.zeros(n + 1, D, dtype=torch.bfloat16, device=DEV) for _ in range(2))
    hot = [(1 << 24) + 5, n - 1]
    for i, r in enumerate(hot):
        k[r, 0] = 1.0
        v[r] = 1.0 + i
    cache = ag.KVCache(k, v, torch.zeros(n + 1, dtype=torch.int32, device=DEV), torch.tensor([0, n + 1], device=DEV),
                       torch.tensor([n], dtype=torch.int32, device=DEV), 1, 1, D, total_rows=n + 1)
    q = torch.zeros(1, 1, D, dtype=torch.bfloat16, device=DEV)
    q[..., 0] = 60.0
    new = torch.zeros(1, 1, D, dtype=torch.bfloat16, device=DEV)
    out = torch.empty_like(q)
    ag.ag_decode_attn(ctx, q, new, new, None, n, 1.0, cache, out)
    assert torch.all(out == 1.5), out
    assert int(cache.len[0]) == n + 1
    ctx.poll_error()
    ctx.close()


@pytest.mark.parametrize("D,lens", [(128, [40, 1, 500, 3000]), (64, [40, 1, 2100, 9000]), (128, [7000] * 40),
                                    (128, [2000, 2500, 1800] * 32), (64, [3500, 2500, 2800, 2600] * 32)])
def test_decode_infinite_values_stay_infinite(D, lens):
    """An infinite value in the first, the last or the new row of a unit (whole units, pieces, equal ranges in the last two): its feature is
    that infinity, the others are the result without it.  The keys draw equal weights, so no weight rounds to 0."""
    lens = np.asarray(lens, dtype=np.int32)
    U = len(lens)
    wl = W.decode_batch(62, "inf", "bf16", 1, 2 * U, U, D, lens, 1, pos0=int(lens.max()) + 1)
    ctx = make_ctx(1, 1, 2 * U, U, D, ag.AG_BF16, cache_rows=int(wl.row_off[-1]))
    cache = cache_from_host(1, U, D, wl.k_cache, wl.v_cache, wl.idx, wl.row_off, wl.len0)
    q, kn, vn, _ = wl.step_inputs(0, 0.5)
    q, kn, vn = dev(q), dev(kn), dev(vn)
    q.zero_()
    want = torch.empty_like(q)
    no = torch.zeros(1, U, dtype=torch.uint8, device=DEV)  # the new token is not appended: both calls see the same rows
    ag.ag_decode_attn(ctx, q, kn, vn, no, wl.pos0, wl.scale, cache, want)
    for u in range(U):
        a = int(wl.row_off[u])
        cache.v[a, 5] = float("inf")
        cache.v[a + int(lens[u]) - 1, D - 1] = float("-inf")
        vn[0, u, 9] = float("inf")
    want[..., 5], want[..., D - 1], want[..., 9] = float("inf"), float("-inf"), float("inf")
    out = torch.empty_like(q)
    ag.ag_decode_attn(ctx, q, kn, vn, no, wl.pos0, wl.scale, cache, out)
    assert torch.equal(out, want)
    ctx.close()


@pytest.mark.parametrize("D,G,half", [(128, 1, 1), (128, 4, 20), (128, 1, 300), (64, 2, 1000), (64, 8, 33), (128, 8, 6000)])
def test_decode_weights_keep_24_bits(D, G, half):
    """Half of a unit's rows have value 1 and score 0, the other half value -1 and a score lower by d, 2^-14 to 2^-13: the output is
    tanh(d / 2), what is left of sums that cancel to a few 2^-15.  A weight of 24 bits has a relative error of up to 2^-23 (one
    unit in the last place from the exponential, half of one from its argument), so the output one of 2 * 2^-23 / 2^-14 = 0.4 %
    plus half a bf16 spacing (0.4 %); of weights of 16 bits up to a quarter of it would be left."""
    U, n = 8, 2 * half
    k, v = torch.zeros(U, n + 1, D, device=DEV), torch.zeros(U, n + 1, D, device=DEV)
    step = 2.0 ** -14 * (1.0 + torch.arange(U, device=DEV) / 8.0)
    k[:, half:n, 3] = -step[:, None]
    v[:, :half], v[:, half:n] = 1.0, -1.0
    ro = torch.arange(U + 1, device=DEV) * (n + 1)
    cache = ag.KVCache(k.view(-1, D).bfloat16(), v.view(-1, D).bfloat16(), torch.zeros(U * (n + 1), dtype=torch.int32, device=DEV), ro,
                       torch.full((U,), n, dtype=torch.int32, device=DEV), 1, U, D)
    ctx = make_ctx(1, 1, U * G, U, D, ag.AG_BF16, cache_rows=U * (n + 1))
    q = torch.zeros(1, U * G, D, dtype=torch.bfloat16, device=DEV)
    q[..., 3], q[..., 5] = 1.0, 64.0
    kn, vn = torch.zeros(1, U, D, dtype=torch.bfloat16, device=DEV), torch.ones(1, U, D, dtype=torch.bfloat16, device=DEV)
    kn[..., 5] = -64.0                                       # the new token has no weight
    out = torch.empty_like(q)
    ag.ag_decode_attn(ctx, q, kn, vn, None, n, 1.0, cache, out)
    want = torch.tanh(step.double() / 2).repeat_interleave(G)[None, :, None].expand(1, U * G, D)
    err = float(((out.double() - want).abs() / want).max())
    print("relative error %.4f" % err)
    assert err <= 0.008
    ctx.close()


@pytest.mark.parametrize("D,G", [(128, 1), (64, 4)])
def test_decode_infinite_value_of_a_tiny_weight(D, G):
    """The infinity comes through at any weight that is not 0: 2^-60 to 2^-124, the least that the exponential gives."""
    U, n = 16, 40
    k, v = torch.zeros(U, n + 1, D, device=DEV), torch.ones(U, n + 1, D, device=DEV)
    low = torch.linspace(60.0, 124.0, U, device=DEV).round()
    k[:, 7, 3] = -low
    v[:, 7, 9] = float("inf")
    v[:, 7, 11] = -float("inf")
    cache = ag.KVCache(k.view(-1, D).bfloat16(), v.view(-1, D).bfloat16(), torch.zeros(U * (n + 1), dtype=torch.int32, device=DEV),
                       torch.arange(U + 1, device=DEV) * (n + 1), torch.full((U,), n, dtype=torch.int32, device=DEV), 1, U, D)
    ctx = make_ctx(1, 1, U * G, U, D, ag.AG_BF16, cache_rows=U * (n + 1))
    q = torch.zeros(1, U * G, D, dtype=torch.bfloat16, device=DEV)
    q[..., 3] = 1.0
    new = torch.zeros(1, U, D, dtype=torch.bfloat16, device=DEV)
    out = torch.empty_like(q)
    ag.ag_decode_attn(ctx, q, new, torch.ones_like(new), None, n, 0.6931471805599453, cache, out)
    want = torch.ones_like(out)
    want[..., 9], want[..., 11] = float("inf"), -float("inf")
    for u in range(U):
        for g in range(G):
            if not torch.equal(out[0, u * G + g], want[0, u * G + g]): print("weight 2^-%d" % int(low[u]), out[0, u * G + g, 7:13].tolist())
    assert torch.equal(out, want)
    ctx.close()


@pytest.mark.parametrize("dtype,G,D", [("bf16", 1, 128), ("f32", 8, 128)])
def test_decode_steps_of_different_sizes_from_several_threads(dtype, G, D):
    """The LDS of a step grows with its units, and its limit belongs to the kernel: threads with contexts and streams of their
    own, each at another number of units."""
    td = torch.bfloat16 if dtype == "bf16" else torch.float32

    def made(U):
        g = torch.Generator(device=DEV)
        g.manual_seed(U)
        k, v = (torch.randn(U * 4, D, generator=g, device=DEV).to(td) for _ in range(2))
        q = torch.randn(1, U * G, D, generator=g, device=DEV).to(td)
        new = torch.randn(1, U, D, generator=g, device=DEV).to(td)
        cache = ag.KVCache(k, v, torch.zeros(U * 4, dtype=torch.int32, device=DEV), torch.arange(U + 1, device=DEV) * 4,
                           torch.full((U,), 3, dtype=torch.int32, device=DEV), 1, U, D)
        no = torch.zeros(1, U, dtype=torch.uint8, device=DEV)
        ctx = make_ctx(1, 1, U * G, U, D, ag.AG_BF16 if dtype == "bf16" else ag.AG_F32, cache_rows=U * 4)
        return ctx, q, new, no, cache
    sizes = [300, 8192, 1000, 5000]
    sets = [made(U) for U in sizes]
    got, errors = [None] * len(sizes), []
    torch.cuda.synchronize()

    def work(i):
        try:
            ctx, q, new, no, cache = sets[i]
            s = torch.cuda.Stream()
            outs = [torch.empty_like(q) for _ in range(20)]
            torch.cuda.synchronize()
            for o in outs:
                ag.ag_decode_attn(ctx, q, new, new, no, 9, 0.1, cache, o, stream=s)
            s.synchronize()
            assert all(torch.equal(o, outs[0]) for o in outs)
            got[i] = outs[0]
        except Exception as e:  # noqa: BLE001  (reported by the main thread)
            errors.append(e)
    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(sizes))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for (ctx, q, new, no, cache), o in zip(sets, got):
        out = torch.empty_like(q)
        ag.ag_decode_attn(ctx, q, new, new, no, 9, 0.1, cache, out)
        assert torch.equal(o, out) and torch.isfinite(out.float()).all()
        ctx.close()


@pytest.mark.parametrize("D,G,lens,by", [(128, 1, [40, 0, 700, 1300, 33], 1), (64, 4, [5, 900, 2100], 4), (128, 8, [6000], 3),
                                         (128, 2, [70, 3, 31, 500] * 66, 5)])
def test_decode_over_caches_at_any_even_address(D, G, lens, by):
    """Caches that do not start at a multiple of 16 bytes: outputs, appended rows and lengths bit for bit those of aligned ones."""
    U = len(lens)
    wl = W.decode_batch(63, "even", "bf16", 1, U * G, U, D, np.asarray(lens, dtype=np.int32), 2, pos0=6100, fill_slack=float("nan"))
    ctx = make_ctx(1, 1, U * G, U, D, ag.AG_BF16, cache_rows=int(wl.row_off[-1]))
    got = []
    for shift in (0, by):
        cache = cache_from_host(1, U, D, wl.k_cache, wl.v_cache, wl.idx, wl.row_off, wl.len0)
        if shift:
            k, v = (torch.zeros(t.numel() + 8, dtype=t.dtype, device=DEV)[shift:shift + t.numel()].view(t.shape).copy_(t) for t in (cache.k, cache.v))
            cache = ag.KVCache(k, v, cache.idx, cache.row_off, cache.len, 1, U, D)
            assert k.data_ptr() % 16 == 2 * shift % 16
        outs = []
        for i in range(2):
            q, kn, vn, flags = wl.step_inputs(i, 0.5)
            outs.append(torch.empty_like(dev(q)))
            ag.ag_decode_attn(ctx, dev(q), dev(kn), dev(vn), dev(flags), wl.pos0 + i, wl.scale, cache, outs[-1])
        got.append(outs + [cache.k, cache.v, cache.idx, cache.len])
    ctx.poll_error()
    for a, b in zip(*got):
        assert torch.equal(a.nan_to_num(-77.0), b.nan_to_num(-77.0))
    assert torch.isfinite(got[0][0].float()).all() and torch.isfinite(got[0][1].float()).all()
    ctx.close()


@pytest.mark.parametrize("dtype,U,G,D,lens,n_recent", [
    ("bf16", 96, 1, 128, [1500, 2900, 40], 64),   # equal ranges of 8 waves: two ring tiles in front of every unit, also at cuts
    ("bf16", 120, 4, 64, [2500, 900, 1300], 64),
    ("f32", 100, 2, 64, [3000, 2000], 40),
    ("bf16", 300, 2, 128, [1100, 30, 0], 33),     # ... of 4 waves
    ("bf16", 9, 1, 128, [0, 700, 1500], 64),      # whole units and pieces
    ("bf16", 300, 1, 64, [100, 0], 64),           # a team of waves per unit
    ("f32", 1, 8, 128, [65], 64),                 # fp32: four ring tiles; fewer records than pieces of one round
    ("f32", 9, 8, 128, [0, 700, 150], 64),
    ("f32", 300, 2, 64, [100, 0], 64),
    ("f32", 600, 4, 64, [60, 0, 17], 49)])
def test_decode_ring_in_every_split(dtype, U, G, D, lens, n_recent):
    """Ring slots of which some are evicted tokens inside the window, some kept ones, some outside or empty, holding NaN where
    they are not to be seen; against the oracle over the cache rows followed by the visible slots."""
    len0 = np.resize(np.asarray(lens, dtype=np.int32), U)
    wl = W.decode_batch(64, "ring", dtype, 1, U * G, U, D, len0, 1, pos0=4000, fill_slack=float("nan"))
    g = np.random.default_rng(U)
    rk, rv = (W.store(g.standard_normal((U, n_recent, D)).astype(np.float32), dtype).f32 for _ in range(2))
    pos = 4000 - 1 - (4000 - 1 - np.arange(n_recent)) % n_recent * np.ones((U, 1), dtype=np.int64)  # slot p % n: p in [pos - n, pos)
    pos = np.where(g.random((U, n_recent)) < 0.2, -(1 << 30), pos).astype(np.int32)
    kept = (g.random((U, n_recent)) < 0.4).astype(np.uint8)
    see = (pos > 4000 - n_recent) & (pos < 4000) & (kept == 0)
    assert see.any() and not see.all()
    # the oracle's cache: a unit's rows, then its visible slots
    n_see = see.sum(axis=1)
    ro = np.concatenate([[0], np.cumsum(len0.astype(np.int64) + n_see + 1)])
    ck, cv = np.zeros((int(ro[-1]), D), np.float32), np.zeros((int(ro[-1]), D), np.float32)
    for u in range(U):
        a, n, m = int(ro[u]), int(len0[u]), int(n_see[u])
        src = int(wl.row_off[u])
        ck[a:a + n], cv[a:a + n] = wl.k_cache.f32[src:src + n], wl.v_cache.f32[src:src + n]
        ck[a + n:a + n + m], cv[a + n:a + n + m] = rk[u, see[u]], rv[u, see[u]]
    ref = oracle.Cache(ck, cv, np.zeros(int(ro[-1]), np.int32), ro, (len0 + n_see).astype(np.int32))
    q, kn, vn, _ = wl.step_inputs(0, 0.5)
    want, _ = oracle.decode_step(q.f32, kn.f32, vn.f32, None, wl.pos0, ref, wl.scale)
    rk[~see], rv[~see] = np.nan, np.nan
    ring = ag.RecentRing(dev(W.store(rk, dtype)), dev(W.store(rv, dtype)), dev(kept), dev(pos), n_recent)
    ctx = make_ctx(1, 1, U * G, U, D, ag.AG_BF16 if dtype == "bf16" else ag.AG_F32, cache_rows=int(wl.row_off[-1]))
    cache = cache_from_host(1, U, D, wl.k_cache, wl.v_cache, wl.idx, wl.row_off, wl.len0)
    out = torch.empty_like(dev(q))
    print("ring", dtype, U, G, D, n_recent, flush=True)
    ag.ag_decode_attn_recent(ctx, dev(q), dev(kn), dev(vn), None, 4000, wl.scale, cache, ring, out)
    got = host_f32(out)
    assert np.isfinite(got).all() and attn_error(dtype, got, want) <= attn_tolerance(dtype, want)
    assert np.array_equal(cache.len.cpu().numpy(), len0 + 1)
    slot = 4000 % n_recent
    assert torch.equal(ring.k[:, slot], dev(kn)[0]) and (ring.pos[:, slot] == 4000).all() and (ring.flags[:, slot] == 1).all()
    ctx.poll_error()
    ctx.close()
