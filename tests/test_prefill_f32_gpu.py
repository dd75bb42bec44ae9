"""The fp32 prefill kernel at the edges of its 16-query, 16-key tiles and of its waves' shares, all head dimensions, grouped
heads, the recent-token window, a kept row that only some queries of a tile see holding NaN."""
import math

import numpy as np
import pytest

import oracle
import workloads as W
from gpu_util import attn_error, ensure_built, host_f32
from test_parity_configs_gpu import _prefill_recent

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    ensure_built()


@pytest.mark.parametrize("B,Hq,Hkv,L,D,keep,n_recent,with_cache", [
    (1, 1, 1, 1, 64, 1.0, 1, True), (1, 2, 2, 16, 64, 1.0, 1, True), (2, 4, 2, 17, 32, 1.0, 1, False),
    (1, 4, 4, 65, 64, 0.9, 1, True), (1, 8, 1, 129, 128, 0.5, 1, True), (1, 2, 2, 200, 256, 0.7, 1, False),
    (3, 4, 4, 333, 128, 0.3, 17, True), (1, 2, 1, 80, 256, 0.4, 64, True), (2, 2, 2, 50, 32, 0.0, 7, True),
    (1, 4, 2, 600, 64, 1.0, 3, True)])
def test_prefill_f32_tiles(B, Hq, Hkv, L, D, keep, n_recent, with_cache):
    g = np.random.default_rng(L + D)
    q, k, v = (W.store(g.standard_normal(s).astype(np.float32), "f32") for s in ((B, Hq, L, D), (B, Hkv, L, D), (B, Hkv, L, D)))
    flags = (g.random((B, Hkv, L)) < keep).astype(np.uint8)
    scale = 1.0 / math.sqrt(D)
    got = host_f32(_prefill_recent(q, k, v, flags, scale, n_recent, with_cache))
    ref = oracle.prefill_attn(q.f32, k.f32, v.f32, flags, scale, n_recent=n_recent)
    assert np.isfinite(got).all() and attn_error("f32", got, ref) <= 1e-5


def test_a_kept_nan_reaches_only_later_queries():
    B, H, L, D = 1, 2, 100, 64
    g = np.random.default_rng(5)
    q, k, v = (g.standard_normal((B, H, L, D)).astype(np.float32) for _ in range(3))
    flags = np.ones((B, H, L), dtype=np.uint8)
    v[:, :, 40] = np.nan
    got = host_f32(_prefill_recent(W.store(q, "f32"), W.store(k, "f32"), W.store(v, "f32"), flags, 0.125, 1, True))
    assert np.isfinite(got[:, :, :40]).all() and np.isnan(got[:, :, 40:]).any(axis=-1).all()


def test_an_infinite_value_stays_in_its_feature():
    """Kept tokens with one infinite feature each, at both ends of a tile that is seen in part and of one that is seen whole:
    queries that see one get that infinity in that feature, everything else is the result without it."""
    B, H, L, D = 1, 2, 100, 64
    g = np.random.default_rng(6)
    q, k, v = (g.standard_normal((B, H, L, D)).astype(np.float32) for _ in range(3))
    flags = np.ones((B, H, L), dtype=np.uint8)
    ref = oracle.prefill_attn(q, k, v, flags, 0.125)
    for t, d, x in ((0, 3, np.inf), (31, 40, -np.inf), (99, 7, np.inf), (50, 63, -np.inf)):
        v[:, :, t, d] = x
        ref[:, :, t:, d] = x
    got = host_f32(_prefill_recent(W.store(q, "f32"), W.store(k, "f32"), W.store(v, "f32"), flags, 0.125, 1, True))
    fin = np.isfinite(ref)
    assert np.array_equal(got[~fin], ref[~fin])
    assert attn_error("f32", np.where(fin, got, 0), np.where(fin, ref, 0)) <= 1e-5
