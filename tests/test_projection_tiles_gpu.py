"""The projection GEMM on each of its tiles (64 x 64, 128 x 128, 256 x 256, and 128 x 64 and 128 x 128 with two waves to a block; the
gate module's three tensors also on the two of 128 x 192: test_projection_tile_choice.py checks that the sizes below take them all)
and the gate module's attention with its items in 2, 4 and 8 chunks: ragged token tiles, feature counts that the deepest stage does not divide, sequences
shorter than a tile, and few k-steps."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2410_12876_amd as ag
import workloads as W
from gpu_util import DEV, dev, ensure_built, host_bits, host_f32, new_cache

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    ensure_built()


PROJECT_COMPACT = [(1, 1, 128, 1), (2, 63, 192, 2), (3, 65, 256, 4), (1, 129, 64, 32), (1, 700, 128, 32), (5, 200, 64, 32), (40, 100, 128, 8),
                   (3, 700, 192, 32), (1, 4100, 128, 32), (1, 130, 1024, 32), (2, 250, 1088, 32)]
GATE_MHA = [(1, 70, 128, 4), (1, 4096, 64, 4), (2, 1900, 128, 4), (1, 1200, 192, 2), (1, 5401, 128, 4), (3, 1801, 64, 4), (1, 3600, 1024, 4),
            (1, 2000, 1088, 4), (1, 1000, 1024, 4), (1, 6000, 64, 4), (1, 4500, 64, 2), (1, 4500, 64, 1), (1, 3999, 2112, 4),
            (1, 4500, 1088, 4), (1, 8203, 192, 4)]


@pytest.mark.parametrize("B,L,d,Hkv", PROJECT_COMPACT)
def test_project_compact_tiles(B, L, d, Hkv):
    g = np.random.default_rng(L + d)
    x = W.store((0.5 * g.standard_normal((B, L, d))).astype(np.float32), "bf16")
    w = W.store((g.standard_normal((d, 2 * Hkv * 128)) / math.sqrt(d)).astype(np.float32), "bf16")
    flags = (g.random((B, Hkv, L)) < g.random((B, Hkv, 1))).astype(np.uint8)
    ro = oracle.slab_row_off(B * Hkv, L)
    cache = new_cache(B, Hkv, 128, torch.bfloat16, ro)
    kv = torch.zeros(2, B, Hkv, L, 128, dtype=torch.bfloat16, device=DEV)
    ctx = ag.Context(0, ag.project_compact_workspace_bytes(B, L, Hkv))
    ag.ag_project_compact_kv(ctx, dev(x), dev(w), dev(flags), 3, kv, cache)
    ctx.poll_error()
    ctx.close()
    # the product in fp32 from bf16 operands: one bf16 spacing of the exact value plus the sum's own rounding
    y = x.f32.reshape(B * L, d).astype(np.float64) @ w.f32.astype(np.float64)
    want = y.reshape(B, L, 2, Hkv, 128).transpose(2, 0, 3, 1, 4)
    got = host_f32(kv).astype(np.float64)
    assert np.all(np.abs(got - want) <= np.maximum(np.abs(want), np.abs(got)) * 2.0 ** -7 + 1e-5 * math.sqrt(d))
    ref, over = oracle.compact_kv(host_bits(kv[0]), host_bits(kv[1]), flags, ro, pos0=3)
    assert over == 0 and np.array_equal(cache.len.cpu().numpy(), ref.len)
    gk, gv, gi = host_bits(cache.k), host_bits(cache.v), cache.idx.cpu().numpy()
    for u in range(B * Hkv):
        a, n = int(ro[u]), int(ref.len[u])
        assert np.array_equal(gi[a:a + n], ref.idx[a:a + n])
        assert np.array_equal(gk[a:a + n], ref.k[a:a + n]) and np.array_equal(gv[a:a + n], ref.v[a:a + n])


@pytest.mark.parametrize("B,L,d,hp", GATE_MHA)
def test_gate_mha_tiles(B, L, d, hp):
    """The gate module end to end on these tiles: logits against fp32 torch on the CPU with the four tensors it stores in bf16
    rounded where it rounds them (the tolerance of the module's own tests for that reference: 1e-2)."""
    g = np.random.default_rng(L)
    H = 8
    x = W.store((0.5 * g.standard_normal((B, L, d))).astype(np.float32), "bf16")
    w = W.store((2.0 * g.standard_normal((d, 3 * hp * 128)) / math.sqrt(d)).astype(np.float32), "bf16")
    wo = W.store((g.standard_normal((hp * 128, H)) / math.sqrt(hp * 128)).astype(np.float32), "bf16")
    bias = torch.zeros(H, device=DEV)
    logits = torch.empty(B, L, H, device=DEV)
    flags = torch.empty(B, H, L, dtype=torch.uint8, device=DEV)
    ctx = ag.Context(0, ag.gate_mha_workspace_bytes(B, L, d, hp, 128, H))
    ag.ag_gate_mha(ctx, dev(x), dev(w), hp, 128, dev(wo), bias, 0.5, 0, logits, flags)
    ctx.poll_error()
    ctx.close()
    bf = lambda t: t.to(torch.bfloat16).float()
    qkv = bf(torch.from_numpy(x.f32).reshape(B * L, d) @ torch.from_numpy(w.f32)).reshape(B, L, 3, hp, 128).permute(2, 0, 3, 1, 4)
    rows = sorted({0, 1, 63, 64, L // 2, L - 2, L - 1} & set(range(L)))
    for j in rows:
        s = (qkv[0][:, :, j:j + 1] @ qkv[1][:, :, :j + 1].transpose(2, 3)) / math.sqrt(128)
        a = bf(torch.softmax(s, dim=-1) @ qkv[2][:, :, :j + 1]).reshape(B, hp * 128)
        want = a @ torch.from_numpy(wo.f32)
        assert (logits[:, j].cpu() - want).abs().max().item() <= 1e-2, j
