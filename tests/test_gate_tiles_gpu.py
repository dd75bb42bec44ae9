"""The gate's launch shapes against the oracle: 16-token tiles (few tokens) with one to eight feature chunks per wave and
more, ragged last tiles, sequences shorter than a tile, one and two column tiles; streams of tiles; the fp32 gate at odd
sizes."""
import math

import numpy as np
import pytest
import torch

import paper_2410_12876_amd as ag
from gpu_util import DEV, dev, ensure_built, make_ctx
from test_parity_gpu import check_gate, rand_t

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    ensure_built()


@pytest.mark.parametrize("dtype,B,L,d_in,H,n_sink", [
    ("bf16", 1, 1, 64, 4, 0), ("bf16", 1, 5, 192, 32, 0), ("bf16", 1, 17, 512, 16, 1), ("bf16", 1, 15, 576, 20, 0), ("bf16", 9, 3, 1024, 32, 1),
    ("bf16", 2, 333, 2048, 8, 0), ("bf16", 1, 100, 4096, 12, 3), ("bf16", 1, 48, 8192, 32, 0), ("bf16", 1, 40, 4160, 28, 0),
    ("bf16", 1, 4095, 512, 32, 0), ("bf16", 2, 4096, 128, 4, 0), ("bf16", 1, 33, 256, 7, 0),
    # two or more 16-token tiles per CU stream through persistent workgroups
    ("bf16", 1, 8192, 64, 4, 0), ("bf16", 3, 3001, 1088, 12, 1), ("bf16", 1, 8321, 4096, 32, 0), ("bf16", 700, 13, 512, 7, 2),
    ("bf16", 1, 8200, 4160, 8, 0),
    ("f32", 1, 1, 3, 1, 0), ("f32", 5, 7, 130, 17, 2), ("f32", 1, 257, 1021, 32, 0), ("f32", 2, 50, 64, 16, 0)])
def test_gate_tiles(dtype, B, L, d_in, H, n_sink):
    x = rand_t(71, (B, L, d_in), dtype, 0.5)
    w = rand_t(72, (d_in, H), dtype, 1.0 / math.sqrt(d_in))
    bias = np.random.default_rng(73).standard_normal(H).astype(np.float32) * 0.2
    check_gate(x, w, bias, 0.5, n_sink, 1e-4 if dtype == "bf16" else 2e-5)


@pytest.mark.parametrize("L,d_in,H,by", [(8200, 512, 32, 1), (8192, 128, 6, 4), (40, 4096, 32, 3)])
def test_gate_features_at_any_even_address(L, d_in, H, by):
    """Features that do not start at a multiple of 16 bytes, few and many tokens: bit for bit what aligned ones give."""
    x, w = dev(rand_t(74, (1, L, d_in), "bf16", 0.5)), dev(rand_t(75, (d_in, H), "bf16", 1.0 / math.sqrt(d_in)))
    moved = torch.zeros(x.numel() + 8, dtype=x.dtype, device=DEV)[by:by + x.numel()].view(x.shape).copy_(x)
    assert moved.data_ptr() % 16 == 2 * by
    bias = torch.zeros(H, device=DEV)
    ctx = make_ctx(1, L, H, H, 64, ag.AG_BF16, d_in=d_in)
    got = []
    for t in (x, moved):
        logits, flags = torch.zeros(1, L, H, device=DEV), torch.full((1, H, L), 7, dtype=torch.uint8, device=DEV)
        ag.ag_gate(ctx, t, w, bias, 0.5, 1, logits, flags)
        got.append((logits, flags))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1]) and got[0][0].abs().max() > 0.1
    ctx.close()
