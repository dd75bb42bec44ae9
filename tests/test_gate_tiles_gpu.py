"""The gate's launch shapes against the oracle: 16-token tiles (few tokens) with one to eight feature chunks per wave and
more, ragged last tiles, sequences shorter than a tile, one and two column tiles; streams of tiles; the fp32 gate at odd
sizes."""
import math

import numpy as np
import pytest

from gpu_util import ensure_built
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
