"""ag_pack_row_off over unit counts and lengths where the count's split over waves changes: one wave, several and all 16 of
a workgroup per unit, units that do not fill the last workgroup, rows of flags that start at odd addresses."""
import numpy as np
import pytest
import torch

import oracle
import paper_2410_12876_amd as ag
from gpu_util import DEV, ensure_built

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    ensure_built()


@pytest.mark.parametrize("B,H,L,room", [(1, 1, 1, 0), (3, 5, 15, 2), (1, 17, 333, 8), (2, 32, 2048, 8), (1, 3, 2049, 1),
                                        (1, 9, 8193, 0), (1, 2, 40001, 5), (70, 16, 33, 3)])
def test_pack_row_off(B, H, L, room):
    g = np.random.default_rng(L + H)
    flags = (g.random((B, H, L)) < g.random((B, H, 1))).astype(np.uint8) * g.integers(1, 256, size=(B, H, L)).astype(np.uint8)
    ctx = ag.Context(0, 4 * B * H + 256)
    df = torch.from_numpy(flags).to(DEV)
    ro = torch.zeros(B * H + 1, dtype=torch.int64, device=DEV)
    need = torch.zeros(1, dtype=torch.int64, device=DEV)
    for total in (10 ** 9, int(flags.astype(bool).sum()) // 2):   # twice in a row: the arrival counter is back at zero
        ag.ag_pack_row_off(ctx, df, room, total, ro, need)
        torch.cuda.synchronize()
        want, want_need = oracle.packed_row_off(flags, room, total)
        assert np.array_equal(ro.cpu().numpy(), want) and int(need.item()) == int(want_need)
    ctx.close()
