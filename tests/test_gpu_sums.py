"""Sums over box tiles at the number from which they go through two levels.
The sums run over whole-row boxes whatever tiles the sweeps take: with rows of
256 cells there is one box per row."""
import math

import numpy as np
import pytest

from gpu_util import say
from paper_1909_13772_amd import inputs, wlb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ny,nz", [(64, 64), (17, 241), (1, 4095), (63, 130)])  # 4,096, 4,097, 4,095 and 8,190 rows
@pytest.mark.parametrize("storage", [wlb.F64, wlb.F32])
def test_totals_and_force_around_two_levels(ny, nz, storage):
    dom = (256, ny, nz)
    say(f"case sums {dom} storage {storage}")
    rho, u = inputs.random_state(dom, seed=6, umag=0.01)
    solid = (np.random.default_rng(4).random((nz, ny, 256)) < 0.05).astype(np.uint8)
    fluid = solid == 0
    B = wlb.Blocks(wlb.single_block(dom), dom, (1, 0, 1), stencil=19, storage=storage)
    try:
        B.init(wlb.TRT, wlb.make_params(tau=0.7), rho, u, solid)
        B.step(3)
        r, v, tot = B.moments()
        alone = B.moments(fields=False)[2]
        f = B.force()
        B.set_tiles(8, 8, 4)  # another partition: 4,096, 5,856, 32,768 and 8,448 boxes
        f4, alone4 = B.force(), B.moments(fields=False)[2]
    finally:
        B.close()
    n = int(fluid.sum())
    # no chain of additions is longer than 140 (64 rows per thread, trees, groups)
    eps = 140 * 2.0**-53 * 1.2 * n
    for t in (tot, alone, alone4):
        assert abs(t[0] - math.fsum(r[fluid])) <= eps
        for a in range(3):
            assert abs(t[1 + a] - math.fsum((r * v[a])[fluid])) <= eps
        assert t[6] == n and abs(t[5] - np.sqrt((v * v).sum(0))[fluid].max()) <= 1e-12
    assert f[6] == f4[6] > 0 and f[7] == f4[7]
    assert np.abs(f[:6] - f4[:6]).max() <= 140 * 2.0**-53 * 0.3 * (f[6] + f[7])
