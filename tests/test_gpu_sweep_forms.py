"""Launch forms that differ only in how the cells are cut up: strips of
consecutive cells against boxes, slot strides, one- and two-level sums, slabs
of fields.  Populations agree bit for bit; sums agree to the rounding of the
order of their terms."""
import math

import numpy as np
import pytest

from gpu_util import say
from paper_1909_13772_amd import inputs, wlb

pytestmark = pytest.mark.gpu

# rounding of an FP64 sum of n terms: no chain of additions is longer than 64
# (16 tiles per thread, then trees), and each term is rounded itself
SUM_EPS = 66 * 2.0**-53


def _solid(dom, seed, share):
    rng = np.random.default_rng(seed)
    return (rng.random((dom[2], dom[1], dom[0])) < share).astype(np.uint8)


# rows of one cell, of a few, just around a strip and its wavefronts, and
# longer than a strip
@pytest.mark.parametrize("dom", [(1, 9, 40), (3, 50, 7), (31, 5, 9), (64, 6, 5), (101, 7, 6), (160, 5, 4), (250, 4, 3), (257, 3, 5), (600, 3, 2)])
@pytest.mark.parametrize("storage", [wlb.F64, wlb.F32, wlb.F16DEV, wlb.BF16DEV])
def test_strips_match_boxes(dom, storage):
    """The default sweeps (strips, closure-free kernels) and box tiles write
    the same bits, on every parity, with walls, and with obstacles that change
    between two inits of one block set."""
    say(f"case strips {dom} storage {storage}")
    rho, u = inputs.random_state(dom, seed=3, umag=0.01)
    p = wlb.make_params(tau=0.7, magic=3 / 16, force=(1e-5, 0.0, 1e-6))
    xs = [dom[0] // 2, dom[0] - dom[0] // 2] if dom[0] > 1 else [1]
    blocks, _ = inputs.rectilinear_blocks(xs, [dom[1] // 3, dom[1] - dom[1] // 3], [1, dom[2] - 1])
    out = []
    for tiles in (None, (32, 4, 2)):
        B = wlb.Blocks(blocks, dom, (1, 0, 1), stencil=19, storage=storage)
        try:
            if tiles:
                B.set_tiles(*tiles)
            got = []
            for solid in (_solid(dom, 1, 0.2), None, _solid(dom, 2, 0.1)):
                B.init(wlb.TRT, p, rho, u, solid)
                for n in (1, 2, 16):
                    B.step(n)
                    got.append(B.pdfs_get())
            out.append(got)
        finally:
            B.close()
    for k, (a, b) in enumerate(zip(*out)):
        assert np.array_equal(a, b), k


# arrays of 274, 114 and 206 MB, whose strips pad rows of 250 cells to whole
# lines, and the same rows just below the sizes from which they do
@pytest.mark.parametrize("dom,storage", [((250, 170, 170), wlb.BF16DEV), ((250, 120, 50), wlb.F32), ((250, 120, 45), wlb.F64),
                                         ((250, 160, 160), wlb.BF16DEV), ((250, 75, 50), wlb.F32), ((250, 30, 34), wlb.F64)])
def test_long_strips_match_boxes(dom, storage):
    say(f"case long strips {dom} storage {storage}")
    rho, u = inputs.random_state(dom, seed=9, umag=0.01)
    p = wlb.make_params(tau=0.7, magic=3 / 16, force=(1e-5, 0.0, 1e-6))
    out = []
    for tiles in (None, (64, 4, 1)):
        B = wlb.Blocks(wlb.single_block(dom), dom, (1, 0, 1), stencil=19, storage=storage)
        try:
            if tiles:
                B.set_tiles(*tiles)
            B.init(wlb.TRT, p, rho, u, _solid(dom, 5, 0.05) if storage == wlb.F32 else None)
            for n in (3, 1):
                B.step(n)
                out.append(B.moments()[:2])
        finally:
            B.close()
    for k in (0, 1):
        assert all(np.array_equal(a, b) for a, b in zip(out[k], out[2 + k])), k


@pytest.mark.parametrize(
    "collision,q,smagorinsky",
    [(wlb.SRT, 9, False), (wlb.SRT, 15, True), (wlb.TRT, 19, True), (wlb.MRT, 19, True), (wlb.MRT, 27, False),
     (wlb.KBC, 27, False), (wlb.CUMULANT, 27, False), (wlb.CUMULANT, 27, True)])
def test_strips_match_boxes_collisions(collision, q, smagorinsky):
    dom = (90, 11, 1 if q == 9 else 7)
    say(f"case strips collision {collision} q {q} closure {smagorinsky}")
    rho, u = inputs.random_state(dom, seed=3, umag=0.01)
    kw = dict(closure=wlb.CLOSURE_SMAG, cs_smag=0.15) if smagorinsky else {}
    p = wlb.make_params(tau=0.6, **kw)
    out = []
    for tiles in (None, (32, 4, 2)):
        B = wlb.Blocks(wlb.single_block(dom), dom, (1, 1, 1), stencil=q, storage=wlb.F32)
        try:
            if tiles:
                B.set_tiles(*tiles)
            B.init(collision, p, rho, u)
            B.step(5)
            out.append(B.pdfs_get())
        finally:
            B.close()
    assert np.array_equal(*out)


@pytest.mark.parametrize("autotune", [0, 1])
@pytest.mark.parametrize("dom,storage", [((168, 160, 157), wlb.F32), ((130, 129, 128), wlb.F64), ((300, 250, 240), wlb.F32)])
def test_slot_strides(dom, storage, autotune):
    """Slots of 16 MiB (17, 17 and 69 MiB here) and more, at each stride."""
    say(f"case slot strides {dom} storage {storage} autotune {autotune}")
    rho, u = inputs.random_state(dom, seed=5, umag=0.01)
    ref = None
    for kib in (0, 2048, 16384, None):
        B = wlb.Blocks(wlb.single_block(dom), dom, (1, 1, 1), stencil=19, storage=storage)
        try:
            if kib is not None:
                B.set_slot_round(kib)
            B.init(wlb.TRT, wlb.make_params(tau=0.8, autotune=autotune), rho, u)
            B.step(3)
            d = B.pdfs_get()
        finally:
            B.close()
        ref = d if ref is None else ref
        assert np.array_equal(d, ref), kib


@pytest.mark.parametrize("tiles", [(256, 1, 1), (35, 2, 1)])
def test_sums_over_few_and_many_tiles(tiles):
    """Totals and force over 1,680 tiles (one level of sums) and over 4,900
    (two levels, groups not full): against exact sums of the fields and
    against the force from the other partition."""
    dom = (70, 70, 70)
    say(f"case sums {tiles}")
    rho, u = inputs.random_state(dom, seed=6, umag=0.01)
    solid = _solid(dom, 4, 0.05)
    p = wlb.make_params(tau=0.7, force=(1e-5, 0.0, 0.0))
    got = []
    for t in (None, tiles):
        B = wlb.Blocks(wlb.single_block(dom), dom, (1, 0, 1), stencil=19, storage=wlb.F64)
        try:
            if t:
                B.set_tiles(*t)
            B.init(wlb.TRT, p, rho, u, solid)
            B.step(3)
            r, uu, tot = B.moments()
            _, _, alone = B.moments(fields=False)
            assert np.abs(tot - alone).max() <= SUM_EPS * r.size
            got.append((r, tot, B.force(), B.info().n_tiles))
        finally:
            B.close()
    fluid = solid == 0
    n = int(fluid.sum())
    for r, tot, _, _ in got:
        assert abs(tot[0] - math.fsum(r[fluid])) <= SUM_EPS * 1.1 * n
    (_, ta, fa, na), (_, tb, fb, nb) = got
    assert na <= 4096 < nb
    assert fa[6] == fb[6] and fa[7] == fb[7] and fa[6] > 0
    # every link hands over at most 2 (w + |d|) < 0.2
    assert np.abs(fa[:6] - fb[:6]).max() <= SUM_EPS * 0.2 * (fa[6] + fa[7])
    assert np.abs(ta[:4] - tb[:4]).max() <= SUM_EPS * 1.1 * n


@pytest.mark.parametrize("storage", [wlb.F64, wlb.F32])
def test_fields_in_slabs_with_totals(storage):
    """Fields of more than one slab of the staging area (75 MB), taken with
    the totals: the populations' sums, and the totals taken alone."""
    dom = (161, 121, 121)
    say(f"case slabs storage {storage}")
    rho, u = inputs.random_state(dom, seed=8, umag=0.01)
    B = wlb.Blocks(wlb.single_block(dom), dom, (1, 1, 1), stencil=19, storage=storage)
    try:
        B.init(wlb.TRT, wlb.make_params(tau=0.8), rho, u)
        for steps in (1, 1):
            B.step(steps)
            r, uu, tot = B.moments()
            ref = 1.0 + B.pdfs_get().sum(0)
            # 19 terms below 1 summed in FP64 in another order
            assert np.abs(r.reshape(-1) - ref).max() <= 19 * 1e-15
            assert np.abs(tot - B.moments(fields=False)[2]).max() <= SUM_EPS * r.size
            assert abs(tot[0] - math.fsum(r.reshape(-1))) <= SUM_EPS * r.size
            assert np.isfinite(uu).all()
    finally:
        B.close()
