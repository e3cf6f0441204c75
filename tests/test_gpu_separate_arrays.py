"""Block sets whose x-runs keep an array each, with the ghost exchange between
them (domains of 2 GiB and more per population slot; short rows padded to that
bound get there with few cells), against the undivided domain, which is one
array: every velocity set, with solids, walls and density faces, in every
tile form and with the other odd-sweep kernels."""
import numpy as np
import pytest

from gpu_util import say
from paper_1909_13772_amd import inputs, wlb

pytestmark = pytest.mark.gpu

DOM = (2, 2400, 2400)
CELLS = DOM[0] * DOM[1] * DOM[2]
BLOCKS = inputs.rectilinear_blocks([2], [1000, 1400], [1100, 1300])[0]
SMALL = inputs.rectilinear_blocks([1, 1], [800, 1000, 600], [1100, 1300])[0]  # list tiles take up to 1024 cells
_state = {}


def _fields():
    if not _state:
        _state["fields"] = inputs.random_state(DOM, seed=1, umag=0.01)
        solid = (np.random.default_rng(2).random(DOM[::-1]) < 0.1).astype(np.uint8)
        solid[:, :3, :] = 0  # faces of the domain and of the blocks hold both kinds
        _state["solid"] = solid
    return _state["fields"], _state["solid"]


def _run(blocks, periodic, q, storage, coll, solid, kw, steps=(3, 1), **params):
    (rho, u), _ = _fields()
    p = wlb.make_params(tau=0.7, magic=3 / 16, omega_bulk=1.1, **params)
    B = wlb.Blocks(blocks, DOM, periodic, stencil=q, storage=storage)
    try:
        B.init(coll, p, rho, u, solid)
        if "tiles" in kw:
            B.set_tiles(*kw["tiles"])
        B.set_lds_staging(kw.get("lds", 0))
        if kw.get("overlap"):
            B.set_overlap(True)
        out = []
        for n in steps:
            if kw.get("halves"):
                for _ in range(n):
                    B.sweep()
                    B.exchange()
            else:
                B.step(n)
            out.append(B.moments())
        B.exchange()
        out.append((B.force(),))
        out.append((B.pdfs_get(),))
        return out, B.info()
    finally:
        B.close()


FORCE = dict(force=(1e-5, -1e-5, 2e-6))
CASES = [
    # q, collision, storage, periodic, solids, launch form
    (19, wlb.TRT, wlb.F32, (1, 1, 1), False, {}),
    (19, wlb.TRT, wlb.F32, (1, 1, 1), True, {}),
    (19, wlb.TRT, wlb.F64, (0, 1, 1), True, dict(halves=True)),
    (19, wlb.TRT, wlb.F32, (1, 0, 1), True, dict(lds=1)),
    (19, wlb.TRT, wlb.F32, (1, 1, 1), True, dict(overlap=True)),
    (19, wlb.TRT, wlb.F32, (1, 1, 1), True, dict(overlap=True, lds=1)),
    (19, wlb.TRT, wlb.F32, (1, 1, 1), True, dict(tiles=(2, 16, 4, 0))),
    (19, wlb.TRT, wlb.F32, (1, 1, 0), True, dict(tiles=(-1, 0, 0, 0), small=True)),
    (19, wlb.TRT, wlb.F32, (1, 1, 1), True, dict(tiles=(-1, 0, 0, -1), small=True, overlap=True)),
    (27, wlb.MRT, wlb.F32, (1, 1, 1), True, {}),
    (27, wlb.MRT, wlb.F32, (1, 1, 1), True, dict(lds=1)),
    (27, wlb.KBC, wlb.F16DEV, (1, 1, 1), True, {}),
    (15, wlb.SRT, wlb.BF16DEV, (0, 1, 0), True, dict(overlap=True)),
]


@pytest.mark.parametrize("q,coll,storage,periodic,solids,kw", CASES)
def test_separate_arrays_match_one_array(q, coll, storage, periodic, solids, kw):
    say(f"case separate q{q} coll{coll} storage {storage} {periodic} solids {solids} {kw}")
    solid = _fields()[1] if solids else None
    a, info = _run(SMALL if kw.get("small") else BLOCKS, periodic, q, storage, coll, solid, kw, **FORCE)
    assert info.xchg_elems > 0 and info.overlap == int(kw.get("overlap", False)) and info.lds_staging == kw.get("lds", 0)
    b, _ = _run(wlb.single_block(DOM), periodic, q, storage, coll, solid, {}, **FORCE)
    for k, (x, y) in enumerate(zip(a[:2], b[:2])):
        assert np.array_equal(x[0], y[0]) and np.array_equal(x[1], y[1]), k
        # FP64 sums of other tiles: chains of at most 300 additions, terms below 1.2
        assert np.abs(x[2] - y[2]).max() <= 300 * 2.0**-53 * 1.2 * CELLS, k
    fa, fb = a[2][0], b[2][0]
    assert fa[6] == fb[6] and fa[7] == fb[7]
    assert np.abs(fa[:6] - fb[:6]).max() <= 300 * 2.0**-53 * 0.3 * (fa[6] + fa[7])
    assert np.array_equal(a[3][0], b[3][0])


@pytest.mark.parametrize("q,odd,lds", [(19, 0, 0), (19, 1, 0), (19, 1, 1), (27, 1, 0)])
def test_every_slot_is_written_once_between_separate_arrays(q, odd, lds):
    """As in the smaller block sets: one sweep and its exchange write every slot
    of every fluid cell once, and no solid cell."""
    say(f"case separate coverage q{q} odd{odd} lds{lds}")
    (rho, u), solid = _fields()
    B = wlb.Blocks(BLOCKS, DOM, (1, 1, 1), stencil=q, storage=wlb.F32)
    try:
        B.init(wlb.TRT, wlb.make_params(tau=0.8, magic=3 / 16), rho, u, solid)
        B.set_lds_staging(lds)
        c = B.write_coverage(odd)
    finally:
        B.close()
    fluid = solid.reshape(-1) == 0
    for k in range(q):
        row = c[k]
        assert row[fluid].min() == 1 and row[fluid].max() == 1 and not row[~fluid].any(), k


def test_separate_arrays_of_aligned_rows():
    """Rows of whole lines (33 FP64 cells start on a line, with ghost cells
    apart), 110 million cells in four arrays."""
    dom = (33, 1833, 1833)
    say(f"case separate aligned {dom}")
    n = dom[0] * dom[1] * dom[2]
    k = np.arange(n, dtype=np.int64)
    rho = 1.0 + 1e-3 * (k % 11)
    u = np.empty((3, n))
    for a, m in enumerate((7, 13, 17)):
        np.multiply(k % m, 1e-3 / m, out=u[a])
    del k
    blocks, _ = inputs.rectilinear_blocks([20, 13], [833, 1000], [900, 933])
    got = []
    for bl in (blocks, wlb.single_block(dom)):
        B = wlb.Blocks(bl, dom, (0, 1, 1), stencil=15, storage=wlb.F64)
        try:
            B.init(wlb.TRT, wlb.make_params(tau=0.7, magic=3 / 16, force=(1e-5, 0, 0)), rho, u)
            B.step(3)
            B.exchange()
            got.append((B.info().xchg_elems, *B.moments()[:2]))
        finally:
            B.close()
    assert got[0][0] > 0 and got[1][0] == 0
    assert np.array_equal(got[0][1], got[1][1]) and np.array_equal(got[0][2], got[1][2])
