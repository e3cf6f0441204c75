"""Block sets laid out as one array over the domain, whose direct sweeps wrap
periodic faces in place, against the separate arrays with a ghost exchange,
the other odd-sweep kernels and the oracle."""
import numpy as np
import pytest

import oracle as O
from gpu_util import gpu_run, oracle_params, oracle_run, pop_err, rel_l2, say
from paper_1909_13772_amd import inputs, wlb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("periodic", [(1, 1, 1), (1, 0, 1)])
def test_separate_arrays_match_one_array(periodic):
    """Short rows padded to more than 2 GiB per slot keep one array per x-run
    and the exchange; the undivided domain is one array.  Populations agree
    bit for bit after an odd and an even number of steps."""
    dom = (2, 2400, 2400)
    say(f"case separate arrays {periodic}")
    rho, u = inputs.random_state(dom, seed=1, umag=0.01)
    p = wlb.make_params(tau=0.7, magic=3 / 16, force=(1e-5, 0.0, 1e-6))
    blocks, _ = inputs.rectilinear_blocks([2], [1000, 1400], [1100, 1300])
    got = []
    for bl in (blocks, wlb.single_block(dom)):
        B = wlb.Blocks(bl, dom, periodic, stencil=9, storage=wlb.F32)
        try:
            B.init(wlb.TRT, p, rho, u)
            out = []
            for n in (3, 1):
                B.step(n)
                out.append(B.pdfs_get())
            B.set_kernel_timing(True)
            B.step(2)
            got.append((out, B.kernel_times()[1]))
        finally:
            B.close()
    assert got[0][1][2:] == [1, 1] and got[1][1][2:] == [0, 0]  # exchanges of the separate arrays only
    for a, b in zip(got[0][0], got[1][0]):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("first,second", [(0, 1), (1, 0), (0, 2), (2, 0), (1, 2)])
@pytest.mark.parametrize("mode", ["step", "split"])
def test_odd_sweep_kernel_changes_between_steps(first, second, mode):
    """Odd-sweep kernels with and without the ghost layer follow each other
    at any step, also between the two halves of a pair."""
    dom = (32, 20, 12)
    say(f"case kernel change {first}->{second} {mode}")
    rho, u = inputs.random_state(dom, seed=2, umag=0.01)
    p = wlb.make_params(tau=0.7, magic=3 / 16, force=(1e-5, 0.0, 1e-6))
    blocks, _ = inputs.rectilinear_blocks([16, 16], [8, 12], [12])

    def advance(B, n):
        if mode == "step":
            B.step(n)
        else:
            for _ in range(n):
                B.sweep()
                B.exchange()

    ref = gpu_run(blocks, dom, (1, 1, 1), 19, wlb.F64, wlb.TRT, p, rho, u, steps=9)
    ref[4].close()
    for before in (1, 2, 3, 4):
        B = wlb.Blocks(blocks, dom, (1, 1, 1), stencil=19, storage=wlb.F64)
        try:
            B.init(wlb.TRT, p, rho, u)
            B.set_lds_staging(first)
            advance(B, before)
            B.set_lds_staging(second)
            r, uu, _ = B.moments()
            advance(B, 9 - before)
            B.exchange()  # repeating the last exchange changes nothing
            assert np.array_equal(B.pdfs_get(), ref[0]), before
        finally:
            B.close()


@pytest.mark.parametrize("ny,nz", [([1], [2]), ([2], [1]), ([1, 2], [2]), ([1, 4], [2, 1, 3]), ([10, 6], [7, 9])])
@pytest.mark.parametrize("nx", [5, 70, 130])
@pytest.mark.parametrize("q,coll", [(19, 1), (27, 2)])
def test_wrapping_in_place_at_small_extents(nx, ny, nz, q, coll):
    """Periodic extents of one to three cells (a cell may sit at both faces of
    an axis), runs away from the domain's origin, short packed rows and rows
    of several wavefronts: FP64 parity with the oracle, which keeps no ghost
    layer and streams by index."""
    blocks, dom = inputs.rectilinear_blocks([nx], ny, nz)
    say(f"case wrap {dom} {ny} {nz} q{q}")
    rho, u = inputs.random_state(dom, seed=3, umag=0.02)
    F = (1e-5, -1e-5, 2e-6)
    p = wlb.make_params(tau=0.7, magic=3 / 16, omega_bulk=1.1, force=F)
    for periodic in ((1, 1, 1), (0, 1, 1), (1, 0, 1)):
        for steps in (4, 5):
            d, r, uu, _, B = gpu_run(blocks, dom, periodic, q, wlb.F64, coll, p, rho, u, steps=steps)
            B.close()
            op = oracle_params(q, coll, 0.7, 3 / 16, periodic, F, omega_bulk=1.1)
            do, ro, uo, _ = oracle_run(op, dom, rho, u, None, steps)
            assert pop_err(d, do, q) <= 1e-12 and rel_l2(uu.reshape(3, -1), uo) <= 1e-12, (periodic, steps)


@pytest.mark.parametrize("he", [0, 5, 16, 24])
def test_long_graph_replays_match_eager_steps(he):
    """Step counts around the longer captured graph (16 steps), replayed with
    eager work and synchronisations between, and health checks due inside,
    at the end of and after a replay: bit for bit the eager steps."""
    say(f"case long graph health {he}")
    dom = (20, 12, 9)
    rho, u = inputs.random_state(dom, seed=6, umag=0.01)
    p = wlb.make_params(tau=0.7, magic=3 / 16, force=(1e-5, 0.0, 1e-6), health_every=he)
    runs = []
    for graph in (True, False):
        B = wlb.Blocks(wlb.single_block(dom), dom, (1, 0, 1), stencil=19, storage=wlb.F64)
        try:
            B.init(wlb.TRT, p, rho, u)
            B.set_graph(graph)
            out = []
            for n in (16, 37, 1, 15, 33, 2, 48):
                B.step(n)
                out.append(B.pdfs_get())
                assert B.info().steps == sum((16, 37, 1, 15, 33, 2, 48)[:len(out)])
            B.set_nontemporal(1, 1)  # drops the captured graphs
            B.step(34)
            out.append(B.pdfs_get())
            runs.append(out)
        finally:
            B.close()
    for k, (a, b) in enumerate(zip(*runs)):
        assert np.array_equal(a, b), k


def test_health_check_stops_a_diverging_run_at_its_step():
    """A run whose velocity leaves the limit is stopped at the first check due,
    as with a graph of one pair."""
    dom = (16, 8, 8)
    rho, u = inputs.uniform_state(dom, u=(0.2, 0.0, 0.0))
    B = wlb.Blocks(wlb.single_block(dom), dom, (1, 1, 1), stencil=19, storage=wlb.F64)
    try:
        B.init(wlb.TRT, wlb.make_params(tau=0.8, health_every=20, health_umax=0.1), rho, u)
        with pytest.raises(wlb.WlbError) as e:
            B.step(100)
        assert e.value.code == wlb.WLB_ERR_DIVERGED and B.info().steps == 20
    finally:
        B.close()


def test_info_reports_the_exchange_that_runs():
    """Nothing where the sweeps cross the faces themselves, the ghost layer
    around the domain for the LDS-staged odd sweep, every face between
    separate arrays."""
    def crossing(n, axes, q):
        """Populations that leave a box of n cells across a y or z face (x
        wraps inside the rows)."""
        c = np.asarray(O.stencil(q)[0])[:q]
        cells = np.stack(np.meshgrid(*[np.arange(v) for v in n], indexing="ij"), -1).reshape(-1, 3)
        out = 0
        for e in c:
            t = cells + e
            m = np.zeros(len(cells), bool)
            for a in axes:
                m |= (t[:, a] < 0) | (t[:, a] >= n[a])
            out += int(m.sum())
        return out

    dom = (32, 20, 12)
    blocks, _ = inputs.rectilinear_blocks([16, 16], [8, 12], [12])
    rho, u = inputs.uniform_state(dom)
    B = wlb.Blocks(blocks, dom, (1, 1, 1), stencil=19, storage=wlb.F64)
    try:
        B.init(wlb.TRT, wlb.make_params(tau=0.8), rho, u)
        assert (B.info().n_xchg_items, B.info().xchg_elems) == (0, 0)
        B.set_lds_staging(1)
        assert B.info().lds_staging == 1 and B.info().xchg_elems == crossing(dom, (1, 2), 19)
        B.set_kernel_timing(True)
        B.step(2)
        assert B.kernel_times()[1][2:] == [1, 1] and B.info().n_xchg_items > 0
        B.set_lds_staging(0)
        assert (B.info().n_xchg_items, B.info().xchg_elems) == (0, 0)
    finally:
        B.close()
    dom = (2, 2400, 2400)
    blocks, _ = inputs.rectilinear_blocks([2], [1000, 1400], [2400])
    B = wlb.Blocks(blocks, dom, (1, 1, 1), stencil=9, storage=wlb.F32)
    try:
        # two faces along y between the two arrays, six populations of D2Q9 each
        assert B.info().n_xchg_items > 0 and B.info().xchg_elems == 2 * 6 * 2 * 2400
    finally:
        B.close()
