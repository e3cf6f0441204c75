"""Fields and populations fetched into, and taken from, every kind of host
array: pageable and pinned, whole and one field alone, at sizes around the
ways a transfer can go."""
import numpy as np
import pytest
import torch

from gpu_util import say
from paper_1909_13772_amd import inputs, wlb

pytestmark = pytest.mark.gpu


def _array(n, pinned):
    a = torch.full((n,), float("nan"), dtype=torch.float64, pin_memory=True).numpy() if pinned else np.full(n, np.nan)
    return a


# fields of 0.1, 0.4, 0.9, 1.2, 2.0, 2.2, 3.9, 5.6 and 93 MB (two slabs)
@pytest.mark.parametrize("dom", [(15, 15, 15), (24, 24, 24), (30, 31, 32), (33, 33, 33), (40, 40, 40), (41, 41, 41),
                                 (50, 49, 50), (56, 56, 56), (143, 143, 143)])
def test_fields_alone_and_into_any_memory(dom):
    n = int(np.prod(dom))
    say(f"case host arrays {dom}")
    rho, u = inputs.random_state(dom, seed=4, umag=0.01)
    solid = (np.random.default_rng(2).random((dom[2], dom[1], dom[0])) < 0.1).astype(np.uint8)
    B = wlb.Blocks(wlb.single_block(dom), dom, (1, 0, 1), stencil=19, storage=wlb.F32)
    try:
        B.init(wlb.TRT, wlb.make_params(tau=0.8), rho, u, solid)
        for steps in (1, 1):
            B.step(steps)
            r0, u0, tot0 = B.moments()
            r0, u0 = r0.reshape(-1), u0.reshape(-1)
            d = B.pdfs_get()
            fluid = solid.reshape(-1) == 0
            # 19 terms below 1 summed in FP64 in another order
            assert np.abs(r0 - 1.0 - d.sum(0))[fluid].max() <= 19e-15
            for want_r, want_u, want_t in ((1, 0, 0), (0, 1, 0), (1, 0, 1), (0, 1, 1), (1, 1, 0), (1, 1, 1)):
                for pr, pu in ((0, 0), (1, 1), (1, 0), (0, 1)):
                    r, v, t = _array(n, pr), _array(3 * n, pu), np.full(8, np.nan)
                    wlb.wlb_moments_get(B.h, r if want_r else None, v if want_u else None, t if want_t else None)
                    assert np.array_equal(r, r0) if want_r else np.isnan(r).all()
                    assert np.array_equal(v, u0) if want_u else np.isnan(v).all()
                    assert np.array_equal(t, tot0) if want_t else np.isnan(t).all()
    finally:
        B.close()


@pytest.mark.parametrize("dom", [(9, 7, 5), (33, 33, 33), (70, 71, 72), (101, 99, 100)])
def test_populations_and_initial_fields_from_any_memory(dom):
    n = int(np.prod(dom))
    say(f"case host populations {dom}")
    rng = np.random.default_rng(5)
    rho, u = inputs.random_state(dom, seed=5, umag=0.01)
    B = wlb.Blocks(wlb.single_block(dom), dom, (1, 1, 1), stencil=19, storage=wlb.F64)
    try:
        states = []
        for pinned in (0, 1):
            r, v = _array(n, pinned), _array(3 * n, pinned)
            r[:], v[:] = rho.reshape(-1), u.reshape(-1)
            B.init(wlb.TRT, wlb.make_params(tau=0.8), r, v)
            B.step(2)
            states.append(B.pdfs_get())
        assert np.array_equal(*states)
        for pin_in, pin_out in ((0, 1), (1, 0), (1, 1)):
            a, b = _array(19 * n, pin_in), _array(19 * n, pin_out)
            a[:] = 1e-3 * rng.standard_normal(19 * n)
            wlb.wlb_pdfs_set(B.h, a)
            wlb.wlb_pdfs_get(B.h, b)
            assert np.array_equal(a, b), (pin_in, pin_out)
    finally:
        B.close()


def test_handles_of_several_threads_share_the_buffers():
    """Four handles, a thread and a stream each, step and fetch at the same
    time, and are closed and made anew meanwhile: every fetch is what the
    handle alone gives."""
    import threading

    say("case host threads")
    doms = [(20, 20, 20), (64, 60, 62), (90, 91, 92), (130, 65, 67)]
    want, got, errors = {}, {}, []

    def work(dom, out):
        try:
            rho, u = inputs.random_state(dom, seed=dom[0], umag=0.01)
            out[dom] = []
            for _ in range(3):
                B = wlb.Blocks(wlb.single_block(dom), dom, (1, 1, 1), stencil=19, storage=wlb.F32)
                try:
                    B.init(wlb.TRT, wlb.make_params(tau=0.8), rho, u)
                    for n in (3, 2):
                        B.step(n)
                        r, v, t = B.moments()
                        d = B.pdfs_get()
                        B.pdfs_set(d)
                        out[dom].append((r, v, t, d, B.moments()[1]))
                finally:
                    B.close()
        except Exception as e:  # noqa: BLE001
            errors.append((dom, e))

    for d in doms:
        work(d, want)
    th = [threading.Thread(target=work, args=(d, got)) for d in doms]
    for t in th:
        t.start()
    for t in th:
        t.join()
    assert not errors, errors
    for d in doms:
        for a, b in zip(want[d], got[d]):
            assert all(np.array_equal(x, y) for x, y in zip(a, b)), d
