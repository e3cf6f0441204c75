"""Transfers between host arrays and the device at sizes around the pieces
and slabs they are split into: populations set and read back bit for bit, and
fields against the sums of those populations."""
import numpy as np
import pytest

import oracle as O
from gpu_util import say
from paper_1909_13772_amd import inputs, wlb

pytestmark = pytest.mark.gpu


# bytes of populations / fields: 16 KB / 3 KB (one piece), 4.5 MB / 0.9 MB
# (a few threads / none), 86 MB / 18 MB (two slabs of the staging area, every
# thread), and 200 MB / 42 MB in rows of one element
@pytest.mark.parametrize("dom", [(7, 5, 3), (33, 31, 29), (130, 65, 67), (1, 1129, 1163)])
@pytest.mark.parametrize("storage", [wlb.F64, wlb.F32])
def test_populations_and_fields_through_the_host(dom, storage):
    say(f"case host io {dom} storage {storage}")
    n = int(np.prod(dom))
    rng = np.random.default_rng(7)
    rho, u = inputs.random_state(dom, seed=4, umag=0.01)
    B = wlb.Blocks(wlb.single_block(dom), dom, (1, 1, 1), stencil=19, storage=storage)
    try:
        B.init(wlb.TRT, wlb.make_params(tau=0.8), rho, u)
        r0, u0, _ = B.moments()
        d0 = B.pdfs_get()
        for k in range(3):  # the same pinned buffers serve every transfer
            d = (1e-3 * rng.standard_normal((19, n))).astype(np.float32).astype(np.float64)
            B.pdfs_set(d)
            assert np.array_equal(B.pdfs_get(), d), k
            r, uu, _ = B.moments()
            c, _, _ = O.stencil(19)
            ref = 1.0 + d.sum(0)
            # 19 terms of up to 5e-3 summed in FP64 in another order
            assert np.abs(r.reshape(-1) - ref).max() <= 1e-15 * 19
            j = np.asarray(c, np.float64)[:19].T @ d
            assert np.abs(uu.reshape(3, -1) * ref - j).max() <= 1e-15 * 19
        B.pdfs_set(d0)
        r1, u1, _ = B.moments()
        assert np.array_equal(r1, r0) and np.array_equal(u1, u0)
    finally:
        B.close()
