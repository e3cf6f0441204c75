"""Tiles of the sweeps that follow the cache hints: strips of consecutive
cells, or whole rows where every access of the odd sweep is hinted."""
import numpy as np
import pytest

from gpu_util import say
from paper_1909_13772_amd import inputs, wlb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,strips", [(70, False), (200, False), (64, True), (192, True)])
@pytest.mark.parametrize("storage", [wlb.F64, wlb.F32, wlb.F16DEV])
def test_hints_change_between_sweeps(nx, strips, storage):
    """Rows of whole wavefronts keep the strips with every access hinted, others
    go back to boxes; the bits do not depend on it, whenever it changes."""
    dom = (nx, 11, 9)
    say(f"case hints {dom} storage {storage}")
    rho, u = inputs.random_state(dom, seed=3, umag=0.01)
    solid = (np.random.default_rng(1).random((9, 11, nx)) < 0.1).astype(np.uint8)
    p = wlb.make_params(tau=0.7, magic=3 / 16, force=(1e-5, 0.0, 1e-6))
    states = []
    for hints in ([], [(1, 1), (0, 2), (1, 1), (0, 0), (1, 0)]):
        B = wlb.Blocks(wlb.single_block(dom), dom, (1, 0, 1), stencil=19, storage=storage)
        try:
            B.init(wlb.TRT, p, rho, u, solid)
            default = B.info().n_tiles
            for k in range(5):
                if hints:
                    B.set_nontemporal(*hints[k])
                    boxes = hints[k][1] == 1 and not strips
                    # strips are cut across rows: ceil(cells / 256) of them
                    assert (B.info().n_tiles == default) == (not boxes), hints[k]
                B.sweep()
                B.exchange()
                B.step(16)
                B.step(2)
            states.append(B.pdfs_get())
        finally:
            B.close()
    assert np.array_equal(*states)
