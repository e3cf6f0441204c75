"""Minibatch sizes and filter factors around the tiles of the training
kernels: 32 samples per wavefront, 256 per workgroup, more than 512
workgroups' worth in rounds; one thread per fine x position of a coarse cell."""
import numpy as np
import pytest
import torch

from gpu_util import say
from paper_1909_13772_amd import inputs, wlb

pytestmark = pytest.mark.gpu


def _data(n, seed):
    rng = np.random.default_rng(seed)
    scale = np.array([1e-4] * 6 + [1e-3])
    raw = torch.tensor((rng.standard_normal((n, 7)) * scale).astype(np.float32), device="cuda")
    target = torch.tensor((1e-3 * rng.standard_normal(n) ** 2).astype(np.float32), device="cuda")
    P = torch.tensor(inputs.mlp_params(3, inv_std=1.0 / scale, out_bias=-5.0), device="cuda")
    return P, raw, target


def _grad(P, raw, target):
    n = target.numel()
    g = torch.empty(wlb.MLP_NPARAM, device="cuda")
    loss = torch.empty(1, device="cuda")
    wsb = wlb.wlb_mlp_grad_workspace(n)
    # a poisoned workspace, and a guard behind it that has to stay
    ws = torch.full((wsb // 4 + 64,), float("nan"), device="cuda")
    s = torch.cuda.current_stream()
    wlb.wlb_mlp_grad(P.data_ptr(), raw.data_ptr(), target.data_ptr(), n, 100.0, g.data_ptr(), loss.data_ptr(),
                     ws.data_ptr(), wsb, s.cuda_stream)
    torch.cuda.synchronize()
    assert bool(torch.isnan(ws[wsb // 4:]).all())
    return g.double().cpu().numpy(), float(loss)


@pytest.mark.parametrize("n,part", [(1, 1), (31, 1), (33, 1), (255, 1), (257, 1), (600, 7), (131077, 65536)])
def test_minibatch_gradient_is_the_mean_of_its_parts(n, part):
    """A sample's own gradient does not depend on its place in the minibatch,
    so the minibatch gradient is the weighted mean of its parts' to the
    rounding of FP32 sums (1e-5 of the norm: some 1e-7 sqrt(n) and more)."""
    say(f"case gradient parts n {n}")
    P, raw, target = _data(n, 11)
    g, loss = _grad(P, raw, target)
    ref, lref = np.zeros_like(g), 0.0
    for k in range(0, n, part):
        gp, lp = _grad(P, raw[k:k + part].contiguous(), target[k:k + part].contiguous())
        w = min(part, n - k) / n
        ref += w * gp
        lref += w * lp
    assert np.isfinite(g).all() and not g[:14].any()
    for a, b in ((14, 238), (238, 270), (270, 1294), (1294, 1326), (1326, 1358), (1358, 1359)):
        assert np.linalg.norm(g[a:b] - ref[a:b]) <= 1e-5 * np.linalg.norm(ref[a:b]), (a, b)
    assert abs(loss - lref) <= 1e-5 * lref


def test_infinite_target_stays_in_its_own_terms():
    """One infinite target makes the loss infinite, as any FP32 sum would."""
    P, raw, target = _data(64, 12)
    target[5] = float("inf")
    _, loss = _grad(P, raw, target)
    assert loss == float("inf")


@pytest.mark.parametrize("fac,cells", [(1, (37, 3, 2)), (3, (23, 2, 5)), (4, (65, 3, 2)), (5, (52, 2, 1)), (130, (2, 1, 1)),
                                       (257, (1, 1, 1))])
@pytest.mark.parametrize("steps", [0, 1])
def test_box_filter_factors(fac, cells, steps):
    """Averages over factor^3 cells against the library's own per-cell
    moments: factors that do and do not divide a workgroup, one coarse cell
    per workgroup, and one wider than a workgroup."""
    dom = tuple(fac * c for c in cells)
    say(f"case filter {fac} {dom} steps {steps}")
    rho, u = inputs.random_state(dom, seed=5, umag=0.01)
    B = wlb.Blocks(wlb.single_block(dom), dom, (1, 1, 1), stencil=9, storage=wlb.F32)
    try:
        B.init(wlb.SRT, wlb.make_params(tau=0.7, force=(1e-5, 0, 0)), rho, u)
        B.step(steps)
        r, v, _ = B.moments()
        nc = cells[0] * cells[1] * cells[2]
        out = torch.full((10 * nc,), float("nan"), dtype=torch.float64, device="cuda")
        wlb.wlb_box_filter(B.h, fac, out.data_ptr())
        got = out.cpu().numpy().reshape(10, nc)
    finally:
        B.close()

    def avg(a):
        return a.reshape(cells[2], fac, cells[1], fac, cells[0], fac).mean(axis=(1, 3, 5)).reshape(-1)

    ref = [avg(r)] + [avg(v[a]) for a in range(3)] + [avg(v[a] * v[b]) for a, b in
                                                      ((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))]
    for k in range(10):  # FP64 sums of factor^3 terms of one size
        assert np.abs(got[k] - ref[k]).max() <= 1e-15 * fac ** 3 * max(1e-30, np.abs(r).max() if k == 0 else 0.02), k
