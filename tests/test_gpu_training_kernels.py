"""Minibatch sizes around the tiles of the gradient kernel: 32 samples per
wavefront, 256 per workgroup, more than 512 workgroups' worth in rounds."""
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
