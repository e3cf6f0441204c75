"""What the training gradient is made of: the bf16 operands of each sample,
decided by FP32 activations, and one order of FP32 additions over the samples.
Training runs are compared step by step with earlier ones, so both are part of
the result."""
import numpy as np
import pytest
import torch
from scipy.special import erfc

from gpu_util import say
from paper_1909_13772_amd import inputs, wlb

pytestmark = pytest.mark.gpu

CHUNK, ROW = 64, 256  # samples added in turn; four such sums, added in turn, per workspace row
W1, B1, W2, B2, W3, B3 = 14, 238, 270, 1294, 1326, 1358
INV = 100.0


def _data(n, seed, wide=1.0):
    rng = np.random.default_rng(seed)
    scale = np.array([1e-4] * 6 + [1e-3])
    raw = (rng.standard_normal((n, 7)) * scale * wide).astype(np.float32)
    target = (1e-3 * rng.standard_normal(n) ** 2).astype(np.float32)
    P = inputs.mlp_params(3, inv_std=1.0 / scale, out_bias=-5.0).astype(np.float32)
    return P, raw, target


def _grads(P, raw, target, parts, alloc=True):
    """Gradient and loss of each slice in `parts`."""
    dP, draw, dt = (torch.tensor(a, device="cuda") for a in (P, raw, target))
    g = torch.full((len(parts), wlb.MLP_NPARAM), float("nan"), device="cuda")
    loss = torch.full((len(parts),), float("nan"), device="cuda")
    wsb = max(wlb.wlb_mlp_grad_workspace(b - a) for a, b in parts)
    ws = torch.full((wsb // 4,), float("nan"), device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    for k, (a, b) in enumerate(parts):
        args = (dP.data_ptr(), draw[a:].data_ptr(), dt[a:].data_ptr(), b - a, INV, g[k].data_ptr(), loss[k:].data_ptr())
        if alloc:
            wlb.wlb_mlp_grad(*args, ws.data_ptr(), wsb, st)
        else:
            wlb.wlb_mlp_grad_noalloc(*args, st)
    torch.cuda.synchronize()
    return g.cpu().numpy(), loss.cpu().numpy()


@pytest.mark.parametrize("n", [2, 64, 128, 512, 2048])
@pytest.mark.parametrize("alloc", [True, False])
def test_samples_are_added_in_one_order(n, alloc):
    """A minibatch of 2^k samples scales each sample's terms by 2^-k without
    rounding, so its gradient is, bit for bit, the terms of one-sample
    minibatches added up in FP32 in the documented order."""
    say(f"case gradient order n {n}")
    P, raw, target = _data(n, 21)
    one, lone = _grads(P, raw, target, [(k, k + 1) for k in range(n)], alloc)
    (got,), (lgot,) = _grads(P, raw, target, [(0, n)], alloc)
    f = np.float32
    terms = one * f(1.0 / n)
    assert np.array_equal(terms.astype(np.float64), one.astype(np.float64) / n)  # nothing became subnormal
    grad, loss = np.zeros(wlb.MLP_NPARAM, f), f(0)
    for r in range(0, n, ROW):
        row, sq = np.zeros(wlb.MLP_NPARAM, f), f(0)
        for c in range(r, min(n, r + ROW), CHUNK):
            a = np.zeros(wlb.MLP_NPARAM, f)
            for q in range(c, min(n, c + CHUNK)):
                a = a + terms[q]
            row = row + a
        for q in range(r, min(n, r + ROW)):
            sq = sq + lone[q]
        grad, loss = grad + row, loss + sq
    assert not got[:W1].any()
    assert np.array_equal(got, grad)
    assert lgot == loss / f(n)


def _bf16(a):
    return torch.tensor(np.asarray(a, np.float64)).to(torch.float32).to(torch.bfloat16).to(torch.float64).numpy()


@pytest.mark.parametrize("wide", [1.0, 3.0])
def test_operands_and_terms_of_single_samples(wide):
    """One-sample minibatches show the operands (dW / db of a layer are its
    inputs): they are bf16 values next to the FP64 activations of the layer
    before, and the terms are those of the chain rule at these operands."""
    n = 512
    say(f"case gradient operands wide {wide}")
    P, raw, target = _data(n, 22, wide)
    g, loss = _grads(P, raw, target, [(k, k + 1) for k in range(n)])
    g, P64 = g.astype(np.float64), P.astype(np.float64)
    w1, w2, w3 = _bf16(P[W1:B1]).reshape(32, 7), _bf16(P[W2:B2]).reshape(32, 32), _bf16(P[W3:B3])
    b1, b2, b3 = P64[B1:W2], P64[B2:W3], P64[B3]

    def cdf(z):
        return 0.5 * erfc(-z / np.sqrt(2.0))

    def slope(z):
        return cdf(z) + z * np.exp(-0.5 * z * z) / np.sqrt(2.0 * np.pi)

    def operand(gw, gb):
        """The inputs behind dW = db x input, from the unit of largest db."""
        j = np.abs(gb).argmax(1)
        i = np.arange(n)
        q = gw[i, j] / gb[i, j][:, None]
        b = _bf16(q)
        # product rounded to FP32 and divided: within 2^-23 of the bf16 value
        assert np.all(np.abs(q - b) <= 2.0**-22 * np.abs(b))
        return b

    def decided(h, z, zerr):
        """h is bf16(GELU(z)), or its neighbour where the FP32 error of GELU
        (z itself, and up to 50 ulp in the far negative tail) spans the
        boundary."""
        a = z * cdf(z)
        half = np.exp2(np.floor(np.log2(np.maximum(np.abs(a), 1e-300))) - 8)
        return np.all(np.abs(h - a) <= half * (1 + 2.0**-14) + 50 * 2.0**-24 * np.abs(a) + 1.2 * zerr)

    x32 = (raw - P[:7]) * P[7:14]  # both operations round in FP32, as in the kernel
    x = operand(g[:, W1:B1].reshape(n, 32, 7), g[:, B1:W2])
    assert np.array_equal(x, _bf16(x32))
    h1 = operand(g[:, W2:B2].reshape(n, 32, 32), g[:, B2:W3])
    z1 = x @ w1.T + b1
    e1 = 9 * 2.0**-24 * (np.abs(x) @ np.abs(w1).T + np.abs(b1))
    assert decided(h1, z1, e1)
    h2 = operand(g[:, None, W3:B3], g[:, B3:])
    z2 = h1 @ w2.T + b2
    e2 = 34 * 2.0**-24 * (np.abs(h1) @ np.abs(w2).T + np.abs(b2))
    assert decided(h2, z2, e2)
    o = h2 @ w3 + b3
    sp = np.logaddexp(0.0, o)
    res = (sp - target.astype(np.float64)) * INV
    go = 2.0 * res * INV / (1.0 + np.exp(-o))
    eo = 34 * 2.0**-24 * (np.abs(h2) @ np.abs(w3) + abs(b3))
    # softplus by log1p(exp): a few ulp; the residual cancels against the target
    esp = eo + 8 * 2.0**-24 * np.maximum(sp, np.abs(target))
    ego = 2.0 * INV * INV / (1.0 + np.exp(-o)) * esp + np.abs(go) * (eo + 16 * 2.0**-24)
    assert np.all(np.abs(g[:, B3] - go) <= ego)
    assert np.all(np.abs(loss - res * res) <= 2 * np.abs(res) * INV * esp + 8 * 2.0**-24 * res * res)
    # from here on with the kernel's own d loss / d o; slopes carry 2^-20
    go = g[:, B3:]
    es = 2.0**-20 + 1.2 * e2
    gz2 = go * w3 * slope(z2)
    eg2 = np.abs(go * w3) * es + 4 * 2.0**-24 * np.abs(gz2)
    assert np.all(np.abs(g[:, B2:W3] - gz2) <= eg2)
    gz2 = g[:, B2:W3]
    back = gz2 @ w2
    eb = 34 * 2.0**-24 * (np.abs(gz2) @ np.abs(w2))
    gz1 = back * slope(z1)
    assert np.all(np.abs(g[:, B1:W2] - gz1) <= np.abs(back) * (2.0**-20 + 1.2 * e1) + 1.2 * eb + 4 * 2.0**-24 * np.abs(gz1))


def test_infinite_target_reaches_its_own_terms_only():
    """One infinite target among 64: d loss / d o of that sample is -inf, and
    every parameter holds what the chain rule makes of it in extended
    arithmetic (an infinity, or NaN where infinities of both signs meet); the
    other samples add finite terms."""
    say("case gradient infinite target")
    P, raw, target = _data(64, 23)
    (one,), _ = _grads(P, raw[5:6], target[5:6], [(0, 1)])
    target[5] = np.inf
    (got,), (loss,) = _grads(P, raw, target, [(0, 64)])
    assert loss == np.inf and got[B3] == -np.inf and not got[:W1].any()
    # signs of the sample's activations and slopes, from its finite gradient
    sign = np.sign(one) * np.sign(one[B3])
    assert np.array_equal(got[W3:B3], -np.inf * sign[W3:B3])
    assert np.array_equal(got[B2:W3], -np.inf * sign[B2:W3])
    assert np.array_equal(got[W2:B2], -np.inf * sign[W2:B2])
    with np.errstate(invalid="ignore"):
        back = ((-np.inf * sign[B2:W3])[:, None] * _bf16(P[W2:B2]).reshape(32, 32)).sum(0)
    assert np.isnan(back).all()  # every column of W2 has both signs
    assert np.isnan(got[W1:W2]).all()
