"""Timed cases of the library's own work: what a program that runs it does.

A case is a dict of plain values; ``listed()`` gives the standing ones and
``draw(rng)`` further ones of the same ranges.  ``prepare`` makes what a
program holds before the call (a block set with its state, or the buffers of
a training loop), ``run`` is one pass through the public entry points, and
``exact`` is the same result from a plain FP64 implementation in torch that
shares nothing with the library.

Kinds of pass
  flow        advance a flow by a number of steps and fetch density, velocity
              and the conserved totals (with obstacles also the force on them)
  checkpoint  write the populations of a running flow to the host, restore
              them and go on
  les_data    box-filter a fine flow and make training pairs of the closure
  train       one optimiser step of the closure network
"""
from __future__ import annotations

import math
import os

import numpy as np
import torch

from paper_1909_13772_amd import inputs, wlb

DEVICE = "cuda"
STORAGE = {"f64": wlb.F64, "f32": wlb.F32, "f16": wlb.F16DEV, "bf16": wlb.BF16DEV}
COLLISION = {"srt": wlb.SRT, "trt": wlb.TRT, "mrt": wlb.MRT, "kbc": wlb.KBC}
CLOSURE = {"none": wlb.CLOSURE_NONE, "smagorinsky": wlb.CLOSURE_SMAG, "mlp": wlb.CLOSURE_MLP}


def _flow(name, nx, ny, nz, steps, **kw):
    """A flow case: defaults are a periodic D3Q19 TRT flow in FP32."""
    c = {"name": name, "kind": "flow", "nx": nx, "ny": ny, "nz": nz, "steps": steps, "q": 19, "collision": "trt",
         "closure": "none", "storage": "f32", "tau": 0.8, "start": "turbulence", "u0": 0.05, "wall_y": False,
         "force_x": 0.0, "pressure_x": False, "blocks": 1, "solid": 0.0, "force_out": False, "autotune": False}
    c.update(kw)
    return c


def listed():
    return [
        # The smallest flow in use: the Taylor-Green validation box, where
        # launches and latency count, not bandwidth.
        _flow("taylor_green_32_f64", 32, 32, 32, 100, collision="srt", storage="f64", start="taylor_green", u0=0.01),
        # Monitoring a small obstacle flow: a few steps, then drag and fields;
        # ragged sizes (rows of no whole wavefronts), walls and spheres.
        _flow("obstacles_ragged_f32", 101, 53, 61, 20, wall_y=True, force_x=1e-5, solid=0.1, u0=0.01,
              force_out=True),
        # The channel of the headline benchmark (walls in y, body force) in
        # the two storage types it is quoted in, tuned as a long run tunes it.
        _flow("channel_256_f64", 256, 256, 256, 200, storage="f64", wall_y=True, force_x=1e-6, u0=0.01, autotune=True),
        _flow("channel_256_f32", 256, 256, 256, 200, wall_y=True, force_x=1e-6, u0=0.01, autotune=True),
        # Decaying turbulence in the 16-bit storage types: a large box, fields
        # every 100 steps as the precision ladder takes them; and a box whose
        # rows are no multiple of anything, without the autotuner.
        _flow("turbulence_320_f16", 320, 320, 320, 100, storage="f16", autotune=True),
        _flow("turbulence_ragged_bf16", 250, 150, 190, 100, storage="bf16"),
        # Porous medium on 512 uneven blocks: D3Q27 MRT, pressure-driven,
        # ghost exchange every step.
        _flow("porous_512_blocks_f32", 0, 0, 0, 200, q=27, collision="mrt", pressure_x=True, blocks=8, solid=0.3,
              u0=0.0, start="rest", autotune=True),
        # Large-eddy simulation with the learned closure; its fields are kept
        # in the storage's precision (the closure's own resolution).
        _flow("les_128_mlp", 128, 128, 128, 200, collision="srt", closure="mlp", tau=0.505, u0=0.03),
        # Entropic collision of under-resolved turbulence.
        _flow("entropic_160_kbc", 160, 160, 160, 100, q=27, collision="kbc", tau=0.51, u0=0.03, autotune=True),
        # Checkpoint and resume of a running flow.
        {"name": "checkpoint_128_f32", "kind": "checkpoint", "nx": 128, "ny": 128, "nz": 128, "storage": "f32"},
        # Closure training data from a fine run: box filter and target pairs.
        {"name": "les_data_256", "kind": "les_data", "nx": 256, "ny": 256, "nz": 256, "factor": 4},
        # One optimiser step of the closure network at the training minibatch.
        {"name": "train_16384", "kind": "train", "n": 16384},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(("flow", "porous", "checkpoint", "les_data", "train"), (6, 2, 1, 1, 2))[0]
    if kind == "train":  # minibatches and validation sets
        return {"kind": "train", "n": _log_int(rng, 512, 262144)}
    if kind == "les_data":
        fac = rng.choice((2, 3, 4))
        return {"kind": "les_data", "nx": fac * rng.randint(12, 240 // fac), "ny": fac * rng.randint(12, 240 // fac),
                "nz": fac * rng.randint(12, 240 // fac), "factor": fac}
    if kind == "checkpoint":
        return {"kind": "checkpoint", "nx": rng.randint(24, 128), "ny": rng.randint(24, 128),
                "nz": rng.randint(24, 128), "storage": rng.choice(("f64", "f32", "f16", "bf16"))}
    if kind == "porous":
        return _unnamed(_flow("", rng.randint(0, 999), 0, 0, rng.randint(20, 120), q=rng.choice((19, 27)),
                              collision="mrt", storage=rng.choice(("f64", "f32")), pressure_x=True,
                              blocks=rng.choice((2, 4, 8)), solid=rng.choice((0.1, 0.2, 0.3)), u0=0.0, start="rest",
                              autotune=rng.random() < 0.5))
    q = rng.choice((19, 19, 19, 27, 15))
    coll = rng.choice({19: ("srt", "trt", "trt", "mrt"), 27: ("mrt", "kbc", "trt"), 15: ("srt", "trt")}[q])
    storage = rng.choice(("f64", "f32", "f32", "f16", "bf16"))
    closure = "none"
    if q == 19 and coll in ("srt", "trt") and storage != "f64":
        closure = rng.choice(("none", "none", "smagorinsky", "mlp"))
    wall = coll != "kbc" and rng.random() < 0.5
    c = _flow("", _log_int(rng, 24, 256), _log_int(rng, 24, 256), _log_int(rng, 24, 256), _log_int(rng, 10, 120), q=q,
              collision=coll, closure=closure, storage=storage, tau=round(rng.uniform(0.55, 0.9), 3), wall_y=wall,
              force_x=1e-6 if wall and coll != "mrt" else 0.0, u0=0.02, autotune=rng.random() < 0.5)
    return _unnamed(c)


def _unnamed(c):
    c.pop("name")
    return c


# --- inputs ----------------------------------------------------------------
def _layout(case):
    """Blocks and domain.  Porous cases: a rectilinear grid of blocks^3 uneven
    blocks, edges drawn from {16, 24, 32} (nx seeds a drawn case's edges)."""
    if case.get("blocks", 1) > 1:
        return inputs.uneven_blocks(case["nx"], case["blocks"], (16, 24, 32))
    dom = (case["nx"], case["ny"], case["nz"])
    return wlb.single_block(dom), dom


def _modes(dom, u0, seed, nmodes=6, kmax=4):
    """Density (ones) and a smooth solenoidal velocity: a few random Fourier
    modes, made on the GPU.  Device FP64 arrays (nz, ny, nx), (3, nz, ny, nx)."""
    rng = np.random.default_rng(seed)
    nx, ny, nz = dom
    f64 = dict(dtype=torch.float64, device=DEVICE)
    x = torch.arange(nx, **f64).view(1, 1, nx) * (2 * math.pi / nx)
    y = torch.arange(ny, **f64).view(1, ny, 1) * (2 * math.pi / ny)
    z = torch.arange(nz, **f64).view(nz, 1, 1) * (2 * math.pi / nz)
    u = torch.zeros(3, nz, ny, nx, **f64)
    for _ in range(nmodes if u0 else 0):
        k = np.zeros(3)
        while not k.any():
            k = rng.integers(-kmax, kmax + 1, 3).astype(float)
        kk = k / np.array(dom)  # direction in lattice units
        a = np.cross(rng.standard_normal(3), kk)
        a *= u0 * math.sqrt(2.0 / nmodes) / max(np.linalg.norm(a), 1e-12)
        s = torch.sin(k[0] * x + k[1] * y + k[2] * z + rng.uniform(0, 2 * math.pi))
        for c in range(3):
            u[c] += float(a[c]) * s
    return torch.ones(nz, ny, nx, **f64), u


def _start(case, seed):
    """Host density and velocity and the solid mask (or None) of a flow."""
    dom = _layout(case)[1]
    solid = None
    if case["solid"]:
        solid, _, _ = inputs.spheres(dom, seed, solid_fraction=case["solid"],
                                     periodic=(0 if case["pressure_x"] else 1, 0 if case["wall_y"] else 1, 1),
                                     clear_x=4 if case["pressure_x"] else 0)
    if case["start"] == "rest":
        rho, u = inputs.uniform_state(dom)
        rho *= 1.0 + 1e-4 * (seed % 97) / 97.0
        return rho, u, solid
    if case["start"] == "taylor_green":
        rho, u = inputs.taylor_green(dom[0], case["u0"] * (1.0 + 0.1 * (seed % 97) / 97.0), dom[2])
        return rho, u, solid
    rho, u = _modes(dom, case["u0"], seed)
    return rho.cpu().numpy(), u.cpu().numpy(), solid


def _mlp_weights():
    """The trained closure network of the repository."""
    return np.load(os.path.join(os.path.dirname(inputs.__file__), "mlp_closure.npy")).astype(np.float32)


def _flow_state(case, seed):
    blocks, dom = _layout(case)
    rho, u, solid = _start(case, seed)
    pr = case["pressure_x"]
    mlp = _mlp_weights() if case["closure"] == "mlp" else None
    p = wlb.make_params(tau=case["tau"], force=(case["force_x"], 0.0, 0.0), closure=CLOSURE[case["closure"]],
                        cs_smag=0.1 if case["closure"] != "none" else 0.0, mlp=mlp, pressure_axis=0 if pr else -1,
                        rho_in=1.0005, rho_out=0.9995, autotune=1 if case["autotune"] else 0)
    B = wlb.Blocks(blocks, dom, (0 if pr else 1, 0 if case["wall_y"] else 1, 1), stencil=case["q"],
                   storage=STORAGE[case["storage"]])
    B.init(COLLISION[case["collision"]], p, rho, u, solid)
    return B


def _as_flow(case):
    """The flow behind a checkpoint or training-data case."""
    if case["kind"] == "checkpoint":
        return _flow("", case["nx"], case["ny"], case["nz"], 3, storage=case["storage"], u0=0.05)
    return _flow("", case["nx"], case["ny"], case["nz"], 2, collision="srt", tau=0.51, u0=0.05)


N_PARAM = 1359
TRAIN_STEP = 1000  # a step in mid-training: the moment buffers are filled


def _train_data(case, seed):
    """Parameters, optimiser moments, features and targets of a minibatch,
    with the sizes of the closure's training pairs: stresses of some 1e-4,
    densities of some 1e-3, positive targets of some 1e-3."""
    rng = np.random.default_rng(seed)
    n = case["n"]
    scale = np.array([1e-4] * 6 + [1e-3])
    raw = (rng.standard_normal((n, 7)) * scale).astype(np.float32)
    target = (1e-3 * np.abs(rng.standard_normal(n)) ** 2).astype(np.float32)
    P = inputs.mlp_params(seed, mean=np.zeros(7), inv_std=1.0 / scale, out_bias=math.log(math.expm1(1e-3)))
    m = np.zeros(N_PARAM, np.float32)
    v = np.zeros(N_PARAM, np.float32)
    m[14:] = 1e-2 * rng.standard_normal(N_PARAM - 14)
    v[14:] = 1e-3 * (0.1 + rng.random(N_PARAM - 14))
    return P, m, v, raw, target


LR, B1, B2, EPS = 2e-3, 0.9, 0.999, 1e-8
INV_SCALE = 500.0


def prepare(case, seed):
    kind = case["kind"]
    if kind == "train":
        P, m, v, raw, target = (torch.tensor(a, device=DEVICE) for a in _train_data(case, seed))
        s = torch.cuda.Stream()
        wsb = wlb.wlb_mlp_grad_workspace(case["n"])
        st = {"kind": kind, "n": case["n"], "P": P, "m": m, "v": v, "raw": raw, "target": target, "stream": s,
              "grad": torch.zeros_like(P), "loss": torch.zeros(1, device=DEVICE), "step": TRAIN_STEP,
              "ws": torch.empty(wsb, dtype=torch.uint8, device=DEVICE), "wsb": wsb}
        torch.cuda.synchronize()
        return st
    if kind == "flow":
        return {"kind": kind, "B": _flow_state(case, seed), "steps": case["steps"], "force": case["force_out"],
                "single": case["closure"] == "mlp"}
    flow = _as_flow(case)
    B = _flow_state(flow, seed)
    B.step(flow["steps"])
    B.synchronize()
    if kind == "checkpoint":
        return {"kind": kind, "B": B}
    fac = case["factor"]
    nc = (case["nx"] // fac, case["ny"] // fac, case["nz"] // fac)
    n3 = nc[0] * nc[1] * nc[2]
    return {"kind": kind, "B": B, "factor": fac, "nc": nc, "tau0": 0.5025,
            "filt": torch.empty(10, n3, dtype=torch.float64, device=DEVICE),
            "raw": torch.empty(n3, 7, dtype=torch.float32, device=DEVICE),
            "target": torch.empty(n3, dtype=torch.float32, device=DEVICE)}


def run(state):
    kind = state["kind"]
    if kind == "flow":
        B = state["B"]
        B.step(state["steps"])
        out = {}
        if state["force"]:
            out["force"] = B.force()
        out["rho"], out["u"], out["totals"] = B.moments()
        if state["single"]:
            out["rho"], out["u"] = out["rho"].astype(np.float32), out["u"].astype(np.float32)
        return out
    if kind == "checkpoint":
        B = state["B"]
        d = B.pdfs_get()
        B.pdfs_set(d)
        B.step(2)
        B.synchronize()
        return {"d": d}
    if kind == "les_data":
        B = state["B"]
        wlb.wlb_box_filter(B.h, state["factor"], state["filt"].data_ptr())
        wlb.wlb_les_targets(state["filt"].data_ptr(), state["nc"], state["tau0"], state["raw"].data_ptr(),
                            state["target"].data_ptr(), B.stream.cuda_stream)
        return {"filt": state["filt"], "raw": state["raw"], "target": state["target"]}
    s = state["stream"].cuda_stream
    wlb.wlb_mlp_grad(state["P"].data_ptr(), state["raw"].data_ptr(), state["target"].data_ptr(), state["n"], INV_SCALE,
                     state["grad"].data_ptr(), state["loss"].data_ptr(), state["ws"].data_ptr(), state["wsb"], s)
    state["step"] += 1
    wlb.wlb_mlp_adam(state["P"].data_ptr(), state["grad"].data_ptr(), state["m"].data_ptr(), state["v"].data_ptr(),
                     state["step"], LR, B1, B2, EPS, s)
    return {"grad": state["grad"], "loss": state["loss"], "P": state["P"], "m": state["m"], "v": state["v"]}


def work(case):
    """Bytes and operations of one pass.  A step reads and writes every
    population once (and a mask word per cell where there are solids); fields
    are written once in FP64."""
    kind = case["kind"]
    if kind == "train":
        n = case["n"]
        macs = 7 * 32 + 32 * 32 + 32  # per sample; forward, and twice that backward
        return {"bytes": 32 * n + 4 * N_PARAM * 8, "flops": 6 * macs * n}
    if kind != "flow":
        flow = _as_flow(case)
        n = case["nx"] * case["ny"] * case["nz"]
        eb = wlb.ELEM_BYTES[STORAGE[flow["storage"]]]
        if kind == "checkpoint":  # populations out in FP64 and back in, then two steps
            return {"bytes": n * 19 * (2 * eb + 2 * 8 + 4 * eb), "flops": 2 * 300 * n}
        nc = n // case["factor"] ** 3
        return {"bytes": n * 19 * eb + nc * (2 * 80 + 32), "flops": 60 * n}
    dom = _layout(case)[1]
    n = dom[0] * dom[1] * dom[2]
    eb = wlb.ELEM_BYTES[STORAGE[case["storage"]]]
    q = case["q"]
    fluid = n * (1.0 - case["solid"])
    flops = {"srt": 15, "trt": 15, "mrt": 25, "kbc": 50}[case["collision"]] * q
    if case["closure"] == "mlp":
        flops += 2 * (7 * 32 + 32 * 32 + 32) + 64 * 20
    return {"bytes": case["steps"] * (fluid * 2 * q * eb + (4 * n if case["solid"] else 0)) + n * (q * eb + 32),
            "flops": case["steps"] * fluid * flops}


# --- the same in plain FP64 -------------------------------------------------
C27 = [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1), (1, 1, 0), (-1, -1, 0),
       (1, -1, 0), (-1, 1, 0), (1, 0, 1), (-1, 0, -1), (1, 0, -1), (-1, 0, 1), (0, 1, 1), (0, -1, -1), (0, 1, -1),
       (0, -1, 1), (1, 1, 1), (-1, -1, -1), (1, 1, -1), (-1, -1, 1), (1, -1, 1), (-1, 1, -1), (-1, 1, 1), (1, -1, -1)]
WEIGHTS = {15: (2 / 9, 1 / 9, 0.0, 1 / 72), 19: (1 / 3, 1 / 18, 1 / 36, 0.0), 27: (8 / 27, 2 / 27, 1 / 54, 1 / 216)}


def _opp(i):
    return 0 if i == 0 else (i + 1 if i % 2 else i - 1)


class _Plain:
    """A plain FP64 run of a flow on the whole lattice: two arrays, collide,
    then stream."""

    def __init__(self, case, seed):
        self.case = case
        q = case["q"]
        self.C = C27[:7] + C27[19:] if q == 15 else C27[:q]
        self.W = [WEIGHTS[q][sum(a * a for a in c)] for c in self.C]
        self.q = q
        self.F = [case["force_x"], 0.0, 0.0]
        rho, u, solid = _start(case, seed)
        rho = torch.tensor(rho, device=DEVICE)
        u = torch.tensor(u, device=DEVICE)
        nz, ny, nx = self.shape = tuple(rho.shape)
        self.solid = None if solid is None else torch.tensor(solid, device=DEVICE).bool()
        self.wall_y, self.press = case["wall_y"], case["pressure_x"]
        uu = (u * u).sum(0)
        self.d = torch.stack([self.W[i] * (rho - 1 + rho * self._e(i, u, uu)) for i in range(q)])
        if self.solid is not None:
            self.d[:, self.solid] = 0.0
        # links by the population that comes in along i: bounced back, or
        # through a density face
        self.bounce, self.face = [], []
        for i, (cx, cy, cz) in enumerate(self.C):
            b = torch.zeros(self.shape, dtype=torch.bool, device=DEVICE)
            f = torch.zeros(self.shape, dtype=torch.bool, device=DEVICE)
            if self.press and cx:
                f[:, :, 0 if cx > 0 else nx - 1] = True
            if self.solid is not None:
                b |= torch.roll(self.solid, (cz, cy, cx), (0, 1, 2)) & ~f
            if self.wall_y and cy:
                w = torch.zeros_like(b)
                w[:, 0 if cy > 0 else ny - 1, :] = True
                # beyond the wall there is nothing, whatever the roll brought
                b |= w
            f &= ~b
            self.bounce.append(b if bool(b.any()) else None)
            self.face.append(f if bool(f.any()) else None)
        if case["collision"] == "mrt" or case["collision"] == "kbc":
            ex = [e for e in ((a, b, c) for a in range(3) for b in range(3) for c in range(3))
                  if q == 27 or 0 in e]  # D3Q19: no moment with an xyz factor
            M = np.array([[float(cx) ** a * float(cy) ** b * float(cz) ** c for cx, cy, cz in self.C] for a, b, c in ex])
            self.ex, self.M = ex, torch.tensor(M, device=DEVICE)
            self.Mi = torch.tensor(np.linalg.inv(M), device=DEVICE)
        if case["closure"] == "mlp":
            self.net = _net(torch.tensor(_mlp_weights(), device=DEVICE))

    def _cdot(self, i, v):
        r = 0.0
        for a in range(3):
            if self.C[i][a]:
                r = r + self.C[i][a] * v[a]
        return r

    def _e(self, i, u, uu):
        cu = self._cdot(i, u)
        return 3 * cu + 4.5 * cu * cu - 1.5 * uu

    def macro(self):
        d = self.d
        drho = d.sum(0)
        j = []
        for a in range(3):
            s = torch.zeros_like(drho)
            for i in range(self.q):
                if self.C[i][a]:
                    s += self.C[i][a] * d[i]
            j.append(s + 0.5 * self.F[a])
        rho = 1 + drho
        u = torch.stack([v / rho for v in j])
        return drho, rho, u

    def step(self, force=None):
        case, q, d, F = self.case, self.q, self.d, self.F
        drho, rho, u = self.macro()
        uu = (u * u).sum(0)
        feq = lambda i: self.W[i] * (drho + rho * self._e(i, u, uu))  # noqa: E731
        om = 1.0 / case["tau"]
        if case["closure"] != "none":
            pi = [torch.zeros_like(rho) for _ in range(6)]
            for i in range(1, q):
                n = d[i] - feq(i)
                cx, cy, cz = self.C[i]
                for k, cc in enumerate((cx * cx, cy * cy, cz * cz, cx * cy, cx * cz, cy * cz)):
                    if cc:
                        pi[k] += cc * n
            k = 18 * math.sqrt(2.0) * 0.1 ** 2
            pp = pi[0] ** 2 + pi[1] ** 2 + pi[2] ** 2 + 2 * (pi[3] ** 2 + pi[4] ** 2 + pi[5] ** 2)
            tau = 0.5 * (case["tau"] + torch.sqrt(case["tau"] ** 2 + k * torch.sqrt(pp) / rho))
            if case["closure"] == "mlp":
                o, bad = _net_forward(self.net, torch.stack(pi + [drho], -1).reshape(-1, 7))
                tau = torch.where(bad.view_as(tau), tau, case["tau"] + torch.nn.functional.softplus(o).view_as(tau))
            om = 1.0 / tau
        post = torch.empty_like(d)
        if case["collision"] in ("srt", "trt"):
            omm = om
            if case["collision"] == "trt":
                tau = 1.0 / om
                omm = 1.0 / (0.5 + (3.0 / 16.0) / (tau - 0.5))
            uF = sum(u[a] * F[a] for a in range(3))
            for i in range(0, q):
                o = _opp(i)
                if i % 2 == 0 and i:
                    continue
                cu, cF = self._cdot(i, u), self._cdot(i, F)
                ep = self.W[i] * (drho + rho * (4.5 * cu * cu - 1.5 * uu))
                Fp = self.W[i] * (9 * cu * cF - 3 * uF)
                if i == 0:
                    post[0] = d[0] - om * (d[0] - ep) + (1 - om / 2) * Fp
                    continue
                em, Fm = self.W[i] * 3 * rho * cu, self.W[i] * 3 * cF
                sp = -om * (0.5 * (d[i] + d[o]) - ep) + (1 - om / 2) * Fp
                sm = -omm * (0.5 * (d[i] - d[o]) - em) + (1 - omm / 2) * Fm
                post[i] = d[i] + sp + sm
                post[o] = d[o] + sp - sm
        else:  # no body force in these cases
            eq = torch.stack([feq(i) for i in range(q)])
            neq = (d - eq).view(q, -1)
            m = self.M @ neq
            at = {e: k for k, e in enumerate(self.ex)}
            dg = [at[(2, 0, 0)], at[(0, 2, 0)], at[(0, 0, 2)]]
            tr = (m[dg[0]] + m[dg[1]] + m[dg[2]]) / 3
            if case["collision"] == "kbc":
                s = torch.zeros_like(m)
                for k in dg:
                    s[k] = m[k] - tr
                for e in ((1, 1, 0), (1, 0, 1), (0, 1, 1)):
                    s[at[e]] = m[at[e]]
                s = self.Mi @ s
                h = neq - s
                f = eq.view(q, -1) + torch.tensor(self.W, dtype=torch.float64, device=DEVICE).view(q, 1)
                sh, hh = (s * h / f).sum(0), (h * h / f).sum(0)
                ib = 2.0 / om
                gamma = torch.where(hh > 1e-30, ib - (2 - ib) * sh / hh, torch.full_like(hh, 2.0))
                post = d - (om * s + 0.5 * om * gamma * h).view_as(d)
            else:  # trace and higher moments at rate 1
                r = m.clone()
                for e, k in at.items():
                    if sum(e) == 2 and k not in dg:
                        r[k] = om * m[k]
                    elif sum(e) <= 1:
                        r[k] = 0.0
                for k in dg:
                    r[k] = om * (m[k] - tr) + 1.0 * tr
                post = d - (self.Mi @ r).view_as(d)
        if self.solid is not None:
            post[:, self.solid] = 0.0
        if force is not None:
            self._force(post, force)
        new = torch.empty_like(d)
        for i, (cx, cy, cz) in enumerate(self.C):
            t = torch.roll(post[i], (cz, cy, cx), (0, 1, 2))
            if self.bounce[i] is not None:
                t = torch.where(self.bounce[i], post[_opp(i)], t)
            if self.face[i] is not None:
                rw = 1.0005 if cx > 0 else 0.9995
                cu = self._cdot(i, u)
                a = -post[_opp(i)] + 2 * self.W[i] * (rw - 1 + rw * (4.5 * cu * cu - 1.5 * uu))
                t = torch.where(self.face[i], a, t)
            new[i] = t
        if self.solid is not None:
            new[:, self.solid] = 0.0
        self.d = new

    def _force(self, post, out):
        """Momentum handed to solids and walls by the links that bounce."""
        fluid = ~self.solid
        ny = self.shape[1]
        for i in range(1, self.q):
            b = self.bounce[_opp(i)]  # leaving along i comes back along opp(i)
            if b is None:
                continue
            cy = self.C[i][1]
            wall = torch.zeros_like(b)
            if self.wall_y and cy:
                wall[:, ny - 1 if cy > 0 else 0, :] = True
            for k, sel in ((0, b & fluid & ~wall), (3, b & fluid & wall)):
                f = (post[i][sel] + self.W[i]).sum()
                for a in range(3):
                    out[k + a] += 2 * self.C[i][a] * float(f)
                out[6 if k == 0 else 7] += int(sel.sum())

    def fields(self):
        drho, rho, u = self.macro()
        n = rho.numel()
        if self.solid is not None:
            rho = torch.where(self.solid, 0.0, rho)
            u = torch.where(self.solid, 0.0, u)
            drho = torch.where(self.solid, 0.0, drho)
            n = int((~self.solid).sum())
        return drho, rho, u, n


def _net(P):
    """Network parameters as FP64 tensors; matrix operands rounded to bf16,
    which is part of the network's definition."""
    P = P.double()
    r = _bf16
    return {"mean": P[:7], "istd": P[7:14], "W1": r(P[14:238].view(32, 7)), "b1": P[238:270],
            "W2": r(P[270:1294].view(32, 32)), "b2": P[1294:1326], "w3": r(P[1326:1358]), "b3": P[1358]}


def _bf16(x):
    return x.float().to(torch.bfloat16).double()


def _gelu(z):
    return 0.5 * z * (1 + torch.special.erf(z / math.sqrt(2.0)))


def _net_forward(net, raw):
    x = (raw - net["mean"]) * net["istd"]
    h1 = _bf16(_gelu(_bf16(x) @ net["W1"].T + net["b1"]))
    h2 = _bf16(_gelu(h1 @ net["W2"].T + net["b2"]))
    o = h2 @ net["w3"] + net["b3"]
    return o, (x.abs() > 8).any(-1) | ~torch.isfinite(o)


def _exact_train(case, seed):
    P32, m, v, raw, target = _train_data(case, seed)
    P, m, v, raw, t = (torch.tensor(a, device=DEVICE).double() for a in (P32, m, v, raw, target))
    net = _net(P)
    n = case["n"]
    x = _bf16((raw - net["mean"]) * net["istd"])
    z1 = x @ net["W1"].T + net["b1"]
    h1 = _bf16(_gelu(z1))
    z2 = h1 @ net["W2"].T + net["b2"]
    h2 = _bf16(_gelu(z2))
    o = h2 @ net["w3"] + net["b3"]
    res = (torch.nn.functional.softplus(o) - t) * INV_SCALE
    slope = lambda z: 0.5 * (1 + torch.special.erf(z / math.sqrt(2))) + z * torch.exp(-z * z / 2) / math.sqrt(2 * math.pi)  # noqa: E731,E501
    go = 2 * res * INV_SCALE * torch.sigmoid(o) / n
    g2 = go[:, None] * net["w3"] * slope(z2)
    g1 = (g2 @ net["W2"]) * slope(z1)
    g = torch.cat([torch.zeros(14, dtype=torch.float64, device=DEVICE), (g1.T @ x).reshape(-1), g1.sum(0),
                   (g2.T @ h1).reshape(-1), g2.sum(0), go @ h2, go.sum()[None]])
    m[14:] = B1 * m[14:] + (1 - B1) * g[14:]
    v[14:] = B2 * v[14:] + (1 - B2) * g[14:] ** 2
    k = TRAIN_STEP + 1
    P[14:] -= LR * (m[14:] / (1 - B1 ** k)) / (torch.sqrt(v[14:] / (1 - B2 ** k)) + EPS)
    return {"grad": g, "loss": (res ** 2).mean()[None], "P": P, "m": m, "v": v}


def _exact_les_data(case, seed):
    s = _Plain(_as_flow(case), seed)
    for _ in range(_as_flow(case)["steps"]):
        s.step()
    _, rho, u, _ = s.fields()
    f = case["factor"]
    nz, ny, nx = s.shape
    avg = lambda a: a.view(nz // f, f, ny // f, f, nx // f, f).mean((1, 3, 5))  # noqa: E731
    pairs = ((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))
    ch = [avg(rho)] + [avg(u[a]) for a in range(3)] + [avg(u[a] * u[b]) for a, b in pairs]
    R, U = ch[0], ch[1:4]
    dim = {0: 2, 1: 1, 2: 0}  # x is the last axis
    G = [[0.5 * (torch.roll(U[b], -1, dim[a]) - torch.roll(U[b], 1, dim[a])) for b in range(3)] for a in range(3)]
    S = [0.5 * (G[a][b] + G[b][a]) for a, b in pairs]
    T = [ch[4 + k] - U[a] * U[b] for k, (a, b) in enumerate(pairs)]
    tr = (T[0] + T[1] + T[2]) / 3
    T = [T[k] - tr for k in range(3)] + T[3:]
    dot = lambda A, B: A[0] * B[0] + A[1] * B[1] + A[2] * B[2] + 2 * (A[3] * B[3] + A[4] * B[4] + A[5] * B[5])  # noqa: E731,E501
    dtau = 3 * torch.clamp(-dot(T, S) / (2 * dot(S, S) + 1e-30), min=0.0)
    raw = torch.stack([-(2 / 3) * R * (0.5025 + dtau) * S[k] for k in range(6)] + [R - 1], -1)
    return {"filt": torch.stack(ch).view(10, -1), "raw": raw.reshape(-1, 7), "target": dtau.reshape(-1)}


def exact(case, seed):
    with torch.no_grad():
        kind = case["kind"]
        if kind == "train":
            return _exact_train(case, seed)
        if kind == "les_data":
            return _exact_les_data(case, seed)
        flow = case if kind == "flow" else _as_flow(case)
        s = _Plain(flow, seed)
        if kind == "checkpoint":
            for _ in range(flow["steps"]):
                s.step()
            return {"d": s.d.view(19, -1).cpu().numpy()}
        out = {}
        force = [0.0] * 8 if flow["force_out"] else None
        for k in range(flow["steps"]):
            s.step(force if k == flow["steps"] - 1 else None)
        drho, rho, u, n = s.fields()
        uu = (u * u).sum(0)
        if force is not None:
            out["force"] = np.array(force)
        out["rho"], out["u"] = rho.cpu().numpy(), u.cpu().numpy()
        mom = [float((rho * u[a]).sum()) for a in range(3)]
        out["totals"] = np.array([n + float(drho.sum()), *mom, 0.5 * float((rho * uu).sum()), math.sqrt(float(uu.max())),
                                  float(n), float(flow["steps"])])
        return out
