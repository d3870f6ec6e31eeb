"""Timing cases of the collision path and of the learned proposal's network.

``listed()`` is the fixed list and ``draw(rng)`` gives further cases of the same
ranges; ``prepare`` makes what a program holds before the call (a context with
its grid, the distribution, a proposal table or the network's weights, output
buffers), ``run`` makes one pass through the public entry points, ``work``
gives the bytes and floating-point operations that pass cannot do without, and
``exact`` computes the same outputs in 64 bits with plain torch (same draws,
nothing of the library), on the GPU if there is one.

Kinds of case:
  term     one collision term on device buffers (qgbe_collision_term)
  noalloc  the same without a context (qgbe_collision_term_noalloc)
  step     `steps` forward-Euler steps from a given f (qgbe_step), f read back
           on the device; `stats` adds the statistics of the last step
  record   training rows for the proposal (qgbe_record_samples)
  grad     the network's loss and gradient of one batch (qgbe_mlp_loss_grad)
  forward  the network's head on given inputs (qgbe_mlp_forward)
  train    `epochs` of Adam over recorded rows (qgbe_train_proposal)
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1912_04457_amd import qgbe
from paper_1912_04457_amd import workloads as W

G = W.GLUON
GLUONS, ALL = 1 << G, 0x7F
SAMPLERS = {"uniform": qgbe.SAMPLER_UNIFORM, "learned": qgbe.SAMPLER_LEARNED, "network": qgbe.SAMPLER_LEARNED,
            "roots": qgbe.SAMPLER_ROOTS, "roots_alt": qgbe.SAMPLER_ROOTS_ALT}
PRECISIONS = {"f64": qgbe.FP64, "f32": qgbe.FP32}
DRIFTS = {"upwind": qgbe.DRIFT_UPWIND, "central": qgbe.DRIFT_CENTRAL}
HBARC = 0.1973269804
K, HIDDEN, N_IN, N_OUT = 8, 128, 8, 88
ALPHA = 0.1                       # defensive uniform share of the proposal tables
LARGEST = 1.6e10                  # samples of the largest listed case
EXACT_SAMPLES = 3e8               # above this many samples exact() would take too long


def _case(name, kind, **kw):
    """A collision case: cells nx x ny x nz, nodes npx x npy x npz."""
    c = dict(name=name, kind=kind, precision="f32", mask=ALL, sampler="uniform", symmetric=True, nx=1, ny=1, nz=1,
             npx=20, npy=20, npz=20, p_half=3.0, samples=256, init="cgc")
    if kind == "step":
        c.update(drift="upwind", steps=1, stats=False, dt=0.01)
    c.update(kw)
    return c


def listed():
    return [
        # The reference-precision gluon cell of the measurement plan: a call of some
        # tens of microseconds, where launches and latency count.
        _case("gluon_cell_f64", "term", precision="f64", mask=GLUONS, npx=10, npy=10, npz=10, p_half=2.0,
              samples=1000),
        # A small FP32 term for callers that must not allocate (serving loops, capture).
        _case("gluon_ragged_noalloc", "noalloc", mask=GLUONS, nx=3, ny=2, npx=13, npy=11, npz=9, p_half=2.0,
              samples=100),
        # The long thermalisation run: many short steps of one gluon cell at 30^3, records
        # taken now and then, so most steps run without statistics.
        _case("gluon_long_run", "step", mask=GLUONS, npx=30, npy=30, npz=30, p_half=2.0, samples=128, steps=10,
              dt=5e-5),
        # The quark-gluon long run: all 70 channels at 30^3, statistics with the step.
        _case("mixture_long_run", "step", npx=30, npy=30, npz=30, p_half=2.0, samples=128, dt=5e-5, stats=True),
        # The pure-gluon spatial run: 256 cells, 2048 samples per point, upwind drift.
        _case("gluon_spatial", "step", mask=GLUONS, nx=16, ny=16, samples=2048, stats=True),
        # The 7-species cell with the plain sampler at the sample count of the fixed-error
        # comparison.
        _case("mixture_cell", "term", samples=4096),
        # The same cell with an installed proposal table.
        _case("mixture_cell_learned", "term", sampler="learned", samples=256),
        # The 7-species spatial run with the network's table re-evaluated on the step's
        # masses: the headline's grid of 16^3 momenta on an eighth of its cells.
        _case("mixture_spatial_network", "step", nx=6, ny=6, nz=6, npx=16, npy=16, npz=16, sampler="network",
              samples=256),
        # Reference precision on a spatial grid, ragged in every axis, central drift.
        _case("mixture_spatial_f64", "step", precision="f64", nx=3, ny=2, nz=2, npx=11, npy=12, npz=10, samples=64,
              drift="central", stats=True, dt=0.002),
        # The stability test of the paper's root parameterisation: direct estimator, 40^3.
        _case("roots_stability", "term", precision="f64", mask=GLUONS, sampler="roots", symmetric=False, npx=40,
              npy=40, npz=40, p_half=2.0, samples=100, init="uniform"),
        # The root parameterisation with symmetric sampling on the 7-species cell.
        _case("roots_symmetric", "term", precision="f64", sampler="roots_alt", npx=15, npy=15, npz=15, p_half=2.0,
              samples=100),
        # Training of the proposal: two epochs of 4096-row batches (forward, backward, Adam).
        dict(name="train_proposal", kind="train", rows=131072, batch=4096, epochs=2),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["term", "term", "term", "step", "step", "noalloc", "record", "grad", "forward", "train"])
    if kind in ("grad", "forward"):
        return dict(kind=kind, rows=_log_int(rng, 64, 16384 if kind == "grad" else 400000))
    if kind == "train":
        return dict(kind=kind, rows=_log_int(rng, 10000, 200000), batch=_log_int(rng, 512, 8192), epochs=1)
    c = _case("", kind)
    del c["name"]
    c["precision"] = rng.choice(["f32", "f32", "f64"])
    c["mask"] = rng.choice([GLUONS, GLUONS, ALL, ALL, 0x01, 0x09, 0x49])
    if kind == "term":
        c["sampler"] = rng.choice(["uniform", "uniform", "learned", "network", "roots", "roots_alt"])
        c["symmetric"] = rng.random() < 0.8
    if kind == "step":
        c.update(drift=rng.choice(["upwind", "central"]), steps=rng.choice([1, 1, 2, 5]),
                 stats=rng.random() < 0.5, dt=0.002)
    if rng.random() < 0.5:
        c.update(nx=rng.randint(1, 6), ny=rng.randint(1, 5), nz=rng.randint(1, 4))
    n = _log_int(rng, 6, 32)
    c.update(npx=n, npy=max(2, n + rng.randint(-2, 2)), npz=max(2, n + rng.randint(-2, 2)))
    c["p_half"] = rng.choice([2.0, 3.0])
    c["samples"] = 4 if kind == "record" else _log_int(rng, 32, 4096)
    # bounded work: fewer samples, then fewer cells
    top = 1e8 if c["precision"] == "f64" or c["sampler"].startswith("roots") else LARGEST / 8
    if kind == "noalloc":
        top = min(top, 1e8)
    elif kind == "record":
        top = 2e7
    while _n_samples(c) > top and c["samples"] > 16:
        c["samples"] = c["samples"] // 2
    while _n_samples(c) > top and c["nx"] * c["ny"] * c["nz"] > 1:
        a = max(("nx", "ny", "nz"), key=lambda k: c[k])
        c[a] -= 1
    while kind == "noalloc" and _cells(c) * _nodes(c) * 7 > 2_000_000 and _cells(c) > 1:
        a = max(("nx", "ny", "nz"), key=lambda k: c[k])
        c[a] -= 1
    return c


# ---- the pieces of a collision case -------------------------------------------

def _cells(c):
    return c["nx"] * c["ny"] * c["nz"]


def _nodes(c):
    return c["npx"] * c["npy"] * c["npz"]


def _n_samples(c):
    return float(_cells(c)) * _nodes(c) * len(_channels(c["mask"])) * c["samples"] * c.get("steps", 1)


def _species(c):
    return [s for s in range(7) if (c["mask"] >> s) & 1]


def _desc(c):
    return dict(n_x=(c["nx"], c["ny"], c["nz"]), n_p=(c["npx"], c["npy"], c["npz"]),
                x_half=(3.0, 3.0, 3.0), p_half=(c["p_half"],) * 3, species_mask=c["mask"],
                precision=PRECISIONS[c["precision"]], symmetric=int(c["symmetric"]),
                drift=DRIFTS[c.get("drift", "upwind")], seed=W.PHILOX_SEED, device=0)


def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _gen(seed):
    g = torch.Generator(device=_device())
    g.manual_seed(seed)
    return g


def _rand(g, *shape, dtype=torch.float64):
    return torch.rand(*shape, generator=g, device=g.device, dtype=dtype)


def _axis(n, half):
    return -half + (torch.arange(n, dtype=torch.float64, device=_device()) + 0.5) * (2.0 * half / n)


def _momenta(c):
    """Node momenta [nodes, 3], pz fastest."""
    ax = [_axis(c[k], c["p_half"]) for k in ("npx", "npy", "npz")]
    return torch.stack(torch.meshgrid(*ax, indexing="ij"), -1).reshape(-1, 3)


def _field(c, seed):
    """f [7][cells][nodes]: the step occupation of gluons with an amplitude of
    its own in every cell and Fermi-Dirac quarks, each value scattered by 10%;
    or occupations uniform in [0, 1] (the stability test)."""
    g = _gen(seed)
    absp = _momenta(c).norm(dim=1)
    f = torch.zeros(7, _cells(c), _nodes(c), dtype=torch.float64, device=g.device)
    amp = 0.2 + 0.8 * _rand(g, _cells(c), 1) if _cells(c) > 1 else torch.ones(1, 1, device=g.device).double()
    for s in _species(c):
        r = _rand(g, _cells(c), _nodes(c))
        if c["init"] == "uniform":
            f[s] = r
        elif s == G:
            f[s] = 0.5 * amp * (absp < 0.5 * c["p_half"]) * (0.9 + 0.2 * r)
        else:
            f[s] = (0.6 + 0.4 * amp) / (torch.exp(absp / 0.3) + 1.0) * (0.9 + 0.2 * r)
    return f


def _table(c, seed):
    """A mixture table (thr int64, mu, sigma float32) for every (channel, node)."""
    g = _gen(seed + 1)
    rows = len(_channels(c["mask"])) * _nodes(c)
    w = -torch.log(_rand(g, rows, K))
    w = w / w.sum(1, keepdim=True)
    cum = torch.cumsum(w, 1) - w
    thr = torch.floor((ALPHA + (1.0 - ALPHA) * cum) * 4294967296.0).clamp(max=4294967295.0).to(torch.int64)
    mu = torch.randn(rows, K, 5, generator=g, device=g.device) * 0.7
    sigma = torch.exp(_rand(g, rows, K, 5, dtype=torch.float32) - 0.3)
    return thr, mu, sigma


def _step_index(seed):
    return seed % 100003


# ---- the network's inputs ------------------------------------------------------

def _weights(seed):
    return W.random_mlp_params(seed % 1000003)


def _rows(n, seed):
    """Rows as qgbe_record_samples writes them: 8 conditioning inputs, the
    logits of 5 uniforms, and the magnitude of the sample value (half of the
    samples fall outside the box and carry 0)."""
    g = _gen(seed)
    dev = g.device
    p = 2.0 * _rand(g, n, 3, dtype=torch.float32) - 1.0
    a = p.norm(dim=1, keepdim=True) / math.sqrt(3.0)
    e = torch.sqrt(a * a + 0.03)
    m = torch.full((n, 1), 0.03, device=dev)
    s = torch.randint(0, 7, (n, 1), generator=g, device=dev).float() / 3.0 - 1.0
    ch = 2.0 * torch.randint(0, 70, (n, 1), generator=g, device=dev).float() / 69.0 - 1.0
    u = _rand(g, n, 5, dtype=torch.float32).clamp(1e-6, 1.0 - 1e-6)
    v = torch.exp(1.5 * torch.randn(n, 1, generator=g, device=dev)) * (_rand(g, n, 1, dtype=torch.float32) < 0.46)
    return torch.cat([p, a, e, m, s, ch, torch.log(u / (1.0 - u)), 1e-4 * v], 1).contiguous()


# ---- one pass ------------------------------------------------------------------

def prepare(case, seed):
    c, dev = case, "cuda"
    st = {"case": c}
    if c["kind"] in ("grad", "forward", "train"):
        st["solver"] = qgbe.Solver(n_p=(8, 8, 8), precision=qgbe.FP32, species_mask=ALL)
        st["w"] = _weights(seed)
        qgbe.qgbe_proposal_set_weights(st["solver"].ctx, st["w"])
        rows = _rows(c["rows"], seed)
        if c["kind"] == "train":
            st["rows"], st["loss"] = rows, np.zeros(c["epochs"])
            st["cfg"] = qgbe.TrainCfg(epochs=c["epochs"], batch=c["batch"], lr=2e-3, lr_final=1e-4, alpha=ALPHA, seed=1)
        else:
            st["X"], st["yw"] = rows[:, :8].contiguous(), rows[:, 8:].contiguous()
            st["grad"] = torch.empty(qgbe.MLP_PARAMS, dtype=torch.float32, device=dev)
            st["Y"] = torch.empty(c["rows"], N_OUT, dtype=torch.float32, device=dev)
        return st
    st["f"] = _field(c, seed)
    st["step"] = _step_index(seed)
    st["out"] = torch.empty_like(st["f"])
    if c["kind"] == "noalloc":
        st["desc"] = qgbe.make_desc(**_desc(c))
        return st
    s = st["solver"] = qgbe.Solver(**_desc(c))
    s.set_f(st["f"])
    if c["kind"] == "record":
        st["rows"] = torch.empty(s.n_channels * _cells(c) * _nodes(c) * c["samples"], qgbe.RECORD_WIDTH,
                                 dtype=torch.float32, device=dev)
    if c["sampler"] == "learned":
        thr, mu, sigma = _table(c, seed)
        # the library reads 32-bit words; torch has no arithmetic on uint32
        thr32 = torch.where(thr > 0x7FFFFFFF, thr - (1 << 32), thr).to(torch.int32)
        qgbe.qgbe_set_proposal_table(s.ctx, thr32, mu, sigma)
    elif c["sampler"] == "network":
        qgbe.qgbe_proposal_set_weights(s.ctx, _weights(seed))
        qgbe.qgbe_proposal_build_table(s.ctx, ALPHA)
    return st


def run(state):
    c, s = state["case"], state.get("solver")
    kind = c["kind"]
    if kind == "train":
        qgbe.qgbe_proposal_set_weights(s.ctx, state["w"])
        qgbe.qgbe_train_proposal(s.ctx, state["rows"], state["cfg"], state["loss"])
        return {"weights": qgbe.qgbe_proposal_get_weights(s.ctx), "loss": state["loss"]}
    if kind == "grad":
        loss = qgbe.qgbe_mlp_loss_grad(s.ctx, state["X"], state["yw"], state["grad"])
        return {"grad": state["grad"], "loss": loss}
    if kind == "forward":
        qgbe.qgbe_mlp_forward(s.ctx, state["X"], state["Y"])
        return state["Y"]
    sampler = SAMPLERS[c["sampler"]]
    if kind == "noalloc":
        qgbe.qgbe_collision_term_noalloc(state["desc"], state["f"], state["step"], c["samples"], sampler, state["out"])
        return state["out"]
    qgbe.qgbe_set_distribution(s.ctx, -1, state["f"])
    qgbe.qgbe_set_step_index(s.ctx, state["step"])
    if kind == "record":
        qgbe.qgbe_record_samples(s.ctx, c["samples"], 1, state["rows"])
        return state["rows"]
    if kind == "term":
        qgbe.qgbe_collision_term(s.ctx, c["samples"], sampler, state["out"])
        return state["out"]
    last = c["steps"] - 1 if c["stats"] else c["steps"]
    if last:
        qgbe.qgbe_step(s.ctx, c["dt"], c["samples"], sampler, last, None)
    out = {}
    if c["stats"]:
        st = qgbe.Stats()
        qgbe.qgbe_step(s.ctx, c["dt"], c["samples"], sampler, 1, qgbe.C.byref(st))
        out["stats"] = np.array([st.N_total, st.E_total, st.E_total_mod, st.entropy, *st.T_ii, *st.mass2_avg])
        out["evals"] = int(st.n_evals)
    qgbe.qgbe_get_distribution(s.ctx, -1, state["out"])
    out["f"] = state["out"]
    return out


def work(case):
    """Bytes: each input read once, each output written once.  Operations: per
    sample as the method states them (geometry and Table I's matrix element,
    three trilinear reads, the bracket and three deposits), with the share of
    samples inside the box seen on these occupations."""
    c = case
    per_row = 2 * (N_IN * HIDDEN + HIDDEN * HIDDEN + HIDDEN * N_OUT)
    if c["kind"] == "forward":
        return {"bytes": c["rows"] * 4.0 * (N_IN + N_OUT), "flops": float(per_row) * c["rows"]}
    if c["kind"] == "grad":
        return {"bytes": c["rows"] * 56.0 + 4.0 * qgbe.MLP_PARAMS, "flops": 3.0 * per_row * c["rows"]}
    if c["kind"] == "train":
        return {"bytes": c["epochs"] * c["rows"] * 56.0, "flops": 3.0 * per_row * c["rows"] * c["epochs"]}
    points = len(_species(c)) * _cells(c) * _nodes(c)
    n = _n_samples(c)
    rows = len(_channels(c["mask"])) * _nodes(c)
    inside, outside, share = 388.7, 179.0, 0.46
    if c["sampler"] in ("learned", "network"):
        inside, outside, share = inside + 519.0, outside + 519.0, 0.8
    elif c["sampler"].startswith("roots"):
        inside, outside, share = 47.3 + 180.3, 47.3, 0.25
    b = 16.0 * points * c.get("steps", 1)
    if c["kind"] == "record":
        b = 8.0 * points + 56.0 * n
    elif c["sampler"] == "learned":
        b += rows * 352.0
    return {"bytes": b, "flops": n * (share * inside + (1.0 - share) * outside)}


# ---- 64-bit values of the same outputs ------------------------------------------
#
# Everything below is plain torch: the channel table of Eq. C_quark and
# Eq. C_gluon, Philox4x32-10, the sample maps, Table I, the symmetric deposits,
# the drift and the Euler update, as include/qgbe.h states them.

def _channels(mask):
    """(row, species tuple, code, symmetric weight, direct weight), by code."""
    anti = [3, 4, 5, 0, 1, 2, 6]
    reactions = [(7, G, G, G, G)]
    reactions += [(6, q, G, q, G) for q in range(6)]
    reactions += [(5, q, q + 3, G, G) for q in range(3)]
    reactions += [(4, i, i + 3, j, j + 3) for i in range(3) for j in range(i + 1, 3)]
    reactions += [(3, q, q + 3, q, q + 3) for q in range(3)]
    reactions += [(2, q, q, q, q) for q in range(6)]
    reactions += [(1, a, b, a, b) for a in range(6) for b in range(a + 1, 6) if b != anti[a]]
    out = []
    for row, *sp in reactions:
        if not all((mask >> x) & 1 for x in sp):
            continue
        same = sorted(sp[:2]) == sorted(sp[2:])
        pairs = (2.0 if sp[0] == sp[1] else 1.0) * (2.0 if sp[2] == sp[3] else 1.0)
        base = (0.5 if same else 1.0) / pairs
        for x in dict.fromkeys(sp):
            i = sp.index(x)
            order = (i, i ^ 1, (i + 2) % 4, ((i ^ 1) + 2) % 4)
            t = tuple(sp[k] for k in order)
            code = ((t[0] * 7 + t[1]) * 7 + t[2]) * 7 + t[3]
            out.append((row, t, code, base / len(set(sp)), base * sp.count(x)))
    return sorted(out, key=lambda r: r[2])


_M32 = 0xFFFFFFFF


def _philox(x0, x1, x2, x3, k0, k1):
    """Ten rounds on int64 tensors holding 32-bit words."""
    for _ in range(10):
        # 32x32 -> 64 bits from 16-bit halves of the constant (no signed overflow)
        def mul(a, const):
            lo, hi = a * (const & 0xFFFF), a * (const >> 16)
            mid = (lo >> 16) + hi
            return (mid >> 16) & _M32, ((mid << 16) | (lo & 0xFFFF)) & _M32
        ah, al = mul(x0, 0xD2511F53)
        bh, bl = mul(x2, 0xCD9E8D57)
        x0, x1, x2, x3 = bh ^ x1 ^ k0, bl, ah ^ x3 ^ k1, al
        k0, k1 = (k0 + 0x9E3779B9) & _M32, (k1 + 0xBB67AE85) & _M32
    return x0, x1, x2, x3


def _unif(v):
    return (v.double() + 0.5) * (1.0 / 8388608.0)


def _dot(a, b):
    return sum(x * y for x, y in zip(a, b))


def _msq(row, s, t, u, mu):
    a, b = t - mu, u - mu
    if row == 1:
        return 16.0 * (s * s + u * u) / a ** 2
    if row == 2:
        return 16.0 * ((s * s + u * u) / a ** 2 + (s * s + t * t) / b ** 2) - 32.0 / 3.0 * s * s / (a * b)
    if row == 3:
        return 16.0 * ((s * s + u * u) / a ** 2 + (u * u + t * t) / s ** 2) - 32.0 / 3.0 * u * u / (a * s)
    if row == 4:
        return 16.0 * (t * t + u * u) / s ** 2
    if row == 5:
        return 128.0 / 3.0 * (u / a + t / b) - 96.0 * (t * t + u * u) / s ** 2
    if row == 6:
        return -128.0 / 3.0 * (u / s + s / b) + 96.0 * (s * s + u * u) / a ** 2
    return 1152.0 * (3.0 - s * u / a ** 2 - s * t / b ** 2 - t * u / s ** 2)


class _Exact:
    def __init__(self, c):
        self.c = c
        self.np = (c["npx"], c["npy"], c["npz"])
        self.ph = c["p_half"]
        self.P = _momenta(c)
        self.dev = self.P.device
        self.g2 = 4.0 * math.pi * 0.3
        self.chans = _channels(c["mask"])

    def masses(self, f, lag):
        """Eq. mg / Eq. mq per cell [7][cells]; energies |p|, or with the lagged masses."""
        c = self.c
        p2 = (self.P ** 2).sum(1)
        m2 = torch.zeros(7, _cells(c), 1, dtype=torch.float64, device=self.dev) if lag is None else lag[:, :, None]
        E = torch.sqrt(p2[None, None, :] + m2)
        w = torch.where(E > 0, 0.5 / torch.where(E > 0, E, 1.0), 0.0)
        meas = np.prod([2.0 * self.ph / n for n in self.np]) / (8.0 * math.pi ** 3)
        I = (f * w).sum(2) * meas
        CF = 4.0 / 3.0
        out = torch.empty_like(I)
        out[G] = 2.0 * self.g2 / 8.0 * (48.0 * I[G] + 6.0 * CF * I[:6].sum(0))
        for q in range(3):
            out[q] = out[q + 3] = 2.0 * CF * self.g2 * (2.0 * I[G] + I[q] + I[q + 3])
        return out

    def stencil(self, p):
        """Base index and weights [(offset, weight)] of the 8 surrounding nodes."""
        base, ws, stride = 0, [], (self.np[1] * self.np[2], self.np[2], 1)
        for a in range(3):
            n = self.np[a]
            t = (p[a] * (n / (2.0 * self.ph)) + 0.5 * n - 0.5).clamp(0.0, n - 1.0)
            i = t.floor().clamp(max=n - 2.0)
            base = base + i.long() * stride[a]
            ws.append(t - i)
        corner = []
        for k in range(8):
            off, w = 0, 1.0
            for a in range(3):
                up = (k >> (2 - a)) & 1
                off += up * stride[a]
                w = w * (ws[a] if up else 1.0 - ws[a])
            corner.append((off, w))
        return base, corner

    def draw_mixture(self, x, y, thr, mu, sigma, mrow):
        """u [5] and 1/q of the mixture sampler from the eight words of two blocks."""
        xw = list(x) + list(y)
        T = thr[mrow]                                    # [items, K]
        k = (xw[0][:, :, None] >= T[:, None, 1:]).sum(-1)
        uni = xw[0] < T[:, None, 0]
        z = []
        for j in range(3):
            r = torch.sqrt(-2.0 * torch.log(_unif(xw[1 + 2 * j] >> 9)))
            phi = 2.0 * math.pi * _unif(xw[2 + 2 * j] >> 9)
            z += [r * torch.cos(phi), r * torch.sin(phi)]
        M, S = mu[mrow].double(), sigma[mrow].double()   # [items, K, 5]
        hi = torch.cat([T[:, 1:], torch.full_like(T[:, :1], 1 << 32)], 1)
        logpi = torch.log((hi - T).double() / 4294967296.0)
        u, yl = [], []
        for d in range(5):
            yd = torch.gather(M[:, :, d], 1, k) + torch.gather(S[:, :, d], 1, k) * z[d]
            ud = _unif(xw[1 + d] >> 9)
            yl.append(torch.where(uni, torch.log(ud / (1.0 - ud)), yd))
            u.append(torch.where(uni, ud, 1.0 / (1.0 + torch.exp(-yd))))
        dens = 0.0
        for j in range(K):
            l = logpi[:, None, j]
            for d in range(5):
                zz = (yl[d] - M[:, None, j, d]) / S[:, None, j, d]
                l = l - 0.5 * zz * zz - torch.log(S[:, None, j, d]) - 0.5 * math.log(2.0 * math.pi)
            dens = dens + torch.exp(l)
        jac = 1.0
        for d in range(5):
            e = torch.exp(-yl[d].abs())
            jac = jac * (1.0 + e) ** 2 / e
        return u, 1.0 / (T[:, None, 0].double() / 4294967296.0 + dens * jac)

    def angles(self, p1, E1, m, u):
        """CM-angle sample: momenta p2, p3, p4, invariants, |p*|/(sqrt s E2), inside."""
        m1, m2, m3, m4 = m
        ph = self.ph
        p2 = [(2.0 * u[a] - 1.0) * ph for a in range(3)]
        E2 = torch.sqrt(_dot(p2, p2) + m2)
        E = E1 + E2
        P = [a + b for a, b in zip(p1, p2)]
        s = E * E - _dot(P, P)
        r3, r4 = torch.sqrt(m3), torch.sqrt(m4)
        above = s > (r3 + r4) ** 2
        s_ = torch.where(above, s, (r3 + r4) ** 2 + 1.0)
        w = torch.sqrt(s_)
        ps = torch.sqrt((s_ - (r3 + r4) ** 2) * (s_ - (r3 - r4) ** 2)) / (2.0 * w)
        c1 = (_dot(P, p1) / (E + w) - E1) / w
        n = [a + b * c1 for a, b in zip(p1, P)]
        rn = torch.sqrt(_dot(n, n))
        n = [a / rn for a in n]
        sgn = torch.copysign(torch.ones_like(n[2]), n[2])
        a = -1.0 / (sgn + n[2])
        b = n[0] * n[1] * a
        e1 = [1.0 + sgn * n[0] * n[0] * a, sgn * b, -sgn * n[0]]
        e2 = [b, sgn + n[1] * n[1] * a, -n[1]]
        ct, st = 2.0 * u[3] - 1.0, 2.0 * torch.sqrt(u[3] * (1.0 - u[3]))
        phi = 2.0 * math.pi * u[4]
        cp, sp = st * torch.cos(phi), st * torch.sin(phi)
        k = [ps * (cp * x + sp * y + ct * z) for x, y, z in zip(e1, e2, n)]
        E3s = 0.5 * (s_ + m3 - m4) / w
        Pk = _dot(P, k)
        c3 = (Pk / (E + w) + E3s) / w
        p3 = [x + y * c3 for x, y in zip(k, P)]
        p4 = [x - y for x, y in zip(P, p3)]
        E3 = (E * E3s + Pk) / w
        E4 = E - E3
        ok = above
        for x in p3 + p4:
            ok = ok & (x.abs() <= ph)
        d3, d4 = [x - y for x, y in zip(p1, p3)], [x - y for x, y in zip(p1, p4)]
        t = (E1 - E3) ** 2 - _dot(d3, d3)
        uu = (E1 - E4) ** 2 - _dot(d4, d4)
        return p2, p3, p4, s_, t, uu, ps / (w * E2), ok

    def roots(self, p1, E1, m, u, alt):
        """The two root candidates of a sample, each (p2, p3, p4, s, t, u, 1/(E2 E3 E4 |J|), ok)."""
        _, m2, m3, m4 = m
        ph = self.ph
        q = [(2.0 * u[a] - 1.0) * ph for a in range(3)]
        kx, ky = (2.0 * u[3] - 1.0) * ph, (2.0 * u[4] - 1.0) * ph
        a3 = kx * kx + ky * ky + m3
        Eq = torch.sqrt(_dot(q, q) + (m4 if alt else m2))
        if not alt:
            Wt = E1 + Eq
            Q = [x + y for x, y in zip(p1, q)]
            C = Wt * Wt + a3 - (Q[0] - kx) ** 2 - (Q[1] - ky) ** 2 - m4 - Q[2] ** 2
            den = Wt * Wt - Q[2] ** 2
            H = C * C - 4.0 * a3 * den
            some = (H >= 0) & (den > 0)
            lin, half = C * Q[2], Wt * torch.sqrt(H.clamp(min=0.0))
        else:
            D = E1 - Eq
            Q = [x - y for x, y in zip(q, p1)]
            C = 2.0 * (kx * Q[0] + ky * Q[1]) + _dot(Q, Q) + m2 - m3 - D * D
            den = Q[2] ** 2 - D * D
            H = C * C + 4.0 * a3 * den
            some = (H >= 0) & (den != 0) & (D != 0)
            lin, half = -C * Q[2], D.abs() * torch.sqrt(H.clamp(min=0.0))
        for sign in (1.0, -1.0):
            z = torch.where(some, (lin + sign * half) / torch.where(some, 2.0 * den, 1.0), 0.0)
            E3 = torch.sqrt(a3 + z * z)
            p3 = [kx, ky, z]
            if not alt:
                ok = some & (C + 2.0 * Q[2] * z > 0) & (E3 < Wt)
                p2, p4 = q, [x - y for x, y in zip(Q, p3)]
                E2, E4 = Eq, torch.sqrt(_dot(p4, p4) + m4)
                J = (z / E3 - p4[2] / E4).abs()
                other = p4
            else:
                ok = some & ((C + 2.0 * Q[2] * z) * D < 0) & (E3 > D)
                p4, p2 = q, [x + y for x, y in zip(p3, Q)]
                E4, E2 = Eq, torch.sqrt(_dot(p2, p2) + m2)
                J = (p2[2] / E2 - z / E3).abs()
                other = p2
            for x in p3 + other:
                ok = ok & (x.abs() <= ph)
            P = [x + y for x, y in zip(p1, p2)]
            d3, d4 = [x - y for x, y in zip(p1, p3)], [x - y for x, y in zip(p1, p4)]
            s = (E1 + E2) ** 2 - _dot(P, P)
            t = (E1 - E3) ** 2 - _dot(d3, d3)
            uu = (E1 - E4) ** 2 - _dot(d4, d4)
            yield p2, p3, p4, s, t, uu, 1.0 / (E2 * E3 * E4 * J), ok

    def samples(self, f, mass2, step, N, table, each):
        """Calls each(channel index, channel, item indices, uniforms, value, inside,
        stencils) for every block of samples ([items, N] tensors)."""
        c = self.c
        nodes, cells = _nodes(c), _cells(c)
        seed = W.PHILOX_SEED
        k0, k1 = seed & _M32, ((seed >> 32) + step) & _M32
        sampler = c["sampler"]
        rooted = sampler.startswith("roots")
        Vp = (2.0 * self.ph) ** 3
        for ci, (row, sp, code, w, sigma) in enumerate(self.chans):
            block = max(1, 1_500_000 // N)
            for lo in range(0, cells * nodes, block):
                item = torch.arange(lo, min(cells * nodes, lo + block), device=self.dev)
                cell, node = item // nodes, item % nodes
                m = [mass2[x][cell][:, None] for x in sp]
                mu = mass2[G][cell][:, None]
                p1 = [self.P[node][:, a:a + 1] for a in range(3)]
                E1 = torch.sqrt(_dot(p1, p1) + m[0])
                live = E1 > 0
                E1 = torch.where(live, E1, 1.0)
                f1 = f[sp[0]][cell, node][:, None]
                smp = torch.arange(N, device=self.dev)[None, :].expand(len(item), N)
                ctr = (smp, node[:, None].expand_as(smp), cell[:, None].expand_as(smp))
                x = _philox(*ctr, torch.full_like(smp, (code << 8) | (2 if rooted else 0)), k0, k1)
                inv_q = 1.0
                if table is not None:
                    y = _philox(*ctr, torch.full_like(smp, (code << 8) | 1), k0, k1)
                    u, inv_q = self.draw_mixture(x, y, *table, ci * nodes + node)
                else:
                    u = [_unif(v >> 9) for v in x]
                    u.append(_unif(((x[0] & 0x1FF) << 14) | ((x[1] & 0x1FF) << 5) | ((x[2] & 0x1FF) >> 4)))
                weight = (w if c["symmetric"] else sigma) * self.g2 ** 2 / N
                if rooted:
                    coef = weight * Vp * (2.0 * self.ph) ** 2 / (32.0 * math.pi ** 5 * 16.0) / E1
                    forms = self.roots(p1, E1, m, u, sampler == "roots_alt")
                else:
                    coef = weight * Vp * 4.0 * math.pi / (8.0 * math.pi ** 3 * 4.0 * 16.0 * math.pi ** 2) / E1
                    forms = (self.angles(p1, E1, m, u),)
                for p2, p3, p4, s, t, uu, pref, ok in forms:
                    ok = ok & live
                    msq = _msq(row, s, t, uu, mu)
                    sts, vals = [], []
                    for x3, q in zip(sp[1:], (p2, p3, p4)):
                        base, corner = self.stencil(q)
                        base = torch.where(ok, base, 0)
                        at = cell[:, None] * nodes + base
                        ff = f[x3].reshape(-1)
                        vals.append(sum(ff[at + off] * wt for off, wt in corner))
                        sts.append((x3, at, corner))
                    f2, f3, f4 = vals
                    F = [1.0 + v if x3 == G else 1.0 - v for x3, v in zip(sp, (f1, f2, f3, f4))]
                    v = coef * msq * pref * inv_q * (f3 * f4 * F[0] * F[1] - f1 * f2 * F[2] * F[3])
                    each(ci, sp, item, u, torch.where(ok, v, 0.0), ok, sts)

    def collision(self, f, mass2, step, N, table):
        A = torch.zeros(7, f[0].numel(), dtype=torch.float64, device=self.dev)
        sym = self.c["symmetric"]

        def each(ci, sp, item, u, v, ok, sts):
            A[sp[0]].index_add_(0, item, v.sum(1))
            if not sym:
                return
            for (x3, at, corner), sign in zip(sts, (1.0, -1.0, -1.0)):
                hit = ok.reshape(-1).nonzero()[:, 0]
                where, vv = at.reshape(-1)[hit], v.reshape(-1)[hit] * sign
                for off, wt in corner:
                    A[x3].index_add_(0, where + off, vv * wt.reshape(-1)[hit])

        self.samples(f, mass2, step, N, table, each)
        return A.reshape(f.shape)

    def drift(self, f, mass2):
        """D[f]: the flux form of Eq. left handside (upwind) or the central differences."""
        c = self.c
        nx, n = (c["nx"], c["ny"], c["nz"]), self.np
        shape = (7, *nx, *n)
        F = f.reshape(shape)
        E = torch.sqrt((self.P ** 2).sum(1).reshape(1, 1, 1, 1, *n) + mass2.reshape(7, *nx, 1, 1, 1))
        P = self.P.reshape(*n, 3)
        D = torch.zeros_like(F)
        for a in range(3):
            if nx[a] == 1:
                continue
            dx, dp = 6.0 / nx[a], 2.0 * self.ph / n[a]
            nxt = lambda t, ax: torch.roll(t, -1, ax)  # noqa: E731
            prv = lambda t, ax: torch.roll(t, 1, ax)  # noqa: E731
            X, Q = 1 + a, 4 + a
            pa = P[..., a]
            if c["drift"] == "upwind":
                vel = pa / E
                face = 0.5 * (vel + nxt(vel, X))
                flux = torch.where(face > 0, face * F, face * nxt(F, X))
                D += (flux - prv(flux, X)) / dx
                force = -(nxt(E, X) - prv(E, X)) / (2.0 * dx)
                face = 0.5 * (force + nxt(force, Q))
                flux = torch.where(face > 0, face * F, face * nxt(F, Q))
                D += (flux - prv(flux, Q)) / dp
            else:
                D += (nxt(pa * F / E, X) - prv(pa * F / E, X)) / (2.0 * dx)
                dE = (nxt(E, X) - prv(E, X)) / (2.0 * dx)
                D -= (nxt(F * dE, Q) - prv(F * dE, Q)) / (2.0 * dp)
        return D.reshape(f.shape)

    def stats(self, f, mass2):
        """The statistics run() returns: N, E, E_mod, entropy, T_ii, mean masses."""
        c = self.c
        deg = torch.tensor([6.0] * 6 + [16.0], dtype=torch.float64, device=self.dev)[:, None, None]
        meas = np.prod([2.0 * self.ph / n for n in self.np]) / (8.0 * math.pi ** 3)
        meas *= np.prod([6.0 / c[k] for k in ("nx", "ny", "nz")])
        E = torch.sqrt((self.P ** 2).sum(1)[None, None, :] + mass2[:, :, None])
        fe = torch.where(E > 0, f / torch.where(E > 0, E, 1.0), 0.0)
        sgn = torch.tensor([-1.0] * 6 + [1.0], dtype=torch.float64, device=self.dev)[:, None, None]
        one = 1.0 + sgn * f
        okay = (f > 0) & (one > 0)
        g, h = torch.where(okay, f, 1.0), torch.where(okay, one, 1.0)
        ent = torch.where(okay, h * torch.log(h) * sgn - g * torch.log(g), 0.0)
        tot = lambda t: float((deg * t).sum() * meas)  # noqa: E731
        energy = tot(E * f)
        T = [tot(self.P[:, a] ** 2 * fe) for a in range(3)]
        return np.array([tot(f), energy, energy - 0.25 * tot(mass2[:, :, None] * fe), tot(ent), *T,
                         *mass2.mean(1).tolist()])


def _exact_network(c, seed):
    """Head (forward) or loss and gradient of the network in 64 bits."""
    dev = _device()
    w = torch.tensor(_weights(seed), dtype=torch.float64, device=dev, requires_grad=c["kind"] == "grad")
    o, parts = 0, []
    for shape in ((N_IN, HIDDEN), (HIDDEN,), (HIDDEN, HIDDEN), (HIDDEN,), (HIDDEN, N_OUT), (N_OUT,)):
        n = int(np.prod(shape))
        parts.append(w[o:o + n].reshape(shape))
        o += n
    rows = _rows(c["rows"], seed).double()
    silu = torch.nn.functional.silu
    Y = silu(silu(rows[:, :8] @ parts[0] + parts[1]) @ parts[2] + parts[3]) @ parts[4] + parts[5]
    if c["kind"] == "forward":
        return Y
    y, wt = rows[:, 8:13], rows[:, 13]
    mu = Y[:, K:6 * K].reshape(-1, K, 5)
    ls = Y[:, 6 * K:].reshape(-1, K, 5).clamp(-7.0, 3.0)
    z = (y[:, None, :] - mu) * torch.exp(-ls)
    lk = torch.log_softmax(Y[:, :K], 1) + (-0.5 * z * z - ls - 0.5 * math.log(2.0 * math.pi)).sum(2)
    loss = -(wt * torch.logsumexp(lk, 1)).sum() / wt.sum()
    loss.backward()
    return {"grad": w.grad, "loss": float(loss.detach())}


def exact(case, seed):
    c = case
    if c["kind"] in ("grad", "forward"):
        return _exact_network(c, seed)
    # training: the shuffled order is the library's own; the network's table: its
    # BF16 products decide where the samples lie, so 64 bits give other samples
    if c["kind"] == "train" or c["sampler"] == "network" or _n_samples(c) > EXACT_SAMPLES:
        return None
    X = _Exact(c)
    f, step = _field(c, seed), _step_index(seed)
    table = _table(c, seed) if c["sampler"] == "learned" else None
    if c["kind"] == "record":
        X.step = step
        return _exact_rows(X, f)
    if c["kind"] != "step":
        return X.collision(f, X.masses(f, None), step, c["samples"], table)
    lag = None
    deg = torch.tensor([6.0] * 6 + [16.0], dtype=torch.float64, device=f.device)[:, None, None]
    live = torch.tensor([float((c["mask"] >> s) & 1) for s in range(7)], device=f.device).double()[:, None, None]
    for k in range(c["steps"]):
        m2 = X.masses(f, lag)
        A = X.collision(f, m2, step + k, c["samples"], table)
        f = f + live * c["dt"] * (A / (deg * HBARC) - X.drift(f, m2))
        lag = m2
    out = {"f": f}
    if c["stats"]:
        out["stats"] = X.stats(f, lag)
    return out


def _exact_rows(X, f):
    """Recorded rows [x (8), logit u (5), |value|] of every work item, node
    fastest, then channel, then cell."""
    c = X.c
    N, nodes, nch = c["samples"], _nodes(c), len(X.chans)
    m2 = X.masses(f, None)
    rows = torch.empty(_cells(c), nch, nodes, N, qgbe.RECORD_WIDTH, dtype=torch.float64, device=X.dev)
    pn = math.sqrt(3.0) * X.ph

    def each(ci, sp, item, u, v, ok, sts):
        cell, node = item // nodes, item % nodes
        p = X.P[node]
        a2 = (p ** 2).sum(1)
        one = torch.ones_like(a2)
        x = [p[:, 0] / X.ph, p[:, 1] / X.ph, p[:, 2] / X.ph, torch.sqrt(a2) / pn,
             torch.sqrt(a2 + m2[sp[0]][cell]) / pn, m2[G][cell] / pn ** 2, one * (sp[0] / 3.0 - 1.0),
             one * (2.0 * ci / (nch - 1) - 1.0 if nch > 1 else 0.0)]
        out = [t[:, None].expand_as(v) for t in x] + [torch.log(t / (1.0 - t)) for t in u] + [v.abs()]
        rows[cell, ci, node] = torch.stack(out, -1)

    X.samples(f, m2, X.step, N, None, each)
    return rows.reshape(-1, qgbe.RECORD_WIDTH)
