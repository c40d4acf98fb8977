"""Timed workloads of the library, through its public entry points.

Each case is a plain dict; `prepare` makes what a program holds before the
call (states, displacement tables, plans), `run` is one pass as such a program
issues it, `work` the bytes and operations the pass cannot do without, and
`exact` the same outputs from plain FP64 torch operations.  `listed` names
the workloads; `draw` gives others of the same ranges.

Kinds:
  steps    split steps of a 1D, 2D (x, v) or 4D (x1, x2, v1, v2) advection
           problem, then the mass diagnostic, in any storage tier
           ("fp16_scaled": FP16 with per-plane scales)
  sweep    one projection sweep, forward or transposed
  adjoint  split steps forward and reverse-mode gradients of a misfit
  batch    split steps of many uneven (x, v) problems, replayed as a HIP graph
  vp       self-consistent Vlasov-Poisson steps, 1D-1V or 2D-2V
  colloc   a sweep with transverse Gauss-node collocation
"""
import math

import numpy as np
import torch

import paper_1603_07008_amd as sl
from paper_1603_07008_amd import autograd as AG
from paper_1603_07008_amd.batch import Batch

TIER_BYTES = {"fp64": 8, "fp32": 4, "bf16": 2, "fp16": 2, "fp16_scaled": 2}
TIERS = ("fp64", "fp32", "bf16", "fp16")
DT = 0.1
VMAX = 6.0


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------

def listed():
    return [
        # the paper's 1D advection study: 64 cells, about one period in steps of
        # 0.37 cells; launches and latency
        {"name": "advect1d_64", "kind": "steps", "n": "64", "k": 2, "tier": "fp64", "steps": 270,
         "sigma": 0.37, "tune": False},
        # one sweep of a small (x, v) grid (the size of the quick check): the
        # latency of a single call
        {"name": "sweep_48x40", "kind": "sweep", "n": "48x40", "k": 2, "tier": "fp32",
         "ndouble": 1, "dim": 1, "adjoint": False},
        # the 2D Vlasov configuration, 256^2, a run of its Strang steps
        {"name": "vlasov2d_256", "kind": "steps", "n": "256x256", "k": 2, "tier": "fp32",
         "steps": 10, "sigma": 0.0, "tune": False},
        # an uneven 2D grid whose rows start at odd addresses, cubic, 16-bit storage
        {"name": "vlasov2d_odd_bf16", "kind": "steps", "n": "511x389", "k": 3, "tier": "bf16",
         "steps": 4, "sigma": 0.0, "tune": False},
        # the 4D benchmark workload, one split step with the autotuner's shapes
        {"name": "vlasov4d_48", "kind": "steps", "n": "48x48x48x48", "k": 2, "tier": "fp32",
         "steps": 1, "sigma": 0.0, "tune": True},
        # the same in the BF16 tier, in the plan's initial shapes
        {"name": "vlasov4d_48_bf16", "kind": "steps", "n": "48x48x48x48", "k": 2, "tier": "bf16",
         "steps": 1, "sigma": 0.0, "tune": False},
        # the same in scaled FP16, in the plan's initial shapes
        {"name": "vlasov4d_48_scaled", "kind": "steps", "n": "48x48x48x48", "k": 2,
         "tier": "fp16_scaled", "steps": 1, "sigma": 0.0, "tune": False},
        # the differentiation workload: 512^2 FP64, 50 steps, checkpoints, gradients
        {"name": "adjoint2d_512", "kind": "adjoint", "n": "512x512", "k": 2, "tier": "fp64",
         "steps": 50, "checkpoint": 10},
        # the batched Landau workload: 512 uneven problems of degrees 1 to 3, two
        # steps as graph replays, the batch tuner's shapes
        {"name": "batch_512", "kind": "batch", "nprob": 512, "nmin": 32, "nmax": 512,
         "problems": 4, "tier": "fp32", "steps": 2, "tune": True},
        # self-consistent 1D-1V Vlasov-Poisson, a run of Strang steps
        {"name": "vp2d_512", "kind": "vp", "n": "512x512", "k": 2, "tier": "fp32", "steps": 10},
        # self-consistent 2D-2V Vlasov-Poisson on an uneven grid
        {"name": "vp4d_uneven", "kind": "vp", "n": "36x32x30x27", "k": 2, "tier": "fp32",
         "steps": 2},
        # Gauss-node collocation of the 4D grid's x1 sweep in v1
        {"name": "colloc4d_48", "kind": "colloc", "n": "48x48x48x48", "k": 2, "tier": "fp32",
         "dim": 0, "tdim": 2},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _grid4(rng, lo, hi, most):
    while True:
        n = [rng.randint(lo, hi) for _ in range(4)]
        if math.prod(n) <= most:
            return "x".join(map(str, n))


def draw(rng):
    kind = rng.choice(("steps1", "steps2", "steps4", "sweep", "adjoint", "batch", "vp2", "vp4",
                       "colloc"))
    k = rng.randint(1, 3)
    if kind == "steps1":
        return {"kind": "steps", "n": str(_log_int(rng, 16, 4096)), "k": k,
                "tier": rng.choice(TIERS), "steps": _log_int(rng, 16, 400),
                "sigma": round(rng.uniform(-3.0, 3.0), 3), "tune": False}
    if kind == "steps2":
        nx, nv = _log_int(rng, 32, 1024), _log_int(rng, 32, 1024)
        return {"kind": "steps", "n": f"{nx}x{nv}", "k": k, "tier": rng.choice(TIERS),
                "steps": rng.randint(1, 20), "sigma": 0.0, "tune": False}
    if kind == "steps4":
        k = rng.randint(1, 2)
        n = _grid4(rng, 12, 56, 48 ** 4)
        return {"kind": "steps", "n": n, "k": k, "tier": rng.choice(TIERS[1:] + ("fp16_scaled",)),
                "steps": 1, "sigma": 0.0, "tune": rng.random() < 0.3}
    if kind == "sweep":
        ndim = rng.randint(1, 3)
        n = [_log_int(rng, 16, (65536, 1024, 96)[ndim - 1]) for _ in range(ndim)]
        return {"kind": "sweep", "n": "x".join(map(str, n)), "k": k, "tier": rng.choice(TIERS),
                "ndouble": rng.choice((0, 1, 1, 2)), "dim": rng.randrange(ndim),
                "adjoint": rng.random() < 0.5}
    if kind == "adjoint":
        nx, nv = _log_int(rng, 48, 512), _log_int(rng, 48, 512)
        return {"kind": "adjoint", "n": f"{nx}x{nv}", "k": rng.randint(1, 2),
                "tier": rng.choice(("fp64", "fp32")), "steps": _log_int(rng, 4, 50),
                "checkpoint": rng.choice((0, 10))}
    if kind == "batch":
        nmax = _log_int(rng, 64, 512)
        return {"kind": "batch", "nprob": _log_int(rng, 16, 400), "nmin": 32, "nmax": nmax,
                "problems": rng.randrange(1 << 16), "tier": rng.choice(TIERS), "steps": 2,
                "tune": False}
    if kind == "vp2":
        nx, nv = _log_int(rng, 32, 1024), _log_int(rng, 32, 1024)
        return {"kind": "vp", "n": f"{nx}x{nv}", "k": k, "tier": rng.choice(TIERS),
                "steps": rng.randint(1, 20)}
    if kind == "vp4":
        return {"kind": "vp", "n": _grid4(rng, 10, 40, 36 ** 4), "k": rng.randint(1, 2),
                "tier": rng.choice(TIERS[1:]), "steps": rng.randint(1, 3)}
    if rng.random() < 0.5:
        nx, nv = _log_int(rng, 32, 1024), _log_int(rng, 32, 1024)
        dim = rng.randrange(2)
        return {"kind": "colloc", "n": f"{nx}x{nv}", "k": k, "tier": rng.choice(TIERS),
                "dim": dim, "tdim": 1 - dim}
    d = rng.randrange(4)
    return {"kind": "colloc", "n": _grid4(rng, 10, 48, 40 ** 4), "k": rng.randint(1, 2),
            "tier": rng.choice(TIERS), "dim": d, "tdim": (d + 2) % 4}


# ---------------------------------------------------------------------------
# inputs, made on the device from the seed
# ---------------------------------------------------------------------------

def _ns(case):
    return tuple(int(v) for v in case["n"].split("x"))


def _store(tier):
    return {"fp64": torch.float64, "fp32": torch.float32, "bf16": torch.bfloat16,
            "fp16": torch.float16}[tier]


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _degree(m, o, ndim):
    return sum((m // o ** e) % o for e in range(ndim))


def _coefficients(ndim, k, cells, g):
    """Coefficients with the magnitudes of smooth Vlasov data: the cell mean
    0.15 (1 + 0.1 N(0, 1)), mode (j_0, ...) 0.15 * 0.05^(sum j) N(0, 1)."""
    o = k + 1
    M = o ** ndim
    c = torch.empty((M, cells), dtype=torch.float64, device="cuda")
    for m in range(M):
        c[m].normal_(0.0, 0.15 * 0.05 ** _degree(m, o, ndim) if m else 0.015, generator=g)
    c[0] += 0.15
    return c


def _centres(n, lo, hi):
    h = (hi - lo) / n
    return lo + (torch.arange(n, dtype=torch.float64, device="cuda") + 0.5) * h, h


def _phase(seed):
    return 2 * math.pi * ((int(seed) * 0.6180339887498949) % 1.0)


def _sweeps_2d(ns, dt, xlen, seed, amp=0.02):
    """Strang step X(dt/2) V(dt) X(dt/2) of an (x, v) problem with a given E(x)."""
    x, hx = _centres(ns[0], 0.0, xlen)
    v, hv = _centres(ns[1], -VMAX, VMAX)
    sx = (v * (0.5 * dt) / hx).contiguous()
    sv = (amp * torch.sin(2 * math.pi * x / xlen + _phase(seed)) * dt / hv).contiguous()
    return [(0, 2, sx), (1, 1, sv), (0, 2, sx)]


def _sweeps_4d(ns, dt, seed, amp=0.01):
    """Split step X1 X2 (dt/2) V1 V2 (dt) X1 X2 (dt/2) with a smooth E(x1, x2)."""
    L = 4 * math.pi
    x1, h1 = _centres(ns[0], 0.0, L)
    x2, h2 = _centres(ns[1], 0.0, L)
    v1, g1 = _centres(ns[2], -VMAX, VMAX)
    v2, g2 = _centres(ns[3], -VMAX, VMAX)
    ph = _phase(seed)
    a, b = x1[None, :], x2[:, None]                    # x1 fastest
    e1 = amp * (torch.sin(0.5 * a + ph) + 0.5 * torch.sin(0.5 * a + b + 1.0))
    e2 = amp * (torch.sin(0.5 * b + 0.3) + 0.5 * torch.sin(a - 0.5 * b + ph))
    s1 = (v1 * (0.5 * dt) / h1).contiguous()
    s2 = (v2 * (0.5 * dt) / h2).contiguous()
    X1, X2 = (0, 4, s1), (1, 8, s2)
    return [X1, X2, (2, 3, (e1 * dt / g1).reshape(-1).contiguous()),
            (3, 3, (e2 * dt / g2).reshape(-1).contiguous()), X1, X2]


def _sequence(case, ns, seed):
    if len(ns) == 1:
        return [(0, 0, torch.full((1,), float(case["sigma"]), dtype=torch.float64, device="cuda"))]
    if len(ns) == 2:
        return _sweeps_2d(ns, DT, 4 * math.pi, seed)
    return _sweeps_4d(ns, DT, seed)


def _sweep_shift(case, ns, seed):
    """The displacements of a single sweep: linear across a velocity-like
    dimension for sweeps along dimension 0, a smooth field for the others."""
    d = case["dim"]
    if len(ns) == 1:
        return 0, torch.full((1,), 0.37 + 1.5 * math.sin(_phase(seed)), dtype=torch.float64,
                             device="cuda")
    e = (d + 1) % len(ns)
    u = (torch.arange(ns[e], dtype=torch.float64, device="cuda") + 0.5) / ns[e]
    if d == 0:
        s = 8.0 * (2.0 * u - 1.0) + 0.1 * math.sin(_phase(seed))
    else:
        s = 0.4 * torch.sin(2 * math.pi * u + _phase(seed))
    return 1 << e, s.contiguous()


def _vp_coefficients(ns, k, g):
    """Near-equilibrium data of a Vlasov-Poisson run: the cell mean
    (1 + 0.01 cos(x1/2) ...) M(v...) with 0.1% noise, small higher modes."""
    ndim, half = len(ns), len(ns) // 2
    cells = math.prod(ns)
    c = _coefficients(ndim, k, cells, g) * 0.01
    shape = tuple(reversed(ns))
    f = torch.ones(shape, dtype=torch.float64, device="cuda")
    for e in range(ndim):
        if e < half:
            x, _ = _centres(ns[e], 0.0, 4 * math.pi)
            w = 1.0 + 0.01 * torch.cos(0.5 * x)
        else:
            v, _ = _centres(ns[e], -VMAX, VMAX)
            w = torch.exp(-0.5 * v * v) / math.sqrt(2 * math.pi)
        f = f * w.reshape((-1,) + (1,) * e)
    env = f.reshape(-1)
    c *= env
    c[0] += env
    return c


def _split(c, k, ndim, tier, ndouble):
    """(mass, hi) of FP64 coefficients in the layout of a plan."""
    o = k + 1
    M = o ** ndim
    lo = [m for m in range(M) if _degree(m, o, ndim) < ndouble]
    hi = [m for m in range(M) if _degree(m, o, ndim) >= ndouble]
    mass = c[lo].clone() if lo else torch.empty((0, c.shape[1]), dtype=torch.float64, device="cuda")
    h = torch.empty((len(hi), c.shape[1]), dtype=_store(tier), device="cuda")
    for i, m in enumerate(hi):
        h[i] = c[m].to(_store(tier))
    return (mass.reshape(-1) if len(lo) == 1 else mass), h


def _join(mass, hi, k, ndim, ndouble):
    """The FP64 coefficients that (mass, hi) hold."""
    o = k + 1
    M = o ** ndim
    c = torch.empty((M, hi.shape[1]), dtype=torch.float64, device="cuda")
    mm = mass.reshape(-1, hi.shape[1])
    a = b = 0
    for m in range(M):
        if _degree(m, o, ndim) < ndouble:
            c[m] = mm[a]
            a += 1
        else:
            c[m] = hi[b].to(torch.float64)
            b += 1
    return c


def _batch_problems(case):
    rng = np.random.default_rng(int(case["problems"]))
    out = []
    for _ in range(case["nprob"]):
        nx, nv = (int(v) for v in rng.integers(case["nmin"], case["nmax"] + 1, size=2))
        out.append(((nx, nv), int(rng.integers(1, 4)), float(rng.uniform(0.02, 0.2)),
                    float(rng.uniform(0.3, 0.8))))
    return out


def _flat_states(probs, tier, g):
    """One state of every problem in two flat buffers, each problem's planes at
    a 512-byte boundary; returns the buffers and the per-problem views."""
    mo, ho, at_m, at_h = [], [], 0, 0
    es = 512 // TIER_BYTES[tier]
    for ns, k, _, _ in probs:
        cells = ns[0] * ns[1]
        mo.append(at_m)
        ho.append(at_h)
        at_m += -(-cells // 64) * 64
        at_h += -(-cells * ((k + 1) ** 2 - 1) // es) * es
    mass = torch.zeros(at_m, dtype=torch.float64, device="cuda")
    hi = torch.zeros(at_h, dtype=_store(tier), device="cuda")
    if g is not None:
        mass.normal_(0.15, 0.015, generator=g)
        hi.normal_(0.0, 1.0, generator=g)
    views = []
    for (ns, k, _, _), a, b in zip(probs, mo, ho):
        cells, o = ns[0] * ns[1], k + 1
        m = mass[a:a + cells]
        h = hi[b:b + cells * (o * o - 1)].view(o * o - 1, cells)
        if g is not None:
            mass[a + cells:a - (-cells // 64) * 64] = 0.0
            hi[b + h.numel():b - (-h.numel() // es) * es] = 0.0
            scale = [0.15 * 0.05 ** _degree(j, o, 2) for j in range(1, o * o)]
            h *= torch.tensor(scale, dtype=h.dtype, device="cuda")[:, None]
        views.append((m, h))
    return mass, hi, views


def _node_shift(case, ns, seed):
    t, o = case["tdim"], case["k"] + 1
    nodes = torch.from_numpy(np.polynomial.legendre.leggauss(o)[0]).cuda()
    u = (torch.arange(ns[t], dtype=torch.float64, device="cuda")[:, None] + 0.5 + 0.5 * nodes) / ns[t]
    if t >= (len(ns) + 1) // 2:                        # a velocity: linear across the domain
        s = 1.5 * (2.0 * u - 1.0) + 0.01 * math.sin(_phase(seed))
    else:
        s = 0.1 * torch.sin(2 * math.pi * u + _phase(seed))
    return s.reshape(-1).contiguous()


# ---------------------------------------------------------------------------
# prepare and run
# ---------------------------------------------------------------------------

def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        return _prepare_batch(case, seed)
    ns, k, tier = _ns(case), case["k"], case["tier"]
    ndim, cells = len(ns), math.prod(ns)
    scaled = tier == "fp16_scaled"
    tier = "fp16" if scaled else tier
    nd = case.get("ndouble", 1)
    g = _gen(seed)
    c = _vp_coefficients(ns, k, g) if kind == "vp" else _coefficients(ndim, k, cells, g)
    plan = sl.Plan(ns, k, tier, ndouble=nd)
    if scaled:
        s0 = (c[0].clone(), torch.empty((plan.n_hi, cells), dtype=torch.float16, device="cuda"),
              plan.empty_scale())
        plan.scaled_import(c[1:], s0[1], s0[2])
        torch.cuda.current_stream().synchronize()       # c is released next
        s1 = plan.empty_state() + (plan.empty_scale(),)
    else:
        s0 = _split(c, k, ndim, tier, nd)
        s1 = plan.empty_state()
    del c
    st = {"kind": kind, "plan": plan, "bufs": (s0, s1), "cur": 0, "scaled": scaled}
    if kind == "steps":
        st["seq"] = _sequence(case, ns, seed)
        st["steps"] = case["steps"]
        st["total"] = torch.zeros(2, dtype=torch.float64, device="cuda")
        if case["tune"]:
            plan.tune(st["seq"], s0[:2], s1[:2], reps=2)
    elif kind == "sweep":
        mask, shift = _sweep_shift(case, ns, seed)
        st["call"] = plan.advect_dim_adjoint if case["adjoint"] else plan.advect_dim
        st["args"] = (case["dim"], shift, mask)
    elif kind == "adjoint":
        st["seq"] = _sweeps_2d(ns, DT, 4 * math.pi, seed)
        st["steps"], st["ckpt"] = case["steps"], case["checkpoint"] or None
        st["target"] = _split(_coefficients(ndim, k, cells, g), k, ndim, tier, 1)
    elif kind == "vp":
        h = [4 * math.pi / n if e < ndim // 2 else 2 * VMAX / n for e, n in enumerate(ns)]
        seq = _sweeps_2d(ns, DT, 4 * math.pi, seed) if ndim == 2 else _sweeps_4d(ns, DT, seed)
        st["x"] = [s for _, _, s in seq[:ndim // 2]]
        st["h"], st["steps"], st["ndim"] = h, case["steps"], ndim
        st["v"] = [torch.empty(math.prod(ns[:ndim // 2]), dtype=torch.float64, device="cuda")
                   for _ in range(ndim // 2)]
    else:
        st["args"] = (case["dim"], case["tdim"], _node_shift(case, ns, seed))
    return st


def _prepare_batch(case, seed):
    probs = _batch_problems(case)
    stream = torch.cuda.Stream()
    mass, hi, s0 = _flat_states(probs, case["tier"], _gen(seed))
    mass1, hi1, s1 = _flat_states(probs, case["tier"], None)
    seqs = [_sweeps_2d(ns, dt, 2 * math.pi / kappa, seed, amp=0.01 / kappa)
            for ns, _, dt, kappa in probs]
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        b = Batch([p[0] for p in probs], [p[1] for p in probs], case["tier"],
                  stream=stream.cuda_stream)
        b.bind(s0, s1)
        b.set_sequence([(seqs[0][q][0], [(s[q][1], s[q][2]) for s in seqs]) for q in range(3)])
        if case["tune"]:
            b.tune(reps=1)
    stream.synchronize()
    return {"kind": "batch", "batch": b, "steps": case["steps"], "seqs": seqs, "stream": stream,
            "flat": ((mass, hi), (mass1, hi1))}


def run(state):
    kind = state["kind"]
    if kind == "batch":
        res = state["batch"].run(state["steps"], use_graph=True)
        return state["flat"][res]
    plan = state["plan"]
    if kind == "steps":
        a, b = state["bufs"][state["cur"]], state["bufs"][1 - state["cur"]]
        call = plan.split_steps_scaled if state["scaled"] else plan.split_steps
        if call(state["seq"], state["steps"], a, b):
            state["cur"] = 1 - state["cur"]
        out = state["bufs"][state["cur"]]
        plan.mass_device(out[0], state["total"])
        return (*out, state["total"])
    if kind == "vp":
        a, b = state["bufs"][state["cur"]], state["bufs"][1 - state["cur"]]
        if state["ndim"] == 2:
            res = plan.vlasov_poisson_steps(state["steps"], state["x"][0], *state["h"], DT, a, b,
                                            shift_v=state["v"][0])
        else:
            res = plan.vlasov_poisson_steps_2d2v(state["steps"], *state["x"], state["h"], DT, a, b,
                                                 *state["v"])
        if res:
            state["cur"] = 1 - state["cur"]
        return (*state["bufs"][state["cur"]], *state["v"])
    s0, s1 = state["bufs"]
    if kind == "sweep":
        state["call"](*state["args"], *s0, *s1)
        return s1
    if kind == "colloc":
        plan.advect_dim_collocated(*state["args"], *s0, *s1)
        return s1
    mass, hi = (t.detach().requires_grad_(True) for t in s0)
    fm, fh = AG.split_steps(plan, state["seq"], state["steps"], mass, hi,
                            checkpoint_every=state["ckpt"])
    loss = AG.weighted_l2_misfit(fm, fh, *state["target"], plan.ndim, plan.k, 1.0)
    loss.backward()
    return loss.detach(), mass.grad, hi.grad


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def _state_bytes(cells, modes, tier, n_lo=1):
    return cells * (8 * n_lo + TIER_BYTES[tier] * (modes - n_lo))


def work(case):
    """Each input state read once and each output state written once, and
    4 (k+1) - 1 operations per coefficient and sweep."""
    kind = case["kind"]
    if kind == "batch":
        b = f = 0
        for (nx, nv), k, _, _ in _batch_problems(case):
            cells, M = nx * nv, (k + 1) ** 2
            b += 2 * _state_bytes(cells, M, case["tier"]) + 8 * (nx + nv)
            f += 3 * case["steps"] * cells * M * (4 * k + 3)
        return {"bytes": b, "flops": f}
    ns, k = _ns(case), case["k"]
    ndim, cells = len(ns), math.prod(ns)
    o, M = k + 1, (k + 1) ** len(ns)
    per = cells * M * (4 * o - 1)
    n_lo = sum(1 for m in range(M) if _degree(m, o, ndim) < case.get("ndouble", 1))
    b = 2 * _state_bytes(cells, M, case["tier"], n_lo)
    if kind == "steps":
        return {"bytes": b, "flops": {1: 1, 2: 3, 4: 6}[ndim] * case["steps"] * per}
    if kind == "sweep":
        return {"bytes": b, "flops": per}
    if kind == "adjoint":                              # the state and the target in, the gradient out
        return {"bytes": 1.5 * b, "flops": 6 * case["steps"] * per}
    if kind == "vp":
        sweeps = (3 if ndim == 2 else 6) * case["steps"]
        return {"bytes": b, "flops": sweeps * per + case["steps"] * cells}
    return {"bytes": b, "flops": per + 2 * cells * M * (2 * o - 1)}


# ---------------------------------------------------------------------------
# the same outputs in FP64
# ---------------------------------------------------------------------------

def _legendre(o, x):
    p = [torch.ones_like(x), x]
    for j in range(1, o - 1):
        p.append(((2 * j + 1) * x * p[j] - j * p[j - 1]) / (j + 1))
    return torch.stack(p[:o], -1)                      # [..., o]


def _tables(sigma, k):
    """floor(sigma) and the projection matrices A, B [n, j, l] by Gauss
    quadrature (exact for the degree-2k integrands) on the two parts of a cell."""
    o = k + 1
    y, w = (torch.from_numpy(a).cuda() for a in np.polynomial.legendre.leggauss(o))
    s = torch.floor(sigma)
    al = (sigma - s)[:, None]
    scale = (2 * torch.arange(o, dtype=torch.float64, device="cuda") + 1) / 2
    xa = 2 * al - 1 + (1 - al) * (1 + y)               # the part fed by cell i - s
    A = torch.einsum("nq,nqj,nql->njl", (1 - al) * w, _legendre(o, xa), _legendre(o, xa - 2 * al))
    xb = -1 + al * (1 + y)                             # the part fed by cell i - s - 1
    B = torch.einsum("nq,nqj,nql->njl", al * w, _legendre(o, xb), _legendre(o, xb + 2 - 2 * al))
    return s.to(torch.int64), A * scale[:, None], B * scale[:, None]


def _shifted(c, ns, d, rows):
    """c [..., cells] with cell index i_d of every line replaced by rows: an
    index tensor over the reversed grid shape (broadcast)."""
    shape = tuple(reversed(ns))
    v = c.reshape(c.shape[:-1] + shape)
    ax = v.dim() - 1 - d
    idx = rows.expand(shape).reshape((1,) * (v.dim() - len(shape)) + shape).expand(v.shape)
    return torch.gather(v, ax, idx).reshape(c.shape)


def _line_view(t, ns, mask):
    """A per-line vector as a broadcast over the reversed grid shape."""
    return t.reshape(tuple(ns[e] if mask >> e & 1 else 1 for e in reversed(range(len(ns)))))


def _sweep64(c, ns, k, d, mask, sigma, adjoint=False):
    """One sweep of the coefficients c [modes, cells] in FP64."""
    ndim, o = len(ns), k + 1
    s, A, B = _tables(sigma, k)
    if adjoint:
        s, A, B = -s - 1, B.transpose(1, 2), A.transpose(1, 2)
    shape = (1,) * (ndim - 1 - d) + (-1,) + (1,) * d
    i = torch.arange(ns[d], device="cuda").reshape(shape)
    sv = _line_view(s, ns, mask)
    ra, rb = torch.remainder(i - sv, ns[d]), torch.remainder(i - sv - 1, ns[d])
    full = tuple(reversed(ns))
    per = lambda t: _line_view(t, ns, mask).expand(full).reshape(-1)
    low, M = o ** d, o ** ndim
    cv = c.reshape(M // (low * o), o, low, -1)
    out = torch.zeros_like(cv)
    for l in range(o):
        x, y = _shifted(cv[:, l], ns, d, ra), _shifted(cv[:, l], ns, d, rb)
        for j in range(o):
            out[:, j].addcmul_(x, per(A[:, j, l])).addcmul_(y, per(B[:, j, l]))
    return out.reshape(c.shape)


def _field64(c, ns, k, hx, hv, dt):
    """Displacements E(x_i) dt / hv of an (x, v) state."""
    o, nx = k + 1, ns[0]
    r = hv * c[:o].reshape(o, ns[1], nx).sum(1)        # density moments
    rho = r[0] - r[0].mean()
    face = torch.cat([torch.zeros(1, dtype=torch.float64, device="cuda"),
                      torch.cumsum(hx * rho, 0)])[:nx]
    mean = (face + 0.5 * hx * rho - hx / 6 * r[1]).mean()
    half = [1.0, -0.5, 0.0, 0.125]                     # int_{-1}^{0} P_j
    e = face - mean + 0.5 * hx * (rho * half[0] + sum(r[j] * half[j] for j in range(1, o)))
    return e * dt / hv


def _field64_2d(c0, ns, h, dt):
    n1, n2 = ns[:2]
    rho = h[2] * h[3] * c0.reshape(ns[3] * ns[2], n2, n1).sum(0)
    hat = torch.fft.fft2(rho)

    def axis(n, hh):
        m = torch.fft.fftfreq(n, 1.0 / n, dtype=torch.float64, device="cuda").round()
        keep = torch.ones(n, dtype=torch.float64, device="cuda")
        if n % 2 == 0:
            keep[n // 2] = 0.0
        return 2 * math.pi * m / (n * hh), torch.sinc(m / n), keep
    q1, c1, k1 = axis(n1, h[0])
    q2, c2, k2 = axis(n2, h[1])
    q1, q2 = q1[None, :], q2[:, None]
    kk = q1 * q1 + q2 * q2
    keep = k1[None, :] * k2[:, None] * (kk > 0)
    hat = hat / (c1[None, :] * c2[:, None]) * keep / torch.where(kk > 0, kk, torch.ones_like(kk))
    e1 = torch.fft.ifft2(-1j * q1 * hat).real
    e2 = torch.fft.ifft2(-1j * q2 * hat).real
    return (e1 * dt / h[2]).reshape(-1).contiguous(), (e2 * dt / h[3]).reshape(-1).contiguous()


def _colloc64(c, ns, k, d, t, node_shift):
    ndim, o = len(ns), k + 1
    y, w = (torch.from_numpy(a).cuda() for a in np.polynomial.legendre.leggauss(o))
    P = _legendre(o, y)                                # [node, j]
    low = o ** t
    cv = c.reshape(-1, o, low, c.shape[1])
    out = torch.zeros_like(cv)
    ns_q = node_shift.reshape(ns[t], o)
    # a node line carries the modes of every dimension but t
    for q in range(o):
        u = sum(cv[:, j] * P[q, j] for j in range(o))  # [high, low, cells]
        full = torch.zeros_like(cv)
        full[:, 0] = u
        swept = _sweep64(full.reshape(c.shape), ns, k, d, 1 << t, ns_q[:, q].contiguous())
        swept = swept.reshape(cv.shape)[:, 0]
        for j in range(o):
            out[:, j] += (2 * j + 1) / 2 * w[q] * P[q, j] * swept
    return out.reshape(c.shape)


def _weights(o, ndim):
    w = torch.ones(o ** ndim, dtype=torch.float64, device="cuda")
    for m in range(o ** ndim):
        for e in range(ndim):
            w[m] /= 2 * ((m // o ** e) % o) + 1
    return w


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        probs = _batch_problems(case)
        mass, hi, views = _flat_states(probs, case["tier"], _gen(seed))
        hi = hi.to(torch.float64)
        at = 0
        es = 512 // TIER_BYTES[case["tier"]]
        for (ns, k, dt, kappa), (m, h) in zip(probs, views):
            c = _join(m, h, k, 2, 1)
            seq = _sweeps_2d(ns, dt, 2 * math.pi / kappa, seed, amp=0.01 / kappa)
            for _ in range(case["steps"]):
                for d, mask, s in seq:
                    c = _sweep64(c, ns, k, d, mask, s)
            m.copy_(c[0])
            n = c[1:].numel()
            hi[at:at + n] = c[1:].reshape(-1)
            at += -(-n // es) * es
        return mass, hi
    ns, k, tier = _ns(case), case["k"], case["tier"]
    ndim, cells, o = len(ns), math.prod(ns), k + 1
    nd = case.get("ndouble", 1)
    g = _gen(seed)
    c = _vp_coefficients(ns, k, g) if kind == "vp" else _coefficients(ndim, k, cells, g)
    if tier == "fp16_scaled":
        # the stored planes carry exponents of their own: only the FP64 cell
        # means and their sum have a value here, from inputs rounded as a plane
        # with its absmax in [2^6, 2^7) is
        for m in range(1, o ** ndim):
            e = 6.0 - math.floor(math.log2(float(c[m].abs().max().float())))
            c[m] = (c[m] * 2.0 ** e).to(torch.float16).to(torch.float64) * 2.0 ** -e
        for _ in range(case["steps"]):
            for d, mask, s in _sequence(case, ns, seed):
                c = _sweep64(c, ns, k, d, mask, s)
        total = math.fsum(c[0].tolist())
        return c[0], None, None, torch.tensor([total, 0.0], dtype=torch.float64)
    c = _join(*_split(c, k, ndim, tier, nd), k, ndim, nd)

    def state(c):
        lo = [m for m in range(o ** ndim) if _degree(m, o, ndim) < nd]
        hi = [m for m in range(o ** ndim) if _degree(m, o, ndim) >= nd]
        mass = c[lo]
        return (mass.reshape(-1) if len(lo) == 1 else mass), c[hi]

    if kind == "sweep":
        mask, shift = _sweep_shift(case, ns, seed)
        return state(_sweep64(c, ns, k, case["dim"], mask, shift, case["adjoint"]))
    if kind == "colloc":
        return state(_colloc64(c, ns, k, case["dim"], case["tdim"], _node_shift(case, ns, seed)))
    if kind == "steps":
        for _ in range(case["steps"]):
            for d, mask, s in _sequence(case, ns, seed):
                c = _sweep64(c, ns, k, d, mask, s)
        total = math.fsum(c[0].tolist())
        return (*state(c), torch.tensor([total, 0.0], dtype=torch.float64))
    if kind == "vp":
        h = [4 * math.pi / n if e < ndim // 2 else 2 * VMAX / n for e, n in enumerate(ns)]
        seq = _sweeps_2d(ns, DT, 4 * math.pi, seed) if ndim == 2 else _sweeps_4d(ns, DT, seed)
        xs = seq[:ndim // 2]
        for _ in range(case["steps"]):
            for d, mask, s in xs:
                c = _sweep64(c, ns, k, d, mask, s)
            if ndim == 2:
                v = (_field64(c, ns, k, h[0], h[1], DT),)
                c = _sweep64(c, ns, k, 1, 1, v[0])
            else:
                v = _field64_2d(c[0], ns, h, DT)
                c = _sweep64(c, ns, k, 2, 3, v[0])
                c = _sweep64(c, ns, k, 3, 3, v[1])
            for d, mask, s in xs:
                c = _sweep64(c, ns, k, d, mask, s)
        return (*state(c), *v)
    seq = _sweeps_2d(ns, DT, 4 * math.pi, seed)
    t = _join(*_split(_coefficients(ndim, k, cells, g), k, ndim, tier, 1), k, ndim, 1)
    for _ in range(case["steps"]):
        for d, mask, s in seq:
            c = _sweep64(c, ns, k, d, mask, s)
    w = _weights(o, ndim)[:, None]
    loss = 0.5 * (w * (c - t) ** 2).sum()
    gr = w * (c - t)
    for _ in range(case["steps"]):
        for d, mask, s in reversed(seq):
            gr = _sweep64(gr, ns, k, d, mask, s, adjoint=True)
    return loss, gr[0], gr[1:]
