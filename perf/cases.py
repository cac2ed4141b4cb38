"""The work that programs have this framework do, as measurable cases.

Every case is a dict of plain values naming one *kind* of use and its sizes:

  grid     solve a pairwise grid on fresh evidence (restoration, labelling):
           evidence in, messages reset, the iterations, beliefs and MAP out;
           with "tol" the solve stops once the messages settle
  rbm      the same on a dense bipartite layer of binary units
  deconv   the same on a graph of OR / AND factors (blind deconvolution)
  triplet  the same on a grid of dense three-way factors
  batch    many grids of mixed sizes and state counts advanced together
  grad     one training step: beliefs and the gradient of a loss on them
  sampler  perturb-and-MAP samples of one deconvolution graph
  serve    a burst of mixed requests through the continuous-batching server

``prepare`` builds what a program keeps (graph, batch, sampler, server) and its
inputs from the seed alone; ``run`` is one pass through the public entry
points; ``exact`` is the same pass in 64-bit torch.
"""
from __future__ import annotations

import math
import os
import tempfile

import numpy as np
import torch

from paper_2202_04110_amd import lbp, learn, tune
from paper_2202_04110_amd import workloads as W
from paper_2202_04110_amd.autograd import lbp_beliefs

DAMPING = 0.5


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # the smallest solve in use: a 32 x 32 binary image, max-product; all
        # launch latency
        {"name": "ising32_map", "kind": "grid", "L": 32, "n": 2, "T": 0.0, "iters": 100},
        # the paper's timing protocol: a 200-unit binary RBM, 200 iterations
        # (at T = 0 one seed in four keeps moving; T = 0.05 settles on all)
        {"name": "rbm100x100_cold", "kind": "rbm", "nv": 100, "nh": 100, "T": 0.05, "iters": 200},
        # an ordinary labelling problem solved until it has settled
        {"name": "potts128x5_until", "kind": "grid", "L": 128, "n": 5, "T": 1.0, "iters": 200, "tol": 1e-3,
         "check": 10},
        # the headline workload: a 512 x 512 image with five labels; its
        # working set fits the last-level cache
        {"name": "potts512x5", "kind": "grid", "L": 512, "n": 5, "T": 1.0, "iters": 200},
        # the largest solve: streams from HBM on every iteration
        {"name": "potts2048x5", "kind": "grid", "L": 2048, "n": 5, "T": 1.0, "iters": 200},
        # marginals of a dense layer: every variable has hundreds of edges
        # (at low temperatures this graph does not settle: 32 and 64 bits part)
        {"name": "rbm784x500", "kind": "rbm", "nv": 784, "nh": 500, "T": 1.0, "iters": 200},
        # the paper's logical-factor example at its size
        {"name": "deconv32_map", "kind": "deconv", "K": 5, "tw": 6, "img": 32, "T": 0.0, "iters": 200},
        # higher-order factors
        {"name": "triplet256x3", "kind": "triplet", "L": 256, "n": 3, "T": 1.0, "iters": 100},
        # many uneven graphs at once (16..256 a side, 2..8 labels)
        {"name": "batch64_mixed", "kind": "batch", "count": 64, "lo": 16, "hi": 256, "T": 1.0, "iters": 50},
        # one step of end-to-end training: forward, loss, reverse sweep
        {"name": "grad64x6", "kind": "grad", "L": 64, "n": 6, "T": 1.0, "iters": 50, "ckpt": 10},
        # 16 posterior samples of the deconvolution latents
        {"name": "samples16_deconv", "kind": "sampler", "S": 16, "K": 5, "tw": 6, "img": 32, "T": 0.0, "iters": 200},
        # a burst of requests on the server, one in ten with a gradient
        {"name": "serve28_mixed", "kind": "serve", "count": 28, "lo": 16, "hi": 192, "T": 1.0, "iters": 50},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["grid", "grid", "grid", "rbm", "rbm", "deconv", "triplet", "batch", "grad", "sampler", "serve"])
    T = rng.choice([0.0, 1.0])
    if kind == "grid":
        n = rng.randint(2, 8)
        L = _log(rng, 8, int(2048 * 5 / max(n, 5)))
        c = {"kind": kind, "L": L, "n": n, "T": T, "iters": _log(rng, 20, 200)}
        if T > 0 and L <= 512 and rng.random() < 0.25:
            c.update(tol=1e-3, check=rng.choice([5, 10, 20]))
        return c
    if kind == "rbm":
        c = {"kind": kind, "nv": _log(rng, 15, 800), "nh": _log(rng, 15, 520), "iters": _log(rng, 50, 200)}
        # max-product and low temperatures where the graph is small enough to settle
        return dict(c, T=rng.choice([0.0, 0.05, 1.0]) if c["nv"] * c["nh"] <= 20000 else 1.0)
    if kind in ("deconv", "sampler"):
        c = {"kind": kind, "K": rng.randint(1, 5), "tw": rng.randint(3, 6), "img": _log(rng, 10, 32), "T": 0.0}
        if kind == "sampler":
            c.update(S=rng.randint(2, 16), iters=_log(rng, 50, 200))
        else:
            c.update(iters=_log(rng, 50, 300))
        return c
    if kind == "triplet":
        return {"kind": kind, "L": _log(rng, 8, 256), "n": rng.randint(2, 4), "T": T, "iters": _log(rng, 20, 100)}
    if kind == "batch":
        return {"kind": kind, "count": _log(rng, 4, 64), "lo": 16, "hi": _log(rng, 32, 256), "T": T, "iters": 50}
    if kind == "grad":
        return {"kind": kind, "L": _log(rng, 8, 160), "n": rng.randint(2, 8), "T": 1.0, "iters": _log(rng, 10, 60),
                "ckpt": rng.choice([5, 10, 20])}
    return {"kind": "serve", "count": _log(rng, 6, 28), "lo": 16, "hi": _log(rng, 32, 192), "T": T, "iters": 50}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _grid(L, n, seed):
    """L x L 4-neighbour grid, n labels: evidence N(0, 1); per-factor table
    1.0 on the diagonal, N(0, 0.2) elsewhere; two labels: an Ising coupling
    J ~ N(0, 0.5) with table [[J, -J], [-J, J]]."""
    rng = np.random.default_rng([seed, L, n])
    ev = rng.standard_normal(L * L * n, dtype=np.float32)
    pairs = W.grid_pairs(L)
    F = pairs.shape[0]
    if n == 2:
        J = 0.5 * rng.standard_normal(F, dtype=np.float32)
        tab = np.stack([J, -J, -J, J], 1)
    else:
        tab = rng.standard_normal((F, n * n), dtype=np.float32)
        tab *= 0.2
        tab[:, np.arange(n) * (n + 1)] = 1.0
    return W.GraphSpec(
        var_num_states=np.full(L * L, n, np.int32), evidence=ev, factor_kind=np.zeros(F, np.int32),
        factor_edge_off=np.arange(F + 1, dtype=np.int64) * 2, edge_var=pairs.reshape(-1).astype(np.int32),
        factor_cfg_table=np.zeros(F, np.int32), cfg_table_num_cfgs=np.zeros(1, np.int32),
        cfg_table_arity=np.full(1, 2, np.int32), cfg_table_off=np.zeros(2, np.int64),
        cfg_table_states=np.zeros(0, np.int32), logpot_off=np.arange(F + 1, dtype=np.int64) * (n * n),
        log_potentials=tab.reshape(-1), name="grid")


def _spec(case, seed):
    k = case["kind"]
    if k in ("grid", "grad"):
        return _grid(case["L"], case["n"], seed)
    if k == "rbm":
        return W.rbm(case["nv"], case["nh"], seed=seed)
    if k in ("deconv", "sampler"):
        return W.deconv(seed=seed, K=case["K"], tw=case["tw"], sd=case["img"] - case["tw"] + 3,
                        img=case["img"])
    return W.triplet_grid(case["L"], case["n"], seed=seed)


def _mix(case, seed):
    """The graphs of a batch or burst: sides log-uniform in [lo, hi], 2..8
    labels."""
    # the mix of sizes belongs to the case; the seed draws the numbers
    rng = np.random.default_rng([11, case["count"], case["lo"], case["hi"]])
    sides = np.rint(np.exp(rng.uniform(math.log(case["lo"]), math.log(case["hi"]), case["count"]))).astype(int)
    labels = rng.integers(2, 9, case["count"])
    return [_grid(int(L), int(n), seed * 1000 + i) for i, (L, n) in enumerate(zip(sides, labels))]


def _burst_losses(case, specs, seed):
    """Every tenth request carries the gradient of sum(c * q), c ~ N(0, 1)
    (sum-product only: a max has no gradient)."""
    if case["T"] == 0.0:
        return [None] * len(specs)
    return [np.random.default_rng([seed, i]).standard_normal(s.num_var_states, dtype=np.float32)
            if i % 10 == 5 else None for i, s in enumerate(specs)]


def _target(case, spec, seed):
    rng = np.random.default_rng([seed, 77])
    z = torch.from_numpy(rng.standard_normal((spec.num_vars, case["n"]), dtype=np.float32))
    return torch.softmax(z, 1).reshape(-1)


def _noise(case, VS, seed):
    rng = np.random.default_rng([seed, 78])
    return torch.from_numpy(rng.gumbel(size=(case["S"], VS)).astype(np.float32))


# ---------------------------------------------------------------------------
# preparing and running
# ---------------------------------------------------------------------------
_context = None


def _ctx():
    global _context
    if _context is None:
        _context = lbp.Context(0)
    return _context


def _tuned(spec, case):
    """The graph with its launch shapes: from the shipped table where that
    covers its size, from the autotuner elsewhere (kept for this process)."""
    g = lbp.Graph(_ctx(), spec)
    cache = os.path.join(tempfile.gettempdir(), "lbp_shapes_%d.json" % os.getpid())
    tune.apply_or_tune(g, DAMPING, case["T"], path=cache)
    return g


def _out(g):
    return (torch.empty(g.VS, device="cuda", dtype=torch.float32), torch.empty(g.V, device="cuda", dtype=torch.int32))


def prepare(case, seed):
    k = case["kind"]
    st = {"case": case}
    if k == "batch":
        st["graphs"] = [lbp.Graph(_ctx(), s) for s in _mix(case, seed)]
        st["batch"] = lbp.Batch(_ctx(), st["graphs"])
        # one buffer each for all beliefs and all MAPs, a slice per graph
        st["q"] = torch.empty(sum(g.VS for g in st["graphs"]), device="cuda", dtype=torch.float32)
        st["map"] = torch.empty(sum(g.V for g in st["graphs"]), device="cuda", dtype=torch.int32)
        st["outs"] = list(zip(st["q"].split([g.VS for g in st["graphs"]]),
                              st["map"].split([g.V for g in st["graphs"]])))
    elif k == "serve":
        st["specs"] = _mix(case, seed)
        st["losses"] = _burst_losses(case, st["specs"], seed)
        st["server"] = lbp.Server(_ctx(), budget_bytes=512 << 20, max_slots=64, steps_per_round=10)
    elif k == "grad":
        spec = _spec(case, seed)
        st["graph"] = _tuned(spec, case)
        st["phi"] = torch.from_numpy(spec.log_potentials).cuda().requires_grad_(True)
        st["theta"] = torch.from_numpy(spec.evidence).cuda().requires_grad_(True)
        st["target"] = _target(case, spec, seed).cuda()
    elif k == "sampler":
        g = st["graph"] = _tuned(_spec(case, seed), case)
        st["sampler"] = lbp.Sampler(g, case["S"])
        st["noise"] = _noise(case, g.VS, seed).cuda()
        st["map"] = torch.empty((case["S"], g.V), device="cuda", dtype=torch.int32)
        st["q"] = torch.empty((case["S"], g.VS), device="cuda", dtype=torch.float32)
    else:
        spec = _spec(case, seed)
        g = st["graph"] = _tuned(spec, case)
        st["evidence"] = torch.from_numpy(spec.evidence).cuda()
        st["q"], st["map"] = _out(g)
    return st


def run(st):
    case = st["case"]
    k, T, iters = case["kind"], case["T"], case["iters"]
    if k == "batch":
        for g in st["graphs"]:
            g.reset_messages()
        st["batch"].run_bp(iters, DAMPING, T)
        for g, (q, m) in zip(st["graphs"], st["outs"]):
            g.get_beliefs(out=q)
            g.decode_map(out=m)
        return st["q"], st["map"]
    if k == "serve":
        srv = st["server"]
        for i, (s, c) in enumerate(zip(st["specs"], st["losses"])):
            srv.submit(s, iters, DAMPING, T, grad_q=c, ckpt_every=10, req_id=i)
        srv.drain()
        done = {}
        while len(done) < len(st["specs"]):
            for rec in srv.poll():
                done[rec["req_id"]] = rec
        out = []
        for i, c in enumerate(st["losses"]):
            rec = done[i]
            out.append((rec["beliefs"], rec["map"]) + (() if c is None else (rec["grad_logpot"],)))
        return out
    if k == "grad":
        q = lbp_beliefs(st["graph"], st["phi"], st["theta"], iters, DAMPING, T, case["ckpt"])
        loss = learn.cross_entropy(q, st["target"], st["graph"].V)
        gphi, gtheta = torch.autograd.grad(loss, (st["phi"], st["theta"]))
        return q.detach(), gphi, gtheta
    if k == "sampler":
        st["sampler"].run(iters, DAMPING, T, st["noise"], st["map"], st["q"])
        return st["q"], st["map"]
    g = st["graph"]
    g.set_evidence(st["evidence"])
    g.reset_messages()
    if "tol" in case:
        done, residual = g.run_bp_until(iters, DAMPING, T, case["tol"], case["check"])
        g.get_beliefs(out=st["q"])
        g.decode_map(out=st["map"])
        return st["q"], st["map"], done, residual
    g.run_bp(iters, DAMPING, T)
    g.get_beliefs(out=st["q"])
    g.decode_map(out=st["map"])
    return st["q"], st["map"]


# ---------------------------------------------------------------------------
# bytes and operations
# ---------------------------------------------------------------------------
def _pair_flops(F, n, T):
    # both directions: add and max per table entry (and exp, add), then
    # subtract, damp (3) and normalise per state
    return 2.0 * F * (n * n * (2 if T == 0 else 4) + 5 * n)


def _grid_work(L, n, T, iters):
    F, V = 2 * L * (L - 1), L * L
    return 4.0 * (F * n * n + 2 * V * n + V), iters * _pair_flops(F, n, T)


def work(case):
    k, T, iters = case["kind"], case["T"], case["iters"]
    if k in ("batch", "serve"):
        rng = np.random.default_rng([11, case["count"], case["lo"], case["hi"]])
        sides = np.rint(np.exp(rng.uniform(math.log(case["lo"]), math.log(case["hi"]), case["count"]))).astype(int)
        labels = rng.integers(2, 9, case["count"])
        b = f = 0.0
        for i, (L, n) in enumerate(zip(sides, labels)):
            gb, gf = _grid_work(int(L), int(n), T, iters)
            back = k == "serve" and T > 0 and i % 10 == 5
            b += gb + (4.0 * 2 * L * (L - 1) * n * n if back else 0)
            f += gf * (3 if back else 1)
        return {"bytes": float(b), "flops": float(f)}
    if k == "grid":
        b, f = _grid_work(case["L"], case["n"], T, iters)
    elif k == "grad":
        b, f = _grid_work(case["L"], case["n"], T, iters)
        b, f = 2 * b, 3 * f
    elif k == "rbm":
        F, V = case["nv"] * case["nh"], case["nv"] + case["nh"]
        b, f = 4.0 * (4 * F + 4 * V + V), iters * _pair_flops(F, 2, T)
    elif k == "triplet":
        L, n = case["L"], case["n"]
        F, V = 2 * L * max(L - 2, 0), L * L
        b = 4.0 * (F * n ** 3 + 2 * V * n + V)
        f = iters * 3.0 * F * (n ** 3 * (3 if T == 0 else 5) + 6 * n)
    else:
        S = case.get("S", 1)
        sd, tw = case["img"] - case["tw"] + 3, case["tw"]
        nSW = case["K"] * sd * sd * tw * tw
        V = case["K"] * (tw * tw + sd * sd) + nSW + case["img"] ** 2
        b = 4.0 * S * (2 * V + 2 * V + V)
        f = S * iters * (nSW * 4) * 12.0
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------
# A max-product solve of a graph with frustrated loops need not settle; its
# messages then magnify any rounding, and after a hundred iterations no value
# is the exact one.  Where the last 64-bit iteration still moves a message by
# more than this, exact() gives None.
SETTLED = 1e-2


def _lse(x, dim, T):
    return x.amax(dim) if T == 0 else T * torch.logsumexp(x / T, dim)


def _norm(B, T):
    return (B - _lse(B, 1, T)[:, None]).reshape(-1), _argmax(B)


def _argmax(B):
    # the lowest state among the largest
    top = B == B.amax(1, keepdim=True)
    return (top.to(torch.int32) * torch.arange(B.shape[1], 0, -1, device=B.device, dtype=torch.int32)).argmax(1).int()


def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _pair_arrays(spec):
    d = _device()
    n = int(spec.var_num_states[0])
    a, b = (torch.from_numpy(spec.edge_var[i::2].astype(np.int64)).to(d) for i in (0, 1))
    th = torch.from_numpy(spec.evidence).to(d).double().view(-1, n)
    phi = torch.from_numpy(spec.log_potentials).to(d).double().view(-1, n, n)
    return a, b, th, phi


def _pair_beliefs(th, a, b, m0, m1):
    return th.index_add(0, a, m0).index_add(0, b, m1)


def _pair_step(th, phi, a, b, m0, m1, T):
    B = _pair_beliefs(th, a, b, m0, m1)
    u0 = _lse(phi + (B[b] - m1)[:, None, :], 2, T)
    u1 = _lse(phi + (B[a] - m0)[:, :, None], 1, T)
    m0 = DAMPING * m0 + (1 - DAMPING) * u0
    m1 = DAMPING * m1 + (1 - DAMPING) * u1
    return m0 - m0.amax(1, keepdim=True), m1 - m1.amax(1, keepdim=True)


def _pair_exact(spec, T, iters, tol=None, check=1, settle=False):
    a, b, th, phi = _pair_arrays(spec)
    m0 = torch.zeros(phi.shape[0], phi.shape[1], device=th.device, dtype=torch.float64)
    m1 = m0.clone()
    done, res = 0, 0.0
    for it in range(iters):
        p0, p1 = m0, m1
        m0, m1 = _pair_step(th, phi, a, b, m0, m1, T)
        done += 1
        if tol is not None and (done % check == 0 or done == iters):
            res = max(float((m0 - p0).abs().max()), float((m1 - p1).abs().max()))
            if res < tol:
                break
    if settle and max(float((m0 - p0).abs().max()), float((m1 - p1).abs().max())) > SETTLED:
        return None
    q, mp = _norm(_pair_beliefs(th, a, b, m0, m1), T)
    return (q, mp) if tol is None else (q, mp, done, res)


def _pair_grad(spec, T, iters, loss):
    a, b, th, phi = _pair_arrays(spec)
    th.requires_grad_(True)
    phi.requires_grad_(True)
    m0 = torch.zeros(phi.shape[0], phi.shape[1], device=th.device, dtype=torch.float64)
    m1 = m0.clone()
    for _ in range(iters):
        m0, m1 = _pair_step(th, phi, a, b, m0, m1, T)
    B = _pair_beliefs(th, a, b, m0, m1)
    q = (B - _lse(B, 1, T)[:, None]).reshape(-1)
    gphi, gth = torch.autograd.grad(loss(q), (phi, th))
    return q.detach(), _argmax(B.detach()), gphi.reshape(-1), gth.reshape(-1)


def _triplet_exact(spec, T, iters):
    d = _device()
    n = int(spec.var_num_states[0])
    v = [torch.from_numpy(spec.edge_var[i::3].astype(np.int64)).to(d) for i in range(3)]
    th = torch.from_numpy(spec.evidence).to(d).double().view(-1, n)
    phi = torch.from_numpy(spec.log_potentials).to(d).double().view(-1, n, n, n)
    m = [torch.zeros(phi.shape[0], n, device=d, dtype=torch.float64) for _ in range(3)]

    def beliefs():
        B = th
        for j in range(3):
            B = B.index_add(0, v[j], m[j])
        return B

    for _ in range(iters):
        B = beliefs()
        x = [B[v[j]] - m[j] for j in range(3)]
        s = phi + x[0][:, :, None, None] + x[1][:, None, :, None] + x[2][:, None, None, :]
        for j in range(3):
            u = _lse(s.movedim(1 + j, 1).reshape(s.shape[0], n, n * n), 2, T) - x[j]
            w = DAMPING * m[j] + (1 - DAMPING) * u
            m[j] = w - w.amax(1, keepdim=True)
    return _norm(beliefs(), T)


def _deconv_exact(spec, iters, noise=None):
    """Max-product on AND factors (S, W, product) and OR factors (products,
    pixel); a message is its difference d = m[1] - m[0], larger state at 0."""
    d = _device()
    kind = spec.factor_kind
    nA = int((kind == W.AND).sum())
    ev = torch.from_numpy(spec.edge_var.astype(np.int64)).to(d)
    off = spec.factor_edge_off
    av = ev[: 3 * nA].view(nA, 3)
    k = np.diff(off[nA:])
    width = int(k.max())
    col = torch.arange(width, device=d)[None, :]
    kt = torch.from_numpy(k).to(d)[:, None]
    start = torch.from_numpy(off[nA:-1]).to(d)[:, None]
    valid = col < kt
    child = col == kt - 1
    parent = col < kt - 1
    ov = ev[torch.where(valid, start + col, start)]
    th = torch.from_numpy(spec.evidence).to(d).double()
    if noise is not None:
        th = th + noise.to(d).double()
    th = th.view(-1, 2)
    ma = torch.zeros(nA, 3, 2, device=d, dtype=torch.float64)
    mo = torch.zeros(len(k), width, 2, device=d, dtype=torch.float64)
    inf = float("inf")

    def beliefs():
        B = th.index_add(0, av.reshape(-1), ma.reshape(-1, 2))
        return B.index_add(0, ov[valid], mo[valid])

    def logical(dl, par, ch):
        """u[0], u[1] of an OR factor from the incoming differences."""
        r = torch.where(par, dl.clamp(min=0), 0.0)
        S = r.sum(1, keepdim=True)
        loo = S - r
        x = torch.where(par, dl, -inf)
        top = x.topk(2, 1) if x.shape[1] > 1 else None
        if top is None:
            M1, M2, am = x[:, :1], torch.full_like(x[:, :1], -inf), torch.zeros_like(x[:, :1], dtype=torch.int64)
        else:
            M1, M2, am = top.values[:, :1], top.values[:, 1:2], top.indices[:, :1]
        Mx = torch.where(torch.arange(x.shape[1], device=d)[None, :] == am, M2, M1)
        dc = torch.where(ch, dl, 0.0).sum(1, keepdim=True)
        u1 = torch.where(ch, S + M1.clamp(max=0), dc + loo)
        u0 = torch.where(ch, 0.0, (dc + loo + Mx.clamp(max=0)).clamp(min=0))
        return u0, u1

    def damp(m, u):
        w = DAMPING * m + (1 - DAMPING) * u
        return w - w.amax(2, keepdim=True)

    apar = torch.tensor([[True, True, False]], device=d).expand(nA, 3)
    for _ in range(iters):
        pa, po = ma, mo
        B = beliefs()
        na, no = B[av] - ma, B[ov] - mo
        u0, u1 = logical(na[..., 0] - na[..., 1], apar, ~apar)
        ma = damp(ma, torch.stack([u1, u0], 2))
        u0, u1 = logical(torch.where(valid, no[..., 1] - no[..., 0], 0.0), parent, child)
        mo = damp(mo, torch.stack([u0, u1], 2))
    if max(float((ma - pa).abs().max()), float((mo - po)[valid].abs().max())) > SETTLED:
        return None
    return _norm(beliefs(), 0.0)


def exact(case, seed):
    k, T, iters = case["kind"], case["T"], case["iters"]
    if k == "batch":
        outs = [_pair_exact(s, T, iters) for s in _mix(case, seed)]
        return torch.cat([o[0] for o in outs]), torch.cat([o[1] for o in outs])
    if k == "serve":
        out = []
        specs = _mix(case, seed)
        for s, c in zip(specs, _burst_losses(case, specs, seed)):
            if c is None:
                out.append(_pair_exact(s, T, iters))
            else:
                w = torch.from_numpy(c).to(_device()).double()
                out.append(_pair_grad(s, T, iters, lambda q: (w * q).sum())[:3])
        return out
    spec = _spec(case, seed)
    if k in ("grid", "rbm"):
        return _pair_exact(spec, T, iters, case.get("tol"), case.get("check", 1), settle=k == "rbm")
    if k == "grad":
        t = _target(case, spec, seed).to(_device()).double()
        q, _, gphi, gth = _pair_grad(spec, T, iters, lambda q: -(t * q).sum() / spec.num_vars)
        return q, gphi, gth
    if k == "triplet":
        return _triplet_exact(spec, T, iters)
    if k == "deconv":
        return _deconv_exact(spec, iters)
    nz = _noise(case, spec.num_var_states, seed)
    outs = [_deconv_exact(spec, iters, nz[s]) for s in range(case["S"])]
    if any(o is None for o in outs):
        return None
    return torch.stack([o[0] for o in outs]), torch.stack([o[1] for o in outs])
