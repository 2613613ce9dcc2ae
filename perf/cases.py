"""Timing cases of the advection library: what a program that uses it has it do.

A case is a dict of plain values; `listed` gives the fixed ones, `draw` more of
the same ranges.  The kinds, by use:

  step      `ram_step` on rows that share one mesh: a polar disk (or one row)
            advanced n steps in place.  One step a call is the hydro loop, whose
            velocities and time step are new at every step, so each call plans
            afresh; many steps a call is pure transport.
  ragged    `ram_step` on rows of their own lengths and meshes.
  split2d   `ram_step_split2d`: a 2D disk, the limited (or Lagrange) row step
            along the azimuth and the radial step across.
  adjoint   `ram_step_adjoint_steps`: back through a recorded trajectory.
  lim_adj   `ram_step_limited_adjoint`: one limited step backwards.
  rollout   the differentiable rollout in FP64, forward and backward, with the
            gradients of the state, the residual velocity and the bulk speed.

Sizes are those of `workloads.py`, the tests and the benchmark, or lie between
them.  Inputs come from the seed alone, made on the GPU: the disk's density
bump with noise, Keplerian bulk speeds, a noisy residual velocity and the time
step its Courant number allows.  `exact` evaluates the same steps from their
definitions in FP64 torch operations, with gradients by torch's autograd.
"""
from __future__ import annotations

import math

import torch

from paper_2305_05362_amd import _lib as R
from paper_2305_05362_amd.autograd import rollout

DEVICE = "cuda"
DTYPES = {"f32": torch.float32, "f64": torch.float64}


# --------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------

def listed():
    return [
        # one periodic row of 256 cells, one step a call: launches and latency
        dict(name="row256_f64_step", kind="step", rows=1, cols=256, mesh="uniform", dtype="f64",
             order=5, scan="f64", dv=False, steps=1),
        # the 512 x 2048 disk inside a hydro loop: one step a call
        dict(name="disk512x2048_f32_step", kind="step", rows=512, cols=2048, mesh="bump",
             dtype="f32", order=5, scan="direct", dv=True, steps=1),
        # the production disk inside a hydro loop: one step a call
        dict(name="disk2048x16384_f32_step", kind="step", rows=2048, cols=16384, mesh="bump",
             dtype="f32", order=5, scan="direct", dv=True, steps=1),
        # the production disk, steps in one call (the headline workload)
        dict(name="disk2048x16384_f32_20", kind="step", rows=2048, cols=16384, mesh="bump",
             dtype="f32", order=5, scan="direct", dv=True, steps=20),
        # an arbitrary mesh (no two cells alike) with an odd row length
        dict(name="stretched1000x6001_f32_10", kind="step", rows=1000, cols=6001,
             mesh="stretched", dtype="f32", order=5, scan="twosum", dv=True, steps=10),
        # the FP64 path with its default cumulative
        dict(name="disk1024x4096_f64_10", kind="step", rows=1024, cols=4096, mesh="bump",
             dtype="f64", order=5, scan="f64", dv=True, steps=10),
        # the ragged batch: 4096 rows of 64..8192 cells, bulk transport only (at
        # order 3: order 5 is unstable over many steps on such meshes)
        dict(name="ragged4096_f32_20", kind="ragged", rows=4096, nmin=64, nmax=8192,
             dtype="f32", order=3, scan="twosum", dv=False, steps=20),
        # rows of their own meshes inside a hydro loop: one step a call
        dict(name="ragged1024_f32_step", kind="ragged", rows=1024, nmin=64, nmax=4096,
             dtype="f32", order=5, scan="twosum", dv=True, steps=1),
        # the 2D split step with the limited parabola
        dict(name="split2d_ppm1024x4096_f32_8", kind="split2d", rows=1024, cols=4096,
             mesh="bump", dtype="f32", order=5, scan="direct", recon="ppm", dv=True, steps=8),
        # the reverse pass through recorded steps (state and residual gradients)
        dict(name="adjoint1024x4096_f32_8", kind="adjoint", rows=1024, cols=4096, mesh="bump",
             dtype="f32", order=5, dv=True, steps=8),
        # one limited step backwards
        dict(name="lim_adj_ppm1024x4096_f32", kind="lim_adj", rows=1024, cols=4096, mesh="bump",
             dtype="f32", recon="ppm", dv=True, steps=1),
        # forward and backward of the differentiable rollout, every gradient
        dict(name="rollout512x2048_f64_8", kind="rollout", rows=512, cols=2048, mesh="bump",
             dtype="f64", order=5, scan="f64", dv=True, steps=8, checkpoint=4),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "ragged", "ragged", "split2d", "adjoint",
                       "lim_adj", "rollout"])
    order = rng.choice([1, 3, 5, 5, 5])
    mesh = rng.choice(["bump", "bump", "stretched", "uniform"])
    if kind == "ragged":
        nmax = _log_int(rng, 128, 8192)
        c = dict(kind=kind, rows=_log_int(rng, 16, 4096), nmin=min(64, nmax // 2), nmax=nmax,
                 dtype=rng.choice(["f32", "f32", "f64"]), order=order, dv=rng.random() < 0.4)
        c["steps"] = rng.choice([1, 8, 20])
        if c["steps"] > 1:
            c["order"] = min(order, 3)
    else:
        most = {"step": 1 << 25, "split2d": 1 << 23, "adjoint": 1 << 23, "lim_adj": 1 << 23,
                "rollout": 1 << 20}[kind]
        cols = _log_int(rng, 64, 16384)
        rows = _log_int(rng, 1 if kind == "step" else 8, min(2048, most // cols))
        if rng.random() < 0.5:            # mesh generators like multiples of four
            cols -= cols % 4
        c = dict(kind=kind, rows=rows, cols=cols, mesh=mesh, order=order,
                 dtype="f64" if kind == "rollout" else "f32", dv=True)
        c["steps"] = 1 if kind == "lim_adj" else rng.choice([1, 4, 10])
        if kind == "step":
            c["dtype"] = rng.choice(["f32", "f32", "f64"])
            c["dv"] = rng.random() < 0.8
            c["steps"] = rng.choice([1, 1, 10, 20])
        if kind == "rollout":
            c["checkpoint"] = rng.choice([0, 2, 4])
        if kind in ("lim_adj", "split2d"):
            c["recon"] = rng.choice(["plm", "ppm"] + (["none"] if kind == "split2d" else []))
    if kind not in ("adjoint", "lim_adj"):
        c["scan"] = (rng.choice(["f64", "direct"]) if c["dtype"] == "f64"
                     else rng.choice(["direct", "twosum", "f64"]))
    return c


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------

def _bump_edges(n, a=0.2, b=0.3, c=9.0):
    """n + 1 nodes on [-pi, pi] of the periodic-bump density (ten times finer in
    |phi| < a, cos^2 ramps to b), by bisection on its integral."""
    def integral(x):
        t = x.abs()
        w = b - a
        ramp = (1 + c) * a + (1 + 0.5 * c) * (t - a) + 0.5 * c * w / math.pi * torch.sin(
            math.pi * (t - a) / w)
        v = torch.where(t <= a, (1 + c) * t,
                        torch.where(t < b, ramp, (1 + c) * a + (1 + 0.5 * c) * w + (t - b)))
        return torch.sign(x) * v
    half = float(integral(torch.tensor(math.pi, dtype=torch.float64)))
    target = (2.0 * torch.arange(1, n, dtype=torch.float64) / n - 1.0) * half
    lo = torch.full((n - 1,), -math.pi, dtype=torch.float64)
    hi = -lo
    for _ in range(58):
        mid = 0.5 * (lo + hi)
        below = integral(mid) < target
        lo, hi = torch.where(below, mid, lo), torch.where(below, hi, mid)
    e = torch.empty(n + 1, dtype=torch.float64)
    e[0], e[-1] = -math.pi, math.pi
    e[1:-1] = 0.5 * (lo + hi)
    return e


def _radii(n):
    e = 0.4 * (2.5 / 0.4) ** (torch.arange(n + 1, dtype=torch.float64) / n)
    e[0], e[-1] = 0.4, 2.5
    return e


def _grid(w):
    """Cell sizes as multiples of 2^-20: their running sums are exact, whatever
    the order they are formed in."""
    return torch.round(w * 2.0 ** 20) / 2.0 ** 20


def _disk(case, seed, device):
    """Rows that share one mesh on [-pi, pi]: a disk's radii, or one row."""
    g = torch.Generator(device=device)
    g.manual_seed(seed)
    dt_ = DTYPES[case["dtype"]]
    nr, n = case["rows"], case["cols"]
    kw = dict(generator=g, device=device, dtype=torch.float64)
    if case["mesh"] == "bump":
        x = _bump_edges(n).to(device)
    elif case["mesh"] == "uniform":
        x = (-math.pi + 2 * math.pi / n * torch.arange(n + 1, dtype=torch.float64)).to(device)
        x[-1] = math.pi
    else:
        w = _grid(8.0 ** torch.rand(n, **kw))
        x = torch.zeros(n + 1, dtype=torch.float64, device=device)
        x[1:] = torch.cumsum(w, 0)
        x = -math.pi + 2 * math.pi * x / x[-1]
        x[-1] = math.pi
    re = _radii(nr).to(device)
    rc = 0.5 * (re[1:] + re[:-1])
    xc, dx = 0.5 * (x[1:] + x[:-1]), x[1:] - x[:-1]
    v0 = rc ** -1.5 * (1 + 1e-3 * torch.randn(nr, **kw))
    d2 = rc[:, None] ** 2 + 1.0 - 2.0 * rc[:, None] * torch.cos(xc)[None, :]
    q = 1.0 + torch.exp(-d2 / (2 * 0.05 ** 2)) + 1e-3 * torch.randn(nr, n, **kw)
    dv = 0.01 * v0[:, None] * torch.sin(x[:-1])[None, :] * torch.randn(nr, n, **kw)
    lim = torch.minimum(dx, torch.roll(dx, 1))
    dt = 0.5 * float((lim[None, :] / dv.abs().clamp_min(1e-12)).min())
    if not case["dv"]:          # ten cells and a fraction a step
        dt = 10.3 * 2 * math.pi / n / float(v0.max())
    inp = dict(x=x, re=re, v0=v0, dt=dt, q=q.to(dt_), dv=dv.to(dt_) if case["dv"] else None,
               shape=(nr, n))
    if case["kind"] == "split2d":
        u = 0.01 * re[:, None] ** -0.5 * torch.sin(xc)[None, :] * torch.randn(nr + 1, n, **kw)
        u[0] = 0.0
        u[-1] = 0.0
        if nr > 1:
            dr = re[1:] - re[:-1]
            limr = torch.minimum(dr[1:], dr[:-1])[:, None] / u[1:-1].abs().clamp_min(1e-12)
            inp["dt"] = min(dt, 0.5 * float(limr.min()))
        inp["u"] = u.to(dt_)
    if case["kind"] in ("adjoint", "lim_adj"):
        # a recorded trajectory: the states and post-shift states of the steps
        inp["qbar"] = torch.randn(nr, n, **kw).to(dt_)
        rows = _Flat.shared(x, nr, n)
        with torch.no_grad():
            traj, half, cur = [], [], inp["q"]
            for _ in range(case["steps"]):
                traj.append(cur.reshape(-1))
                mid = (_shift_limited(rows, cur.double().reshape(-1), v0, inp["dt"], case["recon"])
                       if case["kind"] == "lim_adj" else
                       _shift(rows, cur.double().reshape(-1), v0, inp["dt"], case["order"]))
                mid = mid.to(dt_)
                half.append(mid)
                cur = _residual(rows, mid.double(), inp["dv"].double().reshape(-1),
                                inp["dt"]).to(dt_)
        inp["traj"], inp["half"] = torch.stack(traj), torch.stack(half)
    return inp


def _ragged(case, seed, device):
    """Rows of random lengths on [0, 1), cell sizes up to 20 times apart."""
    g = torch.Generator(device=device)
    g.manual_seed(seed)
    dt_ = DTYPES[case["dtype"]]
    nr = case["rows"]
    kw = dict(generator=g, device=device, dtype=torch.float64)
    # the row lengths are the batch's own, whatever its meshes and states are
    own = torch.Generator().manual_seed(nr)
    lens = torch.randint(case["nmin"], case["nmax"] + 1, (nr,), generator=own).to(device)
    ptr = torch.zeros(nr + 1, dtype=torch.int64, device=device)
    ptr[1:] = torch.cumsum(lens, 0)
    total = int(ptr[-1])
    row = torch.repeat_interleave(torch.arange(nr, device=device), lens)
    i = torch.arange(total, device=device) - ptr[row]
    w = _grid(20.0 ** torch.rand(total, **kw))
    cs = torch.cumsum(w, 0)
    base = cs[ptr[:-1]] - w[ptr[:-1]]
    size = cs[ptr[1:] - 1] - base
    edges = torch.zeros(total + nr, dtype=torch.float64, device=device)
    edges[ptr[:-1][row] + row + i + 1] = (cs - base[row]) / size[row]
    edges[ptr[1:] + torch.arange(nr, device=device)] = 1.0
    rows = _Flat(edges, ptr, row, i)
    q = torch.ones(total, dtype=torch.float64, device=device)
    for _ in range(3):
        amp = 0.25 * torch.rand(nr, **kw)[row]
        m = torch.randint(1, 17, (nr,), generator=g, device=device)[row]
        ph = 2 * math.pi * torch.rand(nr, **kw)[row]
        k = 2 * math.pi * m
        q -= amp * (torch.cos(k * rows.xr + ph) - torch.cos(k * rows.xl + ph)) / (k * rows.dx)
    v0, dt, dv = (0.5 + 19.5 * torch.rand(nr, **kw)) / lens, 1.0, None
    if case["dv"]:
        dv = 0.3 * torch.randn(total, **kw)
        lim = torch.minimum(rows.dx, rows.dx[rows.nb(-1)])
        dt = 0.5 * float((lim / dv.abs().clamp_min(1e-12)).min())
        v0 = v0 / dt
        dv = dv.to(dt_)
    return dict(edges=edges, ptr=ptr, rows=rows, v0=v0, dt=dt, q=q.to(dt_), dv=dv)


def prepare(case, seed):
    ragged = case["kind"] == "ragged"
    inp = (_ragged if ragged else _disk)(case, seed, DEVICE)
    st = dict(case=case, v0=inp["v0"], dt=inp["dt"])
    if ragged:
        st["rows"] = R.Rows(inp["edges"], case["rows"], 0, inp["ptr"], False, inp["q"].numel())
    else:
        st["rows"] = R.Rows(inp["x"], case["rows"], case["cols"], None, True)
    flat = {k: inp[k].reshape(-1) for k in ("q", "dv") if inp.get(k) is not None}
    st["q0"], st["dv"] = flat["q"], flat.get("dv")
    st["scan"] = R.SCANS[case["scan"]] if "scan" in case else None
    st["recon"] = R.RECONS.get(case.get("recon"), 0)
    if case["kind"] in ("step", "ragged", "split2d"):
        st["q"] = flat["q"].clone()
    if case["kind"] == "split2d":
        st["re"], st["u"] = inp["re"], inp["u"].reshape(-1)
    if case["kind"] in ("adjoint", "lim_adj"):
        st["qbar"], st["traj"], st["half"] = inp["qbar"].reshape(-1), inp["traj"], inp["half"]
        st["dvbar"] = torch.empty_like(st["dv"])
        st["work"] = torch.empty_like(st["q0"])
        st["out"] = torch.empty_like(st["q0"])
    return st


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------

def run(st):
    case = st["case"]
    rows, v0, dv, dt, n = st["rows"], st["v0"], st["dv"], st["dt"], case["steps"]
    kind = case["kind"]
    if kind in ("step", "ragged"):
        # a hydro loop goes on from its state; a longer run starts from the kept
        # initial state, as an ensemble's members do
        if n > 1 or kind == "ragged":
            st["q"].copy_(st["q0"])
        return R.ram_step(rows, st["q"], v0, dv, dt, case["order"], n, st["scan"])
    if kind == "split2d":
        st["q"].copy_(st["q0"])
        return R.ram_step_split2d(rows, st["q"], v0, dv, st["re"], st["u"], dt, case["order"], n,
                                  st["scan"], st["recon"])
    if kind == "adjoint":
        st["dvbar"].zero_()
        st["out"].copy_(st["qbar"])
        R.ram_step_adjoint_steps(rows, st["traj"], st["half"], dv, st["out"], st["work"], v0, dt,
                                 case["order"], n, dvbar=st["dvbar"])
        return dict(q=st["out"], dv=st["dvbar"])
    if kind == "lim_adj":
        st["dvbar"].zero_()
        R.ram_step_limited_adjoint(rows, st["traj"][0], st["half"][0], dv, st["qbar"], st["out"],
                                   v0, dt, st["recon"], dvbar=st["dvbar"])
        return dict(q=st["out"], dv=st["dvbar"])
    leaves = [st["q0"].detach().requires_grad_(True), v0.detach().requires_grad_(True),
              dv.detach().requires_grad_(True)]
    out = rollout(leaves[0], rows, leaves[1], leaves[2], dt, case["order"], n,
                  checkpoint=case["checkpoint"], scan=st["scan"])
    grads = torch.autograd.grad(0.5 * out.square().sum(), leaves)
    return dict(out=out.detach(), q=grads[0], v0=grads[1], dv=grads[2])


def work(case):
    """Bytes: each step reads and writes the state and reads its velocities once
    (the backward kinds: gradient in and out, the recorded states, the residual
    gradient read and written); per-row meshes add their nodes.  Operations a
    cell: the interpolant's weights and sums, the residual, the limiter."""
    e = 8 if case["dtype"] == "f64" else 4
    if case["kind"] == "ragged":
        cells = case["rows"] * (case["nmin"] + case["nmax"]) // 2
    else:
        cells = case["rows"] * case["cols"]
    dv = e if case["dv"] else 0
    per = {"step": 2 * e + dv, "ragged": 2 * e + dv + 8, "split2d": 5 * e + dv,
           "adjoint": 6 * e, "lim_adj": 7 * e, "rollout": 2 * e + dv + 7 * e}[case["kind"]]
    order = case.get("order", 5)
    ops = 10 * (order + 1) + (25 if case["dv"] else 0)
    ops = {"split2d": 150, "adjoint": 2 * ops, "lim_adj": 300, "rollout": 3 * ops}.get(
        case["kind"], ops)
    return {"bytes": float(per) * cells * case["steps"], "flops": float(ops) * cells * case["steps"]}


# --------------------------------------------------------------------------
# the same steps from their definitions, in FP64 torch operations
# --------------------------------------------------------------------------

class _Flat:
    """All rows' cells back to back: left and right nodes, sizes, neighbours."""

    def __init__(self, edges, ptr, row, i):
        self.row, self.i = row, i
        self.start = ptr[:-1][row]
        self.n = (ptr[1:] - ptr[:-1])[row]
        at = self.start + row + i
        self.xl, self.xr = edges[at], edges[at + 1]
        self.dx = self.xr - self.xl
        first = ptr[:-1] + torch.arange(len(ptr) - 1, device=ptr.device)
        last = ptr[1:] + torch.arange(len(ptr) - 1, device=ptr.device)
        self.x0, self.len = edges[first], edges[last] - edges[first]
        self._nb = {}

    @classmethod
    def shared(cls, x, nr, n):
        ptr = torch.arange(nr + 1, device=x.device) * n
        row = torch.arange(nr, device=x.device).repeat_interleave(n)
        i = torch.arange(n, device=x.device).repeat(nr)
        return cls(x.repeat(nr), ptr, row, i)

    def nb(self, k):
        if k not in self._nb:
            self._nb[k] = self.start + torch.remainder(self.i + k, self.n)
        return self._nb[k]

    def at(self, cell, k):
        """The cell k cells right of `cell` in its row (periodic)."""
        return self.start + torch.remainder(cell - self.start + k, self.n)


def _sources(rows, v0, dt):
    """Per left node: its source cell, the position in it, its extended index."""
    s = (v0 * dt)[rows.row]
    x0, ln = rows.x0[rows.row], rows.len[rows.row]
    y = rows.xl - s
    k = torch.floor((y.detach() - x0) / ln)
    y = y - k * ln
    yd = y.detach()
    keys = rows.row * 2.0 + (rows.xl - x0) / ln
    c = torch.searchsorted(keys, rows.row * 2.0 + (yd - x0) / ln, right=True) - 1
    c = torch.minimum(torch.maximum(c, rows.start), rows.start + rows.n - 1)
    for _ in range(2):
        c = torch.where((rows.xl[c] > yd) & (c > rows.start), c - 1, c)
        c = torch.where((rows.xr[c] <= yd) & (c < rows.start + rows.n - 1), c + 1, c)
    theta = (y - rows.xl[c]) / rows.dx[c]
    return c, theta, (c - rows.start) + k.to(torch.int64) * rows.n


def _remap(rows, q, c, g, ell):
    """Whole cells between a cell's two shifted nodes plus the partial integrals."""
    nxt = rows.nb(1)
    last = rows.i == rows.n - 1
    count = torch.where(last, g[nxt] + rows.n, g[nxt]) - g
    mass = q * rows.dx
    whole = torch.zeros_like(q)
    for k in range(int(count.max())):
        whole = whole + torch.where(count > k, mass[rows.at(c, k)], torch.zeros_like(q))
    return (whole + ell[nxt] - ell) / rows.dx


def _shift(rows, q, v0, dt, order):
    c, theta, g = _sources(rows, v0, dt)
    lo = (order - 1) // 2
    h = rows.dx[c]
    pos, cum = [None] * (order + 1), [None] * (order + 1)
    pos[lo] = cum[lo] = torch.zeros_like(q)
    for b in range(lo + 1, order + 1):
        m = rows.at(c, b - lo - 1)
        pos[b], cum[b] = pos[b - 1] + rows.dx[m] / h, cum[b - 1] + q[m] * rows.dx[m]
    for b in range(lo - 1, -1, -1):
        m = rows.at(c, b - lo)
        pos[b], cum[b] = pos[b + 1] - rows.dx[m] / h, cum[b + 1] - q[m] * rows.dx[m]
    ell = torch.zeros_like(q)
    for b in range(order + 1):
        if b == lo:
            continue
        w = torch.ones_like(q)
        for a in range(order + 1):
            if a != b:
                w = w * (theta - pos[a]) / (pos[b] - pos[a])
        ell = ell + w * cum[b]
    return _remap(rows, q, c, g, ell)


def _van_leer(up, dn):
    """Harmonic mean of two one-sided slopes, zero where they differ in sign."""
    ok = up * dn > 0
    den = torch.where(ok, up + dn, torch.ones_like(up))
    return torch.where(ok, 2 * up * dn / den, torch.zeros_like(up))


def _plm_slope(rows, q):
    nx, pv = rows.nb(1), rows.nb(-1)
    return _van_leer((q[nx] - q) / (0.5 * (rows.dx + rows.dx[nx])),
                     (q - q[pv]) / (0.5 * (rows.dx + rows.dx[pv])))


def _ppm_edges(rows, q):
    """Colella & Woodward's constrained left and right edge values of every cell."""
    nx, pv = rows.nb(1), rows.nb(-1)
    h, hp, hm = rows.dx, rows.dx[nx], rows.dx[pv]
    hpp = rows.dx[rows.nb(2)]
    up, dn = q[nx] - q, q - q[pv]
    d = h / (hm + h + hp) * ((2 * hm + h) / (hp + h) * up + (h + 2 * hp) / (hm + h) * dn)
    mag = torch.minimum(d.abs(), torch.minimum(2 * up.abs(), 2 * dn.abs()))
    d = torch.where(up * dn > 0, mag * torch.sign(d.detach()), torch.zeros_like(q))
    w1 = 2 * hp * h / (h + hp) * ((hm + h) / (2 * h + hp) - (hpp + hp) / (2 * hp + h))
    w2 = -h * (hm + h) / (2 * h + hp)
    w3 = hp * (hp + hpp) / (h + 2 * hp)
    face = q + h / (h + hp) * up + (w1 * up + w2 * d[nx] + w3 * d) / (hm + h + hp + hpp)
    left, right = face[pv], face
    flat = (right - q) * (q - left) <= 0
    dq, qa = right - left, q - 0.5 * (left + right)
    pull_l = ~flat & (dq * qa > dq * dq / 6)
    pull_r = ~flat & ~pull_l & (-dq * dq / 6 > dq * qa)
    lv = torch.where(flat, q, torch.where(pull_l, 3 * q - 2 * right, left))
    rv = torch.where(flat, q, torch.where(pull_r, 3 * q - 2 * left, right))
    return lv, rv


def _shift_limited(rows, q, v0, dt, recon):
    c, th, g = _sources(rows, v0, dt)
    h = rows.dx[c]
    if recon == "plm":
        ell = h * q[c] * th + 0.5 * (_plm_slope(rows, q) * rows.dx ** 2)[c] * (th * th - th)
    else:
        lv, rv = _ppm_edges(rows, q)
        q6 = (6 * q - 3 * (lv + rv))[c]
        lv, rv = lv[c], rv[c]
        ell = h * (lv * th + 0.5 * (rv - lv) * th ** 2 + q6 * (0.5 * th ** 2 - th ** 3 / 3))
    return _remap(rows, q, c, g, ell)


def _residual(rows, q, dv, dt):
    nx, pv = rows.nb(1), rows.nb(-1)
    slope = _plm_slope(rows, q)
    left = q[pv] + 0.5 * slope[pv] * (rows.dx[pv] - dv * dt)
    right = q - 0.5 * slope * (rows.dx + dv * dt)
    flux = dv * torch.where(dv >= 0, left, right)
    return q - dt * (flux[nx] - flux) / rows.dx


def _radial(re, q, u, dt):
    nr = q.shape[0]
    rc, dr = 0.5 * (re[1:] + re[:-1]), (re[1:] - re[:-1])[:, None]
    slope = torch.zeros_like(q)
    if nr > 2:
        d = (q[1:] - q[:-1]) / (rc[1:] - rc[:-1])[:, None]
        slope[1:-1] = _van_leer(d[1:], d[:-1])
    flux = torch.zeros_like(u)
    v = u[1:-1]
    below = q[:-1] + 0.5 * slope[:-1] * (dr[:-1] - v * dt)
    above = q[1:] - 0.5 * slope[1:] * (dr[1:] + v * dt)
    flux[1:-1] = v * torch.where(v >= 0, below, above)
    rf = re[:, None] * flux
    area = 0.5 * (re[1:] ** 2 - re[:-1] ** 2)[:, None]
    return q - dt * (rf[1:] - rf[:-1]) / area


def _advance(case, rows, q, v0, dv, dt):
    recon = case.get("recon", "none")
    q = (_shift(rows, q, v0, dt, case["order"]) if recon == "none"
         else _shift_limited(rows, q, v0, dt, recon))
    return q if dv is None else _residual(rows, q, dv, dt)


def exact(case, seed):
    return _exact(case, seed, DEVICE)


def _exact(case, seed, device):
    kind, n = case["kind"], case["steps"]
    inp = (_ragged if kind == "ragged" else _disk)(case, seed, device)
    rows = inp["rows"] if kind == "ragged" else _Flat.shared(inp["x"], *inp["shape"])
    v0, dt = inp["v0"], inp["dt"]
    q = inp["q"].double().reshape(-1)
    dv = None if inp["dv"] is None else inp["dv"].double().reshape(-1)
    if kind in ("step", "ragged", "split2d"):
        with torch.no_grad():
            # a hydro loop's state goes on: its first pass is what is compared
            for _ in range(n):
                q = _advance(case, rows, q, v0, dv, dt)
                if kind == "split2d":
                    q = _radial(inp["re"], q.reshape(inp["shape"]), inp["u"].double(),
                                dt).reshape(-1)
        return q
    if kind == "rollout":
        leaves = [t.requires_grad_(True) for t in (q, v0, dv)]
        out = leaves[0]
        for _ in range(n):
            out = _advance(case, rows, out, leaves[1], leaves[2], dt)
        grads = torch.autograd.grad(0.5 * out.square().sum(), leaves)
        return dict(out=out.detach(), q=grads[0], v0=grads[1], dv=grads[2])
    # one step at a time: the shift's transpose at the recorded state, the
    # residual's at the recorded post-shift state
    qbar = inp["qbar"].double().reshape(-1)
    dvbar = torch.zeros_like(qbar)
    for k in range(n - 1, -1, -1):
        half = inp["half"][k].double().requires_grad_(True)
        dvk = dv.clone().requires_grad_(True)
        qbar, gdv = torch.autograd.grad(_residual(rows, half, dvk, dt), [half, dvk], qbar)
        dvbar = dvbar + gdv
        full = inp["traj"][k].double().requires_grad_(True)
        mid = (_shift_limited(rows, full, v0, dt, case["recon"]) if kind == "lim_adj"
               else _shift(rows, full, v0, dt, case["order"]))
        qbar, = torch.autograd.grad(mid, [full], qbar)
    return dict(q=qbar, dv=dvbar)
