"""Workloads of the framework as a user's program runs them, for measuring.

Every case is one call, or one short sequence of calls, through the public
entry points of ``paper_1407_7486_amd``, on inputs made from a seed: unit
loops (closed random walks with the loop law's step variance, any number of
points), uploaded once and kept on the device, and the (rho_cm, T) grids of
the repository's workloads (rho linear from 0, T geometric).

``call`` names the entry point of a case:
  average      wl_average: host grids in, host results out (the usual call)
  average_ex   wl_average_ex: the same with the scale and rounding outputs
  async        wl_average_async: device grids and results on torch's stream
  batch        wl_average_batch: uneven requests in one call
  server       a running Server: submit the requests, wait, collect
  disc         wl_discretisation: the three levels and the extrapolation
  action       wl_average on the action grids, then wl_action
  correlation  wl_average with one loop per group, wl_correlation, wl_regroup
  generate     wl_ensemble_generate, wl_average on it, wl_ensemble_free
"""
import math
import random

import numpy as np
import torch

import paper_1407_7486_amd as wl

KINDS = {"const": wl.WL_CONST, "sech2": wl.WL_SECH2, "gauss": wl.WL_GAUSS,
         "rational": wl.WL_RATIONAL}
PRECISIONS = {"fp32c": wl.WL_FP32C, "fp32": wl.WL_FP32, "fp64": wl.WL_FP64,
              "fp32k": wl.WL_FP32K}
MODES = {"paper": wl.WL_DISC_PAPER, "full": wl.WL_DISC_FULL}

# Operations of one segment evaluation: about 19 common to every field
# (midpoint, radius, cross product, two sums), the field's own, and each
# transcendental as 4 (sech^2: rsq, exp, rcp, log); a scalar needs 4 fewer.
OPS = {"const": 19.0, "sech2": 49.0, "gauss": 33.0, "rational": 28.0}


def _case(name, call, kind, spin, precision, n_loops, n_ppl, groups, n_rho, n_T, **more):
    c = {"call": call, "kind": kind, "spin": spin, "precision": precision, "n_loops": n_loops,
         "n_ppl": n_ppl, "groups": groups, "n_rho": n_rho, "n_T": n_T, "eB0": 1.0, "lam": 1.0,
         "rho_hi": 5.0, "T_lo": 1e-3, "T_hi": 50.0}
    if name:
        c["name"] = name
    c.update(more)
    return c


def listed():
    return [
        # a first look at a tube on a handful of points: latency and launches
        _case("average_tiny", "average", "sech2", 1, "fp32c", 256, 512, 8, 3, 7,
              rho_hi=2.0, T_lo=1e-2, T_hi=20.0),
        # the small constant-field workload, checked against closed forms
        _case("average_const_1k", "average", "const", 0, "fp32c", 1024, 1024, 16, 8, 16,
              rho_hi=2.0, T_lo=1e-2, T_hi=10.0),
        # an ordinary call with everything odd: points per loop not a power
        # of two, a grid that fills no whole wavefront, all outputs
        _case("average_ragged", "average_ex", "gauss", 1, "fp32c", 2040, 1003, 24, 17, 33,
              eB0=2.0, lam=1.5, rho_hi=4.5),
        # the throughput workload: 65536 loops of 4096 points, a 64 x 64 grid
        _case("throughput_64k", "async", "sech2", 1, "fp32c", 65536, 4096, 64, 64, 64),
        # the precision-stress tube: a third of the grid points fail the
        # rounding estimate and are recomputed in FP64
        _case("stress_tube", "average_ex", "sech2", 0, "fp32c", 1024, 8192, 64, 32, 48,
              eB0=20.0, lam=4.0, T_hi=10.0),
        # FP64 throughout, at an ordinary size
        _case("average_fp64", "average", "sech2", 1, "fp64", 2048, 4096, 64, 32, 32),
        # a batch of uneven requests (both tubes, both spins, 4-128 x 8-64 grids)
        _case("batch_mixed", "batch", "", -1, "fp32c", 4096, 1024, 64, 0, 0,
              n_req=8, mix=1, rho_top=128, T_top=64),
        # serving: small requests arriving together at a running server
        _case("serve_burst", "server", "", -1, "fp32c", 1024, 1024, 32, 0, 0,
              n_req=8, mix=2, rho_top=24, T_top=24),
        # the discretisation estimate over an ordinary grid
        _case("discretisation", "disc", "sech2", 1, "fp32c", 4096, 2048, 64, 32, 32,
              mode="paper"),
        # the effective action of a Gaussian tube on its own quadrature grids
        _case("action", "action", "gauss", 1, "fp32c", 2048, 512, 32, 16, 24,
              eB0=2.5, lam=0.8, rho_hi=1.2, T_lo=0.05, T_hi=1.0),
        # correlations between grid points over loops, and shuffled groups
        _case("correlation", "correlation", "sech2", 1, "fp64", 2048, 256, 32, 8, 24,
              eB0=2.0, rho_hi=1.5, T_lo=0.05, T_hi=20.0, n_perms=4),
        # a new ensemble generated on the device and evaluated once
        _case("generate_evaluate", "generate", "sech2", 1, "fp32c", 16384, 4096, 64, 8, 8),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: any call, field, spin and offered
    precision, sizes spread over their logarithm, odd ones among them."""
    while True:
        call = rng.choice(["average", "average", "average_ex", "async", "batch", "server",
                           "disc", "action", "correlation", "generate"])
        kind = rng.choice(["const", "sech2", "sech2", "gauss", "rational"])
        spin = rng.randint(0, 1)
        precision = rng.choice(["fp32c", "fp32c", "fp32c", "fp32c", "fp64", "fp64", "fp32"])
        groups = rng.choice([4, 8, 15, 16, 24, 32, 64])
        n_loops = groups * max(1, _log_int(rng, 256, 32768) // groups)
        n_ppl = _log_int(rng, 200, 8192)
        n_rho, n_T = _log_int(rng, 2, 64), _log_int(rng, 4, 64)
        field = dict(eB0=round(rng.uniform(0.5, 10.0), 3), lam=round(rng.uniform(0.2, 5.0), 3))
        field.update(rho_hi=round(3.0 * field["lam"], 3), T_hi=round(50.0 / field["eB0"], 3))
        more = {}
        if call in ("batch", "server"):
            kind, spin, n_rho, n_T, field = "", -1, 0, 0, {}
            n_loops = min(n_loops, 4096 if call == "batch" else 2048)
            n_loops -= n_loops % groups
            n_ppl = min(n_ppl, 2048)
            top = rng.choice([12, 24, 48])
            more = dict(n_req=rng.randint(2, 16), mix=rng.randint(3, 10 ** 6), rho_top=top,
                        T_top=top)
        elif call == "disc":
            n_ppl -= n_ppl % 4
            more = dict(mode=rng.choice(["paper", "full"]))
        elif call == "action":
            kind = rng.choice(["sech2", "gauss", "rational"])
            n_rho, n_T = 2 * rng.randint(4, 24), 2 * rng.randint(6, 24)
            field.update(rho_hi=round(1.5 * field["lam"], 3), T_hi=1.0)
            more = dict(T_lo=0.05)
        elif call == "correlation":
            kind = rng.choice(["sech2", "gauss"])
            n_loops = min(n_loops, 8192)
            n_loops -= n_loops % groups
            n_rho, n_T = rng.randint(2, 12), rng.randint(4, 32)
            field.update(T_hi=round(20.0 / field["eB0"], 3))
            more = dict(T_lo=0.05, n_perms=rng.randint(1, 8))
        elif call == "generate":
            n_ppl = 1 << rng.randint(8, 13)
        c = _case("", call, kind, spin, precision, n_loops, n_ppl, groups, n_rho, n_T,
                  **{**field, **more})
        evals = _evals(c)
        if 1e6 <= evals <= (3e10 if precision == "fp64" else 1e11):
            return c


# ------------------------------------------------------------------ inputs
def _device():
    return torch.device("cuda", torch.cuda.current_device())


def _unit_loops(n_loops, n_ppl, seed):
    """Unit loops as device float32 (x, y): closed random walks of n_ppl
    steps whose variance per component is (2/N)(1 - 1/N), centred."""
    gen = torch.Generator(device=_device()).manual_seed(1000003 * int(seed) + 17)
    out = []
    for _ in range(2):
        z = torch.randn((n_loops, n_ppl), generator=gen, device=_device(), dtype=torch.float32)
        w = torch.cumsum(z.double(), dim=1)
        del z
        w *= math.sqrt(2.0 / n_ppl)
        frac = torch.arange(1, n_ppl + 1, device=_device(), dtype=torch.float64) / n_ppl
        w -= w[:, -1:].clone() * frac
        w -= w.mean(dim=1, keepdim=True)
        out.append(w.float().contiguous())
        del w
    return out


def _grids(case):
    return (np.linspace(0.0, case["rho_hi"], case["n_rho"]),
            np.geomspace(case["T_lo"], case["T_hi"], case["n_T"]))


def _action_spec(case):
    return wl.action_spec(1.0, case["T_lo"], case["T_hi"], case["n_T"], case["rho_hi"],
                          case["n_rho"])


def _requests(case, seed=0):
    """The uneven requests of a batch: kinds, spins and grid sizes from the
    case's mix, the fields' strengths and widths also from the seed."""
    sizes, fields = random.Random(case["mix"]), random.Random(case["mix"] * 7919 + seed)
    reqs = []
    for _ in range(case["n_req"]):
        eB0, lam = fields.uniform(0.5, 10.0), fields.uniform(0.2, 5.0)
        reqs.append(dict(kind=KINDS[sizes.choice(["sech2", "gauss"])], eB0=eB0, lam=lam,
                         rho=np.linspace(0.0, 3.0 * lam, sizes.randint(4, case["rho_top"])),
                         T=np.geomspace(1e-3, 50.0 / eB0, sizes.randint(8, case["T_top"])),
                         spin=sizes.randint(0, 1), precision=PRECISIONS[case["precision"]]))
    return reqs


class _State:
    """A program's context and ensemble, freed with the object."""

    def __init__(self):
        self.ctx = wl.wl_create(torch.cuda.current_device(),
                                torch.cuda.current_stream().cuda_stream)
        self.ens = self.server = None

    def __del__(self):
        if self.server is not None:
            self.server.close()
        if self.ens is not None:
            wl.wl_ensemble_free(self.ens)
        wl.wl_destroy(self.ctx)


def _perms(case, seed):
    rng = np.random.default_rng(seed)
    perms = np.stack([rng.permutation(case["n_loops"]) for _ in range(case["n_perms"])])
    which = rng.integers(0, case["n_perms"], case["n_rho"] * case["n_T"]).astype(np.int32)
    return perms, which


def prepare(case, seed):
    s = _State()
    s.case, s.seed = case, seed
    s.precision = PRECISIONS[case["precision"]]
    call = case["call"]
    if call != "generate":
        x, y = _unit_loops(case["n_loops"], case["n_ppl"], seed)
        torch.cuda.current_stream().synchronize()
        s.ens = wl.wl_ensemble_upload(s.ctx, x, y, case["groups"])
        del x, y
    if call in ("batch", "server"):
        s.requests = _requests(case, seed)
        if call == "server":
            s.server = wl.Server(s.ctx, s.ens)
        return s
    s.field = wl.field(KINDS[case["kind"]], case["eB0"], case["lam"])
    if call == "action":
        s.spec = _action_spec(case)
        s.T, s.rho = wl.wl_action_grids(s.spec)
        return s
    s.rho, s.T = _grids(case)
    if call == "async":
        dev, n = _device(), case["n_rho"] * case["n_T"]
        s.d_rho, s.d_T = torch.tensor(s.rho, device=dev), torch.tensor(s.T, device=dev)
        s.d_mean = torch.empty(n, dtype=torch.float64, device=dev)
        s.d_err = torch.empty(n, dtype=torch.float64, device=dev)
        s.d_sums = torch.empty(case["groups"] * n, dtype=torch.float64, device=dev)
    elif call == "correlation":
        # the group sums of an evaluation with one loop per group are the
        # loops' own values
        wl.wl_ensemble_set_groups(s.ens, case["n_loops"])
        s.perms, s.which = _perms(case, seed)
    return s


def run(s):
    case, call = s.case, s.case["call"]
    spin = case["spin"]
    if call == "average":
        mean, err, sums = wl.wl_average(s.ctx, s.ens, s.field, s.rho, s.T, spin, s.precision)
        return {"mean": mean, "err": err, "group_sums": sums}
    if call == "average_ex":
        return wl.wl_average_ex(s.ctx, s.ens, s.field, s.rho, s.T, spin, s.precision)
    if call == "async":
        wl.wl_average_async(s.ctx, s.ens, s.field, s.d_rho, s.d_T, spin, s.precision, s.d_mean,
                            s.d_err, s.d_sums)
        return {"mean": s.d_mean, "err": s.d_err, "group_sums": s.d_sums}
    if call == "batch":
        return [list(r) for r in wl.wl_average_batch(s.ctx, s.ens, s.requests)]
    if call == "server":
        tickets = [s.server.submit(q) for q in s.requests]
        out = []
        for t in tickets:
            status, _ = s.server.wait(t)
            if status != wl.WL_OK:
                raise RuntimeError(f"request failed with status {status}")
            out.append(list(s.server.result(t)))
        return out
    if call == "disc":
        mean, err, delta, sums = wl.wl_discretisation(s.ctx, s.ens, s.field, s.rho, s.T, spin,
                                                      s.precision, MODES[case["mode"]])
        return {"mean": mean, "err": err, "delta": delta, "group_sums": sums}
    if call == "action":
        mean, err, sums = wl.wl_average(s.ctx, s.ens, s.field, s.rho, s.T, spin, s.precision)
        act = wl.wl_action(s.ctx, s.spec, s.field, spin, sums, case["n_loops"])
        return {"mean": mean, "err": err, "group_sums": sums, "action": act}
    if call == "correlation":
        _, _, per = wl.wl_average(s.ctx, s.ens, s.field, s.rho, s.T, spin, s.precision)
        per = per.reshape(case["n_loops"], -1)
        corr = wl.wl_correlation(s.ctx, per)
        sums = wl.wl_regroup(s.ctx, per, s.perms, case["groups"], s.which)
        return {"per_loop": per, "corr": corr, "group_sums": sums}
    ens = wl.wl_ensemble_generate(s.ctx, s.seed, 0, case["n_loops"], case["n_ppl"],
                                  case["groups"])
    try:
        mean, err, sums = wl.wl_average(s.ctx, ens, s.field, s.rho, s.T, spin, s.precision)
    finally:
        wl.wl_ensemble_free(ens)
    return {"mean": mean, "err": err, "group_sums": sums}


# -------------------------------------------------------------------- work
def _points(case):
    """(kind, spin, grid points) of every evaluation of a case."""
    if case["call"] in ("batch", "server"):
        names = {v: k for k, v in KINDS.items()}
        return [(names[q["kind"]], q["spin"], len(q["rho"]) * len(q["T"]))
                for q in _requests(case)]
    return [(case["kind"], case["spin"], case["n_rho"] * case["n_T"])]


def _evals(case):
    """Segment evaluations of one pass."""
    n = float(case["n_loops"]) * case["n_ppl"] * sum(p for _, _, p in _points(case))
    return 2.0 * n if case.get("mode") == "full" else n


def work(case):
    """Bytes: each loop point read once (8 bytes; written once when it is
    generated), the grids, and every result written once.  Operations: OPS
    per segment evaluation."""
    segments = float(case["n_loops"]) * case["n_ppl"]
    pts = sum(p for _, _, p in _points(case))
    groups, per_point, flops, moved = case["groups"], 2, 0.0, 8.0 * segments
    for kind, spin, p in _points(case):
        flops += segments * p * (OPS[kind] - (0.0 if spin else 4.0))
    call = case["call"]
    if call == "disc":
        groups, per_point = 4 * groups, 9
        if case["mode"] == "full":
            flops *= 2.0
    elif call == "average_ex":
        per_point = 4.125
    elif call == "correlation":
        n = float(case["n_loops"])
        groups, per_point = case["n_loops"] + groups, 0
        moved += 8.0 * (2.0 * n * pts + pts * pts + case["n_perms"] * n)
        flops += n * pts * (pts + 1)
    return {"bytes": moved + 8.0 * pts * (groups + per_point), "flops": flops}


# ------------------------------------------------------- values in 64 bits
def _field_values(kind, eB0, lam, r2):
    """(eA_phi/rho, eB) at squared radii r2."""
    if kind == wl.WL_CONST:
        return 0.5 * eB0, torch.full_like(r2, eB0)
    if kind == wl.WL_RATIONAL:
        q = 1.0 / (lam * lam + r2)
        return 0.5 * eB0 * lam * lam * q, eB0 * lam ** 4 * q * q
    v = r2 / (lam * lam)
    if kind == wl.WL_GAUSS:
        return 0.5 * eB0 * torch.where(v > 1e-30, -torch.expm1(-v) / v.clamp_min(1e-30),
                                       torch.ones_like(v)), eB0 * torch.exp(-v)
    u = torch.sqrt(v)
    e = torch.exp(-2.0 * u)
    far = (u * (1.0 - e) / (1.0 + e) - (u - math.log(2.0) + torch.log1p(e))) \
        / v.clamp_min(1e-30)
    near = 0.5 + v * (-0.25 + v * (1.0 / 9.0 + v * (-17.0 / 360.0 + v * (31.0 / 1575.0))))
    return eB0 * torch.where(v < 2.5e-3, near, far), eB0 * 4.0 * e / (1.0 + e) ** 2


class _Loops64:
    """Segments of unit loops in 64 bits: closed polygons through `points`."""

    def __init__(self, x, y):
        x1, y1 = torch.roll(x, -1, dims=1), torch.roll(y, -1, dims=1)
        self.n = x.shape[1]
        self.mx, self.my2 = 0.5 * (x + x1), (0.5 * (y + y1)) ** 2
        self.dy, self.c = y1 - y, x * y1 - y * x1

    def values(self, kind, eB0, lam, rho, T):
        """Per-loop phase and spin exponent at one grid point."""
        s = math.sqrt(T)
        r2 = (rho + s * self.mx) ** 2 + T * self.my2
        g, b = _field_values(kind, eB0, lam, r2)
        return ((rho * s * self.dy + T * self.c) * g).sum(1), T / self.n * b.sum(1)


def _w(phi, S, spin):
    return torch.cos(phi) * torch.cosh(S) if spin else torch.cos(phi)


def _statistics(w, groups):
    """(mean, err, group sums) of per-loop values (n_loops, n_rho, n_T)."""
    n = w.shape[0]
    sums = w.reshape(groups, n // groups, *w.shape[1:]).sum(1)
    m = sums.sum(0) / n
    err = torch.sqrt((((sums * (groups / n)) - m) ** 2).sum(0) / (groups * (groups - 1)))
    return m.cpu().numpy(), err.cpu().numpy(), sums.cpu().numpy()


def _generated(n_loops, n_ppl, seed):
    """The d-loops of wl_ensemble_generate from their definition: Philox4x32-10
    keyed by the seed, Box-Muller, midpoint recursion, centred, as float32."""
    dev, m32 = _device(), 0xFFFFFFFF
    blocks = torch.arange((n_ppl + 1) // 2, device=dev, dtype=torch.int64)[None, :]
    loop = torch.arange(n_loops, device=dev, dtype=torch.int64)[:, None]
    c = [blocks.expand(n_loops, -1).clone(), (loop & m32).expand(-1, blocks.shape[1]).clone(),
         (loop >> 32).expand(-1, blocks.shape[1]).clone(),
         torch.zeros((n_loops, blocks.shape[1]), device=dev, dtype=torch.int64)]
    k0, k1 = seed & m32, (seed >> 32) & m32
    for _ in range(10):
        p0, p1 = 0xD2511F53 * c[0], 0xCD9E8D57 * c[2]  # the high word survives the wrap
        c = [((p1 >> 32) & m32) ^ c[1] ^ k0, p1 & m32, ((p0 >> 32) & m32) ^ c[3] ^ k1, p0 & m32]
        k0, k1 = (k0 + 0x9E3779B9) & m32, (k1 + 0xBB67AE85) & m32
    u = [(w.double() + 0.5) / 2.0 ** 32 for w in c]
    z = []
    for trig in (torch.cos, torch.sin):
        pairs = [torch.sqrt(-2.0 * torch.log(u[i])) * trig(2.0 * math.pi * u[i + 1])
                 for i in (0, 2)]
        z.append(torch.stack(pairs, dim=2).reshape(n_loops, -1))
    out = []
    for zc in z:
        v = torch.zeros((n_loops, n_ppl), device=dev, dtype=torch.float64)
        nk, first = 2, 0
        while nk <= n_ppl:
            h = n_ppl // nk
            i = torch.arange(h, n_ppl, 2 * h, device=dev)
            mid = 0.5 * (v[:, i - h] + v[:, (i + h) % n_ppl])
            v[:, i] = mid + zc[:, first:first + nk // 2] / math.sqrt(nk)
            first += nk // 2
            nk *= 2
        out.append((v - v.mean(dim=1, keepdim=True)).float())
    return out


def _per_loop64(loops, kind, eB0, lam, rho, T, spin):
    """(w, S) of every loop on the grid."""
    n = loops.mx.shape[0]
    w = torch.empty((n, len(rho), len(T)), dtype=torch.float64, device=loops.mx.device)
    S = torch.zeros_like(w)
    for j, r in enumerate(rho):
        for k, t in enumerate(T):
            phi, sp = loops.values(kind, eB0, lam, float(r), float(t))
            w[:, j, k] = _w(phi, sp, spin)
            if spin:
                S[:, j, k] = sp
    return w, S


def _exact_disc(case, x, y, rho, T):
    kind, spin = KINDS[case["kind"]], case["spin"]
    whole = _Loops64(x, y)
    sub = [_Loops64(x[:, a::b], y[:, a::b]) for a, b in ((0, 2), (1, 4), (3, 4))]
    level = torch.empty((4, x.shape[0], len(rho), len(T)), dtype=torch.float64, device=x.device)
    for j, r in enumerate(rho):
        for k, t in enumerate(T):
            args = (kind, case["eB0"], case["lam"], float(r), float(t))
            (c, sc), (s, ss), (q, sq) = [l.values(*args) for l in sub]
            level[1, :, j, k] = _w(c, sc, spin)
            if case["mode"] == "full":
                level[0, :, j, k] = _w(*whole.values(*args), spin)
                level[2, :, j, k] = 0.5 * (_w(s, ss, spin) + _w(q, sq, spin))
            else:
                level[0, :, j, k] = _w(c / 2 + s / 4 + q / 4, sc / 2 + ss / 4 + sq / 4, spin)
                level[2, :, j, k] = _w((s + q) / 2, (ss + sq) / 2, spin)
    level[3] = (8.0 * level[0] - 6.0 * level[1] + level[2]) / 3.0
    st = [_statistics(level[i], case["groups"]) for i in range(4)]
    mean, err, sums = (np.stack([v[i] for v in st]) for i in range(3))
    return {"mean": mean, "err": err, "delta": np.abs(mean[0] - mean[3]), "group_sums": sums}


def _exact_action(case, sums, T, rho):
    """The action integrals from group sums, in numpy."""
    spin, eB0, lam, a = case["spin"], case["eB0"], case["lam"], case["T_lo"]
    G, nr, nt = sums.shape
    xa = 1.0 / (1.0 + a / case["T_hi"])
    k = np.arange(nt, 0, -1)
    c = np.where(k == nt, 1.0, np.where(k % 2 == 1, 4.0, 2.0))
    wt = c * (xa / nt) / 3.0 * case["T_hi"] / (k * xa / nt) ** 2
    b = _field_values(KINDS[case["kind"]], eB0, lam,
                      torch.tensor(rho ** 2, dtype=torch.float64))[1].numpy()
    b4, b6 = b ** 4, b ** 6
    if spin:
        ser = (-b4 / 45, b4 / 45, 2 * b6 / 945 - b4 / 90, (7 * b4 - 4 * b6) / 1890)
    else:
        ser = (7 * b4 / 360, -7 * b4 / 360, (147 * b4 - 31 * b6) / 15120,
               (31 * b6 - 49 * b4) / 15120)
    small = sum(co * a ** (i + 2) / (i + 2) for i, co in enumerate(ser))
    th = b[:, None] * T
    counter = 1 + th ** 2 / 3 if spin else 1 - th ** 2 / 6
    safe = np.maximum(th, 1e-12)
    with np.errstate(over="ignore"):
        lcf = np.where(th > 1e-12, safe / np.tanh(safe) if spin else safe / np.sinh(safe), 1.0)
    rows = np.concatenate([sums * (G / case["n_loops"]), lcf[None]])
    dens = small + (wt * np.exp(-T) / T ** 3 * (rows - counter)).sum(2)
    kr = np.arange(nr, 0, -1)
    cr = np.where(kr == nr, 1.0, np.where(kr % 2 == 1, 4.0, 2.0))
    wr = cr / nr / 3.0 * case["rho_hi"] / (kr / nr) ** 2
    act = (wr * rho * dens).sum(1) / (4.0 * math.pi)
    sem = lambda v: v.std(0, ddof=1) / math.sqrt(G)  # noqa: E731
    return {"density": dens[:G], "density_mean": dens[:G].mean(0), "density_err": sem(dens[:G]),
            "action": act[:G], "action_mean": float(act[:G].mean()),
            "action_err": float(sem(act[:G])), "lcf_density": dens[G],
            "lcf_action": float(act[G])}


def exact(case, seed):
    # about 1e10 segment evaluations a second this way, some 0.5 ms a point
    pts = sum(p for _, _, p in _points(case))
    if _evals(case) > 1.2e11 or pts > 20000 or case["n_loops"] * case["n_ppl"] > 7e7:
        return None
    call, groups = case["call"], case["groups"]
    make = _generated if call == "generate" else _unit_loops
    x, y = (v.double() for v in make(case["n_loops"], case["n_ppl"], seed))
    if call in ("batch", "server"):
        loops, out = _Loops64(x, y), []
        for q in _requests(case, seed):
            w, _ = _per_loop64(loops, q["kind"], q["eB0"], q["lam"], q["rho"], q["T"], q["spin"])
            out.append(list(_statistics(w, groups)))
        return out
    rho, T = _grids(case)
    if call == "disc":
        return _exact_disc(case, x, y, rho, T)
    if call == "action":
        k = np.arange(case["n_T"], 0, -1)
        xs = k / (1.0 + case["T_lo"] / case["T_hi"]) / case["n_T"]
        T = case["T_hi"] * (1.0 / xs - 1.0)
        T[0] = case["T_lo"]
        rho = case["rho_hi"] * (case["n_rho"] / np.arange(case["n_rho"], 0, -1) - 1.0)
    w, S = _per_loop64(_Loops64(x, y), KINDS[case["kind"]], case["eB0"], case["lam"], rho, T,
                       case["spin"])
    if call == "correlation":
        per = w.reshape(w.shape[0], -1)
        d = per - per.mean(0)
        gram = d.t().contiguous() @ d
        norm = torch.sqrt(torch.diagonal(gram))
        perms, which = _perms(case, seed)
        sums = np.empty((groups, per.shape[1]))
        P = per.cpu().numpy()
        for p in range(P.shape[1]):
            sums[:, p] = P[perms[which[p]], p].reshape(groups, -1).sum(1)
        return {"per_loop": P, "corr": (gram / norm[:, None] / norm).cpu().numpy(),
                "group_sums": sums}
    mean, err, sums = _statistics(w, groups)
    if call == "action":
        return {"mean": mean, "err": err, "group_sums": sums,
                "action": _exact_action(case, sums, T, rho)}
    if call == "async":
        return {"mean": mean.reshape(-1), "err": err.reshape(-1), "group_sums": sums.reshape(-1)}
    out = {"mean": mean, "err": err, "group_sums": sums}
    if call == "average_ex":
        scale = (w.abs() * S.clamp_min(1.0)).mean(0)
        out.update(scale=scale.cpu().numpy(), fp_err=None, escalated=None)
    return out
