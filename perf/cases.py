"""Performance cases of the library's public entry points.

Each case is one call, or one short sequence of calls, that a parameter
estimation run makes: single proposals, walker ensembles, large batches in the
FP64 and split forms, the time-banded form, multi-event plans, the ensemble
sampler, the surrogate network's gradient, the exact likelihood and the
start-up stage.  Sizes are those of ``paper_2508_04172_amd.workloads``; where
only the shape of the online stage matters (nodes, basis size, modes,
detectors) the data segment is cut to 8 s so that the start-up stays short.

``exact`` is written here in plain torch / numpy (64 bits) from the paper's
equations; the start-up artefacts it reads (nodes, weights, basis) are inputs
of the online stage.
"""
from __future__ import annotations

import math
from collections import OrderedDict

import numpy as np
import torch

from paper_2508_04172_amd import rbfl
from paper_2508_04172_amd import workloads as wl

FORMS = {"fp64": rbfl.FORM_FP64, "split": rbfl.FORM_SPLIT}
TUNE_FROM = 2048          # batches from here on are autotuned once per handle, as bench.py does


# ----------------------------------------------------------------------------
# the cases
# ----------------------------------------------------------------------------

def _eval(net, modes, nodes, q, degree, n, form="fp64", bands=1):
    return {"kind": "eval", "net": net, "modes": modes, "nodes": nodes, "q": q, "degree": degree, "n": n,
            "form": form, "bands": bands}


def listed():
    cases = [
        # a sampler on the host that asks for one ln L at a time (single detector, (2,2) mode)
        ("one_proposal", _eval("one", 1, 200, 20, 1, 1)),
        # one step of a host-driven ensemble on the three-detector network
        ("walkers", _eval("three", 5, 800, 40, 1, 1021)),
        # the headline batch: 1e6 proposals, three detectors, five modes, plain FP64
        ("batch_fp64", _eval("three", 5, 800, 40, 1, 1_000_000)),
        # the same network in the int8 split form, a quarter of the batch
        ("batch_split", _eval("three", 5, 800, 40, 1, 250_000, "split")),
        # single detector with a cubic tail: many nodes, few outputs
        ("cubic_tail", _eval("one", 1, 1500, 60, 3, 100_003)),
        # third-generation shape: 3000 nodes, 2475 outputs
        ("third_generation", _eval("triangle", 5, 3000, 80, 1, 30_011)),
        # rotating Earth: four time bands, 5100 outputs
        ("banded", _eval("three", 5, 800, 40, 1, 4099, bands=4)),
        # a serving batch of twelve uneven events, about a thousand walkers each, replayed as a graph
        ("multi_event", {"kind": "plan", "events": 12, "walkers": 1000}),
        # ten steps of the GPU-resident ensemble
        ("ensemble_steps", {"kind": "sampler", "net": "three", "modes": 5, "nodes": 800, "q": 40, "walkers": 2048,
                            "steps": 10}),
        # one mini-batch of the surrogate's training: loss and gradients
        ("surrogate_gradient", {"kind": "mlp", "hidden": 256, "out": 1275, "batch": 1024, "grad": True}),
        # exact ln L of a posterior sample (the check of the meshfree one)
        ("exact_lnl", {"kind": "brute", "modes": 5, "seg": 16, "n": 301}),
        # an event arrives: start-up, then its first ensemble
        ("start_up", {"kind": "build", "modes": 3, "nodes": 150, "q": 12, "n": 2000}),
    ]
    return [dict(c, name=name) for name, c in cases]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["eval", "sampler", "mlp", "brute", "build", "plan"], [11, 2, 3, 2, 1, 1])[0]
    if kind == "eval":
        net = rng.choice(["one", "three", "three", "triangle"])
        modes = 1 if net == "one" else rng.randint(1, 5)
        nodes = _log_int(rng, 120, 1500)
        q = min(rng.randint(12, 60), nodes)
        degree = rng.choice([1, 1, 2, 3])
        form = rng.choice(["fp64", "fp64", "fp64", "split"])
        bands = rng.choice([1, 1, 1, rng.randint(2, 4)]) if net == "three" else 1
        n = _log_int(rng, 1, 400_000 // bands)
        c = _eval(net, modes, nodes, q, degree, n, form, bands)
        limit = 1.5e12 if form == "fp64" else 4e11
        c["n"] = max(1, min(n, int(limit / (work(c)["flops"] / n))))
        return c
    if kind == "sampler":
        net = rng.choice(["one", "three"])
        return {"kind": kind, "net": net, "modes": 1 if net == "one" else rng.randint(1, 5),
                "nodes": _log_int(rng, 120, 1000), "q": rng.randint(12, 40), "walkers": 2 * _log_int(rng, 32, 8192),
                "steps": rng.randint(2, 12)}
    if kind == "mlp":
        return {"kind": kind, "hidden": rng.choice([64, 100, 128, 256, 512]), "out": rng.randint(41, 1275),
                "batch": _log_int(rng, 64, 8192), "grad": rng.random() < 0.6}
    if kind == "brute":
        return {"kind": kind, "modes": rng.randint(1, 5), "seg": rng.choice([8, 16]), "n": _log_int(rng, 1, 600)}
    if kind == "build":
        return {"kind": kind, "modes": rng.randint(1, 3), "nodes": rng.randint(60, 200), "q": rng.randint(8, 16),
                "n": _log_int(rng, 100, 4000)}
    return {"kind": kind, "events": rng.randint(2, 12), "walkers": _log_int(rng, 40, 2000)}


# ----------------------------------------------------------------------------
# handles: one per event, kept by a user's program for its whole run
# ----------------------------------------------------------------------------

_HANDLES: OrderedDict = OrderedDict()


def _kept(key, make):
    if key not in _HANDLES:
        while len(_HANDLES) >= 3:
            _HANDLES.popitem(last=False)
        _HANDLES[key] = make()
    _HANDLES.move_to_end(key)
    return _HANDLES[key]


def _config(c):
    base = {"one": wl.CFG1, "three": wl.CFG2, "triangle": wl.CFG2.with_(sites=wl.SITES_TRIANGLE)}[c.get("net", "three")]
    bands = c.get("bands", 1)
    # eps 0: the library picks the shape parameter from the RBF system's condition
    return base.with_(name="perf", seg_len=float(c.get("seg", 8)), modes=wl.ALL_MODES[:c["modes"]],
                      n_nodes=c.get("nodes", 60), q=c.get("q", 8), eps=0.0, poly_degree=c.get("degree", 1),
                      earth_rate=2e-2 if bands > 1 else 0.0, n_bands=bands, tc_span=0.027)


def _handle(c):
    cfg = _config(c)

    def make():
        h = rbfl.Handle.from_config(cfg, wl.white_noise(cfg), wl.injection_extrinsics(cfg))
        return h, torch.from_numpy(h.nodes()).cuda(), torch.from_numpy(h.frame()["semi"].copy()).cuda(), set()

    h, nodes, semi, tuned = _kept((c["kind"], c.get("net"), c["modes"], c["nodes"], c["q"], c.get("degree"),
                                   c.get("bands"), c.get("form")), make)
    return cfg, h, nodes, semi, tuned


def _proposals(cfg, nodes, semi, d_ref, n, gen):
    """[11][n] proposals of a running sampler: intrinsic points scattered about
    the interpolation nodes (the physical part of the ellipsoid; a few fall
    outside it), isotropic sky and orientation (single detector: fixed to one
    sky), uniform phase, arrival time in the window, distance uniform in volume."""
    u = lambda *s: torch.rand(*s, generator=gen, device="cuda", dtype=torch.float64)  # noqa: E731
    x = nodes[torch.randint(nodes.shape[0], (n,), generator=gen, device="cuda")]
    x = x + 0.03 * torch.randn(n, 4, generator=gen, device="cuda", dtype=torch.float64)
    x = x / torch.clamp(x.norm(dim=1, keepdim=True) / 0.999999, min=1.0)
    p = torch.empty(11, n, device="cuda", dtype=torch.float64)
    p[0:4] = (x * semi).T
    if cfg.random_sky:
        p[4] = 2 * math.pi * u(n)
        p[5] = torch.asin(2 * u(n) - 1)
        p[6] = math.pi * u(n)
        p[7] = torch.acos(2 * u(n) - 1)
    else:
        inj = wl.injection_extrinsics(cfg)
        for i in range(4):
            p[4 + i] = float(inj[i])
    p[8] = 2 * math.pi * u(n)
    p[9] = cfg.t_trig + cfg.tc_span * (2 * u(n) - 1)
    p[10] = d_ref * (0.125 + (8.0 - 0.125) * u(n)) ** (1.0 / 3.0)
    return p


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _stream():
    return torch.cuda.current_stream().cuda_stream


def prepare(case, seed):
    return {"eval": _prepare_eval, "plan": _prepare_plan, "sampler": _prepare_sampler, "mlp": _prepare_mlp,
            "brute": _prepare_brute, "build": _prepare_build}[case["kind"]](case, seed)


def _prepare_eval(c, seed):
    cfg, h, nodes, semi, tuned = _handle(c)
    n, form = c["n"], FORMS[c["form"]]
    p = _proposals(cfg, nodes, semi, h.d_ref(), n, _generator(seed))
    if n not in tuned:
        h.prepare(form)
        h.reserve(n)
        if n >= TUNE_FROM:
            if form == rbfl.FORM_SPLIT:
                h.autotune(p.data_ptr(), n, rbfl.FORM_FP64, _stream())
            h.autotune(p.data_ptr(), n, form, _stream())
        tuned.add(n)
    return {"kind": "eval", "h": h, "p": p, "n": n, "form": form,
            "lnl": torch.empty(n, device="cuda", dtype=torch.float64)}


def _prepare_plan(c, seed):
    def make():
        cfgs = wl.ragged_events(c["events"], seg_range=(8.0, 32.0))
        hs = rbfl.Handle.from_configs([(e, wl.white_noise(e), wl.injection_extrinsics(e)) for e in cfgs])
        return cfgs, hs, [torch.from_numpy(h.nodes()).cuda() for h in hs], \
            [torch.from_numpy(h.frame()["semi"].copy()).cuda() for h in hs]

    cfgs, hs, nodes, semi = _kept(("plan", c["events"]), make)
    counts = [c["walkers"] + 7 * e for e in range(c["events"])]
    gen = _generator(seed)
    p = torch.cat([_proposals(cfgs[e], nodes[e], semi[e], hs[e].d_ref(), counts[e], gen)
                   for e in range(c["events"])], dim=1).contiguous()
    lnl = torch.empty(p.shape[1], device="cuda", dtype=torch.float64)
    plan = rbfl.Plan(hs, counts, p.data_ptr(), lnl.data_ptr(), rbfl.PLAN_GRAPH | rbfl.PLAN_AUTOTUNE, _stream())
    return {"kind": "plan", "plan": plan, "p": p, "lnl": lnl}


def _prepare_sampler(c, seed):
    cfg, h, nodes, semi, _ = _handle(c)
    W = c["walkers"]
    p = _proposals(cfg, nodes, semi, h.d_ref(), W, _generator(seed))
    d = h.d_ref()
    s = rbfl.Sampler(h, W, (cfg.t_trig - 0.03, cfg.t_trig + 0.03), (0.4 * d, 2.5 * d), seed=seed + 1,
                     init_ptr=p.data_ptr(), stream=_stream())
    chain = torch.empty(12, c["steps"], W, device="cuda", dtype=torch.float64)
    return {"kind": "sampler", "s": s, "steps": c["steps"], "chain": chain}


def _mlp_inputs(c, seed):
    n_par = rbfl.mlp_param_count(4, c["hidden"], c["out"])
    rng = np.random.default_rng(seed)
    x = wl.uniform_ball(rng, c["batch"]).astype(np.float32)
    t = rng.standard_normal((c["batch"], c["out"])).astype(np.float32)     # standardised targets
    return wl.mlp_normals(n_par, seed), x, t


def _prepare_mlp(c, seed):
    z, x, t = _mlp_inputs(c, seed)
    m = rbfl.Mlp(4, c["hidden"], c["out"], z)
    st = {"kind": "mlp", "m": m, "x": torch.from_numpy(x).cuda(), "t": torch.from_numpy(t).cuda(),
          "batch": c["batch"], "grad": c["grad"]}
    if not c["grad"]:
        st["y"] = torch.empty(c["batch"], c["out"], device="cuda")
    return st


# The exact likelihood runs on the caller's own data and PSD.
_D_REF = 100.0


def _brute_config(c):
    return _config(c).with_(q=8, n_nodes=60)


def _psd(f):
    """The analytic aLIGO-like PSD of the workloads, x = f / 215 Hz."""
    x = np.maximum(f, 1.0) / 215.0
    return 1e-49 * (x ** -4.14 - 5.0 * x ** -2 + 111.0 * (1.0 - x ** 2 + 0.5 * x ** 4) / (1.0 + 0.5 * x ** 2))


def _brute_data(cfg):
    """PSD and coloured noise of every detector (no signal: the noise decides nothing about the cost)."""
    f = np.arange(cfg.n_freq) / cfg.seg_len
    psd = np.repeat(_psd(f)[None, :], cfg.n_det, axis=0)
    w = wl.white_noise(cfg)
    data = np.sqrt(psd * cfg.seg_len / 4.0)[:, :, None] * w
    return np.ascontiguousarray(psd), np.ascontiguousarray(data)


def _brute_handle(c):
    cfg = _brute_config(c)

    def make():
        psd, data = _brute_data(cfg)
        keep = []
        spec = rbfl.spec_from_config(cfg, None, wl.injection_extrinsics(cfg), None, keep)
        spec.psd, spec.data_fd, spec.d_ref = rbfl._dptr(psd), rbfl._dptr(data), _D_REF
        h = rbfl.Handle.build(spec)
        return h, torch.from_numpy(h.nodes()).cuda(), torch.from_numpy(h.frame()["semi"].copy()).cuda(), psd, data

    return (cfg,) + _kept(("brute", c["modes"], c["seg"]), make)


def _prepare_brute(c, seed):
    cfg, h, nodes, semi, _, _ = _brute_handle(c)
    p = _proposals(cfg, nodes, semi, _D_REF, c["n"], _generator(seed))
    return {"kind": "brute", "h": h, "p": p, "n": c["n"],
            "lnl": torch.empty(c["n"], device="cuda", dtype=torch.float64)}


def _prepare_build(c, seed):
    cfg = wl.SMALL_MULTI.with_(modes=wl.ALL_MODES[:c["modes"]], n_nodes=c["nodes"], q=c["q"], eps=0.0,
                               noise_seed=seed, inj_seed=seed)
    keep = []
    spec = rbfl.spec_from_config(cfg, wl.white_noise(cfg), wl.injection_extrinsics(cfg), None, keep)
    return {"kind": "build", "spec": spec, "keep": keep, "qd": wl.queries(cfg, n=c["n"], seed=seed), "cfg": cfg}


# ----------------------------------------------------------------------------
# one pass
# ----------------------------------------------------------------------------

def run(st):
    kind = st["kind"]
    if kind == "eval":
        st["h"].eval(st["p"].data_ptr(), st["n"], st["lnl"].data_ptr(), st["form"], _stream())
        return st["lnl"]
    if kind == "plan":
        st["plan"].launch(_stream())
        return st["lnl"]
    if kind == "sampler":
        st["s"].run(st["steps"], 1, st["chain"].data_ptr(), st["steps"], _stream())
        return st["chain"]
    if kind == "mlp":
        if st["grad"]:
            loss = st["m"].loss_grad(st["x"].data_ptr(), st["t"].data_ptr(), st["batch"], _stream())
            return {"loss": loss, "grad": st["m"].get(1)}
        st["m"].forward(st["x"].data_ptr(), st["batch"], st["y"].data_ptr(), _stream())
        return st["y"]
    if kind == "brute":
        st["h"].brute(st["p"].data_ptr(), st["n"], st["lnl"].data_ptr(), _stream())
        return st["lnl"]
    h = rbfl.Handle.build(st["spec"], _stream())
    p = torch.from_numpy(rbfl.params_soa(h, st["qd"], st["cfg"].t_trig)).cuda()
    lnl = torch.empty(p.shape[1], device="cuda", dtype=torch.float64)
    h.eval(p.data_ptr(), p.shape[1], lnl.data_ptr(), rbfl.FORM_FP64, _stream())
    out = {"lnl": lnl, "singular": h.singular(), "weights": h.weights()}
    h.close()
    return out


# ----------------------------------------------------------------------------
# work of one pass
# ----------------------------------------------------------------------------

def _n_det(c):
    return 1 if c.get("net") == "one" else 3


def _outputs(n_blocks, modes, q):
    return n_blocks * (2 * q * modes + modes * modes)


def _online(n, rows, K, n_blocks, modes, q, T):
    """Bytes and flops of one evaluation of n proposals: parameters in, ln L
    out, weights and the basis (spline-folded: 64 bytes per entry) read once."""
    return (96.0 * n + 8.0 * rows * K + 64.0 * n_blocks * modes * T * q,
            2.0 * n * rows * K + 20.0 * n * rows + 30.0 * n * K)


def work(c):
    kind = c["kind"]
    if kind in ("eval", "sampler"):
        cfg = _config(c)
        blocks = _n_det(c) * c.get("bands", 1)
        rows = c["nodes"] + math.comb(c.get("degree", 1) + 4, 4)
        T = 2 * int(cfg.half_window * cfg.fs) + 1
        K = _outputs(blocks, c["modes"], c["q"])
        n = c["n"] if kind == "eval" else c["walkers"]
        b, f = _online(n, rows, K, blocks, c["modes"], c["q"], T)
        if kind == "sampler":
            b, f = c["steps"] * (b + 96.0 * n), c["steps"] * f
        return {"bytes": b, "flops": f}
    if kind == "plan":
        b = f = 0.0
        for e, cfg in enumerate(wl.ragged_events(c["events"], seg_range=(8.0, 32.0))):
            T = 2 * int(cfg.half_window * cfg.fs) + 1
            be, fe = _online(c["walkers"] + 7 * e, cfg.n_nodes + 5, cfg.n_out, 3, len(cfg.modes), cfg.q, T)
            b, f = b + be, f + fe
        return {"bytes": b, "flops": f}
    if kind == "mlp":
        H, K, B = c["hidden"], c["out"], c["batch"]
        par = rbfl.mlp_param_count(4, H, K)
        fwd = 2.0 * B * (4 * H + H * H + H * K)
        if not c["grad"]:
            return {"bytes": 4.0 * (par + B * (4 + K)), "flops": fwd}
        return {"bytes": 4.0 * (2 * par + B * (4 + K)), "flops": 3.0 * fwd - 2.0 * B * 4 * H}
    if kind == "brute":
        cfg = _config(c)
        J = cfg.n_freq
        # per bin and mode: phase series, one sine and cosine, amplitude (about 80 operations);
        # per bin and detector: the shift and the sums over modes and mode pairs
        per_bin = 80.0 * c["modes"] + 3 * (20.0 + 8.0 * c["modes"] + 8.0 * c["modes"] ** 2)
        return {"bytes": 24.0 * 3 * J + 96.0 * c["n"], "flops": c["n"] * J * per_bin}
    cfg = wl.SMALL_MULTI
    T, N, m = 2 * int(cfg.half_window * cfg.fs) + 1, c["nodes"], c["modes"]
    K = _outputs(3, m, c["q"])
    # windowed DFT of every node, detector and mode; the SVDs; the RBF solve; the first batch
    flops = 8.0 * 3 * m * N * T * cfg.n_freq + 3 * m * 16.0 * N * N * T + 2.0 * N * N * K + 2.0 * c["n"] * N * K
    return {"bytes": 24.0 * 3 * cfg.n_freq + 16.0 * N * m * cfg.n_freq + 8.0 * N * K, "flops": flops}


# ----------------------------------------------------------------------------
# the same results in plain 64-bit torch
# ----------------------------------------------------------------------------

MSUN_S = 4.925490947641267e-06
MPC_S = 3.0856775814913673e22 / 299792458.0
EULER = 0.5772156649015329


def _spline_table():
    """w[s][p]: not-a-knot cubic spline through samples 0..9 at 4 + f as sum_s
    y_s sum_p w[s][p] f^p, from the spline's second derivatives."""
    A = np.zeros((10, 10))
    R = np.zeros((10, 10))
    A[0, :3] = A[9, 7:] = (1.0, -2.0, 1.0)
    for i in range(1, 9):
        A[i, i - 1:i + 2] = (1.0, 4.0, 1.0)
        R[i, i - 1:i + 2] = (6.0, -12.0, 6.0)
    M = np.linalg.solve(A, R)
    e = np.eye(10)
    return np.stack([e[4], e[5] - e[4] - (2 * M[4] + M[5]) / 6.0, M[4] / 2.0, (M[5] - M[4]) / 6.0], axis=1)


def _physical(th, f0, chi_max):
    """Chirp-time coordinates [4][n] to (m1, m2, chi1, chi2, inside)."""
    u = 5.0 * th[1] / (32.0 * math.pi * th[0])
    eta = math.pi / (4.0 * th[1]) * u ** (-2.0 / 3.0)
    mt = u / (math.pi * f0) / MSUN_S
    delta = torch.sqrt(1.0 - 4.0 * eta)
    chi_r = 48.0 * math.pi * th[2] / (113.0 * th[1])
    chi_e = 48.0 * math.pi * th[3] / (113.0 * th[1])
    cs = 113.0 * (chi_e - chi_r) / (76.0 * eta)
    ca = (chi_e - cs) / delta
    ok = (u > 0) & (eta > 0) & (eta <= 0.25) & ((cs + ca).abs() <= chi_max) & ((cs - ca).abs() <= chi_max)
    return 0.5 * mt * (1 + delta), 0.5 * mt * (1 - delta), cs + ca, cs - ca, ok


def _ylm(l, m, iota, phi):
    """Spin -2 harmonic by Wigner's finite sum."""
    f = math.factorial
    c, s = torch.cos(0.5 * iota), torch.sin(0.5 * iota)
    pre = math.sqrt(f(l + m) * f(l - m) * f(l + 2) * f(l - 2))
    d = torch.zeros_like(iota)
    for k in range(2 * l + 1):
        a = (l + 2 - k, k, m - 2 + k, l - m - k)
        if min(a) < 0:
            continue
        w = (-1.0) ** (m - 2 + k) * pre / (f(a[0]) * f(a[1]) * f(a[2]) * f(a[3]))
        d = d + w * c ** (2 * l + 2 - m - 2 * k) * s ** (m - 2 + 2 * k)
    return math.sqrt((2 * l + 1) / (4.0 * math.pi)) * d * torch.exp(1j * m * phi)


def _geometry(site):
    lat, lon, az, opening, radius = site
    east = np.array([-math.sin(lon), math.cos(lon), 0.0])
    north = np.array([-math.sin(lat) * math.cos(lon), -math.sin(lat) * math.sin(lon), math.cos(lat)])
    up = np.array([math.cos(lat) * math.cos(lon), math.cos(lat) * math.sin(lon), math.sin(lat)])
    u = math.cos(az) * north + math.sin(az) * east
    v = math.cos(az + opening) * north + math.sin(az + opening) * east
    return torch.from_numpy(0.5 * (np.outer(u, u) - np.outer(v, v))).cuda(), torch.from_numpy(radius * up).cuda()


def _response(site, alpha, dec, psi):
    """(F+, Fx, delay) with frozen patterns."""
    D, r = _geometry(site)
    z = torch.zeros_like(alpha)
    ea = torch.stack([-torch.sin(alpha), torch.cos(alpha), z])
    ed = torch.stack([-torch.sin(dec) * torch.cos(alpha), -torch.sin(dec) * torch.sin(alpha), torch.cos(dec)])
    X = -torch.cos(psi) * ea + torch.sin(psi) * ed
    Y = torch.sin(psi) * ea + torch.cos(psi) * ed
    DX, DY = D @ X, D @ Y
    n = torch.stack([torch.cos(dec) * torch.cos(alpha), torch.cos(dec) * torch.sin(alpha), torch.sin(dec)])
    return (X * DX - Y * DY).sum(0), (X * DY + Y * DX).sum(0), -(r[:, None] * n).sum(0)


def _amplitude(l, m, fp, fc, iota, phi):
    return 0.5 * ((fp + 1j * fc) * _ylm(l, -m, iota, phi)
                  + (-1.0) ** l * (fp - 1j * fc) * torch.conj(_ylm(l, m, iota, phi)))


def _coordinates(h, p):
    fr = h.frame()
    v = torch.from_numpy(fr["vecs"].copy()).cuda()
    return torch.from_numpy(fr["theta_c"].copy()).cuda()[:, None] + v @ p[0:4]


def _poly(x, degree):
    """Monomials of degree <= `degree` of [n][4] in graded lexicographic order."""
    from itertools import combinations_with_replacement
    cols = [torch.ones_like(x[:, 0])]
    for d in range(1, degree + 1):
        for idx in combinations_with_replacement(range(4), d):
            cols.append(torch.prod(x[:, list(idx)], dim=1))
    return torch.stack(cols, dim=1)


def _meshfree(h, cfg, p):
    """ln L of the meshfree online stage for proposals p [11][n]."""
    s = h.sizes()
    q, T, nm, half = s["q"], s["T"], s["n_modes"], s["half_w"]
    x = (p[0:4] / torch.from_numpy(h.frame()["semi"].copy()).cuda()[:, None]).T.contiguous()
    nodes = torch.from_numpy(h.nodes()).cuda()
    W = torch.from_numpy(h.weights()).cuda()
    basis = torch.from_numpy(h.basis()).cuda()
    tab = torch.from_numpy(_spline_table()).cuda()
    bands = h.bands()
    B = 1 if bands is None else bands[1].shape[0]
    out = torch.empty(p.shape[1], device="cuda", dtype=torch.float64)
    eps2, d_ref = h.eps() ** 2, h.d_ref()
    step = 16384 if W.shape[1] < 3000 else 4096
    for b0 in range(0, p.shape[1], step):
        pc, xc = p[:, b0:b0 + step], x[b0:b0 + step]
        d2 = torch.zeros(xc.shape[0], nodes.shape[0], device="cuda", dtype=torch.float64)
        for d in range(4):
            d2 += (xc[:, d, None] - nodes[None, :, d]) ** 2
        Y = torch.cat([torch.exp(-eps2 * d2), _poly(xc, cfg.poly_degree)], dim=1) @ W
        m1, m2, c1, c2, ok = _physical(_coordinates(h, pc), cfg.f_low, cfg.chi_max)
        ok &= (xc * xc).sum(1) <= 1.0
        r = d_ref / pc[10]
        lnl = torch.zeros_like(r)
        for v in range(cfg.n_det * B):
            k, b = divmod(v, B)
            o = v * (2 * q * nm + nm * nm)
            A = []
            for a, (l, m) in enumerate(cfg.modes):
                t_b = 0.0 if bands is None else float(bands[1][b, a])
                alpha = pc[4] if bands is None else pc[4] - cfg.earth_rate * (pc[9] + t_b - cfg.t_trig)
                fp, fc, dt = _response(cfg.sites[k], alpha, pc[5], pc[6])
                pos = (pc[9] + dt - cfg.t_trig) * cfg.fs + half
                n0 = torch.floor(pos)
                f = (pos - n0)[:, None]
                inside = (n0 >= 4) & (n0 <= T - 6)
                ok &= inside
                n0 = torch.where(inside, n0, 4.0 * torch.ones_like(n0)).long()
                w = tab[None, :, 0] + f * (tab[None, :, 1] + f * (tab[None, :, 2] + f * tab[None, :, 3]))
                co = o + 2 * q * a
                C = torch.complex(Y[:, co:co + 2 * q:2], Y[:, co + 1:co + 2 * q:2])
                bt = torch.zeros_like(C)
                for t in range(10):
                    bt += w[:, t, None] * basis[v, a][n0 + t - 4]
                A.append(_amplitude(l, m, fp, fc, pc[7], pc[8]))
                lnl += r * torch.real(torch.conj(A[a]) * (C * bt).sum(1))
            o += 2 * q * nm
            sg = o + nm
            for a in range(nm):
                lnl -= 0.5 * r * r * A[a].abs() ** 2 * Y[:, o + a]
                for c in range(a + 1, nm):
                    lnl -= r * r * torch.real(torch.conj(A[a]) * A[c] * torch.complex(Y[:, sg], Y[:, sg + 1]))
                    sg += 2
        out[b0:b0 + step] = torch.where(ok, lnl, torch.full_like(lnl, -math.inf))
    return out


def _phase22(f, m1, m2, c1, c2):
    """(2,2) stationary-phase PN phase at template t_c = phi_c = 0 and its frequency derivative."""
    pi, mt = math.pi, m1 + m2
    eta, dl, cs, ca = m1 * m2 / mt ** 2, (m1 - m2) / mt, 0.5 * (c1 + c2), 0.5 * (c1 - c2)
    e2, e3 = eta ** 2, eta ** 3
    p = {0: 1.0, 2: 3715.0 / 756 + 55.0 / 9 * eta,
         3: -16 * pi + 113.0 / 3 * dl * ca + (113.0 / 3 - 76.0 / 3 * eta) * cs,
         4: 15293365.0 / 508032 + 27145.0 / 504 * eta + 3085.0 / 72 * e2 + (-405.0 / 8 + 200 * eta) * ca ** 2
            - 405.0 / 4 * dl * ca * cs + (-405.0 / 8 + 2.5 * eta) * cs ** 2,
         6: 11583231236531.0 / 4694215680 - 640.0 / 3 * pi ** 2 - 6848.0 / 21 * EULER
            + eta * (-15737765635.0 / 3048192 + 2255.0 / 12 * pi ** 2) + 76055.0 / 1728 * e2 - 127825.0 / 1296 * e3
            + pi * (2270.0 / 3 * dl * ca + (2270.0 / 3 - 520 * eta) * cs)
            + (75515.0 / 144 - 8225.0 / 18 * eta) * dl * ca * cs
            + (75515.0 / 288 - 263245.0 / 252 * eta - 480 * e2) * ca ** 2
            + (75515.0 / 288 - 232415.0 / 504 * eta + 1255.0 / 9 * e2) * cs ** 2 - 6848.0 / 21 * math.log(4.0),
         7: pi * (77096675.0 / 254016 + 378515.0 / 1512 * eta - 74045.0 / 756 * e2)
            + dl * ca * (-25150083775.0 / 3048192 + 26804935.0 / 6048 * eta - 1985.0 / 48 * e2)
            + cs * (-25150083775.0 / 3048192 + 10566655595.0 / 762048 * eta - 1042165.0 / 3024 * e2
                    + 5345.0 / 36 * e3)}
    p[5] = (pi * (38645.0 / 756 - 65.0 / 9 * eta) + dl * ca * (-732985.0 / 2268 - 140.0 / 9 * eta)
            + cs * (-732985.0 / 2268 + 24260.0 / 81 * eta + 340.0 / 9 * e2))
    logs = {5: 3.0 * p[5], 6: -6848.0 / 21}               # coefficients of ln v
    v = (pi * mt * MSUN_S * f) ** (1.0 / 3.0)
    lv = torch.log(v)
    S, dS = torch.zeros_like(v), torch.zeros_like(v)      # S(v) and v S'(v)
    for k, c in p.items():
        lg = logs.get(k, 0.0)
        S = S + (c + lg * lv) * v ** k
        dS = dS + (k * (c + lg * lv) + lg) * v ** k
    pre = 3.0 / (128.0 * eta) * v ** -5
    return -0.25 * pi + pre * S, pre * (dS - 5.0 * S) / (3.0 * f)


def _brute(h, cfg, p, psd, data):
    """Exact ln L of proposals p: templates on the frequency grid, direct sums."""
    n_s, df = cfg.n_samples, 1.0 / cfg.seg_len
    j0 = max(1, math.ceil(cfg.f_low * cfg.seg_len - 1e-9))
    j = torch.arange(j0, n_s // 2, device="cuda")
    f = j.double() * df
    w = 4.0 * df / torch.from_numpy(psd).cuda()[:, j0:n_s // 2]
    d = torch.view_as_complex(torch.from_numpy(data).cuda()[:, j0:n_s // 2].contiguous())
    m1, m2, c1, c2, ok = _physical(_coordinates(h, p), cfg.f_low, cfg.chi_max)
    f_ref = torch.tensor([h.f_ref()], device="cuda", dtype=torch.float64)
    resp = [_response(site, p[4], p[5], p[6]) for site in cfg.sites]
    amps = [[_amplitude(l, m, fp, fc, p[7], p[8]) for (l, m) in cfg.modes] for fp, fc, _ in resp]
    out = torch.full((p.shape[1],), -math.inf, device="cuda", dtype=torch.float64)
    for i in range(p.shape[1]):
        if not bool(ok[i]):
            continue
        b = [float(v[i]) for v in (m1, m2, c1, c2)]
        mt, dl = b[0] + b[1], (b[0] - b[1]) / (b[0] + b[1])
        eta = b[0] * b[1] / mt ** 2
        mc = (b[0] * b[1]) ** 0.6 / mt ** 0.2 * MSUN_S
        amp = math.sqrt(5.0 / 24.0) * math.pi ** (-2.0 / 3.0) * mc ** (5.0 / 6.0) / (_D_REF * MPC_S)
        rel = {(2, 2): 1.0, (2, 1): 0.1 * dl, (3, 3): 0.3 * dl, (3, 2): 0.05 * (1 - 3 * eta), (4, 4): 0.1 * (1 - 3 * eta)}
        isco = 1.0 / (2.0 * math.pi * 6.0 ** 1.5 * mt * MSUN_S)
        p0, dp0 = (float(v) for v in _phase22(f_ref, *b))
        hs = []
        for (l, m) in cfg.modes:
            x = 2.0 * f / m
            ph = 0.5 * m * (_phase22(x, *b)[0] - p0 - dp0 * (x - float(f_ref)))
            a = rel[(l, m)] * amp * f ** (-7.0 / 6.0)
            a = torch.where(j < math.ceil(m * isco * cfg.seg_len), a, torch.zeros_like(a))
            hs.append(torch.polar(a, -ph))
        tot = 0.0
        r = _D_REF / float(p[10, i])
        for k in range(cfg.n_det):
            tau = float(p[9, i] + resp[k][2][i])
            ns = round(tau * cfg.fs)
            rem = tau - ns / cfg.fs
            frac = ((j * (ns % n_s)) % n_s).double() / n_s
            shift = torch.polar(torch.ones_like(f), -2.0 * math.pi * (frac + f * rem))
            sig = sum(complex(amps[k][a][i]) * hs[a] for a in range(len(hs)))
            dk = r * float((torch.conj(sig * shift) * d[k] * w[k]).real.sum())
            tot += dk - 0.5 * r * r * float((sig.abs() ** 2 * w[k]).sum())
        out[i] = tot
    return out


def _mlp_exact(c, seed):
    z, x, t = _mlp_inputs(c, seed)
    H, K = c["hidden"], c["out"]
    sizes = [(H * 4, 2.0), (H, None), (H * H, math.sqrt(H)), (H, None), (K * H, math.sqrt(H)), (K, None)]
    parts, o = [], 0
    for n, scale in sizes:
        a = (z[o:o + n] / scale).astype(np.float32) if scale else np.zeros(n, np.float32)
        parts.append(torch.from_numpy(a).cuda().double())
        o += n
    par = torch.cat(parts).requires_grad_(True)
    w = torch.split(par, [n for n, _ in sizes])
    act = torch.nn.functional.silu
    X, T = torch.from_numpy(x).cuda().double(), torch.from_numpy(t).cuda().double()
    y = act(X @ w[0].view(H, 4).T + w[1])
    y = act(y @ w[2].view(H, H).T + w[3]) @ w[4].view(K, H).T + w[5]
    if not c["grad"]:
        return y.detach()
    loss = ((y - T) ** 2).mean()
    loss.backward()
    return {"loss": float(loss), "grad": par.grad.cpu().numpy()}


def exact(case, seed):
    kind = case["kind"]
    if kind == "eval":
        cfg, h, nodes, semi, _ = _handle(case)
        return _meshfree(h, cfg, _proposals(cfg, nodes, semi, h.d_ref(), case["n"], _generator(seed)))
    if kind == "plan":
        st = _prepare_plan(case, seed)
        cfgs, hs, _, _ = _kept(("plan", case["events"]), lambda: None)
        counts = [case["walkers"] + 7 * e for e in range(case["events"])]
        cols = torch.split(st["p"], counts, dim=1)
        return torch.cat([_meshfree(hs[e], cfgs[e], cols[e].contiguous()) for e in range(case["events"])])
    if kind == "mlp":
        return _mlp_exact(case, seed)
    if kind == "brute":
        st = _prepare_brute(case, seed)
        cfg, h, _, _, psd, data = _brute_handle(case)
        return _brute(h, cfg, st["p"], psd, data)
    # a Metropolis chain and a start-up's SVD basis have no value of their own in 64 bits
    return None
