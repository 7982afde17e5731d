"""The work that a user of this framework has it do, as measurable cases.

Five kinds, each through the public entry points of `capi`:

  step       ofm_step: time steps of a state that lies in device memory (custom
             drivers, bench.py); 1-D to 3-D, float and double, both WENO orders,
             all three boundary conditions
  solve      ofm_solve: one sample from its bubbles to its quantities of interest
  batch      ofm_solve_batch: samples of uneven grids solved together, the unit
             of work of the multi-level drivers
  net        ofm_nn_forward (the learned level evaluated over many clouds) and
             ofm_nn_grads (forward and backward of a training step)
  estimator  the OF-MLMC statistics of one iteration of the adaptive loop

A step's state is a cloud in mid-collapse: bubbles with a sub-cell interface,
a pressure ramp with waves and a few collapse peaks, inflow; nothing in it is
constant but the gas fields of pure water.  Solves start from the bubbles, as
the drivers' do; they are in double, because the place of the largest pressure
early in a float solve hangs on its rounding (the float kernels are the step
cases').
"""
import math

import numpy as np
import torch

from paper_1705_04374_amd import capi
from paper_1705_04374_amd.state import alloc_state, current

EOS = dict(gamma1=6.12, pc1=3.43e8, gamma2=1.4, pc2=0.0)
RHO1, RHO2, P_BUBBLE, P_INF = 1000.0, 1.0, 2340.0, 1.0e7
# of the clouds that are solved from their bubbles: off the domain's middle, where
# the largest pressure of the first steps would be a tie of mirrored cells
CENTRE = (0.48, 0.53, 0.49)

# the cloud distributions of the repository's workloads
CLOUDS = {
    "cloud2d": dict(ndim=2, n_bubbles=8, cloud_radius=0.3, r_median=0.03, r_sigma=0.25, r_lo=0.0, r_hi=0.0),
    "cloud50": dict(ndim=3, n_bubbles=50, cloud_radius=0.25, r_median=0.02, r_sigma=0.3, r_lo=0.0, r_hi=0.0),
    "cloud500": dict(ndim=3, n_bubbles=500, cloud_radius=0.3, r_median=0.015, r_sigma=0.1, r_lo=0.012, r_hi=0.018),
}
WORD = {"f32": 4, "f64": 8}
# parameters of the set network, in the library's order
LAYERS = [(128, 4), (128,), (128, 128), (128,), (128, 128), (128,), (5, 128), (5,)]
# operations of the scheme per cell, RK stage and axis (reconstruction of 4 + d
# variables, one face), and those that do not depend on the axes
FLOPS_WENO = {5: 100, 3: 45}


def listed():
    return [
        # the finest level of the four-level hierarchy (64^3 to 512^3): the largest grid a solve takes here
        dict(name="step3d_512_f32", kind="step", ndim=3, n=512, precision="f32", order=5, bc="zero_gradient", steps=1),
        # bench.py's grid
        dict(name="step3d_256_f32", kind="step", ndim=3, n=256, precision="f32", order=5, bc="zero_gradient", steps=2),
        # plain double-precision Monte Carlo, the method's comparator
        dict(name="step3d_192_f64", kind="step", ndim=3, n=192, precision="f64", order=5, bc="zero_gradient", steps=2),
        # a grid that no tile divides, the third-order option and the far-field boundary
        dict(name="step3d_150_f32_weno3", kind="step", ndim=3, n=150, precision="f32", order=3, bc="characteristic",
             steps=2),
        # a coarse level's grid alone: too few tiles to fill the GPU
        dict(name="step3d_48_f32", kind="step", ndim=3, n=48, precision="f32", order=5, bc="zero_gradient", steps=4),
        # the smallest call: a few steps of a 2-D state, all launch latency
        dict(name="step2d_64_f64", kind="step", ndim=2, n=64, precision="f64", order=5, bc="periodic", steps=2),
        # one 2-D sample solved alone (samples one at a time, as plain Monte Carlo does), to two Rayleigh times
        dict(name="solve2d_32_f64", kind="solve", n=32, t_rayleigh=2.0),
        # the two-level 2-D workload: 16 solves at 32^2 and 4 (64^2, 32^2) pairs in one batch
        dict(name="batch2d_64_f64", kind="batch", cloud="cloud2d", n=64, single=16, pairs=4, t_rayleigh=2.0),
        # the three-level 3-D workload's shape, scaled down: single coarse solves and (2n, n) pairs
        dict(name="batch3d_96_f64", kind="batch", cloud="cloud50", n=96, single=8, pairs=2, t_rayleigh=1.0),
        # the learned level over one chunk of clouds of 500 bubbles
        dict(name="net_forward_16384x500", kind="net", train=False, sets=16384, bubbles=500, ragged=False),
        # one training batch (256 clouds), forward and backward
        dict(name="net_grads_256x500", kind="net", train=True, sets=256, bubbles=500, ragged=False),
        # the adaptive loop's statistics at the sample counts of a converged run
        dict(name="estimator_65536", kind="estimator", L=3, M0=65536, ratio=20.0),
    ]


def _spread(rng, lo, hi):
    """An integer in [lo, hi], uniform in its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "solve", "batch", "batch", "net", "net", "net", "estimator"])
    if kind == "step":
        ndim = rng.choice([1, 2, 2, 3, 3, 3, 3, 3])
        precision = rng.choice(["f32", "f32", "f64"])
        top = {1: 4096, 2: 2048, 3: 320 if precision == "f32" else 200}[ndim]
        return dict(kind=kind, ndim=ndim, n=_spread(rng, {1: 64, 2: 24, 3: 20}[ndim], top), precision=precision,
                    order=rng.choice([5, 5, 3]), bc=rng.choice(["zero_gradient", "periodic", "characteristic"]),
                    steps=rng.randint(1, 3))
    if kind == "solve":
        return dict(kind=kind, n=rng.randint(24, 64), t_rayleigh=round(rng.uniform(1.0, 2.0), 2))
    if kind == "batch":
        if rng.random() < 0.5:
            return dict(kind=kind, cloud="cloud2d", n=2 * rng.randint(13, 32), single=rng.randint(2, 16),
                        pairs=rng.randint(1, 4), t_rayleigh=round(rng.uniform(1.0, 2.0), 2))
        return dict(kind=kind, cloud="cloud50", n=2 * rng.randint(24, 48), single=rng.randint(1, 8),
                    pairs=rng.randint(1, 2), t_rayleigh=round(rng.uniform(0.5, 1.0), 2))
    if kind == "net":
        train = rng.random() < 0.5
        return dict(kind=kind, train=train, sets=_spread(rng, 16, 512 if train else 16384),
                    bubbles=_spread(rng, 20, 500), ragged=rng.random() < 0.5)
    return dict(kind=kind, L=rng.randint(1, 4), M0=_spread(rng, 64, 65536), ratio=round(rng.uniform(2.0, 20.0), 1))


_ctx = []


def _context():
    """The program's one library context."""
    if not _ctx:
        _ctx.append(capi.Context(0))
    return _ctx[0]


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------


def _cfg(ndim, n, radius, order=5, bc="zero_gradient", center=(0.5, 0.5, 0.5)):
    return dict(ndim=ndim, n=n, eos=EOS, rho1=RHO1, rho2=RHO2, p_bubble=P_BUBBLE, p_inf=P_INF, cfl=0.3, n_sub=4,
                weno_eps=1e-6, weno_order=order, bc=bc, center=center, cloud_radius=radius,
                ramp_delta=radius / 20.0, ramp_width=radius / 3.0)


def _cloud_of(ndim, n):
    return "cloud2d" if ndim < 3 else "cloud500" if n > 100 else "cloud50"


def _gamma(a2):
    return (1.0 - a2) / (EOS["gamma1"] - 1.0) + a2 / (EOS["gamma2"] - 1.0)


def _pi(a2):
    return ((1.0 - a2) * EOS["gamma1"] * EOS["pc1"] / (EOS["gamma1"] - 1.0)
            + a2 * EOS["gamma2"] * EOS["pc2"] / (EOS["gamma2"] - 1.0))


def _collapse_state(case, seed, dtype):
    """[4 + d, n, .., n] state of the library (energy slot E - Pi(a2)), x last."""
    d, n = case["ndim"], case["n"]
    R = CLOUDS[_cloud_of(d, n)]["cloud_radius"]
    rng = np.random.default_rng([seed, 77, d, n])
    if d == 1:      # a column through a few bubbles
        xs = np.sort(rng.uniform(0.25, 0.75, 6))
        bub = np.stack([xs, 0 * xs, 0 * xs, rng.uniform(0.01, 0.03, 6)], axis=1)
    else:
        bub = _bubbles(_cloud_of(d, n), seed, 0)
    ax = (torch.arange(n, dtype=torch.float64, device="cuda") + 0.5) / n
    shape = (n,) * d

    def along(a, v):        # a coordinate's values along axis a (x = 0, the last dimension)
        s = [1] * d
        s[d - 1 - a] = v.numel()
        return v.reshape(s)

    a2 = torch.zeros(shape, dtype=torch.float64, device="cuda")
    for b in bub:
        r = float(b[3]) * 0.8       # shrunk on average by now
        box = [(max(0, int((b[a] - r) * n) - 2), min(n, int((b[a] + r) * n) + 3)) for a in range(d)]
        view = a2[tuple(slice(*box[a]) for a in range(d - 1, -1, -1))]
        if view.numel():
            r2 = sum(along(a, (ax[box[a][0]:box[a][1]] - float(b[a])) ** 2) for a in range(d))
            torch.maximum(view, ((r - r2.sqrt()) * n + 0.5).clamp(0.0, 1.0), out=view)

    def waves(amp, modes=3):
        f = 0.0
        for _ in range(modes):
            k = rng.integers(-4, 5, size=3)
            ph, w = rng.uniform(0, 2 * math.pi), rng.uniform(0.3, 1.0)
            f = f + w * torch.cos(sum(along(a, 2 * math.pi * int(k[a]) * ax) for a in range(d)) + ph)
        return f * (amp / modes)

    r2 = sum(along(a, (ax - 0.5) ** 2) for a in range(d))
    s = ((r2.sqrt() - 0.8 * R) / (0.5 * R)).clamp(0.0, 1.0)
    p = (2.0e5 + (P_INF - 2.0e5) * (s * s * (3.0 - 2.0 * s))) * (1.0 + waves(0.2))
    for k in range(6):      # collapse peaks, each a quarter lower than the one before
        c = 0.5 + rng.uniform(-0.4, 0.4, size=3) * R
        w = max(0.02, 2.5 / n)
        p = p + 4.0e7 * 0.75 ** k * math.prod(
            (along(a, torch.exp(-((ax - float(c[a])) / w) ** 2)) for a in range(d)), start=1.0)
    del r2, s
    rho1 = RHO1 * (1.0 + waves(0.01))
    rho2 = RHO2 * (2.0 + waves(0.5))
    u = torch.empty((4 + d,) + shape, dtype=dtype, device="cuda")
    r1, g1 = (1.0 - a2) * rho1, a2 * rho2
    u[0], u[1] = r1, g1
    rho = r1 + g1
    et = _gamma(a2) * p
    del r1, g1, rho1, rho2, p
    for m in range(d):
        v = waves(8.0) - 15.0 * along(m, torch.sin(2 * math.pi * (ax - 0.5)))
        u[2 + m] = rho * v
        et = et + 0.5 * rho * v * v
    u[2 + d], u[3 + d] = et, a2
    return u


def _rayleigh(cloud):
    return 0.915 * CLOUDS[cloud]["r_median"] * math.sqrt(RHO1 / (P_INF - P_BUBBLE))


def _bubbles(cloud, seed, index):
    """[n_bubbles, 4] centres and radii of a cloud around CENTRE (radii log-normal, clipped by
    redrawing where the cloud says so; bubbles do not overlap)."""
    c, d = CLOUDS[cloud], CLOUDS[cloud]["ndim"]
    rng = np.random.default_rng([seed, 1, index])
    out = np.zeros((c["n_bubbles"], 4))
    k = 0
    while k < c["n_bubbles"]:
        x = rng.uniform(-1.0, 1.0, d)
        r = c["r_median"] * math.exp(c["r_sigma"] * rng.normal())
        if (x * x).sum() >= 1.0 or (c["r_hi"] > 0.0 and not c["r_lo"] <= r <= c["r_hi"]):
            continue
        x = np.array(CENTRE[:d]) + c["cloud_radius"] * x
        if k and (((out[:k, :d] - x) ** 2).sum(axis=1) < (out[:k, 3] + r) ** 2).any():
            continue
        out[k, :d], out[k, 3] = x, r
        k += 1
    return out


def _members(case, seed):
    """(grid sizes, bubbles) of a batch: single coarse solves, then fine and
    coarse members of the pairs, which share their bubbles."""
    ns, bub = [], []
    for i in range(case["single"] + case["pairs"]):
        b = _bubbles(case["cloud"], seed, i)
        for n in ([case["n"] // 2] if i < case["single"] else [case["n"], case["n"] // 2]):
            ns.append(n)
            bub.append(b)
    return ns, bub


def _net_inputs(case, seed):
    rng = np.random.default_rng([seed, 5, case["sets"]])
    S, B = case["sets"], case["bubbles"]
    sizes = rng.integers(max(1, B // 4), B + 1, S) if case["ragged"] else np.full(S, B)
    off = np.concatenate([[0], np.cumsum(sizes)])
    g = torch.Generator(device="cuda").manual_seed(int(seed) * 1000003 + S)
    x = torch.randn((int(off[-1]), 4), generator=g, device="cuda", dtype=torch.float32)
    # centres uniform in the unit ball, log-radii standard normal
    u = torch.rand((int(off[-1]), 1), generator=g, device="cuda", dtype=torch.float32)
    x[:, :3] *= u.pow(1.0 / 3.0) / x[:, :3].norm(dim=1, keepdim=True).clamp_min(1e-6)
    mean = torch.tensor([1.9e8, 0.5, 0.5, 0.5, 4.0e-4])
    std = torch.tensor([2.5e7, 0.15, 0.15, 0.15, 1.0e-4])
    y = mean.cuda() + std.cuda() * torch.randn((S, 5), generator=g, device="cuda", dtype=torch.float32)
    # weights uniform in +-sqrt(6 / inputs), small biases
    P = torch.cat([(torch.rand(math.prod(s), generator=g, device="cuda") * 2.0 - 1.0)
                   * (math.sqrt(6.0 / s[1]) if len(s) == 2 else 0.1) for s in LAYERS])
    return x, torch.tensor(off, dtype=torch.int32, device="cuda"), y, mean, std, P


def _terms(case, seed):
    """Samples of the estimator's terms: fine and coarse values, status flags."""
    rng = np.random.default_rng([seed, 9, case["L"], case["M0"]])
    out = []
    for l in range(case["L"] + 1):
        M = max(8, int(case["M0"] / case["ratio"] ** l))
        y = rng.lognormal(0.0, 0.3, M)
        qf = 1e8 * 2.0 ** l * (y + 0.1 * rng.normal(size=M))
        qc = 1e8 * 2.0 ** (l - 1) * (y + 0.1 * rng.normal(size=M)) if l else None
        out.append((qf, qc, (rng.random(M) > 0.01).astype(np.int32)))
    return out


def _costs(case):
    return [0.01 * 16.0 ** l * (1.0 + 1.0 / 16.0 if l else 1.0) for l in range(case["L"] + 1)]


def prepare(case, seed):
    kind, ctx = case["kind"], _context()
    if kind == "step":
        d, n = case["ndim"], case["n"]
        cfg = _cfg(d, n, CLOUDS[_cloud_of(d, n)]["cloud_radius"], case["order"], case["bc"])
        st, bufs = alloc_state(cfg, case["precision"])
        bufs[0].copy_(_collapse_state(case, seed, bufs[0].dtype).reshape(bufs[0].shape))
        return dict(case=case, ctx=ctx, spec=capi.make_spec(cfg, case["precision"], n_steps=case["steps"]), st=st,
                    bufs=bufs)
    if kind == "solve":
        cfg = _cfg(2, case["n"], CLOUDS["cloud2d"]["cloud_radius"], center=CENTRE)
        return dict(case=case, ctx=ctx, spec=capi.make_spec(cfg, "f64", t_end=case["t_rayleigh"] * _rayleigh("cloud2d")),
                    bubbles=_bubbles("cloud2d", seed, 0))
    if kind == "batch":
        ns, bub = _members(case, seed)
        c = CLOUDS[case["cloud"]]
        specs = [capi.make_spec(_cfg(c["ndim"], n, c["cloud_radius"], center=CENTRE), "f64",
                                t_end=case["t_rayleigh"] * _rayleigh(case["cloud"])) for n in ns]
        return dict(case=case, ctx=ctx, specs=specs, bubbles=bub)
    if kind == "net":
        x, off, y, mean, std, P = _net_inputs(case, seed)
        net = capi.SetNet(ctx, 1.0 / case["bubbles"], out_mean=mean.tolist(), out_std=std.tolist())
        net.set_params(P)
        return dict(case=case, net=net, x=x, off=off, y=y,
                    out=torch.empty((case["sets"], 5), dtype=torch.float32, device="cuda"),
                    grads=torch.empty(net.param_count(), dtype=torch.float32, device="cuda"),
                    loss=torch.empty(1, dtype=torch.float32, device="cuda"))
    dev = lambda v: None if v is None else torch.tensor(v, device="cuda")  # noqa: E731
    L = case["L"]
    f64 = lambda *s: torch.empty(s, dtype=torch.float64, device="cuda")  # noqa: E731
    return dict(case=case, ctx=ctx, terms=[tuple(map(dev, t)) for t in _terms(case, seed)],
                W=torch.tensor(_costs(case), dtype=torch.float64, device="cuda"), mom=f64(L + 1, 6), alpha=f64(L + 1),
                sig=f64(L + 1), eps2=f64(1), E=f64(1), M=torch.empty(L + 1, dtype=torch.int64, device="cuda"),
                have=torch.full((L + 1,), 2, dtype=torch.int64, device="cuda"),
                flag=torch.empty(2, dtype=torch.int32, device="cuda"))


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------


def run(s):
    kind = s["case"]["kind"]
    if kind == "step":
        q, dts = capi.ofm_step(s["ctx"], s["spec"], s["st"], s["case"]["steps"])
        return dict(u=current(s["st"], s["bufs"]), qoi=q, dts=dts.tolist())
    if kind == "solve":
        return capi.ofm_solve(s["ctx"], s["spec"], s["bubbles"])
    if kind == "batch":
        qois = capi.ofm_solve_batch(s["ctx"], s["specs"], s["bubbles"])
        return {k: np.array([q[k] for q in qois]) for k in qois[0]}
    if kind == "net":
        if s["case"]["train"]:
            s["net"].grads(s["x"], s["off"], s["y"], s["grads"], s["loss"])
            return dict(loss=s["loss"], grads=s["grads"])
        s["net"].forward(s["x"], s["off"], s["out"])
        return s["out"]
    ctx, L = s["ctx"], s["case"]["L"]
    for l, (qf, qc, ok) in enumerate(s["terms"]):
        capi.ofm_mlmc_moments(ctx, qf, qc, ok, s["mom"][l])
    capi.ofm_ofmlmc_coefficients(ctx, L, s["mom"], s["W"], s["alpha"], s["flag"][:1])
    capi.ofm_ofmlmc_errors(ctx, L, s["mom"], s["alpha"], s["sig"], s["eps2"])
    capi.ofm_ofmlmc_estimate(ctx, L, s["mom"], s["alpha"], s["E"])
    capi.ofm_ofmlmc_optimal_M(ctx, L, s["sig"], s["W"], s["have"], capi.OFM_MODE_TOLERANCE, 1.0e6, s["M"], s["flag"][1:])
    return dict(mom=s["mom"], alpha=s["alpha"], sig=s["sig"], eps2=s["eps2"], E=s["E"], M=s["M"], flag=s["flag"])


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------


def _flow_work(ndim, cells, steps, order, word):
    nv = 4 + ndim
    per_stage = ndim * (nv * FLOPS_WENO[order] + 28 + 110) + 119
    return 2.0 * nv * cells * word, 3.0 * per_stage * cells * steps


def _steps(cloud, n, rayleigh):
    """Time steps to an end time: the sound speed of water at rest is close to the fastest signal."""
    return math.ceil(rayleigh * _rayleigh(cloud) * n / 0.3 * math.sqrt(EOS["gamma1"] * (P_INF + EOS["pc1"]) / RHO1))


def work(case):
    kind = case["kind"]
    if kind == "step":
        b, f = _flow_work(case["ndim"], case["n"] ** case["ndim"], case["steps"], case["order"], WORD[case["precision"]])
    elif kind == "solve":
        _, f = _flow_work(2, case["n"] ** 2, _steps("cloud2d", case["n"], case["t_rayleigh"]), 5, 8)
        b = 32.0 * CLOUDS["cloud2d"]["n_bubbles"] + 128.0
    elif kind == "batch":
        c = CLOUDS[case["cloud"]]
        k = case["single"] + case["pairs"]
        f = sum(m * _flow_work(c["ndim"], n ** c["ndim"], _steps(case["cloud"], n, case["t_rayleigh"]), 5, 8)[1]
                for m, n in ((k, case["n"] // 2), (case["pairs"], case["n"])))
        b = k * 32.0 * c["n_bubbles"] + 128.0 * (k + case["pairs"])
    elif kind == "net":
        mean = case["bubbles"] * (0.625 if case["ragged"] else 1.0)
        rows, sets = case["sets"] * mean, case["sets"]
        f = rows * 2.0 * (4 * 128 + 128 * 128) + sets * 2.0 * (128 * 128 + 5 * 128)
        b = rows * 16.0 + sets * 24.0 + 34309 * 4.0
        if case["train"]:
            f, b = 3.0 * f, b + sets * 20.0 + 34309 * 4.0
    else:
        M = sum(max(8, int(case["M0"] / case["ratio"] ** l)) for l in range(case["L"] + 1))
        f, b = 14.0 * M, 20.0 * M
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------------------
# the same in 64 bits, by plain torch and numpy
# ---------------------------------------------------------------------------


def _weno(s, order):
    """Right-edge value of the centre cell of five shifted fields."""
    a, b, c, d, e = s
    if order == 3:
        w0, w1 = (1.0 / 3.0) / (1e-6 + (c - b) ** 2) ** 2, (2.0 / 3.0) / (1e-6 + (d - c) ** 2) ** 2
        return (w0 * (3.0 * c - b) / 2.0 + w1 * (c + d) / 2.0) / (w0 + w1)
    w0 = 0.1 / (1e-6 + 13.0 / 12.0 * (a - 2 * b + c) ** 2 + 0.25 * (a - 4 * b + 3 * c) ** 2) ** 2
    w1 = 0.6 / (1e-6 + 13.0 / 12.0 * (b - 2 * c + d) ** 2 + 0.25 * (b - d) ** 2) ** 2
    w2 = 0.3 / (1e-6 + 13.0 / 12.0 * (c - 2 * d + e) ** 2 + 0.25 * (3 * c - 4 * d + e) ** 2) ** 2
    return (w0 * (2 * a - 7 * b + 11 * c) + w1 * (-b + 5 * c + 2 * d) + w2 * (2 * c + 5 * d - e)) / (6.0 * (w0 + w1 + w2))


def _edges(W, dim, n, d, order):
    """Left- and right-edge states of cells -1..n along `dim` from primitives
    padded by three cells, with the positivity rules."""
    cut = lambda v, k: v.narrow(dim - 1, k, n + 2)  # noqa: E731
    lo, hi = [], []
    for v in range(4 + d):
        s = [cut(W[v], k) for k in range(5)]
        l, h, c = _weno(s[::-1], order), _weno(s, order), s[2]
        if v < 2 or v == 3 + d:
            mid = (6.0 * c - l - h) / 4.0 if order == 3 else (12.0 * c - l - h) / 10.0
            if v < 2:
                big = torch.full_like(c, RHO1 if v == 0 else RHO2)
                for q in (s[1:4] if order == 3 else s):
                    big = torch.maximum(big, q.abs())
                low, top = -1e-12 * big, math.inf
            else:
                low, top = -1e-12, 1.0 + 1e-12
            keep = (l >= low) & (h >= low) & (mid >= low) & (l <= top) & (h <= top) & (mid <= top)
            l, h = torch.where(keep, l, c), torch.where(keep, h, c)
        lo.append(l)
        hi.append(h)
    ok = True
    for w in (lo, hi):
        ok = ok & ((_gamma(w[3 + d]) + 1.0) * w[2 + d] + _pi(w[3 + d]) > 0.0)
    c = [cut(W[v], 2) for v in range(4 + d)]
    return [torch.where(ok, x, y) for x, y in zip(lo, c)], [torch.where(ok, x, y) for x, y in zip(hi, c)]


def _hllc(wl, wr, ax, d):
    def side(w):
        rho, a2, p = w[0] + w[1], w[3 + d], w[2 + d]
        G, P = _gamma(a2), _pi(a2)
        E = G * p + P + 0.5 * rho * sum(w[2 + m] ** 2 for m in range(d))
        return rho, w[2 + ax], p, E, torch.sqrt(((G + 1.0) * p + P) / (G * rho))
    (rl, ul, pl, El, cl), (rr, ur, pr, Er, cr) = side(wl), side(wr)
    sl, sr = torch.minimum(ul - cl, ur - cr), torch.maximum(ul + cl, ur + cr)
    ml, mr = rl * (sl - ul), rr * (sr - ur)
    ss = (pr - pl + ml * ul - mr * ur) / (ml - mr)
    left = (sl >= 0) | (ss >= 0)
    up = (left & (sl >= 0)) | (~left & (sr <= 0))
    pick = lambda x, y: torch.where(left, x, y)  # noqa: E731
    w = [pick(x, y) for x, y in zip(wl, wr)]
    rho, un, p, E, S = pick(rl, rr), pick(ul, ur), pick(pl, pr), pick(El, Er), pick(sl, sr)
    chi = torch.where(up, torch.ones_like(S), (S - un) / (S - ss))
    v = torch.where(up, un, ss)
    uf = chi * v
    f = [w[0] * uf, w[1] * uf]
    f += [rho * w[2 + m] * uf if m != ax else rho * uf * v + p + rho * (S - un) * (v - un) for m in range(d)]
    return f + [uf * (E + p + rho * S * (v - un)), w[3 + d] * uf], uf


def _prim(u, d):
    rho = u[0] + u[1]
    vel = [u[2 + m] / rho for m in range(d)]
    ke = 0.5 * rho * sum(v * v for v in vel)
    a2 = u[3 + d]
    return [u[0], u[1]] + vel + [(u[2 + d] - ke) / _gamma(a2), a2]


def _rate(u, d, n, order, bc):
    """L(U), with the energy slot E - Pi(a2)."""
    W = _prim(u, d)
    L, div = [torch.zeros_like(W[0]) for _ in range(4 + d)], torch.zeros_like(W[0])
    for ax in range(d):
        dim = d - 1 - ax
        end = lambda v, low: v.narrow(dim, 0, 1) if low else v.narrow(dim, n - 1, 1)  # noqa: E731
        if bc == "periodic":
            Wp = [torch.cat([v.narrow(dim, n - 3, 3), v, v.narrow(dim, 0, 3)], dim) for v in W]
        else:
            ghost = []
            for low in (True, False):
                g = [end(v, low) for v in W]
                if bc == "characteristic":
                    rho, p, a2, sg = g[0] + g[1], g[2 + d], g[3 + d], -1.0 if low else 1.0
                    z2 = rho * ((_gamma(a2) + 1.0) * p + _pi(a2)) / _gamma(a2)
                    Z = torch.sqrt(z2.clamp_min(1e-300))
                    delta = 0.5 * (0.25 / n) * (P_INF - (p - sg * Z * g[2 + ax]))
                    g = list(g)
                    g[2 + d] = torch.where(z2 > 0, p + delta, p)
                    g[2 + ax] = torch.where(z2 > 0, g[2 + ax] - sg * delta / Z, g[2 + ax])
                ghost.append(g)
            Wp = [torch.cat([a] * 3 + [v] + [b] * 3, dim) for a, v, b in zip(ghost[0], W, ghost[1])]
        lo, hi = _edges(Wp, dim + 1, n, d, order)
        del Wp
        f, uf = _hllc([v.narrow(dim, 0, n + 1) for v in hi], [v.narrow(dim, 1, n + 1) for v in lo], ax, d)
        del lo, hi
        dif = lambda v: (v.narrow(dim, 0, n) - v.narrow(dim, 1, n)) * n  # noqa: E731
        for v in range(4 + d):
            L[v] += dif(f[v])
        f[2 + d] = None
        div -= dif(uf)
    # the energy flux above is that of E with its part Pi(a2_K) u_f; L of
    # E - Pi(a2) is L(E) - dPi L(a2), Pi linear in a2
    a2, p = W[3 + d], W[2 + d]
    a = a2.clamp(0.0, 1.0)
    c1, c2 = EOS["gamma1"] * (p + EOS["pc1"]), EOS["gamma2"] * (p + EOS["pc2"])
    den = (1.0 - a) * c2 + a * c1
    K = (1.0 - a) * a * (c1 - c2) / torch.where(den == 0, torch.ones_like(den), den)
    K = torch.where((a == 0) | (a == 1) | (den == 0), torch.zeros_like(K), torch.minimum(torch.maximum(K, -a), 1.0 - a))
    L[3 + d] += (a2 + K) * div
    L[2 + d] -= (_pi(torch.ones_like(a2)) - _pi(torch.zeros_like(a2))) * L[3 + d]
    return L


def _level(u, d, n, R, centre):
    """Largest signal speed and the quantities of interest of one time level."""
    W = _prim(u, d)
    a2, p = W[3 + d], W[2 + d]
    c = torch.sqrt(((_gamma(a2) + 1.0) * p + _pi(a2)) / (_gamma(a2) * (W[0] + W[1])))
    s = max(float((W[2 + m].abs() + c).max()) for m in range(d))
    ax = (torch.arange(n, dtype=torch.float64, device=p.device) + 0.5) / n
    r2 = 0.0
    for a in range(d):
        shape = [1] * d
        shape[d - 1 - a] = n
        r2 = r2 + ((ax - centre[a]) ** 2).reshape(shape)
    ball, gas = r2 <= max(R / 40.0, 1.01 * 0.5 / n * math.sqrt(d)) ** 2, r2 <= R * R
    at = int(p.reshape(-1).argmax())
    return s, dict(p=float(p.reshape(-1)[at]), at=at, sensor=float(p[ball].mean()) if bool(ball.any()) else 0.0,
                   gas=float(a2[gas].mean()) if bool(gas.any()) else 0.0, c=float(c.max()))


def _advance(u, d, n, R, order, bc, steps, t_end=math.inf, centre=(0.5, 0.5, 0.5)):
    """Steps of the scheme on u (a list of fields) and the quantities of interest."""
    s, l = _level(u, d, n, R, centre)
    q = dict(p_max=l["p"], argmax=l["at"], t_at_max=0.0, p_sensor=l["sensor"], t_p_sensor=0.0, gas_min=l["gas"],
             t_gas_min=0.0, c_max=l["c"], status=0)
    t, k, dts = 0.0, 0, []
    while k < steps and t < t_end:
        dt = 0.3 / n / s
        last = dt >= t_end - t
        dt = t_end - t if last else dt
        dts.append(dt)
        du = None
        for A, B in ((0.0, 0.25), (-17.0 / 32.0, 8.0 / 9.0), (-32.0 / 27.0, 0.75)):
            L = _rate(u, d, n, order, bc)
            du = [dt * x if du is None else dt * x + A * y for x, y in zip(L, du or L)]
            u = [x + B * y for x, y in zip(u, du)]
        t, k = t_end if last else t + dt, k + 1
        s, l = _level(u, d, n, R, centre)
        if l["p"] > q["p_max"]:
            q.update(p_max=l["p"], argmax=l["at"], t_at_max=t)
        if l["sensor"] > q["p_sensor"]:
            q.update(p_sensor=l["sensor"], t_p_sensor=t)
        if l["gas"] < q["gas_min"]:
            q.update(gas_min=l["gas"], t_gas_min=t)
        q["c_max"] = max(q["c_max"], l["c"])
    at = q["argmax"]
    x = [((at // n ** a) % n + 0.5) / n if a < d else 0.0 for a in range(3)]
    q.update(t=t, steps=k, x=tuple(x), peak_distance=math.sqrt(sum((v - c) ** 2 for v, c in zip(x[:d], centre))))
    return u, q, dts


def _initial(bub, n, R):
    """The 2-D state of a cloud at rest (fields of 64 bits, energy slot E - Pi)."""
    ax = (torch.arange(4 * n, dtype=torch.float64, device="cuda") + 0.5) / (4 * n)
    inside = torch.zeros((4 * n, 4 * n), dtype=torch.bool, device="cuda")
    for b in bub:
        inside |= (ax[None, :] - float(b[0])) ** 2 + (ax[:, None] - float(b[1])) ** 2 < float(b[3]) ** 2
    a2 = inside.double().reshape(n, 4, n, 4).mean(dim=(1, 3))
    c = (torch.arange(n, dtype=torch.float64, device="cuda") + 0.5) / n
    s = ((torch.sqrt((c[None, :] - CENTRE[0]) ** 2 + (c[:, None] - CENTRE[1]) ** 2) - R - R / 20.0) / (R / 3.0)).clamp(0.0, 1.0)
    p = P_BUBBLE + (P_INF - P_BUBBLE) * (s * s * (3.0 - 2.0 * s))
    z = torch.zeros_like(a2)
    return [(1.0 - a2) * RHO1, a2 * RHO2, z, z.clone(), _gamma(a2) * p, a2]


def _network(case, seed):
    x, off, y, mean, std, P = _net_inputs(case, seed)
    P = P.double().requires_grad_(case["train"])
    W, at = [], 0
    for s in LAYERS:
        W.append(P[at:at + math.prod(s)].reshape(s))
        at += math.prod(s)
    idx = torch.repeat_interleave(torch.arange(case["sets"], device="cuda"), (off[1:] - off[:-1]).long())
    pool = torch.zeros((case["sets"], 128), dtype=torch.float64, device="cuda")
    for r in range(0, x.shape[0], 1 << 20):     # a chunk of rows at a time
        h = torch.relu(torch.relu(x[r:r + (1 << 20)].double() @ W[0].T + W[1]) @ W[2].T + W[3])
        pool = pool.index_add(0, idx[r:r + (1 << 20)], h)
    out = torch.relu(pool / case["bubbles"] @ W[4].T + W[5]) @ W[6].T + W[7]
    mean, std = mean.cuda().double(), std.cuda().double()
    if not case["train"]:
        return out * std + mean
    loss = ((out - (y.double() - mean) / std) ** 2).mean()
    g, = torch.autograd.grad(loss, P)
    return dict(loss=loss.detach().reshape(1), grads=g)


def _statistics(case, seed):
    L, W = case["L"], np.array(_costs(case))
    mom = np.zeros((L + 1, 6))
    for l, (qf, qc, ok) in enumerate(_terms(case, seed)):
        k = ok != 0
        f, c = qf[k], qc[k] if l else np.zeros(int(k.sum()))
        M = f.size
        mom[l] = (M, f.mean(), c.mean(), ((f - f.mean()) ** 2).sum() / (M - 1), ((c - c.mean()) ** 2).sum() / (M - 1),
                  ((f - f.mean()) * (c - c.mean())).sum() / (M - 1))
    A, b = np.zeros((L, L)), np.zeros(L)
    for k in range(L):
        A[k, k] = mom[k, 3] * W[k] + mom[k + 1, 4] * W[k + 1]
        if k:
            A[k, k - 1] = -mom[k, 5] * W[k]
        if k + 1 < L:
            A[k, k + 1] = -mom[k + 1, 5] * W[k + 1]
    b[L - 1] = mom[L, 5] * W[L]
    al = np.append(np.linalg.solve(A, b), 1.0)
    prev = np.append(0.0, al[:-1])
    sig = al ** 2 * mom[:, 3] + prev ** 2 * mom[:, 4] - 2.0 * al * prev * mom[:, 5]
    E = (al * mom[:, 1] - prev * mom[:, 2]).sum()
    return dict(mom=mom, alpha=al, sig=sig, eps2=np.array([(sig / mom[:, 0]).sum()]), E=np.array([E]), M=None, flag=None)


def exact(case, seed):
    kind = case["kind"]
    if kind == "step":
        d, n = case["ndim"], case["n"]
        u = _collapse_state(case, seed, torch.float32 if case["precision"] == "f32" else torch.float64).double()
        with torch.no_grad():
            u, q, dts = _advance(list(u), d, n, CLOUDS[_cloud_of(d, n)]["cloud_radius"], case["order"], case["bc"],
                                 case["steps"])
        return dict(u=torch.stack([v.reshape(-1) for v in u]), qoi=q, dts=dts)
    if kind == "solve":
        R = CLOUDS["cloud2d"]["cloud_radius"]
        return _advance(_initial(_bubbles("cloud2d", seed, 0), case["n"], R), 2, case["n"], R, 5, "zero_gradient", 1 << 30,
                        case["t_rayleigh"] * _rayleigh("cloud2d"), CENTRE)[1]
    if kind == "batch":
        return None     # a few hundred steps of every member: minutes
    if kind == "net":
        return _network(case, seed)
    return _statistics(case, seed)
