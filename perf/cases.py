"""The framework's work as a user's program has it done, for measurement.

Every case goes through the public entry points (``Net``, ``Mlp``,
``estimate``) on inputs made on the GPU from a seed.  The networks follow the
shapes this repository's tests and benchmark use: two-dimensional ones
(uniform in 1 mm x 1 mm, a pair closer than 150 um connected with probability
0.3, a tenth of the vertices driven at 5 Hz), three-dimensional ones (65,536
vertices per mm^3, connection probability falling as exp(-r / 100 um), about
100 in-edges per vertex, state noise) and the paper's standardized test
networks (10 to 1,000 vertices in a 500 um square).

The range of each kind (``draw`` draws from it, up to the listed case's size):

kind        sizes                                  what it stands for
----------  -------------------------------------  ----------------------------
single      32..256 vertices                       one small network, all steps in one launch
ensemble    8..128 networks of 64..4,096 vertices  many uneven networks, observed through calcium
default     1,000..8,192 vertices                  one network built with no options
fused       4,096..65,536 vertices                 one network, pull delivery fused with the update
push        8,192..262,144 vertices                one network, spikes pushed along out-edges
plastic     2,048..16,384 vertices                 one network whose weights learn (STDP)
izhikevich  4..20 networks of 10..1,000 vertices   the paper's test networks, FP64 state
hh          4..20 networks of 10..1,000 vertices   the same with Hodgkin-Huxley vertices
forward     64..65,536 rows                        scoring candidate pairs
train       1,024..65,536 rows                     an epoch of scorer training
scorer      64..1,024 vertices, 20..600 frames     pair features of one observed network, scored
fit         32..512 vertices, 20..120 frames       the simulation-based fit of one network
"""
from __future__ import annotations

import math
from dataclasses import dataclass
from typing import Optional

import numpy as np
import torch

import paper_0908_3934_amd as gn
from paper_0908_3934_amd import estimate

DT_MS, TAU_C_MS = 0.1, 500.0
FRAME_NUM, FRAME_DEN = 3, 1000          # 30 frames per second at dt = 0.1 ms
RADIUS_UM, DENSITY = 150.0, 65536.0     # 2D connection radius; 3D vertices per mm^3
LAMBDA_UM, CUT_UM = 100.0, 2000.0


def listed():
    return [
        # the smallest call: a 256-vertex network, 1,000 steps, its raster kept
        dict(name="single 256", kind="single", n=256, steps=1000),
        # a batch of uneven networks simulated and observed together, as when training data is made
        dict(name="ensemble 128", kind="ensemble", nets=128, n_max=4096, steps=1000),
        # what a first program gets: no options, a mid-sized network
        dict(name="default 8192", kind="default", n=8192, steps=256),
        # the 65,536-vertex network of the tests, pull delivery
        dict(name="fused 65536", kind="fused", n=65536, steps=128),
        # a large network with 20 % inhibitory sources, push delivery
        dict(name="push 262144", kind="push", n=262144, steps=256),
        # learning weights read back after a stretch of steps
        dict(name="plastic 16384", kind="plastic", n=16384, steps=256),
        # the paper's benchmark: its test networks side by side, alpha synapses
        dict(name="izhikevich test set", kind="izhikevich", nets=20, n_max=1000, psc=2, steps=500),
        dict(name="hh test set", kind="hh", nets=20, n_max=1000, psc=2, steps=500),
        # one 1,024-vertex network's candidate pairs scored
        dict(name="forward 65536", kind="forward", rows=65536),
        # one epoch at the batch size EdgeScorer.fit uses
        dict(name="train 65536", kind="train", rows=65536, batch=16384),
        # features and scores of one 1,024-vertex network observed for 20 s
        dict(name="scorer 1024", kind="scorer", n=1024, frames=600),
        # the fit of one network observed for 4 s
        dict(name="fit 512", kind="fit", n=512, frames=120, realisations=8, sweeps=2),
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice([c["kind"] for c in listed()])
    if kind == "single":
        return dict(kind=kind, n=size(32, 256), steps=size(200, 1000))
    if kind == "ensemble":
        return dict(kind=kind, nets=size(8, 128), n_max=size(256, 4096), steps=size(200, 1000))
    if kind == "default":
        return dict(kind=kind, n=size(1000, 8192), steps=size(64, 256))
    if kind == "fused":
        return dict(kind=kind, n=size(4096, 65536), steps=size(32, 128))
    if kind == "push":
        return dict(kind=kind, n=size(8192, 262144), steps=size(64, 256))
    if kind == "plastic":
        return dict(kind=kind, n=size(2048, 16384), steps=size(64, 256))
    if kind in ("izhikevich", "hh"):
        return dict(kind=kind, nets=size(4, 20), n_max=size(30, 1000), psc=rng.randrange(3), steps=size(100, 500))
    if kind == "forward":
        return dict(kind=kind, rows=size(64, 65536))
    if kind == "train":
        rows = size(1024, 65536)
        return dict(kind=kind, rows=rows, batch=min(rows, size(1024, 16384)))
    if kind == "scorer":
        return dict(kind=kind, n=size(64, 1024), frames=size(20, 600))
    return dict(kind="fit", n=size(32, 512), frames=size(20, 120), realisations=rng.choice([4, 8]),
                sweeps=rng.randrange(3))


# ---------------------------------------------------------------------------
# Networks
# ---------------------------------------------------------------------------
@dataclass
class Spec:
    """One network, with the attributes ``Net`` and ``estimate`` read."""
    pos_um: np.ndarray
    src: np.ndarray
    dst: np.ndarray
    weight: np.ndarray
    seed: int
    delay_steps: Optional[np.ndarray] = None
    dt_ms: float = DT_MS
    v_um_per_ms: float = 100.0
    tau_ms: float = 20.0
    v_rest: float = 0.0
    v_reset: float = 0.0
    v_th: float = 1.0
    n_ref: int = 20
    drive_rate_hz: Optional[np.ndarray] = None
    drive_amp: float = 1.5
    i_ext: Optional[np.ndarray] = None
    noise_sigma: float = 0.0
    v0: Optional[np.ndarray] = None
    tau_c_ms: float = TAU_C_MS
    frame_num: int = FRAME_NUM
    frame_den: int = FRAME_DEN
    plastic: int = 0
    stdp_alpha: float = float(np.float32(0.005))
    stdp_beta: float = float(np.float32(0.1))
    # Izhikevich (regular spiking) and Hodgkin-Huxley (squid axon) constants
    model: int = 0
    psc: int = 0
    iz_C: float = 100.0
    iz_k: float = float(np.float32(0.7))
    iz_vr: float = -60.0
    iz_vt: float = -40.0
    iz_a: float = float(np.float32(0.03))
    iz_b: float = -2.0
    iz_d: float = 100.0
    psc_rate: float = float(np.float32(0.2))
    w0_iz: Optional[np.ndarray] = None
    hh_C: float = 1.0
    hh_gna: float = 120.0
    hh_gk: float = 36.0
    hh_gl: float = float(np.float32(0.3))
    hh_ena: float = 50.0
    hh_ek: float = -77.0
    hh_el: float = float(np.float32(-54.387))

    @property
    def n(self):
        return int(self.pos_um.shape[0])

    @property
    def dims(self):
        return int(self.pos_um.shape[1])

    @property
    def n_edges(self):
        return int(self.src.shape[0])


def gpu_rng(seed, tag=0):
    return torch.Generator(device="cuda").manual_seed((int(seed) * 1000003 + tag) & 0x7FFFFFFFFFFFFFFF)


def uniform(g, *shape, dtype=torch.float64):
    return torch.rand(*shape, generator=g, device="cuda", dtype=dtype)


def fp16_weights(g, m, scale):
    return ((0.5 + uniform(g, m)) * scale).half().float()


def morton(cells, bits):
    """Z-order codes of integer cell coordinates [n][dims]."""
    dims = cells.shape[1]
    code = torch.zeros(cells.shape[0], dtype=torch.int64, device=cells.device)
    for b in range(bits):
        for k in range(dims):
            code |= ((cells[:, k] >> b) & 1) << (b * dims + k)
    return code


def host(t, dtype):
    return np.ascontiguousarray(t.cpu().numpy().astype(dtype, copy=False))


def square_net(n, seed, w0=0.05, noise=0.0, geometry=None):
    """Two-dimensional network of n vertices, vertices numbered in Z order;
    `geometry`: another seed for where they lie and what is connected, so
    that every seed of a size has as many pairs."""
    g = gpu_rng(seed if geometry is None else geometry, 1)
    pos = uniform(g, n, 2) * 1000.0
    pos = pos[torch.argsort(morton((pos * 1.024).long(), 10))]
    d2 = (pos[:, None, :] - pos[None, :, :]).square().sum(-1)
    edge = (d2 < RADIUS_UM ** 2) & (uniform(g, n, n, dtype=torch.float32) < 0.3)
    edge.fill_diagonal_(False)
    dst, src = torch.nonzero(edge, as_tuple=True)     # by target, then source
    g = gpu_rng(seed, 11)
    driven = torch.randperm(n, generator=g, device="cuda") < max(1, n // 10)
    return Spec(pos_um=host(pos, np.float64), src=host(src, np.int32), dst=host(dst, np.int32),
                weight=host(fp16_weights(g, src.numel(), w0), np.float32), seed=seed + 1,
                drive_rate_hz=host(driven.float() * 5.0, np.float32), noise_sigma=noise)


def cube_net(n, seed, w0=0.005, noise=0.05, inhibitory=0.0, geometry=None):
    """Three-dimensional network of n vertices on a jittered grid: every
    target draws displacements with density r^2 exp(-r / 100 um) and takes
    the vertex of the grid cell each one ends in (`geometry`: as above)."""
    g = gpu_rng(seed if geometry is None else geometry, 2)
    side = 1000.0 * (n / DENSITY) ** (1.0 / 3.0)
    k = int(math.ceil(n ** (1.0 / 3.0) - 1e-9))
    h = side / k
    cell = torch.randperm(k ** 3, generator=g, device="cuda")[:n]
    xyz = torch.stack([cell // (k * k), cell // k % k, cell % k], 1)
    order = torch.argsort(morton(xyz, 8))
    cell, xyz = cell[order], xyz[order]
    pos = (xyz + uniform(g, n, 3)) * h
    vertex_of = torch.full((k ** 3,), -1, dtype=torch.int64, device="cuda")
    vertex_of[cell] = torch.arange(n, device="cuda")
    tries = 164 if inhibitory == 0.0 else 117           # in-edges per vertex of an unbounded space
    keys = []
    for lo in range(0, n, 32768):
        p = pos[lo:lo + 32768]
        m = p.shape[0]
        r = -LAMBDA_UM * torch.log(uniform(g, m, tries, 3).clamp_min(1e-12)).sum(-1)
        v = torch.randn(m, tries, 3, generator=g, device="cuda", dtype=torch.float64)
        q = p[:, None, :] + v * (r / v.norm(dim=-1))[..., None]
        c = torch.floor(q / h).long()
        inside = ((c >= 0) & (c < k)).all(-1) & (r < CUT_UM)
        c = c.clamp(0, k - 1)
        i = vertex_of[(c[..., 0] * k + c[..., 1]) * k + c[..., 2]]
        j = torch.arange(lo, lo + m, device="cuda")[:, None].expand_as(i)
        ok = inside & (i >= 0) & (i != j)
        keys.append(torch.unique(j[ok] * n + i[ok]))
    key = torch.cat(keys)
    src, dst = key % n, key // n
    g = gpu_rng(seed, 12)
    w = fp16_weights(g, src.numel(), w0)
    if inhibitory > 0.0:
        w = torch.where((uniform(g, n) < inhibitory)[src], -w, w)
    return Spec(pos_um=host(pos, np.float64), src=host(src, np.int32), dst=host(dst, np.int32),
                weight=host(w, np.float32), seed=seed + 2, noise_sigma=noise)


def test_net(n, seed, model, psc, cls, dense):
    """One of the paper's standardized networks: vertices numbered from the
    centre outwards, edges from the k nearest vertices or from a random tenth
    or fifth of all ordered pairs, tonically driven."""
    g = gpu_rng(seed, 3)
    pos = uniform(g, n, 2) * 500.0
    pos = pos[torch.argsort((pos - 250.0).square().sum(-1))]
    if cls == "lattice":
        d2 = (pos[:, None, :] - pos[None, :, :]).square().sum(-1)
        d2.fill_diagonal_(math.inf)
        k = min(n - 1, 8 if dense else 3)
        src = torch.sort(torch.topk(d2, k, largest=False).indices, 1).values.reshape(-1)
        dst = torch.arange(n, device="cuda").repeat_interleave(k)
    else:
        edge = uniform(g, n, n) < (0.2 if dense else 0.1)
        edge.fill_diagonal_(False)
        dst, src = torch.nonzero(edge, as_tuple=True)
    indeg = max(1.0, src.numel() / n)
    kw = dict(pos_um=host(pos, np.float64), src=host(src, np.int32), dst=host(dst, np.int32), seed=seed + 3,
              n_ref=0, model=model, psc=psc)
    scale = min(1.0, 8.0 / indeg)
    if model == 1:
        w = fp16_weights(g, src.numel(), (4.0, 100.0, 25.0)[psc] * scale)
        return Spec(weight=host(w, np.float32), dt_ms=1.0, v_th=35.0, v_reset=-50.0, drive_amp=3000.0,
                    noise_sigma=1.0, v0=host(-60.0 + 20.0 * uniform(g, n), np.float32),
                    i_ext=np.full(n, 60.0, np.float32), frame_den=FRAME_DEN // 10, **kw)
    w = fp16_weights(g, src.numel(), (4.0, 15.0, 6.0)[psc] * scale)
    return Spec(weight=host(w, np.float32), dt_ms=0.03, v_th=0.0, drive_amp=1000.0, noise_sigma=0.1,
                v0=host(-65.0 + 4.0 * uniform(g, n), np.float32), i_ext=np.full(n, 8.0, np.float32),
                psc_rate=0.5, frame_den=FRAME_DEN * 10 // 3, **kw)


def ensemble_sizes(case):
    """Log-uniform sizes, the largest always there; the same for every seed."""
    r = np.random.RandomState(7)
    s = np.exp(r.uniform(math.log(64), math.log(case["n_max"]), case["nets"])).round().astype(int)
    s[0] = case["n_max"]
    return [int(x) for x in s]


def test_set_sizes(case):
    """(n, class, dense) of each network: the paper's sizes up to n_max, then its classes and densities."""
    sizes = [s for s in (10, 30, 100, 300, 1000) if s < case["n_max"]] + [case["n_max"]]
    kinds = [(n, cls, dense) for cls in ("random", "lattice") for dense in (True, False) for n in reversed(sizes)]
    return [kinds[k % len(kinds)] for k in range(case["nets"])]


# ---------------------------------------------------------------------------
# Observations and scorer inputs
# ---------------------------------------------------------------------------
def observation(n, frames, seed):
    """Fluorescence of a 1 mm^2 network of n vertices firing at about 10 Hz
    with a common modulation, seen at 30 Hz with SNR 5."""
    spec = square_net(n, seed, w0=0.065, noise=0.05, geometry=n)
    g = gpu_rng(seed, 4)
    steps = FRAME_DEN / FRAME_NUM
    rho = (1.0 - DT_MS / TAU_C_MS) ** steps
    rate = 10.0 * (0.5 + uniform(g, 1, n)) * (0.5 + uniform(g, frames, 1))
    spikes = torch.poisson(rate * (steps * DT_MS * 1e-3), generator=g)
    c = torch.empty(frames, n, dtype=torch.float64, device="cuda")
    now = torch.full((n,), 0.02 * TAU_C_MS * DT_MS, dtype=torch.float64, device="cuda")
    for f in range(frames):
        c[f] = now * (1.0 + rho) / 2.0 + 0.5 * DT_MS * spikes[f]
        now = now * rho + DT_MS * spikes[f]
    gamma = float(np.float32(estimate.observation_gamma(spec)))
    F = (c + gamma * torch.randn(frames, n, generator=g, device="cuda", dtype=torch.float64)).float().contiguous()
    pairs, dist, labels = estimate.candidate_pairs(spec)
    return estimate.Observed(spec=spec, F=F, pairs=torch.tensor(pairs, device="cuda"),
                             dist=torch.tensor(dist, device="cuda"), labels=labels, gain=1.0, offset=0.0, gamma=gamma)


def mlp_params(seed):
    p = gn.Mlp.init_params(int(seed) % (1 << 31))
    r = np.random.RandomState(int(seed) % (1 << 31))
    for lo in (64 * 256, 64 * 256 + 256 + 256 * 256):        # the two bias vectors of a trained net are not zero
        p[lo:lo + 256] = r.uniform(-0.1, 0.1, 256)
    return p


def feature_rows(rows, seed):
    """Features as the extractor leaves them (columns of unlike scale, the
    last five zero), their standardisation, and labels that depend on them."""
    g = gpu_rng(seed, 5)
    scale = 10.0 ** (uniform(g, 64) * 3.0 - 2.0)
    shift = uniform(g, 64) * scale
    z = torch.randn(rows, 64, generator=g, device="cuda", dtype=torch.float64)
    z[:, 1:59] = 0.8 * z[:, 1:59] + 0.6 * z[:, :58]          # neighbouring lags are correlated
    x = z * scale + shift
    x[:, 59:] = 0.0
    inv = 1.0 / scale
    inv[59:] = 0.0
    y = (torch.sigmoid(z[:, :8].sum(1)) > uniform(g, rows)).float()
    return x.float().contiguous(), y, host(shift.float(), np.float32), host(inv.float(), np.float32)


# ---------------------------------------------------------------------------
# What a user's program holds, and one pass
# ---------------------------------------------------------------------------
def prepare(case, seed):
    kind, seed = case["kind"], int(seed)
    if kind == "single":
        net = gn.Net(square_net(case["n"], seed), flags=gn.NET_BUILD_SINGLE_LAUNCH)
        net.step(1000)                                        # past the silent start
    elif kind == "ensemble":
        specs = [square_net(n, seed * 131 + m) for m, n in enumerate(ensemble_sizes(case))]
        frames = estimate.frames_in(case["steps"], FRAME_NUM, FRAME_DEN)
        net = gn.Net(specs, frame_capacity=max(frames, 1), flags=gn.NET_BUILD_AUTOTUNE)
        return dict(case=case, net=net, frames=frames, gamma=estimate.observation_gamma(specs[0]))
    elif kind == "default":
        net = gn.Net(cube_net(case["n"], seed))
        net.step(400)
    elif kind == "fused":
        net = gn.Net(cube_net(case["n"], seed), flags=gn.NET_BUILD_FUSED_STEP)
        net.step(400)
    elif kind == "push":
        net = gn.Net(cube_net(case["n"], seed, inhibitory=0.2), flags=gn.NET_BUILD_PUSH)
        net.step(400)
    elif kind == "plastic":
        spec = cube_net(case["n"], seed, geometry=case["n"])
        spec.plastic = 1
        net = gn.Net(spec)
        net.step(400)
    elif kind in ("izhikevich", "hh"):
        specs = [test_net(n, seed * 131 + m, 1 if kind == "izhikevich" else 2, case["psc"], cls, dense)
                 for m, (n, cls, dense) in enumerate(test_set_sizes(case))]
        net = gn.Net(specs, flags=gn.NET_BUILD_AUTOTUNE)
        net.step(200)
    elif kind in ("forward", "train"):
        x, y, shift, scale = feature_rows(case["rows"], seed)
        mlp = gn.Mlp(mlp_params(seed))
        mlp.set_input_norm(shift, scale)
        return dict(case=case, mlp=mlp, x=x, y=y)
    elif kind == "scorer":
        scorer = estimate.EdgeScorer(seed % (1 << 31))
        return dict(case=case, o=observation(case["n"], case["frames"], seed), scorer=scorer)
    else:
        return dict(case=case, o=observation(case["n"], case["frames"], seed))
    return dict(case=case, net=net)


def run(state):
    case, kind = state["case"], state["case"]["kind"]
    if kind == "ensemble":
        net = state["net"]
        net.step(case["steps"])
        return {"v": net.observe(gn.NET_OBS_V), "calcium": net.observe(gn.NET_OBS_CALCIUM),
                "fluor": net.observe(gn.NET_OBS_FLUOR, frames=state["frames"], gamma=state["gamma"])}
    if kind == "plastic":
        net = state["net"]
        r = net.step(case["steps"], raster=True)
        return {"raster": r["raster"], "v": net.observe(gn.NET_OBS_V), "weights": net.observe(gn.NET_OBS_WEIGHTS)}
    if kind == "forward":
        return state["mlp"].forward(state["x"])
    if kind == "train":
        losses = torch.zeros(-(-case["rows"] // case["batch"]), device="cuda")
        state["mlp"].train_epoch(state["x"], state["y"], case["batch"], 1e-3, seed=5, epoch=0, losses=losses)
        return {"losses": losses, "params": state["mlp"].get_params()}
    if kind == "scorer":
        feats = estimate.features(state["o"])
        return {"features": feats, "scores": state["scorer"].score(state["o"], feats)}
    if kind == "fit":
        return estimate.simfit(state["o"], 0.065, realisations=case["realisations"], sweeps=case["sweeps"])
    net = state["net"]
    r = net.step(case["steps"], raster=True)
    return {"raster": r["raster"], "v": net.observe(gn.NET_OBS_V)}


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------
MLP_FLOPS = 2 * (64 * 256 + 256 * 256 + 256)


def square_pairs(n):
    """Ordered pairs closer than 150 um in the 1 mm square, on average."""
    r = RADIUS_UM / 1000.0
    return n * (n - 1) * (math.pi * r * r - 8.0 / 3.0 * r ** 3 + 0.5 * r ** 4)


def work(case):
    """Vertex state in and out once (V and the spike age; FP64 state of the
    other models), the records, and the vertex arithmetic: about 12
    operations a step for LIF, 100 more for a noise draw, 60 and 250 for the
    FP64 models.  Edges are touched only where a spike arrives: at 5 Hz an
    edge's weight, target and delay (8 B) every 2,000 steps."""
    kind = case["kind"]
    if kind in ("single", "default", "fused", "push", "plastic"):
        n, t = case["n"], case["steps"]
        arrivals = n * t * (0.0005 * 100 if kind != "single" else 0.0005 * 5)
        edges = n * 100 * 4 if kind == "plastic" else 0       # every weight read out
        return {"bytes": n * 12 + n * t / 8 + 4 * n + 8 * arrivals + edges,
                "flops": n * t * (12 if kind == "single" else 112) + 2 * arrivals}
    if kind == "ensemble":
        n, t = sum(ensemble_sizes(case)), case["steps"]
        return {"bytes": n * (12 + 32 + 4 * (2 + t * FRAME_NUM // FRAME_DEN)), "flops": n * t * 24}
    if kind in ("izhikevich", "hh"):
        n, t = sum(s[0] for s in test_set_sizes(case)), case["steps"]
        return {"bytes": n * (2 * 8 * (4 if kind == "izhikevich" else 7) + t / 8 + 4),
                "flops": n * t * (160 if kind == "izhikevich" else 350)}
    if kind == "forward":
        return {"bytes": case["rows"] * 260, "flops": case["rows"] * MLP_FLOPS}
    if kind == "train":
        steps = -(-case["rows"] // case["batch"])
        return {"bytes": case["rows"] * 260 + 82689 * 4 * 6 * steps, "flops": 3 * case["rows"] * MLP_FLOPS}
    p = square_pairs(case["n"])
    if kind == "scorer":
        return {"bytes": 4 * case["n"] * case["frames"] + p * (12 + 256 + 4),
                "flops": p * (2 * 53 * case["frames"] + MLP_FLOPS)}
    # every hypothesis (pair or target) stepped for every realisation and sweep, six operations a step
    steps = case["frames"] * FRAME_DEN / FRAME_NUM
    return {"bytes": 4 * case["n"] * case["frames"] + p * 12,
            "flops": (case["sweeps"] + 1) * (p + case["n"]) * case["realisations"] * steps * 6}


# ---------------------------------------------------------------------------
# The same in 64 bits, in plain torch
# ---------------------------------------------------------------------------
def philox(c0, c1, c2, c3, k0, k1):
    """Philox4x32-10 on int64 tensors holding 32-bit words."""
    m = 0xFFFFFFFF

    def mulhilo(a, b):
        lo = (a & 0xFFFF) * b                                  # 48 bits each: no overflow of int64
        hi = (a >> 16) * b
        s = lo + ((hi & 0xFFFF) << 16)
        return ((hi >> 16) + (s >> 32)) & m, s & m

    x = [c0, c1, c2, c3]
    for _ in range(10):
        h0, l0 = mulhilo(x[0], 0xD2511F53)
        h1, l1 = mulhilo(x[2], 0xCD9E8D57)
        x = [h1 ^ x[1] ^ k0, l1, h0 ^ x[3] ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & m, (k1 + 0xBB67AE85) & m
    return x


def exact_forward(p, x):
    p = torch.as_tensor(p, device="cuda").double()
    w1, b1, w2, b2, w3, b3 = torch.split(p, [64 * 256, 256, 256 * 256, 256, 256, 1])
    h1 = torch.relu(x @ w1.view(64, 256) + b1)
    return torch.relu(h1 @ w2.view(256, 256) + b2) @ w3 + b3


def exact_train(case, seed):
    """Adam on the mean BCE of consecutive batches of the keyed permutation
    (a four-round Feistel network over Philox with cycle walking)."""
    x, y, shift, scale = feature_rows(case["rows"], seed)
    x = (x.double() - torch.as_tensor(shift, device="cuda").double()) * torch.as_tensor(scale, device="cuda").double()
    n, bits = case["rows"], 1
    while (1 << bits) < n:
        bits += 1
    h = (bits + 1) // 2
    i = torch.arange(n, device="cuda")
    todo = torch.ones(n, dtype=torch.bool, device="cuda")
    while bool(todo.any()):
        left, right = i >> h, i & ((1 << h) - 1)
        for r in range(4):
            z = torch.zeros_like(right)
            f = philox(right, z + r, z, z + 0x53485546, 5, 0)[0]
            left, right = right, (left ^ f) & ((1 << h) - 1)
        i = torch.where(todo, (left << h) | right, i)
        todo = i >= n
    p = torch.as_tensor(mlp_params(seed), device="cuda").double()
    m, v, losses = torch.zeros_like(p), torch.zeros_like(p), []
    for k, lo in enumerate(range(0, n, case["batch"])):
        at = i[lo:lo + case["batch"]]
        q = p.clone().requires_grad_(True)
        loss = torch.nn.functional.binary_cross_entropy_with_logits(exact_forward(q, x[at]), y[at].double())
        g, = torch.autograd.grad(loss, q)
        losses.append(loss.detach())
        m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
        p = p - 1e-3 * (m / (1 - 0.9 ** (k + 1))) / ((v / (1 - 0.999 ** (k + 1))).sqrt() + 1e-8)
    return {"losses": torch.stack(losses), "params": p.cpu().numpy()}


def exact_scorer(case, seed):
    o = observation(case["n"], case["frames"], seed)
    s, nf = o.spec, case["frames"]
    F = o.F.double().t().contiguous()
    rho = (1.0 - DT_MS / TAU_C_MS) ** (FRAME_DEN / FRAME_NUM)

    def standardise(a):
        a = a - a.mean(1, keepdim=True)
        var = a.square().mean(1, keepdim=True)
        return a * torch.where(var > 1e-12, var.clamp_min(1e-300).rsqrt(), torch.zeros_like(var))

    e = torch.zeros_like(F)
    e[:, :-1] = (F[:, 1:] - rho * F[:, :-1]).clamp_min(0.0)
    en, zn = standardise(e), standardise(F)
    rn = standardise(en - en.mean(0, keepdim=True))
    dc = torch.zeros_like(F)
    t = torch.arange(-(-nf * FRAME_DEN // FRAME_NUM), device="cuda")
    thr = [math.floor(float(r) * (DT_MS * 1e-3) * 4294967296.0) for r in s.drive_rate_hz]
    zero = torch.zeros_like(t)
    for j, th in enumerate(thr):
        if th > 0:
            hit = philox(zero + j, t, zero, zero, s.seed & 0xFFFFFFFF, s.seed >> 32)[0] < th
            dc[j] = torch.bincount(t[hit] * FRAME_NUM // FRAME_DEN, minlength=nf)[:nf].double()
    npulse = dc.sum(1)
    pairs, out = o.pairs.long(), []
    for lo in range(0, pairs.shape[0], 4096):
        i, j = pairs[lo:lo + 4096, 0], pairs[lo:lo + 4096, 1]

        def lag(a, b, L):
            a, b = (a[:, :nf - L], b[:, L:]) if L >= 0 else (a[:, -L:], b[:, :nf + L])
            return (a * b).sum(1) / max(a.shape[1], 1)

        def response(a, count, b, L):
            return (a[:, :nf - L] * b[:, L:]).sum(1) / count.clamp_min(1.0)

        ei, ej, zi, zj, ri, rj, di, dj = en[i], en[j], zn[i], zn[j], rn[i], rn[j], dc[i], dc[j]
        c = [lag(ei, ej, L) for L in range(-8, 9)] + [lag(zi, zj, L) for L in range(-2, 3)]
        c += [response(di, npulse[i], ej, L) for L in range(6)] + [response(dj, npulse[j], ei, L) for L in range(4)]
        c += [torch.log1p(npulse[i]), torch.log1p(npulse[j]), e.mean(1)[i], e.mean(1)[j]]
        sd = (F - F.mean(1, keepdim=True)).square().mean(1).sqrt()
        c += [sd[i], sd[j], o.dist[lo:lo + 4096].double() / 150.0]
        c += [lag(ri, rj, L) for L in range(4)] + [lag(ei, zj, L) for L in range(8)] + [lag(zi, ej, L) for L in range(8)]
        c += [torch.zeros_like(c[0])] * 5
        out.append(torch.stack(c, 1))
    feats = torch.cat(out) if out else torch.zeros(0, 64, dtype=torch.float64, device="cuda")
    return {"features": feats, "scores": exact_forward(gn.Mlp.init_params(seed % (1 << 31)), feats)}


def exact(case, seed):
    kind = case["kind"]
    if kind == "forward":
        x, _, shift, scale = feature_rows(case["rows"], int(seed))
        x = (x.double() - torch.as_tensor(shift, device="cuda").double()) * torch.as_tensor(scale, device="cuda").double()
        return exact_forward(mlp_params(seed), x)
    if kind == "train":
        return exact_train(case, int(seed))
    if kind == "scorer":
        return exact_scorer(case, int(seed))
    # Simulations and the fit step thresholded units: one rounding that moves a spike changes all that
    # follows, so a 64-bit run is another trajectory; their rasters are whole numbers and stay equal.
    return None
