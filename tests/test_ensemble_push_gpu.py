"""Single-launch kernel at the edges of its shapes: against the per-step
kernels, whose arithmetic is the same (tolerance 0), over calls that end
within a block of steps, are too short for noise drawn ahead, or cross the
buffer it is drawn into, with records and from the state left by them; and
against the FP64 oracle's delivered sums."""
import numpy as np
import pytest

import oracle
import synth
from tests import fixtures as fx
from tests.test_parity_gpu import check_parity

pytestmark = pytest.mark.gpu

CALLS = (1, 7, 40, 3, 1049)      # ends off the 32-step blocks; below 16 steps; past 1,024 steps


def _lif(n, k, sigma, delays=None):
    """n vertices at random, up to 12 in-edges each, a fifth of them driven,
    vertex 0 firing every ~23 steps."""
    rng = np.random.default_rng(1000 * n + k)
    e = 12 * n if n > 1 else 0
    src, dst = rng.integers(0, n, e).astype(np.int32), rng.integers(0, n, e).astype(np.int32)
    _, first = np.unique(src.astype(np.int64) * n + dst, return_index=True)
    src, dst = src[first], dst[first]
    src, dst = src[src != dst], dst[src != dst]
    d = rng.choice(np.array(delays or [1, 2, 5, 12]), src.size).astype(np.uint8)
    i_ext = np.zeros(n, np.float32)
    i_ext[0] = 0.5
    rate = np.where(rng.random(n) < 0.2, 150.0, 0.0).astype(np.float32)
    return synth.NetSpec(name="n%d" % n, pos_um=rng.uniform(0, 500, (n, 2)), src=src, dst=dst,
                         weight=synth.round_fp16(rng.uniform(0.1, 0.4, src.size)), delay_steps=d, drive_rate_hz=rate,
                         i_ext=i_ext, noise_sigma=sigma, seed=17 + k)


def _wide_weights():
    """Rows of 2^-24 and rows of 4096: no unit holds both in 31 bits."""
    s = _lif(70, 5, 0.05)
    s.weight = np.where(s.dst % 2 == 0, 2.0 ** -24, 4096.0).astype(np.float32)
    return s


def _models(n, k, hh):
    make = fx.hodgkin_huxley_tiny if hh else fx.izhikevich_tiny
    a, b, c = make(5, k % 3, 3), make(6, (k + 1) % 3, 4, sigma=0.0), make(7, 0, 5)
    big = _lif(n, k, 0.0)
    big = (synth.hodgkin_huxley if hh else synth.izhikevich)(big, psc=k % 3)
    big.i_ext = None
    return [a, b, c, big]


CASES = {
    "lif edges of a wave": lambda: [_lif(n, 0, s) for n in (1, 63, 64, 65) for s in (0.0, 0.05)],
    "lif two groups a wave": lambda: [_lif(1025, 1, 0.05), _lif(2048, 2, 0.0)],
    "lif four groups a wave": lambda: [_lif(2049, 1, 0.0), _lif(70, 2, 0.05)],
    "lif eight groups a wave": lambda: [_lif(4097, 1, 0.05), _lif(8192, 2, 0.0, [1, 2, 3])],
    "several windows": lambda: [_lif(3, 1, 0.05, [1, 254, 255]), _lif(700, 2, 0.05, [1, 60, 128, 255]),
                                _lif(3000, 3, 0.0, [1, 9, 31, 70])],
    "sums of floats": lambda: [_wide_weights(), _lif(130, 2, 0.0)],
    "one network": lambda: [_lif(300, 3, 0.0)],
    "izhikevich": lambda: _models(513, 1, False),
    "izhikevich four groups a wave": lambda: _models(1100, 2, False),
    "hodgkin-huxley": lambda: _models(513, 2, True),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_single_launch_equals_per_step(case):
    import torch
    import paper_0908_3934_amd as gn
    specs = CASES[case]()
    print(case, [len(s.pos_um) for s in specs], flush=True)
    one = gn.NET_BUILD_SINGLE_LAUNCH if len(specs) == 1 else 0
    nets = [gn.Net(specs, flags=one | extra, frame_capacity=64)
            for extra in (0, gn.NET_BUILD_REORDER, gn.NET_BUILD_GRAPH)] + [gn.Net(specs, flags=gn.NET_BUILD_PER_STEP, frame_capacity=64)]
    assert all(x.info()["ensemble_blocks"] == len(specs) for x in nets[:3]) and nets[3].info()["ensemble_blocks"] == 0
    spikes = 0
    for c, T in enumerate(CALLS):
        outs = [x.step(T, raster=True, v=True, inp=True) if c != 2 else x.step(T) for x in nets]   # (call 2: no records)
        torch.cuda.synchronize()
        for out in outs[:3] if c != 2 else []:
            for key in ("raster", "v", "input"):
                assert torch.equal(out[key], outs[3][key]), (c, key)
        if c != 2:
            spikes += int(gn.unpack_raster(outs[3]["raster"], nets[3].n_total).sum())
    assert spikes > 20
    done = nets[3].info()["frames_done"]
    for what, kw in [(gn.NET_OBS_CALCIUM, {})] + ([(gn.NET_OBS_FRAMES, {"frames": done})] if done else []):
        ref = nets[3].observe(what, **kw).cpu().double()
        for x in nets[:3]:
            got = x.observe(what, **kw).cpu().double()
            # FP64 recursion by blocks of up to 32 steps instead of single steps: a few ulp of 2^-53
            # per step and factor, read out in FP32 at least
            assert float((got - ref).abs().max()) <= 2.0 ** -23 * max(1.0, float(ref.abs().max())), what
    for x in nets:
        x.close()


@pytest.mark.parametrize("case", ["sums of floats", "several windows"])
def test_single_launch_sums_are_the_oracles(case):
    import torch
    import paper_0908_3934_amd as gn
    specs, T = CASES[case](), 300
    net = gn.Net(specs)
    out = net.step(T, raster=True, v=True, inp=True)
    torch.cuda.synchronize()
    r = gn.unpack_raster(out["raster"], net.n_total)
    v, inp = out["v"].cpu().numpy().astype(np.float64), out["input"].cpu().numpy().astype(np.float64)
    offs = net.node_offsets()
    for k, s in enumerate(specs):
        sl = slice(offs[k], offs[k + 1])
        if case == "sums of floats" and k == 0:
            # (V after sums of 4096s is not within the parity bar's absolute 1e-4: delivered sums alone)
            o = oracle.OracleNet(s).step(T, v=False, inp=True)
            rows = np.nonzero((r[:, sl] != o["raster"]).any(1))[0]
            upto = rows[0] + 1 if rows.size else T
            assert upto > 20 and np.array_equal(inp[:upto, sl], o["input"][:upto])
        else:
            check_parity({"raster": r[:, sl], "v": v[:, sl], "input": inp[:, sl]}, oracle.OracleNet(s).step(T, v=True, inp=True))
    net.close()
