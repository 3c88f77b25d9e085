"""One network resident on the chip for the steps of a call against the
per-step kernels, whose arithmetic is the same (tolerance 0): workgroups with
few and with no vertices to spare, arrivals inside and beyond the LDS window,
steps in which more vertices fire than a published word holds, and calls that
pass between the two paths."""
import numpy as np
import pytest

import oracle
import synth
from tests.test_ensemble_push_gpu import _lif
from tests.test_parity_gpu import check_parity

pytestmark = pytest.mark.gpu

# resident; per step; too short to rebuild the arrivals; rebuilt; resident, with no records; the same with
CALLS = (200, 3, 40, 130, 8, 300)


def _burst(n, k):
    """Every vertex fires every ~23 steps, in step at first."""
    s = _lif(n, k, 0.0)
    s.i_ext = np.full(n, 0.5, np.float32)
    return s


CASES = {
    "one vertex": lambda: _lif(1, 0, 0.0),
    "two workgroups": lambda: _lif(257, 1, 0.05),
    "partial word": lambda: _lif(1000, 2, 0.05),
    "late arrivals": lambda: _lif(1500, 3, 0.05, [1, 149, 150, 151, 152, 254, 255]),
    "bursts": lambda: _burst(700, 4),
    "wider workgroups": lambda: _lif(70000, 5, 0.05, [1, 3, 120, 121, 255]),
    "full width": lambda: _lif(200001, 6, 0.0, [1, 31, 32, 33, 200]),
}


@pytest.mark.parametrize("flag", ["default", "FUSED_STEP", "PUSH", "REORDER"])
@pytest.mark.parametrize("case", list(CASES))
def test_resident_equals_per_step(case, flag):
    import torch
    import paper_0908_3934_amd as gn
    spec = CASES[case]()
    print(case, flag, spec.src.size, flush=True)
    a = gn.Net(spec, flags=0 if flag == "default" else getattr(gn, "NET_BUILD_" + flag), frame_capacity=8)
    b = gn.Net(spec, flags=gn.NET_BUILD_PER_STEP, frame_capacity=8)
    spikes = 0
    for c, T in enumerate(CALLS):
        if c == 4:
            a.step(T)
            b.step(T)
            continue
        x, y = a.step(T, raster=True, v=True, inp=True), b.step(T, raster=True, v=True, inp=True)
        torch.cuda.synchronize()
        for key in ("raster", "v", "input"):
            assert torch.equal(x[key], y[key]), (c, key)
        spikes += int(gn.unpack_raster(y["raster"], b.n_total).sum())
    assert spikes > 5
    assert a.info()["frames_done"] == b.info()["frames_done"] == 2
    for what, kw in ((gn.NET_OBS_CALCIUM, {}), (gn.NET_OBS_FRAMES, {"frames": 2}), (gn.NET_OBS_REF, {})):
        p, q = a.observe(what, **kw), b.observe(what, **kw)
        torch.cuda.synchronize()
        assert torch.equal(p, q), what
    a.close()
    b.close()


def test_resident_timing_window_and_oracle():
    """A timing window runs the per-step kernels; the state passes through it."""
    import torch
    import paper_0908_3934_amd as gn
    spec = _lif(900, 7, 0.05)
    net = gn.Net(spec)
    parts = [net.step(300, raster=True, v=True, inp=True)]
    net.timing_begin(64, every=1)
    parts.append(net.step(20, raster=True, v=True, inp=True))
    torch.cuda.synchronize()
    assert net.timing_end()["deliver_launches"] == 20
    parts.append(net.step(400, raster=True, v=True, inp=True))
    torch.cuda.synchronize()
    g = {"raster": np.concatenate([gn.unpack_raster(p["raster"], net.n_total) for p in parts])}
    for key, name in (("v", "v"), ("input", "input")):
        g[key] = torch.cat([p[name] for p in parts]).cpu().numpy().astype(np.float64)
    check_parity(g, oracle.OracleNet(spec).step(720, v=True, inp=True))
    net.close()


def _learning(n, k, delays=None, burst=False):
    """A plastic network with inhibitory weights and weights that start at zero."""
    s = _burst(n, k) if burst else _lif(n, k, 0.05, delays)
    s.weight = s.weight.copy()
    s.weight[::5] *= -1.0
    s.weight[::7] = 0.0
    return synth.plastic(s, alpha=0.02, beta=0.1)


@pytest.mark.parametrize("args", [(2, 0), (65, 1, [1, 254, 255]), (1000, 2, [1, 2, 30, 90]), (700, 3, None, True),
                                  (20001, 4, [1, 2, 25])])
def test_resident_plastic_equals_per_step(args):
    """The same for weights that learn: every weight, and the spike times that
    the next call starts from."""
    import torch
    import paper_0908_3934_amd as gn
    spec = _learning(*args)
    print(args, spec.src.size, flush=True)
    nets = [gn.Net(spec), gn.Net(spec, flags=gn.NET_BUILD_REORDER), gn.Net(spec, flags=gn.NET_BUILD_PER_STEP)]
    for c, T in enumerate(CALLS):
        outs = [x.step(T, raster=True, v=True, inp=True) for x in nets]
        w = [x.observe(gn.NET_OBS_WEIGHTS) for x in nets]
        torch.cuda.synchronize()
        for k in range(2):
            for key in ("raster", "v", "input"):
                assert torch.equal(outs[k][key], outs[2][key]), (c, k, key)
            assert torch.equal(w[k], w[2]), (c, k)
    assert spec.src.size < 10 or int((w[2].cpu() != torch.tensor(spec.weight)).sum()) > spec.src.size // 20
    for x in nets:
        x.close()


def test_resident_on_streams_of_two_threads():
    """Two networks, a thread and a stream each: cooperative launches of one
    process take turns on the device, and each gives what it gives alone."""
    import threading
    import torch
    import paper_0908_3934_amd as gn
    specs = [_lif(1000, 8, 0.05), _lif(20000, 9, 0.05)]
    alone = []
    for s in specs:
        net = gn.Net(s)
        alone.append([net.step(64, raster=True, v=True) for _ in range(4)])
        torch.cuda.synchronize()
        net.close()
    nets, got = [gn.Net(s) for s in specs], [None, None]
    torch.cuda.synchronize()

    def work(k):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            got[k] = [nets[k].step(64, raster=True, v=True) for _ in range(4)]
        stream.synchronize()

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
        assert not t.is_alive()
    torch.cuda.synchronize()
    for k in range(2):
        for a, b in zip(alone[k], got[k]):
            for key in ("raster", "v"):
                assert torch.equal(a[key], b[key]), (k, key)
        nets[k].close()
