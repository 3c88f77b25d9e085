"""Resident launches whose workgroups do not all get onto the chip, or lose each
other: forced from the host through the library's test hook, every kernel ends
normally.  One workgroup alone gives the results of the per-step kernels
(tolerance 0); a launch that gives up says so in everything it leaves."""
import pytest

import synth
from tests.test_ensemble_push_gpu import _lif
from tests.test_resident_gpu import _burst, _learning

pytestmark = pytest.mark.gpu


def _lose(net, how):
    import paper_0908_3934_amd as gn
    assert gn.library().net_simulate_lost_workgroups(net.h, how) == 0


# (steps, whether the launch's workgroups come together)
CALLS = ((200, False), (130, True), (3, True), (150, False), (9, False), (300, True), (40, False), (64, True))
CASES = {
    "one vertex": lambda: _lif(1, 0, 0.0),
    "partial word": lambda: _lif(1000, 2, 0.05),
    "bursts": lambda: _burst(700, 4),
    "late arrivals": lambda: _lif(70000, 5, 0.05, [1, 3, 106, 107, 108, 255]),
}


@pytest.mark.parametrize("flag", ["default", "PUSH", "REORDER"])
@pytest.mark.parametrize("case", list(CASES))
def test_one_workgroup_alone(case, flag):
    import torch
    import paper_0908_3934_amd as gn
    from paper_0908_3934_amd import _abi
    spec = CASES[case]()
    print(case, flag, spec.src.size, flush=True)
    a = gn.Net(spec, flags=0 if flag == "default" else getattr(gn, "NET_BUILD_" + flag), frame_capacity=8)
    b = gn.Net(spec, flags=gn.NET_BUILD_PER_STEP, frame_capacity=8)
    assert a.resident()["workgroups"] > 0 and b.resident()["workgroups"] == 0
    for c, (T, together) in enumerate(CALLS):
        _lose(a, _abi.NET_LOST_NEVER if together else _abi.NET_LOST_AT_START)
        x, y = a.step(T, raster=True, v=True, inp=c != 4), b.step(T, raster=True, v=True, inp=c != 4)
        torch.cuda.synchronize()
        for key in x:
            assert x[key] is None or torch.equal(x[key], y[key]), (c, key)
    assert a.resident()["launches"] >= 5 and a.resident()["failed"] == 0
    frames = b.info()["frames_done"]
    assert a.info()["frames_done"] == frames >= 2
    for what, kw in ((gn.NET_OBS_V, {}), (gn.NET_OBS_CALCIUM, {}), (gn.NET_OBS_FRAMES, {"frames": frames}), (gn.NET_OBS_REF, {})):
        p, q = a.observe(what, **kw), b.observe(what, **kw)
        torch.cuda.synchronize()
        assert torch.equal(p, q), what
    a.close()
    b.close()


@pytest.mark.parametrize("args", [(65, 1, [1, 254, 255]), (700, 3, None, True), (5001, 4, [1, 2, 25])])
def test_one_workgroup_alone_learns(args):
    import torch
    import paper_0908_3934_amd as gn
    from paper_0908_3934_amd import _abi
    spec = _learning(*args)
    a, b = gn.Net(spec), gn.Net(spec, flags=gn.NET_BUILD_PER_STEP)
    for c, (T, together) in enumerate(CALLS):
        _lose(a, _abi.NET_LOST_NEVER if together else _abi.NET_LOST_AT_START)
        x, y = a.step(T, raster=True, v=True, inp=True), b.step(T, raster=True, v=True, inp=True)
        u, w = a.observe(gn.NET_OBS_WEIGHTS), b.observe(gn.NET_OBS_WEIGHTS)
        torch.cuda.synchronize()
        for key in x:
            assert torch.equal(x[key], y[key]), (c, key)
        assert torch.equal(u, w), c
    assert a.resident()["launches"] >= 7
    a.close()
    b.close()


def test_tags_after_launches_alone():
    """65,536 steps without published words, after which 16-bit tags come round again."""
    import torch
    import paper_0908_3934_amd as gn
    from paper_0908_3934_amd import _abi
    spec = _burst(130, 6)
    a, b = gn.Net(spec), gn.Net(spec, flags=gn.NET_BUILD_PER_STEP)
    for T, how in ((50, _abi.NET_LOST_NEVER), (65536, _abi.NET_LOST_AT_START), (200, _abi.NET_LOST_NEVER)):
        _lose(a, how)
        rec = T < 1000
        x, y = a.step(T, raster=rec, v=rec), b.step(T, raster=rec, v=rec)
        torch.cuda.synchronize()
        for key in x:
            assert x[key] is None or torch.equal(x[key], y[key]), (T, key)
    assert a.resident()["launches"] >= 1 + 4 + 1
    a.close()
    b.close()


@pytest.mark.parametrize("plastic", [False, True])
def test_given_up_launch_shows(plastic):
    import torch
    import paper_0908_3934_amd as gn
    from paper_0908_3934_amd import _abi
    spec = _lif(1000, 2, 0.05)
    net = gn.Net(synth.plastic(spec) if plastic else spec, frame_capacity=8)
    net.step(400)
    _lose(net, _abi.NET_LOST_IN_STEP)
    r = net.step(64, raster=True, v=True, inp=True)
    # enqueued behind it: the call and these see no status yet
    kinds = [(gn.NET_OBS_V, {}), (gn.NET_OBS_CALCIUM, {}), (gn.NET_OBS_FRAMES, {"frames": 1}), (gn.NET_OBS_FLUOR, {"frames": 1}),
             (gn.NET_OBS_REF, {})] + ([(gn.NET_OBS_WEIGHTS, {})] if plastic else [])
    out = []
    for what, kw in kinds:
        try:
            out.append((what, net.observe(what, **kw)))
        except gn.GeonetError as e:                     # (the launch has ended already)
            assert e.status == _abi.NET_E_DEVICE if not out or out[-1][1] is not None else e.status == _abi.NET_E_STATE
            break
    torch.cuda.synchronize()
    for what, x in out:
        assert bool((x == -1).all()) if what == gn.NET_OBS_REF else bool(torch.isnan(x).all()), what
    assert not bool(torch.isnan(r["v"][0]).any())
    assert bool(torch.isnan(r["v"][1:]).all()) and bool(torch.isnan(r["input"][1:]).all())
    assert bool((gn.unpack_raster(r["raster"][1:], 1000) == 1).all())
    assert net.resident()["failed"] == 1
    with pytest.raises(gn.GeonetError):
        net.step(64)
    with pytest.raises(gn.GeonetError):
        net.observe(gn.NET_OBS_V)
    net.close()


def test_busy_chip():
    """Another stream's launch holds every CU's LDS for a second or two: a
    resident call beside it gives what it gives alone."""
    import torch
    import paper_0908_3934_amd as gn
    spec = _lif(20000, 9, 0.05)
    a, b = gn.Net(spec), gn.Net(spec, flags=gn.NET_BUILD_PER_STEP)
    others = gn.Net([_lif(1500, k, 0.0, [1, 100, 255]) for k in range(4)] * 64)
    torch.cuda.synchronize()
    one, two = torch.cuda.Stream(), torch.cuda.Stream()
    others.step(300000, stream=one)
    for T in (100, 40):
        x = a.step(T, raster=True, v=True, stream=two)
        y = b.step(T, raster=True, v=True, stream=two)
        two.synchronize()
        for key in ("raster", "v"):
            assert torch.equal(x[key], y[key]), (T, key)
    torch.cuda.synchronize()
    assert a.resident()["failed"] == 0
    for x in (a, b, others):
        x.close()
