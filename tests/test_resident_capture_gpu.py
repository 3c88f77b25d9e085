"""A short call recorded into a HIP graph whose replays come between eager
calls: the arrivals that the resident kernel keeps must not survive them.
Against the per-step kernels, recorded and replayed alike (tolerance 0)."""
import pytest

from tests.test_ensemble_push_gpu import _lif

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flag", ["default", "FUSED_STEP", "PUSH"])
def test_captured_short_call(flag):
    import torch
    import paper_0908_3934_amd as gn
    spec = _lif(900, 3, 0.05)
    flags = 0 if flag == "default" else getattr(gn, "NET_BUILD_" + flag)
    got = []
    for net in (gn.Net(spec, flags=flags), gn.Net(spec, flags=flags | gn.NET_BUILD_PER_STEP)):
        out = [net.step(150, raster=True, v=True)]
        torch.cuda.synchronize()
        graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        with torch.cuda.graph(graph, stream=stream):
            net.step(4, stream=stream)
        for T in (200, 50, 9):
            graph.replay()
            torch.cuda.synchronize()
            out.append(net.step(T, raster=True, v=True, inp=True))
            torch.cuda.synchronize()
        got.append(out)
        del graph
        net.close()
    for x, y in zip(*got):
        for key in x:
            assert x[key] is None or torch.equal(x[key], y[key]), key
    assert sum(int(gn.unpack_raster(y["raster"], 900).sum()) for y in got[1]) > 20
