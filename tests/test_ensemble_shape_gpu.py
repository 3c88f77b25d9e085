"""blocks_per_cu pins the shape of the single-launch kernel that has one (the
push kernel runs one workgroup per network), with the same results."""
import pytest

from tests.test_ensemble_push_gpu import _lif

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("per_cu,threads", [(1, 0), (2, 0), (4, 256)])
def test_workgroups_per_cu(per_cu, threads):
    import torch
    import paper_0908_3934_amd as gn
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    specs = [_lif(40 + k, k, 0.05 * (k % 2)) for k in range(7)] * (4 * cus // 7 + 2)
    a = gn.Net(specs, blocks_per_cu=per_cu, block_threads=threads)
    b = gn.Net(specs)
    c = gn.Net(specs, flags=gn.NET_BUILD_PER_STEP)
    assert a.info()["ensemble_blocks"] == cus * per_cu
    assert a.info()["ensemble_threads"] == (threads or (512 if per_cu >= 2 else 1024))
    assert b.info()["ensemble_blocks"] == len(specs)
    for T in (150, 33):
        x, y, z = [net.step(T, raster=True, v=True, inp=True) for net in (a, b, c)]
        torch.cuda.synchronize()
        for key in z:
            assert torch.equal(x[key], z[key]) and torch.equal(y[key], z[key]), key
    for net in (a, b, c):
        net.close()


def test_lds_of_two_handles():
    """A handle that needs little LDS, built after one that needs most of it and
    stepped before it."""
    import torch
    import paper_0908_3934_amd as gn
    big, small = [_lif(900, 1, 0.0, [1, 100, 255]), _lif(64, 2, 0.05)], [_lif(900, 3, 0.0, [1]), _lif(64, 4, 0.05)]
    ref = [gn.Net(s, flags=gn.NET_BUILD_PER_STEP) for s in (small, big)]
    b, a = gn.Net(big), gn.Net(small)
    for T in (40, 200):
        for net, per_step in zip((a, b), ref):
            x, y = net.step(T, raster=True, v=True), per_step.step(T, raster=True, v=True)
            torch.cuda.synchronize()
            assert torch.equal(x["raster"], y["raster"]) and torch.equal(x["v"], y["v"])
    for net in [a, b] + ref:
        net.close()
