"""net_build where device memory runs out: the tables of the resident and of the
push ensemble kernel are not needed for a handle that works, so no allocation
of theirs that fails may fail the build.  Results against the per-step kernels
(tolerance 0)."""
import contextlib

import pytest

import synth
from tests.test_ensemble_push_gpu import _lif

pytestmark = pytest.mark.gpu


@contextlib.contextmanager
def _allocator(fails):
    """Device memory from PyTorch's allocator; allocation number k (from 0)
    fails where fails(k).  Yields the list of the sizes asked for."""
    import torch
    import paper_0908_3934_amd as gn
    from paper_0908_3934_amd import _abi
    asked = []

    def alloc(nbytes, stream, ctx):
        asked.append(int(nbytes))
        return None if fails(len(asked) - 1) else torch.cuda.caching_allocator_alloc(int(nbytes), stream=int(stream or 0))

    def release(ptr, stream, ctx):
        torch.cuda.caching_allocator_delete(int(ptr))

    gn._register_torch_allocator()
    keep = _abi.ALLOC_FN(alloc), _abi.RELEASE_FN(release)
    assert gn.library().net_set_allocator(*keep, None) == 0
    try:
        yield asked
    finally:
        assert gn.library().net_set_allocator(gn._alloc_cb, gn._release_cb, None) == 0


def _noisy_ensemble():
    return [_lif(300, 1, 0.05), _lif(70, 2, 0.0), _lif(900, 3, 0.05, [1, 2, 40])]


@pytest.mark.parametrize("make,flags", [(lambda: _lif(900, 1, 0.05), 0), (lambda: _lif(900, 1, 0.05), "PUSH"),
                                        (lambda: synth.plastic(_lif(700, 2, 0.05)), 0), (_noisy_ensemble, 0)],
                         ids=["resident", "resident push", "plastic", "ensemble"])
def test_no_memory_for_optional_tables(make, flags):
    import torch
    import paper_0908_3934_amd as gn
    specs = make()
    flags = gn.NET_BUILD_PUSH if flags == "PUSH" else 0
    ensemble = isinstance(specs, list)

    def run(fails, extra=0):
        with _allocator(fails) as asked:
            net = gn.Net(specs, flags=flags | extra, torch_allocator=False)
            uses = net.resident()["workgroups"] > 0 or net.info()["ensemble_blocks"] > 0
            held = net.info()["device_bytes"]
            out = [net.step(T, raster=True, v=True, inp=True) for T in (150, 40)]
            torch.cuda.synchronize()
            net.close()
        return out, len(asked), uses, held

    ref, base, uses, small = run(lambda k: False, gn.NET_BUILD_PER_STEP)
    assert not uses
    _, most, uses, large = run(lambda k: False)
    assert uses and most > base and large > small
    for bad in range(base, most):
        print("allocation", bad, "of", most, flush=True)
        out, asked, uses, held = run(lambda k: k == bad)
        # (an ensemble has another single-launch kernel, or only draws its noise in the steps)
        assert uses if ensemble else (not uses and held == small)
        for x, y in zip(out, ref):
            for key in x:
                assert torch.equal(x[key], y[key]), (bad, key)
