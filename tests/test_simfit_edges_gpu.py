"""The fit's evaluation kernel at the edges of its work split: one to 64
realisations, more variants per target than one workgroup holds (64
realisations: 16 variants each), frames shorter than its 32-step blocks and
not a multiple of them, no noise, no hold and a hold that never ends.
Against the FP64 fit reference; the sums over frames and realisations differ
in order only (about 1e-12 of a likelihood of 1e3 nats), so 1e-6 holds as in
the full-size comparison."""
from dataclasses import replace

import numpy as np
import pytest

import synth
from tests.test_simfit_gpu import _case, _gpu, _ref

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,nf,den,sigma,n_ref", [
    (64, 4, 1000, 0.05, 20),
    (1, 20, 1000, 0.05, 20),
    (2, 20, 100, 0.05, 0),
    (8, 20, 20, 0.05, 20),
    (4, 9, 1000, 0.0, 20),
    (4, 6, 1000, 0.05, 255),
])
def test_evaluation_split_matches_reference(K, nf, den, sigma, n_ref):
    spec, F, gamma, pairs, dist, labels = _case(n_targets=3)
    spec = replace(spec, frame_den=den, noise_sigma=sigma, n_ref=n_ref)
    F = np.ascontiguousarray(F[:nf])
    print("simfit split: K=%d nf=%d den=%d sigma=%g n_ref=%d P=%d" % (K, nf, den, sigma, n_ref, len(pairs)), flush=True)
    g = _gpu(spec, F, gamma, pairs, dist, labels, w_assumed=synth.W0, realisations=K, sweeps=1, fit_seed=5)
    ref, _, _ = _ref(spec, F, gamma, pairs, w=synth.W0, K=K, sweeps=1, fit_seed=5)
    assert np.isfinite(g).all()
    assert (np.abs(g - ref) <= 1e-6 * np.maximum(1.0, np.abs(ref))).all(), np.abs(g - ref).max()
