"""The every-step reverse sweep at the ends of its read-ahead: series of one to three steps, series that
cross the 64-step window of flags, and resampling at no, some and every step."""
import numpy as np
import pytest

from gpu_util import gpu_pf, spread_theta
from paper_2407_17296_amd import smc2, synth
from test_gpu_pf_parity import _check_fp64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ess_frac", [0.0, 0.5, 1.5])
@pytest.mark.parametrize("T", [1, 2, 3, 64, 65, 66, 130])
@pytest.mark.parametrize("index", [0, 3, 4, 5])
def test_fp64_reverse_reads(oracle, index, T, ess_frac):
    if index == 3 and T > 66:
        T = 67  # the growth model's gradient is ill-conditioned on longer series
    w = synth.make(index, S=1, N=2, M=100 if index else 256, T=T)
    w.T_len[:] = T
    if w.y.shape[1] < T:
        w.y = np.concatenate([w.y] * (T // w.y.shape[1] + 1), axis=1)[:, :T].copy()
    theta = spread_theta(w, 0.03, seed=T)
    items = [(0, 0), (0, 1)]
    ll, g, tr = gpu_pf(w, theta, ckpt=1, k=6, store_noise=T % 2, ess_frac=ess_frac,
                       trace_items=items)
    _check_fp64(oracle, w, theta, ll, g, tr, k=6, ess_frac=ess_frac)
    ll32, g32, _ = gpu_pf(w, theta, precision=smc2.MIXED, ckpt=1, k=6, store_noise=T % 2,
                          ess_frac=ess_frac)
    assert np.all(np.isfinite(ll32)) and np.all(np.isfinite(g32))


@pytest.mark.parametrize("ess_frac", [0.0, 0.5, 1.5])
@pytest.mark.parametrize("T", [1, 2, 3, 64, 65, 66, 130])
@pytest.mark.parametrize("index", [0, 3, 4, 5])
def test_mixed_reverse_reads_against_segments(index, T, ess_frac):
    """The mixed form at a checkpoint every step, noise stored and recovered, against the segments that
    are recomputed from every third (which read neither ancestors nor carry ahead): the same estimate,
    the gradient within the mixed form's bar."""
    if index == 3 and T > 3:
        T = 4 + T % 3  # the growth model's gradient is ill-conditioned on longer series
    w = synth.make(index, S=1, N=4, M=100 if index else 256, T=T)
    w.T_len[:] = T
    if w.y.shape[1] < T:
        w.y = np.concatenate([w.y] * (T // w.y.shape[1] + 1), axis=1)[:, :T].copy()
    theta = spread_theta(w, 0.03, seed=T)
    kw = dict(precision=smc2.MIXED, k=6, ess_frac=ess_frac)
    ll, g, _ = gpu_pf(w, theta, ckpt=3, store_noise=1, **kw)
    assert np.any(g != 0)
    for store_noise in (0, 1):
        ll1, g1, _ = gpu_pf(w, theta, ckpt=1, store_noise=store_noise, **kw)
        assert np.array_equal(ll, ll1)
        for i in range(w.N):
            assert np.linalg.norm(g1[0, i] - g[0, i]) <= 1e-3 * np.linalg.norm(g[0, i]), (i, store_noise)
