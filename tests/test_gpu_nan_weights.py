"""Particles whose weight is not a number count as particles of weight zero, in the forward sweep, the
adjoint and beside padding slots.  The SV density at y = 0 is 0 * exp(-x) - x / 2: not a number where
the exponential overflows (x below -709.78 in FP64, -88.72 in FP32)."""
import numpy as np
import pytest

from gpu_util import gpu_pf
from paper_2407_17296_amd import smc2, synth
from test_gpu_pf_parity import _check_fp64

pytestmark = pytest.mark.gpu


def _workload(M, T, mu):
    w = synth.make(4, S=1, N=4, M=M, T=T)
    w.y[:] = 0.0
    theta = np.empty((1, 4, 3))
    theta[..., 0] = mu + np.array([0.6, 0.2, -0.1, 0.0])
    theta[..., 1], theta[..., 2] = 0.5, -1.0
    return w, theta


@pytest.mark.parametrize("ckpt", [1, 3])
@pytest.mark.parametrize("M", [50, 100, 256, 500])
@pytest.mark.parametrize("ess_frac", [0.0, 0.5, 1.5])
def test_fp64_nan_weights(oracle, M, ckpt, ess_frac):
    w, theta = _workload(M, 5, -709.78)
    items = [(0, i) for i in range(w.N)]
    ll, g, tr = gpu_pf(w, theta, ckpt=ckpt, k=2, ess_frac=ess_frac, trace_items=items)
    assert np.all(np.isfinite(ll)) and np.all(np.isfinite(g))
    _check_fp64(oracle, w, theta, ll, g, tr, k=2, ess_frac=ess_frac)


@pytest.mark.parametrize("ckpt", [1, 3])
@pytest.mark.parametrize("M", [50, 100, 256, 500])
def test_mixed_nan_weights(oracle, M, ckpt):
    """One step: log of the mean of the weights exp(-x / 2) / sqrt(2 pi) of the particles whose exponential
    is finite, the states from the oracle's normals.  A particle within 1e-4 of the limit may fall on
    either side: it moves the mean by less than 2 / M."""
    k, lim = 2, 128 * np.log(2.0)
    w, theta = _workload(M, 1, -88.72)
    ll, g, _ = gpu_pf(w, theta, precision=smc2.MIXED, ckpt=ckpt, k=k)
    assert np.all(np.isfinite(g))
    some = 0
    for i in range(w.N):
        mu, s = theta[0, i, 0], np.exp(theta[0, i, 2])
        z = [np.concatenate([oracle.normals(w.seed, b, i, oracle.c3(k, st), 4 * t, 4)
                             for b in range((M + 3) // 4)])[:M] for t, st in ((0, 1), (1, 2))]
        x = mu + np.tanh(theta[0, i, 1]) * s * np.cosh(theta[0, i, 1]) * z[0] + s * z[1]
        near = np.abs(x + lim) < 1e-4
        ok = x > -lim
        some += int(np.sum(~ok & ~near))
        wt = np.exp(-0.5 * (x - mu))
        want = np.log(wt[ok].sum() / M) - 0.5 * mu - 0.5 * np.log(2 * np.pi)
        slack = np.log1p(wt[near].sum() / wt[ok & ~near].sum())
        assert abs(ll[0, i] - want) <= 1e-4 + slack, (i, ll[0, i], want)
    assert some > 0


@pytest.mark.parametrize("ckpt,store_noise", [(1, 0), (1, 1), (3, 0)])
def test_mixed_overflowed_adjoint_shows_in_the_gradient(ckpt, store_noise):
    """An adjoint beyond FP32's range (one particle, one step, log sy = -46: d log g / dx above 3.4e38 at
    a finite density) is not lost in the products that give 0 for 0 times anything."""
    w = synth.make(0, N=256, M=1, T=1)
    w.y[:] = 0.0
    theta = np.broadcast_to([0.8, 0.0, -46.0], (1, 256, 3)).copy()
    ll, g, _ = gpu_pf(w, theta, ckpt=ckpt, store_noise=store_noise, k=2)
    ll32, g32, _ = gpu_pf(w, theta, precision=smc2.MIXED, ckpt=ckpt, store_noise=store_noise, k=2)
    adjoint = np.sqrt(g[..., 2] + 1) * np.exp(46.0)  # |r| / sy, from d ll / d log sy = r^2 - 1
    over = np.isfinite(ll32) & (adjoint > 4e38)
    assert over.sum() > 5
    assert not np.any(np.all(np.isfinite(g32[over]), axis=-1))
