"""The wide state's reverse scatter over sorted ancestors (sums across lanes, rows and waves before one
addition per run and wave), at every spread of the weights from even to a single survivor."""
import numpy as np
import pytest

from gpu_util import gpu_pf
from paper_2407_17296_amd import smc2, synth
from test_gpu_pf_parity import _check_fp64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ckpt,store_noise", [(1, 0), (1, 1), (4, 0), (4, 1)])
@pytest.mark.parametrize("M,tile", [(1, 1), (60, 1), (128, 2), (250, 4), (500, 7), (1024, 11),
                                    (2047, 14)])
@pytest.mark.parametrize("resampler", [smc2.SYSTEMATIC, smc2.MULTINOMIAL])
def test_fp64_wide_scatter(oracle, M, tile, ckpt, store_noise, resampler):
    """Resampling at every step (threshold above M); the three samples' observation spreads go from
    wide (runs of one or two offspring) to narrow (one parent for nearly all)."""
    w = synth.make(2, N=3, M=M, T=6)
    theta = np.broadcast_to(w.theta_true, (1, 3, w.D)).copy()
    theta[0, :, -1] = [3.0, 0.5, -1.5]
    items = [(0, i) for i in range(w.N)]
    ll, g, tr = gpu_pf(w, theta, tile=tile, ckpt=ckpt, k=4, store_noise=store_noise,
                       resampler=resampler, ess_frac=1.5, trace_items=items)
    _check_fp64(oracle, w, theta, ll, g, tr, k=4, resampler=resampler, ess_frac=1.5)
    if tile != 2:  # the mixed form, where no ancestor flipped
        ll32, g32, _ = gpu_pf(w, theta, precision=smc2.MIXED, tile=tile, ckpt=ckpt, k=4,
                              store_noise=store_noise, resampler=resampler, ess_frac=1.5)
        same = np.abs(ll32 - ll) <= 1e-4 * 6
        assert same.any()
        rel = np.linalg.norm(g32 - g, axis=-1) / np.linalg.norm(g, axis=-1)
        assert np.all(rel[same] <= 1e-3)


@pytest.mark.parametrize("store_noise", [0, 1])
@pytest.mark.parametrize("M,tile", [(1, 1), (60, 1), (65, 2), (128, 2), (250, 4), (500, 7), (1024, 11),
                                    (2047, 14), (2047, 17), (2048, 17)])
@pytest.mark.parametrize("resampler", [smc2.SYSTEMATIC, smc2.MULTINOMIAL])
def test_mixed_wide_segments_against_every_step(M, tile, store_noise, resampler):
    """The mixed form's segments against its own every-step checkpoints, on every shape: the forward
    sweep is the same, so the estimates agree bit for bit, whatever ancestors they take, and the
    gradients to rounding (their sums take another order)."""
    w = synth.make(2, N=3, M=M, T=6)
    theta = np.broadcast_to(w.theta_true, (1, 3, w.D)).copy()
    theta[0, :, -1] = [3.0, 0.5, -1.5]
    kw = dict(precision=smc2.MIXED, tile=tile, k=4, resampler=resampler, ess_frac=1.5)
    ll, g, _ = gpu_pf(w, theta, ckpt=1, store_noise=store_noise, **kw)
    ll4, g4, _ = gpu_pf(w, theta, ckpt=4, store_noise=store_noise, **kw)
    assert np.array_equal(ll, ll4)
    rel = np.linalg.norm(g4 - g, axis=-1) / np.linalg.norm(g, axis=-1)
    assert np.all(rel <= 1e-4), rel
