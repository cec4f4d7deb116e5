"""The filter's noise on lanes with fewer slots than a Philox block serves: several steps drawn at a
time and exchanged between lanes, with series and segments that end inside such a group of steps."""
import pytest

from gpu_util import gpu_pf, spread_theta
from paper_2407_17296_amd import smc2, synth
from test_gpu_pf_parity import _check_fp64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ckpt,store_noise", [(1, 0), (3, 0), (3, 1), (7, 0)])
@pytest.mark.parametrize("index,M,tile", [
    (0, 64, 1),    # one component, one slot a lane: four steps at a time
    (0, 100, 2),   # ... on two waves, ragged
    (0, 256, 4),   # ... on four waves
    (0, 512, 7),   # two slots a lane: two steps at a time
    (0, 200, 3),   # four slots a lane: a block a step
    (5, 60, 1),    # two components, one slot a lane: two steps at a time
    (5, 256, 4),
])
def test_fp64_noise_groups(oracle, index, M, tile, ckpt, store_noise):
    """Every item's estimate, gradient and ancestry against the oracle, T = 10 (a remainder of two)."""
    w = synth.make(index, N=3, M=M, T=10)
    theta = spread_theta(w, 0.05, seed=90 + M)
    items = [(0, i) for i in range(w.N)]
    ll, g, tr = gpu_pf(w, theta, tile=tile, ckpt=ckpt, k=5, store_noise=store_noise,
                       trace_items=items)
    _check_fp64(oracle, w, theta, ll, g, tr, k=5)
    # the mixed form draws the same words: the same estimate to FP32 rounding, where no ancestor flips
    ll32, _, _ = gpu_pf(w, theta, precision=smc2.MIXED, tile=tile, ckpt=ckpt, k=5,
                        store_noise=store_noise)
    assert (abs(ll32 - ll) <= 1e-4 * 10).mean() >= 0.3


@pytest.mark.parametrize("ckpt,store_noise", [(1, 0), (3, 0), (3, 1)])
@pytest.mark.parametrize("index,M,tile", [(0, 64, 1), (0, 100, 2), (0, 256, 4), (0, 512, 7), (0, 200, 3),
                                          (0, 500, 5), (5, 60, 1), (5, 256, 4), (5, 200, 3)])
def test_mixed_noise_groups(index, M, tile, ckpt, store_noise):
    """The mixed form draws the same words: without resampling no ancestor can flip, and every estimate
    and gradient follows the FP64 form's."""
    w = synth.make(index, N=16, M=M, T=10)
    theta = spread_theta(w, 0.05, seed=90 + M)
    kw = dict(tile=tile, ckpt=ckpt, k=5, store_noise=store_noise, ess_frac=0.0)
    ll, g, _ = gpu_pf(w, theta, **kw)
    ll32, g32, _ = gpu_pf(w, theta, precision=smc2.MIXED, **kw)
    assert abs(ll32 - ll).max() <= 1e-4 * 10
    for i in range(w.N):
        assert ((g32[0, i] - g[0, i]) ** 2).sum() <= (1e-3 ** 2) * (g[0, i] ** 2).sum()
