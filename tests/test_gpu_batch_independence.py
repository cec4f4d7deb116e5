"""FP64 results do not depend on how many filters a call holds: the library's own launch shape goes by
the number of filters, and the shapes it chooses between sum the weights in one order."""
import numpy as np
import pytest

from gpu_util import gpu_pf, spread_theta
from paper_2407_17296_amd import smc2, synth

pytestmark = pytest.mark.gpu


def _cut(w, N):
    """The workload with its first N samples."""
    import copy
    c = copy.copy(w)
    c.N = N
    return c


@pytest.mark.parametrize("index,M,line", [
    (0, 130, 256), (0, 250, 256), (3, 256, 256), (4, 255, 256), (5, 250, 1024), (0, 300, 512),
    (4, 512, 512), (5, 511, 512), (5, 600, 256), (5, 1024, 256)])
def test_fp64_estimate_in_a_small_and_in_a_large_batch(index, M, line):
    """The same samples in a call on either side of the line: the estimates bit for bit."""
    w = synth.make(index, S=1, N=line + 1, M=M, T=12)
    theta = spread_theta(w, 0.02, seed=M)
    items = [(0, i) for i in (0, line // 2, line - 1)]
    ll, g, tr = gpu_pf(w, theta, k=3, trace_items=items)
    ll1, g1, tr1 = gpu_pf(_cut(w, line), theta[:, :line], k=3, trace_items=items)
    assert np.array_equal(ll[:, :line], ll1)
    for it in items:
        assert np.array_equal(tr[it][0], tr1[it][0]) and np.array_equal(tr[it][1], tr1[it][1])
    assert np.linalg.norm(g[:, :line] - g1) <= 1e-9 * np.linalg.norm(g1)


@pytest.mark.parametrize("resampler", [smc2.SYSTEMATIC, smc2.MULTINOMIAL])
@pytest.mark.parametrize("index,M,wide,narrow", [
    (1, 129, 3, 4), (1, 256, 3, 4), (5, 200, 3, 4), (1, 257, 6, 7), (4, 512, 6, 7), (5, 400, 6, 7),
    (1, 513, 10, 11), (5, 1000, 10, 11), (1, 1024, 10, 11)])
def test_fp64_estimate_on_lanes_of_four_and_of_fewer_particles(index, M, wide, narrow, resampler):
    """Resampled at no, some and every step; 70 steps (SIR 35): more than one a thread of the smallest
    shape."""
    w = synth.make(index, S=1, N=5, M=M, T=70)
    theta = spread_theta(w, 0.02, seed=M)
    items = [(0, i) for i in range(w.N)]
    for ess_frac in (0.0, 0.5, 1.5):
        a = gpu_pf(w, theta, k=3, tile=wide, want_grad=0, trace_items=items, ess_frac=ess_frac,
                   resampler=resampler)
        b = gpu_pf(w, theta, k=3, tile=narrow, want_grad=0, trace_items=items, ess_frac=ess_frac,
                   resampler=resampler)
        assert np.array_equal(a[0], b[0]), ess_frac
        for it in items:
            assert np.array_equal(a[2][it][0], b[2][it][0])
            assert np.array_equal(a[2][it][1], b[2][it][1])


@pytest.mark.parametrize("resampler", [smc2.SYSTEMATIC, smc2.MULTINOMIAL])
@pytest.mark.parametrize("index,ckpt", [(0, 1), (0, 3), (5, 1), (5, 3)])
def test_fp64_gradient_of_up_to_256_particles_is_the_same_from_launch_to_launch(index, ckpt, resampler):
    w = synth.make(index, S=1, N=64, M=250, T=20)
    theta = spread_theta(w, 0.02, seed=8)
    kw = dict(k=3, ckpt=ckpt, ess_frac=1.5, resampler=resampler)
    first = gpu_pf(w, theta, **kw)
    for _ in range(3):
        again = gpu_pf(w, theta, **kw)
        assert np.array_equal(first[0], again[0]) and np.array_equal(first[1], again[1])
