"""Systematic resampling where rounding decides a count: steps at which the kernel's estimate lies within
its margin of an integer and the counting rule's own comparisons are taken.  Such steps are rare (a
prefix in 2^28), so the seeds below were searched for; T = 2, resampled after step 1."""
import numpy as np
import pytest

from gpu_util import gpu_pf, oracle_pf
from paper_2407_17296_amd import smc2, synth

pytestmark = pytest.mark.gpu


def _word(oracle, seed):
    """The word of the offset of filter 0, iteration 3, step 1."""
    return int(oracle.philox([2**32 - 1, 1, 0, oracle.c3(3, 3)], [seed & 0xFFFFFFFF, seed >> 32])[0])


def _run(oracle, w, theta, precision, tile=0):
    items = [(0, i) for i in range(w.N)]
    ll, _, tr = gpu_pf(w, theta, precision=precision, k=3, ess_frac=1.5, ckpt=1, tile=tile,
                       trace_items=items)
    for (s, i) in items:
        r = oracle_pf(oracle, w, theta, s, i, k=3, ess_frac=1.5, want_trace=True)
        fl, anc = tr[(s, i)]
        assert fl[0] == 1 and np.array_equal(fl, r["flags"])
        assert np.array_equal(anc, r["ancestors"])
        if precision == smc2.FP64:
            assert abs(ll[s, i] - r["loglik"]) <= 1e-12 * abs(r["loglik"])


# the offset nu = (word + 1) 2^-32 of filter 0 at step 1: words 2^32 - 1 (every prefix of even weights
# on a target), 2^32 - 2, 1 and 5 (within the margin above and below)
@pytest.mark.parametrize("seed,word", [(63462225, 2**32 - 1), (4707225464, 2**32 - 2), (4892334448, 1),
                                       (437685311, 5)])
@pytest.mark.parametrize("M", [1, 3, 49, 64, 100, 250, 256, 300, 512, 1000, 2049, 4095, 4096])
@pytest.mark.parametrize("precision", [smc2.FP64, smc2.MIXED])
def test_every_prefix_near_a_target(oracle, seed, word, M, precision):
    """Observations that say nothing (log sy = 40): every weight is 1, every prefix a whole number, also
    in the lane that holds the last particle and the padding, and ((i + nu) / M) M rounds to either
    side of it."""
    assert _word(oracle, seed) == word
    w = synth.make(0, N=1, M=M, T=2)
    w.seed = seed
    theta = np.array([[[0.8, 0.0, 40.0]]])
    _run(oracle, w, theta, precision)


# weights of a filter at ordinary parameters, one prefix near a target
@pytest.mark.parametrize("seed,M,tile", [
    (27895, 4096, 15), (27895, 4096, 16), (21981, 4001, 15), (21981, 4001, 16), (129988, 4001, 16),
    (180725, 4001, 15)])
def test_one_prefix_near_a_target(oracle, seed, M, tile):
    w = synth.make(0, N=1, M=M, T=2)
    w.seed = seed
    w.y[:] = 0.5
    theta = np.broadcast_to(w.theta_true, (1, 1, w.D)).copy()
    a, sx, sy = theta[0, 0, 0], np.exp(theta[0, 0, 1]), np.exp(theta[0, 0, 2])
    e0, e1 = (np.concatenate([oracle.normals(seed, b, 0, oracle.c3(3, st), 4 * t, 4)
                              for b in range((M + 3) // 4)])[:M] for t, st in ((0, 1), (1, 2)))
    lw = -0.5 * ((0.5 - (a * e0 + sx * e1)) / sy) ** 2
    P = np.cumsum(np.exp(lw - lw.max()))
    z = P[:-1] / P[-1] * M - (_word(oracle, seed) + 1.0) * 2.0**-32
    assert np.abs(z - np.rint(z)).min() < 1e-9
    _run(oracle, w, theta, smc2.FP64, tile)
