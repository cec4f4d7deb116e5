"""Multinomial ancestors from a lane's binary searches run in step: the same as the oracle's at particle
counts about the powers of two where a search's probes pass the end, at each number of particles a lane."""
import numpy as np
import pytest

from gpu_util import gpu_pf
from paper_2407_17296_amd import smc2, synth
from test_gpu_pf_parity import _check_fp64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,tile", [(1, 1), (2, 1), (3, 1), (63, 1), (64, 1), (65, 2), (129, 3),
                                    (255, 3), (256, 3), (257, 5), (511, 5), (512, 5), (513, 9),
                                    (1000, 9), (1024, 9)])
def test_multinomial_search(oracle, M, tile):
    """Resampling at every step (threshold above M), FP64: ancestors bit for bit."""
    w = synth.make(1, N=3, M=M, T=6)
    theta = np.broadcast_to(w.theta_true, (1, 3, w.D)).copy()
    items = [(0, i) for i in range(w.N)]
    ll, g, tr = gpu_pf(w, theta, tile=tile, ckpt=1, k=2, resampler=smc2.MULTINOMIAL,
                       ess_frac=1.5, trace_items=items)
    _check_fp64(oracle, w, theta, ll, g, tr, k=2, resampler=smc2.MULTINOMIAL, ess_frac=1.5)


@pytest.mark.parametrize("M,tile", [(200, 4), (511, 7), (512, 7), (1000, 8), (1024, 8), (1023, 11),
                                    (2047, 12), (2048, 12), (2049, 15), (4095, 15), (4096, 16)])
def test_multinomial_search_in_chunks(oracle, M, tile):
    """The same on lanes of one and two slots, and of sixteen (two chunks of eight searches)."""
    test_multinomial_search(oracle, M, tile)
