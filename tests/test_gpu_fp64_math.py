"""FP64 elementary functions of the kernels: the Box-Muller normals (logarithm, square root, sine and
cosine) against extended precision on the device's own Philox words."""
import numpy as np
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed", [1, 0xFFFFFFFF00000001])
def test_fp64_normals_against_extended_precision(seed):
    """Each normal is r cos a or r sin a with a = 2 pi u2 rounded to double.  The logarithm is
    within 1.1 ulp (halved by the root), the root, sine / cosine and product within 0.5, 0.6 and
    0.5: together below 2.2 ulp, that is 2.2 * 2^-52 of the value."""
    import torch
    from paper_2407_17296_amd import smc2
    R = 1 << 18
    rng = np.random.default_rng(seed & 0xFFFF)
    ctr = rng.integers(0, 2**32, size=(R, 4), dtype=np.uint64).astype(np.uint32)
    ctr[:, 1] = 0
    n = (np.arange(R) % 4).astype(np.int32)  # both pairs of a block, cosine and sine
    dev = torch.device("cuda:0")
    say("  normals R=%d" % R)
    out, nz, _, _, _ = smc2.smc2_philox_probe(torch.tensor(ctr.view(np.int32), device=dev),
                                              torch.tensor(n, device=dev), seed)
    torch.cuda.synchronize()
    w = out.cpu().numpy().view(np.uint32)
    ld = np.longdouble
    wa, wb = np.where(n < 2, w[:, 0], w[:, 2]), np.where(n < 2, w[:, 1], w[:, 3])
    r = np.sqrt(-2 * np.log((wa.astype(ld) + 1) / ld(2)**32))
    a = (2 * np.pi * (wb * 2.0**-32)).astype(ld)
    want = r * np.where(n % 2 == 0, np.cos(a), np.sin(a))
    rel = np.abs(nz.cpu().numpy().astype(ld) - want) / np.abs(want)
    say("  max relative error %.3e" % float(rel.max()))
    assert float(rel.max()) < 2.2 * 2.0**-52


def _sv_at(mu, y, M=1):
    """Log-likelihoods [S][N] and gradients of one-step SV filters whose particles all lie at mu [S][N]
    (log s = -45), each series with its observation y [S]."""
    from gpu_util import gpu_pf
    from paper_2407_17296_amd import synth
    S, N = mu.shape
    w = synth.make(4, S=S, N=N, M=M, T=1)
    w.y[:, 0, 0] = y
    theta = np.stack([mu, np.zeros_like(mu), np.full_like(mu, -45.0)], axis=-1)
    ll, g, _ = gpu_pf(w, theta)
    return ll, g


def test_fp64_exponential():
    """log g = -(y^2 exp(-mu) + mu + log 2 pi) / 2 with y^2 exp(-mu) above 1e4 |mu| is the exponential to
    1e-4 and four roundings (y^2, two fused sums and, with it below 0.9 units, the exponential's own):
    together below 1.1 * (0.9 + 3 * 0.5) units of 2^-52."""
    rng = np.random.default_rng(3)
    ld = np.longdouble
    centre = np.concatenate([np.linspace(-690, -20, 24), np.linspace(-19, 685, 40)])
    y = np.where(centre < -19.5, 1.0, 3e3 * np.exp(centre / 2))
    mu = centre[:, None] + rng.uniform(-0.5, 0.5, (64, 256))
    ll, _ = _sv_at(mu, y)
    y2 = (y * y)[:, None].astype(ld)
    want = -(y2 * np.exp(-mu.astype(ld)) + mu + np.log(2 * ld(np.pi))) / 2
    rel = np.abs((ll.astype(ld) - want) / want)
    say("  exponential: max %.2f units" % (float(rel.max()) * 2.0**52))
    assert float(rel.max()) < 1.1 * (0.9 + 3 * 0.5) * 2.0**-52


def test_fp64_exponential_at_its_ends():
    """0 below the smallest subnormal, infinity above the largest double."""
    mu = np.array([[746.0, 800.0, 1e6, 1e300], [-709.7, -709.79, -711.0, -1e300]])
    ll, g = _sv_at(mu, np.array([1.0, 1.0]))
    half = 0.5 * np.log(2 * np.pi)
    assert np.array_equal(ll[0], -0.5 * mu[0] - half)  # y^2 exp(-mu) = 0
    assert np.allclose(g[0, :, 0], -0.5, rtol=1e-15)
    assert np.isfinite(ll[1, 0]) and ll[1, 0] < -1e307
    assert np.all(ll[1, 1:] == -np.inf) and np.all(g[1, 1:] == 0.0)


@pytest.mark.parametrize("M", [1, 2, 3, 7, 64, 100, 1000, 1024, 4095, 4096])
def test_fp64_logarithm_of_the_weight_sum(M):
    """Even weights whose log density is zero (y = 0, mu = -log 2 pi): the estimate is log S - log M with
    S = M, zero to the roundings of the two logarithms (0.6 units each) and of the sum."""
    mu = np.full((1, 4), -np.log(2 * np.pi))
    ll, _ = _sv_at(mu, np.zeros(1), M)
    assert np.all(np.abs(ll) <= 1.2 * np.spacing(np.log(M)) + 2.0**-52)


def test_fp64_normals_rms():
    """Three correctly rounded operations (root, sine or cosine, product; one has an rms error of
    2^-53 (0.541 / 3)^(1/2) of the value for logarithmically spread mantissas) come to 8.17e-17; the
    logarithm enters the root unrounded and adds next to nothing."""
    import torch
    from paper_2407_17296_amd import smc2
    R = 1 << 19
    rng = np.random.default_rng(11)
    ctr = rng.integers(0, 2**32, size=(R, 4), dtype=np.uint64).astype(np.uint32)
    ctr[:, 1] = 0
    n = (np.arange(R) % 2).astype(np.int32)
    dev = torch.device("cuda:0")
    out, nz, _, _, _ = smc2.smc2_philox_probe(torch.tensor(ctr.view(np.int32), device=dev),
                                              torch.tensor(n, device=dev), 5)
    w = out.cpu().numpy().view(np.uint32)
    ld = np.longdouble
    r = np.sqrt(-2 * np.log((w[:, 0].astype(ld) + 1) / ld(2)**32))
    a = (2 * np.pi * (w[:, 1] * 2.0**-32)).astype(ld)
    want = r * np.where(n == 0, np.cos(a), np.sin(a))
    rms = float(np.sqrt(np.mean(((nz.cpu().numpy().astype(ld) - want) / want) ** 2)))
    say("  rms relative error %.4e" % rms)
    assert rms <= 1.01 * 2.0**-53 * np.sqrt(0.541)


def test_fp64_normal_of_a_unit_uniform_is_zero():
    """u1 = 1 (a word of 2^32 - 1: word 0 of block 1 of this stream): radius zero, both normals zero."""
    import torch
    from paper_2407_17296_amd import smc2
    dev = torch.device("cuda:0")
    ctr = torch.tensor([[-1, 1, 0, (3 << 8) | 3]] * 2, dtype=torch.int32, device=dev)
    out, nz, _, _, _ = smc2.smc2_philox_probe(ctr, torch.tensor([4, 5], dtype=torch.int32, device=dev),
                                              63462225)
    assert out[0, 0].item() == -1
    assert torch.all(nz == 0)
