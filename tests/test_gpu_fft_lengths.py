"""FFT passes over grid lengths of every radix schedule, with the zero gap
starting inside, at and between the radix segments, against numpy's FFT in
float64, and the coil combination in one and in several rounds of a tile."""
import numpy as np
import pytest

from nudft import rel_l2

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# A float32 transform of length K loses about 6e-8 per pass and per rounded
# twiddle and scale (at most 7 passes): below 1e-6 in relative L2.
TOL = 1e-6

LENGTHS = [(2, 2), (4, 2), (6, 4), (8, 8), (10, 6), (12, 12), (16, 10), (18, 10), (20, 14), (24, 16), (30, 16), (36, 24),
           (40, 22), (48, 32), (50, 30), (54, 40), (60, 60), (64, 34), (72, 48), (90, 50), (96, 48), (100, 74), (108, 72),
           (128, 64), (150, 100), (162, 110), (192, 96), (240, 120), (250, 126), (360, 182), (400, 216), (486, 250),
           (512, 256), (640, 322), (768, 384), (810, 406), (1152, 600), (1250, 700), (1458, 730), (2048, 1024),
           (4096, 2050)]


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def _plan(N, K, J, dev, **options):
    from paper_1710_03197_amd import Plan
    r = np.random.default_rng(3)
    om = r.uniform(-np.pi, np.pi, (40, len(N))).astype(np.float32)
    return om, Plan(torch.from_numpy(om).to(dev), N, K, J, options=options)


@pytest.mark.parametrize("schedule", [0, 1, 2, 3])
@pytest.mark.parametrize("K0,N0", LENGTHS)
def test_passes_match_numpy(orc, dev, K0, N0, schedule):
    """K0 on the strided axis, on the contiguous one and alone."""
    r = np.random.default_rng(K0)
    J = min(4, K0)
    cases = [((N0,), (K0,)), ((N0, 6), (K0, 10)), ((6, N0), (10, K0))]
    if K0 <= 128:
        cases.append(((4, N0, 6), (6, K0, 8)))
    for N, K in cases:
        x = (r.standard_normal(N) + 1j * r.standard_normal(N)).astype(np.complex64)
        h = (r.standard_normal(K) + 1j * r.standard_normal(K)).astype(np.complex64)
        jj = min(J, min(K))
        _, plan = _plan(N, K, jj, dev, fft_radix=schedule)
        with plan:
            G = plan.stage_fs(torch.from_numpy(x).to(dev)).cpu().numpy()
            img = plan.stage_shfh(torch.from_numpy(h).to(dev)).cpu().numpy()
        assert rel_l2(G, np.fft.fftn(orc.pad_scale(x, N, K, jj))) < TOL, (N, K)
        want = orc.crop_scale(np.fft.ifftn(h.astype(np.complex128)) * np.prod(K), N, K, jj)
        assert rel_l2(img, want) < TOL, (N, K)


@pytest.mark.parametrize("C,N,K", [(1, (12, 20), (24, 36)), (3, (10, 40), (20, 60)), (7, (8, 322), (16, 640)),
                                   (9, (6, 600), (12, 1152)), (5, (4, 8, 30), (8, 12, 54))])
def test_coil_rounds_match_oracle(orc, dev, C, N, K):
    """Coil sums in one round (C K <= 4096) and several, several rows per tile and one."""
    r = np.random.default_rng(C)
    coils = (r.standard_normal((C,) + N) + 1j * r.standard_normal((C,) + N)).astype(np.complex64)
    x = (r.standard_normal(N) + 1j * r.standard_normal(N)).astype(np.complex64)
    om, plan = _plan(N, K, 4, dev)
    ys = (r.standard_normal((C, len(om))) + 1j * r.standard_normal((C, len(om)))).astype(np.complex64)
    with plan:
        plan.set_coils(torch.from_numpy(coils).to(dev))
        y = plan.forward(torch.from_numpy(x).to(dev)).cpu().numpy()
        z = plan.adjoint(torch.from_numpy(ys).to(dev)).cpu().numpy()
    assert rel_l2(y, orc.forward_coils(x, coils, om, N, K, 4)) < TOL
    assert rel_l2(z, orc.adjoint_coils(ys, coils, om, N, K, 4)) < TOL
