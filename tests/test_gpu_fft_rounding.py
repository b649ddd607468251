"""Rounding of the FFT passes: lengths whose default schedule takes radix 6
against the same lengths in radices 8, 4, 2, 3, 5."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# Both errors are rms over at least 20000 complex values, 0.5% standard error
# each: three of them on either side of equality.
TOL = 1.02


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def _errors(orc, dev, K, schedule):
    """rms error of the forward and the inverse transform of length K, scaling
    left out (it is applied in float32 to the reference as well)."""
    from paper_1710_03197_amd import Plan
    N = K // 2
    ones = orc.pad_scale(np.ones(N, np.complex64), (N,), (K,), 4).real
    live = ones > 0
    at = np.rint(orc.pad_scale(np.arange(1, N + 1).astype(np.complex64), (N,), (K,), 4).real[live] / ones[live]) - 1
    scale = ones[live].astype(np.float32)
    crop = orc.crop_scale(np.ones(K, np.complex128), (N,), (K,), 4).real
    crop32 = crop.astype(np.float32).astype(np.float64)
    r = np.random.default_rng(K)
    sums = np.zeros(4)
    om = torch.zeros((4, 1), dtype=torch.float32, device=dev)
    with Plan(om, (N,), (K,), 4, options=dict(fft_radix=schedule)) as p:
        for _ in range(20000 // K + 20):
            x = (r.standard_normal(N) + 1j * r.standard_normal(N)).astype(np.complex64)
            h = (r.standard_normal(K) + 1j * r.standard_normal(K)).astype(np.complex64)
            G = p.stage_fs(torch.from_numpy(x).to(dev)).cpu().numpy()
            g = p.stage_shfh(torch.from_numpy(h).to(dev)).cpu().numpy()
            t = np.zeros(K, np.complex64)
            t.real[live], t.imag[live] = x.real[at.astype(int)] * scale, x.imag[at.astype(int)] * scale
            G_ref = np.fft.fft(t.astype(np.complex128))
            g_ref = orc.crop_scale(np.fft.ifft(h.astype(np.complex128)) * K, (N,), (K,), 4) / crop * crop32
            for k, (got, ref) in enumerate(((G, G_ref), (g, g_ref))):
                sums[2 * k] += np.sum(np.abs(got - ref) ** 2)
                sums[2 * k + 1] += np.sum(np.abs(ref) ** 2)
    return np.sqrt(sums[::2] / sums[1::2])


@pytest.mark.parametrize("K", [36, 144, 216, 288, 432, 648, 864, 1296])
def test_radix_6_rounds_no_more_than_8_4_2_3_5(orc, dev, K):
    default, greedy = _errors(orc, dev, K, 0), _errors(orc, dev, K, 3)
    print(f"K={K}: {default} against {greedy}", flush=True)
    assert (default <= TOL * greedy).all()
