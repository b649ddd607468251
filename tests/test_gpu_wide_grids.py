"""Strided FFT passes over grids whose rows between two elements of a butterfly
hold more than 4 GiB (lengths that start or end in radix 2 or 3), as single
and as multi-problem launches, against the exact sums in float64."""
import numpy as np
import pytest

from nudft import rel_l2

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


# N, K, options, samples: the default schedule's last radix of 162 is 3 (forward
# stores); schedule 1 of 162 starts in 2 (inverse loads); schedule 2 of 1458
# starts in 3, with the crowded centre's partial tiles summed in that pass.
CASES = [((2, 2, 2), (162, 4096, 3200), dict(), 2000),
         ((4, 2, 2), (162, 4096, 3200), dict(fft_radix=1), 2000),
         ((2, 4, 2), (1458, 1024, 1080), dict(fft_radix=2, fuse_reduce=1, grid_chunk=64), 2000)]


@pytest.mark.parametrize("N,K,options,M", CASES)
def test_pair_on_wide_slabs(dev, N, K, options, M):
    from paper_1710_03197_amd.plan import MultiPlan, Plan
    r = np.random.default_rng(sum(N))
    om = r.uniform(-np.pi, np.pi, (M, 3)).astype(np.float32)
    om[: M // 4] *= 1e-4  # a crowded tile at the centre
    x = (r.standard_normal(N) + 1j * r.standard_normal(N)).astype(np.complex64)
    y = (r.standard_normal(M) + 1j * r.standard_normal(M)).astype(np.complex64)
    pos = np.stack(np.meshgrid(*[np.arange(n) - n // 2 for n in N], indexing="ij"), -1).reshape(-1, 3)
    E = np.exp(-1j * (om.astype(np.float64) @ pos.T))
    y_ref = E @ x.reshape(-1).astype(np.complex128)
    x_ref = (E.conj().T @ y.astype(np.complex128)).reshape(N)
    t = [torch.from_numpy(v).to(dev) for v in (om, x, y)]
    print(f"N={N} K={K} {options}: single plan", flush=True)
    with Plan(t[0], N, K, 6, options=options) as p:
        ys, xs = p.forward(t[1]).cpu().numpy(), p.adjoint(t[2]).cpu().numpy()
    assert rel_l2(ys, y_ref) < 1e-5
    assert rel_l2(xs, x_ref) < 1e-5
    print("multi-problem plan", flush=True)
    mp = MultiPlan([dict(om=t[0], N=N, K=K, options=options)], J=6)
    ym, xm = mp.forward([t[1]])[0].cpu().numpy(), mp.adjoint([t[2]])[0].cpu().numpy()
    mp.close()
    assert np.array_equal(ym, ys) and np.array_equal(xm, xs)
