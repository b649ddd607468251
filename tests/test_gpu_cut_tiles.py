"""Default tiles on grids that 16- and 8-cell tiles do not divide (evenly cut
tiles of at most that size): gather, every gridding form on the matrix cores,
both sums of split tiles, against the FP64 oracle, and the tile arithmetic."""
import numpy as np
import pytest

from nudft import rel_l2

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TOL = 1e-5  # the suite's bar against the oracle
TOL_NO_OVERSAMPLING = 5e-4  # and its bar where an axis has K = N (the scaling magnifies float32 rounding)


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


@pytest.mark.parametrize("N,K,J,options", [
    ((12, 20), (24, 40), 6, dict(fuse_reduce=1)),            # 24 = 12 + 12, 40 = 12 + 14 + 14
    ((12, 20), (24, 40), 6, dict(fuse_reduce=2)),
    ((27 * 2, 50), (108, 100), 6, dict(grid_chunk=64)),
    ((82, 90), (162, 180), 5, dict(grid_chunk=64, weight_table=1)),
    ((64, 100), (128, 162), 7, dict(grid_mfma=3)),           # one axis divides, row tiles
    ((60, 45 * 2), (90, 150), 8, dict(interp_merge=3)),
    ((100, 60), (200, 120), 6, dict(interpolator=1)),
    ((30, 50), (50, 90), 11, {}),
    ((11 * 2, 18), (36, 30), 4, dict(interp_direct=1)),
    ((20, 12, 16), (40, 20, 30), 6, {}),                     # 8 x 8 x 16 tiles cut on every axis
    ((10, 18, 22), (18, 36, 40), 5, dict(grid_waves=1, grid_chunk=64, weight_table=1)),
    ((12, 14, 20), (20, 27 * 2, 36), 4, dict(fuse_reduce=1, grid_chunk=128)),
    ((12, 14, 20), (20, 27 * 2, 36), 7, dict(grid_mfma=3)),
    ((12, 10, 9 * 2), (18, 20, 18), 6, {}),                  # an axis too short for cut tiles
])
def test_pair_on_cut_tiles(orc, dev, N, K, J, options):
    from paper_1710_03197_amd import Plan
    r = np.random.default_rng(sum(K) + J)
    d, M, B = len(N), 3001, 4
    om = r.uniform(-np.pi, np.pi, (M, d))
    om[: M // 4] = r.normal(0.0, 0.1, (M // 4, d))
    om[M // 4: M // 3] = np.pi - r.uniform(0, 0.2, (M // 3 - M // 4, d))  # windows across the wrap
    om = om.astype(np.float32)
    x = (r.standard_normal((B,) + N) + 1j * r.standard_normal((B,) + N)).astype(np.complex64)
    y = (r.standard_normal((B, M)) + 1j * r.standard_normal((B, M))).astype(np.complex64)
    mm = options.get("interpolator")
    fwd, adj = (orc.minmax_forward, orc.minmax_adjoint) if mm else (orc.forward, orc.adjoint)
    with Plan(torch.from_numpy(om).to(dev), N, K, J, options=options) as p:
        f = p.forward_batched(torch.from_numpy(x).to(dev)).cpu().numpy()
        a = p.adjoint_batched(torch.from_numpy(y).to(dev)).cpu().numpy()
        a0 = p.adjoint(torch.from_numpy(y[0]).to(dev)).cpu().numpy()
        h = None if mm else p.stage_vh(torch.from_numpy(y[0]).to(dev)).cpu().numpy()
    tol = TOL_NO_OVERSAMPLING if any(n == k for n, k in zip(N, K)) else TOL
    for b in (0, B - 1):
        assert rel_l2(f[b], fwd(x[b], om, N, K, J)) < tol
        assert rel_l2(a[b], adj(y[b], om, N, K, J)) < tol
    assert rel_l2(a0, adj(y[0], om, N, K, J)) < tol
    if h is not None:
        assert rel_l2(h, orc.grid(y[0], om, N, K, J)) < TOL


def test_column_form_on_cut_tiles(orc, dev):
    from paper_1710_03197_amd import Plan
    r = np.random.default_rng(5)
    N, K, M, B = (50, 82), (100, 162), 9001, 5
    om = r.uniform(-np.pi, np.pi, (M, 2)).astype(np.float32)
    y = (r.standard_normal((B, M)) + 1j * r.standard_normal((B, M))).astype(np.complex64)
    for chunk in (64, 512):
        with Plan(torch.from_numpy(om).to(dev), N, K, 6, options=dict(grid_chunk=chunk)) as p:
            a = p.adjoint_batched(torch.from_numpy(y).to(dev)).cpu().numpy()
        for b in (0, B - 1):
            assert rel_l2(a[b], orc.adjoint(y[b], om, N, K, 6)) < TOL
