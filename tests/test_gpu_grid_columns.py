"""Gridding of several grids on the matrix cores with the grids as columns
(2D, 16 x 16 tiles), against the row-tile form of the same plan and the FP64
oracle: numbers of grids around a column group, taps around the instance
widths, the window table, split tiles, one-tile axes and wrapped windows."""
import numpy as np
import pytest

from nudft import rel_l2

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TOL = 1e-5       # the suite's bar against the oracle
TOL_FORMS = 2e-6  # two float32 summation orders of the same products, each within 1e-6


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def _points(M, r):
    om = r.uniform(-np.pi, np.pi, (M, 2))
    om[: M // 3] = r.normal(0.0, 0.1, (M // 3, 2))   # a crowded centre: split tiles
    om[: M // 10] += 2 * np.pi * r.integers(-1, 2, (M // 10, 2))  # wrapped coordinates
    return om.astype(np.float32)


@pytest.mark.parametrize("B,N,K,J,options", [
    (3, (32, 40), (64, 80), 6, {}),
    (8, (24, 32), (48, 64), 6, dict(weight_table=1)),
    (9, (24, 24), (48, 48), 5, dict(grid_chunk=64)),
    (17, (16, 24), (32, 48), 4, dict(presort=1, fuse_reduce=2)),
    (4, (8, 24), (16, 48), 6, dict(weight_table=1, grid_chunk=128)),     # one tile on axis 0
    (3, (8, 8), (16, 16), 8, dict(weight_table=1)),                      # one tile on both
    (5, (32, 32), (64, 64), 8, {}),
    (3, (32, 24), (64, 48), 11, {}),
    (3, (32, 32), (64, 64), 16, dict(grid_chunk=256)),
    (4, (24, 32), (48, 64), 6, dict(interpolator=1)),
    (3, (24, 32), (48, 64), 2, {}),
])
def test_column_form_matches_row_tiles_and_oracle(orc, dev, B, N, K, J, options):
    from paper_1710_03197_amd import Plan
    r = np.random.default_rng(B * 100 + J)
    M = 4001 if B > 8 else 11003  # enough samples times grids for the column form
    om = _points(M, r)
    ys = (r.standard_normal((B, M)) + 1j * r.standard_normal((B, M))).astype(np.complex64)
    out = {}
    for mfma in (0, 3):
        opts = dict(options, tile=(16, 16), grid_mfma=mfma)
        with Plan(torch.from_numpy(om).to(dev), N, K, J, options=opts) as p:
            y = torch.from_numpy(ys).to(dev)
            out[mfma] = p.adjoint_batched(y).cpu().numpy()
            again = p.adjoint_batched(y).cpu().numpy()
        assert np.array_equal(again.view(np.uint32), out[mfma].view(np.uint32))  # reproducible
    for b in range(B):
        assert rel_l2(out[0][b], out[3][b]) < TOL_FORMS
    adj = orc.minmax_adjoint if options.get("interpolator") else orc.adjoint
    for b in (0, B - 1):
        assert rel_l2(out[0][b], adj(ys[b], om, N, K, J)) < TOL


@pytest.mark.parametrize("C", [3, 8])
def test_column_form_in_a_multi_problem_launch(orc, dev, C):
    """One wavefront per item (the multi-problem form), two problems of one launch."""
    from paper_1710_03197_amd.plan import MultiPlan
    r = np.random.default_rng(C)
    probs, ys, want = [], [], []
    for N, M in (((32, 32), 11003), ((48, 24), 12001)):
        K = (2 * N[0], 2 * N[1])
        om = _points(M, r)
        coils = (r.standard_normal((C,) + N) + 1j * r.standard_normal((C,) + N)).astype(np.complex64)
        y = (r.standard_normal((C, M)) + 1j * r.standard_normal((C, M))).astype(np.complex64)
        probs.append(dict(om=torch.from_numpy(om).to(dev), N=N, K=K, coils=torch.from_numpy(coils).to(dev),
                          options=dict(tile=(16, 16), grid_chunk=512)))
        ys.append(torch.from_numpy(y).to(dev))
        want.append(orc.adjoint_coils(y, coils, om, N, K, 6))
    m = MultiPlan(probs, 6)
    got = [v.cpu().numpy() for v in m.adjoint(ys)]
    m.close()
    for g, w in zip(got, want):
        assert rel_l2(g, w) < TOL
