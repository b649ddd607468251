"""The 2D gridding that takes the grids as matrix columns, at the sizes where the
plan takes it (five grids and more, 1024 workgroups of four grids and more): the
edges of tiles, windows, grid groups and batches, against the row-tile form and
the FP64 oracle."""
import numpy as np
import pytest

from nudft import rel_l2

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TOL = 1e-5        # the suite's bound against the oracle
# Two summation orders of the same float32 products: a sum of n terms differs by
# about sqrt(n) eps of its largest partial sums, n up to 11003 in one cell.
TOL_FORMS = 2e-6


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


# grids, N, K, J, samples, options: at least 172 work items where a chunk holds 64 samples
@pytest.mark.parametrize("B,N,K,J,M,options", [
    (24, (8, 8), (16, 16), 8, 11003, dict(grid_chunk=64)),                   # one tile on both axes
    (24, (8, 24), (16, 48), 6, 11003, dict(grid_chunk=64)),                  # one tile on axis 0
    (25, (32, 40), (64, 80), 6, 11003, dict(grid_chunk=64, weight_table=-1)),
    (29, (24, 24), (48, 48), 5, 11003, dict(grid_chunk=64)),
    (204, (16, 24), (32, 48), 4, 11003, dict(presort=1, fuse_reduce=2)),     # eight batches an item
    (160, (32, 32), (64, 64), 8, 11003, dict(grid_chunk=300)),               # part of a batch at the end
    (24, (24, 32), (48, 64), 11, 11003, dict(grid_chunk=64)),
    (24, (32, 32), (64, 64), 16, 11003, dict(grid_chunk=64)),
    (24, (24, 32), (48, 64), 6, 11003, dict(grid_chunk=64, interpolator=1)),
    (24, (24, 32), (48, 64), 2, 11003, dict(grid_chunk=64)),
    (5, (256, 300), (512, 600), 6, 2003, {}),                                # tiles cut unevenly, few samples
    (33, (320, 320), (640, 640), 6, 4001, {}),                               # one wavefront an item
])
def test_column_form_matches_row_tiles_and_oracle(orc, dev, B, N, K, J, M, options):
    from paper_1710_03197_amd import Plan
    r = np.random.default_rng(B * 100 + J)
    om = r.uniform(-np.pi, np.pi, (M, 2))
    om[: M // 3] = r.normal(0.0, 0.1, (M // 3, 2))   # a crowded centre: split tiles
    om[: M // 10] += 2 * np.pi * r.integers(-1, 2, (M // 10, 2))  # wrapped coordinates
    om = om.astype(np.float32)
    ys = (r.standard_normal((B, M)) + 1j * r.standard_normal((B, M))).astype(np.complex64)
    out = {}
    for mfma in (0, 3):
        with Plan(torch.from_numpy(om).to(dev), N, K, J, options=dict(options, grid_mfma=mfma)) as p:
            y = torch.from_numpy(ys).to(dev)
            out[mfma] = p.adjoint_batched(y).cpu().numpy()
            assert np.array_equal(p.adjoint_batched(y).cpu().numpy(), out[mfma])  # reproducible
    assert not np.array_equal(out[0], out[3])  # two forms, not one twice
    for b in range(B):
        assert rel_l2(out[0][b], out[3][b]) < TOL_FORMS
    adj = orc.minmax_adjoint if options.get("interpolator") else orc.adjoint
    for b in (0, B - 1):
        assert rel_l2(out[0][b], adj(ys[b], om, N, K, J)) < TOL
