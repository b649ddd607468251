"""2D staged gather: tiles whose samples fill one workgroup, one work item or just
more, regions wider than the workgroup, against the FP64 oracle."""
import numpy as np
import pytest

from nudft import rel_l2

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TOL = 1e-5  # the suite's bar against the oracle


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


@pytest.mark.parametrize("grids", [1, 3])
@pytest.mark.parametrize("M", [1, 127, 128, 129, 255, 256, 257, 511, 513])
def test_one_full_tile(orc, dev, M, grids):
    from paper_1710_03197_amd import Plan
    r = np.random.default_rng(M)
    om = r.uniform(0.02, 0.3, (M, 2)).astype(np.float32)  # 16 cells of 64 are 1.57 wide
    x = (r.standard_normal((grids, 32, 32)) + 1j * r.standard_normal((grids, 32, 32))).astype(np.complex64)
    with Plan(torch.from_numpy(om).to(dev), (32, 32), (64, 64), 6) as p:
        f = p.forward_batched(torch.from_numpy(x).to(dev)).cpu().numpy()
    for b in range(grids):
        assert rel_l2(f[b], orc.forward(x[b], om, (32, 32), (64, 64), 6)) < TOL


@pytest.mark.parametrize("merge", [2, 8, 15, 16, 17, 32])
def test_regions_wider_than_the_workgroup(orc, dev, merge):
    from paper_1710_03197_amd import Plan
    r = np.random.default_rng(merge)
    N, K, J, M = (64, 256), (128, 512), 6, 801  # few samples a tile: runs of `merge` tiles of 16 cells share an item
    om = r.uniform(-np.pi, np.pi, (M, 2)).astype(np.float32)
    x = (r.standard_normal(N) + 1j * r.standard_normal(N)).astype(np.complex64)
    with Plan(torch.from_numpy(om).to(dev), N, K, J, options=dict(interp_merge=merge)) as p:
        f = p.forward(torch.from_numpy(x).to(dev)).cpu().numpy()
    assert rel_l2(f, orc.forward(x, om, N, K, J)) < TOL
