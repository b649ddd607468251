"""Kaiser-Bessel windows read from the plan's table and evaluated on the fly
(weight_table = 1 and -1) give the same bits in every sample kernel that has
both forms, and both match the FP64 oracle."""
import numpy as np
import pytest

from nudft import rel_l2

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# N, J, coils, samples, options: the staged gather in 1D to 3D at the narrowest,
# odd and widest windows; gridding on the vector ALUs, by row tiles, with the
# grids as columns (four wavefronts), by blocks with four and one wavefront
CASES = [
    ((40,), 6, 0, 700, {}),
    ((32, 48), 2, 0, 3000, {}),
    ((32, 48), 6, 0, 3000, {}),
    ((50, 36), 7, 2, 3000, {}),
    ((32, 32), 8, 0, 3000, dict(grid_mfma=2)),
    ((48, 64), 5, 3, 12000, {}),
    ((48, 64), 8, 9, 6000, {}),
    ((16, 20, 24), 6, 0, 5000, {}),
    ((16, 16, 16), 8, 0, 5000, dict(grid_waves=1)),
    ((16, 16, 16), 3, 0, 5000, dict(grid_mfma=3)),
    ((12, 12, 12), 4, 0, 3000, dict(grid_mfma=2)),
    ((18, 20, 30), 7, 2, 4000, {}),
]


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


@pytest.mark.parametrize("N,J,C,M,options", CASES)
def test_table_and_on_the_fly_agree(orc, dev, N, J, C, M, options):
    from paper_1710_03197_amd import Plan
    r = np.random.default_rng(M + J)
    K = tuple(2 * n for n in N)
    om = (r.standard_normal((M, len(N))) * 1.2).clip(-np.pi, np.pi).astype(np.float32)  # crowded at the centre
    cn = lambda *s: (r.standard_normal(s) + 1j * r.standard_normal(s)).astype(np.complex64)  # noqa: E731
    x, y, coils = cn(*N), cn(*((C, M) if C else (M,))), cn(C, *N) if C else None
    t = [None if v is None else torch.from_numpy(v).to(dev) for v in (om, x, y, coils)]
    got = []
    for table in (1, -1):
        with Plan(t[0], N, K, J, coils=t[3], options=dict(options, weight_table=table)) as p:
            got.append([v.cpu().numpy() for v in (p.forward(t[1]), p.adjoint(t[2]), p.density_compensation(2))])
    for a, b in zip(*got):
        assert np.array_equal(a, b)
    yo = orc.forward_coils(x, coils, om, N, K, J) if C else orc.forward(x, om, N, K, J)
    xo = orc.adjoint_coils(y, coils, om, N, K, J) if C else orc.adjoint(y, om, N, K, J)
    assert rel_l2(got[1][0], yo) < 1e-5
    assert rel_l2(got[1][1], xo) < 1e-5
