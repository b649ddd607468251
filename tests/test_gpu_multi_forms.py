"""Multi-problem launches at sizes where the gridding takes the grids as matrix
columns, with four wavefronts per work item or, in full launches, one: each
problem's results are bit for bit those of its own single plan, whatever shares
the launch, and match the FP64 oracle."""
import numpy as np
import pytest

from nudft import rel_l2
from paper_1710_03197_amd import data

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


# N, coils, samples, options.  Five coils and more and 1024 workgroups of four grids
# and more: work items from part of a batch of 64 samples to 32 batches, one and
# two groups of eight grids, the last one partly filled, tiles cut unevenly,
# on-the-fly windows; and one problem that stays with the row-tile form.
PROBLEMS = [((192, 160), 8, 40000, {}),
            ((100, 180), 13, 30000, dict(grid_chunk=2048)),
            ((96, 96), 9, 20000, dict(grid_chunk=64, weight_table=-1)),
            ((256, 256), 8, 30000, dict(grid_chunk=1536, presort=1, fuse_reduce=2)),
            ((32, 32), 2, 5000, {})]


@pytest.mark.parametrize("which", [[0], [1, 2], [0, 1, 2, 3, 4], [3] * 20 + [0, 1]],
                         ids=["one", "two", "five", "many"])
def test_bits_are_those_of_single_plans(orc, dev, which):
    from paper_1710_03197_amd.plan import MultiPlan, Plan
    r = np.random.default_rng(len(which))
    cn = lambda *s: torch.from_numpy((r.standard_normal(s) + 1j * r.standard_normal(s)).astype(np.complex64)).to(dev)  # noqa: E731
    probs = []
    for k in which:
        N, C, M, options = PROBLEMS[k]
        om = torch.from_numpy(data.spiral_2d(M, 8, 11 + k)).to(dev)
        probs.append(dict(om=om, N=N, coils=cn(C, *N), options=options, x=cn(*N), y=cn(C, om.shape[0])))
    mp = MultiPlan([{k: p[k] for k in ("om", "N", "coils", "options")} for p in probs], J=6)
    ys = mp.forward([p["x"] for p in probs])
    xs = mp.adjoint([p["y"] for p in probs])
    torch.cuda.synchronize()
    for p, y, x in zip(probs, ys, xs):
        with Plan(p["om"], p["N"], None, 6, coils=p["coils"], options=p["options"]) as sp:
            assert torch.equal(sp.forward(p["x"]), y)
            assert torch.equal(sp.adjoint(p["y"]), x)
    p, x = probs[-1], xs[-1].cpu().numpy()
    om, K = p["om"].cpu().numpy(), tuple(2 * n for n in p["N"])
    xo = orc.adjoint_coils(p["y"].cpu().numpy(), p["coils"].cpu().numpy(), om, p["N"], K, 6)
    assert rel_l2(x, xo) < 1e-5
    mp.close()
