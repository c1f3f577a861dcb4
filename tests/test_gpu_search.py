"""The density by single waves that walk the octree, where groups are plenty.
"""
import numpy as np
import pytest

from paper_2003_10850_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def dev_t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.mark.parametrize("fp64", [False, True])
def test_density_without_a_team_has_the_same_bits(fp64):
    # 1.9e6 targets in unsplit groups take no team; the first 2^15 in tree order
    # form the same groups and take teams of 12 (FP64 positions: 16)
    from paper_2003_10850_amd import g3, ops
    n = 1900000
    w = inputs.uniform(n=n, seed=23)
    p = inputs.Params(n_ngb=48.0)
    c = ops.Context(torch.device("cuda", 0))
    c.set_tuning(g3.G3_TUNE_DENSITY, 128, -1)
    tree = ops.Tree(c, dev_t(w.pos if fp64 else w.pos.astype(np.float32)),
                    dev_t(w.mass.astype(np.float32)), None, tuple(w.box), p)
    few = torch.sort(tree.export(1)["order"][: 1 << 15]).values
    g = torch.Generator(device="cuda").manual_seed(2)
    h = (2.25 * n ** (-1.0 / 3.0) * (0.8 + 0.4 * torch.rand(n, generator=g, device="cuda"))).to(
        torch.float64 if fp64 else torch.float32)
    a, b = ops.density(tree, h=h), ops.density(tree, h=h, active=few)
    at = few.long()
    for k in a:
        assert torch.equal(a[k][at], b[k][at]), k
    assert c.nonconverged() == 0
