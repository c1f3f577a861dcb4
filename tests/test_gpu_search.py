"""The density by single waves that walk the octree, where groups are plenty, and
the lists of small trees.
"""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2003_10850_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BOX = (0.0, 0.0, 0.0, 1.0)


def dev_t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.mark.parametrize("pad", [(), (0, 9, 1)])
@pytest.mark.parametrize("nodes", [1, 700, 2048, 2049])
def test_lists_of_small_trees(nodes, pad):
    # a list by one workgroup up to 2048 nodes, by three launches above: the most
    # particles in leaves of one with so many nodes, or the fewest with more
    from paper_2003_10850_amd import ops
    rng = np.random.default_rng(nodes)
    pos = rng.random((2048, 3)).astype(np.float32)
    h = (0.05 + 0.2 * rng.random(2048)).astype(np.float32)
    u, rho = rng.uniform(0.5, 1.5, (2, 2048)).astype(np.float32)
    mass = np.full(2048, 1e-3, np.float32)
    p = inputs.Params(n_ngb=32.0, leaf_size=1)
    c = ops.Context(torch.device("cuda", 0))

    def tree(m):
        off = np.concatenate([[0], np.cumsum((m,) + pad)])
        n = int(off[-1])
        return off, ops.Tree(c, dev_t(pos[:n]), dev_t(mass[:n]), None, [BOX] * (len(off) - 1), p,
                             snap_off=[int(x) for x in off])

    lo, hi = 1, 2000  # nodes(lo) <= 2048 (or the least there is) < nodes(hi)
    while hi - lo > 1:
        m = (lo + hi) // 2
        lo, hi = (m, hi) if tree(m)[1].info(1)[1] <= min(nodes, 2048) else (lo, m)
    off, t = tree(hi if nodes > 2048 else lo)
    n = int(off[-1])
    print(f"small {off} nodes={t.info(1)[1]}", flush=True)
    assert (t.info(1)[1] > 2048) == (nodes > 2048)
    nngb = ops.density(t, h=dev_t(h[:n]), solve_h=False)["nngb"].cpu().numpy()
    pairs = ops.conduction(t, dev_t(u[:n]), dev_t(h[:n]), dev_t(rho[:n]), 1.0, 0.0)["npairs"]
    pairs = pairs.cpu().numpy()
    pr = dataclasses.replace(p, flags=0)
    for a, b in zip(off[:-1], off[1:]):
        if a == b:
            continue
        r, H = slice(a, b), h[a:b].astype(np.float64)
        o = oracle.Tree(pos[r].astype(np.float64), mass[r].astype(np.float64), BOX, gas_only=True,
                        type=np.zeros(b - a, np.uint8))
        ref = oracle.density(o, pr, h=H, solve_h=False)["nngb"]
        np.testing.assert_array_equal(nngb[r], ref)
        ref = oracle.conduction(o, pr, u[r], H, rho[r], 1.0, 0.0)["npairs"]
        np.testing.assert_array_equal(pairs[r], ref)


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
