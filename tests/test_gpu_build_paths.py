"""The octree build on both sides of its size rules (one-workgroup sort and
moments, subtree and top moments, node-depth windows at snapshot and block
edges), against the oracle's tree: members, keys and topology exact, moments to
FP64 rounding; and refits of the same trees.
"""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BOX = (0.0, 0.0, 0.0, 1.0)


def dev_t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.fixture(scope="module")
def ctx():
    from paper_2003_10850_amd import ops
    return ops.Context(torch.device("cuda", 0))


def points(kind, n):
    rng = np.random.default_rng(n)
    if kind == "halo":
        pos = 0.5 + 0.01 * rng.normal(0, 1, (n, 3))
    elif kind == "chains":  # pairs 1e-6 apart: chains to the deepest levels
        pos = rng.random((n, 3))
        pos[1::2] = pos[: n - n // 2][: len(pos[1::2])] + 1e-6
    elif kind == "coincident":  # a deepest leaf larger than a subtree
        pos = rng.random((n, 3))
        pos[: n // 2] = 0.3
    else:
        pos = rng.random((n, 3))
    return np.clip(pos, 0.0, 1.0 - 1e-6)


def compare(tree, which, pos, mass, typ, leaf, k=None):
    got = {q: v.cpu().numpy() for q, v in tree.export(which).items()}
    ref = oracle.Tree(pos.astype(np.float64), mass.astype(np.float64), BOX, type=typ,
                      leaf_size=leaf, gas_only=which == 1).export()
    np.testing.assert_array_equal(got["order"], ref["order"])
    np.testing.assert_array_equal(got["keys"].view(np.uint64), ref["keys"])
    for q in ("start", "count", "level", "skip"):
        np.testing.assert_array_equal(got[q], ref[q], err_msg=q)
    np.testing.assert_allclose(got["mass"], ref["mass"], rtol=1e-12)
    np.testing.assert_allclose(got["com"], ref["com"], rtol=1e-12, atol=1e-12)


@pytest.mark.parametrize("leaf", [1, 8, 64])
@pytest.mark.parametrize("kind,n", [("uniform", 1), ("uniform", 2), ("uniform", 257),
                                    ("uniform", 8192), ("uniform", 8193), ("halo", 12000),
                                    ("chains", 9001), ("coincident", 6000),
                                    ("halo", 70001)])
def test_build_against_oracle(ctx, kind, n, leaf):
    from paper_2003_10850_amd import inputs, ops
    print(f"build {kind} n={n} leaf={leaf}", flush=True)
    pos = points(kind, n).astype(np.float32)
    rng = np.random.default_rng(1)
    mass = rng.uniform(0.5, 1.5, n).astype(np.float32)
    typ = (rng.random(n) < 0.4).astype(np.uint8)
    p = inputs.Params(leaf_size=leaf)
    tree = ops.Tree(ctx, dev_t(pos), dev_t(mass), dev_t(typ), BOX, p)
    for which in (0, 1):
        if (typ == 0).any() or which == 0:
            compare(tree, which, pos, mass, typ, leaf)
    # a second build into the same object, smaller, and a refit of it
    m = max(1, n // 3)
    tree.build(dev_t(pos[:m]), dev_t(mass[:m]), None, BOX)
    compare(tree, 1, pos[:m], mass[:m], np.zeros(m, np.uint8), leaf)
    before = tree.export(0)
    tree.refit(dev_t(pos[:m]), dev_t(mass[:m]))
    after = tree.export(0)
    for q in before:
        assert torch.equal(before[q], after[q]), q


@pytest.mark.parametrize("sizes", [[5, 0, 300, 1, 9000], [300] * 70])
def test_forest_edges(ctx, sizes):
    # snapshots shorter than a block and than a window of members
    from paper_2003_10850_amd import inputs, ops
    off = np.concatenate([[0], np.cumsum(sizes)])
    pos = np.concatenate([points("halo", max(m, 1))[:m] for m in sizes]).astype(np.float32)
    n = len(pos)
    mass = np.full(n, 1.0 / n, np.float32)
    tree = ops.Tree(ctx, dev_t(pos), dev_t(mass), None, [BOX] * len(sizes), inputs.Params(),
                    snap_off=off)
    for which in (0, 1):
        got = {q: v.cpu().numpy() for q, v in tree.export(which).items()}
        m0 = n0 = 0
        for k, m in enumerate(sizes):
            if m == 0:
                continue
            r = slice(off[k], off[k + 1])
            ref = oracle.Tree(pos[r].astype(np.float64), mass[r].astype(np.float64), BOX,
                              type=np.zeros(m, np.uint8)).export()
            nn = len(ref["start"])
            np.testing.assert_array_equal(got["order"][m0:m0 + m] - off[k], ref["order"])
            np.testing.assert_array_equal(got["start"][n0:n0 + nn] - m0, ref["start"])
            np.testing.assert_array_equal(got["skip"][n0:n0 + nn] - n0, ref["skip"])
            np.testing.assert_allclose(got["com"][n0:n0 + nn], ref["com"], rtol=1e-12, atol=1e-12)
            m0, n0 = m0 + m, n0 + nn
        assert m0 == len(got["order"]) and n0 == len(got["start"])


@pytest.mark.parametrize("n", [1, 2047, 2048, 2049, 16383, 16384, 16385, 40960])
def test_target_lists_at_the_edges_of_the_scans(n):
    # one tile, one workgroup, two launches: the listed rows are computed (the
    # same counts as in a call for every member), the others stay
    from paper_2003_10850_amd import inputs, ops
    c = ops.Context(torch.device("cuda", 0))
    g = torch.Generator(device="cuda").manual_seed(n)
    pos, mass = torch.rand(n, 3, generator=g, device="cuda"), torch.ones(n, device="cuda")
    tree = ops.Tree(c, pos, mass, None, (0.0, 0.0, 0.0, 1.0), inputs.Params(n_ngb=16.0))
    every = ops.gravity(tree)["nterms"]
    h = torch.full((n,), 0.9 * n ** (-1.0 / 3.0), device="cuda")
    nngb = ops.density(tree, h=h, solve_h=False)["nngb"]
    for part in (0.0, 0.3, 1.0):
        on = torch.rand(n, generator=g, device="cuda") < part
        on[-1] = True
        act = on.nonzero().flatten().int().flip(0).contiguous()
        for a, b in ((ops.gravity(tree, active=act)["nterms"], every),
                     (ops.density(tree, h=h, active=act, solve_h=False)["nngb"], nngb)):
            assert torch.equal(a, torch.where(on, b, torch.zeros_like(b)))


def test_scans_of_more_than_four_thousand_tiles():
    # 8.4e6 members: the tiles' sums are scanned by themselves first
    from paper_2003_10850_amd import inputs, ops
    n = 4096 * 2048 + 4321
    c = ops.Context(torch.device("cuda", 0))
    g = torch.Generator(device="cuda").manual_seed(8)
    pos, mass = torch.rand(n, 3, generator=g, device="cuda"), torch.ones(n, device="cuda")
    typ = torch.zeros(n, dtype=torch.uint8, device="cuda")
    typ[: n // 100] = 1  # the gas octree keeps more than 4096 tiles less one
    tree = ops.Tree(c, pos, mass, typ, (0.0, 0.0, 0.0, 1.0), inputs.Params(theta=1.0))
    order = tree.export(1)["order"]
    assert torch.equal(order.sort().values, torch.arange(n // 100, n, device="cuda").int())
    act = torch.tensor([n - 1, 0, 4096 * 2048, 17], dtype=torch.int32, device="cuda")
    r = ops.gravity(tree, active=act)
    on = torch.zeros(n, dtype=torch.bool, device="cuda")
    on[act.long()] = True
    assert torch.equal(r["nterms"] > 0, on)
