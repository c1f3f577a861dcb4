"""The ways a group's neighbours are found beside the plain team search (a wave
that walks the octree by itself, the deep search of long lists and of few targets
among many members, lists at the ends of walk_leaf), at the sizes where they can
go wrong, against the oracle or the other way; and team sizes that no other test
takes.

Tolerances: counts exact; the density within 2e-6 of the FP64 sums (FP32 terms
of one sign, each good to a few 1e-7, added with compensation), accelerations,
rates and gradients within 1e-5 of the L1 sum of their terms, as the parity tests
have.
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


def gas_set(kind, n, rng):
    pos = rng.random((n, 3))
    if kind == "halo":
        pos = np.clip(0.5 + 0.05 * rng.normal(0, 1, (n, 3)), 0.0, 1.0 - 1e-6)
    elif kind == "line":
        pos[:, 1:] = 0.5 + 1e-2 * (pos[:, 1:] - 0.5)
    return pos


def within(what, got, ref, S):
    # 1e-5 of the L1 sum, and 1e-7 of its median for what only the edge of the
    # support feeds (the adjoint tests' bar)
    err, floor = np.abs(got - ref), 1e-7 * np.median(S[S > 0]) if np.any(S > 0) else 0.0
    assert (err <= 1e-5 * S + floor).all(), (what, (err / (1e-5 * S + floor + 1e-300)).max())


# deep by the targets: 64 or a few thousand of 2e5 (terminals of 16 and 64
# members: 2 to 7 blocks); deep by the list: all of them with terminals of 4; not
# deep: terminals of up to 4096 members, nodes of more than 65535; deep in a tree
# of fewer than 2048 nodes
@pytest.mark.parametrize("kind,n,sizes,leaf,few,fp64", [
    ("uniform", 200000, None, 16, 1, False), ("uniform", 200000, None, 16, 64, False),
    ("uniform", 200000, None, 64, 3001, False), ("line", 200000, None, 16, 200, False),
    ("uniform", 200000, None, 16, 130, True), ("uniform", 200000, None, 4, None, False),
    ("uniform", 200000, None, 4, None, True), ("uniform", 190011, [10, 100000, 1, 90000], 2, 900, False),
    ("uniform", 190011, [10, 100000, 1, 90000], 2, None, False),
    ("uniform", 140000, None, 4096, None, False), ("uniform", 3000, None, 1, 40, False)])
def test_searches_against_oracle(kind, n, sizes, leaf, few, fp64):
    from paper_2003_10850_amd import g3, ops
    print(f"search {kind} n={n} leaf={leaf} few={few} fp64={fp64}", flush=True)
    rng = np.random.default_rng(n + leaf)
    ft = np.float64 if fp64 else np.float32
    pos = gas_set(kind, n, rng).astype(ft)
    mass = np.full(n, 1.0 / n, np.float32)
    vel = rng.normal(0, 0.1, (n, 3)).astype(np.float32)
    u, rho, om = [rng.uniform(0.5, 1.5, n).astype(np.float32) for _ in range(3)]
    h = (2.2 * n ** (-1.0 / 3.0) * rng.uniform(0.7, 1.3, n)).astype(ft)
    if kind == "line":
        h *= 0.1
    off = [0, n] if sizes is None else list(np.concatenate([[0], np.cumsum(sizes)]))
    p = inputs.Params(n_ngb=48.0)
    c = ops.Context(torch.device("cuda", 0))
    for k in (g3.G3_TUNE_DENSITY, g3.G3_TUNE_HYDRO):
        c.set_tuning(k, leaf, -1)
    tree = ops.Tree(c, dev_t(pos), dev_t(mass), None, BOX if sizes is None else [BOX] * len(sizes),
                    p, snap_off=None if sizes is None else off)
    act = np.arange(n) if few is None else np.sort(rng.choice(n, few, replace=False))
    a = None if few is None else dev_t(act.astype(np.int32))
    got = dict(ops.density(tree, h=dev_t(h), active=a, solve_h=False))
    got |= {"f_" + k: v for k, v in ops.hydro_force(
        tree, dev_t(vel), dev_t(u), dev_t(h), dev_t(rho), dev_t(om), active=a).items()}
    if not fp64:
        got |= {"c_" + k: v for k, v in ops.conduction(
            tree, dev_t(u), dev_t(h), dev_t(rho), 1.0, 0.0, active=a).items()}
        got |= {"v_" + k: v for k, v in ops.velocity_gradients(
            tree, dev_t(vel), dev_t(h), dev_t(rho), dev_t(om), active=a).items()}
    got = {k: v.cpu().numpy() for k, v in got.items()}
    pr = dataclasses.replace(p, flags=oracle.FLAG_FP64_DECISIONS if fp64 else 0)
    for lo, hi in zip(off[:-1], off[1:]):
        r = slice(lo, hi)
        ids = act[(act >= lo) & (act < hi)] - lo
        if ids.size == 0:
            continue
        ids = ids if ids.size < 20000 else np.sort(rng.choice(ids, 20000, replace=False))
        t = oracle.Tree(pos[r].astype(np.float64), mass[r].astype(np.float64), BOX, gas_only=True,
                        type=np.zeros(hi - lo, np.uint8))
        H = h[r].astype(np.float64)

        def rel(key, ref, val, S):
            d = got[key][r][ids] - ref[val][ids]
            e = np.linalg.norm(d.reshape(len(ids), -1), axis=1)
            s = ref[S][ids]
            assert (e[s > 0] / s[s > 0]).max(initial=0) < 1e-5, key

        ref = oracle.density(t, pr, active=ids, h=H, solve_h=False)
        np.testing.assert_array_equal(got["nngb"][r][ids], ref["nngb"][ids])
        assert (np.abs(got["rho"][r][ids] / ref["rho"][ids] - 1.0)).max() < 2e-6
        ref = oracle.hydro(t, pr, vel[r], u[r], H, rho[r], om[r], active=ids)
        np.testing.assert_array_equal(got["f_npairs"][r][ids], ref["npairs"][ids])
        rel("f_acc", ref, "acc", "S")
        if not fp64:
            ref = oracle.conduction(t, pr, u[r], H, rho[r], 1.0, 0.0, active=ids)
            np.testing.assert_array_equal(got["c_npairs"][r][ids], ref["npairs"][ids])
            rel("c_dudt", ref, "dudt", "S")
            ref = oracle.velgrad(t, pr, vel[r], H, rho[r], om[r], active=ids)
            within("v_div", got["v_div"][r][ids], ref["div"][ids], ref["S_div"][ids])
            within("v_curl", np.abs(got["v_curl"][r] - ref["curl"])[ids].max(1), 0.0,
                   ref["S_curl"][ids])


def test_adjoints_of_long_lists_against_oracle():
    # lists of 16 rows of windows: the deep adjoints, upstream gradients at every
    # particle (at few, the edge of the support alone would feed many entries)
    from paper_2003_10850_amd import g3, ops
    n = 2000000
    print(f"deep adjoints n={n}", flush=True)
    rng = np.random.default_rng(14)
    pos = rng.random((n, 3)).astype(np.float32)
    mass = ((0.5 + rng.random(n)) / n).astype(np.float32)
    h = (2.2 * n ** (-1.0 / 3.0) * rng.uniform(0.7, 1.3, n)).astype(np.float32)
    vel, ga = rng.normal(0, 0.1, (2, n, 3)).astype(np.float32)
    u, rho, om, gr, gd, go = rng.uniform(0.5, 1.5, (6, n)).astype(np.float32)
    p = inputs.Params(n_ngb=48.0)
    c = ops.Context(torch.device("cuda", 0))
    tree = ops.Tree(c, dev_t(pos), dev_t(mass), None, BOX, p)
    t = oracle.Tree(pos.astype(np.float64), mass.astype(np.float64), BOX, gas_only=True,
                    type=np.zeros(n, np.uint8))
    H = h.astype(np.float64)
    f = oracle.density(t, p, h=H, solve_h=False)
    new = lambda *k: torch.zeros(*k, device="cuda")
    D = {k: dev_t(v) for k, v in dict(
        h=h, u=u, rho=rho, om=om, vel=vel, ga=ga, gr=gr, gd=gd, go=go,
        fr=f["rho"].astype(np.float32), fd=f["drho_dh"].astype(np.float32)).items()}
    P = lambda *k: [D[x].data_ptr() for x in k]
    prm, st = g3.g3_params.of(p), torch.cuda.current_stream().cuda_stream
    o = dict(pos=new(n, 3), mass=new(n), h=new(n))
    g3.g3_density_backward(c.handle, tree.handle, n, 0, prm,
                           *P("h", "fr", "fd", "gr", "gd", "go"),
                           *[o[k].data_ptr() for k in ("pos", "mass", "h")], st)
    ref = oracle.density_backward(t, p, H, gr, gd, go)
    for k in o:
        within("density " + k, o[k].cpu().numpy(), ref[k], ref["S"][k])
    names = ("pos", "vel", "mass", "h", "u", "rho", "omega")
    o = {k: new(n, 3) if k in ("pos", "vel") else new(n) for k in names}
    g3.g3_hydro_force_backward(c.handle, tree.handle, n, 0, prm,
                               *P("vel", "u", "h", "rho", "om", "ga", "gd"),
                               *[o[k].data_ptr() for k in names], st)
    ref = oracle.hydro_backward(t, p, vel, u, H, rho, om, ga, gd)
    for k in names:
        within("hydro " + k, o[k].cpu().numpy(), ref[k], ref["S"][k])


@pytest.mark.parametrize("kind,leaf,few,fp64", [
    ("uniform", 16, 1, False), ("uniform", 64, 3000, False), ("halo", 16, 2500, False),
    ("halo", 64, 65, False), ("line", 16, 700, False), ("halo", 16, 1500, True),
    ("line", 64, 130, True)])
def test_the_deep_search_has_the_bits_of_the_plain_one(kind, leaf, few, fp64):
    # few targets of the first snapshot take the deep search, with the members of
    # the second one (whose groups are others) beside them the plain one
    from paper_2003_10850_amd import g3, ops
    print(f"deep {kind} leaf={leaf} few={few} fp64={fp64}", flush=True)
    m, pad = 200000, 20000
    n = m + pad
    rng = np.random.default_rng(leaf + few)
    ft = np.float64 if fp64 else np.float32
    pos = np.concatenate([gas_set(kind, m, rng), rng.random((pad, 3))]).astype(ft)
    h = (2.2 * m ** (-1.0 / 3.0) * rng.uniform(0.7, 1.3, n)).astype(ft)
    h *= dict(uniform=1.0, halo=0.4, line=0.1)[kind]
    c = ops.Context(torch.device("cuda", 0))
    for k in (g3.G3_TUNE_DENSITY, g3.G3_TUNE_HYDRO):
        c.set_tuning(k, leaf, -1)
    tree = ops.Tree(c, dev_t(pos), dev_t(np.full(n, 1.0 / m, np.float32)), None, [BOX] * 2,
                    inputs.Params(n_ngb=48.0), snap_off=[0, m, n])
    g = torch.Generator(device="cuda").manual_seed(2)
    R = lambda *s: torch.rand(*s, generator=g, device="cuda")
    vel, u, rho, om, hh = R(n, 3) - 0.5, 0.5 + R(n), 0.5 + R(n), 0.5 + R(n), dev_t(h)
    ids = np.sort(rng.choice(m, few, replace=False)).astype(np.int32)
    sets = [dev_t(ids), dev_t(np.concatenate([ids, np.arange(m, n, dtype=np.int32)]))]
    at = sets[0].long()
    calls = [lambda a: ops.density(tree, h=hh, active=a, solve_h=False),
             lambda a: ops.density(tree, h=hh, active=a),
             lambda a: ops.hydro_force(tree, vel, u, hh, rho, om, active=a)]
    for call in calls:
        x, y = [call(a) for a in sets]
        for k in x:
            assert torch.equal(x[k][at], y[k][at]), k
    if not fp64:
        x, y = [ops.conduction(tree, u, hh, rho, 1.0, 0.0, active=a) for a in sets]
        assert torch.equal(x["npairs"][at], y["npairs"][at])


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


@pytest.mark.parametrize("theta,eps", [(0.5, 1e-3), (0.8, 1e-3), (0.6, 0.0)])
def test_gravity_adjoint_without_a_team_adds_up(theta, eps):
    # the gradients are linear in the upstream ones: all of 10^6 targets (no team)
    # against two halves in tree order (teams of 4, the same groups), 1e-5 of the
    # largest (sums of a few hundred FP32 terms that cancel in part)
    from paper_2003_10850_amd import ops
    n = 1000000
    g = torch.Generator(device="cuda").manual_seed(9)
    R = lambda *s: torch.rand(*s, generator=g, device="cuda")
    pos, mass = R(n, 3), (0.5 + R(n)) / n
    c = ops.Context(torch.device("cuda", 0))
    tree = ops.Tree(c, pos, mass, None, BOX, inputs.Params(n_ngb=16.0, theta=theta, eps=eps))
    x = [pos.clone().requires_grad_(True), mass.clone().requires_grad_(True)]
    ups = (R(n, 3) - 0.5, R(n) - 0.5)
    order = tree.export(0)["order"]

    def grads(active):
        f = ops.gravity_ad(tree, x[0], x[1], active=active)
        return torch.autograd.grad(f, x, ups)

    cut = 64 * (n // 128)
    halves = [grads(torch.sort(q).values) for q in (order[:cut], order[cut:])]
    for a, b, s in zip(*halves, grads(None)):
        assert (a + b - s).abs().max() <= 1e-5 * s.abs().max()


@pytest.mark.parametrize("log_few,fp64", [(14, False), (17, False), (19, False), (14, True),
                                          (17, True), (19, True)])
def test_switches_in_teams_have_the_bits_of_single_waves(log_few, fp64):
    # 2^20 targets take no team; the first 2^14, 2^17 and 2^19 in tree order, the
    # same groups, take teams of 16 (and the deep search), 8 and 4
    from paper_2003_10850_amd import g3, ops
    n = 1 << 20
    g = torch.Generator(device="cuda").manual_seed(8)
    R = lambda *s: torch.rand(*s, generator=g, device="cuda")
    ft = torch.float64 if fp64 else torch.float32
    c = ops.Context(torch.device("cuda", 0))
    c.set_tuning(g3.G3_TUNE_HYDRO, 128, -1)
    tree = ops.Tree(c, R(n, 3).to(ft), torch.full((n,), 1.0 / n, device="cuda"), None, BOX,
                    inputs.Params(n_ngb=48.0))
    few = torch.sort(tree.export(1)["order"][: 1 << log_few]).values
    h = (2.25 * n ** (-1.0 / 3.0) * (0.8 + 0.4 * R(n))).to(ft)
    x = [R(n, 3) - 0.5, 0.5 + R(n), h, 0.5 + R(n), 0.5 + R(n), inputs.SwitchParams(alpha_u=0.7)]
    kw = dict(alpha=0.05 + R(n), balsara=R(n))
    a = ops.hydro_force_switches(tree, *x, **kw)
    b = ops.hydro_force_switches(tree, *x, **kw, active=few)
    at = few.long()
    for k in a:
        assert torch.equal(a[k][at], b[k][at]), k


@pytest.mark.parametrize("fp64", [False, True])
def test_gravity_with_the_inside_test_in_teams_of_4(fp64):
    # 1.4e6 targets in teams of 4 and 5600 of them in teams of 16: the same terms,
    # in sums of 64 that are cut elsewhere (64 roundings of 6e-8 at the worst, of
    # terms that mostly point one way)
    from paper_2003_10850_amd import ops
    n = 1400000
    g = torch.Generator(device="cuda").manual_seed(10)
    pos = torch.rand(n, 3, generator=g, device="cuda").to(torch.float64 if fp64 else torch.float32)
    tree = ops.Tree(ops.Context(torch.device("cuda", 0)), pos,
                    torch.full((n,), 1.0 / n, device="cuda"), None, BOX,
                    inputs.Params(theta=0.7, eps=1e-3))
    few = torch.arange(0, n, 250, dtype=torch.int32, device="cuda")
    a, b = ops.gravity(tree), ops.gravity(tree, active=few)
    at = few.long()
    assert torch.equal(a["nterms"][at], b["nterms"][at])
    for k in ("acc", "pot"):
        x, y = a[k][at].double(), b[k][at].double()
        assert float((x - y).abs().max()) <= 4e-6 * float(y.abs().max()), k
