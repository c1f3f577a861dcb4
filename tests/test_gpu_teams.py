"""Teams of waves that serve one group (density, hydro force): the terminal
list, its windows and the tiles at the sizes where they can go wrong, against
the oracle, and the same bits from every team size.

Tolerances: counts exact; the density within 2e-6 of the FP64 sums (FP32 terms
of one sign, each good to a few 1e-7, added with compensation), the hydro
acceleration within 1e-5 of the L1 sum of its terms, as the parity tests have.
"""
import numpy as np
import pytest

import oracle
from paper_2003_10850_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def dev_t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.fixture(scope="module")
def ctx():
    from paper_2003_10850_amd import ops
    return ops.Context(torch.device("cuda", 0))


def gas_set(kind, n, seed=3):
    rng = np.random.default_rng(seed)
    pos = rng.random((n, 3))
    if kind == "coincident":  # one leaf larger than a tile and a round
        pos[: n - n // 4] = 0.371
    elif kind == "line":  # wide groups, many terminals each
        pos[:, 1:] = 0.5 + 1e-3 * pos[:, 1:]
    return pos.astype(np.float32)


def check(ctx, pos, h, p, box, snap_off=None, act=None):
    """Density at given h and hydro of one set (or forest) with the oracle,
    snapshot by snapshot."""
    from paper_2003_10850_amd import ops
    n = len(pos)
    rng = np.random.default_rng(11)
    mass = np.full(n, 1.0 / n, np.float32)
    vel = rng.normal(0, 0.1, (n, 3)).astype(np.float32)
    u, rho, om = [rng.uniform(0.5, 1.5, n).astype(np.float32) for _ in range(3)]
    off = [0, n] if snap_off is None else list(snap_off)
    boxes = [box] if snap_off is None else box
    tree = ops.Tree(ctx, dev_t(pos), dev_t(mass), None, box, p, snap_off=snap_off)
    a_dev = None if act is None else dev_t(act)
    d = ops.density(tree, h=dev_t(h), active=a_dev, solve_h=False)
    f = ops.hydro_force(tree, dev_t(vel), dev_t(u), dev_t(h), dev_t(rho), dev_t(om), active=a_dev)
    act = np.arange(n) if act is None else act
    for k, b in enumerate(boxes):
        r = slice(off[k], off[k + 1])
        a = act[(act >= off[k]) & (act < off[k + 1])] - off[k]
        if a.size == 0:
            continue
        t = oracle.Tree(pos[r].astype(np.float64), mass[r].astype(np.float64), b,
                        type=np.zeros(off[k + 1] - off[k], np.uint8), gas_only=True)
        ref = oracle.density(t, p, active=a, h=h[r].astype(np.float64), solve_h=False)
        got = {q: v.cpu().numpy()[r] for q, v in {**d, **f}.items()}
        np.testing.assert_array_equal(got["nngb"][a], ref["nngb"][a])
        assert (np.abs(got["rho"][a] - ref["rho"][a]) / ref["rho"][a]).max() < 2e-6
        ry = oracle.hydro(t, p, vel[r], u[r], h[r].astype(np.float64), rho[r].astype(np.float64),
                          om[r].astype(np.float64), active=a)
        np.testing.assert_array_equal(got["npairs"][a], ry["npairs"][a])
        S = ry["S"][a]
        err = np.linalg.norm(got["acc"][a] - ry["acc"][a], axis=1)
        assert (err[S > 0] / S[S > 0]).max(initial=0) < 1e-5


@pytest.mark.parametrize("kind,n", [("uniform", 1), ("uniform", 2), ("uniform", 63),
                                    ("uniform", 65), ("uniform", 129), ("uniform", 4100),
                                    ("coincident", 5000), ("line", 3000)])
def test_sets_against_oracle(ctx, kind, n):
    print(f"teams {kind} n={n}", flush=True)
    p = inputs.Params(n_ngb=64.0)
    rng = np.random.default_rng(n)
    h = (min(1.0, 0.9 * n ** (-1.0 / 3.0) * 2.5) * rng.uniform(0.4, 1.6, n)).astype(np.float32)
    check(ctx, gas_set(kind, n), h, p, (0.0, 0.0, 0.0, 1.0))


def test_forest_of_uneven_snapshots_against_oracle(ctx):
    # snapshots' terminals share windows; one snapshot is empty, one has one particle
    sizes = [1, 200, 0, 3000, 70, 64, 900]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    rng = np.random.default_rng(5)
    boxes, pos = [], []
    for k, m in enumerate(sizes):
        boxes.append((float(k), 0.0, 0.0, 1.0))
        pos.append(rng.random((m, 3)) + [k, 0, 0])
    pos = np.concatenate(pos).astype(np.float32)
    h = np.concatenate([np.full(m, 2.3 * max(m, 1) ** (-1.0 / 3.0)) for m in sizes])
    act = np.sort(rng.choice(len(pos), 1700, replace=False)).astype(np.int32)
    check(ctx, pos, h.astype(np.float32), inputs.Params(n_ngb=64.0), boxes, off, act)


@pytest.mark.parametrize("fp64", [False, True])
def test_every_team_size_gives_the_same_bits(ctx, fp64):
    # 2^19 targets in unsplit groups take teams of 4; the first 2^15 in tree
    # order form the same groups and take teams of 16 (the hydro force of 2^20
    # targets takes no team)
    from paper_2003_10850_amd import g3, ops
    n = 1 << (19 if fp64 else 20)
    w = inputs.uniform(n=n, seed=21)
    pos = w.pos if fp64 else w.pos.astype(np.float32)
    ht = torch.float64 if fp64 else torch.float32
    p = inputs.Params(n_ngb=48.0)
    c = ops.Context(torch.device("cuda", 0))
    c.set_tuning(g3.G3_TUNE_DENSITY, 128, -1)
    tree = ops.Tree(c, dev_t(pos), dev_t(w.mass.astype(np.float32)), None, tuple(w.box), p)
    order = tree.export(1)["order"]
    few = torch.sort(order[: 1 << 15]).values
    g = torch.Generator(device="cuda").manual_seed(2)
    R = lambda *s: torch.rand(*s, generator=g, device="cuda")
    h = (2.25 * n ** (-1.0 / 3.0) * (0.8 + 0.4 * R(n))).to(ht)
    vel, u, rho, om = R(n, 3) - 0.5, 0.5 + R(n), 0.5 + R(n), 0.5 + R(n)
    all_d, few_d = ops.density(tree, h=h), ops.density(tree, h=h, active=few)
    all_f = ops.hydro_force(tree, vel, u, h, rho, om)
    few_f = ops.hydro_force(tree, vel, u, h, rho, om, active=few)
    at = few.long()
    for a, b in ((all_d, few_d), (all_f, few_f)):
        for k in a:
            assert torch.equal(a[k][at], b[k][at]), k



@pytest.mark.parametrize("log_few,fp64", [(14, False), (16, False), (17, False), (18, False),
                                          (14, True), (17, True)])
def test_middle_team_sizes_give_the_same_bits(ctx, log_few, fp64):
    # 2^20 targets: density in teams of 4, hydro force without; the first 2^18
    # in tree order take teams of 8, 2^17 and 2^16 of 12, 2^14 of 16 (with FP64
    # positions 2^17 take teams of 8)
    from paper_2003_10850_amd import g3, ops
    n = 1 << 20
    w = inputs.uniform(n=n, seed=22)
    p = inputs.Params(n_ngb=48.0)
    c = ops.Context(torch.device("cuda", 0))
    for kind in (g3.G3_TUNE_DENSITY, g3.G3_TUNE_HYDRO):
        c.set_tuning(kind, 128, -1)
    tree = ops.Tree(c, dev_t(w.pos if fp64 else w.pos.astype(np.float32)), dev_t(w.mass.astype(np.float32)), None,
                    tuple(w.box), p)
    few = torch.sort(tree.export(1)["order"][: 1 << log_few]).values
    g = torch.Generator(device="cuda").manual_seed(2)
    R = lambda *s: torch.rand(*s, generator=g, device="cuda")
    h = (2.25 * n ** (-1.0 / 3.0) * (0.8 + 0.4 * R(n))).to(torch.float64 if fp64 else torch.float32)
    vel, u, rho, om = R(n, 3) - 0.5, 0.5 + R(n), 0.5 + R(n), 0.5 + R(n)
    at = few.long()
    for a, b in ((ops.density(tree, h=h), ops.density(tree, h=h, active=few)),
                 (ops.hydro_force(tree, vel, u, h, rho, om),
                  ops.hydro_force(tree, vel, u, h, rho, om, active=few))):
        for k in a:
            assert torch.equal(a[k][at], b[k][at]), k


def close(a, b, what):
    # the same 64-candidate partial sums, compensated over the tiles in another
    # order: a last rounding of the total and one or two of each factor on it
    a, b = a.double(), b.double()
    lim = 2e-6 * b.abs() + 1e-7 * b.abs().max()
    assert bool(((a - b).abs() <= lim).all()), what


@pytest.mark.parametrize("m,total", [(64, 125000), (641, 210000), (5000, 125000),
                                     (5000, 210000)])
def test_adjoints_of_a_forest_equal_the_single_trees(ctx, m, total):
    # the forest's members take teams of 8 or 4, the single snapshots (which
    # other tests hold against the oracle) teams of 16
    from paper_2003_10850_amd import ops
    count = -(-total // m)
    some = 25
    print(f"teams adjoint forest {count} x {m}", flush=True)
    p = inputs.Params(n_ngb=48.0)
    g = torch.Generator(device="cuda").manual_seed(m)
    R = lambda *s: torch.rand(*s, generator=g, device="cuda")
    n = count * m
    pos, mass = R(n, 3), (0.5 + R(n)) / m
    h = 2.25 * m ** (-1.0 / 3.0) * (0.8 + 0.4 * R(n))
    vel, u, rho, om = R(n, 3) - 0.5, 0.5 + R(n), 0.5 + R(n), 0.5 + R(n)
    box = (0.0, 0.0, 0.0, 1.0)
    ups = [R(n) - 0.5 for _ in range(3)] + [R(n, 3) - 0.5, R(n) - 0.5]

    def grads(tree, r):
        x = [t[r].clone().requires_grad_(True) for t in (pos, mass, h, vel, u, rho, om)]
        d = ops.density_ad(tree, x[0], x[1], x[2])
        f = ops.hydro_force_ad(tree, x[0], x[3], x[1], x[4], x[2], x[5], x[6])
        gd = torch.autograd.grad(d, x[:3], [t[r] for t in ups[:3]])
        return gd + torch.autograd.grad(f, x, [t[r] for t in ups[3:]])

    off = np.arange(count + 1, dtype=np.int64) * m
    all_g = grads(ops.Tree(ctx, pos, mass, None, [box] * count, p, snap_off=off), slice(0, n))
    for k in np.linspace(0, count - 1, some).astype(int):
        r = slice(k * m, (k + 1) * m)
        one = grads(ops.Tree(ctx, pos[r].clone(), mass[r].clone(), None, box, p), r)
        for i, (a, b) in enumerate(zip(all_g, one)):
            close(a[r], b, (int(k), i))


@pytest.mark.parametrize("log_few", [10, 15, 18, 20])
def test_conduction_and_gradients_of_every_team_size(ctx, log_few):
    # 1.6e6 targets: conduction without teams, gradients in teams of 4; the
    # first 2^20 in teams of 4, 2^18 of 8, fewer of 16
    from paper_2003_10850_amd import g3, ops
    n = 1600000
    w = inputs.uniform(n=n, seed=21)
    p = inputs.Params(n_ngb=48.0)
    c = ops.Context(torch.device("cuda", 0))
    for kind in (g3.G3_TUNE_DENSITY, g3.G3_TUNE_HYDRO):
        c.set_tuning(kind, 128, -1)
    tree = ops.Tree(c, dev_t(w.pos.astype(np.float32)), dev_t(w.mass.astype(np.float32)), None,
                    tuple(w.box), p)
    few = torch.sort(tree.export(1)["order"][: 1 << log_few]).values
    g = torch.Generator(device="cuda").manual_seed(2)
    R = lambda *s: torch.rand(*s, generator=g, device="cuda")
    h = 2.25 * n ** (-1.0 / 3.0) * (0.8 + 0.4 * R(n))
    vel, u, rho, om = R(n, 3) - 0.5, 0.5 + R(n), 0.5 + R(n), 0.5 + R(n)
    at = few.long()
    a, b = [ops.conduction(tree, u, h, rho, 1.0, 2.5, active=x) for x in (None, few)]
    assert torch.equal(a["npairs"][at], b["npairs"][at])
    close(a["dudt"][at], b["dudt"][at], "dudt")
    a, b = [ops.velocity_gradients(tree, vel, h, rho, om, active=x) for x in (None, few)]
    for k in a:
        close(a[k][at], b[k][at], k)


def test_targets_without_neighbours_have_no_rates(ctx):
    # h = 0, h whose h^-5 overflows, and rho = 0 where no pair is at r > 0
    from paper_2003_10850_amd import ops
    n = 200
    g = torch.Generator(device="cuda").manual_seed(5)
    pos, one = torch.rand(n, 3, generator=g, device="cuda"), torch.ones(n, device="cuda")
    tree = ops.Tree(ctx, pos, one, None, (0.0, 0.0, 0.0, 1.0), inputs.Params(n_ngb=16.0))
    h = torch.full((n,), 1e-9, device="cuda")
    h[::3] = 0.0
    rho = one.clone()
    c = ops.conduction(tree, one, h, torch.zeros(n, device="cuda"), 1.0, 0.0)
    assert torch.equal(c["dudt"], torch.zeros(n, device="cuda"))
    v = ops.velocity_gradients(tree, pos.clone(), h, rho, one)
    assert not v["div"].any() and not v["curl"].any()


@pytest.mark.parametrize("approach", [0.0, 1.0, -1.0])
def test_an_infinite_factor_without_upstream_stays_out_of_the_adjoint(ctx, approach):
    # rho = 0 makes the second particle's pressure factor infinite; only the
    # first has an upstream gradient, of its acceleration alone, and no term of
    # its velocity, u, h and rho gradients holds that factor
    from paper_2003_10850_amd import ops
    pos = dev_t(np.float32([[0.45, 0.5, 0.5], [0.55, 0.5, 0.5]]))
    one = torch.ones(2, device="cuda")
    tree = ops.Tree(ctx, pos, one, None, (0.0, 0.0, 0.0, 1.0), inputs.Params(n_ngb=16.0))
    vel = torch.zeros_like(pos)
    vel[0, 0] = approach
    rho = dev_t(np.float32([1.0, 0.0]))
    x = [t.clone().requires_grad_(True) for t in (pos, vel, one, one, 0.3 * one, rho, one)]
    acc = ops.hydro_force_ad(tree, *x)[0]
    up = torch.zeros_like(acc)
    up[0] = torch.tensor([1.0, 0.5, -0.25])
    _, gv, _, gu, gh, gr, go = torch.autograd.grad(acc, x, up)
    assert torch.isfinite(gv).all()
    for g in (gu, gh, gr, go):
        assert torch.isfinite(g[0])


@pytest.mark.parametrize("n", [2, 65, 1000, 30000])
def test_hydro_adjoint_of_parts_of_the_upstream_adds_up(ctx, n):
    # the gradients are linear in the upstream ones, whichever side of a pair
    # holds them: sums of a few hundred FP32 terms that cancel in part, 1e-5 of
    # the largest
    from paper_2003_10850_amd import ops
    g = torch.Generator(device="cuda").manual_seed(n)
    R = lambda *s: torch.rand(*s, generator=g, device="cuda")
    pos, mass = R(n, 3), (0.5 + R(n)) / n
    tree = ops.Tree(ctx, pos, mass, None, (0.0, 0.0, 0.0, 1.0), inputs.Params(n_ngb=16.0))
    x = [t.requires_grad_(True) for t in (pos.clone(), R(n, 3) - 0.5, mass.clone(), 0.5 + R(n),
                                          1.2 * n ** (-1.0 / 3.0) * (0.8 + 0.4 * R(n)),
                                          0.5 + R(n), 0.5 + R(n))]
    ups = (R(n, 3) - 0.5, R(n) - 0.5)

    def grads(on):
        f = ops.hydro_force_ad(tree, *x)
        return torch.autograd.grad(f[:2], x, [u * (on if u.dim() == 1 else on[:, None]) for u in ups])

    few = (torch.arange(n, device="cuda") % 7 == 1).float()
    for a, b, c in zip(grads(few), grads(1.0 - few), grads(torch.ones_like(few))):
        assert (a + b - c).abs().max() <= 1e-5 * c.abs().max()
