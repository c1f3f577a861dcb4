"""Finite inputs in units far from one, where single terms or node sums leave
FP32's range though every result lies in it, against the oracle (or counts by
brute force).

Tolerances: counts exact; accelerations and gradients within 1e-5 of the L1 sum
of their terms and potentials within 2e-6, as the parity tests have them.
"""
import dataclasses

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


def host(d):
    return {k: v.cpu().numpy() for k, v in d.items()}


@pytest.mark.parametrize("n", [67, 2001])
def test_fp64_pair_counts_where_the_decision_band_overflows(ctx, n):
    # the groups are wider than the root of FP32's largest number, so the band
    # around the threshold is infinite and every entry takes the FP64 test
    from paper_2003_10850_amd import ops
    print(f"range: band n={n}", flush=True)
    rng = np.random.default_rng(n)
    side = 1e20
    pos = rng.random((n, 3)) * side
    h = 1.05e19 * rng.uniform(0.8, 1.2, n)
    one = np.ones(n, np.float32)
    tree = ops.Tree(ctx, dev_t(pos), dev_t(one), None, (0.0, 0.0, 0.0, side),
                    inputs.Params(n_ngb=32.0))
    f = ops.hydro_force(tree, dev_t(np.zeros((n, 3), np.float32)), dev_t(one), dev_t(h),
                        dev_t(one), dev_t(one))
    d = pos[:, None] - pos[None]
    H = np.maximum(h[:, None], h[None])
    want = ((d[..., 0] ** 2 + d[..., 1] ** 2) + d[..., 2] ** 2 < H * H).sum(1) - 1
    np.testing.assert_array_equal(f["npairs"].cpu().numpy(), want)


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("theta", [0.5, 0.7])
def test_gravity_below_nodes_heavier_than_fp32_holds(ctx, theta, fp64):
    # the root's mass overflows FP32; no particle accepts it
    from paper_2003_10850_amd import ops
    n, side = 4096, 1e6
    rng = np.random.default_rng(3)
    pos = rng.random((n, 3)) * side
    if not fp64:
        pos = pos.astype(np.float32)
    mass = (1.5e35 * rng.uniform(0.7, 1.3, n)).astype(np.float32)
    p = inputs.Params(n_ngb=32.0, theta=theta, eps=1e4, G=1e-30)
    box = (0.0, 0.0, 0.0, side)
    tree = ops.Tree(ctx, dev_t(pos), dev_t(mass), None, box, p)
    g = host(ops.gravity(tree))
    pr = dataclasses.replace(p, flags=oracle.FLAG_FP64_DECISIONS if fp64 else 0)
    ref = oracle.gravity(oracle.Tree(pos.astype(np.float64), mass.astype(np.float64), box), pr)
    np.testing.assert_array_equal(g["nterms"], ref["nterms"])
    assert (np.linalg.norm(g["acc"] - ref["acc"], axis=1) / ref["S"]).max() < 1e-5
    assert (np.abs(g["pot"] - ref["pot"]) / np.abs(ref["pot"])).max() < 2e-6


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("n,theta", [(1 << 18, 0.7), (1400000, 0.5)])
def test_gravity_below_a_heavy_root_in_teams_of_8_and_4(ctx, n, theta, fp64):
    # masses, lengths and G scaled by powers of two (an even one for the lengths,
    # whose square root is taken of r^2): every product and sum has the same digits,
    # but the root's mass is above FP32's largest number
    from paper_2003_10850_amd import ops
    g = torch.Generator(device="cuda").manual_seed(12)
    pos = torch.rand(n, 3, generator=g, device="cuda").to(torch.float64 if fp64 else torch.float32)
    mass = (0.5 + torch.rand(n, generator=g, device="cuda")) / n
    out = []
    for m, x in ((1.0, 1.0), (2.0 ** 130, 2.0 ** 20)):
        tree = ops.Tree(ctx, pos * x, (mass.double() * m).float(), None, (0.0, 0.0, 0.0, x),
                        inputs.Params(theta=theta, eps=2.0 ** -9 * x, G=1.0 / m))
        f = ops.gravity(tree)
        out.append((f["acc"] * x * x, f["pot"] * x, f["nterms"]))
    for a, b in zip(*out):
        assert torch.equal(a, b)


@pytest.mark.parametrize("mass,speed,side", [(2e33, 1e7, 3e3), (1e-36, 1e-3, 0.1), (1e-3, 1.0, 1.0)])
def test_velocity_gradients_in_large_and_small_units(ctx, mass, speed, side):
    from paper_2003_10850_amd import ops
    n = 3000
    rng = np.random.default_rng(8)
    pos = (rng.random((n, 3)) * side).astype(np.float32)
    vel = (speed * rng.normal(0, 1, (n, 3))).astype(np.float32)
    m = (mass * rng.uniform(0.7, 1.3, n)).astype(np.float32)
    h = (2.3 * side * n ** (-1.0 / 3.0) * rng.uniform(0.8, 1.2, n)).astype(np.float32)
    rho = (n * mass / side ** 3 * rng.uniform(0.7, 1.3, n)).astype(np.float32)
    om = rng.uniform(0.8, 1.2, n).astype(np.float32)
    box = (0.0, 0.0, 0.0, side)
    p = inputs.Params(n_ngb=48.0)
    tree = ops.Tree(ctx, dev_t(pos), dev_t(m), None, box, p)
    v = host(ops.velocity_gradients(tree, dev_t(vel), dev_t(h), dev_t(rho), dev_t(om)))
    t = oracle.Tree(pos.astype(np.float64), m.astype(np.float64), box, gas_only=True,
                    type=np.zeros(n, np.uint8))
    ref = oracle.velgrad(t, p, vel, h, rho, om)
    assert (np.abs(v["div"] - ref["div"]) / ref["S_div"]).max() < 1e-5
    assert (np.linalg.norm(v["curl"] - ref["curl"], axis=1) / ref["S_curl"]).max() < 1e-5


@pytest.mark.parametrize("fp64", [False, True])
def test_hydro_force_on_a_particle_with_a_tiny_h_and_a_large_pressure(ctx, fp64):
    # A h^-5 of the first particle overflows; its pairs lie beyond its own h,
    # where its kernel is zero
    from paper_2003_10850_amd import ops
    n = 130
    rng = np.random.default_rng(4)
    pos = 0.3 + 0.4 * rng.random((n, 3))
    if not fp64:
        pos = pos.astype(np.float32)
    mass = np.full(n, 1.0 / n, np.float32)
    vel = rng.normal(0, 0.1, (n, 3)).astype(np.float32)
    h = rng.uniform(0.15, 0.2, n).astype(pos.dtype)
    u, rho = [rng.uniform(0.5, 1.5, n).astype(np.float32) for _ in range(2)]
    h[0], u[0], rho[0] = 1e-6, 1e6, 1e-3
    one = np.ones(n, np.float32)
    p = inputs.Params(n_ngb=32.0)
    box = (0.0, 0.0, 0.0, 1.0)
    tree = ops.Tree(ctx, dev_t(pos), dev_t(mass), None, box, p)
    f = host(ops.hydro_force(tree, dev_t(vel), dev_t(u), dev_t(h), dev_t(rho), dev_t(one)))
    t = oracle.Tree(pos.astype(np.float64), mass.astype(np.float64), box, gas_only=True,
                    type=np.zeros(n, np.uint8))
    pr = dataclasses.replace(p, flags=oracle.FLAG_FP64_DECISIONS if fp64 else 0)
    ref = oracle.hydro(t, pr, vel, u, h, rho, one)
    assert ref["npairs"][0] > 0
    np.testing.assert_array_equal(f["npairs"], ref["npairs"])
    assert (np.linalg.norm(f["acc"] - ref["acc"], axis=1) / ref["S"]).max() < 1e-5
    assert np.isfinite(f["dudt"]).all()
