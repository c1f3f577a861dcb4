"""The launchers refuse a team of waves that has no kernel, before they touch a
device (a kernel of another team's size would run past its LDS arrays), and the
rules name only teams that have one.
"""
import ctypes
import re
import subprocess

import pytest

from paper_2003_10850_amd import g3

INVALID = 1  # hipErrorInvalidValue


@pytest.fixture(scope="module")
def lib():
    handle = g3.lib()
    names = subprocess.run(["nm", "-D", "--defined-only", handle._name], capture_output=True,
                           text=True, check=True).stdout
    def get(name):
        return handle[re.search(rf"\b_ZN2g3{len(name)}{name}[A-Za-z0-9_]*", names).group(0)]
    return get


def octree():
    b = (ctypes.c_int64 * 64)(*([64] * 64))  # members, nodes, and pointers that nothing reads
    return ctypes.byref(b)


def sph(f64, team):
    class Sph(ctypes.Structure):
        _fields_ = [("f", ctypes.c_float * 4), ("max_iter", ctypes.c_int), ("leaf", ctypes.c_int),
                    ("f64", ctypes.c_int), ("team", ctypes.c_int), ("absmax", ctypes.c_void_p)]
    return ctypes.byref(Sph(max_iter=1, leaf=8, f64=f64, team=team))


def grav(f64, team):
    class Grav(ctypes.Structure):
        _fields_ = [("f", ctypes.c_float * 3), ("inside", ctypes.c_int), ("f64", ctypes.c_int),
                    ("theta", ctypes.c_double), ("team", ctypes.c_int)]
    return ctypes.byref(Grav(f64=f64, team=team))


I64, P0 = ctypes.c_int64(1), ctypes.c_void_p(0)
NONE = [P0] * 8


def density(lib, f64, team):
    return lib("launch_density")(octree(), octree(), I64, sph(f64, team), octree(),
                                 ctypes.c_int(0), *NONE[:7])


def hydro(lib, f64, team, ext=False):
    return lib("launch_hydro")(octree(), octree(), I64, sph(f64, team), octree(), *NONE[:5],
                               ctypes.c_void_p(64 if ext else 0), ctypes.c_float(0))


def gravity(lib, f64, team):
    return lib("launch_gravity")(octree(), octree(), I64, grav(f64, team), *NONE[:4])


def gravity_bwd(lib, f64, team):
    return lib("launch_gravity_bwd")(octree(), octree(), I64, grav(f64, team), I64, *([P0] * 13))


def conduction(lib, team):
    return lib("launch_conduction")(octree(), octree(), I64, ctypes.c_int(8), octree(),
                                    ctypes.c_int(team), *NONE[:4])


def velgrad(lib, team):
    return lib("launch_velgrad")(octree(), octree(), I64, octree(), ctypes.c_int(team), *NONE[:5])


@pytest.mark.parametrize("call,teams", [
    (lambda l, t: density(l, 0, t), {1, 4, 8, 12, 16}),
    (lambda l, t: density(l, 1, t), {1, 4, 8, 16}),
    (lambda l, t: hydro(l, 0, t), {1, 8, 12, 16}),
    (lambda l, t: hydro(l, 0, t, True), {1, 4, 8, 16}),
    (lambda l, t: hydro(l, 1, t), {1, 4, 8, 16}),
    (lambda l, t: hydro(l, 1, t, True), {1, 4, 8, 16}),
    (lambda l, t: gravity(l, 0, t), {4, 8, 16}),
    (lambda l, t: gravity(l, 1, t), {4, 8, 16}),
    (lambda l, t: gravity_bwd(l, 0, t), {1, 4, 8, 16}),
    (lambda l, t: conduction(l, t), {1, 4, 8, 16}),
    (lambda l, t: velgrad(l, t), {4, 8, 16})])
def test_teams_without_a_kernel_are_refused(lib, call, teams):
    for t in set(range(0, 18)) - teams:
        assert call(lib, t) == INVALID, t


@pytest.mark.parametrize("rule,args,teams", [
    ("density_team", (0, 1), {1, 4, 8, 12, 16}), ("density_team", (1, 0), {1, 4, 8, 16}),
    ("hydro_team", (0,), {1, 8, 12, 16}), ("hydro_team", (1,), {1, 4, 8, 16}),
    ("gravity_team", (), {4, 8, 16}), ("gravity_bwd_team", (), {1, 4, 8, 16}),
    ("adjoint_team", (), {4, 8, 16}), ("velgrad_team", (), {4, 8, 16}),
    ("conduction_team", (), {1, 4, 8, 16})])
def test_the_rules_name_teams_that_have_a_kernel(lib, rule, args, teams):
    got = {lib(rule)(ctypes.c_int64(n), *map(ctypes.c_int, args))
           for k in range(31) for n in ((1 << k) - 1, 1 << k, 3 << k)}
    assert got <= teams and len(got) == len(teams)
