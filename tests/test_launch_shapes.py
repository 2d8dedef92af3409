"""Launch shapes chosen on the host (no GPU): the resident 1D lines, whose
blocks wait for each other, and the fused 2D Euler stage follow the number of
compute units they are given."""
import ctypes as C

import pytest

from paper_2603_26272_amd import za
from paper_2603_26272_amd.problem import ADVECTION, EULER, Problem

ARGS = "RK10za_problemiPiS2_"


def _shape(name, P, cus):
    f = getattr(C.CDLL(za.LIB_PATH), f"_Z{len(name)}{name}{ARGS}")
    f.restype = None
    a, b = C.c_int(-1), C.c_int(-1)
    f(C.byref(za.ZaProblem.from_problem(P)), C.c_int(cus), C.byref(a), C.byref(b))
    return a.value, b.value


@pytest.mark.parametrize("cus", [8, 32, 64, 128, 256, 304])
@pytest.mark.parametrize("system,waves_per_cu", [(EULER, 8), (ADVECTION, 16)])
def test_lines_take_at_most_a_quarter_of_the_device(cus, system, waves_per_cu):
    """Four lines at once (one per hardware queue) have all their blocks
    resident: a line of several blocks takes a quarter of the wavefronts."""
    several = 0
    for N in (64, 500, 600, 1021, 1500, 4096, 5000, 16321, 32640, 32704, 65472):
        blocks, waves = _shape("line_shape", Problem(dim=1, system=system, nx=N), cus)
        if blocks > 1:
            assert 4 * blocks * waves <= cus * waves_per_cu, (N, blocks, waves)
            assert blocks * (64 * waves - 1) >= N
            several += 1
    assert several > 0 or cus < 16


def test_line_of_one_block_needs_one_cu():
    assert _shape("line_shape", Problem(dim=1, nx=200), 1) == (1, 4)


def test_fused_bands_follow_the_device():
    """128^2: 3 strips; bands of one step (3 rows) while every block finds a
    CU of its own, taller ones on a device that would take rounds of them."""
    P = Problem(dim=2, nx=128, ny=128)
    assert _shape("fused_shape", P, 256) == (3, 43)
    gx, gy = _shape("fused_shape", P, 16)
    assert gx == 3 and gx * gy <= 3 * 16


def _model(P, res, cus=256):
    """The cost rule of fused_shape for `res` resident blocks per CU."""
    strips, best = -(-P.nx // 63), None
    for s in range(1, 257):
        nb = -(-P.ny // (4 * s - 1))
        m = -(-strips * nb // cus)
        full, rest = divmod(m, res)
        idle = 1.5 if rest == 1 else (1.15 if rest == 2 and res > 2 else 1.0)
        start = 0.5 if res == 1 else 2.0
        cost = full * (res * s + start) + (idle * rest * s + start if rest else 0.0)
        if best is None or cost < best[0]:
            best = (cost, strips, nb)
        if m <= 1:
            break
    return best[1:]


JS = dict(weight_L=0.0, p=2.0)
F32 = dict(precision=1, eps=1e-20, mu0=1e-8)


@pytest.mark.parametrize("n", [64, 300, 512, 700, 1024, 2048])
@pytest.mark.parametrize("kind,res", [(dict(), 3), (dict(order=2), 3), (dict(order=4), 2), (dict(order=5), 2),
                                      (JS, 2), (dict(order=2, **JS), 2), (dict(order=4, **JS), 2),
                                      (dict(order=5, **JS), 1), (F32, 4), (dict(**F32, **JS), 3)])
def test_fused_bands_use_the_kernels_own_occupancy(kind, res, n):
    """The bands are those for as many resident blocks per CU as the kernel
    of these weights, this order and this precision is launched for."""
    P = Problem(dim=2, nx=n, ny=n, **kind)
    assert _shape("fused_shape", P, 256) == _model(P, res)
    assert _waves(P) == res


def _waves(P):
    f = getattr(C.CDLL(za.LIB_PATH), "_Z11fused_wavesRK10za_problem")
    return f(C.byref(za.ZaProblem.from_problem(P)))


P15 = dict(p=1.5)


@pytest.mark.parametrize("kind,res", [(dict(order=2, **P15), 3), (P15, 2), (dict(order=4, **P15), 2),
                                      (dict(order=5, **P15), 1), (dict(**F32, **P15), 3)])
def test_pow_kernels_share_the_cu(kind, res):
    """Weights with pow() leave most issue slots of a CU idle with one block:
    the fused kernels are compiled, and their bands chosen, for several (but
    at r = 5, where two would take too much scratch memory)."""
    P = Problem(dim=2, nx=512, ny=512, **kind)
    assert _waves(P) == res
    assert _shape("fused_shape", P, 256) == _model(P, res)


@pytest.mark.parametrize("env,on", [({}, True), (dict(ZA_STEP_GRAPHS="1"), True), (dict(ZA_STEP_GRAPHS="0"), False),
                                    (dict(ZA_RESIDENT="1"), True), (dict(ZA_RESIDENT="0"), False),
                                    (dict(ZA_XL_CHUNKS="3"), False)])
def test_environment_that_leaves_the_resident_kernel_on(monkeypatch, env, on):
    for k in ("ZA_RESIDENT", "ZA_STEP_GRAPHS", "ZA_XL_CHUNKS"):
        monkeypatch.delenv(k, raising=False)
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    f = getattr(C.CDLL(za.LIB_PATH), "_Z15resident_wantedv")
    f.restype = C.c_bool
    assert f() is on
