"""GPU: 1D problems whose steps run in one resident launch (one block, or
several that exchange halo cells and wave speeds through memory) against the
same steps as ordinary launches (ZA_RESIDENT=0).  Both evaluate every flux,
update and wave speed with the same arithmetic and take exact maxima, so the
states, times and step sizes agree bit for bit.  Sizes sit at the edges of
the launch shapes (wavefronts, blocks, the largest line); the options cover
every kernel; a wait limit of zero ticks makes the blocks give up, and the
steps must then be repeated by ordinary launches with the same result."""
import numpy as np
import pytest

from paper_2603_26272_amd import workloads as W
from paper_2603_26272_amd.problem import ADVECTION, BUCKLEY, BURGERS, EULER, PERIODIC, TRANSMISSIVE, Problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _data(system, N, seed=3):
    if system == EULER:
        P, q = W.riemann_1d(seed, N) if N >= 8 else W.entropy_wave_1d(N)
        return P.with_(dt_rule=0), q
    x = W.centres(N, -1.0, 1.0)
    u = 0.5 + 0.3 * np.sin(np.pi * x + 0.3) + np.where((x > -0.4) & (x < 0.1), 0.15, 0.0)
    return Problem(dim=1, system=system, nx=N, ny=1, xlo=-1.0, xhi=1.0, cfl=0.45), u.reshape(1, 1, N)


def _run(monkeypatch, P, q0, resident, t_final=0.0, steps=7, spin=None, calls=1, step=False):
    from paper_2603_26272_amd.za import Context
    for k in ("ZA_RESIDENT", "ZA_LINE_SPIN", "ZA_XL_CHUNKS", "ZA_STEP_GRAPHS"):
        monkeypatch.delenv(k, raising=False)
    if not resident:
        monkeypatch.setenv("ZA_RESIDENT", "0")
    if spin is not None:
        monkeypatch.setenv("ZA_LINE_SPIN", str(spin))
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    q = torch.from_numpy(np.ascontiguousarray(q0)).cuda()
    with Context(P) as ctx:
        if step:
            out = [ctx.step(q, sync=True) for _ in range(steps)]
        else:
            out = [ctx.solve(q, t_final, steps, check=False) for _ in range(calls)]
        rhs = ctx.rhs(q)
    return q.cpu().numpy(), out, rhs.cpu().numpy()


def _same(monkeypatch, P, q0, **kw):
    a, b = _run(monkeypatch, P, q0, True, **kw), _run(monkeypatch, P, q0, False, **{**kw, "spin": None})
    assert a[1] == b[1], (P.nx, a[1], b[1])
    assert np.array_equal(a[0], b[0], equal_nan=True), P.nx
    assert np.array_equal(a[2], b[2], equal_nan=True), P.nx
    return a


@pytest.mark.parametrize("bc", [PERIODIC, TRANSMISSIVE])
@pytest.mark.parametrize("N", [1, 2, 3, 5, 7, 63, 64, 65, 200, 255, 256, 511, 512, 513, 765, 1021, 4096, 16320,
                               16321, 32640, 32641, 32704, 32705])
def test_euler_sizes(monkeypatch, N, bc):
    P, q0 = _data(EULER, N)
    _same(monkeypatch, P.with_(bc_x=bc), q0)


@pytest.mark.parametrize("bc", [PERIODIC, TRANSMISSIVE])
@pytest.mark.parametrize("system", [ADVECTION, BURGERS, BUCKLEY])
@pytest.mark.parametrize("N", [2, 64, 400, 1023, 1024, 5000, 16321, 32641, 65408, 65472, 65473])
def test_scalar_sizes(monkeypatch, system, N, bc):
    P, q0 = _data(system, N)
    _same(monkeypatch, P.with_(bc_x=bc), q0, steps=5)


OPTIONS = [dict(precision=1, eps=1e-20, mu0=1e-8), dict(weight_L=0.0, p=2.0), dict(affine_invariant=1), dict(order=2),
           dict(order=4), dict(order=5), dict(lf=1), dict(alt_tau=1), dict(linear_weights=1), dict(p=1.5),
           dict(pp_limiter=1, cfl=0.45), dict(dt_rule=1, cfl=0.3), dict(precision=1, eps=1e-20, weight_L=0.0, p=2.0)]


@pytest.mark.parametrize("opt", OPTIONS)
@pytest.mark.parametrize("N", [130, 1500])
@pytest.mark.parametrize("system", [EULER, BURGERS])
def test_options(monkeypatch, system, N, opt):
    if system != EULER and "pp_limiter" in opt:
        pytest.skip("the limiter applies to the Euler equations")
    P, q0 = _data(system, N)
    P = P.with_(**opt)
    _same(monkeypatch, P, q0, steps=4)
    _same(monkeypatch, P, q0, steps=3, step=True)


@pytest.mark.parametrize("N", [200, 1500])
@pytest.mark.parametrize("dt_rule", [0, 1])
def test_final_time_and_repeated_calls(monkeypatch, N, dt_rule):
    P, q0 = _data(EULER, N)
    P = P.with_(dt_rule=dt_rule)
    T = 40.3 * 0.5 * P.dx / 2.5 if dt_rule == 0 else 40.3 * 0.5 * P.dx ** 2
    _same(monkeypatch, P, q0, t_final=T, steps=0, calls=2)
    _same(monkeypatch, P, q0, t_final=T, steps=11)


@pytest.mark.parametrize("N", [200, 1500])
def test_inadmissible_states(monkeypatch, N):
    P, q0 = _data(EULER, N)
    bad = q0.copy()
    bad[2, 0, N // 3] = -1.0          # negative pressure at the start
    a = _same(monkeypatch, P, bad, steps=3)
    assert a[1][0]["nonfinite_step"] == 0 and a[1][0]["status"] != 0
    (Pv, qv), _ = W.vacuum_tube(N, speed=8.0)   # fails some steps in
    a = _same(monkeypatch, Pv, qv, steps=60)
    assert a[1][0]["nonfinite_step"] >= 0


@pytest.mark.parametrize("N", [700, 4096])
def test_blocks_that_wait_too_long(monkeypatch, N):
    P, q0 = _data(EULER, N)
    _same(monkeypatch, P, q0, steps=40, spin=0, calls=2)
    _same(monkeypatch, P, q0, t_final=20 * 0.4 * P.dx / 2.5, steps=0, spin=0)


def test_two_streams(monkeypatch):
    from paper_2603_26272_amd.za import Context
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    P, q0 = _data(EULER, 4096)
    ref = _run(monkeypatch, P, q0, False, steps=50)[0]
    monkeypatch.delenv("ZA_RESIDENT", raising=False)
    import threading
    got = [None] * 4

    def work(i):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            q = torch.from_numpy(q0).cuda()
            with Context(P, stream=s) as ctx:
                ctx.solve(q, 0.0, 50)
            got[i] = q.cpu().numpy()

    th = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    [t.start() for t in th]
    [t.join() for t in th]
    assert all(np.array_equal(g, ref) for g in got)


def _blow_up(N=1100):
    """Advection with linear weights and a fixed step just beyond the limit of
    the scheme: the state overflows after 5819 of 300,000 steps."""
    x = W.centres(N, -1.0, 1.0)
    P = Problem(dim=1, system=ADVECTION, nx=N, ny=1, xlo=-1.0, xhi=1.0, bc_x=PERIODIC, linear_weights=1)
    P = P.with_(dt_rule=1, cfl=1.22 / P.dx)
    return P, (0.5 + 0.3 * np.sin(np.pi * x + 0.3)).reshape(1, 1, N), 1.22 * P.dx * 300000


def test_launches_after_a_long_wait_are_checked_as_often(monkeypatch):
    """Once the blocks have given up, ordinary launches must stop as soon
    after the end (or an inadmissible state) as without the resident kernel:
    32 steps (2048 equal steps) between host checks, not 4096 (262,144)."""
    import time
    from paper_2603_26272_amd.za import Context
    P, q0, T = _blow_up()
    Pe, qe = _data(EULER, 700)
    if not torch.cuda.is_available():
        pytest.skip("no GPU")

    def seconds(P, q0, T, **env):
        for k in ("ZA_RESIDENT", "ZA_LINE_SPIN", "ZA_XL_CHUNKS", "ZA_STEP_GRAPHS"):
            monkeypatch.delenv(k, raising=False)
        for k, v in env.items():
            monkeypatch.setenv(k, v)
        best, res = 1e9, None
        for _ in range(3):
            q = torch.from_numpy(np.ascontiguousarray(q0)).cuda()
            with Context(P) as ctx:
                torch.cuda.synchronize()
                t = time.perf_counter()
                res = ctx.solve(q, T, 0, check=False)
                best = min(best, time.perf_counter() - t)
        return best, res, q.cpu().numpy()

    # (4096 steps between checks: 31 ms against 0.6 ms for the first of these)
    for P, q0, T in ((Pe, qe, 20.3 * 0.5 * Pe.dx / 2.5), (P, q0, T)):
        ref = seconds(P, q0, T, ZA_RESIDENT="0")
        got = seconds(P, q0, T, ZA_LINE_SPIN="0")
        assert got[1] == ref[1] and np.array_equal(got[2], ref[2], equal_nan=True)
        assert got[0] < 4.0 * ref[0], (got[0], ref[0])


@pytest.mark.parametrize("spin", [None, "0", "0:1"])
@pytest.mark.parametrize("dt_rule", [0, 1])
def test_several_launches_of_several_blocks(monkeypatch, dt_rule, spin):
    """More steps than one launch takes (4096): the second launch goes on from
    the control block that the first left, whether both run, the first gives
    up, or the second does (the steps go back to where it began)."""
    P, q0 = _data(EULER, 700)
    P = P.with_(dt_rule=dt_rule)
    if dt_rule == 0:
        _same(monkeypatch, P, q0, steps=4500, spin=spin)
    else:
        _same(monkeypatch, P, q0, t_final=4500.4 * P.cfl * P.dx ** 2, steps=0, spin=spin)
