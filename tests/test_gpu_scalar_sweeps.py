"""GPU: stages that are pairs of sweeps (2D scalar laws, limited 2D Euler
stages): the looped x-sweep against the one-shot sweep and the oracle, on
ragged and tiny widths and with both boundary conditions, and sweeps of so
many blocks that a launch of its own prepares their constants (more than
3072) against a periodic tile that stays below that."""
import numpy as np
import pytest

import oracle as orc
from paper_2603_26272_amd import workloads as W
from paper_2603_26272_amd.problem import ADVECTION, BUCKLEY, BURGERS, PERIODIC, TRANSMISSIVE, Problem

from tests.test_gpu_parity import assert_close

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SYSTEMS = [ADVECTION, BURGERS, BUCKLEY]


def _data(system, nx, ny, bc):
    x = np.arange(nx)[None, :] / 64.0
    y = np.arange(ny)[:, None] / 64.0
    u = 0.5 + 0.2 * np.sin(2.1 * x + 0.3) * np.cos(1.7 * y + 0.1) + 0.15 * ((x * 3) % 2 > 1) * (y % 1 < 0.6)
    u = u + 0.01 * np.sin(29.0 * x + 17.0 * y)
    P = Problem(dim=2, system=system, nx=nx, ny=ny, xhi=nx / 64.0, yhi=ny / 64.0, bc_x=bc[0], bc_y=bc[1], cfl=0.45,
                adv_speed=(1.0, -0.5))
    return P, np.ascontiguousarray(u.reshape(1, ny, nx))


def _run(monkeypatch, P, q0, steps, chunks=None):
    from paper_2603_26272_amd.za import Context
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    monkeypatch.delenv("ZA_XL_CHUNKS", raising=False)
    if chunks is not None:
        monkeypatch.setenv("ZA_XL_CHUNKS", str(chunks))
    q = torch.from_numpy(q0).cuda()
    with Context(P) as ctx:
        rhs = ctx.rhs(q).cpu().numpy()
        fx, fy = ctx.rhs_fluxes(q)
        info = ctx.solve(q, 0.0, steps)
    monkeypatch.delenv("ZA_XL_CHUNKS", raising=False)
    assert info["steps"] == steps
    return {"state": q.cpu().numpy(), "t": info["t"], "rhs": rhs, "fx": fx.cpu().numpy(), "fy": fy.cpu().numpy()}


@pytest.mark.parametrize("nx,ny", [(1, 3), (2, 5), (5, 4), (63, 5), (64, 5), (65, 3), (127, 4), (128, 4), (300, 6),
                                   (703, 3), (1500, 2)])
@pytest.mark.parametrize("system", SYSTEMS)
def test_looped_equals_one_shot_and_oracle(monkeypatch, system, nx, ny):
    for bc in ((TRANSMISSIVE, PERIODIC), (PERIODIC, TRANSMISSIVE)):
        P, q0 = _data(system, nx, ny, bc)
        ref = _run(monkeypatch, P, q0, 3, 0)
        for nc in (1, 2, 3, 5, 11, None):
            got = _run(monkeypatch, P, q0, 3, nc)
            assert np.array_equal(got["state"], ref["state"]) and got["t"] == ref["t"], (bc, nc)
        want, steps, t, st = orc.solve(P, q0, 0.0, 3)
        assert st == 0 and steps == 3
        assert_close(ref["state"], want, 1e-10, f"{system} {nx}x{ny} {bc}")


def _tiles(P, q0, k):
    big = P.with_(nx=P.nx * k, ny=P.ny * k, xhi=P.xhi * k, yhi=P.yhi * k)
    assert big.dx == P.dx and big.dy == P.dy
    return big, np.ascontiguousarray(np.tile(q0, (1, k, k)))


def _same_tiles(one, big, k, ny, nx):
    assert big["t"] == one["t"]
    for f in ("state", "rhs"):
        assert np.array_equal(big[f], np.tile(one[f], (1, k, k))), f
    assert np.array_equal(big["fx"][:, :, :-1], np.tile(one["fx"][:, :, :-1], (1, k, k)))
    assert np.array_equal(big["fy"][:, :-1, :], np.tile(one["fy"][:, :-1, :], (1, k, k)))


# 900 rows of 15 one-shot (or one-chunk) segments: 3375 blocks
@pytest.mark.parametrize("kind,chunks", [({}, 0), ({}, 1), ({}, None), (dict(order=5), None),
                                         (dict(weight_L=0.0, p=2.0), None), (dict(precision=1, eps=1e-20), None)],
                         ids=["one-shot", "one-chunk", "default", "r5", "js", "fp32"])
@pytest.mark.parametrize("system", SYSTEMS)
def test_scalar_sweeps_of_many_blocks(monkeypatch, system, kind, chunks):
    nt, k = 30, 30
    P, q0 = _data(system, nt, nt, (PERIODIC, PERIODIC))
    P = P.with_(**kind)
    one = _run(monkeypatch, P, q0, 3, chunks)
    Pk, qk = _tiles(P, q0, k)
    _same_tiles(one, _run(monkeypatch, Pk, qk, 3, chunks), k, nt, nt)


@pytest.mark.parametrize("kind", [{}, dict(weight_L=0.0, p=2.0), dict(p=1.5)], ids=["z", "js", "p15"])
def test_limited_sweeps_of_many_blocks(monkeypatch, kind):
    """Near-vacuum quadrants, periodic: the limiter acts from the first step.
    The tile's steps are checked against the oracle's by the limiter tests."""
    nt, k = 30, 30
    P, q0 = W.vacuum_quadrants_2d(nt)
    P = P.with_(pp_limiter=1, bc_x=PERIODIC, bc_y=PERIODIC, xlo=0.0, ylo=0.0, xhi=nt / 32.0, yhi=nt / 32.0, **kind)
    one = _run(monkeypatch, P, q0, 3)
    free = _run(monkeypatch, P.with_(pp_limiter=0), q0, 1)
    assert not np.array_equal(_run(monkeypatch, P, q0, 1)["state"], free["state"])   # it acts
    Pk, qk = _tiles(P, q0, k)
    _same_tiles(one, _run(monkeypatch, Pk, qk, 3), k, nt, nt)
