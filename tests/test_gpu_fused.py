"""GPU: the fused 2D Euler stage (both sweeps of a stage in one kernel, strips
of at most 63 columns, bands of rows, four interface rows per step) at the
edges of its tiles: widths around one and two strips and around the halo
columns that one wavefront loads in turn, heights around one step and one
band, grids narrower than a stencil, both boundary conditions, every order
and weight kind, and both precisions.  Right-hand sides against the oracle
at the bar of the other right-hand-side tests (1e-11 of the component scale;
FP32 reconstruction: 3e-5 of the flux scale over the cell size), three steps
at the state bar (1e-10, FP64)."""
import numpy as np
import pytest

import oracle as orc
from paper_2603_26272_amd import workloads as W
from paper_2603_26272_amd.problem import PERIODIC, TRANSMISSIVE

from tests.test_gpu_parity import assert_close

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [(1, 1), (2, 5), (5, 2), (7, 3), (57, 4), (58, 7), (59, 8), (62, 3), (63, 5), (64, 11), (65, 12), (125, 4),
          (126, 6), (127, 33), (190, 9), (16, 130)]
KINDS = [dict(), dict(order=2), dict(order=4), dict(order=5), dict(weight_L=0.0, p=2.0), dict(affine_invariant=1),
         dict(p=1.5), dict(order=5, weight_L=0.0, p=2.0), dict(precision=1, eps=1e-20, mu0=1e-8),
         dict(precision=1, eps=1e-20, mu0=1e-8, weight_L=0.0, p=2.0), dict(lf=1)]


def _data(nx, ny):
    P, q0 = W.quadrants_2d(nx + 5 * ny, max(nx, 2), max(ny, 2))
    q0 = np.ascontiguousarray(q0[:, :ny, :nx])
    # a ripple rules out exactly tied indicators on tiny and periodic grids
    x = np.arange(nx)[None, :] + 0.37 * np.arange(ny)[:, None]
    q0[0] *= 1 + 1e-2 * np.sin(1.3 * x + 0.2)
    return P.with_(nx=nx, ny=ny, xhi=nx / 64.0, yhi=ny / 64.0), q0


@pytest.mark.parametrize("kind", KINDS, ids=lambda k: "-".join(f"{a}{b}" for a, b in k.items()) or "z")
@pytest.mark.parametrize("bc", [TRANSMISSIVE, PERIODIC])
def test_rhs_and_steps_against_oracle(kind, bc):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_26272_amd.za import Context, rhs_noalloc
    for nx, ny in SHAPES:
        P, q0 = _data(nx, ny)
        P = P.with_(bc_x=bc, bc_y=bc, **kind)
        f32 = P.precision == 1
        tag = f"{nx}x{ny} {kind}"
        ref, st = orc.rhs(P, q0)
        assert st == 0
        q = torch.from_numpy(q0).cuda()
        with Context(P) as ctx:
            got = ctx.rhs(q).cpu().numpy()
            info = ctx.solve(q, 0.0, 3)
        alone = rhs_noalloc(P, torch.from_numpy(q0).cuda()).cpu().numpy()
        assert np.array_equal(alone, got), tag
        if f32:
            fx, fy, _ = orc.fluxes(P, q0)
            scale = np.abs(fx).max(axis=(1, 2), keepdims=True) + np.abs(fy).max(axis=(1, 2), keepdims=True)
            assert (np.abs(got - ref) <= 3e-5 * 64.0 * 2.0 * scale).all(), tag
        else:
            assert_close(got, ref, 1e-11 if nx > 5 and ny > 5 else 1e-10, tag)
        rq, steps, t, st = orc.solve(P, q0, 0.0, 3)
        assert st == 0 and info["steps"] == 3 == steps
        if not f32:   # (FP32 states: the FP32 tests of test_gpu_parity and test_gpu_large)
            assert_close(q.cpu().numpy(), rq, 1e-10, tag)


def test_bands_do_not_change_the_result():
    """A tall grid (many bands and steps per band) equals its pieces: a
    periodic tile repeated vertically gives the tile's right-hand side."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_26272_amd.za import Context
    P, q0 = _data(130, 37)
    P = P.with_(bc_x=PERIODIC, bc_y=PERIODIC)
    with Context(P) as ctx:
        one = ctx.rhs(torch.from_numpy(q0).cuda()).cpu().numpy()
    for k in (7, 61):
        Pk = P.with_(ny=37 * k, yhi=P.yhi * k)
        with Context(Pk) as ctx:
            got = ctx.rhs(torch.from_numpy(np.tile(q0, (1, k, 1))).cuda()).cpu().numpy()
        if Pk.dy == P.dy:
            assert np.array_equal(got, np.tile(one, (1, k, 1)))
        else:
            assert_close(got, np.tile(one, (1, k, 1)), 1e-12, f"{k} tiles")


@pytest.mark.parametrize("kind", [dict(order=4, weight_L=0.0, p=2.0), dict(order=4, p=1.5), dict(order=2, p=1.5)],
                         ids=["r4-js", "r4-p15", "r2-p15"])
def test_kernels_of_few_and_many_blocks_agree_bitwise(kind):
    """Some weights run one kernel where few blocks share a CU and another, of
    fewer registers, where many do: a periodic tile gives the same bits
    through either."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_26272_amd.za import Context
    P, q0 = _data(128, 32)
    P = P.with_(bc_x=PERIODIC, bc_y=PERIODIC, **kind)
    k = 128                                  # 33 blocks, then more than two per CU
    Pk = P.with_(ny=32 * k, yhi=P.yhi * k)
    assert Pk.dy == P.dy
    out = []
    for Pi, qi in ((P, q0), (Pk, np.tile(q0, (1, k, 1)))):
        q = torch.from_numpy(qi).cuda()
        with Context(Pi) as ctx:
            rhs = ctx.rhs(q).cpu().numpy()
            ctx.solve(q, 0.0, 3)
        out.append((rhs, q.cpu().numpy()))
    for a, b in zip(*out):
        assert np.array_equal(np.tile(a, (1, k, 1)), b)


@pytest.mark.parametrize("kind", [dict(precision=1, eps=1e-20, mu0=1e-8),
                                  dict(precision=1, eps=1e-20, mu0=1e-8, weight_L=0.0, p=2.0),
                                  dict(precision=1, eps=1e-20, mu0=1e-8, p=1.5)], ids=["z", "js", "p15"])
@pytest.mark.parametrize("bc", [TRANSMISSIVE, PERIODIC])
def test_fp32_stages(kind, bc):
    """One step with FP32 reconstruction (whose stages reload the FP64 state
    for the update) at the edges of the tiles, against the oracle's FP32
    reading and against the step put together from right-hand sides.

    Oracle: each flux agrees to 3e-5 of its component scale S_F, so a stage's
    update to 4 * 3e-5 * S_F dt / dx over both faces and directions, and the
    step to three times that.  Right-hand sides: stage states that differ in
    an FP64 rounding give the same FP32 records but where a value sits on a
    rounding boundary; one such flip (2^-24) moves a flux by at most 8 * 2^-23
    of its scale, hence 4 * 1e-6 * S_F dt / dx."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_26272_amd.za import Context
    for nx, ny in SHAPES:
        P, q0 = _data(nx, ny)
        P = P.with_(bc_x=bc, bc_y=bc, **kind)
        q = torch.from_numpy(q0).cuda()
        with Context(P) as ctx:
            dt = ctx.step(q, 0.0, sync=True)
            L = lambda u: ctx.rhs(torch.from_numpy(u).cuda()).cpu().numpy()
            q1 = q0 + dt * L(q0)
            q2 = 0.75 * q0 + 0.25 * (q1 + dt * L(q1))
            q3 = q0 / 3.0 + (2.0 / 3.0) * (q2 + dt * L(q2))
        got = q.cpu().numpy()
        ref, dt_ref, st = orc.step(P, q0, dt)
        assert st == 0
        fx, fy, _ = orc.fluxes(P, q0)
        SF = np.maximum(np.abs(fx).max(axis=(1, 2), keepdims=True), np.abs(fy).max(axis=(1, 2), keepdims=True))
        SQ = np.abs(q0).max(axis=(1, 2), keepdims=True)
        unit = 4.0 * SF * dt / P.dx
        assert (np.abs(got - ref) <= 3 * 3e-5 * unit + 1e-10 * SQ).all(), (nx, ny)
        assert (np.abs(got - q3) <= 1e-6 * unit + 1e-13 * SQ).all(), (nx, ny)


FLUX_KINDS = [dict(), dict(weight_L=0.0, p=2.0), dict(affine_invariant=1), dict(p=1.5), dict(alt_tau=1), dict(lf=1),
              dict(linear_weights=1)] + [dict(order=r, **w) for r in (2, 4, 5)
                                         for w in (dict(), dict(weight_L=0.0, p=2.0), dict(p=1.5))]


@pytest.mark.parametrize("kind", FLUX_KINDS, ids=lambda k: "-".join(f"{a}{b}" for a, b in k.items()) or "z")
def test_rhs_at_the_flux_bar(kind):
    """The fused kernel has no flux output (za_rhs_fluxes runs the separate
    sweeps), so its fluxes are held to their bar through the right-hand side:
    every cell within what the bar of 1e-12 (|F| + max |F|) allows its four
    faces, against the oracle's fluxes, and twice that against the library's
    own flux output."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_26272_amd.za import Context
    for (nx, ny), bc in (((63, 65), TRANSMISSIVE), ((130, 67), PERIODIC)):
        P, q0 = W.quadrants_2d(nx * 7 + ny, nx, ny)
        q0 = np.ascontiguousarray(q0)
        q0[0] *= 1.0 + 1e-2 * np.random.default_rng(nx).random(q0[0].shape)   # rules out tied indicators
        P = P.with_(bc_x=bc, bc_y=bc, **kind)
        q = torch.from_numpy(q0).cuda()
        with Context(P) as ctx:
            got = ctx.rhs(q).cpu().numpy()
            own = [f.cpu().numpy() for f in ctx.rhs_fluxes(q)]
        fx, fy, st = orc.fluxes(P, q0)
        assert st == 0
        bx, by = (1e-12 * (np.abs(f) + np.abs(f).max(axis=(1, 2), keepdims=True)) for f in (fx, fy))
        bar = (bx[:, :, 1:] + bx[:, :, :-1]) / P.dx + (by[:, 1:, :] + by[:, :-1, :]) / P.dy
        for k, (gx, gy) in ((1, (fx, fy)), (2, own)):
            ref = -(gx[:, :, 1:] - gx[:, :, :-1]) / P.dx - (gy[:, 1:, :] - gy[:, :-1, :]) / P.dy
            assert (np.abs(got - ref) <= k * bar).all(), (nx, ny, k, float((np.abs(got - ref) / bar).max()))
