"""GPU: the resolution of headings, at quarter turns and away from them, and of
progress.

At rest, with the heading terms alone in the cost, a sample of one step costs
2 (Q1 e1^2 + Q2 e2^2), e1 and e2 the start headings' distances from the path's.
Headings are held in revolutions from the quarter turn nearest the start heading, so
an angle of up to an eighth of a turn has half a unit in the last place of 2^-28
revolutions, 2.3e-8 rad, and start and path are rounded twice each: 9.4e-8 rad of
1e-3 is a relative 1.9e-4 of the cost.
"""
import numpy as np
import pytest

from paper_2508_05773_amd import brmppi as B
from paper_2508_05773_amd import workloads as W

pytestmark = pytest.mark.gpu

HEADINGS = [0.0, 0.3, 0.78, 1.5709, 1.62, 1.7, 2.0, 3.1417, 3.15, 3.2, 3.3, -1.5709, -1.7, -3.15, -3.3, 4.8, 6.4, 20.0]


def wrap(x):
    return x - 2 * np.pi * np.round(x / (2 * np.pi))


@pytest.mark.parametrize("S,shape", [(64, (0, 0)), (65, (256, 0)), (9000, (0, 0))])
@pytest.mark.parametrize("turn", [0.0, 6.283185307179586])
def test_heading_costs(S, shape, turn):
    """(turn: the path's headings a whole turn further than the start's)"""
    with B.Context(arena_bytes=64 << 20, n_streams=1, max_controllers=1) as c:
        B.brmppi_set_launch(c.h, *shape)
        for th in HEADINGS:
            p = W.random_small(7, S=64, T=1, n_obs=0)
            path = p.path.copy()
            path[:, 2] = np.float32(th + turn)
            path[:, 3] = np.float32(th + turn + 0.01)
            x0 = p.x0.copy()
            x0[2:4] = 0.0
            x0[4] = np.float32(path[0, 2] - np.float32(turn)) + np.float32(1e-3)
            x0[5] = np.float32(path[0, 3] - np.float32(turn)) - np.float32(1e-3)
            q = dict(p.params, Qc=0.0, Ql=0.0, Qth1=3.0, Qth2=2.0, R_j=0.0, R_w=0.0, mu=0.0)
            p = p.copy(S=S, path=path, x0=x0, params=q, flags=W.FLAG_GUIDANCE_OFF)
            e1 = wrap(np.float64(x0[4]) - np.float64(path[0, 2]))
            e2 = wrap(np.float64(x0[5]) - np.float64(path[0, 3]))
            want = 2.0 * (3.0 * e1**2 + 2.0 * e2**2)
            c.set_path(0, p.path, p.ds)
            J = B.brmppi_solve_ex(c.h, B.ProblemBuffers(p, controller=0), want_J=True)["J"]
            err = np.max(np.abs(J - want) / want)
            print(f"  S={S} heading {th} + {turn:.2f}: {err:.1e}", flush=True)
            assert err <= 2e-4, th


@pytest.mark.parametrize("shape", [(256, 0), (0, 0)])
def test_terminal_heading(shape):
    """The sine and cosine of the terminal cost's reference heading are the library's.
    At rest on the first waypoint, one step of progress away from the second, 10 m off:
    the contour error there is 10 m times a sine and cosine product, and a sample's
    cost its square.  With correctly rounded functions its root mean square error over
    400 headings is 3.2e-8 of the distance, with the hardware's (3.0 to 3.4e-8 rms)
    4.2 to 4.8e-8: the bar lies between."""
    rng = np.random.default_rng(3)
    q = None
    err = []
    with B.Context(arena_bytes=64 << 20, n_streams=1, max_controllers=1) as c:
        B.brmppi_set_launch(c.h, *shape)
        for _ in range(400):
            p = W.random_small(7, S=64, T=1, n_obs=0)
            th, way = np.float32(rng.uniform(-3.1, 3.1)), rng.uniform(-np.pi, np.pi)
            xy = np.float32([10 * np.cos(way), 10 * np.sin(way)])
            path = np.zeros((3, 4), np.float32)
            path[:, :2] = np.arange(3, dtype=np.float32)[:, None] * xy
            path[:, 2:] = th
            x0 = np.zeros(8, np.float32)
            x0[4:6] = np.float32(th + rng.uniform(-0.7, 0.7))
            q = q or dict(p.params, Ts=0.5, sigma_nu=0.0, Qc=1.0, Ql=0.0, Qth1=0.0, Qth2=0.0, R_j=0.0, R_w=0.0, mu=0.0)
            p = p.copy(path=path, ds=0.5, x0=x0, params=q, u_nom=np.float32([[0.0, 0.0, 1.0]]), flags=W.FLAG_GUIDANCE_OFF)
            c.set_path(0, p.path, p.ds)
            J = B.brmppi_solve_ex(c.h, B.ProblemBuffers(p, controller=0), want_J=True)["J"].astype(np.float64)
            h, e = np.float64(th), -xy.astype(np.float64)
            err.append((np.sqrt(J[0]) - abs(np.sin(h) * e[0] - np.cos(h) * e[1])) / 10)
    rms = np.sqrt(np.mean(np.square(err)))
    print(f"  rms {rms:.2e} of the distance", flush=True)
    assert rms <= 3.9e-8


@pytest.mark.parametrize("S,shape", [(64, (0, 0)), (65, (256, 0)), (9000, (0, 0))])
def test_progress(S, shape):
    """At rest on a straight path with progress of 1/16 m a step, exact in FP32 over 512
    steps, the lag errors are the progress itself.  Its waypoint index is rounded twice
    (1/ds and the product), the point and the error once each, the square once: 4.5
    units of 2^-24, twice that in the square, 5.4e-7 of the cost."""
    T = 512
    p = W.random_small(7, S=64, T=1, n_obs=0)
    path = np.zeros((400, 4), np.float32)
    path[:, 0] = np.float32(0.3) * np.arange(400, dtype=np.float32)
    u = np.zeros((T, 3), np.float32)
    u[:, 2] = 1.0
    q = dict(p.params, Ts=0.0625, sigma_j=0.0, sigma_w=0.0, sigma_nu=0.0, Qc=0.0, Ql=1.0, Qth1=0.0, Qth2=0.0, R_j=0.0, R_w=0.0,
             mu=0.0)
    p = p.copy(S=S, T=T, path=path, ds=float(np.float32(0.3)), x0=np.zeros(8, np.float32), params=q, u_nom=u, flags=W.FLAG_GUIDANCE_OFF)
    f = np.arange(T + 1) * 0.0625 / np.float64(np.float32(0.3))
    want = np.sum(np.interp(f, np.arange(400), path[:, 0].astype(np.float64)) ** 2)
    with B.Context(arena_bytes=256 << 20, n_streams=1, max_controllers=1) as c:
        B.brmppi_set_launch(c.h, *shape)
        c.set_path(0, p.path, p.ds)
        J = B.brmppi_solve_ex(c.h, B.ProblemBuffers(p, controller=0), want_J=True)["J"].astype(np.float64)
    print(f"  S={S}: {np.max(np.abs(J - want)) / want:.1e}", flush=True)
    assert np.max(np.abs(J - want)) <= 5.4e-7 * want
