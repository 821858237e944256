"""GPU: the obstacle rows at the edges of their slots and row kinds.

Every count of obstacles at which a kernel's slots, pairs of rows or lanes of a
sample run out (0, 1, 2, 3, ... 32), with ellipses at rest, some of them moving,
and some super-ellipses: each sample's cost against the FP64 oracle at the
stated bar (relative 1e-4, FP32 against FP64), and every launch shape's costs
and nominal sequence bit for bit the same.
"""
import os
import sys

import numpy as np
import pytest

from paper_2508_05773_amd import brmppi as B
from paper_2508_05773_amd import workloads as W

pytestmark = pytest.mark.gpu

J_RTOL = 1e-4
SHAPES = [(256, 0), (64, 0), (256, 1), (256, 2), (256, 3), (256, 4), (64, 4)]


@pytest.fixture(scope="module")
def ctx():
    c = B.Context(arena_bytes=256 << 20, n_streams=1, max_controllers=4)
    yield c
    c.close()


def problem(kind, n_obs, flags=0):
    p = W.random_small(40 + n_obs, S=67, T=9, n_obs=n_obs, moving=False)
    obs = p.obstacles.copy()
    if kind != "rest":
        obs[::3, 6:8] = (0.7, -0.9)
    if kind == "e4":
        obs[1::2, 5] = 4.0
    return p.copy(obstacles=obs, flags=flags)


@pytest.mark.parametrize("kind", ["rest", "moving", "e4"])
@pytest.mark.parametrize("n_obs", [0, 1, 2, 3, 7, 8, 9, 15, 16, 17, 31, 32])
def test_rows_at_slot_edges(ctx, kind, n_obs):
    from oracle import oracle as O

    for flags in (0, W.FLAG_HITCH_OFF, W.FLAG_GUIDANCE_OFF | W.FLAG_COLLISION_PENALTY):
        p = problem(kind, n_obs, flags)
        ctx.set_path(0, p.path, p.ds)
        want = O.solve(p, nthreads=min(8, os.cpu_count() or 1))
        first = None
        for block, variant in SHAPES:
            print(f"  rows {kind} n_obs={n_obs} flags={flags} shape=({block},{variant})", flush=True)
            sys.stdout.flush()
            B.brmppi_set_launch(ctx.h, block, variant)
            try:
                got = B.brmppi_solve_ex(ctx.h, B.ProblemBuffers(p, controller=0), want_J=True)
            finally:
                B.brmppi_set_launch(ctx.h, 0, 0)
            assert np.max(np.abs(got["J"] - want["J"]) / np.abs(want["J"])) <= J_RTOL
            if first is None:
                first = got
            else:
                assert np.array_equal(got["J"], first["J"])
                assert np.array_equal(got["U_new"], first["U_new"])


def test_batch_of_every_form(ctx):
    """One batch over every bucket, row kind and lane count: bit for bit the
    plain solves."""
    with B.Context(arena_bytes=512 << 20, n_streams=1, max_controllers=64) as c:
        probs = []
        for kind in ("rest", "moving", "e4"):
            for n_obs in (0, 2, 3, 8, 9, 16, 17, 32):
                probs.append(problem(kind, n_obs))
        probs.append(problem("e4", 5, W.FLAG_GUIDANCE_OFF | W.FLAG_COLLISION_PENALTY))
        prm = W.make_params(0.05, disc_tractor=(0.0, 2.0), disc_trailer=(1.5,))
        for n_obs in (1, 3, 5, 10):
            p = problem("e4", n_obs)
            p.params.update(prm)
            probs.append(p)
        pbs = []
        for i, p in enumerate(probs):
            q = p.copy(S=65 + 61 * i, T=5 + i % 7, u_nom=p.u_nom[:1].repeat(5 + i % 7, axis=0))
            c.set_path(i, q.path, q.ds)
            pbs.append(B.ProblemBuffers(q, controller=i))
        plain = [B.brmppi_solve(c.h, pb)[0].copy() for pb in pbs]
        for block in (0, 64, 192):
            B.brmppi_set_launch(c.h, block, 0)
            got = B.brmppi_solve_batch(c.h, pbs)[0]
            for i, (u, v) in enumerate(zip(got, plain)):
                assert np.array_equal(u, v), (block, i)
        B.brmppi_set_launch(c.h, 0, 0)


@pytest.mark.parametrize("n_obs", [9, 16, 17, 32])
def test_no_room_for_normals(ctx, n_obs):
    """A plain solve whose normals do not fit half the arena draws them in the
    kernel, several lanes per sample: the same bits."""
    p = problem("moving", n_obs).copy(S=1030, T=60, u_nom=np.zeros((60, 3), np.float32))
    ctx.set_path(0, p.path, p.ds)
    want = B.brmppi_solve_ex(ctx.h, B.ProblemBuffers(p, controller=0), want_J=True)
    with B.Context(arena_bytes=6 << 20, n_streams=1, max_controllers=2) as c:
        c.set_path(0, p.path, p.ds)
        got = B.brmppi_solve_ex(c.h, B.ProblemBuffers(p, controller=0), want_J=True)
    assert np.array_equal(got["J"], want["J"])
    assert np.array_equal(got["U_new"], want["U_new"])


@pytest.mark.parametrize("S", [1, 33, 1024, 1025])
def test_one_group_and_two(ctx, S):
    """Up to 1024 samples an instance is merged by the block that merges its one
    group: bit for bit the batch's separate reduction, update after update, with
    either log of the closed loop."""
    p = problem("moving", 3).copy(S=S)
    ctx.set_path(0, p.path, p.ds)
    ctx.set_path(1, p.path, p.ds)
    x, u = B.brmppi_closed_loop(ctx.h, B.ProblemBuffers(p, controller=0), 3)
    B.brmppi_set_state(ctx.h, 1, p.x0.astype(np.float64))
    for k in range(3):
        pb = B.ProblemBuffers(p, controller=1, with_nominal=(k == 0), seed=p.seed + k,
                              flags=p.flags | B.X0_RESIDENT | B.ADVANCE_PLANT)
        assert np.array_equal(B.brmppi_solve_batch(ctx.h, [pb])[0][0][0], u[k])
        assert np.array_equal(B.brmppi_get_state(ctx.h, 1), x[k + 1])
    ctx.set_path(0, p.path, p.ds)
    assert np.array_equal(B.brmppi_closed_loop(ctx.h, B.ProblemBuffers(p, controller=0), 3, want_u=False)[0], x)
    ctx.set_path(0, p.path, p.ds)
    assert np.array_equal(B.brmppi_closed_loop(ctx.h, B.ProblemBuffers(p, controller=0), 3, want_x=False)[1], u)


@pytest.mark.parametrize("S,T", [(67, 120), (70001, 2), (300001, 1)])
def test_downloads_in_pieces(ctx, S, T):
    """Costs and applied sequences that reach the caller in several pieces: ends
    of pieces in a row's padding, rows longer than a piece, costs past the size
    that the rollout writes to the host itself.  Against the FP64 oracle at the
    stated bars (costs 1e-4 relative, inputs 1e-4 of their range)."""
    from oracle import oracle as O
    p = problem("rest", 0, W.FLAG_GUIDANCE_OFF).copy(S=S, T=T, u_nom=np.zeros((T, 3), np.float32))
    ctx.set_path(0, p.path, p.ds)
    want = O.solve(p, nthreads=min(8, os.cpu_count() or 1), want_useq=True)
    got = B.brmppi_solve_ex(ctx.h, B.ProblemBuffers(p, controller=0), want_J=True, want_useq=True)
    only = B.brmppi_solve_ex(ctx.h, B.ProblemBuffers(p, controller=0), want_J=True)
    tol = 1e-4 * np.array([4.0, 1.8, p.params["nu_bar"]])
    assert np.max(np.abs(got["J"] - want["J"]) / np.abs(want["J"])) <= J_RTOL
    assert np.all(np.abs(got["useq"].reshape(T, 3, S).transpose(2, 0, 1) - want["useq"]) <= tol)
    assert np.array_equal(only["J"], got["J"])


@pytest.mark.parametrize("n_obs", [0, 2, 8, 16, 32])
def test_normals_drawn_in_runs(ctx, n_obs):
    """Eight lanes per sample with the normals drawn by the rollout's launch, as
    many steps at a time as LDS holds: one step, an odd last step, one to several
    runs, the longest horizons that it takes and the first that it leaves to the
    noise kernel, a partial tile, the largest sample count and the first above
    it.  Bit for bit the four-lane form with the noise kernel."""
    for S, T in ((1, 1), (33, 2), (65, 11), (100, 24), (100, 25), (100, 49), (100, 50), (64, 155), (64, 156), (64, 217), (8191, 3), (8193, 3)):
        p = problem("moving", n_obs).copy(S=S, T=T, u_nom=np.full((T, 3), 0.1, np.float32))
        ctx.set_path(0, p.path, p.ds)
        print(f"  n_obs={n_obs} S={S} T={T}", flush=True)
        got = []
        for shape in ((256, 4), (256, 3)):
            B.brmppi_set_launch(ctx.h, *shape)
            try:
                got.append(B.brmppi_solve_ex(ctx.h, B.ProblemBuffers(p, controller=0), want_J=True))
            finally:
                B.brmppi_set_launch(ctx.h, 0, 0)
        assert np.array_equal(got[0]["J"], got[1]["J"])
        assert np.array_equal(got[0]["U_new"], got[1]["U_new"])


def test_noalloc_limit_counts_the_normals(ctx):
    """The scratch limit of the allocation-free solve is the stated one, normals
    included, whichever launch draws them."""
    for T, rc_want in ((30, B.OK), (100, B.ENOMEM)):
        p = problem("rest", 32).copy(S=8192, T=T, u_nom=np.zeros((T, 3), np.float32))
        ctx.set_path(0, p.path, p.ds)
        rc = B.brmppi_solve_noalloc(ctx.h, B.ProblemBuffers(p, controller=0), allow=(B.OK, B.ENOMEM))[2]
        assert rc == rc_want, T


@pytest.mark.parametrize("S,T,n_obs,drawn", [
    (3000, 12, 7, True), (8191, 3, 7, True), (8193, 12, 7, False),       # up to a block per CU
    (8192, 162, 32, True), (8192, 163, 32, False), (600, 162, 0, True), (600, 163, 0, False),   # the epilogue's LDS
    (256, 40, 32, True), (256, 60, 32, True), (256, 81, 32, False), (255, 60, 32, False), (256, 162, 32, False),   # runs
])
def test_which_launch_draws(S, T, n_obs, drawn):
    """The default form at the edges of what the rollout's own launch draws (its noise
    is counted without a time; the noise kernel's has one), and the four-lane form's
    bits in either."""
    p = problem("moving", n_obs).copy(S=S, T=T, u_nom=np.full((T, 3), 0.1, np.float32))
    with B.Context(arena_bytes=512 << 20, n_streams=1, max_controllers=4, flags_extra=B.CTX_PROFILE_ROLLOUT) as c:
        c.set_path(0, p.path, p.ds)
        print(f"  n_obs={n_obs} S={S} T={T}", flush=True)
        got = B.brmppi_solve_ex(c.h, B.ProblemBuffers(p, controller=0), want_J=True)
        prof = B.brmppi_profile_read(c.h)
        assert prof["rollout"]["count"] == 1 and prof["noise"]["count"] == 1
        assert (prof["noise"]["ms"] == 0.0) == drawn
        B.brmppi_set_launch(c.h, 256, 3)
        want = B.brmppi_solve_ex(c.h, B.ProblemBuffers(p, controller=0), want_J=True)
    assert np.array_equal(got["J"], want["J"]) and np.array_equal(got["U_new"], want["U_new"])


@pytest.mark.parametrize("S", [65535, 65536, 65537])
def test_downloads_at_the_piece_size(ctx, S):
    """Applied sequences whose rows are just under, exactly and just over the size from
    which they are copied whole.  Against the FP64 oracle at the stated bars, as above."""
    test_downloads_in_pieces(ctx, S, 2)


def test_batches_without_guidance(ctx):
    """Batches of unguided instances, with and without the penalty, over the kinds of
    rows that the penalty tells apart: bit for bit the plain solves, also where a batch
    of the same sizes has a guided instance."""
    with B.Context(arena_bytes=512 << 20, n_streams=1, max_controllers=64) as c:
        prm = W.make_params(0.05, disc_tractor=(0.0, 2.0), disc_trailer=(1.5,))
        probs = []
        for flags in (W.FLAG_GUIDANCE_OFF, W.FLAG_GUIDANCE_OFF | W.FLAG_COLLISION_PENALTY):
            for kind in ("rest", "moving", "e4"):
                for n_obs in (0, 3, 4, 9, 32):
                    probs.append(problem(kind, n_obs, flags))
            p = problem("e4", 7, flags)
            p.params.update(prm)
            probs.append(p)
        pbs = []
        for i, p in enumerate(probs):
            q = p.copy(S=1 + 67 * i, T=1 + i % 9, u_nom=p.u_nom[:1].repeat(1 + i % 9, axis=0))
            c.set_path(i, q.path, q.ds)
            pbs.append(B.ProblemBuffers(q, controller=i))
        guided = problem("moving", 9)
        c.set_path(63, guided.path, guided.ds)
        plain = [B.brmppi_solve(c.h, pb)[0].copy() for pb in pbs]
        for block in (0, 64, 192):
            B.brmppi_set_launch(c.h, block, 0)
            for extra in ([], [B.ProblemBuffers(guided, controller=63)], []):
                got = B.brmppi_solve_batch(c.h, pbs + extra)[0]
                for i, v in enumerate(plain):
                    assert np.array_equal(got[i], v), (block, len(extra), i)
        B.brmppi_set_launch(c.h, 0, 0)
