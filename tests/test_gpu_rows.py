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
