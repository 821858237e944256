"""GPU: what a call needs of the arena, and what it leaves of it.

A plain solve or closed loop whose precomputed normals find no room draws them in
the rollout, and gives what they took back when it returns: the same bits on any
arena that holds the applied inputs (12 S T bytes and a few percent).
"""
import numpy as np
import pytest

from paper_2508_05773_amd import brmppi as B
from paper_2508_05773_amd import workloads as W

pytestmark = pytest.mark.gpu


def problem(S, T, n_obs, flags=0):
    p = W.random_small(60 + n_obs, S=64, T=T, n_obs=n_obs)
    return p.copy(S=S, flags=flags)


def context(arena):
    return B.Context(arena_bytes=arena, n_streams=1, max_controllers=4, flags_extra=B.CTX_PROFILE_ROLLOUT)


def solve(c, p, controller=0):
    """(costs and sequence, launches of the noise kernel)"""
    c.set_path(controller, p.path, p.ds)
    B.brmppi_profile_reset(c.h)
    print(f"  S={p.S} T={p.T} n_obs={len(p.obstacles)} flags={p.flags}", flush=True)
    r = B.brmppi_solve_ex(c.h, B.ProblemBuffers(p, controller=controller), want_J=True)
    return r, B.brmppi_profile_read(c.h)["noise"]["count"]


def test_normals_without_room():
    """24.3 MB of normals are less than half of a 48.75 MB arena, but do not fit beside
    the 25.1 MB of the rest: drawn in the rollout, where 256 MiB take the buffer"""
    p = problem(20011, 100, 0, W.FLAG_GUIDANCE_OFF)
    with context(256 << 20) as c, context(48750000) as small:
        (want, n_want), (got, n_got) = solve(c, p), solve(small, p)
    assert (n_want, n_got) == (1, 0)
    assert np.array_equal(got["J"], want["J"]) and np.array_equal(got["U_new"], want["U_new"])


@pytest.mark.parametrize("S,T,n_obs", [(20011, 40, 12), (65536, 40, 2)])
def test_normals_are_given_back(S, T, n_obs):
    """after a solve with precomputed normals no more of the arena is in use than after
    one without"""
    p = problem(S, T, n_obs)
    used = []
    for shape in ((256, 0), (0, 0)):
        with context(1 << 30) as c:
            B.brmppi_set_launch(c.h, *shape)
            _, n = solve(c, p)
            assert n == (shape == (0, 0))
            used.append(B.brmppi_get_info(c.h)["arena_used"])
    assert used[1] <= used[0]


def test_normals_behind_the_kept_scratch():
    """a scratch kept from a larger call holds a smaller one's normals, also when the
    rest of the arena does not"""
    big, p = problem(45056, 100, 0, W.FLAG_GUIDANCE_OFF), problem(9000, 40, 12)
    with context(512 << 20) as c:
        want, _ = solve(c, p)
    with context(64 << 20) as c:
        B.brmppi_set_launch(c.h, 128, 0)
        solve(c, big)
        B.brmppi_set_launch(c.h, 0, 0)
        before = B.brmppi_get_info(c.h)
        got, n = solve(c, p, 1)
        after = B.brmppi_get_info(c.h)
    assert n == 1 and after["scratch_grows"] == before["scratch_grows"]
    assert np.array_equal(got["J"], want["J"]) and np.array_equal(got["U_new"], want["U_new"])


@pytest.mark.parametrize("S,T,n_obs,flags,arena", [(65536, 55, 32, 0, 1 << 30), (20011, 100, 0, W.FLAG_GUIDANCE_OFF, 48750000),
                                                   (20011, 40, 12, 0, 110 << 20)])
def test_closed_loop_in_a_small_arena(S, T, n_obs, flags, arena):
    """normals of one update past a quarter of the arena, without room at all, and of
    some updates of a chunk"""
    p = problem(S, T, n_obs, flags)
    got = []
    for a in (4 << 30, arena):
        with context(a) as c:
            c.set_path(0, p.path, p.ds)
            print(f"  S={S} T={T} n_obs={n_obs} arena={a >> 20} MiB", flush=True)
            got.append(B.brmppi_closed_loop(c.h, B.ProblemBuffers(p, controller=0), 19))
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])


@pytest.mark.parametrize("S,T,n_obs,flags,arena,ok", [
    (65536, 50, 8, 0, 512 << 20, True),                       # 41 MB, normals not counted
    (40000, 40, 8, 0, 512 << 20, True),
    (32768, 100, 0, W.FLAG_GUIDANCE_OFF, 512 << 20, True),
    (65536, 100, 0, W.FLAG_GUIDANCE_OFF, 512 << 20, False),   # 79 MB
    (8192, 100, 32, 0, 200 << 20, True),                      # normals above half the arena: not counted
    (20000, 100, 8, 0, 512 << 20, False),                     # 105 MB of normals
    (8192, 300, 0, W.FLAG_GUIDANCE_OFF, 512 << 20, True),     # 30 MB and as much of normals
    (8192, 400, 0, W.FLAG_GUIDANCE_OFF, 512 << 20, False),
])
def test_noalloc_limit(S, T, n_obs, flags, arena, ok):
    """the allocation-free solve takes what its stated limit allows, with or without
    room for the normals in its array, and gives the plain solve's bits"""
    p = problem(S, T, n_obs, flags)
    with context(arena) as c:
        c.set_path(0, p.path, p.ds)
        pb = B.ProblemBuffers(p, controller=0)
        print(f"  S={S} T={T} n_obs={n_obs} flags={flags}", flush=True)
        u, _, rc = B.brmppi_solve_noalloc(c.h, pb, allow=(B.OK, B.ENOMEM))
        assert rc == (B.OK if ok else B.ENOMEM)
        if ok:
            u = u.copy()
            assert np.array_equal(u, B.brmppi_solve(c.h, pb)[0])


@pytest.mark.parametrize("n_obs", [0, 2, 3, 8, 9, 16, 17, 32])
@pytest.mark.parametrize("T", [20, 60, 90])
def test_drawn_for_lack_of_room(n_obs, T):
    """8300 samples (a partial tile in every form) whose normals exceed half the arena:
    the rollout draws them itself, on one lane up to eight rows, two up to 16, four up
    to 32, with tiles that reduce themselves (T = 20; 60 on four lanes) and without.
    The bits of the buffered form; the launch counts tell the two apart."""
    p = problem(8300, T, n_obs)
    normals = 4 * (5 + n_obs) * T * 8448
    sequences = 4 * 3 * T * 8448
    room = int(1.05 * sequences) + (600 << 10)
    small = min(2 * normals - 4096, room + normals)
    assert small >= room
    with context(512 << 20) as a, context(small) as b:
        (want, n_want), (got, n_got) = solve(a, p), solve(b, p)
    assert (n_want, n_got) == (1, 0)
    assert np.array_equal(got["J"], want["J"]) and np.array_equal(got["U_new"], want["U_new"])
