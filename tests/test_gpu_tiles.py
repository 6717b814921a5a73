"""The 4 x 4 tiles at the sizes where they can go wrong, against the oracle:
chains that end inside a tile, the first chains with inner splits, budgets
around a wave and around the windows, shifts within their overlap, past it and
beyond whole windows, and the three kinds of keys; and that large sizes and
many budgets do not make tiles walk their budgets in turn."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_1911_13214_amd import chaingen

pytestmark = pytest.mark.gpu


def check(params, M, schedule="diagonal"):
    from gpu_util import chain_tables, solve_on_gpu

    print(f"tiles L={params.shape[-1]} M={M} n={params.shape[0]} {schedule}", flush=True)
    _, cost, dec = solve_on_gpu(params, M, schedule=schedule)
    for c in range(params.shape[0]):
        C, D = orc.solve(params[c], M)
        gc, gd = chain_tables(cost, dec, c, params.shape[-1], M)
        assert np.array_equal(gc, C) and np.array_equal(gd, D), c


# costs x 2^0: 32-bit keys; x 2^14 (L = 70): 4-byte values that leave no room
# for them; x 2^26: 64-bit values
@pytest.mark.parametrize("shift", [0, 14, 26])
@pytest.mark.parametrize("L,M", [(1, 0), (2, 64), (3, 63), (4, 65), (5, 127), (8, 128), (9, 200), (12, 191), (13, 192),
                                 (16, 300), (17, 301), (29, 511), (70, 257)])
def test_tile_edges(L, M, shift):
    p = chaingen.random_chains(2, L, seed=100 + L)
    p[:, :2] <<= shift
    check(p, M)


# windows of 320 and 512 budgets, their overlaps of 128 and 192 and budgets one
# around their ends; sizes x 1 stay within the overlap, the larger ones reach
# past it (windows apart, a launch after another) and past whole windows
@pytest.mark.parametrize("scale", [1, 4, 30])
@pytest.mark.parametrize("L,M", [(22, 319), (22, 320), (23, 448), (22, 511), (24, 575), (33, 703), (33, 704),
                                 (45, 1023), (45, 1024), (50, 1151), (90, 2000)])
def test_tile_windows(L, M, scale):
    p = chaingen.random_chains(1, L, seed=200 + L)
    p[:, 2:] *= scale
    check(p, M)


# batches whose tile-diagonals go from budgets in turn to windows as they get
# fewer than 128 tiles
@pytest.mark.parametrize("n,L,M", [(9, 75, 330), (20, 50, 600), (40, 21, 900)])
def test_tile_windows_change(n, L, M):
    check(chaingen.random_chains(n, L, seed=300 + L), M)


# chains of one call whose windows overlap and chains whose windows lie apart,
# also where budgets in turn come before, and chains of one block, which have
# no overlap
@pytest.mark.parametrize("n,L,M", [(1, 8, 400), (1, 11, 511), (2, 16, 500), (3, 40, 330), (3, 30, 1023), (2, 61, 1464),
                                   (12, 45, 600), (30, 22, 700), (2, 66, 5119)])
def test_windows_apart_beside_overlapping_ones(n, L, M):
    p = chaingen.random_chains(n, L, seed=800 + L)
    p[::2, 2:] *= 40
    check(p, M)


# the edges of the blocked order by windows that lie apart: one pass each, two
# passes each, beside chains whose windows overlap
@pytest.mark.parametrize("n,L,M", [(2, 53, 700), (3, 37, 880), (2, 70, 1600), (1, 130, 2047)])
def test_block_edges_apart_beside_overlapping_ones(n, L, M):
    p = chaingen.random_chains(n, L, seed=1200 + L)
    p[::2, 2:] *= 25
    check(p, M, "blocked")


# a chain outside the domain (negative, huge and 32-bit sizes) among windows
# that overlap and lie apart: its neighbours' tables are the oracle's
@pytest.mark.parametrize("schedule", ["diagonal", "blocked"])
def test_windows_beside_a_chain_out_of_the_domain(schedule):
    import torch

    from gpu_util import chain_tables
    from paper_1911_13214_amd import rotor
    L, M = 40, 700
    p = chaingen.random_chains(4, L, seed=1250)
    p[3, 2:] *= 40
    p[1, chaingen.WA, 7], p[1, chaingen.WABAR, 12] = -9, 1 << 62
    p[2, chaingen.WA, 20], p[2, chaingen.WABAR, 30], p[2, chaingen.UF, 9] = (1 << 32) + 3, -7, -100
    print(f"domain L={L} M={M} {schedule}", flush=True)
    d_params = torch.from_numpy(p).to("cuda")
    cost, dec = rotor.alloc_tables(4, L, M)
    work = rotor.alloc_workspace(4, L, M)
    rotor.rotor_solve_schedule(d_params, 4, L, M, cost, dec, work, schedule)
    torch.cuda.synchronize()
    st, per = rotor.rotor_solve_status(work, 4, L, M)
    assert st == rotor.ROTOR_EDOMAIN
    assert per.tolist() == [rotor.ROTOR_OK, rotor.ROTOR_EDOMAIN, rotor.ROTOR_EDOMAIN, rotor.ROTOR_OK]
    for c in (0, 3):
        C, D = orc.solve(p[c], M)
        gc, gd = chain_tables(cost, dec, c, L, M)
        assert np.array_equal(gc, C) and np.array_equal(gd, D), c


def limited(n, L, M, seed, share):
    """Chains whose sizes add up to M / share: a memory limit of that share."""
    p = chaingen.random_chains(n, L, seed=seed)
    scale = M / share / p[:, chaingen.WABAR].sum(axis=1)
    p[:, 2:] = np.ceil(p[:, 2:] * scale[:, None, None]).astype(np.int64)
    return p


def solve_ms(params, M, schedule="auto"):
    """Shortest of four timed solves."""
    import torch

    from paper_1911_13214_amd import rotor
    n, _, L = params.shape
    d_params = rotor.upload_params(params, M)
    cost, dec = rotor.alloc_tables(n, L, M)
    work = rotor.alloc_workspace(n, L, M)
    best = float("inf")
    for _ in range(5):
        start, stop = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        torch.cuda.synchronize()
        start.record()
        rotor.rotor_solve_schedule(d_params, n, L, M, cost, dec, work, schedule)
        stop.record()
        torch.cuda.synchronize()
        best = min(best, start.elapsed_time(stop))
    return best, cost, dec


# budgets far beyond the stages, sizes from half the memory of store-everything:
# the automatic order (2.4, 5.0 and 0.7 ms) stays within twice the edges by rounds, whose
# waves cover all budgets at once (tiles, window by window, took 16, 110 and 1.9)
@pytest.mark.parametrize("n,L,M", [(1, 100, 20000), (1, 16, 4000000), (8, 40, 5000)])
def test_many_budgets_are_not_filled_in_turn(n, L, M):
    import torch

    p = limited(n, L, M, 1300 + L, 0.5)
    print(f"many budgets L={L} M={M} n={n}", flush=True)
    ms, cost, dec = solve_ms(p, M)
    ms_rounds, cost_r, dec_r = solve_ms(p, M, "rounds")
    assert torch.equal(cost[..., :M + 1], cost_r[..., :M + 1]) and torch.equal(dec[..., :M + 1], dec_r[..., :M + 1])
    assert ms < 2 * ms_rounds, (ms, ms_rounds)


# the edges of a batch from 1024 budgets on: by rounds (29 or 30 launches per
# block-diagonal) where it holds few blocks, by tiles (at most 10) where many
@pytest.mark.parametrize("n,L,M,by_tiles", [(8, 200, 1500, False), (40, 120, 1100, True), (12, 200, 800, True)])
def test_edges_of_batches(n, L, M, by_tiles):
    from paper_1911_13214_amd import rotor

    print(f"edges of batches n={n} L={L} M={M}", flush=True)
    p = limited(n, L, M, 1350, 0.5)
    stats = rotor.rotor_solve_timed(rotor.upload_params(p, M), n, L, M, *rotor.alloc_tables(n, L, M),
                                    rotor.alloc_workspace(n, L, M))
    diagonals = (L + 15) // 16 - 1
    launches = stats["edge"]["launches"]
    assert 8 * diagonals <= launches <= 10 * diagonals if by_tiles else launches >= 29 * diagonals


# sizes past the windows' overlap cost a launch per window (0.25 and 0.48 ms against 0.21
# and 0.35), not the windows of every tile in turn (0.48 and 1.2)
@pytest.mark.parametrize("L,M", [(64, 1500), (100, 2400)])
def test_large_sizes_are_not_filled_in_turn(L, M):
    print(f"large sizes L={L} M={M}", flush=True)
    near = solve_ms(chaingen.random_chains(1, L, seed=1400 + L), M)[0]
    far = solve_ms(limited(1, L, M, 1400 + L, 0.1), M)[0]
    assert far < 1.8 * near, (far, near)


# streamed tiles of 8-byte values take twice the operands: the automatic order
# (9.8 ms) follows the blocked one in time (streamed 12.4)
def test_automatic_order_of_large_costs():
    L, M = 450, 1000
    p = chaingen.random_chains(1, L, seed=1600)
    p[:, :2] <<= 16
    print(f"automatic order of 8-byte values L={L} M={M}", flush=True)
    ms, ms_blocked = solve_ms(p, M)[0], solve_ms(p, M, "blocked")[0]
    assert ms < 1.15 * ms_blocked, (ms, ms_blocked)


# double keys change runs every 512 splits: chains past that, enough of them that
# no waves share a tile's splits; 4-byte values (too large for 32-bit keys) and
# 8-byte ones
@pytest.mark.parametrize("shift", [8, 14])
def test_runs_of_double_keys(shift):
    import torch

    from gpu_util import chain_tables, solve_on_gpu
    L, M, n = 610, 12, 256
    p = chaingen.random_chains(2, L, seed=1500, wa_hi=1)
    p[:, :2] <<= shift
    p[:, 2:] = np.minimum(p[:, 2:], 1)
    print(f"runs of double keys L={L} M={M} n={n} shift={shift}", flush=True)
    _, cost, dec = solve_on_gpu(np.tile(p, (n // 2, 1, 1)), M, schedule="diagonal")
    for c in range(2, n):
        assert torch.equal(cost[c, :, :M + 1], cost[c % 2, :, :M + 1]), c
        assert torch.equal(dec[c, :, :M + 1], dec[c % 2, :, :M + 1]), c
    for c in range(2):
        C, D = orc.solve(p[c], M)
        gc, gd = chain_tables(cost, dec, c, L, M)
        assert np.array_equal(gc, C) and np.array_equal(gd, D), c
        assert (D[orc.row(L, 1, L):orc.row(L, 1, L) + 1] > 530).any()  # splits of the second run


# many budgets against few stages: diagonals instead of tiles
@pytest.mark.parametrize("L,M", [(20, 480), (20, 481), (21, 512), (30, 800)])
def test_diagonals_of_short_chains(L, M):
    check(chaingen.random_chains(2, L, seed=400 + L), M)


def test_inner_runs():
    # 32-bit keys with 4 to 5 split bits: runs of 16 and 32 splits
    p = chaingen.random_chains(1, 150, seed=7)
    p[:, :2] *= 230
    check(p, 90)


# the blocked order's edges by tiles: one block-diagonal and more, chains that
# end inside a block and a tile, windows in turn and overlapping ones, the kinds
# of keys and of stored middle partials
@pytest.mark.parametrize("shift", [0, 14, 26])
@pytest.mark.parametrize("n,L,M", [(1, 17, 70), (1, 32, 130), (2, 37, 300), (1, 50, 321), (1, 53, 900), (9, 64, 400),
                                   (1, 70, 1600), (1, 35, 3300)])
def test_tile_block_edges(n, L, M, shift):
    p = chaingen.random_chains(n, L, seed=600 + L)
    p[:, :2] <<= shift
    for schedule in ("blocked", "serial"):
        check(p, M, schedule)


def test_tile_block_edges_past_the_overlap():
    p = chaingen.random_chains(1, 52, seed=700)
    p[:, 2:] *= 30
    check(p, 1300, "blocked")


def test_tile_block_edges_of_large_batches():
    # past 3e10 candidates short chains keep edges by tiles: the same tables as
    # by rows, which other tests hold against the oracle
    import torch

    from gpu_util import solve_on_gpu
    n, L, M = 256, 100, 760
    p = chaingen.random_chains(n, L, seed=900)
    print(f"tiles L={L} M={M} n={n}", flush=True)
    _, cost, dec = solve_on_gpu(p, M)
    _, cost_rows, dec_rows = solve_on_gpu(p, M, schedule="rows")
    assert torch.equal(cost[..., :M + 1], cost_rows[..., :M + 1])
    assert torch.equal(dec[..., :M + 1], dec_rows[..., :M + 1])
