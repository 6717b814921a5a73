"""The streamed order's 4 x 4 tiles at the sizes where they can go wrong,
against the oracle: chains that end inside a tile, the first chains with inner
splits, budgets around a wave and around a workgroup's window of 1024, shifts
beyond a window, and the three kinds of keys."""
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
# past it (the windows in turn) and past whole windows
@pytest.mark.parametrize("scale", [1, 4, 30])
@pytest.mark.parametrize("L,M", [(22, 319), (22, 320), (23, 448), (22, 511), (24, 575), (33, 703), (33, 704),
                                 (45, 1023), (45, 1024), (50, 1151), (90, 2000)])
def test_tile_windows(L, M, scale):
    p = chaingen.random_chains(1, L, seed=200 + L)
    p[:, 2:] *= scale
    check(p, M)


# batches whose tile-diagonals go from windows in turn to overlapping ones as
# they get fewer than 128 tiles
@pytest.mark.parametrize("n,L,M", [(9, 75, 330), (20, 50, 600), (40, 21, 900)])
def test_tile_windows_change(n, L, M):
    check(chaingen.random_chains(n, L, seed=300 + L), M)


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
