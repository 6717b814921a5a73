"""GPU parity: the HIP tables (through the C ABI) against the CPU oracle, bit
for bit.  Costs are int64 and decisions int16, so the bar is exact equality
of every cell.  Run on an MI355X with ``pytest -m gpu``."""
import os

import numpy as np
import pytest

import model
from gpu_util import canonical_hashes, chain_tables, gpu_rows_in_oracle_order, solve_on_gpu
from oracle import oracle as orc
from paper_1911_13214_amd import chaingen
from test_oracle_pins import TINY_M, tiny_chain, wide_chain

pytestmark = pytest.mark.gpu
GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden")


def say(msg):
    print(msg, flush=True)


# the blocked fill with its edges by tiles (at these sizes) and by anti-diagonal
# rounds (both with the inner middle products beside the previous edges, on the
# side stream), by rows, and by tiles on one stream; and the streamed tiles
SCHEDULES = ["blocked", "rounds", "rows", "serial", "diagonal"]
EDGE_ORDERS = ["blocked", "rounds", "rows", "serial"]
_oracle_cache = {}


def oracle_tables(params, M):
    """The oracle's tables of one chain, kept for the next schedule's run of
    the same case."""
    key = (params.tobytes(), params.shape, M)
    if key not in _oracle_cache:
        if len(_oracle_cache) > 8:
            _oracle_cache.clear()
        _oracle_cache[key] = orc.solve(params, M)
    return _oracle_cache[key]


def assert_same(params, M, cost, dec, c=0, order=None):
    L = params.shape[-1]
    C, D = oracle_tables(params[c:c + 1] if params.ndim == 3 else params, M)
    gc, gd = chain_tables(cost, dec, c, L, M, order)
    if not np.array_equal(gc, C):
        bad = np.argwhere(gc != C)[0]
        raise AssertionError(f"cost differs first at oracle row {bad[0]} m={bad[1]}: gpu {gc[tuple(bad)]} "
                             f"oracle {C[tuple(bad)]}")
    if not np.array_equal(gd, D):
        bad = np.argwhere(gd != D)[0]
        raise AssertionError(f"decision differs first at oracle row {bad[0]} m={bad[1]}: gpu {gd[tuple(bad)]} "
                             f"oracle {D[tuple(bad)]}")


@pytest.mark.parametrize("schedule", SCHEDULES)
@pytest.mark.parametrize("cfg", [1, 2, 3])
def test_parity_full_tables(cfg, schedule):
    params, L, M, _, name = chaingen.config(cfg)
    say(f"parity {name} {schedule}")
    _, cost, dec = solve_on_gpu(params, M, schedule=schedule)
    assert_same(params, M, cost, dec)


@pytest.mark.parametrize("schedule", SCHEDULES)
def test_parity_batch_256_chains(schedule):
    params, L, M, n, name = chaingen.config(4)
    say(f"parity {name} {schedule}")
    _, cost, dec = solve_on_gpu(params, M, schedule=schedule)
    order = gpu_rows_in_oracle_order(L)
    for c in list(range(0, n, 17)) + [n - 1]:
        assert_same(params, M, cost, dec, c, order)
    g = np.load(os.path.join(GOLDEN, "batch256_L64_M640.npz"))
    hc, hd = canonical_hashes(cost, dec, L, M)
    assert hc == str(g["hash_cost"]) and hd == str(g["hash_dec"])


def check_large_chain(params, M, cost, dec, g):
    """The stored records of a large chain: top row, seeded cells, three
    36-stage windows solved by the oracle now (C(s,t,.) depends on stages
    s..t only), and the hashes of both whole tables."""
    L = params.shape[2]
    order = gpu_rows_in_oracle_order(L)
    top = order[orc.row(L, 1, L)]
    np.testing.assert_array_equal(cost[0, top, :M + 1].cpu().numpy(), g["top_cost"])
    np.testing.assert_array_equal(dec[0, top, :M + 1].cpu().numpy(), g["top_dec"])
    cells = g["cells"]
    rows = order[[orc.row(L, int(s), int(t)) for s, t, _ in cells]]
    gc = cost[0].cpu().numpy()
    gd = dec[0].cpu().numpy()
    np.testing.assert_array_equal(gc[rows, cells[:, 2]], g["cell_cost"])
    np.testing.assert_array_equal(gd[rows, cells[:, 2]], g["cell_dec"])
    for a, b in [(1, 36), (233, 268), (L - 35, L)]:
        sub = np.ascontiguousarray(params[:, :, a - 1:b])
        C, D = orc.solve(sub, M)
        Ls = b - a + 1
        for s in range(1, Ls + 1):
            for t in range(s, Ls + 1):
                r = order[orc.row(L, s + a - 1, t + a - 1)]
                np.testing.assert_array_equal(gc[r, :M + 1], C[orc.row(Ls, s, t)])
                ds = D[orc.row(Ls, s, t)].astype(np.int64)
                np.testing.assert_array_equal(gd[r, :M + 1], np.where(ds > 0, ds + a - 1, ds))
    del gc, gd
    hc, hd = canonical_hashes(cost, dec, L, M)
    assert hc == str(g["hash_cost"]), "whole cost table hash"
    assert hd == str(g["hash_dec"]), "whole decision table hash"


@pytest.mark.parametrize("schedule", SCHEDULES)
def test_parity_large_chain(schedule):
    params, L, M, _, name = chaingen.config(5)
    say(f"parity {name} {schedule}")
    g = np.load(os.path.join(GOLDEN, "random_L500_M5000.npz"))
    _, cost, dec = solve_on_gpu(params, M, schedule=schedule)
    check_large_chain(params, M, cost, dec, g)


@pytest.mark.parametrize("schedule", SCHEDULES)
def test_parity_large_chain_costs_x8(schedule):
    # The large chain with u_f and u_b times 8: its block-diagonals take
    # whole packed keys, runs of 128 splits (several per range, one
    # workgroup holding the whole range and finishing the corner cell) and
    # (value, split) pairs.
    params, L, M, _, name = chaingen.config(5)
    g = np.load(os.path.join(GOLDEN, "random_L500_M5000_x8.npz"))
    params[:, :2] <<= int(g["cost_shift"])
    modes = middle_modes(params[0], L, M, 1)
    kinds = {m if isinstance(m, str) else m[0] for m in modes.values()}
    assert kinds == {"packed", "runs", "pairs"}
    assert any(m[0] == "runs" and m[2] == 1 and m[3] > 2 << m[1] for m in modes.values() if m != "pairs")
    say(f"parity {name} costs x 8 {schedule}")
    _, cost, dec = solve_on_gpu(params, M, schedule=schedule)
    check_large_chain(params, M, cost, dec, g)


@pytest.mark.parametrize("M", [62, 63, 64, 126, 127, 128, 191])
@pytest.mark.parametrize("schedule", SCHEDULES)
def test_budget_counts_around_the_lane_layout(M, schedule):
    # The edge and diagonal kernels give each lane two budgets 64 apart in
    # workgroups of 128 budgets: budget counts M + 1 just below, at and above
    # 64 and 128 leave the second budget of some lanes, or a whole second
    # workgroup, with nothing or part to do.
    L = 48
    params = chaingen.random_chains(1, L, seed=100 + M)
    say(f"lane layout L={L} M={M} {schedule}")
    _, cost, dec = solve_on_gpu(params, M, schedule=schedule)
    assert_same(params, M, cost, dec)


@pytest.mark.parametrize("L,M,seed", [(1, 0, 1), (1, 37, 2), (2, 15, 3), (3, 16, 4), (5, 1, 9), (17, 255, 5),
                                      (33, 257, 6), (40, 1023, 7), (64, 300, 8)])
@pytest.mark.parametrize("schedule", SCHEDULES)
def test_edge_shapes(L, M, seed, schedule):
    say(f"edge L={L} M={M} {schedule}")
    params = chaingen.random_chains(1, L, seed=seed)
    _, cost, dec = solve_on_gpu(params, M, schedule=schedule)
    assert_same(params, M, cost, dec)


@pytest.mark.parametrize("schedule", SCHEDULES)
def test_tiny_and_wide_chains(schedule):
    for seed in range(40):
        p = tiny_chain(seed)
        _, cost, dec = solve_on_gpu(p, TINY_M, schedule=schedule)
        assert_same(p, TINY_M, cost, dec)
    for seed in range(6):
        p = wide_chain(seed, L=12, size_hi=40, over_hi=30)
        _, cost, dec = solve_on_gpu(p, 400, schedule=schedule)
        assert_same(p, 400, cost, dec)


@pytest.mark.parametrize("schedule", SCHEDULES)
def test_shifts_beyond_the_budget(schedule):
    # sizes larger than M: every shifted read falls below budget 0
    p = chaingen.random_chains(1, 9, seed=12)
    p[0, 2, ::2] += 300
    p[0, 3, ::3] += 500
    _, cost, dec = solve_on_gpu(p, 200, schedule=schedule)
    assert_same(p, 200, cost, dec)


@pytest.mark.parametrize("schedule", SCHEDULES)
def test_zero_sizes_any_length(schedule):
    # no memory needed anywhere: with u_f >= 1 the no-recomputation schedule
    # is optimal for every budget, F_all first everywhere
    L, M = 700, 3
    p = chaingen.random_chains(1, L, seed=13)
    p[0, 2:] = 0
    d_params, cost, dec = solve_on_gpu(p, M, schedule=schedule)
    pre = np.concatenate([[0], np.cumsum(p[0, 0] + p[0, 1])])
    gc = cost[0].cpu().numpy()
    gd = dec[0].cpu().numpy()
    for d in (0, 1, 2, 350, L - 1):
        for s in sorted({1, min(2, L - d), L - d}):
            t = s + d
            from paper_1911_13214_amd import rotor
            r = rotor.rotor_row_index(L, s, t)
            assert (gc[r, :M + 1] == pre[t] - pre[s - 1]).all()
            assert (gd[r, :M + 1] == 0).all()
    from paper_1911_13214_amd import rotor
    seq = rotor.reconstruct(d_params, 1, L, M, dec, 0, [0])[0]
    assert seq == [(orc.F_ALL, l) for l in range(1, L + 1)] + [(orc.B, l) for l in range(L, 0, -1)]


def test_large_budget_range():
    p = chaingen.random_chains(1, 4, seed=14)
    M = (1 << 18) + 5
    _, cost, dec = solve_on_gpu(p, M)
    assert_same(p, M, cost, dec)


def test_batch_equals_single_solves():
    params = chaingen.random_chains(9, 23, seed=15)
    M = 230
    _, cost, dec = solve_on_gpu(params, M)
    for c in range(9):
        _, c1, d1 = solve_on_gpu(params[c:c + 1], M)
        assert np.array_equal(cost[c].cpu().numpy()[:, :M + 1], c1[0].cpu().numpy()[:, :M + 1])
        assert np.array_equal(dec[c].cpu().numpy()[:, :M + 1], d1[0].cpu().numpy()[:, :M + 1])
        assert_same(params, M, cost, dec, c)


def test_deterministic():
    params, L, M, _, _ = chaingen.config(3)
    _, c1, d1 = solve_on_gpu(params, M)
    _, c2, d2 = solve_on_gpu(params, M)
    assert np.array_equal(c1[..., :M + 1].cpu().numpy(), c2[..., :M + 1].cpu().numpy())
    assert np.array_equal(d1[..., :M + 1].cpu().numpy(), d2[..., :M + 1].cpu().numpy())


def test_non_default_stream():
    import torch
    params, L, M, _, _ = chaingen.config(2)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        _, cost, dec = solve_on_gpu(params, M, stream=st)
    assert_same(params, M, cost, dec)


@pytest.mark.parametrize("cfg", [1, 2, 3])
def test_reconstruct_matches_oracle(cfg):
    from paper_1911_13214_amd import rotor
    params, L, M, _, name = chaingen.config(cfg)
    say(f"reconstruct {name}")
    d_params, cost, dec = solve_on_gpu(params, M)
    C, _ = orc.solve(params, M)
    budgets = list(range(0, M + 1, max(1, (M + 1) // 97))) + [M]
    seqs = rotor.reconstruct(d_params, 1, L, M, dec, 0, budgets)
    for m, seq in zip(budgets, seqs):
        assert seq == orc.reconstruct(params, M, C, m), m


def test_reconstruct_batch_chain_and_replay():
    from paper_1911_13214_amd import rotor
    params, L, M, n, _ = chaingen.config(4)
    d_params, cost, dec = solve_on_gpu(params, M)
    for c in (0, 77, 255):
        C, _ = orc.solve(params[c:c + 1], M)
        budgets = [100, 200, 400, M]
        for m, seq in zip(budgets, rotor.reconstruct(d_params, n, L, M, dec, c, budgets)):
            assert seq == orc.reconstruct(params[c:c + 1], M, C, m)


def test_reconstruct_large_chain_replays():
    from paper_1911_13214_amd import rotor
    params, L, M, _, _ = chaingen.config(5)
    g = np.load(os.path.join(GOLDEN, "random_L500_M5000.npz"))
    d_params, cost, dec = solve_on_gpu(params, M)
    ch = model.Chain(params)
    budgets = [m for m in range(0, M + 1, 250) if g["top_cost"][m] != orc.INF] + [M]
    for m, seq in zip(budgets, rotor.reconstruct(d_params, 1, L, M, dec, 0, budgets)):
        time, peak = model.simulate(ch, 1, L, seq)
        assert time == g["top_cost"][m] and peak <= m


@pytest.mark.parametrize("L,seed", [(40, 1), (77, 2)])
def test_plan_discretise_solve_and_walk_ten_budgets(L, seed):
    # Sections 5.2 and 5.3: sizes in bytes -> 500 slots of the store-everything
    # memory, one table, ten equally spaced budgets walked in one call
    from paper_1911_13214_amd import rotor
    p = chaingen.byte_sized_chain(L, seed=seed)
    say(f"plan bytes L={L}")
    S = 500
    res = rotor.plan(p, slots=S, n_budgets=10)
    ps = res["params_slots"]
    assert res["top_bytes"] == orc.store_all_peak(p)
    assert np.array_equal(ps, orc.discretize(p, orc.store_all_peak(p), S))
    assert res["budgets"] == [S * i // 10 for i in range(1, 11)]
    C, _ = orc.solve(ps, S)
    top = orc.table_view(C, L)(1, L)
    ch = model.Chain(ps)
    feasible = 0
    for b, t, seq in zip(res["budgets"], res["times"], res["sequences"]):
        if top[b] == orc.INF:
            assert t is None and seq is None
            continue
        feasible += 1
        assert t == top[b] and seq == orc.reconstruct(ps, S, C, b)
        time, peak = model.simulate(ch, 1, L, seq)
        assert time == t and peak <= b
    assert feasible >= 3


def test_discretise_one_limit_per_chain_of_a_batch():
    # the paper's reading: every memory limit gets its own slot size; a batch
    # of ten copies of a chain with ten limits is filled in one call
    from paper_1911_13214_amd import rotor
    p = chaingen.byte_sized_chain(30, seed=9)
    top = orc.store_all_peak(p)
    limits = np.array([top * i // 10 for i in range(1, 11)], dtype=np.int64)
    S = 200
    ps = rotor.rotor_discretize(np.repeat(p[None], 10, axis=0), limits, S)
    for c in range(10):
        assert np.array_equal(ps[c], orc.discretize(p, int(limits[c]), S))
    _, cost, dec = solve_on_gpu(ps, S)
    for c in range(10):
        assert_same(ps, S, cost, dec, c)


def test_reconstruct_status_codes():
    import torch

    from paper_1911_13214_amd import rotor
    params, L, M, _, _ = chaingen.config(1)
    d_params, cost, dec = solve_on_gpu(params, M)
    assert rotor.reconstruct(d_params, 1, L, M, dec, 0, [0, 24]) == [None, None]
    budgets = torch.tensor([50, M + 1, -1, 100], dtype=torch.int64, device="cuda")
    cap = 5
    ops = torch.zeros((4, cap, 2), dtype=torch.int32, device="cuda")
    count = torch.zeros(4, dtype=torch.int64, device="cuda")
    status = torch.zeros(4, dtype=torch.int32, device="cuda")
    rotor.rotor_reconstruct(d_params, 1, L, M, dec, 0, budgets, cap, ops, count, status)
    torch.cuda.synchronize()
    C, _ = orc.solve(params, M)
    full50 = orc.reconstruct(params, M, C, 50)
    st, cnt = status.cpu().tolist(), count.cpu().tolist()
    assert st == [rotor.ROTOR_ECAPACITY, rotor.ROTOR_EINVAL, rotor.ROTOR_EINVAL, rotor.ROTOR_ECAPACITY]
    assert cnt[0] == len(full50)
    assert [tuple(x) for x in ops[0].cpu().tolist()] == full50[:cap]
    # a table the library did not write is reported, not walked out of bounds
    bad = dec.clone()
    top = rotor.rotor_row_index(L, 1, L)
    bad[0, top, 60] = L + 5
    rotor.rotor_reconstruct(d_params, 1, L, M, bad, 0, torch.tensor([60], device="cuda"), 200, ops.new_zeros(1, 200, 2),
                            count[:1], status[:1])
    torch.cuda.synchronize()
    assert status[0].item() == rotor.ROTOR_ECORRUPT


@pytest.mark.parametrize("cfg,n", [(2, 1), (3, 1), (4, 256), (4, 320)])
def test_timed_solve_matches_and_counts_the_work(cfg, n):
    # random L=50, ResNet-like L=100 and the batch workload take the streamed
    # order, a larger batch the blocked one (middle and edge classes)
    import torch

    from paper_1911_13214_amd import rotor
    params, L, M, n_cfg, _ = chaingen.config(cfg)
    if n > n_cfg:
        params = np.concatenate([params, params[:n - n_cfg]])
    say(f"timed cfg {cfg} n={n}")
    d_params, cost, dec = solve_on_gpu(params, M)
    c2, d2 = rotor.alloc_tables(n, L, M)
    stats = rotor.rotor_solve_timed(d_params, n, L, M, c2, d2, rotor.alloc_workspace(n, L, M))
    torch.cuda.synchronize()
    assert torch.equal(cost[..., :M + 1], c2[..., :M + 1]) and torch.equal(dec[..., :M + 1], d2[..., :M + 1])
    blocked = n == 320
    assert (stats["middle"]["launches"] > 0) == blocked and (stats["edge"]["launches"] > 0) == blocked
    W = M + 1
    assert sum(s["split_candidates"] for s in stats.values()) == (L ** 3 - L) // 6 * W * n
    assert sum(s["all_candidates"] for s in stats.values()) == L * (L - 1) // 2 * W * n
    assert sum(s["cells"] for s in stats.values()) == L * (L + 1) // 2 * W * n
    assert all(s["ms"] >= 0 for s in stats.values()) and stats["leaf"]["launches"] == 1
    assert stats["prep"]["launches"] == 1


# the narrow (4-byte) value path takes block-diagonals whose cost bound is
# below NARROW_BOUND; the 64-bit path's middle keys are doubles below F64_BOUND
NARROW_BOUND = (1 << 32) - 1
F64_BOUND = 1 << 38


def cost_bound(p):
    """sum_l P[l] + sum u_b = sum_j (L - j + 1) u_f^j + sum u_b: no stage runs
    forward more often than the stages after it plus one, so every finite cost
    is at most this; the library picks its value path from it."""
    return int(np.cumsum(p[0].astype(object)).sum() + p[1].astype(object).sum())


def scaled_chain(seed, L, shift):
    p = chaingen.random_chains(1, L, seed=seed)
    p[0, 0] *= 1 << shift
    p[0, 1] *= 1 << shift
    return p


def wide_costs_chain(seed, L):
    """A chain whose cost bound exceeds 2^32 - 2, so the solver takes its
    64-bit value path."""
    p = scaled_chain(seed, L, 22)
    assert cost_bound(p[0]) >= NARROW_BOUND
    return p


@pytest.mark.parametrize("schedule", SCHEDULES)
@pytest.mark.parametrize("L,M,seed", [(5, 60, 1), (23, 230, 2), (40, 400, 3), (70, 300, 4)])
def test_wide_value_path(L, M, seed, schedule):
    p = wide_costs_chain(seed, L)
    say(f"wide L={L} M={M} {schedule}")
    _, cost, dec = solve_on_gpu(p, M, schedule=schedule)
    assert_same(p, M, cost, dec)


@pytest.mark.parametrize("L,M,seed", [(70, 300, 5), (90, 200, 6)])
@pytest.mark.parametrize("edges", EDGE_ORDERS)
def test_narrow_chain_beyond_packed_keys(L, M, seed, edges):
    # costs below 2^30 (compact copy, 4-byte values) but too large to leave
    # the split field room once the middle range has 16 splits or more: the first
    # block-diagonal takes packed keys, the later ones the (value, split) pairs
    # (their own bounds too leave too few bits)
    p = scaled_chain(seed, L, 12)
    v = cost_bound(p[0])
    assert (1 << 26) < v < (1 << 30)
    say(f"narrow beyond packed L={L} M={M} bound={v}")
    _, cost, dec = solve_on_gpu(p, M, schedule=edges)
    assert_same(p, M, cost, dec)


def key_bits(v):
    """Largest S with (v + 1) << S <= 2^32 - 1: the split bits a packed key
    has left beside a value of at most v."""
    return (((1 << 32) - 1) // (v + 1)).bit_length() - 1


def block_diagonal_bounds(p, L):
    """cost_bound of the longest pairs of each block-diagonal D of 16-stage
    blocks: the pairs of the blocks (I, I + D) lie within the stages
    [16I + 1, min(16(I + D + 1), L)]."""
    nb = (L + 15) // 16
    return {D: max(cost_bound(p[:, 16 * I:min(16 * (I + D + 1), L)]) for I in range(nb - D)) for D in range(1, nb)}


@pytest.mark.parametrize("seed,shift", [(8, 7), (8, 8), (8, 9), (7, 6)])
@pytest.mark.parametrize("edges", EDGE_ORDERS)
def test_packed_keys_per_block_diagonal(seed, shift, edges):
    # The packed middle keys of block-diagonal D need (V_D + 1) << S to fit
    # in 32 bits, with S the bits of its split range and V_D the bound of its
    # longest pairs.  At these cost scales some block-diagonals fit with no
    # bit to spare, others miss by one, and the whole chain's bound would
    # have packed fewer of them.
    L, M = 160, 240
    p = scaled_chain(seed, L, shift)
    v = cost_bound(p[0])
    assert v < 1 << 30
    vd = block_diagonal_bounds(p[0], L)
    span_bits = {D: (16 * (D - 1)).bit_length() for D in vd}
    packed = {D for D in vd if span_bits[D] <= key_bits(vd[D])}
    assert {D for D in vd if span_bits[D] <= key_bits(v)} < packed
    assert any(span_bits[D] == key_bits(vd[D]) for D in packed)
    assert any(span_bits[D] == key_bits(vd[D]) + 1 for D in vd)
    say(f"packed per block-diagonal seed={seed} shift={shift} bound={v} packed={sorted(packed)}")
    _, cost, dec = solve_on_gpu(p, M, schedule=edges)
    assert_same(p, M, cost, dec)


def middle_modes(p, L, M, n_chains):
    """How the blocked fill relaxes the middle splits of each block-diagonal
    D >= 1 of one chain: ("packed", parts) when its whole range fits a packed
    key, ("runs", S, parts, splits per part) when runs of 2^S splits do (S >=
    7), "pairs" or "wide" otherwise.  A range is cut into parts when its
    launch has fewer than 256 workgroups of 64 budgets."""
    nb = (L + 15) // 16
    vd = block_diagonal_bounds(p, L)
    out = {}
    for D in range(1, nb):
        n = 16 * (D - 1)  # last split minus first
        if vd[D] >= NARROW_BOUND:
            out[D] = "wide"
            continue
        wgs = (M + 64) // 64 * (nb - D) * n_chains
        parts = max(1, min(-(-512 // wgs), (n + 1) // 32)) if wgs < 256 else 1
        S = key_bits(vd[D])
        if n.bit_length() <= S:
            out[D] = ("packed", parts)
        elif S >= 7:
            out[D] = ("runs", S, parts, (n + parts) // parts)
        else:
            out[D] = "pairs"
    return out


@pytest.mark.parametrize("L,M,seed,shift", [(200, 240, 8, 5), (240, 200, 7, 4), (256, 300, 9, 4)])
@pytest.mark.parametrize("edges", EDGE_ORDERS)
def test_packed_runs_per_block_diagonal(L, M, seed, shift, edges):
    # Block-diagonals whose bound leaves a packed key 7 bits or more, but
    # fewer than their split range needs, relax the range in runs of 2^S
    # splits and merge the runs' (value, split) results in the cost table by
    # atomic minima.  At these sizes their ranges are cut into parts of one
    # run each; the large chain with costs x 8 (stored hashes) has whole
    # ranges of several runs.
    p = scaled_chain(seed, L, shift)
    modes = middle_modes(p[0], L, M, 1)
    runs = {D: m for D, m in modes.items() if m[0] == "runs"}
    assert runs and all(m[2] > 1 for m in runs.values())
    say(f"packed runs L={L} M={M} seed={seed} shift={shift} {sorted(runs.items())}")
    _, cost, dec = solve_on_gpu(p, M, schedule=edges)
    assert_same(p, M, cost, dec)


@pytest.mark.parametrize("schedule", SCHEDULES)
@pytest.mark.parametrize("shift", [13, 14, 16, 18])
def test_value_path_per_block_diagonal(shift, schedule):
    # A chain whose cost bound is past 2^32 - 2 while the bounds of its shorter
    # sub-chains are not: the pairs of the first block-diagonals take the
    # 4-byte path (compact copy, saturating adds), the later ones the 64-bit
    # keys, in the three orders.
    L, M = 160, 240
    p = scaled_chain(8, L, shift)
    nb = (L + 15) // 16
    vd = {0: max(cost_bound(p[0][:, 16 * I:min(16 * (I + 1), L)]) for I in range(nb))}
    vd.update(block_diagonal_bounds(p[0], L))
    narrow = [D for D in range(nb) if vd[D] < NARROW_BOUND]
    assert cost_bound(p[0]) >= NARROW_BOUND and narrow == list(range(len(narrow))) and 0 < len(narrow) < nb
    say(f"value path per block-diagonal shift={shift} narrow={narrow} {schedule}")
    _, cost, dec = solve_on_gpu(p, M, schedule=schedule)
    assert_same(p, M, cost, dec)


@pytest.mark.parametrize("schedule", SCHEDULES)
def test_double_keys_per_block_diagonal(schedule):
    # Costs x 2^20: every block-diagonal on the 64-bit path, the first ones
    # with bounds below 2^38, whose middle keys value * 2^15 + split offset
    # are exact as doubles, the later ones with 64-bit integer keys.
    L, M = 160, 240
    p = scaled_chain(8, L, 20)
    vd = block_diagonal_bounds(p[0], L)
    f64 = [D for D in sorted(vd) if vd[D] < F64_BOUND]
    assert min(vd.values()) >= NARROW_BOUND and f64 == list(range(1, len(f64) + 1)) and 0 < len(f64) < len(vd)
    say(f"double keys per block-diagonal f64={f64} {schedule}")
    _, cost, dec = solve_on_gpu(p, M, schedule=schedule)
    assert_same(p, M, cost, dec)


@pytest.mark.parametrize("bound", [NARROW_BOUND - 1, NARROW_BOUND, F64_BOUND - 1, F64_BOUND])
@pytest.mark.parametrize("edges", EDGE_ORDERS)
def test_value_paths_at_their_limits(bound, edges):
    # Block-diagonal D takes the 4-byte values when its bound V_D is below
    # 2^32 - 1, double keys when it is below 2^38, else 64-bit keys.  Three
    # blocks of 16 stages with u_f = c, u_b = 2c, w_a = 1, w_abar = 2: D = 2
    # is the whole chain, its bound put on each side of both limits through
    # u_b of stage 1, and the oracle shows the top cell reaching it (the
    # schedule that recomputes every forward step, at the smallest budgets).
    L, M = 48, 120
    c = bound // 1272 - 1  # the whole chain's bound is 1176 c + 48 u_b
    p = np.zeros((1, 6, L), dtype=np.int64)
    p[0, chaingen.UF], p[0, chaingen.UB] = c, 2 * c
    p[0, chaingen.WA], p[0, chaingen.WABAR] = 1, 2
    p[0, chaingen.UB, 0] = 2 * c + bound - 1272 * c
    vd = block_diagonal_bounds(p[0], L)
    assert vd[2] == bound and vd[1] < bound // 2
    C, _ = oracle_tables(p, M)
    top = C[orc.row(L, 1, L)]
    assert top[top != orc.INF].max() == bound
    say(f"value paths at their limits V_2={bound} {edges}")
    _, cost, dec = solve_on_gpu(p, M, schedule=edges)
    assert_same(p, M, cost, dec)


@pytest.mark.parametrize("schedule", SCHEDULES)
def test_saturated_budgets(schedule):
    # From G(s, t) on (the peak of storing every activation) a cell holds the
    # least time sum(u_f + u_b), and C_2 when u_f^s > 0: the kernels store
    # that without loading operands, by edge workgroup of 128 budgets, by row
    # of 64 and by middle block.  Here G spreads over the whole budget range
    # (pairs of 2 to 100 stages, M = 999), crossing the workgroups' bounds;
    # the second chain has u_f = 0 on about one stage in five, where C_1 can
    # tie C_2 and no shortcut applies; the third has every size 0 but one.
    L, M = 100, 999
    p = chaingen.random_chains(3, L, seed=77)
    rng = np.random.default_rng(77)
    p[1, chaingen.UF, rng.random(L) < 0.2] = 0
    p[2, chaingen.WA:] = 0
    p[2, chaingen.WABAR, 50] = 7
    say(f"saturated budgets L={L} M={M} {schedule}")
    _, cost, dec = solve_on_gpu(p, M, schedule=schedule)
    for c in range(3):
        assert_same(p, M, cost, dec, c)


@pytest.mark.parametrize("v0", [32752, 32766, 32767, 32768, 33600])
@pytest.mark.parametrize("edges", EDGE_ORDERS)
def test_two_byte_copy_of_the_diagonal_blocks_at_its_limit(v0, edges):
    # The edges read the diagonal blocks' cells from a 2-byte copy when their
    # bound V_0 (largest over the 16-stage blocks) is at most 2^15 - 2, else
    # from the 4-byte copy.  Here u_f = 200, w_a = 1, w_abar = 2 on every
    # stage and u_b = 347 but on stage 1, so V_0 is the first block's bound,
    # and the oracle shows block cells reaching it: a value of 2^15 or more
    # in the 2-byte copy would come back negative.
    L, M = 40, 120
    p = np.zeros((1, 6, L), dtype=np.int64)
    p[0, chaingen.UF], p[0, chaingen.UB] = 200, 347
    p[0, chaingen.WA], p[0, chaingen.WABAR] = 1, 2
    p[0, chaingen.UB, 0] = 347 + v0 - (200 * 136 + 16 * 347)
    assert max(cost_bound(p[0][:, b:b + 16]) for b in range(0, L, 16)) == v0
    C, _ = oracle_tables(p, M)
    block_cells = [orc.row(L, s, t) for s in range(1, L + 1) for t in range(s, min(L, (s - 1) // 16 * 16 + 16) + 1)]
    finite = C[block_cells][C[block_cells] != np.iinfo(np.int64).max]
    assert finite.max() == v0
    say(f"two-byte diagonal blocks V_0={v0}")
    _, cost, dec = solve_on_gpu(p, M, schedule=edges)
    assert_same(p, M, cost, dec)


@pytest.mark.parametrize("schedule", SCHEDULES)
def test_batch_mixing_value_paths(schedule):
    # chains of one call may take different value paths
    params = chaingen.random_chains(6, 37, seed=21)
    for c in (1, 4):
        params[c, 0] *= 1 << 22
        params[c, 1] *= 1 << 22
    params[2, 0] *= 1 << 13
    params[2, 1] *= 1 << 13
    assert cost_bound(params[1]) >= NARROW_BOUND and (1 << 27) < cost_bound(params[2]) < NARROW_BOUND
    M = 200
    _, cost, dec = solve_on_gpu(params, M, schedule=schedule)
    for c in range(6):
        assert_same(params, M, cost, dec, c)


@pytest.mark.parametrize("edges", EDGE_ORDERS)
def test_batch_mixing_middle_paths(edges):
    # One blocked fill whose chains take different middle paths in the same
    # launches: packed keys and packed runs, packed keys only, packed keys
    # with (value, split) pairs and 64-bit keys, 64-bit keys only.
    L, M = 200, 240
    shifts = (5, 0, 14, 22)
    p = np.concatenate([scaled_chain(30 + i, L, sh) for i, sh in enumerate(shifts)])
    kinds = [{m if isinstance(m, str) else m[0] for m in middle_modes(p[c], L, M, len(shifts)).values()}
             for c in range(len(shifts))]
    assert kinds == [{"packed", "runs"}, {"packed"}, {"packed", "pairs", "wide"}, {"wide"}]
    say(f"batch mixing middle paths L={L} M={M} {kinds}")
    _, cost, dec = solve_on_gpu(p, M, schedule=edges)
    for c in range(len(shifts)):
        assert_same(p, M, cost, dec, c)


@pytest.mark.parametrize("L,M", [(5, (1 << 28) - 1), (20, (1 << 24) + 3)])
def test_largest_budgets(L, M):
    # M at the domain's limit: C(s, t, m) depends only on budgets up to m, and
    # from the store-everything peak on it no longer changes, so the oracle
    # at a small budget range gives every column exactly
    import torch
    from paper_1911_13214_amd import rotor
    p = chaingen.random_chains(1, L, seed=L)
    small = 2000
    assert orc.store_all_peak(p[0]) < small
    say(f"largest budgets L={L} M={M}")
    d_params = rotor.upload_params(p, M)
    cost, dec = rotor.alloc_tables(1, L, M)
    work = rotor.alloc_workspace(1, L, M)
    rotor.rotor_solve(d_params, 1, L, M, cost, dec, work)
    torch.cuda.synchronize()
    del work
    C, D = orc.solve(p, small)
    order = torch.as_tensor(gpu_rows_in_oracle_order(L), device="cuda")
    g = torch.Generator().manual_seed(L)
    cols = torch.cat([torch.arange(small + 1), torch.randint(small + 1, M + 1, (4000,), generator=g),
                      torch.tensor([M - 1, M])]).cuda()
    gc = cost[0][:, cols][order].cpu().numpy()
    gd = dec[0][:, cols][order].cpu().numpy()
    want = np.minimum(cols.cpu().numpy(), small)
    assert np.array_equal(gc, C[:, want]) and np.array_equal(gd, D[:, want])
    del cost, dec
    torch.cuda.empty_cache()


def test_long_chain_windows():
    # L = 4000: 8 million pairs, 250 blocks a side.  Small sizes keep the
    # costs near 4e8, too large for packed keys once the middle range passes
    # 8 splits, so the (value, split) middle path runs at scale.  Windows of
    # 36 stages are solved by the oracle: C(s, t, .) depends on s..t only.
    import torch
    from paper_1911_13214_amd import rotor
    L, M = 4000, 63
    p = chaingen.random_chains(1, L, seed=11, wa_hi=1)
    assert (1 << 26) < cost_bound(p[0]) < (1 << 30)
    say(f"long chain L={L} M={M}")
    _, cost, dec = solve_on_gpu(p, M)
    for a in (1, 1983, 3965):
        b = a + 35
        C, D = orc.solve(np.ascontiguousarray(p[:, :, a - 1:b]), M)
        pairs = [(s, t) for s in range(1, 37) for t in range(s, 37)]
        rows = torch.tensor([rotor.rotor_row_index(L, s + a - 1, t + a - 1) for s, t in pairs], device="cuda")
        gc = cost[0][rows][:, :M + 1].cpu().numpy()
        gd = dec[0][rows][:, :M + 1].cpu().numpy().astype(np.int64)
        want_c = np.stack([C[orc.row(36, s, t)] for s, t in pairs])
        want_d = np.stack([D[orc.row(36, s, t)] for s, t in pairs]).astype(np.int64)
        np.testing.assert_array_equal(gc, want_c)
        np.testing.assert_array_equal(gd, np.where(want_d > 0, want_d + a - 1, want_d))
    top = cost[0, rotor.rotor_row_index(L, 1, L), :M + 1].cpu().numpy()
    assert np.all(top[1:] <= top[:-1]) and top[M] != orc.INF


def test_orders_agree_on_a_table_beyond_4_gb():
    # L = 1000, M = 4000: 500,500 pairs, a 16 GB cost table and an 8 GB
    # compact copy, so row offsets pass 32 bits; the cost bound (~2.5e7)
    # leaves 7 bits of split field, so block-diagonals up to 8 take packed
    # middle keys and the later ones the (value, split) middle kernel.  The
    # blocked order with edges by rounds and the streamed one (by tiles) share
    # no kernel, and the blocked order's own choice takes tiles for the last
    # block-diagonals; every cell must agree, and 36-stage windows must equal
    # the oracle's tables.
    import torch
    from paper_1911_13214_amd import rotor
    L, M = 1000, 4000
    p = chaingen.random_chains(1, L, seed=1000)
    assert (1 << 24) < cost_bound(p[0]) < (1 << 25)
    say(f"orders at scale L={L} M={M}")
    _, c1, d1 = solve_on_gpu(p, M, schedule="rounds")
    for other in ("diagonal", "blocked"):
        _, c2, d2 = solve_on_gpu(p, M, schedule=other)
        assert torch.equal(c1[..., :M + 1], c2[..., :M + 1]) and torch.equal(d1[..., :M + 1], d2[..., :M + 1]), other
        del c2, d2
        torch.cuda.empty_cache()
    for a in (1, 483, 965):
        b = a + 35
        C, D = oracle_tables(np.ascontiguousarray(p[:, :, a - 1:b]), M)
        pairs = [(s, t) for s in range(1, 37) for t in range(s, 37)]
        rows = torch.tensor([rotor.rotor_row_index(L, s + a - 1, t + a - 1) for s, t in pairs], device="cuda")
        gc = c1[0][rows][:, :M + 1].cpu().numpy()
        gd = d1[0][rows][:, :M + 1].cpu().numpy().astype(np.int64)
        np.testing.assert_array_equal(gc, np.stack([C[orc.row(36, s, t)] for s, t in pairs]))
        want_d = np.stack([D[orc.row(36, s, t)] for s, t in pairs]).astype(np.int64)
        np.testing.assert_array_equal(gd, np.where(want_d > 0, want_d + a - 1, want_d))
    top = c1[0, rotor.rotor_row_index(L, 1, L), :M + 1].cpu().numpy()
    assert np.all(top[1:] <= top[:-1]) and top[M] != orc.INF


@pytest.mark.parametrize("n,L,M", [(65535, 3, 4), (8192, 40, 20)])
def test_largest_batches(n, L, M):
    # the chain index rides on the grid's z dimension (65535 at most): the two
    # fill orders agree on every chain, and sampled chains equal the oracle
    import torch
    params = chaingen.random_chains(n, L, seed=n + L)
    say(f"batch n={n} L={L} M={M}")
    _, c1, d1 = solve_on_gpu(params, M, schedule="blocked")
    _, c2, d2 = solve_on_gpu(params, M, schedule="diagonal")
    assert torch.equal(c1[..., :M + 1], c2[..., :M + 1]) and torch.equal(d1[..., :M + 1], d2[..., :M + 1])
    del c2, d2
    order = gpu_rows_in_oracle_order(L)
    rng = np.random.default_rng(n)
    for c in sorted({0, 1, n // 2, n - 1, *rng.integers(0, n, 24).tolist()}):
        assert_same(params, M, c1, d1, c, order)


def test_fill_replays_from_a_captured_graph():
    # the fill only enqueues kernels (no allocation, no memset, no host wait),
    # so a caller may capture it; every replay, with eager work in between,
    # must rebuild the same tables
    import torch
    from paper_1911_13214_amd import rotor
    params, L, M, n, _ = chaingen.config(3)
    say("graph replay resnet-like L=100 M=1000")
    d_params = rotor.upload_params(params, M)
    cost, dec = rotor.alloc_tables(n, L, M)
    work = rotor.alloc_workspace(n, L, M)
    st = torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(st):
        rotor.rotor_solve(d_params, n, L, M, cost, dec, work, st)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        rotor.rotor_solve(d_params, n, L, M, cost, dec, work, st)
    torch.cuda.synchronize()
    for _ in range(3):
        cost.fill_(-7)
        dec.fill_(-7)
        work.fill_(-7)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert_same(params, M, cost, dec)


@pytest.mark.parametrize("schedule", ["blocked", "rounds"])
def test_two_stream_fill_replays_from_a_captured_graph(schedule):
    # the blocked order forks its inner middle products onto the library's
    # side stream and joins it back with events: under capture that is a
    # fork and a join of the graph, and every replay must rebuild the tables
    import torch
    from paper_1911_13214_amd import rotor
    L, M = 80, 300
    params = chaingen.random_chains(1, L, seed=808)
    say(f"graph replay of the two-stream blocked fill L={L} M={M} {schedule}")
    d_params = rotor.upload_params(params, M)
    cost, dec = rotor.alloc_tables(1, L, M)
    work = rotor.alloc_workspace(1, L, M)
    st = torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(st):
        rotor.rotor_solve_schedule(d_params, 1, L, M, cost, dec, work, schedule, st)
    torch.cuda.synchronize()
    assert_same(params, M, cost, dec)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        rotor.rotor_solve_schedule(d_params, 1, L, M, cost, dec, work, schedule, st)
    torch.cuda.synchronize()
    for _ in range(3):
        cost.fill_(-7)
        dec.fill_(-7)
        work.fill_(-7)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert_same(params, M, cost, dec)


@pytest.mark.parametrize("schedule", ["blocked", "rounds"])
def test_two_stream_fills_from_two_host_threads(schedule):
    # solves from several host threads share the device's side stream: each
    # enqueues under the library's lock, and every table must come out whole
    import threading
    import torch
    from paper_1911_13214_amd import rotor
    L, M = 72, 260
    chains = [chaingen.random_chains(1, L, seed=900 + i) for i in range(2)]
    say(f"two host threads, two-stream blocked fills L={L} M={M} {schedule}")
    bufs = []
    for p in chains:
        bufs.append((rotor.upload_params(p, M), *rotor.alloc_tables(1, L, M), rotor.alloc_workspace(1, L, M),
                     torch.cuda.Stream()))
    torch.cuda.synchronize()
    errors = []

    def run(i):
        try:
            d_params, cost, dec, work, st = bufs[i]
            for _ in range(4):
                rotor.rotor_solve_schedule(d_params, 1, L, M, cost, dec, work, schedule, st)
            st.synchronize()
        except Exception as e:  # reported in the main thread
            errors.append(e)

    threads = [threading.Thread(target=run, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    torch.cuda.synchronize()
    for p, (_, cost, dec, _, _) in zip(chains, bufs):
        assert_same(p, M, cost, dec)


def test_workspace_too_small_is_rejected():
    import torch
    from paper_1911_13214_amd import rotor
    params, L, M, n, _ = chaingen.config(2)
    d_params = rotor.upload_params(params, M)
    cost, dec = rotor.alloc_tables(n, L, M)
    need = rotor.rotor_workspace_bytes(n, L, M)
    small = torch.empty(need // 8 - 1, dtype=torch.int64, device="cuda")
    with pytest.raises(rotor.RotorError) as e:
        rotor.rotor_solve(d_params, n, L, M, cost, dec, small)
    assert e.value.status == rotor.ROTOR_EINVAL
