"""The sequence walk reads ahead in runs of 32 frames: chains whose runs of F_all
end just before, at and past that, against the oracle's Algorithm 2."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_1911_13214_amd import chaingen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [1, 2, 31, 32, 33, 63, 64, 65, 66, 98])
def test_walk_runs(L):
    from gpu_util import solve_on_gpu
    from paper_1911_13214_amd import rotor

    p = chaingen.random_chains(1, L, seed=500 + L, wa_hi=4)
    top = rotor.rotor_store_all_peak(p)
    M = min(top + 3, 700)
    print(f"walk L={L} M={M}", flush=True)
    d_params, _, dec = solve_on_gpu(p, M)
    C, _ = orc.solve(p, M)
    budgets = sorted(set(np.linspace(0, M, 25).astype(int)) | {M, max(0, M - 1)})
    for m, seq in zip(budgets, rotor.reconstruct(d_params, 1, L, M, dec, 0, budgets)):
        assert seq == orc.reconstruct(p, M, C, int(m)), m


def test_walk_longest_chain():
    # the longest chain the walk takes: no memory limit, one run of F_all
    import torch

    from paper_1911_13214_amd import rotor
    L = rotor.MAX_L_RECONSTRUCT
    d_params = torch.ones((1, 6, L), dtype=torch.int64, device="cuda")
    rows = L * (L + 1) // 2
    pitch = rotor.rotor_layout(1, L, 0)[0]
    d_params[0, 2:] = 0  # no sizes: M = 0 is enough
    dec = torch.zeros((rows, pitch), dtype=torch.int16, device="cuda")
    ops = torch.zeros((1, 2 * L, 2), dtype=torch.int32, device="cuda")
    count = torch.zeros(1, dtype=torch.int64, device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    print(f"walk L={L} M=0", flush=True)
    rotor.rotor_reconstruct(d_params, 1, L, 0, dec, 0, torch.zeros(1, dtype=torch.int64, device="cuda"), 2 * L, ops,
                            count, status)
    torch.cuda.synchronize()
    assert status.item() == rotor.ROTOR_OK and count.item() == 2 * L
    o = ops[0].cpu().numpy()
    assert (o[:L, 0] == rotor.F_ALL).all() and (o[:L, 1] == np.arange(1, L + 1)).all()
    assert (o[L:, 0] == rotor.B).all() and (o[L:, 1] == np.arange(L, 0, -1)).all()
