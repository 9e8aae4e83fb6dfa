"""ELL,TM with the distances from row to column kept behind the arrays: the same bits as without them, on
matrices that have one distance per 64 rows everywhere, mostly, in half of the slots, and nowhere."""
import numpy as np
import pytest

import paper_2403_17017_amd as S
from workloads import csr_gen as G

from gpu_util import announce, assert_parity, oracle_of, upload

pytestmark = pytest.mark.gpu


def half_scattered(rows, n, seed):
    """n near columns at one distance, then n anywhere behind them."""
    rng = np.random.default_rng(seed)
    near = np.arange(rows)[:, None] + np.arange(n)[None, :]
    far = np.sort(rng.integers(rows + n, 2 * rows, (rows, n)), axis=1)
    ci = np.concatenate([near, far], axis=1).astype(np.int32).ravel()
    rp = (np.arange(rows + 1) * 2 * n).astype(np.int32)
    return G.HostCSR(rows, 2 * rows, rp, ci, rng.uniform(-1, 1, ci.size).astype(np.float32), f"half-scattered-{rows}")


CASES = [
    (lambda: G.laplacian_5pt(1000), True),           # 15 000 blocks, one in eight with a grid row's end
    (lambda: G.laplacian_5pt(700), True),
    (lambda: G.laplacian_5pt(9), False),             # 81 rows: arrays below 16 MB, like the next
    (lambda: G.banded(64_000, 4, 6), False),
    (lambda: G.banded(699_968, 1, 5), True),         # whole blocks of 64
    (lambda: G.banded(240_003, 4, 6), True),         # nine slots: one past the eight fetched together
    (lambda: G.banded(40_001, 30, 7), True),         # 61 slots
    (lambda: G.banded(26_001, 40, 7), True),         # 81: more than a wave has lanes
    (lambda: G.banded(17_001, 64, 8), True),         # 129
    (lambda: half_scattered(350_007, 3, 9), False),
    (lambda: G.random_lengths(240_007, 240_007, 0, 9, 10), False),
]


@pytest.mark.parametrize("k", range(len(CASES)))
def test_same_bits_with_and_without(k):
    import torch
    make, kept = CASES[k]
    A = make()
    announce(f"ELL,TM distances {A.name} rows={A.rows} nnz={A.nnz}")
    dA = upload(A)
    width = int(np.diff(A.row_ptr).max())
    x = G.dense_vector(A.cols, 3)
    x[A.cols // 2] = np.inf                          # reaches exactly the rows that have the column
    xd = torch.from_numpy(x).cuda()
    need = S.ell_plan_bytes(A.rows, width)
    arena = S.alloc_workspace(max(need, S.features_workspace_bytes(A.rows)) + need // 100 + (1 << 20))
    plan = S.seer_spmv_prepare(S.ELL_TM, dA, plan_mem=arena)
    used = int(plan.c.device_bytes)
    assert used == need + (-(-A.rows // 64) * width * 4 + 255) // 256 * 256 + 256 if kept else used == need
    arena[used:] = 0x5A                              # what lies behind the plan is the program's again
    exact = S.alloc_workspace(max(S.ell_plan_bytes(A.rows, width), S.features_workspace_bytes(A.rows)))
    # (the reduction's workspace may leave room behind a small matrix's arrays: cut it off)
    plain = S.seer_spmv_prepare(S.ELL_TM, dA, plan_mem=exact)
    assert plan.n_blocks == int(kept) and plain.n_blocks == 0 and int(plain.c.device_bytes) == need
    ys = []
    for p in (plan, plain):
        y = torch.full((A.rows,), float("nan"), dtype=torch.float32, device="cuda:0")
        S.seer_spmv_prepared(p, dA, xd, y)
        torch.cuda.synchronize()
        ys.append(y.cpu().numpy())
    assert ys[0].tobytes() == ys[1].tobytes()
    got_c, got_v = plan.ell_arrays()
    want_c, want_v = plain.ell_arrays()
    assert np.array_equal(got_c, want_c) and got_v.tobytes() == want_v.tobytes()
    x[A.cols // 2] = 1.0
    y = torch.full((A.rows,), float("nan"), dtype=torch.float32, device="cuda:0")
    S.seer_spmv_prepared(plan, dA, torch.from_numpy(x).cuda(), y)
    torch.cuda.synchronize()
    assert_parity(y.cpu().numpy(), *oracle_of(A, x), f"ELL,TM on {A.name}")
