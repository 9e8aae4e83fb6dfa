"""GPU parity of the schedules whose gathers are ordered in time by column range, forced on small
matrices with the "gather_range" knob: against the oracle, against the plain order of gathers
(bit for bit where the sums are the same), and inside seer_spmv_auto."""
import numpy as np
import pytest

import paper_2403_17017_amd as S
from workloads import csr_gen as G

from gpu_util import announce, assert_parity, oracle_of, run_spmv, upload

pytestmark = pytest.mark.gpu

RANGED = (S.CSR_BM, S.CSR_MP, S.CSR_WO, S.CSR_A)


@pytest.fixture(autouse=True)
def restore_knob():
    yield
    S.set_tuning("gather_range", -1)


def cases():
    """(matrix, log2 of the columns per range): 2 ranges, the 32 that are the most, and between;
    chunks of whole tiles and with remainders of every length mod 4 at their ends, rows cut by
    chunks, waves that gather at once (bands) and waves that wait, columns up to the last one."""
    out = [(G.random_lengths(3_001, 70_000, 9, 60, 1), 16), (G.random_lengths(3_001, 65_536, 9, 60, 2), 11),
           (G.random_lengths(997, 4_099, 0, 300, 3), 8), (G.explicit_lengths([0] * 70 + [9_001] + [17] * 513, 9_001, 4), 12),
           (G.banded(5_003, 20, 5), 10), (G.laplacian_5pt(90), 9), (G.zipf_rows(20_011, s=1.6, cap=6_000, seed=6), 12),
           (G.empty_poisson(40_003, 9_999, 0.3, 4.0, seed=7), 10)]
    for n in (4095, 4096, 4097, 4098, 8191, 1, 3):
        out.append((G.explicit_lengths([n], 50_000, 10 + n, f"one-row-{n}"), 12))
    for n in (2047, 2049):
        out.append((G.explicit_lengths([11] * 7 + [n] + [10] * 9, 33_000, 30 + n, f"short-then-{n}"), 11))
    return out


@pytest.mark.parametrize("i", range(len(cases())))
def test_ranged_gathers_match_the_oracle_and_the_plain_order(i):
    import torch
    A, shift = cases()[i]
    x = G.dense_vector(A.cols, 50 + i)
    y_ref, bound = oracle_of(A, x)
    dA, xd = upload(A), torch.from_numpy(x).cuda()
    for k in RANGED:
        announce(f"gather_range={shift} kernel {k} {A.name} rows={A.rows} cols={A.cols} nnz={A.nnz}")
        S.set_tuning("gather_range", 0)
        plain = run_spmv(k, dA, xd, A.rows)
        S.set_tuning("gather_range", shift)
        ranged = run_spmv(k, dA, xd, A.rows)
        assert_parity(ranged, y_ref, bound, f"kernel {k} on {A.name}, ranges of 2^{shift}")
        if k != S.CSR_BM:
            assert ranged.tobytes() == plain.tobytes(), f"kernel {k} on {A.name}: the order of gathers changed y"
        plan = S.seer_spmv_prepare(k, dA)
        y = torch.full((A.rows,), float("nan"), device="cuda:0")
        S.seer_spmv_prepared(plan, dA, xd, y)
        torch.cuda.synchronize()
        assert y.cpu().numpy().tobytes() == ranged.tobytes(), f"prepared kernel {k} on {A.name}"


@pytest.mark.parametrize("kid", range(S.NUM_DIRECT_KERNELS))
@pytest.mark.parametrize("gathered", [False, True])
def test_combined_kernel_by_range_is_the_stand_alone_one(kid, gathered):
    """The choice made on the host alone (a one-leaf tree) and on the device; long and short rows."""
    import torch
    S.set_tuning("gather_range", 12)
    tree = S.Tree([6, -1, -1], [-1.0, 0, 0], [1, -1, -1], [2, -1, -1], [-1, (kid + 1) % 5, kid]) if gathered \
        else S.Tree.constant(kid)
    for A in (G.random_lengths(4_001, 60_001, 0, 30, 71), G.random_lengths(301, 60_001, 200, 500, 72),
              G.random_lengths(9_001, 30_001, 0, 9, 73)):
        announce(f"auto by range kernel {kid} {A.name} rows={A.rows} cols={A.cols} nnz={A.nnz}")
        x = G.dense_vector(A.cols, 3)
        y_ref, bound = oracle_of(A, x)
        dA, xd = upload(A), torch.from_numpy(x).cuda()
        y = torch.full((A.rows,), float("nan"), device="cuda:0")
        ws = S.alloc_workspace(S.spmv_auto_workspace_bytes(A.rows, A.nnz))
        S.seer_spmv_auto(dA, tree, xd, y, ws)
        assert S.seer_spmv_auto_result(ws)[1] == kid
        torch.cuda.synchronize()
        assert_parity(y.cpu().numpy(), y_ref, bound, f"auto kernel {kid} on {A.name}")
        assert y.cpu().numpy().tobytes() == run_spmv(kid, dA, xd, A.rows).tobytes()


def test_infinite_and_nan_entries_of_x_reach_only_their_rows():
    import torch
    A = G.random_lengths(2_003, 20_011, 9, 40, 81)
    x = G.dense_vector(A.cols, 4)
    x[[5, 9_999]] = np.inf
    x[20_010] = np.nan
    dA, xd = upload(A), torch.from_numpy(x).cuda()
    for k in RANGED:
        S.set_tuning("gather_range", 0)
        plain = run_spmv(k, dA, xd, A.rows)
        S.set_tuning("gather_range", 11)
        ranged = run_spmv(k, dA, xd, A.rows)
        assert np.array_equal(np.isnan(plain), np.isnan(ranged)) and np.array_equal(np.isinf(plain), np.isinf(ranged))


def test_misaligned_entries_and_odd_range_counts_take_the_plain_order():
    import torch
    A = G.random_lengths(1_003, 40_000, 9, 30, 91)
    x = G.dense_vector(A.cols, 5)
    xd = torch.from_numpy(x).cuda()
    y_ref, bound = oracle_of(A, x)
    for dA, shift in ((upload(A, misalign=True), 12), (upload(A), 10), (upload(A), 20)):   # 40 ranges, one range
        for k in RANGED:
            S.set_tuning("gather_range", 0)
            plain = run_spmv(k, dA, xd, A.rows)
            S.set_tuning("gather_range", shift)
            got = run_spmv(k, dA, xd, A.rows)
            assert_parity(got, y_ref, bound, f"kernel {k}")
            assert got.tobytes() == plain.tobytes()


@pytest.mark.parametrize("nnz", [(1 << 21) - 1, 1 << 21])
def test_adaptive_from_two_million_entries_on(nnz):
    """Either side of the size from which CSR,A orders its gathers by itself: the same bits."""
    import torch
    A = G.explicit_lengths([21] * (nnz // 21) + [nnz % 21], (11 << 17) + 1, 95, f"rows-of-21-{nnz}")
    assert A.nnz == nnz
    dA, xd = upload(A), torch.from_numpy(G.dense_vector(A.cols, 6)).cuda()
    S.set_tuning("gather_range", 0)
    plain = run_spmv(S.CSR_A, dA, xd, A.rows)
    S.set_tuning("gather_range", -1)
    y_ref, bound = oracle_of(A, xd.cpu().numpy())
    plan, y = S.seer_spmv_prepare(S.CSR_A, dA), torch.full((A.rows,), float("nan"), device="cuda:0")
    S.seer_spmv_prepared(plan, dA, xd, y)
    torch.cuda.synchronize()
    for got in (run_spmv(S.CSR_A, dA, xd, A.rows), y.cpu().numpy()):
        assert_parity(got, y_ref, bound, f"CSR,A at {nnz} entries")
        assert got.tobytes() == plain.tobytes()
