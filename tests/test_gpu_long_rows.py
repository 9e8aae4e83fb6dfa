"""CSR,WO's long rows summed apart with slabs of x in LDS: parity against the oracle where rows begin and
end at chunk boundaries, beside empty rows, at either end of the matrix, with columns that do not ascend, that
are local, and with too little scratch memory; the same through the selection on the device."""
import numpy as np
import pytest

import paper_2403_17017_amd as S
from workloads import csr_gen as G

from gpu_util import announce, assert_parity, oracle_of, upload

pytestmark = pytest.mark.gpu
CHUNK, COLS = 4096, 1_400_000
LEAST = 32 * -(-COLS // 32768)               # entries of the shortest long row


@pytest.fixture
def long_rows():
    S.set_tuning("long_rows", 1)
    yield
    S.set_tuning("long_rows", -1)


def edges():
    """Rows placed against the chunks, then Zipf-like ones up to 9 M nonzeros."""
    lens = [0, 0, 0, 3 * CHUNK, 0, 0]                       # begins at 0 behind empty rows, ends on a boundary, empties behind
    lens += [2 * CHUNK, 0]                                  # whole chunks, both ends on a boundary
    lens += [5, LEAST, 7]                                   # inside one chunk: stays with CSR,WO
    lens += [CHUNK - 12 - LEAST - 1, LEAST, 0, 0, LEAST + CHUNK, 1, LEAST - 1, LEAST - 1, LEAST - 1]
    lens += [100_000, 100_000, 0, 200_000] + [0] * 3000 + [150_000]
    lens += [2 * CHUNK - 1, 2 * CHUNK + 1, 1, 1, CHUNK + 1]
    rng = np.random.default_rng(5)
    while sum(lens) < 8_700_000:
        lens += [int(v) for v in np.minimum(rng.zipf(1.5, 400), 60_000)]
    lens += [0, 40_000]                                     # the matrix ends with a long row
    return G.explicit_lengths(lens, COLS, 41, "edges")


def reordered(A):
    """Long rows whose columns ascend nearly, not at all, and all lie in a few slabs."""
    ci = A.col_idx.copy()
    rng = np.random.default_rng(6)
    lens = np.diff(A.row_ptr)
    for n, i in enumerate(np.flatnonzero(lens >= LEAST)):
        a, e = int(A.row_ptr[i]), int(A.row_ptr[i + 1])
        if n % 5 == 1:                                      # neighbours swapped
            m = (e - a) // 2 * 2
            ci[a:a + m] = ci[a:a + m].reshape(-1, 2)[:, ::-1].ravel()
        elif n % 5 == 2:                                    # quarters in place, the rest shuffled between them
            for q in range(4):
                s, t = a + (e - a) * q // 4 + 1, a + (e - a) * (q + 1) // 4
                ci[s:t] = rng.permutation(ci[s:t])
        elif n % 5 == 3:
            ci[a:e] = rng.permutation(ci[a:e])
        elif n % 5 == 4:                                    # local
            ci[a:e] = np.sort(rng.integers(700_000, 760_000, e - a))
    return G.HostCSR(A.rows, A.cols, A.row_ptr, ci, A.values, "reordered")


def no_long_rows():
    return G.random_lengths(450_007, COLS, 0, 40, 42)


def all_long():
    return G.random_lengths(2_900, COLS, 1_500, 4_700, 43)


@pytest.mark.parametrize("make", [edges, lambda: reordered(edges()), no_long_rows, all_long],
                         ids=["edges", "reordered", "none", "all"])
def test_parity(long_rows, make):
    import torch
    A = make()
    assert A.nnz >= 1 << 23
    announce(f"long rows {A.name} rows={A.rows} nnz={A.nnz}")
    dA = upload(A)
    x = G.dense_vector(A.cols, 3)
    xd = torch.from_numpy(x).cuda()
    y_ref, bound = oracle_of(A, x)

    def wo(ws):
        y = torch.full((A.rows,), float("nan"), dtype=torch.float32, device="cuda:0")
        S.seer_spmv(S.CSR_WO, dA, xd, y, workspace=ws)
        torch.cuda.synchronize()
        return y.cpu().numpy()
    need = S.spmv_workspace_bytes(S.CSR_WO, A.rows, A.nnz)
    ws = S.alloc_workspace(need)
    ws.fill_(0x5A)
    y = wo(ws)
    assert_parity(y, y_ref, bound, f"CSR,WO on {A.name}")
    assert np.array_equal(y, wo(ws)), "again, the same bits"
    S.set_tuning("long_rows", 0)
    small = S.alloc_workspace(S.spmv_workspace_bytes(S.CSR_WO, A.rows, A.nnz))
    plain = wo(small)
    S.set_tuning("long_rows", 1)
    assert small.numel() < need
    assert np.array_equal(wo(small), plain), "without the scratch memory: as without the stage"
    assert np.array_equal(plain, y) == (A.name.startswith("unif") and "1500" not in A.name)
    # through the selection: decided by the host, and gathered on the device (with and without CSR,WO chosen)
    for tree, kid in ((S.Tree.constant(S.CSR_WO), S.CSR_WO),
                      (S.Tree([4, -1, -1], [0.5, 0, 0], [1, -1, -1], [2, -1, -1], [-1, S.CSR_MP, S.CSR_WO]), S.CSR_WO),
                      (S.Tree([4, -1, -1], [0.5, 0, 0], [1, -1, -1], [2, -1, -1], [-1, S.CSR_WO, S.CSR_MP]), S.CSR_MP)):
        aws = S.alloc_workspace(S.spmv_auto_workspace_bytes(A.rows, A.nnz))
        aws.fill_(0x5A)
        g, out = torch.cuda.CUDAGraph(), torch.full((A.rows,), float("nan"), dtype=torch.float32, device="cuda:0")
        with torch.cuda.graph(g):
            S.seer_spmv_auto(dA, tree, xd, out, aws)
        for _ in range(3):
            out.fill_(float("nan"))
            g.replay()
            torch.cuda.synchronize()
            assert S.seer_spmv_auto_result(aws)[1] == kid
            got = out.cpu().numpy()
            assert_parity(got, y_ref, bound, f"auto on {A.name}")
            assert kid != S.CSR_WO or np.array_equal(got, y)


def test_non_finite_x_reaches_only_the_rows_that_use_it(long_rows):
    import torch
    A = all_long()
    x = G.dense_vector(A.cols, 3)
    x[7::900_001] = np.inf
    announce(f"long rows, non-finite x {A.name}")
    y = torch.full((A.rows,), float("nan"), dtype=torch.float32, device="cuda:0")
    S.seer_spmv(S.CSR_WO, upload(A), torch.from_numpy(x).cuda(), y)
    torch.cuda.synchronize()
    row = np.repeat(np.arange(A.rows), np.diff(A.row_ptr))
    touched = np.zeros(A.rows, bool)
    touched[row[~np.isfinite(x[A.col_idx])]] = True
    assert np.array_equal(~np.isfinite(y.cpu().numpy()), touched)
