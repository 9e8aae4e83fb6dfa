"""Long rows of CSR,WO that the feature pass of seer_spmv_auto finds (by default from 2^25 nonzeros on): against sums in 64
bits, and where they are not to be summed apart -- another schedule chosen, too few of them, too little scratch
memory -- against the bits of seer_spmv."""
import numpy as np
import pytest

import paper_2403_17017_amd as S

from gpu_util import announce

pytestmark = pytest.mark.gpu
COLS = 1_500_000
LEAST = 32 * -(-COLS // 32768)               # entries of the shortest long row


def tree(yes, no=S.CSR_TM):
    """Gathers (the longest row decides), then `yes`."""
    return S.Tree([4, -1, -1], [0.5, 0, 0], [1, -1, -1], [2, -1, -1], [-1, no, yes])


def deep_tree(yes):
    """Seven comparisons deep: walked node by node."""
    n = 7
    return S.Tree([4] * n + [-1] * (n + 1), [0.5] * n + [0.0] * (n + 1), [n + k for k in range(n)] + [-1] * (n + 1),
                  [k + 1 for k in range(n - 1)] + [2 * n] + [-1] * (n + 1), [-1] * n + [S.CSR_MP] * n + [yes])


@pytest.fixture(scope="module", params=["many", "few", "ends"])
def matrix(request):
    import torch
    rng = np.random.default_rng(7)
    if request.param == "few":               # long rows of fewer than 2^23 entries together
        lens = rng.integers(0, 40, 1_760_003)
        lens[rng.integers(0, len(lens), 60)] = 30_000
    else:
        lens = np.minimum(rng.zipf(1.7, 700_001), 150_000)
        if request.param == "ends":          # the first and the last row long, one exactly at the limit
            lens[[0, -1]] = 60_000, LEAST
    while lens.sum() < 1 << 25:
        lens = np.concatenate([lens, np.minimum(rng.zipf(1.7, 40_001), 150_000)])
    rp = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).cuda()
    nnz, rows = int(rp[-1]), len(lens)
    g = torch.Generator(device="cuda:0")
    g.manual_seed(8)
    row = torch.repeat_interleave(torch.arange(rows, device="cuda:0"), torch.from_numpy(lens).cuda(), output_size=nnz)
    key, _ = torch.sort(row * COLS + torch.randint(0, COLS, (nnz,), generator=g, device="cuda:0"))
    ci = (key - row * COLS).to(torch.int32)
    va = torch.rand(nnz, generator=g, device="cuda:0") * 2 - 1
    x = torch.rand(COLS, generator=g, device="cuda:0") * 2 - 1
    p = va.double() * x.double()[ci.long()]
    off = rp.long()
    ref = torch.segment_reduce(p, "sum", offsets=off, initial=0.0)
    bound = torch.segment_reduce(p.abs(), "sum", offsets=off, initial=0.0)
    return request.param, S.DeviceCSR(rows, COLS, rp, ci, va, nnz), x, ref, bound


def auto(A, t, x, ws, want):
    import torch
    y = torch.full((A.rows,), float("nan"), device="cuda:0")
    S.seer_spmv_auto(A, t, x, y, ws)
    assert S.seer_spmv_auto_result(ws)[1] == want
    return y


def check(y, ref, bound, what):
    import torch
    assert not bool(torch.isnan(y).any()), what
    assert bool(((y.double() - ref).abs() <= 1e-5 * bound).all()), what


def test_parity_and_graph(matrix):
    import torch
    name, A, x, ref, bound = matrix
    announce(f"gathered long rows {name} rows={A.rows} nnz={A.nnz}")
    ws = torch.randint(0, 256, (S.spmv_auto_workspace_bytes(A.rows, A.nnz),), dtype=torch.uint8, device="cuda:0")
    y = auto(A, tree(S.CSR_WO), x, ws, S.CSR_WO)
    check(y, ref, bound, name)
    plain = torch.empty_like(y)
    S.seer_spmv(S.CSR_WO, A, x, plain)
    assert torch.equal(y, plain) == (name == "few")
    out, g = torch.empty_like(y), torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        S.seer_spmv_auto(A, tree(S.CSR_WO), x, out, ws)
    for _ in range(3):
        out.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, y)


def test_features_are_the_same(matrix):
    name, A, x, _, _ = matrix
    announce(f"features beside long rows {name}")
    ws = S.alloc_workspace(S.spmv_auto_workspace_bytes(A.rows, A.nnz))
    auto(A, tree(S.CSR_WO), x, ws, S.CSR_WO)
    f, _ = S.seer_spmv_auto_result(ws)
    assert f.vector().tobytes() == S.seer_features(A).vector().tobytes()


@pytest.mark.parametrize("kid", [S.CSR_MP, S.CSR_BM])
def test_another_schedule_chosen(matrix, kid):
    import torch
    name, A, x, ref, bound = matrix
    announce(f"gathered long rows {name}, kernel {kid} chosen")
    ws = S.alloc_workspace(S.spmv_auto_workspace_bytes(A.rows, A.nnz))
    y = auto(A, tree(kid, S.CSR_WO), x, ws, kid)             # (CSR,WO stays reachable)
    check(y, ref, bound, name)
    want = torch.empty_like(y)
    S.seer_spmv(kid, A, x, want)
    assert torch.equal(y, want)


def test_deep_trees_misaligned_offsets_and_little_memory(matrix):
    import torch
    name, A, x, ref, bound = matrix
    announce(f"gathered long rows {name}: deep tree, offsets at 4 bytes, little memory")
    ws = S.alloc_workspace(S.spmv_auto_workspace_bytes(A.rows, A.nnz))
    y = auto(A, tree(S.CSR_WO), x, ws, S.CSR_WO)
    check(auto(A, deep_tree(S.CSR_WO), x, ws, S.CSR_WO), ref, bound, name)
    at4 = torch.empty(A.rows + 2, dtype=torch.int32, device="cuda:0")
    at4[1:] = A.row_ptr
    B = S.DeviceCSR(A.rows, A.cols, at4[1:], A.col_idx, A.values, A.nnz)
    assert torch.equal(auto(B, tree(S.CSR_WO), x, ws, S.CSR_WO), y)
    S.set_tuning("long_rows", 0)
    try:
        small = S.alloc_workspace(S.spmv_auto_workspace_bytes(A.rows, A.nnz))
    finally:
        S.set_tuning("long_rows", -1)
    assert small.numel() < ws.numel()
    plain = torch.empty_like(y)
    S.seer_spmv(S.CSR_WO, A, x, plain)
    assert torch.equal(auto(A, tree(S.CSR_WO), x, small, S.CSR_WO), plain)


def test_short_rows_have_the_bits_of_the_direct_product(matrix):
    """Rows too short to go apart are added up as without the stage, also in a chunk that a long row shares."""
    import torch
    name, A, x, _, _ = matrix
    announce(f"rows beside long rows {name}")
    ws = S.alloc_workspace(S.spmv_auto_workspace_bytes(A.rows, A.nnz))
    y = auto(A, tree(S.CSR_WO), x, ws, S.CSR_WO)
    plain = torch.empty_like(y)
    S.seer_spmv(S.CSR_WO, A, x, plain)
    short = A.row_ptr[1:] - A.row_ptr[:-1] < LEAST
    assert int((y != plain)[short].sum()) == 0


@pytest.mark.parametrize("walk", ["deep", "workgroup"])
def test_few_long_rows_stay_whoever_selects(matrix, walk):
    """A tree that the nodes are walked for, or a selection by a workgroup: the same rows go apart as where one wave selects."""
    import torch
    name, A, x, _, _ = matrix
    announce(f"gathered long rows {name}, selection {walk}")
    ws = S.alloc_workspace(S.spmv_auto_workspace_bytes(A.rows, A.nnz))
    y = auto(A, tree(S.CSR_WO), x, ws, S.CSR_WO)
    t = deep_tree(S.CSR_WO) if walk == "deep" else tree(S.CSR_WO)
    S.set_tuning("auto_select_wave", 0 if walk == "workgroup" else -1)
    try:
        z = auto(A, t, x, ws, S.CSR_WO)
    finally:
        S.set_tuning("auto_select_wave", -1)
    assert torch.equal(z, y)
