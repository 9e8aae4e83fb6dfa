"""GPU parity of CSR,S in bins (slabs of x in LDS): what the preparation keeps against the oracle's
slab plan for the same width, the product against the oracle's row sums, repeatability, and the rule
that takes a matrix to this form."""
import numpy as np
import pytest

import paper_2403_17017_amd as S
from oracle import seer_oracle as O
from workloads import csr_gen as G

from gpu_util import announce, assert_parity, oracle_of, upload

pytestmark = pytest.mark.gpu
W = 15                       # log2 of the columns per slab
NOMINAL, MOST = 15360, 16384  # nonzeros per chunk


@pytest.fixture
def bins():
    S.set_tuning("slab_bins", 1)
    yield
    S.set_tuning("slab_bins", -1)


def product(plan, dA, x):
    import torch
    y = torch.full((dA.rows,), float("nan"), dtype=torch.float32, device="cuda:0")
    S.seer_spmv_prepared(plan, dA, torch.from_numpy(x).cuda(), y)
    torch.cuda.synchronize()
    return y.cpu().numpy()


def check(A, width=W):
    announce(f"CSR,S in bins {A.name} rows={A.rows} cols={A.cols} nnz={A.nnz}")
    dA = upload(A)
    plan = S.seer_spmv_prepare(S.CSR_S, dA)
    assert plan.kernel_id == S.CSR_S and plan.ell_width == W and int(plan.c.split_rows) in (-1, -2)
    assert plan.n_blocks == -(-A.cols // (1 << W))
    assert int(plan.c.device_bytes) == S.slab_plan_bytes(A.rows, A.cols, A.nnz)
    want = O.slab_plan(A.rows, A.cols, A.row_ptr, A.col_idx, W)
    rp_z, p_idx, rp_j, ci, va = plan.slab_arrays(A.cols)
    assert np.array_equal(rp_z.astype(np.int64), want["rp_z"]) and np.array_equal(rp_j.astype(np.int64), want["rp_j"])
    assert np.array_equal(p_idx.astype(np.int64), want["p_idx"])
    assert np.array_equal(ci, A.col_idx[want["perm"]]) and np.array_equal(va, A.values[want["perm"]])
    x = G.dense_vector(A.cols, 3)
    y_ref, bound = oracle_of(A, x)
    y = product(plan, dA, x)
    assert_parity(y, y_ref, bound, f"CSR,S in bins on {A.name}")
    assert np.array_equal(y, product(S.seer_spmv_prepare(S.CSR_S, dA), dA, x)), "another plan, the same bits"
    return plan


def edge_cases():
    c = 600_011                                            # 19 slabs, the last one ragged
    return [
        G.explicit_lengths([0, 0, 0], c, 1, "no-nonzeros"),
        G.explicit_lengths([1], c, 2, "one"),
        G.explicit_lengths([0, 7, 0, 0, 3, 0], c, 4, "empties"),
        G.explicit_lengths([NOMINAL], c, 5, "one-chunk"),
        G.explicit_lengths([NOMINAL - 1, 2, 5], c, 6, "row-begins-one-before-the-cut"),
        G.explicit_lengths([NOMINAL, 1, 0, 0, 9], c, 7, "row-begins-at-the-cut"),
        G.explicit_lengths([2 * NOMINAL - MOST, MOST], c, 8, "a-row-that-just-moves-whole"),
        G.explicit_lengths([2 * NOMINAL - MOST - 1, MOST + 1], c, 9, "a-row-that-is-just-cut"),
        G.explicit_lengths([0] * 5000 + [200_000] + [0] * 5000 + [3, 70_000, 2], c, 10, "giant-rows-among-empties"),
        G.explicit_lengths([129] * 119 + [128] * 40, c, 11, "about-the-lanes-per-row-limit"),
        G.random_lengths(5_003, c, 0, 40, 21),
        G.random_lengths(1_237, 8_388_608, 50, 700, 22),   # 256 slabs, the most
        # runs of one row in one slab, of lengths about 4, 16 and 64, and across the 64 entries looked at together
        G.explicit_lengths([3, 4, 5, 15, 16, 17, 20, 63, 64, 65, 81, 3, 50, 16, 300, 4] * 40, c, 12, "short-runs"),
        G.explicit_lengths([70, 200, 500, 1100, 1300, 2000, 5000, 0, 1, 12_000] * 4, c, 13, "rows-of-runs"),
        G.zipf_rows(20_011, cols=c, s=1.6, cap=50_000, seed=23),
        G.banded(530_001, 3, 26),                          # buckets of one slab, and of two
    ]


def test_plan_and_product(bins):
    cut = [int(check(A).c.split_rows) for A in edge_cases()]
    assert -1 in cut and -2 in cut


def test_what_x_holds_reaches_only_the_rows_that_use_it(bins):
    """Infinities and NaN in x: padding entries read column 0 of their slab and must add nothing."""
    A = G.random_lengths(3_001, 600_011, 0, 30, 33)
    announce(f"CSR,S in bins, non-finite x {A.name}")
    x = G.dense_vector(A.cols, 3)
    x[:: 1 << W] = np.inf                                  # the first column of every slab
    x[(1 << W) + 5] = np.nan
    row = np.repeat(np.arange(A.rows), np.diff(A.row_ptr))
    touched = np.zeros(A.rows, bool)
    touched[row[~np.isfinite(x[A.col_idx])]] = True
    y = product(S.seer_spmv_prepare(S.CSR_S, upload(A)), upload(A), x)
    assert np.array_equal(~np.isfinite(y), touched)


@pytest.mark.parametrize("n", [5, 200, 40_000])
@pytest.mark.parametrize("what", ["descends", "outside"])
def test_refused_as_by_the_other_form(bins, n, what):
    B = G.random_lengths(60, 600_011, n, n, 6)
    ci = B.col_idx.copy()
    a = int(B.row_ptr[17])
    if what == "descends":
        ci[a + n - 2], ci[a + n - 1] = ci[a + n - 1] + 1 if ci[a + n - 1] + 1 < B.cols else B.cols - 1, ci[a + n - 2]
    else:
        ci[a + n - 1] = B.cols
    bad = G.HostCSR(B.rows, B.cols, B.row_ptr, ci, B.values, f"{what}-{n}")
    announce(f"CSR,S in bins refuses {bad.name}")
    with pytest.raises(S.SeerError) as ei:
        S.seer_spmv_prepare(S.CSR_S, upload(bad))
    assert ei.value.status == -1


def test_rule_and_scratch_limits():
    """From 9 * 2^20 nonzeros on by default, unless the columns are local; a plan keeps its form whatever
    the knobs say later; a product without enough scratch is refused."""
    import torch
    A = G.random_lengths(300_007, 1_300_000, 20, 50, 77)
    B = G.banded(600_011, 8, 78)
    assert A.nnz >= 9 << 20 and B.nnz >= 9 << 20
    announce(f"CSR,S in bins by rule {A.name} nnz={A.nnz}")
    dA = upload(A)
    plan = S.seer_spmv_prepare(S.CSR_S, dA)
    assert plan.ell_width == W and int(plan.c.split_rows) == -1
    x = G.dense_vector(A.cols, 3)
    y_ref, bound = oracle_of(A, x)
    S.set_tuning("slab_bins", 0)
    S.set_tuning("slab_shift", 18)
    try:
        assert_parity(product(plan, dA, x), y_ref, bound, "a plan in bins")
        other = S.seer_spmv_prepare(S.CSR_S, dA)
        assert other.ell_width == 18
        assert_parity(product(other, dA, x), y_ref, bound, "the other form")
    finally:
        S.set_tuning("slab_bins", -1)
        S.set_tuning("slab_shift", -1)
    local = S.seer_spmv_prepare(S.CSR_S, upload(B))
    assert local.ell_width == 19 and int(local.c.split_rows) >= 0
    xb = G.dense_vector(B.cols, 4)
    assert_parity(product(local, upload(B), xb), *oracle_of(B, xb), "a band")
    need = S.spmv_prepared_workspace_bytes(plan)
    xd, y = torch.from_numpy(x).cuda(), torch.empty(A.rows, device="cuda:0")
    with pytest.raises(S.SeerError) as ei:
        S.seer_spmv_prepared(plan, dA, xd, y, workspace=S.alloc_workspace(need - 256))
    assert ei.value.status == -4
    S.seer_spmv_prepared(plan, dA, xd, y, workspace=S.alloc_workspace(need))
    # captured and replayed, with eager work in between
    ws, ref = S.alloc_workspace(need), torch.clone(y)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        S.seer_spmv_prepared(plan, dA, xd, y, workspace=ws)
    for _ in range(3):
        y.fill_(float("nan"))
        ws.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, ref)


@pytest.mark.parametrize("by_bins", [True, False])
def test_lines_shared_within_a_long_row(by_bins):
    """Entries of one long row share lines of x without being local; a wide band is local although 256 of
    its entries lie in a few rows."""
    A = G.explicit_lengths([100_003] * 100, 1_100_011, 81) if by_bins else G.banded(530_003, 40, 82)
    announce(f"CSR,S by rule {A.name} nnz={A.nnz}")
    assert A.nnz >= 9 << 20
    plan = S.seer_spmv_prepare(S.CSR_S, upload(A))
    assert (int(plan.c.split_rows) < 0) == by_bins
    if by_bins:
        x = G.dense_vector(A.cols, 5)
        assert_parity(product(plan, upload(A), x), *oracle_of(A, x), A.name)


def test_more_preparations_at_once_than_mailboxes(bins):
    """A preparation waits for the device twice, each time with one of 64 result mailboxes: 70 at once end."""
    import threading

    import torch
    A = G.random_lengths(3_001, 600_011, 0, 30, 33)
    announce(f"70 preparations at once {A.name}")
    dA, x = upload(A), G.dense_vector(A.cols, 3)
    mem = [S.alloc_workspace(S.slab_plan_bytes(A.rows, A.cols, A.nnz)) for _ in range(70)]
    streams = [torch.cuda.Stream() for _ in range(4)]
    plans = [None] * len(mem)

    def prepare(k):
        plans[k] = S.seer_spmv_prepare(S.CSR_S, dA, plan_mem=mem[k], stream=streams[k % 4])
    torch.cuda.synchronize()
    threads = [threading.Thread(target=prepare, args=(k,)) for k in range(len(mem))]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
    y_ref, bound = oracle_of(A, x)
    for plan in plans[::10]:
        assert_parity(product(plan, dA, x), y_ref, bound, A.name)
    assert all(int(p.c.split_rows) == int(plans[0].c.split_rows) for p in plans)


@pytest.mark.parametrize("where", ["first", "middle", "last"])
@pytest.mark.parametrize("run", [30_000, 400_000])
def test_a_long_run_of_empty_rows_is_not_for_bins(where, run):
    """One workgroup would have it to itself, in the preparation and in every product."""
    n, at = 320_003, {"first": 0, "middle": 150_001, "last": 320_003}[where]
    lens = np.full(n, 30)
    lens[0] += 7
    A = G.explicit_lengths(np.insert(lens, at, np.zeros(run, lens.dtype)).tolist(), 1_300_001, 91, f"{run}-empty-rows-{where}")
    announce(f"CSR,S by rule {A.name} nnz={A.nnz}")
    assert A.nnz >= 9 << 20
    plan = S.seer_spmv_prepare(S.CSR_S, upload(A))
    assert (int(plan.c.split_rows) < 0) == (run == 30_000)
    x = G.dense_vector(A.cols, 5)
    assert_parity(product(plan, upload(A), x), *oracle_of(A, x), A.name)


def test_memory_for_the_arrays_alone_is_enough():
    """Where bins take more than the arrays (few rows, many columns) memory for the arrays still gives them; less is
    refused; and what the library chooses is prepared rather than another schedule."""
    import ctypes as C
    A = G.explicit_lengths([2_001] * 5_003, 8_000_011, 61, "few-rows-many-columns")
    announce(f"CSR,S with memory for the arrays alone {A.name} nnz={A.nnz}")
    assert A.nnz >= 9 << 20
    both = S.slab_plan_bytes(A.rows, A.cols, A.nnz)
    S.set_tuning("slab_bins", 0)
    arrays = S.slab_plan_bytes(A.rows, A.cols, A.nnz)
    S.set_tuning("slab_bins", -1)
    assert 0 < arrays < both
    dA, x = upload(A), G.dense_vector(A.cols, 5)
    y_ref, bound = oracle_of(A, x)
    model = S.Model(S.Tree.constant(S.CSR_S), S.Tree.constant(S.CSR_S), S.Tree([-1], [0.0], [-1], [-1], [0], n_classes=2))
    for size, in_bins in ((both, True), (both - 1, False), (arrays, False)):
        mem = S.alloc_workspace(both)
        mem[size:] = 0x5A
        for plan in (S.seer_spmv_prepare(S.CSR_S, dA, plan_mem=mem[:size]), S.seer_spmv_plan(dA, model, 50, plan_mem=mem[:size])[0]):
            assert plan.kernel_id == S.CSR_S and (int(plan.c.split_rows) < 0) == in_bins
            assert int(plan.c.device_bytes) == (both if in_bins else arrays)
            assert_parity(product(plan, dA, x), y_ref, bound, A.name)
        assert bool((mem[size:] == 0x5A).all())
    cs, c, mem = dA.c_struct(), S.binding.seer_plan(), S.alloc_workspace(arrays)
    rc = S.lib().seer_spmv_prepare(S.CSR_S, C.byref(cs), mem.data_ptr(), arrays - 1, None, C.byref(c))
    assert rc == -4 and c.device_bytes == both and c.kernel_id == 0


@pytest.mark.parametrize("cols,in_bins", [(1 << 23, True), ((1 << 23) + 1, False)])
def test_more_slabs_than_bins_hold(bins, cols, in_bins):
    """256 slabs, and one more: size, preparation and product agree on the form."""
    A = G.random_lengths(2_003, cols, 5, 60, 51)
    announce(f"CSR,S of {cols} columns {A.name}")
    dA, x = upload(A), G.dense_vector(A.cols, 5)
    size = S.slab_plan_bytes(A.rows, A.cols, A.nnz)
    plan = S.seer_spmv_prepare(S.CSR_S, dA)
    assert (int(plan.c.split_rows) < 0) == in_bins and plan.n_blocks == (256 if in_bins else 9)
    assert int(plan.c.device_bytes) == size
    S.set_tuning("slab_bins", 0)
    assert (S.slab_plan_bytes(A.rows, A.cols, A.nnz) == size) == (not in_bins)
    assert_parity(product(plan, dA, x), *oracle_of(A, x), A.name)
