"""GPU parity of the asynchronous path (seer_spmv_auto): device-side feature
derivation and tree walk must match the oracle bit for bit, and y must match both
the oracle (tolerance) and seer_spmv with the same kernel id (bit for bit)."""
import numpy as np
import pytest

import paper_2403_17017_amd as S
from oracle import seer_oracle as O
from workloads import csr_gen as G

from gpu_util import announce, assert_features_equal, assert_parity, oracle_of, run_spmv, upload
from test_gpu_parity import ALL

pytestmark = pytest.mark.gpu

# var_len <= 50 ? (mean_len <= 8 ? (rows <= 20000 ? TM : BM) : WM) : MP
REAL_TREE = ([6, 3, 0, -1, -1, -1, -1], [50.0, 8.0, 20000.0, 0, 0, 0, 0],
             [1, 2, 3, -1, -1, -1, -1], [6, 5, 4, -1, -1, -1, -1], [-1, -1, -1, 0, 2, 1, 3])


def check_record(A, tree, f, kid, what):
    """The record seer_spmv_auto left: the kernel id is the oracle's walk over the full feature
    vector; the features are the gathered ones, bit for bit -- unless the known features alone
    leave one kernel reachable (the oracle's definition), in which case nothing was gathered
    and the record holds the known features and the mark."""
    want = O.features(A.rows, A.cols, A.row_ptr)
    assert kid == O.select(want["f"], *tree.arrays), what
    kf = O.known_features(A.rows, A.cols, A.nnz)
    reach = O.reachable_classes(kf, *tree.arrays)
    assert kid in reach, what
    if len(reach) == 1:
        assert int(f.max_len) == int(f.min_len) == int(f.empty_rows) == -1, f"{what}: gathered although decided"
        assert (int(f.rows), int(f.cols), int(f.nnz)) == (A.rows, A.cols, A.nnz), what
        assert f.vector().tobytes() == kf.tobytes(), what
    else:
        assert_features_equal(f, want, what)
    return len(reach) == 1


@pytest.fixture
def no_pruning():
    """Every schedule counts as reachable, features are always gathered (the tests of the
    device-side derivation and of the combined kernel force schedules with one-leaf trees)."""
    S.set_tuning("auto_prune", 0)
    yield
    S.set_tuning("auto_prune", -1)


def run_auto(dA, tree, xd, rows, ws):
    import torch
    y = torch.full((max(rows, 1),), float("nan"), dtype=torch.float32, device="cuda:0")
    S.seer_spmv_auto(dA, tree, xd, y, ws)
    f, kid = S.seer_spmv_auto_result(ws)
    return y[:rows].cpu().numpy(), f, kid


@pytest.fixture(scope="module")
def cases():
    out = []
    for A in ALL:
        x = G.dense_vector(A.cols, 1000 + len(out))
        y_ref, bound = oracle_of(A, x)
        out.append((A, x, y_ref, bound))
    return out


@pytest.mark.parametrize("prune", [1, 0])
@pytest.mark.parametrize("forced", [0, 1, 2, 3, 4, "tree"])
def test_auto_matches_oracle_and_three_call_path(cases, forced, prune):
    import torch
    tree = S.Tree(*REAL_TREE) if forced == "tree" else S.Tree.constant(forced)
    S.set_tuning("auto_prune", prune)
    try:
        for A, x, y_ref, bound in cases:
            announce(f"auto path tree={forced} prune={prune} {A.name} rows={A.rows} nnz={A.nnz}")
            dA = upload(A)
            xd = torch.from_numpy(x).cuda()
            ws = S.alloc_workspace(S.spmv_auto_workspace_bytes(A.rows, A.nnz))
            y, f, kid = run_auto(dA, tree, xd, A.rows, ws)
            want_f = O.features(A.rows, A.cols, A.row_ptr)
            if prune:
                decided = check_record(A, tree, f, kid, f"auto record {A.name}")
                assert decided == (forced != "tree" or len(O.reachable_classes(
                    O.known_features(A.rows, A.cols, A.nnz), *tree.arrays)) == 1)
            else:
                assert_features_equal(f, want_f, f"auto features {A.name}")
                assert kid == O.select(want_f["f"], *tree.arrays)
            assert_parity(y, y_ref, bound, f"auto (kernel {kid}) on {A.name}")
            y3 = run_spmv(kid, dA, xd, A.rows)
            assert y.tobytes() == y3.tobytes(), f"auto and seer_spmv({kid}) differ on {A.name}"
            # and the three-call path agrees on the features and the id
            f3 = S.seer_features(dA)
            assert f3.vector().tobytes() == want_f["f"].tobytes() and S.seer_select(f3, tree) == kid
    finally:
        S.set_tuning("auto_prune", -1)


def test_pruning_changes_nothing_but_the_launches(cases):
    """Trees that mix known and gathered features (so that some matrices leave one kernel, some
    a few, some all): with and without pruning the kernel id and y are the same bits, and the
    pruned call's record says "decided" exactly where the oracle's reachable set has one class."""
    import torch
    trees = [
        S.Tree(*REAL_TREE),
        # rows <= 5000 ? TM : (nnz <= 200000 ? (max_len <= 40 ? BM : WO) : (var_len <= 9 ? WM : MP))
        S.Tree([0, -1, 2, 4, 6, -1, -1, -1, -1], [5000.0, 0, 200000.0, 40.0, 9.0, 0, 0, 0, 0],
               [1, -1, 3, 5, 7, -1, -1, -1, -1], [2, -1, 4, 6, 8, -1, -1, -1, -1], [-1, 0, -1, -1, -1, 2, 4, 1, 3]),
        # mean_len <= 6 ? (empty_frac <= 0.1 ? TM : BM) : WM     -- never merge path / nonzero split
        S.Tree([3, 7, -1, -1, -1], [6.0, 0.1, 0, 0, 0], [1, 3, -1, -1, -1], [2, 4, -1, -1, -1], [-1, -1, 1, 0, 2]),
    ]
    decided_seen, undecided_seen = 0, 0
    for A, x, y_ref, bound in cases:
        dA, xd = upload(A), torch.from_numpy(x).cuda()
        ws = S.alloc_workspace(S.spmv_auto_workspace_bytes(A.rows, A.nnz))
        for ti, tree in enumerate(trees):
            announce(f"pruned against unpruned, tree #{ti}, {A.name} rows={A.rows} nnz={A.nnz}")
            y1, f1, k1 = run_auto(dA, tree, xd, A.rows, ws)
            decided = check_record(A, tree, f1, k1, f"tree #{ti} on {A.name}")
            S.set_tuning("auto_prune", 0)
            try:
                y0, f0, k0 = run_auto(dA, tree, xd, A.rows, ws)
            finally:
                S.set_tuning("auto_prune", -1)
            assert k0 == k1 and y0.tobytes() == y1.tobytes(), f"tree #{ti} on {A.name}: pruning changed the result"
            assert_parity(y1, y_ref, bound, f"pruned auto tree #{ti} (kernel {k1}) on {A.name}")
            decided_seen += decided
            undecided_seen += not decided
    assert decided_seen > 0 and undecided_seen > 0


def test_auto_with_trees_of_every_depth(cases):
    """Trees up to six comparisons deep are evaluated from a flattened copy, deeper ones by
    walking the node array: both must agree with the oracle's walk.  Chains of comparisons on
    nnz with leaves that cycle through the direct kernels, 1 to 9 levels deep, plus a full
    depth-6 tree over several features."""
    import torch
    rng = np.random.default_rng(17)
    trees = []
    for depth in range(1, 10):
        # node 2j: nnz <= t_j ? leaf (node 2j + 1) : node 2j + 2; the last node is a leaf
        feat, thr, left, right, kl = [], [], [], [], []
        for j in range(depth):
            feat += [2, -1]; thr += [float(10 ** (j * 0.9)), 0.0]
            left += [2 * j + 1, -1]; right += [2 * j + 2, -1]; kl += [-1, j % S.NUM_DIRECT_KERNELS]
        feat.append(-1); thr.append(0.0); left.append(-1); right.append(-1); kl.append(depth % S.NUM_DIRECT_KERNELS)
        trees.append(S.Tree(feat, thr, left, right, kl))
    # full binary tree, depth 6, heap order, random features and thresholds near typical values
    n_int, feat, thr, left, right, kl = 63, [], [], [], [], []
    for i in range(127):
        if i < n_int:
            f = int(rng.choice([0, 2, 3, 4, 5, 6, 7, 9, 11]))
            t = float({0: 3000, 2: 50000, 3: 6, 4: 40, 5: 1, 6: 30, 7: 0.2, 9: 0.01, 11: 1e-6}[f] * rng.uniform(0.3, 3))
            feat.append(f); thr.append(t); left.append(2 * i + 1); right.append(2 * i + 2); kl.append(-1)
        else:
            feat.append(-1); thr.append(0.0); left.append(-1); right.append(-1); kl.append(int(rng.integers(S.NUM_DIRECT_KERNELS)))
    trees.append(S.Tree(feat, thr, left, right, kl))
    seen = set()
    for A, x, y_ref, bound in cases:
        dA, xd = upload(A), torch.from_numpy(x).cuda()
        ws = S.alloc_workspace(S.spmv_auto_workspace_bytes(A.rows, A.nnz))
        want_f = O.features(A.rows, A.cols, A.row_ptr)["f"]
        for ti, tree in enumerate(trees):
            announce(f"auto path, tree #{ti} ({len(tree.arrays[0])} nodes), {A.name}")
            y, f, kid = run_auto(dA, tree, xd, A.rows, ws)
            assert kid == O.select(want_f, *tree.arrays), (ti, A.name)
            assert_parity(y, y_ref, bound, f"auto tree #{ti} (kernel {kid}) on {A.name}")
            seen.add((ti, kid))
    assert len({k for _, k in seen}) == S.NUM_DIRECT_KERNELS


def test_auto_misaligned_and_repeated(cases):
    import torch
    tree = S.Tree(*REAL_TREE)
    for A, x, y_ref, bound in cases:
        if A.nnz == 0:
            continue
        dA = upload(A, misalign=True)
        xd = torch.from_numpy(x).cuda()
        ws = S.alloc_workspace(S.spmv_auto_workspace_bytes(A.rows, A.nnz))
        announce(f"auto path misaligned {A.name}")
        for _ in range(3):   # the workspace is reused as it was left
            y, f, kid = run_auto(dA, tree, xd, A.rows, ws)
            assert_parity(y, y_ref, bound, f"auto misaligned on {A.name}")


def test_auto_in_a_hip_graph(cases):
    """The whole path captured once and replayed, with eager work between replays."""
    import torch
    tree = S.Tree(*REAL_TREE)
    picks = [c for c in cases if c[0].name.startswith(("zipf1.6_20011", "laplace5_100", "unif0-40"))]
    for A, x, y_ref, bound in picks:
        dA = upload(A)
        xd = torch.from_numpy(x).cuda()
        ws = S.alloc_workspace(S.spmv_auto_workspace_bytes(A.rows, A.nnz))
        y = torch.full((A.rows,), float("nan"), device="cuda:0")
        S.seer_spmv_auto(dA, tree, xd, y, ws)
        torch.cuda.synchronize()
        eager = y.clone()
        announce(f"auto path graph capture {A.name}")
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            S.seer_spmv_auto(dA, tree, xd, y, ws)
        for rep in range(4):
            y.fill_(float("nan"))                       # eager work between replays
            _ = S.seer_features(dA)                     # shares nothing with the graph but the device
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(y, eager), f"replay {rep} differs on {A.name}"
        assert_parity(y.cpu().numpy(), y_ref, bound, f"graph replay on {A.name}")


def test_auto_status_codes():
    import torch
    A = G.random_lengths(1000, 500, 0, 9, 3)
    dA = upload(A)
    xd = torch.zeros(500, device="cuda:0")
    y = torch.zeros(1000, device="cuda:0")
    ws = S.alloc_workspace(S.spmv_auto_workspace_bytes(A.rows, A.nnz))
    cyc = S.Tree([0, 0, -1], [1e30, 1e30, 0], [1, 0, -1], [2, 2, -1], [-1, -1, 0])
    with pytest.raises(S.SeerError) as ei:
        S.seer_spmv_auto(dA, cyc, xd, y, ws)
    assert ei.value.status == -3
    big = S.Tree([0] * 127 + [-1] * 128, [1.0] * 255, list(range(1, 128)) + [-1] * 128,
                 list(range(128, 255)) + [-1] * 128, [-1] * 127 + [0] * 128)
    with pytest.raises(S.SeerError) as ei:
        S.seer_spmv_auto(dA, big, xd, y, ws)
    assert ei.value.status == -3
    with pytest.raises(S.SeerError) as ei:
        S.seer_spmv_auto(dA, S.Tree.constant(2), xd, y, torch.empty(64, dtype=torch.uint8, device="cuda:0"))
    assert ei.value.status == -4
    with pytest.raises(S.SeerError) as ei:     # a kernel that needs preprocessing cannot be a leaf here
        S.seer_spmv_auto(dA, S.Tree.constant(S.CSR_A), xd, y, ws)
    assert ei.value.status == -3
    fresh = torch.zeros(4096, dtype=torch.uint8, device="cuda:0")
    with pytest.raises(S.SeerError):
        S.seer_spmv_auto_result(fresh)        # nothing has selected into this workspace


def test_auto_wide_integer_features(no_pruning):
    """rows * sum(len^2) beyond 2^64: the device's 128-bit variance numerator and its
    conversion to fp64 against exact Python integers (all values 1, x = 1, so y = len)."""
    import torch
    rows, long_rows, L = 20_000, 1_000, 1_000_000
    lens = np.zeros(rows, np.int64)
    lens[::20] = L
    assert int(lens.sum()) == long_rows * L < 2**31 and rows * int((lens**2).sum()) > 2**64
    rp = np.zeros(rows + 1, np.int64)
    rp[1:] = np.cumsum(lens)
    nnz = int(rp[-1])
    dA = S.DeviceCSR(rows, 64, torch.from_numpy(rp.astype(np.int32)).cuda(),
                     torch.zeros(nnz, dtype=torch.int32, device="cuda:0"),
                     torch.ones(nnz, dtype=torch.float32, device="cuda:0"), nnz)
    xd = torch.ones(64, device="cuda:0")
    ws = S.alloc_workspace(S.spmv_auto_workspace_bytes(rows, nnz))
    want = O.features(rows, 64, rp.astype(np.int32))
    for forced in (3, 4, 2, 1):
        announce(f"auto path wide integers, kernel {forced}, nnz={nnz}")
        y, f, kid = run_auto(dA, S.Tree.constant(forced), xd, rows, ws)
        assert kid == forced
        assert_features_equal(f, want, "wide-integer features (device)")
        assert np.array_equal(y, lens.astype(np.float32))
    assert_features_equal(S.seer_features(dA), want, "wide-integer features (host derivation)")


def test_auto_wm_when_its_tiles_outnumber_the_grid():
    """The combined kernel caps CSR,WM's share of the grid and lets its workgroups take
    several tiles: every row must still be written exactly once, and the result must be
    the stand-alone kernel's bit for bit.  Short rows (2 lanes per row, twice the
    thread-mapped tile count) and medium rows (8 lanes per row)."""
    import torch
    for A in (G.laplacian_5pt(1100), G.random_lengths(300_001, 300_001, 30, 50, 77)):
        x = G.dense_vector(A.cols, 5)
        y_ref, bound = oracle_of(A, x)
        dA = upload(A)
        xd = torch.from_numpy(x).cuda()
        ws = S.alloc_workspace(S.spmv_auto_workspace_bytes(A.rows, A.nnz))
        for forced in (S.CSR_WM, S.CSR_TM, S.CSR_WO):
            for prune in (0, 1):      # 0: the grid is sized for all five schedules; 1: for the forced one alone
                announce(f"auto path, capped CSR,WM share: kernel {forced} prune={prune} on {A.name} rows={A.rows} nnz={A.nnz}")
                S.set_tuning("auto_prune", prune)
                try:
                    y, f, kid = run_auto(dA, S.Tree.constant(forced), xd, A.rows, ws)
                finally:
                    S.set_tuning("auto_prune", -1)
                assert kid == forced
                assert_parity(y, y_ref, bound, f"auto kernel {forced} on {A.name}")
                assert np.array_equal(y, run_spmv(forced, dA, xd, A.rows))


def test_classifier_selection_path(cases):
    """seer_spmv_model: the selector runs on the host, the known model launches a kernel
    directly, the gathered model goes through the asynchronous path; path and kernel id
    must match the oracle's three-tree inference, y must match the oracle."""
    import torch
    # selector: nnz <= 100000 -> known model, else gather
    selector = S.Tree([2, -1, -1], [100000.0, 0, 0], [1, -1, -1], [2, -1, -1], [-1, 0, 1], n_classes=2)
    # known: mean_len <= 6 ? BM : WM
    known = S.Tree([3, -1, -1], [6.0, 0, 0], [1, -1, -1], [2, -1, -1], [-1, 2, 1])
    gathered = S.Tree(*REAL_TREE)
    model = S.Model(gathered, known, selector)
    paths = set()
    for A, x, y_ref, bound in cases:
        announce(f"model path {A.name}")
        dA = upload(A)
        xd = torch.from_numpy(x).cuda()
        ws = S.alloc_workspace(S.spmv_auto_workspace_bytes(A.rows, A.nnz))
        y = torch.full((max(A.rows, 1),), float("nan"), device="cuda:0")
        path, kid = S.seer_spmv_model(dA, model, xd, y, ws)
        if path == 1:
            _, kid = S.seer_spmv_auto_result(ws)
        torch.cuda.synchronize()
        fg = O.features(A.rows, A.cols, A.row_ptr)["f"]
        assert (path, kid) == O.model_select(A.rows, A.cols, A.nnz, fg, selector.arrays, known.arrays, gathered.arrays)
        assert_parity(y[:A.rows].cpu().numpy(), y_ref, bound, f"model path {path} kernel {kid} on {A.name}")
        paths.add(path)
    assert paths == {0, 1}
    # no selector: always gather
    A, x, y_ref, bound = cases[-1]
    dA, xd = upload(A), torch.from_numpy(x).cuda()
    ws = S.alloc_workspace(S.spmv_auto_workspace_bytes(A.rows, A.nnz))
    y = torch.empty(A.rows, device="cuda:0")
    assert S.seer_spmv_model(dA, S.Model(gathered), xd, y, ws)[0] == 1


def test_shipped_model_loads_and_runs(cases):
    import os
    import torch
    from paper_2403_17017_amd import training as T
    path = os.path.join(os.path.dirname(T.__file__), "selector_model.json")
    model, meta = T.load_model(path)
    for A, x, y_ref, bound in cases[12:]:
        dA, xd = upload(A), torch.from_numpy(x).cuda()
        ws = S.alloc_workspace(S.spmv_auto_workspace_bytes(A.rows, A.nnz))
        y = torch.full((A.rows,), float("nan"), device="cuda:0")
        p, kid = S.seer_spmv_model(dA, model, xd, y, ws)
        torch.cuda.synchronize()
        assert_parity(y.cpu().numpy(), y_ref, bound, f"shipped model on {A.name}")


def test_builtin_model_chooses_like_the_shipped_trees(cases):
    """model == NULL (the generated if/else code compiled into the library) against the same
    trees loaded from selector_model.json and passed as node arrays: same path, same kernel,
    same y, for single products and for planned ones."""
    import ctypes as C
    import os
    import torch
    from paper_2403_17017_amd import training as T
    path_json = os.path.join(os.path.dirname(T.__file__), "selector_model.json")
    model, _ = T.load_model(path_json)
    it_model, _ = T.load_model(path_json, iterative=True)
    L = S.lib()
    for A, x, y_ref, bound in cases:
        if A.rows == 0:
            continue
        announce(f"built-in model against the loaded trees, {A.name}")
        dA, xd = upload(A), torch.from_numpy(x).cuda()
        ws = S.alloc_workspace(S.spmv_auto_workspace_bytes(A.rows, A.nnz))
        y1 = torch.full((A.rows,), float("nan"), device="cuda:0")
        p1, k1 = S.seer_spmv_model(dA, model, xd, y1, ws)
        if p1 == 1:
            _, k1 = S.seer_spmv_auto_result(ws)
        y0 = torch.full((A.rows,), float("nan"), device="cuda:0")
        cs = dA.c_struct()
        p0, k0 = C.c_int(-1), C.c_int(-1)
        rc = L.seer_spmv_model(C.byref(cs), None, xd.data_ptr(), y0.data_ptr(), ws.data_ptr(), ws.numel(),
                               None if torch.cuda.current_stream().cuda_stream == 0 else C.c_void_p(torch.cuda.current_stream().cuda_stream),
                               C.byref(p0), C.byref(k0))
        assert rc == 0
        k0 = S.seer_spmv_auto_result(ws)[1] if p0.value == 1 else k0.value
        torch.cuda.synchronize()
        assert (p0.value, k0) == (p1, k1), A.name
        assert torch.equal(y0, y1)
        assert_parity(y0.cpu().numpy(), y_ref, bound, f"built-in model on {A.name}")
        for n in (1, 19, 100):
            plan1, pp1 = S.seer_spmv_plan(dA, it_model, n)
            plan_mem = S.alloc_workspace(plan1.plan_mem.numel() if plan1.plan_mem is not None else 256)
            fws = S.alloc_workspace(S.features_workspace_bytes(A.rows))
            c, pp0 = S.binding.seer_plan(), C.c_int(-1)
            rc = L.seer_spmv_plan(C.byref(cs), None, n, plan_mem.data_ptr(), plan_mem.numel(), fws.data_ptr(), fws.numel(),
                                  None, C.byref(c), C.byref(pp0))
            assert rc == 0 and (pp0.value, c.kernel_id) == (pp1, plan1.kernel_id), (A.name, n)


@pytest.mark.parametrize("rows", [1, 3, 4, 5, 255, 1023, 1024, 1025, 8191, 8192, 8193, 10_241, 32_771, 524_287, 2_097_152,
                                  2_097_155, 4_300_001])
def test_statistics_at_the_edges_of_the_reduction(rows):
    """Row counts around one workgroup's lanes, its loads in flight, the single launch, whole and
    ragged parts of the first pass; lengths whose squares need 64 bits and empty rows at both ends."""
    import torch
    rng = np.random.default_rng(rows)
    lens = rng.integers(0, 5, rows).astype(np.int64)
    lens[0] = 0
    lens[rows // 2] = 1_000_003
    lens[rows - 1] = 0 if rows > 2 else 77
    rp = np.zeros(rows + 1, np.int32)
    rp[1:] = np.cumsum(lens)
    announce(f"statistics of {rows} rows")
    want = O.features(rows, 2_000_000, rp)
    for shift in (0, 1):                                  # row_ptr on 16 bytes, and 4 bytes past that
        d = torch.zeros(rows + 1 + shift, dtype=torch.int32, device="cuda:0")
        d[shift:] = torch.from_numpy(rp).cuda()
        A = S.DeviceCSR(rows, 2_000_000, d[shift:], torch.zeros(1, dtype=torch.int32, device="cuda:0"),
                        torch.zeros(1, device="cuda:0"), 0)
        f = S.seer_features(A)
        for k in ("max_len", "min_len", "empty_rows", "sum_sq_len"):
            assert int(getattr(f, k)) == int(want[k]), k
        assert f.vector().tobytes() == want["f"].tobytes()


@pytest.mark.parametrize("rows,launches", [(200_003, 2), (262_144, 2), (262_145, 3), (500_003, 3)])
def test_where_the_wavefront_schedule_lets_the_selection_into_the_product(rows, launches):
    """CSR,BM or CSR,WM, selected on the device: a first pass and the product, up to as many rows as the first pass
    reads in one trip; with a selection launch between them beyond, where CSR,WM would loop for too long."""
    import ctypes

    import torch
    A = G.random_lengths(rows, rows, 0, 6, 61)
    dA, x = upload(A), G.dense_vector(A.cols, 3)
    xd, y = torch.from_numpy(x).cuda(), torch.empty(A.rows, device="cuda:0")
    ws = S.alloc_workspace(S.spmv_auto_workspace_bytes(A.rows, A.nnz))
    hip = ctypes.CDLL(next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line))
    y_ref, bound = oracle_of(A, x)
    for kids in ((1, 2), (2, 1)):
        tree = S.Tree([6, -1, -1], [50.0, 0, 0], [1, -1, -1], [2, -1, -1], [-1, *kids])
        announce(f"launches of a step rows={rows} tree={kids}")
        g = torch.cuda.CUDAGraph(keep_graph=True)
        with torch.cuda.graph(g):
            S.seer_spmv_auto(dA, tree, xd, y, ws)
        n = ctypes.c_size_t(0)
        assert hip.hipGraphGetNodes(ctypes.c_void_p(g.raw_cuda_graph()), None, ctypes.byref(n)) == 0
        assert n.value == launches
        g.instantiate()
        for _ in range(2):
            y.fill_(float("nan"))
            g.replay()
            torch.cuda.synchronize()
            assert_parity(y.cpu().numpy(), y_ref, bound, f"tree {kids}")
