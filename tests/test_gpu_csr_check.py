"""GPU parity of seer_csr_check with the oracle's count of contract violations
(bit-exact: integer work).  The check only reads the two index arrays, so a matrix
with planted defects is safe to hand to it (and to nothing else)."""
import numpy as np
import pytest

import paper_2403_17017_amd as S
from oracle import seer_oracle as O
from workloads import csr_gen as G

from gpu_util import announce

pytestmark = pytest.mark.gpu


def device_counts(rows, cols, nnz, rp, ci):
    import torch
    d = S.DeviceCSR(rows, cols, torch.from_numpy(rp).cuda(),
                    torch.from_numpy(ci).cuda() if ci.size else torch.zeros(1, dtype=torch.int32, device="cuda:0"),
                    torch.zeros(max(nnz, 1), device="cuda:0"), nnz)
    return S.seer_csr_check(d)


def test_well_formed_matrices_pass():
    for A in (G.laplacian_5pt(300), G.fixed_degree(), G.random_lengths(200_001, 5000, 0, 40, seed=2),
              G.explicit_lengths([0, 0, 0, 100_000, 0, 1], 777, seed=4), G.explicit_lengths([0] * 5000, 10, seed=1)):
        announce(f"csr check, well formed: {A.name} rows={A.rows} nnz={A.nnz}")
        assert device_counts(A.rows, A.cols, A.nnz, A.row_ptr, A.col_idx) == (0, 0)


def test_small_defects_match_the_oracle():
    i32 = lambda *v: np.array(v, dtype=np.int32)
    ci = i32(0, 1, 2, 3)
    for rows, cols, nnz, rp, c in (
            (2, 4, 4, i32(1, 2, 4), ci), (2, 4, 4, i32(0, 2, 3), ci), (2, 4, 4, i32(0, 5, 4), ci),
            (3, 4, 4, i32(2, 1, 0, 3), ci), (2, 4, 4, i32(0, -1, 4), ci),
            (2, 4, 4, i32(0, 2, 4), i32(-1, 4, 2, 9)), (2, 0, 4, i32(0, 2, 4), ci), (0, 5, 0, i32(0), i32())):
        announce(f"csr check, small case rows={rows} rp={rp.tolist()} ci={c.tolist()}")
        want = O.csr_defects(rows, cols, nnz, rp, c)
        assert device_counts(rows, cols, nnz, rp, c) == want


def test_planted_defects_in_a_large_matrix_match_the_oracle():
    """Several grid-stride trips per lane, defects spread over many waves."""
    A = G.random_lengths(1_300_003, 40_000, 0, 9, seed=21)
    rng = np.random.default_rng(8)
    ci = A.col_idx.copy()
    where = rng.choice(A.nnz, 5000, replace=False)
    ci[where[:3000]] = A.cols + rng.integers(0, 2**20, 3000)
    ci[where[3000:]] = -1 - rng.integers(0, 2**20, 2000)
    rp = A.row_ptr.copy()
    hit = rng.choice(A.rows - 2, 700, replace=False) + 1
    rp[hit] = rp[hit + 1] + rng.integers(1, 50, 700).astype(np.int32)     # offsets pushed past their successors
    rp[0] = 3
    announce(f"csr check, planted defects rows={A.rows} nnz={A.nnz}")
    want = O.csr_defects(A.rows, A.cols, A.nnz, rp, ci)
    assert want[1] == 5000 and want[0] >= 700
    assert device_counts(A.rows, A.cols, A.nnz, rp, ci) == want
    # the same workspace again, now on the intact matrix: the counters start from zero
    import torch
    ws = S.alloc_workspace(16)
    vals = torch.zeros(A.nnz, device="cuda:0")
    d_bad = S.DeviceCSR(A.rows, A.cols, torch.from_numpy(rp).cuda(), torch.from_numpy(ci).cuda(), vals, A.nnz)
    d_ok = S.DeviceCSR(A.rows, A.cols, torch.from_numpy(A.row_ptr).cuda(), torch.from_numpy(A.col_idx).cuda(), vals, A.nnz)
    assert S.seer_csr_check(d_bad, ws) == want
    assert S.seer_csr_check(d_ok, ws) == (0, 0)


def test_status_codes():
    import torch
    A = G.laplacian_5pt(20)
    d = S.DeviceCSR.from_host(A)
    small = torch.zeros(8, dtype=torch.uint8, device="cuda:0")
    with pytest.raises(S.SeerError) as ei:
        S.seer_csr_check(d, small)
    assert ei.value.status == -4


@pytest.mark.parametrize("rows,nnz", [(1, 1), (2, 3), (3, 4), (4, 5), (5, 2), (1023, 4099), (4096, 16384), (70_001, 131_075)])
@pytest.mark.parametrize("shift", [0, 1])
def test_every_position_counts_whatever_the_alignment(rows, nnz, shift):
    """The first and the last few offsets and columns, in arrays that start on 16 bytes and 4
    bytes past that (the kernel reads four of them at a time)."""
    import torch
    rng = np.random.default_rng(rows + nnz)
    rp = np.zeros(rows + 1, np.int32)
    rp[1:] = np.sort(rng.integers(0, nnz + 1, rows))
    rp[-1] = nnz
    ci = rng.integers(0, 50, nnz).astype(np.int32)

    def counts(p, c):
        dp, dc = torch.zeros(rows + 1 + shift, dtype=torch.int32, device="cuda:0"), \
            torch.zeros(nnz + shift, dtype=torch.int32, device="cuda:0")
        dp[shift:] = torch.from_numpy(p).cuda()
        dc[shift:] = torch.from_numpy(c).cuda()
        return S.seer_csr_check(S.DeviceCSR(rows, 50, dp[shift:], dc[shift:], torch.zeros(nnz, device="cuda:0"), nnz))
    announce(f"csr check at every position rows={rows} nnz={nnz} shift={shift}")
    assert counts(rp, ci) == O.csr_defects(rows, 50, nnz, rp, ci)
    for k in sorted({k for k in (0, 1, 2, 3, 4, nnz // 2, nnz - 4, nnz - 3, nnz - 2, nnz - 1) if 0 <= k < nnz}):
        bad = ci.copy()
        bad[k] = 50 if k % 2 else -1
        assert counts(rp, bad) == O.csr_defects(rows, 50, nnz, rp, bad), f"column {k}"
    for i in sorted({i for i in (0, 1, 2, 3, 4, 5, rows // 2, rows - 3, rows - 2, rows - 1, rows) if 0 <= i <= rows}):
        bad = rp.copy()
        bad[i] += nnz + 1
        assert counts(bad, ci) == O.csr_defects(rows, 50, nnz, bad, ci), f"offset {i}"


@pytest.mark.parametrize("first", ["check", "features"])
def test_a_call_behind_long_work_holds_up_no_other_thread(first):
    """One thread's call waits for its own stream, which is busy; the others' streams are not."""
    import threading

    import torch
    A = G.random_lengths(2_003, 5_000, 0, 20, 7)
    dA = S.DeviceCSR.from_host(A)
    S.seer_features(dA)
    assert S.seer_csr_check(dA) == (0, 0)                             # code loaded, mailboxes allocated
    streams = [torch.cuda.Stream() for _ in range(5)]
    left = torch.cuda.Event()
    done, results = [], []
    torch.cuda.synchronize()

    def call(k):
        ws = S.alloc_workspace(max(256, S.features_workspace_bytes(A.rows)))
        if k == 0 and first == "features":
            results.append((0, 0) if int(S.seer_features(dA, ws, streams[0]).nnz) == A.nnz else None)
        else:
            results.append(S.seer_csr_check(dA, ws, streams[k]))
        done.append((k, left.query()))                                # was the busy stream through by then?
    with torch.cuda.stream(streams[0]):
        torch.cuda._sleep(1_500_000_000)                              # 0.6 s and more of the GPU's clock
        left.record()
    announce(f"one {first} behind a busy stream, csr checks on four others")
    threads = [threading.Thread(target=call, args=(k,)) for k in range(5)]
    threads[0].start()
    threads[0].join(0.05)
    for t in threads[1:]:
        t.start()
    for t in threads:
        t.join(60)
    assert results == [(0, 0)] * 5
    # (a few streams share a hardware queue, so not necessarily all of them)
    assert any(k != 0 and not through for k, through in done), "every call waited for the busy stream"


def test_counters_start_from_zero_after_a_bad_matrix():
    """Alternating good and bad matrices, each call gets its own counts, on one stream and on two."""
    import torch
    A = G.random_lengths(5_003, 3_000, 0, 40, 21)
    ci = A.col_idx.copy()
    ci[[3, 700, 701, ci.size - 1]] = A.cols
    bad = S.DeviceCSR.from_host(G.HostCSR(A.rows, A.cols, A.row_ptr, ci, A.values, "four-outside"))
    good = S.DeviceCSR.from_host(A)
    announce("seer_csr_check, good and bad in turn")
    other = torch.cuda.Stream()
    torch.cuda.synchronize()
    for k in range(12):
        stream = other if k % 3 == 2 else None
        assert tuple(S.seer_csr_check(bad, stream=stream)) == (0, 4)
        assert tuple(S.seer_csr_check(good, stream=stream)) == (0, 0)


def test_calls_share_nothing_but_what_they_are_handed():
    """Two threads with a stream and a workspace each, one matrix bad and one good: each gets its own counts.
    What a call adds up lies in the caller's workspace, whatever that holds on entry."""
    import threading

    import torch
    A = G.random_lengths(5_003, 3_000, 0, 40, 21)
    ci, rp = A.col_idx.copy(), A.row_ptr.copy()
    ci[[3, 700, 701, ci.size - 1]] = A.cols
    rp[0] = 1
    bad = S.DeviceCSR.from_host(G.HostCSR(A.rows, A.cols, rp, ci, A.values, "offset-and-four-outside"))
    good = S.DeviceCSR.from_host(A)
    want = O.csr_defects(A.rows, A.cols, A.nnz, rp, ci)
    assert want[0] > 0 and want[1] == 4
    announce("seer_csr_check, good and bad on two threads")
    poison = torch.full((4,), 0x5A5A5A5A, dtype=torch.int32, device="cuda:0").view(torch.uint8)
    ws = poison.clone()
    assert tuple(S.seer_csr_check(bad, ws)) == want
    assert not torch.equal(ws, poison)
    results = {}

    def calls(name, matrix):
        stream = torch.cuda.Stream()
        results[name] = {tuple(S.seer_csr_check(matrix, poison.clone(), stream)) for _ in range(200)}
    torch.cuda.synchronize()
    threads = [threading.Thread(target=calls, args=a) for a in (("bad", bad), ("good", good))]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
    assert results == {"bad": {want}, "good": {(0, 0)}}


@pytest.mark.parametrize("call", ["check", "features", "prepare CSR,S", "prepare ELL,TM"])
def test_a_call_that_fails_leaves_no_kernel_behind(call):
    """An error that another library left in the thread is reported behind the launches.  Such a call ends when its
    kernels have: they write into a result mailbox that is another call's next."""
    import ctypes

    import torch
    hip = ctypes.CDLL(next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line))
    A = G.random_lengths(300_007, 1_300_000, 20, 50, 77) if call != "prepare ELL,TM" else G.banded(699_968, 1, 5)
    dA = S.DeviceCSR.from_host(A)
    good = S.DeviceCSR.from_host(G.random_lengths(2_003, 5_000, 0, 20, 7))
    busy, other = torch.cuda.Stream(), torch.cuda.Stream()
    ws = S.alloc_workspace(max(S.features_workspace_bytes(A.rows), 256))
    mem = S.alloc_workspace(1 << 30) if call.startswith("prepare") else None
    run = {"check": lambda: S.seer_csr_check(dA, ws, busy), "features": lambda: S.seer_features(dA, ws, busy),
           "prepare CSR,S": lambda: S.seer_spmv_prepare(S.CSR_S, dA, plan_mem=mem, stream=busy),
           "prepare ELL,TM": lambda: S.seer_spmv_prepare(S.ELL_TM, dA, plan_mem=mem, stream=busy)}[call]
    run()
    assert tuple(S.seer_csr_check(good, ws, other)) == (0, 0)
    torch.cuda.synchronize()
    announce(f"{call} with an error left in the thread")
    with torch.cuda.stream(busy):
        torch.cuda._sleep(20_000_000)                                          # 8 ms and more of the GPU's clock
    assert hip.hipSetDevice(12345) != 0                                        # refused; remembered by the runtime
    with pytest.raises(S.SeerError) as ei:
        run()
    assert ei.value.status == -5
    assert busy.query(), "the call's kernels were still to run"
    for _ in range(20):
        assert tuple(S.seer_csr_check(good, ws, other)) == (0, 0)
    run()
    torch.cuda.synchronize()
