"""Rows that the tiles of CSR,MP and CSR,WO cut: their parts meet inside the product, in the workspace.  Small whole
numbers throughout, so every sum is exact in any order and a part that is lost, doubled or left over from an earlier
product shows as a wrong number."""
import numpy as np
import pytest

import paper_2403_17017_amd as S

from gpu_util import announce

pytestmark = pytest.mark.gpu

CHUNK, MP_TILE = 2048, 1792
COLS = 997


def lengths():
    rng = np.random.default_rng(4)
    out = {
        "1x1": [1], "no nonzeros": [0, 0, 0], "one chunk": [CHUNK], "one more": [CHUNK + 1], "one less": [CHUNK - 1],
        "row ends at the boundary": [7, CHUNK - 7, 5], "row begins at the boundary, empty rows there": [CHUNK, 0, 0, 3, 0],
        "two tiles of merge path": [MP_TILE - 2, 1, 9], "row end alone in its tile": [MP_TILE, 4],
        "one row": [100_003], "one row of 64 chunks": [64 * CHUNK], "one row among empty ones": [0] * 5000 + [300_000] + [0] * 5000,
        "rows over several tiles": list(rng.integers(2000, 9000, 60)), "rows of 14": [14] * 5000,
        "mixed": list(rng.choice([0, 1, 3, 50, 3000, 9000], 300)), "short": list(rng.integers(0, 40, 20_011)),
        "the last that meet": [8388, 0, 3] * 999 + [2**23 - 1 - 8391 * 999], "the first that do not": [8388, 0, 3] * 999 + [2**23 - 8391 * 999],
    }
    return {k: np.asarray(v, dtype=np.int64) for k, v in out.items()}


def matrix(lens, seed):
    import torch
    rng = np.random.default_rng(seed)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ci = rng.integers(0, COLS, rp[-1]).astype(np.int32)
    va = rng.integers(-3, 4, rp[-1]).astype(np.float32)
    A = S.DeviceCSR(len(lens), COLS, torch.from_numpy(rp).cuda(), torch.from_numpy(ci).cuda(), torch.from_numpy(va).cuda(), int(rp[-1]))
    return A, rp, ci, va


def product(rp, ci, va, x):
    total = np.concatenate([[0.0], np.cumsum(va.astype(np.float64) * x[ci])])
    return (total[rp[1:]] - total[rp[:-1]]).astype(np.float32)


def carries_bytes(tiles):
    return 2 * (-(-4 * tiles // 256) * 256)


@pytest.mark.parametrize("kid", [S.CSR_WO, S.CSR_MP])
@pytest.mark.parametrize("call", ["direct", "auto", "gathered", "carries"])
def test_cut_rows_on_one_workspace(kid, call):
    """All matrices one after the other on one workspace that held anything before, each with three x."""
    import torch
    ws = torch.randint(0, 256, (4 << 20,), dtype=torch.uint8, device="cuda:0")
    other = S.CSR_MP if kid == S.CSR_WO else S.CSR_WO
    tree = S.Tree.constant(kid) if call == "auto" else S.Tree([4, -1, -1], [-1.0, 0, 0], [1, -1, -1], [2, -1, -1], [-1, other, kid])
    for name, lens in lengths().items():
        A, rp, ci, va = matrix(lens, len(name))
        announce(f"cut rows, kernel {kid}, {call}: {name}, rows={A.rows} nnz={A.nnz}")
        least = carries_bytes(max(1, -(-A.nnz // (CHUNK if A.nnz < 2**23 else 2 * CHUNK)) if kid == S.CSR_WO
                                  else -(-(A.rows + A.nnz) // MP_TILE)))
        for k in range(3):
            x = np.random.default_rng(k).integers(-3, 4, COLS).astype(np.float32)
            xd = torch.from_numpy(x).cuda()
            y = torch.full((A.rows,), float("nan"), device="cuda:0")
            if call in ("auto", "gathered"):
                S.seer_spmv_auto(A, tree, xd, y, ws)
                assert S.seer_spmv_auto_result(ws)[1] == kid
            else:
                S.seer_spmv(kid, A, xd, y, workspace=ws[:least] if call == "carries" else ws)
            assert np.array_equal(y.cpu().numpy(), product(rp, ci, va, x)), (name, k)


@pytest.mark.parametrize("kid", [S.CSR_WO, S.CSR_MP])
def test_cut_rows_in_a_graph(kid):
    """Products of two matrices share one workspace in one graph; values change between the replays."""
    import torch
    names = lengths()
    pair = [matrix(names["rows over several tiles"], 1), matrix(names["one row"], 2)]
    ws = torch.randint(0, 256, (1 << 20,), dtype=torch.uint8, device="cuda:0")
    x = torch.ones(COLS, device="cuda:0")
    ys = [torch.empty(A.rows, device="cuda:0") for A, *_ in pair]
    announce(f"cut rows in a graph, kernel {kid}")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for (A, *_), y in zip(pair, ys):
            S.seer_spmv(kid, A, x, y, workspace=ws)
    for rep in range(4):
        vals = [np.random.default_rng(10 * rep + k).integers(-3, 4, A.nnz).astype(np.float32) for k, (A, *_) in enumerate(pair)]
        for (A, *_), v, y in zip(pair, vals, ys):
            A.values.copy_(torch.from_numpy(v))
            y.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        for (A, rp, ci, _), v, y in zip(pair, vals, ys):
            assert np.array_equal(y.cpu().numpy(), product(rp, ci, v, np.ones(COLS, dtype=np.float32)))


@pytest.mark.parametrize("kid", [S.CSR_WO, S.CSR_MP])
def test_cut_rows_same_bits_on_every_run(kid):
    """The order in which workgroups come to a meeting does not show in y."""
    import torch
    lens = lengths()["rows over several tiles"]
    A, *_ = matrix(lens, 3)
    A.values.copy_(torch.rand(A.nnz, device="cuda:0"))
    x = torch.rand(COLS, device="cuda:0")
    ws = S.alloc_workspace(S.spmv_workspace_bytes(kid, A.rows, A.nnz))
    announce(f"cut rows, the same bits, kernel {kid}")
    runs = torch.empty(40, A.rows, device="cuda:0")
    for y in runs:
        S.seer_spmv(kid, A, x, y, workspace=ws)
    assert torch.equal(runs, runs[:1].expand_as(runs))


@pytest.mark.parametrize("kid", [S.CSR_WO, S.CSR_MP])
@pytest.mark.parametrize("call", ["direct", "auto"])
def test_marks_are_the_calls_own(kid, call):
    """What one call leaves in the slots is never taken for another call's: the second words show its proof."""
    import torch
    A, rp, ci, va = matrix(lengths()["one row"], 5)
    x = torch.ones(COLS, device="cuda:0")
    y = torch.empty(A.rows, device="cuda:0")
    ws = torch.zeros(1 << 20, dtype=torch.uint8, device="cuda:0")
    announce(f"marks of each call, kernel {kid}, {call}")
    slots = 0 if call == "direct" else 33024                 # (behind the partials and the record)
    seen = set()
    for k in range(4):
        if call == "auto":
            S.seer_spmv_auto(A, S.Tree.constant(kid), x, y, ws)
        else:
            S.seer_spmv(kid, A, x, y, workspace=ws)
        words = ws[slots:slots + 64 * 16].cpu().numpy().view(np.uint64).reshape(16, 8)
        assert not words[:, 0].any()                         # at rest
        proofs = set((words[:, 1] >> np.uint64(32)).tolist())
        assert len(proofs) == 1 and not proofs & seen, (k, proofs, seen)
        seen |= proofs
        assert np.array_equal(y.cpu().numpy(), product(rp, ci, va, np.ones(COLS, dtype=np.float32)))


@pytest.mark.parametrize("kid", [S.CSR_WO, S.CSR_MP])
def test_less_workspace_gives_the_bits_of_the_direct_product_with_less(kid):
    """Both calls take a workspace with room for carries alone, and add cut rows up in the same order then."""
    import torch
    A, *_ = matrix(lengths()["rows over several tiles"], 6)
    A.values.copy_(torch.rand(A.nnz, device="cuda:0"))
    x = torch.rand(COLS, device="cuda:0")
    announce(f"cut rows, little workspace, kernel {kid}")

    def run(auto, ws):
        y = torch.full((A.rows,), float("nan"), device="cuda:0")
        if auto:
            S.seer_spmv_auto(A, S.Tree.constant(kid), x, y, ws)
        else:
            S.seer_spmv(kid, A, x, y, workspace=ws)
        return y

    carries = carries_bytes(max(-(-A.nnz // CHUNK), -(-(A.rows + A.nnz) // MP_TILE)))
    few, much = (torch.zeros(n, dtype=torch.uint8, device="cuda:0") for n in (33024 + carries, 4 << 20))
    assert few.numel() < S.spmv_auto_workspace_bytes(A.rows, A.nnz)
    assert torch.equal(run(True, few), run(False, few[:carries]))
    assert torch.equal(run(True, much), run(False, much))
    with pytest.raises(S.SeerError):
        run(True, few[:-256])
