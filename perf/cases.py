"""The work that a program built on this library has it do, as measurable cases.

A case is a matrix (a family of synthetic CSR matrices, its sizes) and an operation on it
(`op`), always through the package's public entry points:

  step      seer_spmv_auto: gather the features, walk the tree, run the chosen schedule -- a
            matrix that is multiplied once
  steps     the same, `n` right-hand sides one after the other, captured in one HIP graph as a
            launch-bound program does (the entry point is documented as capturable)
  model     seer_spmv_model: classifier selection with the shipped trees, one product
  spmv      seer_spmv with a schedule the program has settled on
  repeat    seer_spmv_prepared from a plan the program keeps (seer_spmv_plan for 100 products):
            one of the many products of an iterative solver
  solve     seer_spmv_plan for `n` products, then the n products: selection, preprocessing and
            repetition together
  admit     seer_csr_check and seer_features on a matrix that has just come in

Matrices are drawn on the GPU from the seed: structure, values and vectors all depend on it,
except for the grid stencils, whose structure and values are fixed by the grid.
"""
import math
import os

import numpy as np
import torch

import paper_2403_17017_amd as S
from paper_2403_17017_amd.training import load_model

_MODEL = os.path.join(os.path.dirname(os.path.abspath(S.__file__)), "selector_model.json")
_DEVICE = "cuda:0"


def listed():
    return [
        # the smallest matrix anyone benchmarks here: 4096 rows of 16, all latency and launches
        {"name": "step_fixed16_4096", "op": "step", "family": "fixed", "rows": 4096, "cols": 4096, "k": 16},
        # a batch of right-hand sides on a small ragged matrix: launch-bound, hence captured
        {"name": "steps_uniform_20011", "op": "steps", "n": 16, "family": "uniform", "rows": 20011, "cols": 20011,
         "lo": 2, "hi": 37},
        # the framework's headline workload: a 5-point Laplacian of a million rows, one product
        {"name": "step_laplace_1024", "op": "step", "family": "stencil", "grid": 1024, "dim": 2},
        # power-law rows (graphs): two million rows, rows of up to 200 000 entries
        {"name": "step_zipf1.85_2M", "op": "step", "family": "zipf", "rows": 2000000, "cols": 2000000, "s": 1.85},
        # the same with a heavier tail, 4.8e8 nonzeros: the largest matrix of the benchmark
        {"name": "step_zipf1.6_2M", "op": "step", "family": "zipf", "rows": 2000000, "cols": 2000000, "s": 1.6},
        # rectangular, eight million very short rows, three in ten empty: classifier selection
        {"name": "model_empty_8M", "op": "model", "family": "empty", "rows": 8000000, "cols": 1000000, "lam": 4.0},
        # a wide band (a discretised operator of higher order): the program knows its schedule
        {"name": "spmv_band_1M", "op": "spmv", "kernel": S.CSR_WO, "family": "banded", "rows": 1000003, "half": 30},
        # iterations on a power-law matrix of four million rows: one product from the plan that the
        # library chose (the column-slabbed copy)
        {"name": "repeat_zipf1.9_4M", "op": "repeat", "family": "zipf", "rows": 4000000, "cols": 4000000, "s": 1.9},
        # iterations on a large stencil: one product from the plan that the library chose
        {"name": "repeat_laplace_4096", "op": "repeat", "family": "stencil", "grid": 4096, "dim": 2},
        # a whole short solve on a large matrix of scattered columns, preprocessing included (19
        # products: the count at which the paper shows preprocessing amortised)
        {"name": "solve_uniform_2M", "op": "solve", "n": 19, "family": "uniform", "rows": 2000003, "cols": 2000003,
         "lo": 0, "hi": 40},
        # a short solve on a mid-sized 3-D grid of odd size
        {"name": "solve_laplace3d_71", "op": "solve", "n": 19, "family": "stencil", "grid": 71, "dim": 3},
        # a matrix arrives: input check, then its statistics
        {"name": "admit_poisson_3M", "op": "admit", "family": "poisson", "rows": 3000001, "cols": 3000001, "lam": 9.0},
    ]


_OPS = ("step", "steps", "model", "spmv", "repeat", "solve", "admit")
_FAMILIES = ("fixed", "uniform", "banded", "poisson", "zipf", "stencil", "empty")
_MOST_NNZ = 60_000_000


def draw(rng):
    """Rows from a thousand to eight million, mean row lengths from one to about two hundred,
    every family and operation; schedules named directly are ones that suit the family."""
    while True:
        op = rng.choice(_OPS)
        fam = rng.choice(_FAMILIES)
        if op == "admit" and fam in ("fixed", "banded", "stencil"):
            continue                                    # nothing in their statistics depends on the seed
        rows = int(round(10 ** rng.uniform(3.0, 6.9)))
        c = {"op": op, "family": fam}
        if op == "steps":
            rows = int(round(10 ** rng.uniform(3.0, 4.8)))
            c["n"] = rng.randint(4, 24)
        if op == "solve":
            c["n"] = rng.choice((3, 5, 8, 12, 19, 30))
        if fam == "stencil":
            c["dim"] = rng.randint(2, 3)
            c["grid"] = max(8, int(round(rows ** (1.0 / c["dim"]))))
        else:
            c["rows"] = rows
            if fam != "banded":
                c["cols"] = rows if rng.random() < 0.7 else int(round(10 ** rng.uniform(3.0, 6.9)))
            if fam == "fixed":
                c["k"] = rng.randint(1, 64)
            elif fam == "uniform":
                c["lo"] = rng.randint(0, 4)
                c["hi"] = c["lo"] + int(round(10 ** rng.uniform(0.0, 2.5)))
            elif fam == "banded":
                c["half"] = int(round(10 ** rng.uniform(0.0, 2.0)))
            elif fam == "zipf":
                c["s"] = round(rng.uniform(1.6, 2.5), 3)
            else:
                c["lam"] = round(10 ** rng.uniform(0.0, 1.8), 2)
        rows, _, nnz = _sizes(c)
        if nnz > _MOST_NNZ or (op == "solve" and nnz * c["n"] > 4e8):
            continue
        if op == "spmv":
            balanced = [S.CSR_MP, S.CSR_WO, S.CSR_A, S.COO_WM]
            if fam not in ("zipf",):
                balanced += [S.CSR_WM, S.CSR_BM]
            if fam == "stencil" or nnz <= 8 * rows and fam in ("fixed", "banded", "empty", "poisson"):
                balanced.append(S.CSR_TM)
            c["kernel"] = rng.choice(balanced)
        return c


# ------------------------------------------------------------------ the matrices
def _lengths(case, gen):
    fam, rows = case["family"], case["rows"]

    def uniform01(n):
        return torch.rand(n, generator=gen, device=_DEVICE, dtype=torch.float64)
    if fam == "fixed":
        return torch.full((rows,), min(case["k"], case["cols"]), device=_DEVICE, dtype=torch.int64)
    if fam == "uniform":
        return torch.randint(case["lo"], case["hi"] + 1, (rows,), generator=gen, device=_DEVICE).clamp(max=case["cols"])
    if fam == "poisson":
        lam = torch.full((rows,), case["lam"], device=_DEVICE, dtype=torch.float32)
        return torch.poisson(lam, generator=gen).to(torch.int64).clamp(max=case["cols"])
    if fam == "zipf":          # min(Zipf(s), 200 000) by its distribution function
        cap = min(200_000, case["cols"])
        p = torch.arange(1, cap + 1, device=_DEVICE, dtype=torch.float64) ** -case["s"]
        tail = cap ** (1.0 - case["s"]) / (case["s"] - 1.0)           # what lies beyond the cap, close enough
        cdf = torch.cumsum(p, 0) / (p.sum() + tail)
        return (torch.searchsorted(cdf, uniform01(rows)) + 1).clamp(max=cap)
    # empty: three rows in ten empty, the others Poisson of at least one
    lam = case["lam"]
    k = torch.arange(0, int(lam + 12 * math.sqrt(lam) + 20), device=_DEVICE, dtype=torch.float64)
    pmf = torch.exp(k * math.log(lam) - lam - torch.lgamma(k + 1))
    cdf = torch.cumsum(pmf, 0)
    u = math.exp(-lam) + uniform01(rows) * (1.0 - math.exp(-lam)) * (1 - 1e-12)
    lens = torch.searchsorted(cdf, u).clamp(min=1, max=case["cols"])
    lens[uniform01(rows) < 0.3] = 0
    return lens


def _matrix(case, gen):
    """(rows, cols, row_ptr, col_idx, values): columns ascending inside a row."""
    fam = case["family"]
    if fam == "stencil":
        n, dim = case["grid"], case["dim"]
        rows = cols = n ** dim
        i = torch.arange(rows, device=_DEVICE, dtype=torch.int64)
        coord = [(i // n ** d) % n for d in range(dim)]
        mask = torch.stack([coord[d] > 0 for d in reversed(range(dim))] + [torch.ones_like(i, dtype=torch.bool)]
                           + [coord[d] < n - 1 for d in range(dim)], dim=1)
        offs = torch.tensor([-n ** d for d in reversed(range(dim))] + [0] + [n ** d for d in range(dim)],
                            device=_DEVICE, dtype=torch.int64)
        ci = (i[:, None] + offs[None, :])[mask].to(torch.int32)
        va = torch.where(offs == 0, 2.0 * dim, -1.0).to(torch.float32).expand(rows, -1)[mask].contiguous()
        lens = mask.sum(1)
    else:
        if fam == "banded":
            rows = cols = case["rows"]
            i = torch.arange(rows, device=_DEVICE, dtype=torch.int64)
            first = (i - case["half"]).clamp(min=0)
            lens = (i + case["half"]).clamp(max=rows - 1) - first + 1
        else:
            rows, cols = case["rows"], case["cols"]
            lens = _lengths(case, gen)
        nnz = int(lens.sum())
        row_id = torch.repeat_interleave(torch.arange(rows, device=_DEVICE, dtype=torch.int64), lens, output_size=nnz)
        if fam == "banded":
            start = torch.cumsum(lens, 0) - lens
            ci = (torch.arange(nnz, device=_DEVICE, dtype=torch.int64) - (start - first)[row_id]).to(torch.int32)
        else:
            key = row_id * cols + torch.randint(0, cols, (nnz,), generator=gen, device=_DEVICE)
            key, _ = torch.sort(key)
            ci = (key - row_id * cols).to(torch.int32)
            del key
        del row_id
        va = torch.rand(nnz, generator=gen, device=_DEVICE, dtype=torch.float32) * 2 - 1
    rp = torch.zeros(rows + 1, device=_DEVICE, dtype=torch.int32)
    rp[1:] = torch.cumsum(lens, 0)
    return rows, cols, rp, ci.contiguous(), va


def _inputs(case, seed):
    gen = torch.Generator(device=_DEVICE)
    gen.manual_seed(int(seed) * 2654435761 % (1 << 31) + 17)
    A = S.DeviceCSR(*_matrix(case, gen))
    xs = [torch.rand(A.cols, generator=gen, device=_DEVICE, dtype=torch.float32) * 2 - 1 for _ in range(case.get("n", 1))]
    return A, xs


_models = {}


def _model(iterative):
    if iterative not in _models:
        _models[iterative] = load_model(_MODEL, iterative=iterative)[0]
    return _models[iterative]


# ------------------------------------------------------------------ the cases
def prepare(case, seed):
    A, xs = _inputs(case, seed)
    st = {"case": case, "op": case["op"], "A": A, "xs": xs}
    op = case["op"]
    if op != "admit":
        ys = torch.empty(len(xs), A.rows, device=_DEVICE, dtype=torch.float32)
        st["out"], st["ys"] = ys, list(ys.unbind(0))
    if op in ("step", "steps", "model"):
        st["model"] = _model(False)
        st["ws"] = S.alloc_workspace(S.spmv_auto_workspace_bytes(A.rows, A.nnz))
    elif op == "spmv":
        st["ws"] = S.alloc_workspace(S.spmv_workspace_bytes(case["kernel"], A.rows, A.nnz))
    elif op == "repeat":
        st["plan"], _ = S.seer_spmv_plan(A, _model(True), 100)
        st["ws"] = S.alloc_workspace(S.spmv_prepared_workspace_bytes(st["plan"]))
    elif op == "solve":
        st["model"] = _model(True)
        st["feature_ws"] = S.alloc_workspace(S.features_workspace_bytes(A.rows))
        # one block that holds whatever plan the library chooses, and the products' scratch
        st["plan_mem"] = S.alloc_workspace(max(S.plan_bytes(S.CSR_A, A.rows, A.nnz), S.plan_bytes(S.COO_WM, A.rows, A.nnz),
                                               12 * A.nnz + (1 << 20), S.slab_plan_bytes(A.rows, A.cols, A.nnz)))
        st["ws"] = S.alloc_workspace(4 * A.nnz + (1 << 20) + 2 * max(S.spmv_workspace_bytes(k, A.rows, A.nnz)
                                                                     for k in S.ONE_CALL_KERNELS))
    elif op == "admit":
        st["ws"] = S.alloc_workspace(max(16, S.features_workspace_bytes(A.rows)))
    if op == "steps":
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _steps(st)
        torch.cuda.current_stream().wait_stream(side)
        st["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(st["graph"]):
            _steps(st)
    return st


def _steps(st):
    for x, y in zip(st["xs"], st["ys"]):
        S.seer_spmv_auto(st["A"], st["model"].gathered, x, y, st["ws"])


def run(state):
    op, A = state["op"], state["A"]
    if op == "admit":
        bad_rp, bad_ci = S.seer_csr_check(A, workspace=state["ws"])
        f = S.seer_features(A, workspace=state["ws"])
        return {"bad": [bad_rp, bad_ci],
                "counts": [int(f.rows), int(f.cols), int(f.nnz), int(f.max_len), int(f.min_len), int(f.empty_rows),
                           int(f.sum_sq_len)],
                "f": f.vector()}
    xs, ys = state["xs"], state["ys"]
    if op == "step":
        S.seer_spmv_auto(A, state["model"].gathered, xs[0], ys[0], state["ws"])
    elif op == "steps":
        state["graph"].replay()
    elif op == "model":
        S.seer_spmv_model(A, state["model"], xs[0], ys[0], state["ws"])
    elif op == "spmv":
        S.seer_spmv(state["case"]["kernel"], A, xs[0], ys[0], workspace=state["ws"])
    elif op == "repeat":
        S.seer_spmv_prepared(state["plan"], A, xs[0], ys[0], workspace=state["ws"])
    else:
        plan, _ = S.seer_spmv_plan(A, state["model"], state["case"]["n"], plan_mem=state["plan_mem"],
                                   workspace=state["feature_ws"])
        for x, y in zip(xs, ys):
            S.seer_spmv_prepared(plan, A, x, y, workspace=state["ws"])
        return {"y": state["out"], "kernel": plan.kernel_id}
    return state["out"]


def _sizes(case):
    """(rows, cols, expected nnz)."""
    if case["family"] == "stencil":
        n, d = case["grid"], case["dim"]
        return n ** d, n ** d, (2 * d + 1) * n ** d - 2 * d * n ** (d - 1)
    rows = case["rows"]
    if case["family"] == "banded":
        b = min(case["half"], rows - 1)
        return rows, rows, rows * (2 * b + 1) - b * (b + 1)
    cols = case["cols"]
    if case["family"] == "fixed":
        mean = min(case["k"], cols)
    elif case["family"] == "uniform":
        mean = (case["lo"] + case["hi"]) / 2
    elif case["family"] == "poisson":
        mean = case["lam"]
    elif case["family"] == "empty":
        mean = 0.7 * case["lam"] / (1.0 - math.exp(-case["lam"]))
    else:
        k = np.arange(1, min(200_000, cols) + 1, dtype=np.float64)
        p = k ** -case["s"]
        tail = k[-1] ** (1.0 - case["s"]) / (case["s"] - 1.0)
        mean = (float((k * p).sum()) + k[-1] * tail) / (float(p.sum()) + tail)
    return rows, cols, int(rows * mean)


def work(case):
    """8 bytes per nonzero, 4 per row offset, x once, y once, per product."""
    rows, cols, nnz = _sizes(case)
    if case["op"] == "admit":
        return {"bytes": 4 * (rows + 1) + 4 * nnz, "flops": 0}
    n = case.get("n", 1)
    return {"bytes": n * (8 * nnz + 4 * (rows + 1) + 4 * cols + 4 * rows), "flops": n * 2 * nnz}


def tolerance(case):
    if case["op"] == "admit":
        return "exact"                      # integers, and quotients of them rounded once
    # fp32 products and sums of up to 200 000 terms in some order: two schedules of this library
    # differ from each other by up to 1.8e-7 in the 2-norm and 3.5e-5 in the worst row
    return {"rel": 7e-7, "max": 1.4e-4}


def exact(case, seed):
    A, xs = _inputs(case, seed)
    rp = A.row_ptr.to(torch.int64)
    if case["op"] == "admit":
        lens = (rp[1:] - rp[:-1])
        R, C, N = float(A.rows), float(A.cols), float(A.nnz)
        mean, sq = N / R, int((lens * lens).sum())
        var = float(A.rows * sq - A.nnz * A.nnz) / (R * R)
        mx, mn, em = int(lens.max()), int(lens.min()), int((lens == 0).sum())
        f = np.array([R, C, N, mean, mx, mn, var, em / R, mean / C, mx / C, mn / C, var / (C * C), 1.0])
        return {"bad": [0, 0], "counts": [A.rows, A.cols, A.nnz, mx, mn, em, sq], "f": f}
    va = A.values.to(torch.float64)
    ci = A.col_idx.to(torch.int64)
    y = torch.zeros(len(xs), A.rows, device=_DEVICE, dtype=torch.float64)
    step = 2_000_000                        # rows whose sums are formed together
    for k, x in enumerate(xs):
        for i in range(0, A.rows, step):
            off = rp[i:i + step + 1]
            a, e = int(off[0]), int(off[-1])
            if e > a:
                part = va[a:e] * x.to(torch.float64)[ci[a:e]]
                y[k, i:i + step] = torch.segment_reduce(part, "sum", offsets=off - a, initial=0.0)
    return {"y": y, "kernel": None} if case["op"] == "solve" else y
