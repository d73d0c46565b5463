"""Performance cases of the RBT solver: the work that programs have it do,
through the public binding, over the range of sizes, shapes, precisions and
directions the library serves.

Matrices (see `workloads`): "randn" is N(0,1), the family of the method's
paper, always solved with the paper's two fixed refinement steps (tol 0, two
corrections), so that X is accurate to the matrix's condition; "shifted"
(N(0,1)/sqrt(n) + I) is the adjoint's workload; "dominant"
(I + 0.3 N(0,1)/sqrt(n)) is the family whose low-precision factors suffice in
every precision, for the mixed and batched paths at their default tolerance.
"""
import math

import numpy as np
import torch

from paper_2312_09376_amd import rbt, workloads

PREC = {"fp32": rbt.RBT_FP32, "bf16": rbt.RBT_BF16}
SOLVER = {"classic": rbt.RBT_IR_CLASSIC, "gmres": rbt.RBT_IR_GMRES}
RBT_SEED = workloads.RBT_SEED


def listed():
    return [
        # one small dense system: a call in an outer loop, all latency
        {"name": "refine_100", "kind": "refine", "n": 100, "k": 1, "depth": 2},
        # the smallest configured system (n = 1000) as a plain solve
        {"name": "refine_1000", "kind": "refine", "n": 1000, "k": 1, "depth": 2},
        # the headline system: n = 20000, one right-hand side
        {"name": "refine_20000", "kind": "refine", "n": 20000, "k": 1, "depth": 2},
        # odd order and a wide block of right-hand sides
        {"name": "refine_5003_k64", "kind": "refine", "n": 5003, "k": 64, "depth": 2},
        # a differentiable solve in a training step: forward, dA and dB
        {"name": "autograd_4096_k8", "kind": "autograd", "n": 4096, "k": 8, "depth": 2,
         "prec": "fp64"},
        # factors kept, new right-hand sides as they come (serving), both directions
        {"name": "getrs_12000", "kind": "getrs", "n": 12000, "k": 1, "trans": 0},
        # mixed precision: FP32 factors, classical refinement, and its adjoint
        {"name": "mixed_adjoint_8191_k8", "kind": "mixed_adjoint", "n": 8191, "k": 8, "depth": 2},
        # mixed precision: BF16 updates, classical refinement, a large system
        {"name": "mixed_bf16_16384", "kind": "mixed", "n": 16384, "k": 1, "depth": 2,
         "prec": "bf16", "solver": "classic"},
        # mixed precision with GMRES refinement, several right-hand sides
        {"name": "mixed_gmres_3000_k4", "kind": "mixed", "n": 3000, "k": 4, "depth": 2,
         "prec": "fp32", "solver": "gmres"},
        # the pivoted solver that the fallback runs, and on its own
        {"name": "gepp_4000", "kind": "gepp", "n": 4000, "k": 1},
        # a batch of many small uneven systems
        {"name": "batched_1024_small", "kind": "batched", "count": 1024, "lo": 37, "hi": 300,
         "depth": 2, "prec": "fp32"},
        # a batch over the configured range of orders, 37 to 1500
        {"name": "batched_512", "kind": "batched", "count": 512, "lo": 37, "hi": 1500,
         "depth": 2, "prec": "fp32"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["refine", "refine", "autograd", "getrs", "mixed_adjoint", "mixed", "gepp",
                       "batched"])
    depth = rng.choice([1, 2, 2, 3])
    if kind == "refine":
        return {"kind": kind, "n": _log(rng, 50, 16000), "k": rng.choice([1, 1, 3, 8, 16, 40, 64]),
                "depth": depth}
    if kind == "autograd":
        return {"kind": kind, "n": _log(rng, 200, 8000), "k": rng.choice([1, 2, 8, 16]),
                "depth": depth, "prec": rng.choice(["fp64", "fp64", "fp32"])}
    if kind == "getrs":
        return {"kind": kind, "n": _log(rng, 500, 16000), "k": rng.choice([1, 1, 4, 16, 48]),
                "trans": rng.choice([0, 1])}
    if kind == "mixed_adjoint":
        return {"kind": kind, "n": _log(rng, 500, 9000), "k": rng.choice([1, 4, 8, 16]),
                "depth": depth}
    if kind == "mixed":
        return {"kind": kind, "n": _log(rng, 500, 18000), "k": rng.choice([1, 1, 4, 16]),
                "depth": depth, "prec": rng.choice(["fp32", "bf16"]),
                "solver": rng.choice(["classic", "classic", "gmres"])}
    if kind == "gepp":
        return {"kind": kind, "n": _log(rng, 100, 6000), "k": rng.choice([1, 4, 32])}
    lo = rng.randrange(17, 200)
    hi = lo + _log(rng, 50, 1300)
    return {"kind": "batched", "count": _log(rng, 16, 600), "lo": lo, "hi": hi, "depth": depth,
            "prec": rng.choice(["fp32", "fp32", "bf16"])}


def _dominant(n, seed):
    A = workloads.device_randn(n, n, seed)
    A *= 0.3 / math.sqrt(n)
    A.diagonal().add_(1.0)
    return A


def _cols(n, k, dtype=torch.float64):
    return torch.empty_strided((n, k), (1, n), dtype=dtype, device="cuda")


def _sizes(case, seed):
    # the sizes of a batch belong to the program, not to its inputs
    return workloads.batch_sizes(case["count"], case["lo"], case["hi"], seed=7)


def _inputs(case, seed):
    """Matrix, right-hand sides and (for the adjoints) the incoming gradient."""
    kind, n, k = case["kind"], case["n"], case["k"]
    if kind in ("refine", "gepp"):
        A = workloads.device_randn(n, n, 2 * seed + 1)
    elif kind in ("getrs",) or (kind == "autograd" and case["prec"] == "fp64"):
        A = workloads.device_shifted(n, 2 * seed + 1)
    else:
        A = _dominant(n, 2 * seed + 1)
    B = workloads.device_randn(n, k, 2 * seed + 2)
    G = workloads.device_randn(n, k, 2 * seed + 3) if kind in ("autograd", "mixed_adjoint") else None
    return A, B, G


def _batch_inputs(case, seed):
    """Every system's matrix and right-hand sides, each a slice of one buffer."""
    ns, ks = _sizes(case, seed)
    g = torch.Generator(device="cuda")
    g.manual_seed(2 * seed + 1)
    a = torch.randn(int((ns * ns).sum()), generator=g, device="cuda", dtype=torch.float64)
    b = torch.randn(int((ns * ks).sum()), generator=g, device="cuda", dtype=torch.float64)
    As, Bs, oa, ob = [], [], 0, 0
    for n, k in zip(ns.tolist(), ks.tolist()):
        A = a[oa:oa + n * n].view(n, n).t()
        A *= 0.3 / math.sqrt(n)
        A.diagonal().add_(1.0)
        As.append(A)
        Bs.append(b[ob:ob + n * k].view(k, n).t())
        oa, ob = oa + n * n, ob + n * k
    return ns, ks, As, Bs


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind == "batched":
        ns, ks, As, Bs = _batch_inputs(case, seed)
        x = torch.empty(int((ns * ks).sum()), dtype=torch.float64, device="cuda")
        Xs, o = [], 0
        for n, k in zip(ns.tolist(), ks.tolist()):
            Xs.append(x[o:o + n * k].view(k, n).t())
            o += n * k
        plan = rbt.batched_plan(ns, ks, case["depth"], PREC[case["prec"]])
        s.update(plan=plan, args=rbt.BatchArgs(plan, As, Bs, Xs), x=x)
        return s
    A, B, G = _inputs(case, seed)
    n, k = case["n"], case["k"]
    s.update(A=A, B=B, G=G)
    if kind == "refine":
        s.update(LU=_cols(n, n), X=_cols(n, k), work=_work(n, k, case["depth"], rbt.RBT_FP64))
    elif kind == "autograd":
        A.requires_grad_(True)
        B.requires_grad_(True)
    elif kind == "getrs":
        LU, _ = rbt.genp(A)
        s.update(LU=LU, X=_cols(n, k), work=_work(n, k, 0, rbt.RBT_FP64))
    elif kind == "mixed":
        s.update(LU=_cols(n, n, torch.float32), X=_cols(n, k),
                 work=_work(n, k, case["depth"], PREC[case["prec"]]))
    elif kind == "mixed_adjoint":
        s.update(LU=_cols(n, n, torch.float32), X=_cols(n, k),
                 work=_work(n, k, case["depth"], rbt.RBT_FP32))
    elif kind == "gepp":
        s.update(LU=_cols(n, n), X=_cols(n, k), work=_work(n, k, 0, rbt.RBT_FP64))
    return s


def _work(n, k, depth, prec):
    return torch.empty(rbt.workspace_size(n, k, depth, prec), dtype=torch.uint8, device="cuda")


def run(s):
    case = s["case"]
    kind, depth = case["kind"], case.get("depth", 0)
    if kind == "refine":
        X, _, _, _, info, _ = rbt.solve_refine(s["A"], s["B"], depth, RBT_SEED, tol=0.0, max_iter=2,
                                               LU=s["LU"], X=s["X"], work=s["work"])
        return {"X": X, "info": info}
    if kind == "autograd":
        prec = rbt.RBT_FP64 if case["prec"] == "fp64" else PREC[case["prec"]]
        X = rbt.rbt_solve(s["A"], s["B"], depth, RBT_SEED, prec=prec)
        dA, dB = torch.autograd.grad(X, (s["A"], s["B"]), s["G"])
        return {"X": X, "dA": dA, "dB": dB}
    if kind == "getrs":
        X = s["X"].copy_(s["B"])
        return {"X": rbt.getrs(s["LU"], X, case["trans"], work=s["work"])}
    if kind == "mixed":
        X, _, _, _, info, _ = rbt.solve_mixed(s["A"], s["B"], depth, RBT_SEED, PREC[case["prec"]],
                                              SOLVER[case["solver"]], LU=s["LU"], X=s["X"],
                                              work=s["work"])
        return {"X": X, "info": info}
    if kind == "mixed_adjoint":
        X, LU, _, _, info, _ = rbt.solve_mixed(s["A"], s["B"], depth, RBT_SEED, rbt.RBT_FP32,
                                               rbt.RBT_IR_CLASSIC, LU=s["LU"], X=s["X"],
                                               work=s["work"])
        dA, dB, _, _ = rbt.solve_backward_mixed(LU, s["A"], X, s["G"], depth, RBT_SEED,
                                                work=s["work"])
        return {"X": X, "dA": dA, "dB": dB, "info": info}
    if kind == "gepp":
        LU, ipiv, info = rbt.gepp(s["LU"].copy_(s["A"]), work=s["work"])
        X = rbt.gepp_solve(LU, ipiv, s["X"].copy_(s["B"]), work=s["work"])
        return {"LU": LU, "ipiv": ipiv, "X": X, "info": info}
    rbt.solve_batched_launch(s["plan"], s["args"], RBT_SEED)
    return {"x": s["x"], "info": s["args"].info}


def work(case):
    kind = case["kind"]
    if kind == "batched":
        ns, ks = (v.astype(np.float64) for v in _sizes(case, 0))
        # A read once, X and B; elimination, two triangular solves
        return {"bytes": float((8 * ns * ns + 16 * ns * ks).sum()),
                "flops": float((2 / 3 * ns**3 + 2 * ns * ns * ks).sum())}
    n, k = float(case["n"]), float(case["k"])
    lu, solve, mv = 2 / 3 * n**3, 2 * n * n * k, 2 * n * n * k
    if kind == "refine":  # A in, factors out; three solves, two residuals
        return {"bytes": 16 * n * n + 16 * n * k, "flops": lu + 3 * solve + 2 * mv}
    if kind == "autograd":  # A in, dA out
        return {"bytes": 16 * n * n + 32 * n * k, "flops": lu + 2 * solve + 2 * n * n * k}
    if kind == "getrs":  # the factors in
        return {"bytes": 8 * n * n + 16 * n * k, "flops": solve}
    if kind == "mixed":  # A in, FP32 factors out
        return {"bytes": 12 * n * n + 16 * n * k, "flops": lu + solve + mv}
    if kind == "mixed_adjoint":  # A in, FP32 factors and dA out
        return {"bytes": 20 * n * n + 32 * n * k, "flops": lu + 2 * solve + 2 * mv + 2 * n * n * k}
    return {"bytes": 16 * n * n + 16 * n * k, "flops": lu + solve}


def exact(case, seed):
    kind = case["kind"]
    if kind == "batched":
        ns, ks, As, Bs = _batch_inputs(case, seed)
        return {"x": torch.cat([torch.linalg.solve(A, B).t().reshape(-1) for A, B in zip(As, Bs)]),
                "info": None}
    A, B, G = _inputs(case, seed)
    if kind == "getrs" and case["trans"]:
        return {"X": torch.linalg.solve(A.t(), B)}
    if kind == "getrs":
        return {"X": torch.linalg.solve(A, B)}
    X = torch.linalg.solve(A, B)
    if kind in ("refine", "mixed"):
        # one step of refinement of the pivoted solution
        return {"X": X + torch.linalg.solve(A, B - A @ X), "info": None}
    if kind == "gepp":
        return {"LU": None, "ipiv": None, "X": X + torch.linalg.solve(A, B - A @ X), "info": None}
    dB = torch.linalg.solve(A.t(), G)
    out = {"X": X, "dA": -dB @ X.t(), "dB": dB}
    if kind == "mixed_adjoint":
        out["info"] = None
    return out
