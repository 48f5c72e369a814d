"""The workloads this library is timed on: whole solves from a seed to the
solution, factorisations alone and grouped, the refinement of several
right-hand sides with a factor in hand, single trailing updates, the
regenerating residual, and the FP64 LU with and without pivoting.

``listed()`` names twelve of them, ``draw`` gives more of the same ranges,
``prepare`` makes what a caller holds before the call, ``run`` is one pass
through the public entry points, ``work`` counts what a pass cannot do
without, and ``exact`` gives the results in FP64 from plain torch.
"""
import math

import torch

import paper_2509_19618_amd as mxp

_KIND = {"dominant": mxp.GEN_DOMINANT, "sqrtn": mxp.GEN_SQRTN, "uniform": mxp.GEN_UNIFORM}
_BYTES = {"f64": 8, "f32": 4, "f16": 2, "bf16": 2, "f8": 1}
_TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16, "f8": torch.float8_e4m3fn}


def _solve(name, n, nb, update, store, nrhs=1, kind="dominant", gamma=0.0):
    return {"name": name, "path": "solve", "n": n, "nb": nb, "update": update, "store": store, "nrhs": nrhs,
            "kind": kind, "gamma": gamma}


def listed():
    return [
        # whole solves: generate, factor, refine to the FP64 backward error.
        # The benchmark workload:
        _solve("solve_32768_f16", 32768, 512, "f16", "f16"),
        # the all-FP32 configuration at the size it is quoted on
        _solve("solve_2048_f32", 2048, 256, "f32", "f32"),
        # the smallest requests of the serving mix (latency and launch count)
        _solve("solve_600_bf16", 600, 128, "bf16", "bf16", nrhs=2),
        # FP8 update on FP16 storage, an odd size, the harder diagonal
        _solve("solve_20001_f8", 20001, 512, "f8", "f16", kind="sqrtn", gamma=1.0),
        # a factorisation alone, as a caller with many later right-hand sides runs it
        {"name": "factor_12013_bf16", "path": "factor", "n": 12013, "nb": 512, "update": "bf16", "store": "bf16",
         "kind": "dominant", "gamma": 0.0},
        # a group of mixed-size requests factored together, as the solve server does
        {"name": "group_bf16", "path": "group", "sizes": "520,777,1536,2100,3001,5003", "nb": 256, "update": "bf16",
         "store": "bf16"},
        # a factor in hand, eight new right-hand sides refined together
        {"name": "refine_8192x8_bf16", "path": "refine", "n": 8192, "nb": 512, "update": "bf16", "store": "bf16",
         "nrhs": 8, "kind": "dominant", "gamma": 0.0},
        # the Schur-complement update on its own: two block steps in one pass ...
        {"name": "update2_16384_f16", "path": "update", "M": 16384, "N": 16384, "K1": 512, "K2": 512, "update": "f16",
         "store": "f16"},
        # ... and one step with FP8 operands at a ragged size
        {"name": "update_5000x3001_f8", "path": "update", "M": 5000, "N": 3001, "K1": 512, "K2": 0, "update": "f8",
         "store": "f16"},
        # b - A x with A regenerated, at the benchmark's size
        {"name": "residual_32768", "path": "residual", "n": 32768, "nrhs": 1, "kind": "dominant", "gamma": 0.0},
        # FP64 LU and solve with partial pivoting on uniform entries (the pivoting study)
        {"name": "lu64_pivot_3000", "path": "lu64", "n": 3000, "pivot": True, "nrhs": 1, "kind": "uniform"},
        # FP64 LU and solve without pivoting (the baseline the figure of merit divides by)
        {"name": "lu64_8192", "path": "lu64", "n": 8192, "pivot": False, "nrhs": 2, "kind": "dominant"},
    ]


def _log_int(rng, lo, hi):
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    # half of the sizes are multiples of 64, the others as they fall
    return max(lo, min(hi, n // 64 * 64)) if rng.random() < 0.5 else n


def _pair(rng):
    return rng.choice([("f16", "f16"), ("bf16", "bf16"), ("f8", "f16"), ("f8", "bf16"), ("f32", "f32"),
                       ("f16", "f32"), ("bf16", "f32")])


def _diagonal(rng):
    return rng.choice([("dominant", 0.0), ("dominant", 0.0), ("sqrtn", 1.0)])


def draw(rng):
    path = rng.choice(["solve", "solve", "factor", "group", "refine", "update", "update", "residual", "lu64", "lu64"])
    nb = rng.choice([128, 256, 512, 512, 1024])
    if path in ("solve", "refine"):
        update, store = _pair(rng)
        kind, gamma = _diagonal(rng)
        hi = 8192 if update == "f32" else 24000
        if path == "refine":
            hi = min(hi, 12000)
        return {"path": path, "n": _log_int(rng, 200, hi), "nb": nb, "update": update, "store": store,
                "nrhs": 1 if path == "solve" and rng.random() < 0.6 else rng.randint(1, 8), "kind": kind,
                "gamma": gamma}
    if path == "factor":
        # storage formats whose factor carries no strip scales (results comparable entry by entry)
        update, store = rng.choice([("bf16", "bf16"), ("f8", "bf16"), ("f16", "f32"), ("f32", "f32")])
        kind, gamma = _diagonal(rng)
        return {"path": path, "n": _log_int(rng, 300, 8192 if update == "f32" else 16000), "nb": nb, "update": update,
                "store": store, "kind": kind, "gamma": gamma}
    if path == "group":
        sizes = [_log_int(rng, 512, 6000) for _ in range(rng.randint(2, 8))]
        return {"path": path, "sizes": ",".join(str(v) for v in sizes), "nb": min(nb, 512), "update": "bf16",
                "store": "bf16"}
    if path == "update":
        update, store = _pair(rng)
        hi = 4096 if update == "f32" else 20000
        K1 = rng.choice([128, 256, 512, 1024])
        return {"path": path, "M": _log_int(rng, 100, hi), "N": _log_int(rng, 100, hi), "K1": K1,
                "K2": rng.choice([0, K1]), "update": update, "store": store}
    if path == "residual":
        kind = rng.choice(["dominant", "sqrtn", "uniform"])
        return {"path": path, "n": _log_int(rng, 100, 32768), "nrhs": rng.randint(1, 8), "kind": kind,
                "gamma": 1.0 if kind == "sqrtn" else 0.0}
    pivot = rng.random() < 0.5
    return {"path": "lu64", "n": _log_int(rng, 100, 4000 if pivot else 8192), "pivot": pivot,
            "nrhs": rng.randint(1, 4), "kind": "uniform" if pivot else "dominant"}


# ------------------------------------------------------------------ inputs
def _bytes(nbytes):
    return torch.empty(max(int(nbytes), 1), dtype=torch.uint8, device="cuda")


def _generate(case, seed, nrhs, store, with_matrix=True):
    return mxp.mxp_generate(case["n"], nrhs, seed, store=store, kind=_KIND[case["kind"]],
                            gamma=case.get("gamma", 0.0), with_matrix=with_matrix)


def _pow2_strips(g, rows, top):
    """per 32 rows a power of two: 2^top or 2^(top - 1)"""
    return torch.pow(2.0, top - torch.randint(0, 2, (rows // 32,), generator=g, device="cuda").float())


def _operands(case, K, g):
    """The operands of one block step as the factorisation forms them: L21
    entries of about 2^-8 (a diagonal of the order of sqrt(n)), U12 entries of
    about 1/2, each 32-row strip under its own power of two."""
    up = case["update"]
    top = {"f16": 15, "f8": 8, "bf16": 0, "f32": 0}[up]
    out = []
    for rows, size in ((case["M"], 8), (case["N"], 1)):
        r = mxp.round_up(rows, 256)
        x = (torch.rand((r, K), generator=g, device="cuda") - 0.5) * 2.0 ** (1 - size)
        x[rows:] = 0
        s = _pow2_strips(g, r, float(top + size)) if top else torch.ones(r // 32, device="cuda")
        out.append(((x * s.repeat_interleave(32)[:, None]).to(_TORCH[up]), 1.0 / s))
    (a, ia), (b, ib) = out
    return a, b, ia, ib


def _update_inputs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    ldc = mxp.round_up(case["M"], 128)
    C = (torch.rand((case["N"], ldc), generator=g, device="cuda") - 0.5).to(_TORCH[case["store"]])
    return ldc, C, [_operands(case, K, g) for K in (case["K1"], case["K2"]) if K]


def prepare(case, seed):
    L, path = mxp.lib(), case["path"]
    if path == "update":
        ldc, C, segs = _update_inputs(case, seed)
        return {"case": case, "ldc": ldc, "C": C, "segs": segs}
    st = {"case": case, "seed": seed}
    if path in ("solve", "factor", "refine"):
        n, nb = case["n"], case["nb"]
        # the buffers a program keeps from one system to the next
        st["aux"] = _bytes(L.mxp_factor_aux_bytes(n, nb))
        st["fwork"] = _bytes(L.mxp_factor_work_bytes(n, nb, mxp.dtype_code(case["update"])))
        if path != "factor":
            st["swork"] = _bytes(L.mxp_solve_work_bytes(n, case["nrhs"], 30))
        if path == "refine":
            st["prob"] = _generate(case, seed, case["nrhs"], case["store"])
            st["fac"] = mxp.mxp_factor(st["prob"], nb, case["update"], work=st["fwork"], aux=st["aux"])
    if path == "residual":
        st["prob"] = _generate(case, seed, case["nrhs"], "f32", with_matrix=False)
        st["X"] = _residual_x(case, seed)
    if path == "lu64":
        st["work"] = _bytes(L.mxp_lu64_work_bytes(case["n"]))
    return st


def _residual_x(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.rand((case["nrhs"], case["n"]), generator=g, device="cuda", dtype=torch.float64) - 0.5


# ------------------------------------------------------------------ one pass
def run(st):
    case = st["case"]
    path = case["path"]
    if path == "solve":
        prob = _generate(case, st["seed"], case["nrhs"], case["store"])
        fac = mxp.mxp_factor(prob, case["nb"], case["update"], work=st["fwork"], aux=st["aux"])
        return mxp.mxp_solve_ir(prob, fac, work=st["swork"]).X
    if path == "factor":
        prob = _generate(case, st["seed"], 0, case["store"])
        fac = mxp.mxp_factor(prob, case["nb"], case["update"], work=st["fwork"], aux=st["aux"])
        return mxp.as_matrix(fac.LU, case["n"])
    if path == "group":
        sizes = [int(v) for v in case["sizes"].split(",")]
        probs = [mxp.mxp_generate(n, 0, st["seed"] + i, store=case["store"]) for i, n in enumerate(sizes)]
        facs = mxp.mxp_factor_group(probs, [case["nb"]] * len(sizes), case["update"])
        return [mxp.as_matrix(f.LU, f.n) for f in facs]
    if path == "refine":
        return mxp.mxp_solve_ir(st["prob"], st["fac"], work=st["swork"]).X
    if path == "update":
        C, ldc, M, N = st["C"], st["ldc"], case["M"], case["N"]
        if case["K2"]:
            (a1, b1, ia1, ib1), (a2, b2, ia2, ib2) = st["segs"]
            mxp.mxp_trailing_update2(C, ldc, M, N, case["K1"], case["K2"], case["update"], case["store"], a1, b1,
                                     ia1, ib1, a2, b2, ia2, ib2)
        else:
            a, b, ia, ib = st["segs"][0]
            mxp.mxp_trailing_update(C, ldc, M, N, case["K1"], case["update"], case["store"], a, b, ia, ib)
        return mxp.as_matrix(C, M)
    if path == "residual":
        return mxp.mxp_residual(st["prob"], st["X"], st["prob"].B)
    prob = _generate(case, st["seed"], case["nrhs"], "f64")
    fac = mxp.mxp_lu64_factor(prob.A, case["n"], prob.lda, case["pivot"], work=st["work"])
    X = mxp.mxp_lu64_solve(fac, prob.B)
    out = {"LU": mxp.as_matrix(fac.LU, case["n"]), "X": X}
    if case["pivot"]:
        out["ipiv"] = fac.ipiv
    return out


# ------------------------------------------------------------------ work
def _philox_ops(n):
    # ten rounds of two multiplies (both halves) and four xors per four entries
    return 10.0 * 8.0 / 4.0 * n * n


def work(case):
    path = case["path"]
    if path == "group":
        w = [work({"path": "factor", "n": int(v), "nb": case["nb"], "update": case["update"],
                   "store": case["store"]}) for v in case["sizes"].split(",")]
        return {k: sum(x[k] for x in w) for k in ("bytes", "flops")}
    if path == "update":
        M, N, K = case["M"], case["N"], case["K1"] + case["K2"]
        return {"bytes": 2.0 * M * N * _BYTES[case["store"]] + float(M + N) * K * _BYTES[case["update"]],
                "flops": 2.0 * M * N * K}
    n = case["n"]
    if path == "residual":
        return {"bytes": 24.0 * n * case["nrhs"] + 8.0 * n, "flops": 2.0 * n * n * case["nrhs"] + _philox_ops(n)}
    if path == "lu64":
        # the matrix is written by the generator and its factor by the LU; the solve reads the factor
        return {"bytes": 24.0 * n * n, "flops": 2.0 / 3.0 * n ** 3 + 2.0 * n * n * case["nrhs"] + _philox_ops(n)}
    s = _BYTES[case["store"]]
    if path == "factor":
        return {"bytes": 2.0 * s * n * n, "flops": 2.0 / 3.0 * n ** 3}
    # a refinement reads the factor for the start and for at least one
    # correction step, and regenerates the matrix for the two residuals
    refine = {"bytes": 2.0 * s * n * n, "flops": 2.0 * _philox_ops(n) + 8.0 * n * n * case["nrhs"]}
    if path == "refine":
        return refine
    return {"bytes": 2.0 * s * n * n + refine["bytes"], "flops": 2.0 / 3.0 * n ** 3 + refine["flops"]}


# ------------------------------------------------------------------ FP64 results from plain torch
def _philox(c0, c1, stream, seed):
    """four 32-bit words (int64 tensors) of Philox4x32-10 for counters (c0, c1, stream, 0)"""
    lo32 = 0xFFFFFFFF
    x0, x1, x2, x3 = torch.broadcast_tensors(c0, c1, torch.full_like(c0, stream), torch.zeros_like(c0))
    k0, k1 = seed & lo32, (seed >> 32) & lo32
    for _ in range(10):
        # the products wrap in int64; their halves do not depend on the sign
        p0, p1 = x0 * 0xD2511F53, x2 * 0xCD9E8D57
        x0, x1, x2, x3 = ((p1 >> 32) & lo32) ^ x1 ^ k0, p1 & lo32, ((p0 >> 32) & lo32) ^ x3 ^ k1, p0 & lo32
        k0, k1 = (k0 + 0x9E3779B9) & lo32, (k1 + 0xBB67AE85) & lo32
    return x0, x1, x2, x3


def _matrix64(case, n, seed):
    """A (n x n, FP64) and its diagonal"""
    kind = case.get("kind", "dominant")
    unit = 2.0 ** -31 if kind == "uniform" else 2.0 ** -32
    A = torch.empty((n, n), dtype=torch.float64, device="cuda")
    rowsum = torch.zeros(n, dtype=torch.int64, device="cuda")
    rows = torch.arange(n, device="cuda")[:, None]
    step = max(4, (1 << 26) // n // 4 * 4)
    for j in range(0, n, step):
        q = torch.arange(j // 4, (min(j + step, n) + 3) // 4, device="cuda")[None, :]
        w = torch.stack(_philox(rows + 0 * q, q + 0 * rows, 0, seed), dim=2).reshape(n, -1)[:, :min(step, n - j)]
        w = w - (1 << 31)
        rowsum += w.abs().sum(dim=1)
        A[:, j:j + w.shape[1]] = w.double() * unit
    d = A.diagonal()
    if kind == "dominant":
        d.copy_(rowsum.double() * 2.0 ** -32)
    elif kind == "sqrtn":
        d.add_(case["gamma"] * math.sqrt(n))
    return A


def _rhs64(n, nrhs, seed):
    i = torch.arange(n, device="cuda")
    words = []
    for q in range((nrhs + 3) // 4):
        words += list(_philox(i, torch.full_like(i, q), 1, seed))
    return torch.stack([(w - (1 << 31)).double() * 2.0 ** -32 for w in words[:nrhs]])


def exact(case, seed):
    path = case["path"]
    if path == "update":
        _, C, segs = _update_inputs(case, seed)
        M, N = case["M"], case["N"]
        out = C[:, :M].t().double()
        for a, b, ia, ib in segs:
            a = a[:M].double() * ia.double().repeat_interleave(32)[:M, None]
            b = b[:N].double() * ib.double().repeat_interleave(32)[:N, None]
            out -= a @ b.t()
        return out
    if path == "group":
        return [torch.linalg.lu_factor(_matrix64({}, int(v), seed + i))[0]
                for i, v in enumerate(case["sizes"].split(","))]
    n = case["n"]
    A = _matrix64(case, n, seed)
    if path == "residual":
        return _rhs64(n, case["nrhs"], seed) - _residual_x(case, seed) @ A.t()
    if path == "factor":
        return torch.linalg.lu_factor(A)[0]
    B = _rhs64(n, case["nrhs"], seed)
    if case.get("pivot"):
        # on the CPU: LAPACK takes the largest magnitude of every column; the
        # device library's blocked LU was seen to take other rows
        A, B = A.cpu(), B.cpu()
    lu, piv = torch.linalg.lu_factor(A)
    X = torch.linalg.lu_solve(lu, piv, B.t()).t()
    if path == "lu64":
        out = {"LU": lu, "X": X}
        if case["pivot"]:
            out["ipiv"] = piv.long() - 1
        return out
    return X
