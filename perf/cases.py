"""What the framework is timed on: the work that a user's program has it do,
each piece through the package's public entry points.

Kinds of case:

* heq     one solve of the Chandrasekhar H-equation (eq. (3.2)) by Newton's
          method in three precisions, from a given iterate to the stopping
          rule; LU precision, linear solver and the FFT form are options;
* dense   one solve of the dense system F(x) = A x + 0.1 tanh(x) - b, whose
          factorisation interchanges rows;
* getrf   one LU factorisation of a matrix that the caller has;
* getrs   one solve with factors that the caller has, rows interchanged;
* parts   the pieces of a caller's own Newton loop: F, J and the refinement
          residual r = b - J u;
* engine  a burst of H-equation requests of mixed sizes through the batched
          engine, from admission to the collected results.

Sizes are those of the benchmark, the tests and the stored references
(256, 1000, 4096, 8192, 16384; 128 to 2048 for requests) or odd ones between.
"""
import math

import numpy as np
import torch

import paper_2307_16051_amd as n3p

DEVICE = "cuda"
TORCH = {"FP16": torch.float16, "BF16": torch.bfloat16, "FP32": torch.float32, "FP64": torch.float64}
REQUEST_SIZES = (128, 256, 512, 1024, 2048)


def listed():
    return [
        # the smallest whole solve (the size of the smoke check): launches and host waits
        {"name": "heq_256_fp16_ir", "kind": "heq", "n": 256, "c": 0.9, "prec": "FP16",
         "solver": "IR", "fft": False},
        # an ordinary small system of a ragged size in the other half precision
        {"name": "heq_1000_bf16_ir", "kind": "heq", "n": 1000, "c": 0.99, "prec": "BF16",
         "solver": "IR", "fft": False},
        # the paper's ill-conditioned table: GMRES-IR, many triangular solves a step
        {"name": "heq_4096_fp16_gmres", "kind": "heq", "n": 4096, "c": 0.9999, "prec": "FP16",
         "solver": "GMRES_IR", "fft": False},
        # the operator form: FFT residual and J v without a stored J
        {"name": "heq_8192_fp16_fft", "kind": "heq", "n": 8192, "c": 0.9, "prec": "FP16",
         "solver": "IR", "fft": True},
        # the benchmark's solve, the largest
        {"name": "heq_16384_fp16_ir", "kind": "heq", "n": 16384, "c": 0.99, "prec": "FP16",
         "solver": "IR", "fft": False},
        # the comparison column: Newton with a double-precision factorisation
        {"name": "heq_3000_fp64_direct", "kind": "heq", "n": 3000, "c": 0.9, "prec": "FP64",
         "solver": "DIRECT", "fft": False},
        # a dense system that needs row interchanges
        {"name": "dense_2048_fp16_ir", "kind": "dense", "n": 2048, "cond": 100.0, "prec": "FP16",
         "solver": "IR"},
        # the factorisation by itself: half precision, no interchange, odd size
        {"name": "getrf_5001_fp16", "kind": "getrf", "n": 5001, "prec": "FP16", "matrix": "heq"},
        # the factorisation by itself: double precision with partial pivoting
        {"name": "getrf_2500_fp64_pivot", "kind": "getrf", "n": 2500, "prec": "FP64",
         "matrix": "gaussian"},
        # one right-hand side against factors kept in half precision
        {"name": "getrs_6001_fp16", "kind": "getrs", "n": 6001, "prec": "FP16"},
        # a caller's own Newton loop: residual, Jacobian, refinement residual
        {"name": "parts_5003", "kind": "parts", "n": 5003, "c": 0.9},
        # a server's burst of small systems
        {"name": "engine_32", "kind": "engine", "count": 32, "prec": "FP16"},
    ]


def _size(rng, lo, hi):
    """A size spread over the logarithm of the range; half of them odd."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.5:
        n |= 1
    return max(lo, min(hi, n))


def draw(rng):
    kind = rng.choice(["heq", "heq", "heq", "dense", "getrf", "getrf", "getrs", "parts", "engine"])
    if kind == "heq":
        which = rng.choice(["FP16", "FP16", "BF16", "FP32", "FP64", "GMRES", "FFT"])
        if which == "GMRES":
            return {"kind": kind, "n": _size(rng, 256, 6000), "c": 0.9999, "prec": "FP16",
                    "solver": "GMRES_IR", "fft": False}
        c = round(rng.uniform(0.5, 0.99), 3)
        if which == "FP64":
            return {"kind": kind, "n": _size(rng, 128, 4096), "c": c, "prec": "FP64",
                    "solver": "DIRECT", "fft": False}
        if which == "FP32":
            return {"kind": kind, "n": _size(rng, 128, 4096), "c": c, "prec": "FP32",
                    "solver": "IR", "fft": False}
        return {"kind": kind, "n": _size(rng, 128, 12000), "c": c,
                "prec": "FP16" if which == "FFT" else which, "solver": "IR", "fft": which == "FFT"}
    if kind == "dense":
        return {"kind": kind, "n": _size(rng, 256, 4096), "cond": round(rng.uniform(10.0, 100.0), 1),
                "prec": "FP16", "solver": rng.choice(["IR", "GMRES_IR"])}
    if kind == "getrf":
        prec = rng.choice(["FP16", "BF16", "FP32", "FP64"])
        hi = {"FP16": 12000, "BF16": 12000, "FP32": 6000, "FP64": 4100}[prec]
        return {"kind": kind, "n": _size(rng, 128, hi), "prec": prec,
                "matrix": "gaussian" if prec == "FP64" and rng.random() < 0.6 else "heq"}
    if kind == "getrs":
        return {"kind": kind, "n": _size(rng, 128, 12000),
                "prec": rng.choice(["FP16", "BF16", "FP32", "FP64"])}
    if kind == "parts":
        return {"kind": kind, "n": _size(rng, 128, 12000), "c": round(rng.uniform(0.5, 0.99), 3)}
    return {"kind": kind, "count": rng.randint(4, 48), "prec": rng.choice(["FP16", "BF16"])}


# ---------------------------------------------------------------------- inputs
def _gen(seed):
    return torch.Generator(device=DEVICE).manual_seed(seed)


def _uniform(g, lo, hi, *shape, dtype=torch.float64):
    return torch.rand(*shape, generator=g, device=DEVICE, dtype=dtype) * (hi - lo) + lo


def _mu(n):
    return (torch.arange(n, device=DEVICE, dtype=torch.float64) + 0.5) / n


def _heq_like(g, n, scale):
    """Column-major FP64 matrix of the H-equation Jacobian's kind: the identity
    less a kernel of norm below one half, every entry of it at random, times
    `scale` (half precision keeps its small entries normal that way)."""
    mu = _mu(n)
    B = mu[None, :] / (mu[None, :] + mu[:, None])  # transposed: row-major here
    B *= _uniform(g, 0.25, 0.75, n, n)
    B *= -scale / n
    B.diagonal().add_(scale)
    return B.t()


def _dense_system(case, seed):
    """A = P diag(s) Q with orthogonal P, Q (signed cosine transforms), s from
    1 to cond over its logarithm, and b with the solution x* in [0.5, 1.5]."""
    n, g = case["n"], _gen(seed)
    k = torch.arange(n, device=DEVICE, dtype=torch.float64)
    C = torch.cos((math.pi / n) * (k[None, :] + 0.5) * k[:, None]) * math.sqrt(2.0 / n)
    C[0] *= math.sqrt(0.5)

    def signs():
        return torch.randint(0, 2, (n,), generator=g, device=DEVICE).double() * 2 - 1

    s = case["cond"] ** (k / max(n - 1, 1))
    s = s[torch.randperm(n, generator=g, device=DEVICE)]
    left = signs()[:, None] * C.t() * s[None, :]
    right = signs()[:, None] * C * signs()[None, :]
    A = (right.t() @ left.t()).contiguous().t()  # column-major
    xs = _uniform(g, 0.5, 1.5, n)
    return A, A @ xs + 0.1 * torch.tanh(xs)


def _requests(case, seed):
    rng = np.random.default_rng(seed)
    # the mix of sizes is the case's, so that every seed is the same amount of work
    ns = [REQUEST_SIZES[i % len(REQUEST_SIZES)] for i in range(case["count"])]
    return ns, rng.uniform(0.5, 0.999, case["count"]).tolist()


def prepare(case, seed):
    s = {"case": case}
    kind, g = case["kind"], _gen(seed)
    if kind in ("heq", "dense"):
        n = case["n"]
        prec, solver = getattr(n3p, case["prec"]), getattr(n3p, case["solver"])
        fft = int(case.get("fft", False))
        s.update(prec=prec, solver=solver,
                 opts=n3p.Options.default(fft_residual=fft, matrix_free=fft))
        s["ws"] = torch.empty(n3p.workspace_size(n, prec, solver, s["opts"]), dtype=torch.uint8,
                              device=DEVICE)
        if kind == "heq":
            s["x0"] = _uniform(g, 1.0, 1.1, n)
        else:
            s["A"], s["b"] = _dense_system(case, seed)
            s["x0"] = torch.zeros(n, dtype=torch.float64, device=DEVICE)
        s["x"] = torch.empty_like(s["x0"])
    elif kind == "getrf":
        s["A"] = _getrf_matrix(case, seed)
        s["LU"] = torch.empty_like(s["A"])
    elif kind == "getrs":
        s["LU"], s["ipiv"], s["b"] = _factors(case, seed)
        s["x"] = torch.empty_like(s["b"])
    elif kind == "parts":
        n = case["n"]
        s["x"] = _uniform(g, 1.0, 1.1, n)
        s["u"] = _uniform(g, -1.0, 1.0, n, dtype=torch.float32)
        s["b"] = _uniform(g, -1.0, 1.0, n, dtype=torch.float32)
    else:
        ns, cs = _requests(case, seed)
        prec = getattr(n3p, case["prec"])
        cfg = n3p.EngineConfig.default(max_slots=64, max_n=max(REQUEST_SIZES), lu_prec=prec)
        pool = n3p.engine_fixed_bytes(64) + sum(n3p.engine_request_bytes(n, prec) for n in ns) + 4096
        s["engine"] = n3p.Engine(torch.empty(pool, dtype=torch.uint8, device=DEVICE), cfg)
        s["x"] = torch.empty(sum(ns), dtype=torch.float64, device=DEVICE)
        s["requests"] = list(zip(ns, cs, s["x"].split(ns)))
    return s


def _getrf_matrix(case, seed):
    n, g = case["n"], _gen(seed)
    if case["matrix"] == "gaussian":
        A = torch.randn(n, n, generator=g, device=DEVICE, dtype=torch.float64).t()
    else:
        A = _heq_like(g, n, 256.0)
    return A.to(TORCH[case["prec"]])


def _factors(case, seed):
    """Unit lower and upper factors of the H-equation's kind, and an
    interchange list as partial pivoting leaves it."""
    n, g = case["n"], _gen(seed)
    LU = _heq_like(g, n, 256.0)
    LU = (LU * (torch.tril(torch.full_like(LU, 1.0 / 256.0), -1) + torch.triu(torch.ones_like(LU))))
    LU = LU.t().contiguous().t().to(TORCH[case["prec"]])
    k = torch.arange(n, device=DEVICE)
    ipiv = k + (torch.rand(n, generator=g, device=DEVICE) * (n - k)).long().clamp_(min=0)
    ipiv = torch.minimum(ipiv, torch.full_like(ipiv, n - 1)).to(torch.int32)
    b = _uniform(g, -1.0, 1.0, n)
    return LU, ipiv, b if case["prec"] == "FP64" else b.float()


# ------------------------------------------------------------------------ run
def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "heq":
        state["x"].copy_(state["x0"])
        x, rep = n3p.solve_heq(case["n"], case["c"], x=state["x"], prec=state["prec"],
                               solver=state["solver"], opts=state["opts"], ws=state["ws"])
        return {"x": x, "its": rep.its, "status": rep.status}
    if kind == "dense":
        state["x"].copy_(state["x0"])
        x, rep = n3p.solve_dense_tanh(state["A"], state["b"], state["x"], prec=state["prec"],
                                      solver=state["solver"], opts=state["opts"], ws=state["ws"])
        return {"x": x, "its": rep.its, "status": rep.status}
    if kind == "getrf":
        state["LU"].copy_(state["A"])
        ipiv, info = n3p.getrf(state["LU"])
        return {"LU": state["LU"], "ipiv": ipiv, "info": info}
    if kind == "getrs":
        state["x"].copy_(state["b"])
        return {"x": n3p.getrs(state["LU"], state["ipiv"], state["x"])}
    if kind == "parts":
        F, D = n3p.heq_residual(state["x"], case["c"])
        J = n3p.heq_jacobian(D, case["c"])
        return {"F": F, "D": D, "J": J, "r": n3p.gemv_resid(J, state["u"], state["b"])}
    eng = state["engine"]
    slots = [eng.admit(n, c) for n, c, _ in state["requests"]]
    left = len(slots)
    while left:
        left = len(slots) - eng.step()
    its = [eng.collect(slot, x).its for slot, (_, _, x) in zip(slots, state["requests"])]
    return {"x": state["x"], "its": np.array(its)}


# ----------------------------------------------------------------------- work
def _newton_steps(c):
    """Newton steps to 1e-10 from ones (the same at every size)."""
    return 3 if c <= 0.5 else 4 if c <= 0.9 else 6 if c <= 0.99 else 9


def work(case):
    kind = case["kind"]
    if kind == "engine":
        ns, _ = _requests(case, 0)
        return {"bytes": sum(16.0 * n for n in ns),
                "flops": sum(5 * (2.0 / 3.0 * n ** 3 + 2 * 6.0 * n * n) for n in ns)}
    n = float(case["n"])
    es = {"FP16": 2, "BF16": 2, "FP32": 4, "FP64": 8}[case.get("prec", "FP32")]
    lu = 2.0 / 3.0 * n ** 3
    if kind == "heq":  # each step: the factorisation, two sweeps of refinement, F
        return {"bytes": 16 * n, "flops": _newton_steps(case["c"]) * (lu + 10.0 * n * n)}
    if kind == "dense":
        return {"bytes": 8 * n * n + 24 * n, "flops": 3 * (lu + 22.0 * n * n)}
    if kind == "getrf":
        return {"bytes": 2 * es * n * n + 4 * n, "flops": lu}
    if kind == "getrs":
        return {"bytes": es * n * n + (20 if case["prec"] == "FP64" else 12) * n, "flops": 2 * n * n}
    return {"bytes": 4 * n * n + 36 * n, "flops": 6 * n * n}


# ---------------------------------------------------------------------- exact
def _heq_operator(n, c):
    mu = _mu(n)
    K = mu[:, None] / (mu[:, None] + mu[None, :])
    K *= c / (2.0 * n)
    return K


def _heq_solution(n, c, x):
    """Newton's method in 64 bits to the rounding floor."""
    K = _heq_operator(n, c)
    best, xb = math.inf, x
    for _ in range(30):
        D = 1.0 - K @ x
        F = x - 1.0 / D
        f = float(F.norm())
        if not f < 0.5 * best:
            break
        best, xb = f, x
        J = K / (-(D * D)[:, None])
        J.diagonal().add_(1.0)
        x = x - torch.linalg.solve(J, F)
        del J
    return xb


def exact(case, seed):
    kind = case["kind"]
    if kind == "heq":
        x = _heq_solution(case["n"], case["c"], _uniform(_gen(seed), 1.0, 1.1, case["n"]))
        return {"x": x, "its": None, "status": None}
    if kind == "dense":
        A, b = _dense_system(case, seed)
        x = torch.zeros_like(b)
        for _ in range(8):
            F = A @ x + 0.1 * torch.tanh(x) - b
            J = A + torch.diag(0.1 * (1.0 - torch.tanh(x) ** 2))
            x = x - torch.linalg.solve(J, F)
        return {"x": x, "its": None, "status": None}
    if kind == "getrf":
        # partial pivoting in 64 bits of the matrix as it is stored
        A = _getrf_matrix(case, seed).double()
        if case["matrix"] == "gaussian":
            A = A.cpu()  # LAPACK's rule: the largest entry of the column, the lowest row of equals
        return {"LU": torch.linalg.lu_factor(A)[0], "ipiv": None, "info": None}
    if kind == "getrs":
        LU, ipiv, b = _factors(case, seed)
        perm = np.arange(case["n"])
        for k, p in enumerate(ipiv.cpu().numpy()):
            perm[k], perm[p] = perm[p], perm[k]
        LU, x = LU.double(), b.double()[torch.from_numpy(perm).to(DEVICE)][:, None]
        x = torch.linalg.solve_triangular(LU, x, upper=False, unitriangular=True)
        return {"x": torch.linalg.solve_triangular(LU, x, upper=True)[:, 0]}
    if kind == "parts":
        n, g = case["n"], _gen(seed)
        x = _uniform(g, 1.0, 1.1, n)
        u = _uniform(g, -1.0, 1.0, n, dtype=torch.float32)
        b = _uniform(g, -1.0, 1.0, n, dtype=torch.float32)
        K = _heq_operator(n, case["c"])
        D = 1.0 - K @ x
        J = K / (-(D * D)[:, None])
        J.diagonal().add_(1.0)
        # r is formed from the J that is stored in 32 bits
        return {"F": x - 1.0 / D, "D": D, "J": J, "r": b.double() - J.float().double() @ u.double()}
    ns, cs = _requests(case, seed)
    xs = [_heq_solution(n, c, torch.ones(n, dtype=torch.float64, device=DEVICE))
          for n, c in zip(ns, cs)]
    return {"x": torch.cat(xs), "its": None}
