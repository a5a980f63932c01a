"""The calls a program makes on this framework, over the sizes it makes them at.

Every case goes through a public entry point of `paper_1502_07806_amd` on
inputs of the kind the method is for: a symmetric matrix with the density of
states of the synthetic workloads (occupied square-root band, flat unoccupied
band; levels at jittered quantiles of it, so that neighbouring levels repel
each other as those of a system without symmetry do and every eigenvector is
determined by its matrix), and previous eigenvectors a small rotation away.

`exact` is the same method written down in 64 bits with plain torch / numpy:
basis change, LAPACK on the submatrices, folded-spectrum iterations,
Cholesky-QR, Rayleigh quotients, ordering.
"""
import math

import numpy as np
import torch

import paper_1502_07806_amd as pf

DEV = "cuda:0"
ETA = 1e-8  # Lorentzian broadening of the adjoint (the entry points' default)


# ---------------------------------------------------------------- the cases
def listed():
    return [
        # The smallest step a program makes: N = 256, every launch and every
        # latency of the FP64 path counts.
        {"name": "solve_fp64_256", "kind": "solve", "precision": "fp64", "n": 256, "slice": 64, "halo": 32,
         "iterations": 3, "power": 2},
        # A serving loop that may not allocate: the library's own workspace,
        # an odd order and a ragged last slice, mixed precision.
        {"name": "static_mixed_607", "kind": "static", "precision": "mixed_bf16", "n": 607, "slice": 100, "halo": 50,
         "iterations": 3, "power": 2},
        # One guarded SCF step of the driver (dominance monitor, FP64 step,
        # residual monitor) at the order of the SCF-like sequence.
        {"name": "scf_step_2048", "kind": "scf", "precision": "fp64", "n": 2048, "slice": 256, "halo": 128,
         "iterations": 3, "power": 2},
        # The full diagonalisation of the first SCF steps, without a start basis.
        {"name": "full_diag_1024", "kind": "full", "precision": "fp64", "n": 1024, "slice": 1024, "halo": 0,
         "iterations": 0, "power": 2},
        # The order of the paper's smallest system (Cu256), submatrices of 0.3 N, FP64.
        {"name": "solve_fp64_1664", "kind": "solve", "precision": "fp64", "n": 1664, "slice": 208, "halo": 146,
         "iterations": 3, "power": 2},
        # An odd order in the middle of the range, slices that do not divide
        # it, mixed precision, residuals guarded by a threshold.
        {"name": "solve_mixed_3001", "kind": "solve", "precision": "mixed_bf16", "n": 3001, "slice": 250, "halo": 125,
         "iterations": 3, "power": 2, "resid_tol": 1e-2},
        # The headline step: N = 8192, 32 slices, submatrices of 512, mixed precision.
        {"name": "solve_mixed_8192", "kind": "solve", "precision": "mixed_bf16", "n": 8192, "slice": 256, "halo": 128,
         "iterations": 3, "power": 2},
        # The same step in FP64 throughout, the largest case.
        {"name": "solve_fp64_8192", "kind": "solve", "precision": "fp64", "n": 8192, "slice": 256, "halo": 128,
         "iterations": 3, "power": 2},
        # Submatrices of the paper's width, 0.3 N, where the submatrix eigensolver rules.
        {"name": "wide_mixed_4096", "kind": "solve", "precision": "mixed_bf16", "n": 4096, "slice": 256, "halo": 486,
         "iterations": 3, "power": 2},
        # k-points of uneven order in one call, as the batched workload draws them.
        {"name": "batched_mixed_12", "kind": "batched", "precision": "mixed_bf16", "n": 2048, "count": 12, "slice": 128,
         "halo": 64, "iterations": 3, "power": 2},
        # Gradient of a loss over the occupied half (backward of a training step).
        {"name": "backward_4096", "kind": "backward", "precision": "mixed_bf16", "n": 4096, "slice": 256, "halo": 128,
         "iterations": 3, "power": 2, "split": False},
        # Generalized -> standard conversion, eight steps.
        {"name": "convert_4096", "kind": "convert", "precision": "fp64", "n": 4096, "iterations": 8},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve64", "solve64", "mixed", "mixed", "mixed", "static", "scf", "full", "wide", "batched",
                       "backward", "convert"])
    if kind == "convert":
        return {"kind": "convert", "precision": "fp64", "n": _log(rng, 500, 6000), "iterations": rng.randint(4, 8)}
    if kind == "full":
        n = _log(rng, 100, 1100)
        return {"kind": "full", "precision": "fp64", "n": n, "slice": n, "halo": 0, "iterations": 0, "power": 2}
    c = {"kind": "solve", "precision": rng.choice(["fp64", "mixed_bf16"]), "n": 0, "slice": 0, "halo": 0,
         "iterations": rng.choice([2, 3, 3, 3, 4]), "power": 2}
    if kind == "solve64":
        c["precision"] = "fp64"
        c["n"] = _log(rng, 200, 5000)
        c["power"] = rng.choice([2, 2, 2, 1])
    elif kind == "mixed":
        c["precision"] = "mixed_bf16"
        c["n"] = _log(rng, 300, 8192)
        c["fs_split"] = rng.random() < 0.2
    elif kind == "static":
        c["kind"] = "static"
        c["n"] = _log(rng, 200, 740)
    elif kind == "scf":
        c["kind"] = "scf"
        c["precision"] = "fp64"
        c["n"] = _log(rng, 400, 3000)
    elif kind == "backward":
        c["kind"] = "backward"
        c["n"] = _log(rng, 400, 5000)
        c["split"] = c["precision"] == "mixed_bf16" and rng.random() < 0.5
    elif kind == "batched":
        c["kind"] = "batched"
        c["precision"] = "mixed_bf16"
        c["n"] = rng.choice([1024, 1536, 2048])
        c["count"] = rng.randint(4, 16)
    else:  # wide
        c["n"] = _log(rng, 1000, 4096)
    if kind == "wide":
        c["slice"] = c["n"] // rng.randint(6, 16)
        c["halo"] = max(1, int(rng.uniform(0.2, 0.3) * c["n"] - c["slice"]) // 2)
    else:
        c["slice"] = rng.randint(max(32, min(c["n"], 512) // 8), max(64, min(256, c["n"] // 3)))
        c["halo"] = c["slice"] // 2
    if c["kind"] == "solve" and rng.random() < 0.25:
        c["resid_tol"] = 1e-2
    return c


# ---------------------------------------------------------------- inputs
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _levels(n, g):
    """Ascending levels: occupied half -0.8 + u^(2/3), unoccupied half 0.2 + 1.3 u, at jittered quantiles."""
    m = n // 2
    j = 0.6 * (torch.rand(n, generator=g, device=DEV, dtype=torch.float64) - 0.5)
    u0 = (torch.arange(m, device=DEV, dtype=torch.float64) + 0.5 + j[:m]) / max(m, 1)
    u1 = (torch.arange(n - m, device=DEV, dtype=torch.float64) + 0.5 + j[m:]) / (n - m)
    return torch.cat([-0.8 + u0 ** (2.0 / 3.0), 0.2 + 1.3 * u1])


def _basis(n, g):
    """A dense orthogonal matrix: cosine basis, random signs, 32 random reflections."""
    i = torch.arange(n, device=DEV, dtype=torch.int64)
    C = torch.cos(((2 * i[:, None] + 1) * i[None, :] % (4 * n)).to(torch.float64) * (math.pi / (2 * n)))
    C *= math.sqrt(2.0 / n)
    C[:, 0] *= math.sqrt(0.5)
    C *= (torch.randint(0, 2, (n, 1), generator=g, device=DEV) * 2 - 1).to(torch.float64)
    k = min(32, n)
    U = torch.randn(n, k, generator=g, device=DEV, dtype=torch.float64)
    U /= torch.linalg.vector_norm(U, dim=0, keepdim=True)
    T = torch.triu(U.T @ U, 1).cpu() + 0.5 * torch.eye(k, dtype=torch.float64)
    return C - (C @ U) @ (torch.linalg.inv(T).to(DEV) @ U.T)


def _colmajor(M):
    return M.t().contiguous().t()


def _problem(n, g, kappa=1e-2):
    """(A, V_prev, levels, eigenvectors): A symmetric, V_prev = Q exp(K), ||K||_F = kappa."""
    lam = _levels(n, g)
    Q = _basis(n, g)
    A = (Q * lam) @ Q.T
    A = 0.5 * (A + A.T)
    K = torch.randn(n, n, generator=g, device=DEV, dtype=torch.float64)
    K = K - K.T
    K *= kappa / torch.linalg.matrix_norm(K)
    E = torch.eye(n, device=DEV, dtype=torch.float64)
    for j in range(6, 0, -1):
        E = (K @ E) / j
        E.diagonal().add_(1.0)
    return _colmajor(A), _colmajor(Q @ E), lam, Q


def _offsets(n, size):
    return list(range(0, n, size)) + [n]


def _batch_orders(case):
    sizes = [s for s in (384, 512, 768, 1024, 1536, 2048) if s <= case["n"]]
    return [sizes[(b * b + b // 2) % len(sizes)] for b in range(case["count"])]


def _options(case):
    o = {"halo": case["halo"], "iterations": case["iterations"], "fs_power": case["power"],
         "precision": case["precision"]}
    if case.get("resid_tol"):
        o["resid_tol"] = case["resid_tol"]
    if case.get("fs_split"):
        o["fs_split"] = True
    if case.get("split"):
        o["backward_split"] = True
    return o


def _adjoint_inputs(case, g):
    n, m = case["n"], case["n"] // 2
    lam, V = _levels(n, g), _colmajor(_basis(n, g))
    gl = torch.zeros(n, device=DEV, dtype=torch.float64)
    gl[:m] = torch.rand(m, generator=g, device=DEV, dtype=torch.float64)
    w = torch.rand(m, generator=g, device=DEV, dtype=torch.float64)
    d = torch.randn(n, generator=g, device=DEV, dtype=torch.float64)
    gV = torch.zeros(n, n, device=DEV, dtype=torch.float64)
    gV[:, :m] = 2.0 * d[:, None] * V[:, :m] * w  # gradient of sum_i w_i v_i^T diag(d) v_i over the occupied half
    return lam, V, gl, _colmajor(gV)


def _overlap(n, g):
    G = torch.randn(n, n, generator=g, device=DEV, dtype=torch.float64)
    B = (G @ G.T) * (0.05 / n)
    B = 0.5 * (B + B.T)
    B.diagonal().add_(1.0)
    return _colmajor(B)


def _scf_matrix(A, g):
    """The next SCF step's matrix: A plus a symmetric perturbation of Frobenius norm 5e-3."""
    n = A.shape[0]
    E = torch.randn(n, n, generator=g, device=DEV, dtype=torch.float64)
    E = E + E.T
    return _colmajor(A + E * (5e-3 / torch.linalg.matrix_norm(E)))


def prepare(case, seed):
    g = _gen(seed)
    kind, n = case["kind"], case["n"]
    s = {"kind": kind}
    if kind == "batched":
        orders = _batch_orders(case)
        probs = [_problem(nb, g)[:2] for nb in orders]
        s["A"], s["V"] = [p[0] for p in probs], [p[1] for p in probs]
        s["plan"] = pf.BatchedPlan([dict(_options(case), n=nb, part_offsets=_offsets(nb, case["slice"]))
                                    for nb in orders])
    elif kind == "convert":
        s["A"], s["B"] = _problem(n, g)[0], _overlap(n, g)
        s["iterations"] = case["iterations"]
    elif kind == "backward":
        s["lam"], s["V"], s["gl"], s["gV"] = _adjoint_inputs(case, g)
        s["plan"] = pf.Plan(n, _offsets(n, case["slice"]), **_options(case))
    elif kind == "full":
        s["A"] = _problem(n, g)[0]
        s["plan"] = pf.FullDiag(n)
    elif kind == "scf":
        A0, V, lam, Q = _problem(n, g)
        drv = pf.SCFDriver(n, _offsets(n, case["slice"]), halo=case["halo"], iterations=case["iterations"],
                           precision=case["precision"], full_steps=1)
        drv.V = V
        s["lam0"], s["V0"] = drv.step(A0)  # the sequence's first step, a full diagonalisation
        s["A"] = _scf_matrix(A0, g)
        s["driver"] = drv
    else:
        s["A"], s["V"] = _problem(n, g)[:2]
        s["plan"] = pf.Plan(n, _offsets(n, case["slice"]), **_options(case))
    return s


# ---------------------------------------------------------------- one pass
def run(s):
    kind = s["kind"]
    if kind == "solve":
        lam, V = s["plan"].solve(s["A"], s["V"])
    elif kind == "static":
        lam, V = s["plan"].solve_static(s["A"], s["V"])
    elif kind == "full":
        lam, V = s["plan"].solve(s["A"])
    elif kind == "scf":
        d = s["driver"]
        d.lam, d.V = s["lam0"], s["V0"]
        lam, V = d.step(s["A"])
    elif kind == "batched":
        lams, Vs = s["plan"].solve(s["A"], s["V"])
        return {"lam": lams, "V": Vs}
    elif kind == "backward":
        return {"grad": s["plan"].backward(s["lam"], s["V"], s["gl"], s["gV"], ETA)}
    else:
        Z, _ = pf.generalized_to_standard(s["A"], s["B"], s["iterations"])
        return {"Z": Z}
    return {"lam": lam, "V": V}


# ---------------------------------------------------------------- what a pass cannot do without
def _step_work(n, size, halo, iterations, power):
    """Basis change 3 n^3, overlap n^3, back-rotation 2 n^3, orthonormalisation n^3, folded-spectrum products on
    the submatrix rows, about 9 M^3 per submatrix eigenproblem; A and V_prev read, V and lambda written."""
    M = min(n, min(size, n) + 2 * halo)
    parts = -(-n // size)
    flops = 7.0 * n ** 3 + 2.0 * power * iterations * n * n * M + 9.0 * parts * M ** 3
    return 24.0 * n * n + 8.0 * n, flops


def work(case):
    kind, n = case["kind"], case["n"]
    if kind == "convert":
        return {"bytes": 24.0 * n * n, "flops": 2.0 * case["iterations"] * n ** 3}
    if kind == "backward":
        return {"bytes": 24.0 * n * n + 16.0 * n, "flops": 5.0 * n ** 3}
    if kind == "full":
        return {"bytes": 16.0 * n * n + 8.0 * n, "flops": 9.0 * n ** 3}
    args = (case["slice"], case["halo"], case["iterations"], case["power"])
    if kind == "batched":
        each = [_step_work(nb, *args) for nb in _batch_orders(case)]
        return {"bytes": sum(b for b, _ in each), "flops": sum(f for _, f in each)}
    b, f = _step_work(n, *args)
    if kind == "scf":  # and the two monitors, A V and the lower half of V^T V each
        f += 2 * 3.0 * n ** 3
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------- 64 bits
def _eigh(B):
    w, U = np.linalg.eigh(B.cpu().numpy())
    return torch.from_numpy(w).to(DEV), torch.from_numpy(U).to(DEV)


def _inv_lower(L):
    """Inverse of a lower triangular matrix, halved down to blocks that numpy inverts."""
    n = L.shape[0]
    if n <= 256:
        return torch.from_numpy(np.tril(np.linalg.inv(L.cpu().numpy()))).to(DEV)
    h = n // 2
    a, c = _inv_lower(L[:h, :h]), _inv_lower(L[h:, h:])
    top = torch.cat([a, torch.zeros(h, n - h, device=DEV, dtype=torch.float64)], 1)
    return torch.cat([top, torch.cat([-c @ (L[h:, :h] @ a), c], 1)], 0)


def _pfsm(A, V, offs, halo, iterations, power):
    n = A.shape[0]
    At = V.T @ (A @ V)
    At = 0.5 * (At + At.T)
    d = At.diagonal()
    r = At.abs().sum(1) - d.abs()
    alpha = 1.0 / float((d + r).max() - (d - r).min()) ** power
    X = torch.zeros(n, n, device=DEV, dtype=torch.float64)
    eps = torch.empty(n, device=DEV, dtype=torch.float64)
    for s, e in zip(offs[:-1], offs[1:]):
        M = min(n, e - s + 2 * halo)
        w0 = min(max(s - halo, 0), n - M)
        w, U = _eigh(At[w0:w0 + M, w0:w0 + M])
        X[w0:w0 + M, s:e] = U[:, s - w0:e - w0]
        eps[s:e] = w[s - w0:e - w0]
    for _ in range(iterations):
        Y = X
        for _ in range(power):
            Y = At @ Y - Y * eps
        X = X - alpha * Y
    L = torch.linalg.cholesky(X.T @ X)
    X = X @ _inv_lower(L).T
    lam = (X * (At @ X)).sum(0)
    top = X.abs().argmax(0)
    X = X * torch.sign(X[top, torch.arange(n, device=DEV)])
    lam, order = torch.sort(lam, stable=True)
    return lam, V @ X[:, order]


def exact(case, seed):
    g = _gen(seed)
    kind, n = case["kind"], case["n"]
    if kind == "convert":
        A, B = _problem(n, g)[0], _overlap(n, g)
        Z, d = A, B.diagonal()[:, None]
        for _ in range(case["iterations"]):
            Z = Z + (A - B @ Z) / d
        return {"Z": Z}
    if kind == "backward":
        lam, V, gl, gV = _adjoint_inputs(case, g)
        D = lam[None, :] - lam[:, None]
        T = V.T @ gV
        M = 0.5 * D / (D * D + ETA * ETA) * (T - T.T)
        M.diagonal().copy_(gl)
        G = V @ M @ V.T
        return {"grad": 0.5 * (G + G.T)}
    args = (case["halo"], case["iterations"], case["power"])
    if kind == "batched":
        out = []
        for nb in _batch_orders(case):
            A, V = _problem(nb, g)[:2]
            out.append(_pfsm(A, V, _offsets(nb, case["slice"]), *args))
        return {"lam": [x[0] for x in out], "V": [x[1] for x in out]}
    if kind == "full":
        A = _problem(n, g)[0]
        lam, V = _pfsm(A, torch.eye(n, device=DEV, dtype=torch.float64), [0, n], 0, 0, 2)
        return {"lam": lam, "V": V}
    A, V, lam, Q = _problem(n, g)
    if kind == "scf":  # from the eigenvectors of the first step's matrix, signed as its start basis is
        V = Q * torch.sign((Q * V).sum(0))
        A = _scf_matrix(A, g)
    lam, V = _pfsm(A, V, _offsets(n, case["slice"]), *args)
    return {"lam": lam, "V": V}
