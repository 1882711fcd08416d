"""Performance cases of the AltGDmin-LR+S library on one GPU.

Each case is work that a program using this library has it do, through the entry
points of ``paper_2311_03824_amd.altgdmin``:

  * ``solve``: one ``altgdmin_solve`` call on a Gaussian (or Philox-generated)
    problem: initialisation, graph capture, ``iters`` GDmin iterations, results;
  * ``serve``: a round of the serving loop: ``altgdmin_init`` of several problems
    of mixed sizes and A forms, batched ``altgdmin_step_many``, one status poll;
  * ``fourier``: one ``altgdmin_solve`` call on partial Fourier frames;
  * ``subspace``: the spectral initialisation's subspace iteration on its own.

``start`` says where the subspace estimate comes from.  "cold": the library's own
spectral initialisation (Alg. 1).  "auto": the same with the automatic rank of
Sec. 2.6.  "warm": the subspace is known to 1e-4 from an earlier batch of columns
(``U_start``, no subspace iteration) and ``eta_c`` is scaled to that accuracy, as
the fixed step of Sec. 2.6 asks for; B and S of the new columns are recovered.

Inputs follow the protocol of Sec. 3 (U* an orthonormalised Gaussian, B* i.i.d.
Gaussian, supports drawn uniformly, noise-free y) with gross outliers: S* values of
magnitude U[5, 15].
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2311_03824_amd import altgdmin as lib
from paper_2311_03824_amd import instances

WARM = 1e-4          # accuracy of a warm start's subspace
POWER_TOL = 1e-4     # subspace accuracy asked of a cold start: GDmin contracts from there
RANK_ENERGY = 0.57   # energy fraction asked of the automatic rank
TAU0, TAU = 10, 3    # IHT iterations of the initialisation and per GDmin iteration (library defaults)
CACHE_BYTES = 256 << 20   # the GPU's last-level cache


def listed():
    """The listed cases; the comments say what each stands for."""
    def solve(name, form, n, q, m, r, rho, iters, start):
        return {"name": name, "kind": "solve", "form": form, "n": n, "q": q, "m": m, "r": r, "rho": rho,
                "iters": iters, "start": start}

    def fourier(name, n1, n2, q, m, r, rho, iters, start):
        return {"name": name, "kind": "fourier", "n1": n1, "n2": n2, "q": q, "m": m, "r": r, "rho": rho,
                "iters": iters, "start": start}

    return [
        # the exact-recovery size: a whole solve from scratch, all launches and latency
        solve("solve_100", "f32", 100, 100, 40, 2, 2, 60, "cold"),
        # the mid-size throughput shape, A exact in two BF16 planes
        solve("solve_600_bf16x2", "bf16x2", 600, 600, 250, 4, 30, 40, "warm"),
        # the benchmark shape, FP32 plane and mixed BF16 form
        solve("solve_1000", "f32", 1000, 1000, 400, 10, 50, 40, "warm"),
        solve("solve_1000_mixed", "mixed", 1000, 1000, 400, 10, 50, 40, "warm"),
        # one GPU's share of the benchmark shape split by columns over eight
        solve("solve_shard_125", "f32", 1000, 125, 400, 10, 50, 40, "warm"),
        # odd sizes with A regenerated in the kernels (problems whose A is not stored)
        solve("solve_philox_777", "philox", 777, 333, 301, 7, 23, 20, "warm"),
        # 128 x 128 frames: the longest columns
        solve("solve_frames_128", "f32", 16384, 100, 1000, 10, 40, 10, "warm"),
        # rank chosen by the energy rule
        solve("solve_auto_rank", "f32", 300, 200, 120, 2, 2, 20, "auto"),
        # a round of the serving loop over eight requests of mixed sizes and forms
        {"name": "serve_8", "kind": "serve", "count": 8, "sizes": 28, "iters": 20},
        # the 96 x 96 partial Fourier workload (FFT path)
        fourier("fourier_96", 96, 96, 64, 1536, 6, 92, 40, "warm"),
        # the Table 1 shape: small frames through direct DFTs, from scratch
        fourier("fourier_20", 20, 20, 400, 100, 4, 2, 10, "cold"),
        # the spectral start of the benchmark shape on its own
        {"name": "subspace_1000", "kind": "subspace", "n": 1000, "q": 1000, "r": 10, "iters": 100},
    ]


def _log_int(rng: random.Random, lo: float, hi: float) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _gaussian_sizes(rng: random.Random, n_lo, n_hi, q_lo, q_hi, a_max):
    """n, q, m, r, rho of a recoverable problem whose FP32 A takes at most a_max bytes."""
    n = _log_int(rng, n_lo, n_hi)
    m = min(1024, max(40, int(round(n * rng.uniform(0.3, 0.5)))))
    q = max(q_lo, min(_log_int(rng, q_lo, q_hi), int(a_max / (4 * n * m))))
    r = max(2, min(_log_int(rng, 2, 16), m // 12))
    rho = max(2, min(int(round(n * rng.uniform(0.005, 0.05))), m // 10))
    return n, q, m, r, rho


def draw(rng: random.Random) -> dict:
    """One more case of the ranges the listed ones stand for."""
    kind = rng.choice(("solve", "solve", "solve", "long", "small", "serve", "frames", "fourier", "subspace"))
    if kind == "solve":
        n, q, m, r, rho = _gaussian_sizes(rng, 200, 4000, 100, 1200, 1.5e9)
        return {"kind": "solve", "form": rng.choice(("f32", "f32", "mixed", "bf16x2", "philox")), "n": n, "q": q,
                "m": m, "r": r, "rho": rho, "iters": rng.randint(10, 30), "start": "warm"}
    if kind == "long":
        n, m = _log_int(rng, 5000, 13000), rng.randint(600, 1024)
        return {"kind": "solve", "form": rng.choice(("f32", "mixed")), "n": n, "q": int(rng.uniform(1.2e9, 3e9) / (4 * n * m)),
                "m": m, "r": rng.randint(2, 12), "rho": rng.randint(5, m // 25), "iters": rng.randint(5, 10),
                "start": "warm"}
    if kind == "small":
        m = rng.randint(40, 120)
        n = rng.randint(2 * m, 3 * m)
        start = rng.choice(("cold", "auto"))
        return {"kind": "solve", "form": "f32", "n": n, "q": rng.randint(150, 250), "m": m,
                "r": 2 if start == "auto" else rng.randint(2, 2 + m // 40), "rho": 2, "iters": rng.randint(20, 60),
                "start": start}
    if kind == "serve":
        return {"kind": "serve", "count": rng.randint(4, 8), "sizes": rng.randrange(1 << 20),
                "iters": rng.randint(10, 20)}
    if kind == "frames":
        m = rng.randint(900, 2048)
        return {"kind": "fourier", "n1": 96, "n2": 96, "q": rng.randint(16, 64), "m": m, "r": rng.randint(2, 8),
                "rho": rng.randint(20, m // 16), "iters": rng.randint(20, 40), "start": "warm"}
    if kind == "fourier":
        n1, n2 = rng.choice(((1, rng.randint(200, 600)), (rng.randint(12, 40), rng.randint(12, 40))))
        n = n1 * n2
        m = rng.randint(n // 4, n // 2)
        return {"kind": "fourier", "n1": n1, "n2": n2, "q": _log_int(rng, 50, 400), "m": m, "r": rng.randint(2, 4),
                "rho": max(2, m // 24), "iters": rng.randint(10, 30), "start": "warm"}
    return {"kind": "subspace", "n": _log_int(rng, 100, 4000), "q": _log_int(rng, 100, 2000),
            "r": rng.randint(2, 16), "iters": 100}


# ---------------------------------------------------------------- inputs

def _gen(seed: int, tag: int = 0) -> torch.Generator:
    return torch.Generator(device="cuda").manual_seed((int(seed) * 64 + tag) % (1 << 62))


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float64)


def _supports(g, q, n, rho):
    keys = torch.rand(q, n, generator=g, device="cuda")
    return torch.sort(torch.topk(keys, rho, dim=1).indices, dim=1).values


def _magnitudes(g, q, rho):
    return 5.0 + 10.0 * torch.rand(q, rho, generator=g, device="cuda", dtype=torch.float64)


def _columns(q, bytes_each, budget=1 << 30):
    """Ranges of columns whose FP64 working set stays within the budget."""
    step = max(1, int(budget // bytes_each))
    return [(k, min(q, k + step)) for k in range(0, q, step)]


def _orth(X):
    """Q of the thin QR with a positive (real) diagonal R."""
    Q, R = torch.linalg.qr(X.cpu())   # a few columns: the host's factorisation
    d = torch.diagonal(R)
    return (Q * (d / d.abs())).cuda()


def _gaussian_inputs(case, seed):
    """A (and its BF16 planes), Y, and the start block of a Gaussian problem, on the GPU."""
    n, q, m, r, rho, form = (case[k] for k in ("n", "q", "m", "r", "rho", "form"))
    g = _gen(seed)
    U = _orth(_normal(g, n, r))
    X = _normal(g, q, r) @ U.T
    supp = _supports(g, q, n, rho)
    sign = torch.where(torch.rand(q, rho, generator=g, device="cuda") < 0.5, -1.0, 1.0).double()
    X.scatter_add_(1, supp, sign * _magnitudes(g, q, rho))
    start = U + WARM / math.sqrt(n) * _normal(g, n, r) if case["start"] == "warm" else _normal(g, n, r)
    d = {"start": start.float().contiguous(), "a_seed": int(seed) % (1 << 31) + 7}
    lda = (m + 7) // 8 * 8
    A = torch.zeros(q, n, lda, device="cuda")
    if form == "philox":
        d["table"] = torch.from_numpy(instances.normal_table()).cuda()
        lib.altgdmin_op_philox_fill(d["a_seed"], d["table"], q, n, m, A)
    else:
        for k0, k1 in _columns(q, 4 * n * lda):
            a = torch.randn(k1 - k0, n, m, generator=g, device="cuda")
            if form != "f32":
                hi = a.bfloat16()
                a = hi.float() + (a - hi.float()).bfloat16().float()
            A[k0:k1, :, :m] = a
    Y = torch.empty(q, m, device="cuda")
    for k0, k1 in _columns(q, 8 * n * lda):
        Y[k0:k1] = torch.bmm(X[k0:k1, None, :], A[k0:k1].double())[:, 0, :m].float()
    d.update(A=A, Y=Y)
    if form in ("bf16x2", "mixed"):
        d["hi"] = A.bfloat16()
        d["lo"] = (A - d["hi"].float()).bfloat16()
    return d


def _complex_normal(g, *shape):
    return torch.complex(_normal(g, *shape), _normal(g, *shape)) / math.sqrt(2.0)


def _fourier_inputs(case, seed):
    n1, n2, q, m, r, rho = (case[k] for k in ("n1", "n2", "q", "m", "r", "rho"))
    n = n1 * n2
    g = _gen(seed)
    U = _orth(_complex_normal(g, n, r))
    X = _complex_normal(g, q, r) @ U.T
    supp = _supports(g, q, n, rho)
    phase = 2.0 * math.pi * torch.rand(q, rho, generator=g, device="cuda", dtype=torch.float64)
    X.scatter_add_(1, supp, torch.polar(_magnitudes(g, q, rho), phase))
    mask = _supports(g, q, n, m)
    F = torch.fft.fft2(X.reshape(q, n1, n2), norm="ortho").reshape(q, n)
    start = (U + WARM / math.sqrt(n) * _complex_normal(g, n, r) if case["start"] == "warm"
             else _complex_normal(g, n, r))
    return {"mask": mask.int().contiguous(), "Y": torch.gather(F, 1, mask).to(torch.complex64).contiguous(),
            "start": start.to(torch.complex64).contiguous()}


def _subspace_inputs(case, seed):
    """A low-rank matrix in noise of a tenth of its smallest singular value, as L_0 of a
    problem with enough measurements is, and a Gaussian start block."""
    n, q, r = case["n"], case["q"], case["r"]
    g = _gen(seed)
    L = _normal(g, q, r) @ _orth(_normal(g, n, r)).T
    gap = max(math.sqrt(q) - math.sqrt(r), 0.3 * math.sqrt(q))
    L = L + 0.3 * gap / (math.sqrt(n) + math.sqrt(q)) * _normal(g, q, n)
    return {"L0t": L.float().contiguous(), "start": _normal(g, n, r).float().contiguous()}


def _serve_sizes(case):
    """The requests of a serving round: sizes within the serving workload's ranges, the
    stored form of A alternating between the FP32 plane and the mixed BF16 planes."""
    rng = random.Random(case["sizes"])
    reqs = []
    for i in range(case["count"]):
        n, q, m, r, rho = _gaussian_sizes(rng, 256, 2000, 128, 1000, 5e8)
        reqs.append({"form": "mixed" if i % 2 else "f32", "n": n, "q": q, "m": m, "r": r, "rho": rho,
                     "iters": case["iters"], "start": "warm"})
    return reqs


# ---------------------------------------------------------------- prepare and run

def _rank_budget(case):
    return max(1, min(case["n"], case["q"], case["m"], 160) // 10)


def _params(case):
    kw = {"t_max": case["iters"], "tau0": TAU0, "tau": TAU}
    if case["start"] == "warm":
        kw.update(power_iters=0, eta_c=0.5 * WARM)
    else:
        kw.update(power_iters=100, power_tol=POWER_TOL, rank_energy=RANK_ENERGY)
    if case.get("form") == "mixed":
        kw["flags"] = lib.FLAG_BF16_MIXED
    return lib.default_params(**kw)


def _outputs(n, q, r, rho, dtype):
    return {"U": torch.empty(n, r, dtype=dtype, device="cuda"), "Bt": torch.empty(q, r, dtype=dtype, device="cuda"),
            "S_idx": torch.empty(q, rho, dtype=torch.int32, device="cuda"),
            "S_val": torch.empty(q, rho, dtype=dtype, device="cuda")}


def _workspace(prob, par):
    return torch.empty(lib.altgdmin_workspace_bytes(prob, par), dtype=torch.uint8, device="cuda")


def _gaussian_state(case, seed):
    d = _gaussian_inputs(case, seed)
    r = 0 if case["start"] == "auto" else case["r"]
    start = None if case["start"] == "auto" else d["start"]
    if case["form"] == "philox":
        del d["A"]
        prob = lib.make_problem(None, d["Y"], r, case["rho"], U_start=start, m=case["m"], philox_seed=d["a_seed"],
                                normal_table=d["table"], n=case["n"])
    elif case["form"] == "f32":
        prob = lib.make_problem(d["A"], d["Y"], r, case["rho"], U_start=start, m=case["m"])
    else:
        del d["A"]
        prob = lib.make_problem(d["hi"].view(torch.int16), d["Y"], r, case["rho"], A_lo=d["lo"].view(torch.int16),
                                U_start=start, m=case["m"])
    par = _params(case)
    # the automatic rank may pick any r up to a tenth of the smallest size (and at most 16)
    r_out = _rank_budget(case) if case["start"] == "auto" else case["r"]
    out = _outputs(case["n"], case["q"], r_out, case["rho"], torch.float32)
    return {"kind": "solve", "data": d, "prob": prob, "par": par, "ws": _workspace(prob, par), "out": out,
            "auto": case["start"] == "auto"}


def prepare(case: dict, seed: int):
    """The problem, its workspace and result buffers, as a program holds them before a call."""
    if case["kind"] == "solve":
        return _gaussian_state(case, seed)
    if case["kind"] == "fourier":
        d = _fourier_inputs(case, seed)
        prob = lib.make_fourier_problem(d["mask"], d["Y"], case["n1"], case["n2"], case["r"], case["rho"], d["start"])
        par = _params(case)
        return {"kind": "solve", "data": d, "prob": prob, "par": par, "ws": _workspace(prob, par), "auto": False,
                "out": _outputs(prob.n, prob.q, case["r"], case["rho"], torch.complex64)}
    if case["kind"] == "serve":
        jobs = [_gaussian_state(c, seed * 16 + i) for i, c in enumerate(_serve_sizes(case))]
        return {"kind": "serve", "jobs": jobs, "iters": case["iters"], "group": None}
    d = _subspace_inputs(case, seed)
    n, q, r = case["n"], case["q"], case["r"]
    return {"kind": "subspace", "data": d, "r": r, "iters": case["iters"],
            "scratch": torch.empty(lib.altgdmin_op_scratch_bytes(n, q, r) + 256, dtype=torch.uint8, device="cuda"),
            "U": torch.empty(n, r, device="cuda"), "count": torch.zeros(1, dtype=torch.int32, device="cuda")}


def run(state):
    """One pass through the public entry points."""
    if state["kind"] == "solve":
        o = state["out"]
        _, rep = lib.altgdmin_solve(state["prob"], state["par"], state["ws"], o["U"], o["Bt"], o["S_idx"], o["S_val"])
        if not state["auto"]:
            return o
        r, n, q = rep["rank"], state["prob"].n, state["prob"].q   # U and B have the columns of the rank chosen
        return {"U": o["U"].view(-1)[: n * r].view(n, r), "Bt": o["Bt"].view(-1)[: q * r].view(q, r),
                "S_idx": o["S_idx"], "S_val": o["S_val"], "rank": r}
    if state["kind"] == "serve":
        jobs = state["jobs"]
        hs = [lib.altgdmin_init(j["prob"], j["par"], j["ws"]) for j in jobs]
        need = lib.altgdmin_group_bytes(hs)
        if state["group"] is None or state["group"].numel() < need:
            state["group"] = torch.empty(need, dtype=torch.uint8, device="cuda")
        lib.altgdmin_step_many(hs, state["iters"], state["group"])
        lib.altgdmin_status_many(hs)
        for h, j in zip(hs, jobs):
            o = j["out"]
            lib.altgdmin_get(h, o["U"], o["Bt"], o["S_idx"], o["S_val"])
            lib.altgdmin_destroy(h)
        return [j["out"] for j in jobs]
    d = state["data"]
    lib.altgdmin_op_subspace(d["L0t"], state["r"], d["start"], state["iters"], POWER_TOL, state["U"], state["count"],
                             scratch=state["scratch"])
    return {"U": state["U"], "iterations": state["count"]}


# ---------------------------------------------------------------- work

def _solve_work(n, q, m, r, rho, iters, a_bytes, out_bytes):
    """A is read once by the initialisation and once per GDmin iteration (U changes in
    between); an A that fits in the last-level cache is read once in all.  The products
    of Alg. 1: tau0 IHT steps on all columns, then per iteration A_k U and its Gram,
    tau steps on the support, A_k^T r_k and the gradient."""
    reads = 1 if a_bytes <= CACHE_BYTES else 1 + iters
    flops = q * (TAU0 * 2.0 * m * n + iters * (2.0 * m * n * (r + 1) + TAU * 4.0 * m * rho + 2.0 * m * r * r
                                               + 2.0 * n * r))
    return {"bytes": reads * a_bytes + 4.0 * q * m + out_bytes, "flops": flops}


def work(case: dict) -> dict:
    if case["kind"] == "serve":
        ws = [work(dict(c, kind="solve")) for c in _serve_sizes(case)]
        return {"bytes": sum(w["bytes"] for w in ws), "flops": sum(w["flops"] for w in ws)}
    if case["kind"] == "solve":
        n, q, m, r, rho = (case[k] for k in ("n", "q", "m", "r", "rho"))
        a = 0.0 if case["form"] == "philox" else 4.0 * q * n * m
        return _solve_work(n, q, m, r, rho, case["iters"], a, 4.0 * (n * r + q * r + 2 * q * rho))
    if case["kind"] == "fourier":
        n1, n2, q, m, r, rho = (case[k] for k in ("n1", "n2", "q", "m", "r", "rho"))
        n = n1 * n2
        fft = 5.0 * n * math.log2(n)
        per = case["iters"] * ((2 * TAU + 2) * fft + 8.0 * m * r * (r + 2 * TAU + 3) + 8.0 * n * r) + 2 * TAU0 * fft
        return {"bytes": 12.0 * q * m + 8.0 * (n * r + q * r + 1.5 * q * rho), "flops": q * per}
    n, q, r = case["n"], case["q"], case["r"]
    return {"bytes": 4.0 * n * q + 8.0 * n * r, "flops": 10 * 4.0 * n * q * r}


# ---------------------------------------------------------------- FP64 values

def _keep(V, rho):
    """HardThreshold's support: the rho entries of largest magnitude, lower index on ties."""
    idx = torch.sort(V.abs(), dim=1, descending=True, stable=True).indices[:, :rho]
    return torch.zeros(V.shape, dtype=torch.bool, device=V.device).scatter_(1, idx, True)


def _iht(fwd, fwd_t, adj, z, proj, S, T, rho, tau):
    """tau steps of Alg. 2 with the normalised step on the current support."""
    for _ in range(tau):
        g = adj(proj(fwd(S) - z))
        if T is None:
            T = _keep(g, rho)
        gT = g * T
        w = proj(fwd_t(gT))
        ww = (w.abs() ** 2).sum(1)
        mu = torch.where(ww > 0, (gT.abs() ** 2).sum(1) / ww, torch.zeros_like(ww))
        V = S - mu[:, None] * g
        T = _keep(V, rho)
        S = V * T
    return S, T


def _qr_power(L0t, U, iters, tol):
    """Subspace iteration; returns the block and the number of steps."""
    for it in range(1, iters + 1):
        V = _orth(L0t.T @ (L0t.conj() @ U))
        sd = torch.linalg.norm(V - U @ (U.conj().T @ V))
        U = V
        if sd <= tol:
            return U, it
    return U, iters


def _altgdmin64(chunks, ops, n, q, r, rho, iters, start, warm, Y, budget=0):
    """Alg. 1 in FP64.  ops(k0, k1) gives the products of a range of columns: A s, the
    step-length product, A^H v and A U."""
    dt = Y.dtype
    S = torch.zeros(q, n, dtype=dt, device="cuda")
    T = torch.zeros(q, n, dtype=torch.bool, device="cuda")
    L0t = torch.zeros(q, n, dtype=dt, device="cuda")
    for k0, k1 in chunks:
        fwd, fwd_t, adj, _ = ops(k0, k1)
        S[k0:k1], T[k0:k1] = _iht(fwd, fwd_t, adj, Y[k0:k1], lambda v: v, S[k0:k1], None, rho, TAU0)
        if not warm:
            L0t[k0:k1] = adj(Y[k0:k1] - fwd(S[k0:k1]))
    if budget:   # automatic rank: the energy rule on the leading singular values of L_0
        energy = torch.cumsum(torch.linalg.svdvals(L0t.cpu())[:budget] ** 2, 0)
        r = int((energy < RANK_ENERGY * energy[-1]).sum()) + 1
    U = _orth(start[:, :r])
    if not warm:
        U, _ = _qr_power(L0t, U, 100, POWER_TOL)
    eta, U_fit, B = None, U, torch.zeros(q, U.shape[1], dtype=dt, device="cuda")
    for _ in range(iters):
        grad = torch.zeros_like(U)
        for k0, k1 in chunks:
            fwd, fwd_t, adj, au = ops(k0, k1)
            P = au(U)
            Ph = P.conj().transpose(1, 2).contiguous()
            Gi = torch.linalg.inv(torch.bmm(Ph, P).cpu()).cuda()

            def coef(v):
                return torch.bmm(Gi, torch.bmm(Ph, v[:, :, None]))

            def proj(v):
                return v - torch.bmm(P, coef(v))[:, :, 0]

            S[k0:k1], T[k0:k1] = _iht(fwd, fwd_t, adj, Y[k0:k1], proj, S[k0:k1], T[k0:k1], rho, TAU)
            e = Y[k0:k1] - fwd(S[k0:k1])
            b = coef(e)
            B[k0:k1] = b[:, :, 0]
            H = adj(torch.bmm(P, b)[:, :, 0] - e)
            grad += H.T @ B[k0:k1].conj()
        if eta is None:
            eta = (0.5 * WARM if warm else 0.14) / float(torch.linalg.matrix_norm(grad.cpu(), 2))
        U_fit = U
        U = _orth(U - eta * grad)
    idx = torch.sort(torch.topk(T.to(torch.uint8), rho, dim=1).indices, dim=1).values
    return {"U": U_fit, "Bt": B, "S_idx": None, "S_val": torch.gather(S, 1, idx)}


def _gaussian64(case, seed):
    n, q, m, r, rho = (case[k] for k in ("n", "q", "m", "r", "rho"))
    d = _gaussian_inputs(case, seed)

    def ops(k0, k1):
        A = d["A"][k0:k1, :, :m].double()
        At = d["hi"][k0:k1, :, :m].double() if case["form"] == "mixed" else A
        return (lambda s: torch.bmm(s[:, None, :], A)[:, 0], lambda s: torch.bmm(s[:, None, :], At)[:, 0],
                lambda v: torch.bmm(At, v[:, :, None])[:, :, 0],
                lambda U: torch.stack([a.T @ U for a in A]))

    out = _altgdmin64(_columns(q, 16 * n * m), ops, n, q, r, rho, case["iters"], d["start"].double(),
                      case["start"] == "warm", d["Y"].double(), _rank_budget(case) if case["start"] == "auto" else 0)
    if case["start"] == "auto":   # the basis of U depends on the rank estimate's block: only S is fixed by the data
        out.update(U=None, Bt=None, rank=None)
    return out


def _fourier64(case, seed):
    n1, n2, q, m, r, rho = (case[k] for k in ("n1", "n2", "q", "m", "r", "rho"))
    n = n1 * n2
    d = _fourier_inputs(case, seed)
    mask = d["mask"].long()

    def ops(k0, k1):
        mk = mask[k0:k1]

        def fwd(s):
            return torch.gather(torch.fft.fft2(s.reshape(-1, n1, n2), norm="ortho").reshape(-1, n), 1, mk)

        def adj(v):
            f = torch.zeros(k1 - k0, n, dtype=v.dtype, device="cuda").scatter_(1, mk, v)
            return torch.fft.ifft2(f.reshape(-1, n1, n2), norm="ortho").reshape(-1, n)

        def au(U):
            FU = torch.fft.fft2(U.T.reshape(r, n1, n2), norm="ortho").reshape(r, n).T.contiguous()
            return FU[mk]

        return fwd, fwd, adj, au

    return _altgdmin64([(0, q)], ops, n, q, r, rho, case["iters"], d["start"].to(torch.complex128),
                       case["start"] == "warm", d["Y"].to(torch.complex128))


def exact(case: dict, seed: int):
    """What run() returns, computed in 64 bits by torch."""
    if case["kind"] == "solve":
        return _gaussian64(case, seed)
    if case["kind"] == "fourier":
        return _fourier64(case, seed)
    if case["kind"] == "serve":
        return [_gaussian64(c, seed * 16 + i) for i, c in enumerate(_serve_sizes(case))]
    d = _subspace_inputs(case, seed)
    U, _ = _qr_power(d["L0t"].double(), _orth(d["start"].double()), case["iters"], POWER_TOL)
    return {"U": U, "iterations": None}
