"""Workloads of the library, each through its public entry points.

The library finds the lowest eigenpairs of a sectored symmetric sparse matrix
by bootstrapped block Lanczos.  A solve spends its time in a handful of calls
that a program can also make by itself: the product with H (plain CSR and
planned), the Gram-Schmidt sweep against the stored blocks (gram and block
update), the band eigensolve of a convergence check, and, for the learned
pivot, the network's inference and its training step.  Most cases are these
calls at the shapes of the bundled workloads; two are whole solves.  The whole
solves are float64: there the eigenpairs are pinned to rounding, while a
float32 basis leaves them free at the level of the residual tolerance.

listed() gives the fixed cases, draw() one more of the same ranges, prepare()
the state a program holds before the call, run() one pass, work() the bytes
and operations of a pass, exact() the same outputs in 64 bits from plain torch.
"""
import math
import os

import numpy as np
import torch

import paper_2210_15763_amd as bbl

WEIGHTS = os.path.join(os.path.dirname(os.path.abspath(bbl.__file__)), "weights",
                       "pivot_mlp_sectored.npy")
SAMPLE_KEY = 0x9E3779B97F4A7C12   # key of the training step's row sampling
M_MAX = 200                       # block cap of the whole solves


def listed():
    return [
        # The small float64 workload: pivot and solve, blocks of 0.1 ms, so
        # launches, latency and the band eigensolves decide.
        dict(name="solve_f64_n2e4_b4", kind="solve", n=20_000, R=400, q=20, p=0.7, b=4, k=4,
             n_t=2_000, tol=1e-8, planned=False),
        # An ordinary float64 solve through a plan: blocks of 0.3-1 ms.
        dict(name="solve_f64_n4e5_b8", kind="solve", n=400_000, R=1_000, q=31, p=0.7, b=8, k=8,
             n_t=4_000, tol=1e-8, planned=True),
        # The smallest product: one block of the small workload.
        dict(name="spmm_csr_f64_n2e4_b4", kind="spmm", n=20_000, R=400, q=20, p=0.7, b=4,
             dtype="f64", planned=False),
        # The plain product at the n = 2e6 workload: a matrix without the
        # locality hint, or a single product that no plan pays for.
        dict(name="spmm_csr_f32_n2e6_b8", kind="spmm", n=2_000_000, R=1_000, q=105, p=0.7, b=8,
             dtype="f32", planned=False),
        # The recurrence's product at the n = 2e6 workload.
        dict(name="spmm_plan_f32_n2e6_b8", kind="spmm", n=2_000_000, R=1_000, q=105, p=0.7, b=8,
             dtype="f32", planned=True),
        # The 16-wide product of the 400-nonzeros-a-row workload (sectors of
        # 2000 rows), on a tenth of its rows.
        dict(name="spmm_plan_f32_n2e6_b16", kind="spmm", n=2_000_000, R=2_000, q=210, p=0.7, b=16,
             dtype="f32", planned=True),
        # The far-reaching product of the 50-nonzeros-a-row workload (half the
        # entries outside the own sector), on a tenth of its rows.
        dict(name="spmm_plan_f32_n1e7_b8", kind="spmm", n=10_000_000, R=2_000, q=25, p=0.5, b=8,
             dtype="f32", planned=True),
        # One Gram-Schmidt sweep of the n = 2e6 solve against 50 stored blocks.
        dict(name="sweep_f32_n2e6_b8", kind="sweep", n=2_000_000, b=8, nblk=50, dtype="f32"),
        # The 16-wide sweep of the restarted solves, halfway through a cycle.
        dict(name="sweep_f32_n4e6_b16", kind="sweep", n=4_000_000, b=16, nblk=20, dtype="f32"),
        # A late convergence check of the n = 2e6 solve: 181 blocks of 8.
        dict(name="band_eig_N1448_kd8", kind="band", nblk=181, kd=8, k=10),
        # Inference of the learned pivot on the n = 5e6 instance.
        dict(name="mlp_forward_5e6", kind="mlp_forward", rows=5_000_000),
        # One step of the proposer's training at its default batch.
        dict(name="mlp_train_16384", kind="mlp_train", rows=1_000_000, batch=16_384),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "csr", "csr", "plan", "plan", "sweep", "sweep", "band",
                       "mlp_forward", "mlp_train"])
    if kind == "solve":
        n = _log_int(rng, 4_000, 100_000)
        b = rng.choice([4, 8])
        return dict(kind="solve", n=n, R=rng.choice([400, 500, 1_000]), q=rng.randint(15, 40),
                    p=0.7, b=b, k=rng.randint(2, b), n_t=max(400, n // 10), tol=1e-8,
                    planned=n > 50_000)
    if kind == "csr":
        return dict(kind="spmm", n=_log_int(rng, 1_000, 1_500_000), R=rng.choice([400, 1_000]),
                    q=rng.randint(15, 105), p=rng.choice([0.5, 0.7]),
                    b=rng.choice([1, 2, 3, 4, 8, 10, 12, 16]), dtype=rng.choice(["f32", "f64"]),
                    planned=False)
    if kind == "plan":
        wide = rng.random() < 0.3
        return dict(kind="spmm", n=_log_int(rng, 100_000, 1_500_000),
                    R=2_000 if wide else rng.choice([400, 1_000]), q=rng.randint(20, 150),
                    p=rng.choice([0.5, 0.7]), b=16 if wide else rng.choice([4, 8, 10]),
                    dtype="f32" if wide else rng.choice(["f32", "f32", "f64"]), planned=True)
    if kind == "sweep":
        n = _log_int(rng, 20_000, 3_000_000)
        b = rng.choice([4, 8, 10, 16])
        dt = rng.choice(["f32", "f32", "f64"])
        most = int(5.0e9 / (n * b * (4 if dt == "f32" else 8)))
        return dict(kind="sweep", n=n, b=b, nblk=_log_int(rng, 1, min(most, 180)), dtype=dt)
    if kind == "band":
        kd = rng.choice([4, 8, 10, 16])
        return dict(kind="band", nblk=_log_int(rng, 4, 640 // kd if kd == 16 else 1_448 // kd),
                    kd=kd, k=rng.randint(4, 10))
    if kind == "mlp_forward":
        return dict(kind="mlp_forward", rows=_log_int(rng, 1_000, 4_000_000))
    return dict(kind="mlp_train", rows=_log_int(rng, 100_000, 1_000_000),
                batch=_log_int(rng, 256, 65_536))


# ------------------------------------------------------------------- inputs
def _gen(seed, salt):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1_000_003 + salt) & 0x7FFFFFFFFFFF)
    return g


def _rand(g, *shape):
    return torch.rand(shape, generator=g, device="cuda", dtype=torch.float64)


def _randn(g, *shape, dtype=torch.float64):
    return torch.randn(shape, generator=g, device="cuda", dtype=dtype)


def _matrix(case, seed):
    """Sectored symmetric CSR matrix: q draws a row, a share p of them in the
    row's own sector of R rows and the rest in one of its 3 partner sectors,
    N(0, 1) values, mirrored; diagonal sorted U(-40, 40) + N(0, 0.25)."""
    n, R, q, p = case["n"], case["R"], case["q"], case["p"]
    g = _gen(seed, 1)
    S = -(-n // R)
    partners = torch.randint(0, S, (S, 3), generator=g, device="cuda")
    keys = []
    step = max(1, 100_000_000 // q)
    for lo in range(0, n, step):
        hi = min(n, lo + step)
        i = torch.arange(lo, hi, device="cuda").repeat_interleave(q)
        sec = i // R
        other = partners[sec, torch.randint(0, 3, i.shape, generator=g, device="cuda")]
        own = torch.rand(i.shape, generator=g, device="cuda") < p
        sec = torch.where(own, sec, other)
        j = torch.clamp(sec * R + torch.randint(0, R, i.shape, generator=g, device="cuda"),
                        max=n - 1)
        a, b = torch.minimum(i, j), torch.maximum(i, j)
        keys.append((a * n + b)[a != b])
        del i, sec, other, own, j, a, b
    keys = torch.unique_consecutive(torch.sort(torch.cat(keys))[0])
    off = _randn(g, keys.numel(), dtype=torch.float32)
    i, j = keys // n, keys % n
    del keys
    d = torch.arange(n, device="cuda")
    key = torch.cat([i * n + j, j * n + i, d * (n + 1)])
    diag = torch.sort(_rand(g, n) * 80.0 - 40.0)[0] + 0.5 * _randn(g, n)
    del i, j, d
    key, order = torch.sort(key)
    f64 = case.get("dtype", "f64") == "f64"
    dt = torch.float64 if f64 else torch.float32
    val = torch.cat([off.to(dt), off.to(dt), diag.to(dt)])[order]
    del order, off
    row_ptr = torch.searchsorted(key, torch.arange(n + 1, device="cuda") * n)
    col = (key % n).to(torch.int32)
    return row_ptr, col, val


def _device_csr(case, seed):
    row_ptr, col, val = _matrix(case, seed)
    return bbl.DeviceCSR(case["n"], row_ptr, col, val, case["R"] if case["planned"] else 0)


def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.float64


def _vectors(case, seed):
    """A block of roughly orthonormal vectors, as the recurrence multiplies."""
    return _randn(_gen(seed, 2), case["n"], case["b"], dtype=_dtype(case)) / math.sqrt(case["n"])


def _sweep_inputs(case, seed):
    n, b = case["n"], case["b"]
    X = _randn(_gen(seed, 3), case["nblk"], n, b, dtype=_dtype(case)) / math.sqrt(n)
    Y = _randn(_gen(seed, 4), n, b) / math.sqrt(n)
    return X, Y


def _band_inputs(case, seed):
    """Band matrix of a block recurrence (band[i, d] = T[i, i - d]): diagonal
    blocks near zero after a pivot block of low Ritz values, upper triangular
    couplings of half the spectral radius."""
    b, J = case["kd"], case["nblk"]
    g = _gen(seed, 5)
    N = b * J
    A = _randn(g, J, b, b)
    A = 0.5 * (A + A.transpose(1, 2))
    A[0] += torch.diag(torch.sort(_rand(g, b) * 7.0 - 47.0)[0])
    B = torch.triu(_randn(g, J, b, b), 1) + torch.diag_embed(22.0 + _randn(g, J, b))
    band = torch.zeros(N, b + 1, device="cuda", dtype=torch.float64)
    r = torch.arange(b, device="cuda")
    for d in range(b):                      # within the diagonal blocks
        rows = r[d:]
        band.view(J, b, b + 1)[:, rows, d] = A[:, rows, rows - d]
    for d in range(1, b + 1):               # couplings: T[J b + r, (J - 1) b + c]
        rows = r[:d] if d < b else r
        cols = rows + b - d
        if J > 1:
            band.view(J, b, b + 1)[1:, rows, d] = B[:-1, rows, cols]
    return band


def _mlp_params():
    return torch.from_numpy(np.load(WEIGHTS, allow_pickle=False).astype(np.float32)).cuda()


def _features(rows, seed):
    """Per-row features: standardised diagonal, 16 Fourier values of the row's
    sector, degree, and 10 amplitudes of unit scale."""
    g = _gen(seed, 6)
    F = torch.empty(rows, 28, device="cuda", dtype=torch.float32)
    F[:, 0] = (torch.rand(rows, generator=g, device="cuda") - 0.5) * 3.4641
    x = torch.rand(rows, 1, generator=g, device="cuda")
    w = 2.0 * math.pi * torch.pow(2.0, torch.arange(8, device="cuda"))
    F[:, 1:9] = torch.sin(x * w)
    F[:, 9:17] = torch.cos(x * w)
    F[:, 17] = 0.1 * _randn(g, rows, dtype=torch.float32)
    F[:, 18:] = _randn(g, rows, 10, dtype=torch.float32)
    return F.to(torch.bfloat16)


def _targets(F, seed):
    return 0.8 * F[:, 18:].float() + 0.6 * _randn(_gen(seed, 7), F.shape[0], 10,
                                                  dtype=torch.float32)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "solve":
        H = _device_csr(case, seed)
        b, k = case["b"], case["k"]
        plan = bbl.spmm_plan(H, b) if case["planned"] else None
        need = bbl.lanczos_workspace_bytes(case["n"], b, k, M_MAX, bbl.BBL_F64)
        return dict(case=case, seed=seed, H=H, plan=plan,
                    ws=torch.empty(need, dtype=torch.uint8, device="cuda"))
    if kind == "spmm":
        H = _device_csr(case, seed)
        V = _vectors(case, seed)
        plan = bbl.spmm_plan(H, case["b"]) if case["planned"] else None
        return dict(case=case, H=H, V=V, W=torch.empty_like(V), plan=plan)
    if kind == "sweep":
        X, Y = _sweep_inputs(case, seed)
        return dict(case=case, X=X, Y=Y, out=torch.empty_like(Y))
    if kind == "band":
        return dict(case=case, band=_band_inputs(case, seed))
    if kind == "mlp_forward":
        F = _features(case["rows"], seed).view(torch.int16)
        return dict(case=case, params=_mlp_params(), F=F)
    if kind == "mlp_train":
        F = _features(case["rows"], seed)
        tr = bbl.MlpTrainer(_mlp_params(), case["batch"], SAMPLE_KEY + int(seed))
        return dict(case=case, F=F.view(torch.int16), T=_targets(F, seed), trainer=tr)
    raise ValueError(kind)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "solve":
        # the residual norms that come with the pairs are not returned: below
        # the tolerance they are what rounding leaves
        P, _ = bbl.bootstrap_pivot(state["H"], case["n_t"], case["b"], case["tol"], m_max=M_MAX,
                                   seed=state["seed"])
        r = bbl.block_lanczos(state["H"], P, case["k"], case["tol"], m_max=M_MAX,
                              seed=state["seed"], workspace=state["ws"],
                              spmm_plan=state["plan"])
        return {"eigvals": r.eigvals, "eigvecs": r.eigvecs}
    if kind == "spmm":
        if state["plan"] is not None:
            return bbl.spmm_planned(state["plan"], state["V"], state["W"])
        return bbl.spmm(state["H"], state["V"], state["W"])
    if kind == "sweep":
        X, Y = state["X"], state["Y"]
        C = bbl.gram(X, case["nblk"], case["b"], Y)
        W = bbl.block_update(X, case["nblk"], case["b"], C, -1.0, Y, 1.0, state["out"])
        return {"C": C, "W": W}
    if kind == "band":
        theta, S, top = bbl.band_eig(state["band"], case["kd"] * case["nblk"], case["kd"],
                                     case["k"])
        return {"theta": theta, "S": S, "top": top}
    if kind == "mlp_forward":
        return bbl.mlp_forward(state["params"], state["F"])
    tr = state["trainer"]
    loss = tr.step(state["F"], state["T"], 1e-3)
    return {"params": tr.params, "m": tr.m, "v": tr.v, "loss": loss}


# -------------------------------------------------------------------- work
def _nnz(case):
    return case["n"] * (2 * case["q"] + 1)


def _csr_bytes(case, dt):
    return _nnz(case) * (4 + dt) + 8 * (case["n"] + 1)


def work(case):
    kind = case["kind"]
    if kind == "solve":
        # the matrix once, the pairs once; some ten products a wanted vector
        n, b = case["n"], case["b"]
        return {"bytes": _csr_bytes(case, 8) + 8.0 * n * case["k"],
                "flops": 10.0 * b * 2.0 * _nnz(case)}
    if kind == "spmm":
        dt = 4 if case["dtype"] == "f32" else 8
        return {"bytes": _csr_bytes(case, dt) + 2.0 * case["n"] * case["b"] * dt,
                "flops": 2.0 * _nnz(case) * case["b"]}
    if kind == "sweep":
        dt = 4 if case["dtype"] == "f32" else 8
        n, b, M = case["n"], case["b"], case["b"] * case["nblk"]
        return {"bytes": float(n) * M * dt + 16.0 * n * b + 8.0 * M * b,
                "flops": 4.0 * n * M * b}
    if kind == "band":
        N, kd, k = case["kd"] * case["nblk"], case["kd"], case["k"]
        return {"bytes": 8.0 * N * (kd + 1) + 8.0 * N * k,
                "flops": float(k) * N * (2.0 * kd * kd + 16.0 * kd)}
    mats = 28 * 128 + 2 * 128 * 128 + 128 * 10
    if kind == "mlp_forward":
        return {"bytes": case["rows"] * (56.0 + 40.0), "flops": 2.0 * mats * case["rows"]}
    return {"bytes": case["batch"] * (56.0 + 40.0) + 7.0 * 4 * bbl.MLP_PARAMS,
            "flops": 6.0 * mats * case["batch"]}


# ------------------------------------------------------------------- exact
def _csr64(row_ptr, col, val, n):
    return torch.sparse_csr_tensor(row_ptr, col.to(torch.int64), val.to(torch.float64),
                                   size=(n, n), device="cuda")


def _orthonormal(W):
    for _ in range(2):
        L = torch.linalg.cholesky(W.T @ W)
        W = torch.linalg.solve_triangular(L, W.T, upper=False).T.contiguous()
    return W


def _exact_solve(case, seed):
    """Lowest k pairs by a plain block Lanczos run to rounding."""
    n, k = case["n"], case["k"]
    H = _csr64(*_matrix(case, seed), n)
    w = 16
    most = min(160, n // w)
    V = torch.empty(n, (most + 1) * w, device="cuda", dtype=torch.float64)
    T = torch.zeros(most * w, most * w, device="cuda", dtype=torch.float64)
    V[:, :w] = _orthonormal(_randn(_gen(seed, 8), n, w))
    for j in range(most):
        Q = V[:, :(j + 1) * w]
        W = H @ V[:, j * w:(j + 1) * w].contiguous()
        h = torch.zeros((j + 1) * w, w, device="cuda", dtype=torch.float64)
        for _ in range(2):
            c = Q.T @ W
            W = W - Q @ c
            h += c
        T[:(j + 1) * w, j * w:(j + 1) * w] = h
        Qn = _orthonormal(W)
        for _ in range(2):
            Qn = _orthonormal(Qn - Q @ (Q.T @ Qn))
        V[:, (j + 1) * w:(j + 2) * w] = Qn
        if (j + 1) % 10 == 0 or j == most - 1:
            M = T[:(j + 1) * w, :(j + 1) * w].cpu().numpy()
            M = np.triu(M) + np.triu(M, 1).T
            lam, s = np.linalg.eigh(M)
            last = torch.from_numpy(np.ascontiguousarray(s[-w:, :k])).cuda()
            res = torch.linalg.norm((Qn.T @ W) @ last, dim=0).max().item()
            if res <= 1e-11 * abs(lam).max():
                break
    else:
        return None
    X = Q @ torch.from_numpy(np.ascontiguousarray(s[:, :k])).cuda()
    X = X / torch.linalg.norm(X, dim=0)
    big = X.abs().argmax(dim=0)
    X = X * torch.sign(X[big, torch.arange(k, device="cuda")])
    return {"eigvals": lam[:k].copy(), "eigvecs": X}


def _net(params):
    p = params.double()
    out, o = [], 0
    for shape in ((128, 28), (128,), (128, 128), (128,), (128, 128), (128,), (10, 128), (10,)):
        m = math.prod(shape)
        out.append(p[o:o + m].reshape(shape))
        o += m
    return out


def _exact_forward(params, F):
    W1, b1, W2, b2, W3, b3, W4, b4 = _net(params)
    x = F.double()
    h = torch.relu(x @ W1.T + b1)
    h = torch.relu(h @ W2.T + b2)
    h = torch.relu(h @ W3.T + b3)
    return h @ W4.T + b4 + x[:, 18:]


def _philox(c, key):
    """Philox4x32-10 (Salmon et al., SC 2011) on uint64 arrays of 32-bit words."""
    m32 = np.uint64(0xFFFFFFFF)
    k0, k1 = np.uint64(key & 0xFFFFFFFF), np.uint64((key >> 32) & 0xFFFFFFFF)
    for r in range(10):
        if r:
            k0 = (k0 + np.uint64(0x9E3779B9)) & m32
            k1 = (k1 + np.uint64(0xBB67AE85)) & m32
        p0, p1 = np.uint64(0xD2511F53) * c[0], np.uint64(0xCD9E8D57) * c[2]
        c = [(p1 >> np.uint64(32)) ^ c[1] ^ k0, p1 & m32, (p0 >> np.uint64(32)) ^ c[3] ^ k1,
             p0 & m32]
    return c


def _exact_train(case, seed):
    F = _features(case["rows"], seed)
    T = _targets(F, seed)
    r = np.arange(case["batch"], dtype=np.uint64)
    z = np.zeros_like(r)
    c = _philox([r, z, z + np.uint64(1), z + np.uint64(12)],
                (SAMPLE_KEY + int(seed)) & (2**64 - 1))
    idx = ((c[0] << np.uint64(32)) | c[1]) % np.uint64(case["rows"])
    idx = torch.from_numpy(idx.astype(np.int64)).cuda()
    p = _mlp_params().double().requires_grad_(True)
    d = _exact_forward(p, F[idx]) - T[idx].double()
    loss = (d * d).mean()
    g, = torch.autograd.grad(loss, p)
    m, v = 0.1 * g, 0.001 * g * g
    new = p.detach() - 1e-3 * (m / 0.1) / (torch.sqrt(v / 0.001) + 1e-8)
    return {"params": new, "m": m, "v": v, "loss": loss.detach().reshape(1)}


def exact(case, seed):
    kind = case["kind"]
    if kind == "solve":
        return _exact_solve(case, seed)
    if kind == "spmm":
        n = case["n"]
        H = _csr64(*_matrix(case, seed), n)
        return H @ _vectors(case, seed).double()
    if kind == "sweep":
        X, Y = _sweep_inputs(case, seed)
        C = torch.cat([x.double().T @ Y for x in X])
        W = Y.clone()
        for x, c in zip(X, C.reshape(case["nblk"], case["b"], -1)):
            W -= x.double() @ c
        return {"C": C, "W": W}
    if kind == "band":
        # the vectors' signs are free, so only the values have a reference
        band = _band_inputs(case, seed).cpu().numpy()
        N, kd = case["kd"] * case["nblk"], case["kd"]
        T = np.zeros((N, N))
        for d in range(min(kd, N - 1) + 1):
            i = np.arange(d, N)
            T[i, i - d] = T[i - d, i] = band[d:, d]
        lam = np.linalg.eigvalsh(T)
        return {"theta": lam[:case["k"]].copy(), "S": None, "top": float(lam[-1])}
    if kind == "mlp_forward":
        F = _features(case["rows"], seed)
        p = _mlp_params()
        return torch.cat([_exact_forward(p, F[a:a + 500_000])
                          for a in range(0, F.shape[0], 500_000)])
    return _exact_train(case, seed)
