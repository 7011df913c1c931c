"""The work that programs have this library do, as measurable cases.

A trajectory optimizer calls the library once per outer iteration: it hands over the linearised dynamics and cost
blocks of a batch of problems, has S and the preconditioner built, solves S lambda = gamma and recovers the primal
step.  The cases are such calls from one short problem to the ragged 4096-problem batch, in both storage precisions,
with each kind of preconditioner, with matrices given by their blocks, with the learned start, and one training step
of the network behind it.  Inputs follow the recipe of ``paper_2309_06427_amd.inputs`` (the same distributions, drawn
on the GPU).  A handle's sizes are fixed by the case, its numbers by the seed.

Solves return lambda, the iteration counts and the statuses.  The achieved residual and the number of refinement steps
stay in their buffers: below the tolerance the residual is rounding noise of the iterates.
"""
from __future__ import annotations

import math
import types

import numpy as np
import torch

from paper_2309_06427_amd import _lib, inputs
from paper_2309_06427_amd.solver import BatchSolver
from paper_2309_06427_amd.train_warmstart import weights_path
from paper_2309_06427_amd.warmstart import WarmStartNet

DEV = "cuda"
HIDDEN = 128
F64 = torch.float64

# Fields of a case: kind (step: build + solve; kkt: build, right-hand side, solve, recovery; kkt_calls: the two KKT
# calls on a built handle; blocks: S given by blocks, build + solve; warm: build, network start, solve with fallback;
# train: loss, gradient and one Adam step), P problems with N uniform on [n_lo, n_hi] and nx from the list in nx,
# nu = floor(nu_frac nx), sizes: seed of the size draw, pc, precision, tol, cond: 0 for the Wishart Q_k, else the
# largest condition number of the log-uniform recipe.
_BASE = dict(kind="step", P=1, n_lo=50, n_hi=50, nx="14", nu_frac=0.5, sizes=1, pc="sym", precision="fp32_refine64",
             tol=1e-6, cond=0.0)


def _case(name=None, **over):
    c = dict(_BASE, **over)
    return c if name is None else dict(c, name=name)


def listed():
    return [
        # one short problem, as a controller that re-plans at a fixed rate solves it: latency
        _case("single_n50_nx14_fp64", precision="fp64", tol=1e-8),
        # one long horizon with a large state: all of the chip for one problem
        _case("single_n512_nx36", n_lo=512, n_hi=512, nx="36", nu_frac=0.34, cond=1e4),
        # a handful of problems in a serving loop that may not allocate
        _case("serve_16", kind="serve", P=16, n_lo=32, n_hi=256, nx="6,14,26", sizes=2),
        # the headline batch: every state size, ragged horizons
        _case("ragged_4096", P=4096, n_lo=32, n_hi=256, nx="6,14,26", sizes=3),
        # a quarter of it with the polynomial preconditioner of degree 3
        _case("ragged_1024_poly3", P=1024, n_lo=32, n_hi=256, nx="6,14,26", sizes=4, pc="poly3"),
        # ill-conditioned costs: all in FP64, and FP32 with FP64 refinement
        _case("cond1e6_1024_fp64", P=1024, n_lo=128, n_hi=128, nx="26", nu_frac=0.47, precision="fp64", cond=1e6),
        _case("cond1e6_1024_refine64", P=1024, n_lo=128, n_hi=128, nx="26", nu_frac=0.47, cond=1e6),
        # a whole KKT step of an optimizer's iteration, an odd number of problems
        _case("kkt_step_517", kind="kkt", P=517, n_lo=32, n_hi=256, nx="6,14,26", sizes=6),
        # the KKT calls alone: new cost gradients on an unchanged matrix
        _case("kkt_calls_4096", kind="kkt_calls", P=4096, n_lo=32, n_hi=256, nx="6,14,26", sizes=7),
        # any SPD block-tridiagonal matrix, state sizes outside the compiled ones among them
        _case("blocks_256_add", kind="blocks", P=256, n_lo=1, n_hi=90, nx="3,6,9,14,20,26,36", sizes=8, pc="add",
              precision="fp64", tol=1e-10),
        # the trained network's start in front of the solve
        _case("warm_1024", kind="warm", P=1024, n_lo=32, n_hi=256, nx="6,14,26", sizes=9),
        # one step of that network's training: the problems of one range of the pool, built in FP64
        _case("train_nx14_16", kind="train", P=16, n_lo=32, n_hi=256, precision="fp64", sizes=10),
    ]


def draw(rng):
    kind = rng.choice(("step", "step", "step", "serve", "kkt", "kkt_calls", "blocks", "warm", "train"))
    c = _case(kind=kind, sizes=rng.randrange(1 << 20))
    most = {"step": 4096, "serve": 64, "kkt": 2048, "kkt_calls": 4096, "blocks": 512, "warm": 2048, "train": 64}[kind]
    c["P"] = int(round(math.exp(rng.uniform(0.0, math.log(most)))))
    c["n_lo"] = rng.choice((1, 17, 32))
    c["n_hi"] = rng.randrange(c["n_lo"] + 8, 257)
    c["nx"] = rng.choice(("6,14,26", "6", "14", "26", "14,26"))
    if c["nx"] in ("26", "14,26"):  # no more work than the ragged batch
        c["P"] = max(1, c["P"] // 3)
    if kind in ("step", "serve", "kkt"):
        c["pc"] = rng.choice(("sym", "sym", "add", "bj", "poly2", "poly3"))
        c["cond"] = rng.choice((0.0, 0.0, 1e4))
        if kind != "serve" and c["P"] <= 1024 and rng.random() < 0.3:
            c["precision"], c["tol"], c["pc"] = "fp64", rng.choice((1e-6, 1e-8)), rng.choice(("sym", "add", "bj"))
        elif c["P"] <= 256 and rng.random() < 0.3:
            c["nx"], c["nu_frac"] = rng.choice(("36", "9,12", "20", "6,14,26,36")), rng.choice((0.34, 0.5, 1.0))
            c["pc"] = rng.choice(("sym", "add", "bj"))
    elif kind == "blocks":
        c["n_hi"] = min(c["n_hi"], 160)
        c["nx"] = rng.choice(("3,6,9,14,20,26,36", "6,14,26", "5,12,31"))
        c["pc"], c["precision"], c["tol"] = rng.choice(("sym", "add", "bj", "jacobi")), "fp64", 1e-10
    elif kind == "train":
        c["nx"], c["precision"] = rng.choice(("6", "14", "26")), "fp64"
        c["n_lo"] = 32
        c["n_hi"] = max(c["n_hi"], 40)
    return c


def _sizes(c):
    rng = np.random.default_rng(int(c["sizes"]))
    N = rng.integers(c["n_lo"], c["n_hi"] + 1, size=c["P"]).astype(np.int32)
    nxs = np.array([int(v) for v in c["nx"].split(",")], dtype=np.int32)
    nx = nxs[rng.integers(0, len(nxs), size=c["P"])]
    nu = np.zeros_like(nx) if c["kind"] == "blocks" else np.floor(nx * c["nu_frac"]).astype(np.int32)
    return N, nx, nu


def work(case):
    N, nx, nu = (a.astype(np.float64) for a in _sizes(case))
    kind = case["kind"]
    nn, vec, ctl = (N * nx * nx).sum(), (N * nx).sum(), (N * nu).sum()
    dyn = ((N - 1) * (nx * nu + nu * nu)).sum()  # B and R
    kkt = 2.0 * (2 * nn + dyn)
    if kind == "kkt_calls":
        return {"bytes": 8.0 * (2 * nn + dyn + 5 * vec + 2 * ctl), "flops": 2 * kkt}
    blocks = 8.0 * (2 * nn + dyn)
    # assembly: two inverses and three products of size nx per knot, the products with R^-1; PCG: 4 nx^2 per product
    # with the off-diagonal blocks, two (block-Jacobi one) of them per iteration, a typical iteration count
    n3 = (N * nx ** 3).sum()
    build = 0.0 if kind == "blocks" else 2.0 * (6 * n3 + (N * (nu ** 3 + nx * nu * nu + nx * nx * nu)).sum())
    iters = {"jacobi": 70, "bj": 45, "add": 28, "sym": 23, "poly2": 19, "poly3": 16}[case["pc"]]
    iters *= 4 if case["cond"] >= 1e6 else 1
    steps = {"jacobi": 1, "bj": 1, "add": 2, "sym": 2, "poly2": 3, "poly3": 4}[case["pc"]]
    solve = 4.0 * nn * steps * iters
    out = {"bytes": blocks + 16.0 * vec, "flops": build + solve}
    if kind == "kkt":
        out["bytes"] += 8.0 * (4 * vec + 2 * ctl)
        out["flops"] += 2 * kkt
    net = 2.0 * (N * ((2 * nx * nx + nx) * HIDDEN + HIDDEN * HIDDEN + HIDDEN * nx)).sum()
    if kind == "warm":
        out["flops"] += net
    if kind == "train":
        x = float(nx[0])
        par = (2 * x * x + x) * HIDDEN + HIDDEN * HIDDEN + HIDDEN * x
        return {"bytes": 8.0 * (2 * nn + 2 * vec) + 4.0 * 7 * par, "flops": 3 * net + 12.0 * nn}
    return out


# ------------------------------------------------------------------ inputs --

def _householder(M):
    """The orthogonal factor of each Gaussian matrix of the batch as a product of its reflectors."""
    K, n, _ = M.shape
    U = torch.eye(n, dtype=F64, device=DEV).repeat(K, 1, 1)
    for j in range(n - 1):
        v = M[:, j:, j].clone()  # an independent Gaussian of its own for each reflector
        v[:, 0] += torch.where(v[:, 0] < 0, -1.0, 1.0) * v.norm(dim=1)
        v /= v.norm(dim=1, keepdim=True)
        s = U[:, :, j:]
        s -= 2.0 * (s @ v[:, :, None]) * v[:, None, :]
    return U


def _inputs(case, seed):
    """Packed device arrays of the ragged layout, grouped draws per state size scattered to problem order."""
    N, nx, nu = _sizes(case)
    g = torch.Generator(device=DEV).manual_seed(int(seed))
    randn = lambda *s: torch.randn(*s, generator=g, dtype=F64, device=DEV)
    d = types.SimpleNamespace(N=N, nx=nx, nu=nu)
    keys = ("D", "L") if case["kind"] == "blocks" else ("A", "B", "Q", "R")
    parts = {k: [None] * case["P"] for k in keys}
    for x in sorted(set(nx.tolist())):
        ids = np.nonzero(nx == x)[0]
        K, u = int(N[ids].sum()), int(nu[ids[0]])
        if case["kind"] == "blocks":
            L = randn(K, x, x) / math.sqrt(x)
            starts = torch.from_numpy(np.cumsum(N[ids]) - N[ids]).to(DEV)
            L[starts] = 0.0
            W = randn(K, x, x)
            # the Frobenius norm bounds the 2-norm: S stays positive definite by block diagonal dominance
            nrm = L.flatten(1).norm(dim=1)
            c = nrm + torch.cat([nrm[1:], nrm.new_zeros(1)]) + 0.5
            D = W @ W.transpose(1, 2).contiguous() / x + c[:, None, None] * torch.eye(x, dtype=F64, device=DEV)
            blocks = {"D": 0.5 * (D + D.transpose(1, 2)), "L": L}
        else:
            A = torch.eye(x, dtype=F64, device=DEV) + inputs.H_STEP * randn(K, x, x) / math.sqrt(x)
            B = inputs.B_STD * randn(K, x, u)
            W = randn(K, x, x)
            if case["cond"]:
                U = _householder(W)
                c = torch.rand(K, generator=g, dtype=F64, device=DEV) * math.log10(case["cond"])
                e = torch.arange(x, dtype=F64, device=DEV) / max(x - 1, 1)
                Q = (U * 10.0 ** (c[:, None] * e)[:, None, :]) @ U.transpose(1, 2).contiguous()
                Q = 0.5 * (Q + Q.transpose(1, 2))
            else:
                Q = torch.eye(x, dtype=F64, device=DEV) + W @ W.transpose(1, 2).contiguous() / x
            R = inputs.R_SCALE * torch.eye(u, dtype=F64, device=DEV).repeat(K, 1, 1)
            blocks = {"A": A, "B": B, "Q": Q, "R": R}
        for k, t in blocks.items():
            for p, piece in zip(ids, t.split(N[ids].tolist())):
                parts[k][p] = piece.reshape(-1)
    for k in keys:
        setattr(d, k, torch.cat(parts[k]))
    nv, nc = int((N.astype(np.int64) * nx).sum()), int((N.astype(np.int64) * nu).sum())
    d.gamma = randn(nv)
    d.q, d.c, d.r, d.lam_in = randn(nv), randn(nv), randn(max(nc, 1)), randn(nv)
    return d


def _training(case, seed, n_params):
    """Weights and Adam moments of a network in the middle of its training."""
    rng = np.random.default_rng(int(seed))
    theta = inputs.mlp_init(int(case["nx"]), HIDDEN, seed=int(seed)).astype(np.float32)
    m1 = (0.1 * rng.standard_normal(n_params)).astype(np.float32)
    m2 = rng.uniform(0.5, 1.5, n_params).astype(np.float32)
    return theta, m1, m2


def prepare(case, seed):
    d = _inputs(case, seed)
    P, kind = case["P"], case["kind"]
    s = types.SimpleNamespace(case=case, d=d, kind=kind, nets=[])
    s.solver = BatchSolver(d.N, d.nx, d.nu)
    s.gamma = d.gamma
    s.lam = torch.zeros_like(d.gamma)
    s.iters = torch.zeros(P, dtype=torch.int32, device=DEV)
    s.relres = torch.zeros(P, dtype=F64, device=DEV)
    s.status = torch.zeros(P, dtype=torch.int32, device=DEV)
    s.dx = torch.empty_like(d.gamma)
    s.du = torch.zeros_like(d.r)
    if kind in ("step", "serve", "warm", "train"):
        s.solver.set_keep_inverses(False)
    if kind == "serve":  # a serving loop's set-up: what the first build and solve lay out is kept
        _build(s)
        s.solver.solve(case["tol"], 0, s.gamma, s.lam, 0, s.iters, s.relres, s.status)
    elif kind == "kkt_calls":
        _build(s)
    elif kind == "warm":
        s.nets = [WarmStartNet.load(weights_path(x)) for x in sorted(set(d.nx.tolist()))]
    elif kind == "train":
        s.solver.build("sym", "fp64", d.A, d.B, d.Q, d.R, s.status)
        s.solver.solve(1e-10, 0, s.gamma, s.lam, 0, s.iters, s.relres, s.status)
        net = WarmStartNet(int(case["nx"]), HIDDEN)
        s.nets = [net]
        theta, m1, m2 = _training(case, seed, net.n_params)
        net.set_params(theta)
        net.fit_scaling(s, s.lam)
        net.set_state(m1, m2, 100)
        s.loss = torch.zeros(1, dtype=F64, device=DEV)
        s.theta = torch.empty(net.n_params, dtype=torch.float32, device=DEV)
        s.grad = torch.empty_like(s.theta)
    return s


def _build(s):
    c, d = s.case, s.d
    if s.kind == "blocks":
        s.solver.build_from_blocks(c["pc"], c["precision"], d.D, d.L, s.status)
    else:
        s.solver.build(c["pc"], c["precision"], d.A, d.B, d.Q, d.R, s.status)


def run(s):
    c, d, kind = s.case, s.d, s.kind
    if kind == "kkt_calls":
        s.solver.kkt_rhs(d.A, d.B, d.q, d.r, d.c, s.gamma)
        s.solver.kkt_recover(d.A, d.B, d.q, d.r, d.lam_in, s.dx, s.du)
        return {"gamma": s.gamma, "dx": s.dx, "du": s.du}
    if kind == "train":
        net = s.nets[0]
        net.loss_grad(s, 0, c["P"], s.lam, s.loss)
        net.adam(1e-3)
        _lib.check(_lib.load().ssp_mlp_get_params(net._h, s.theta.data_ptr(), s.grad.data_ptr(),
                                                  torch.cuda.current_stream().cuda_stream), "ssp_mlp_get_params")
        return {"loss": s.loss, "grad": s.grad, "theta": s.theta}
    _build(s)
    if kind == "kkt":
        s.solver.kkt_rhs(d.A, d.B, d.q, d.r, d.c, s.gamma)
    for net in s.nets:
        net.predict(s)
    solve = s.solver.solve_noalloc if kind == "serve" else s.solver.solve
    solve(c["tol"], 0, s.gamma, s.lam, 2 if kind == "warm" else 0, s.iters, s.relres, s.status)
    out = {"lam": s.lam, "iters": s.iters, "status": s.status}
    if kind == "kkt":
        s.solver.kkt_recover(d.A, d.B, d.q, d.r, s.lam, s.dx, s.du)
        out.update(gamma=s.gamma, dx=s.dx, du=s.du)
    return out


# ------------------------------------------------------- 64-bit references --

def _inv(M):
    """Inverses of a batch of SPD matrices by Gauss-Jordan elimination."""
    M = M.clone()
    for j in range(M.shape[-1]):
        p = M[:, j, j].clone()
        row = M[:, j, :] / p[:, None]
        col = M[:, :, j].clone()
        M -= col[:, :, None] * row[:, None, :]
        M[:, j, :] = row
        M[:, :, j] = -col / p[:, None]
        M[:, j, j] = 1.0 / p
    return M


class _Group:
    """The problems of one state size padded to one horizon, knots first: arrays [Nmax, problems, ...]."""

    def __init__(self, d, x):
        self.ids = np.nonzero(d.nx == x)[0]
        self.x, self.u = x, int(d.nu[self.ids[0]])
        self.N = d.N[self.ids].astype(np.int64)
        self.n = int(self.N.max())
        self.d = d

    def index(self, rows, cols):
        """(positions in the packed array, which of them exist) of blocks rows x cols."""
        d = self.d
        per = {"x": d.nx.astype(np.int64), "u": d.nu.astype(np.int64), "1": np.ones_like(d.nx, dtype=np.int64)}
        size = d.N * per[rows] * per[cols]
        off = torch.from_numpy((np.cumsum(size) - size)[self.ids]).to(DEV)
        blk = int((per[rows] * per[cols])[self.ids[0]])
        k = torch.arange(self.n, device=DEV)
        idx = off[None, :, None] + k[:, None, None] * blk + torch.arange(blk, device=DEV)
        real = (k[:, None] < torch.from_numpy(self.N).to(DEV)[None, :])[:, :, None].expand(idx.shape)
        return idx, real

    def take(self, flat, rows, cols):
        idx, real = self.index(rows, cols)
        t = torch.where(real, flat[torch.where(real, idx, 0)], 0.0)
        dim = {"x": self.x, "u": self.u, "1": 1}
        return t.reshape(self.n, len(self.ids), dim[rows], dim[cols])

    def put(self, flat, t, rows):
        idx, real = self.index(rows, "1")
        flat[idx[real]] = t.reshape(idx.shape)[real]

    def pad_eye(self, M):
        """M with the identity in the place of the blocks past each horizon."""
        out = torch.arange(self.n, device=DEV)[:, None] >= torch.from_numpy(self.N).to(DEV)[None, :]
        return M + out[:, :, None, None] * torch.eye(M.shape[-1], dtype=F64, device=DEV)


def _shift(M):
    """M of the knot before (zero at the first knot)."""
    return torch.cat([torch.zeros_like(M[:1]), M[:-1]])


def _next(M):
    """M of the next knot (zero past the last one)."""
    return torch.cat([M[1:], torch.zeros_like(M[:1])])


def _flat_inv(M):
    return _inv(M.reshape(-1, *M.shape[2:])).reshape(M.shape) if M.numel() else M


def _thomas(D, L, g):
    """Block elimination of the padded block-tridiagonal systems."""
    n = D.shape[0]
    E, y = torch.empty_like(D), torch.empty_like(g)
    E[0], y[0] = _inv(D[0]), g[0]
    for k in range(1, n):
        G = L[k] @ E[k - 1]
        E[k] = _inv(D[k] - G @ L[k].transpose(1, 2).contiguous())
        y[k] = g[k] - G @ y[k - 1]
    x = torch.empty_like(g)
    x[n - 1] = E[n - 1] @ y[n - 1]
    for k in range(n - 2, -1, -1):
        x[k] = E[k] @ (y[k] - L[k + 1].transpose(1, 2).contiguous() @ x[k + 1])
    return x


def _schur(gr):
    """D, L, Q^-1, R^-1, A, B of a group; A and B of each problem's last knot do not enter."""
    d = gr.d
    Qi, Ri = _flat_inv(gr.pad_eye(gr.take(d.Q, "x", "x"))), _flat_inv(gr.pad_eye(gr.take(d.R, "u", "u")))
    live = (torch.arange(gr.n, device=DEV)[:, None] < torch.from_numpy(gr.N - 1).to(DEV)[None, :])[:, :, None, None]
    A, B = gr.take(d.A, "x", "x") * live, gr.take(d.B, "x", "u") * live
    AQ = A @ Qi
    D = Qi + _shift(AQ @ A.transpose(2, 3).contiguous() + (B @ Ri) @ B.transpose(2, 3).contiguous())
    return D, -_shift(AQ), Qi, Ri, A, B


def exact(case, seed):
    kind = case["kind"]
    d = _inputs(case, seed)
    if kind == "train":
        return _exact_training(case, seed, d)
    out = {k: torch.zeros_like(d.gamma) for k in ("lam", "gamma", "dx")}
    out["du"] = torch.zeros_like(d.r)
    for x in sorted(set(d.nx.tolist())):
        gr = _Group(d, x)
        if kind == "blocks":
            D, L = gr.pad_eye(gr.take(d.D, "x", "x")), gr.take(d.L, "x", "x")
        else:
            D, L, Qi, Ri, A, B = _schur(gr)
        g = gr.take(d.gamma, "x", "1")
        if kind in ("kkt", "kkt_calls"):
            q, r = gr.take(d.q, "x", "1"), gr.take(d.r, "u", "1")
            Qq = Qi @ q
            g = gr.take(d.c, "x", "1") - Qq + _shift(A @ Qq + B @ (Ri @ r))
            gr.put(out["gamma"], g, "x")
        if kind == "kkt_calls":
            lam = gr.take(d.lam_in, "x", "1")
        else:
            lam = _thomas(D, L, g)
            gr.put(out["lam"], lam, "x")
        if kind in ("kkt", "kkt_calls"):
            nxt = _next(lam)
            gr.put(out["dx"], Qi @ (q + lam - A.transpose(2, 3).contiguous() @ nxt), "x")
            du = Ri @ (r - B.transpose(2, 3).contiguous() @ nxt)
            live = (torch.arange(gr.n, device=DEV)[:, None] < torch.from_numpy(gr.N - 1).to(DEV)[None, :])
            gr.put(out["du"], du * live[:, :, None, None], "u")
    if kind == "kkt_calls":
        return {k: out[k] for k in ("gamma", "dx", "du")}
    if kind == "kkt":
        return {**out, "iters": None, "status": None}
    return {"lam": out["lam"], "iters": None, "status": None}


def _exact_training(case, seed, d):
    x, P = int(case["nx"]), case["P"]
    gr = _Group(d, x)
    D, L = _schur(gr)[:2]
    g = gr.take(d.gamma, "x", "1")
    lam = _thomas(D, L, g)
    real = (torch.arange(gr.n, device=DEV)[:, None] < torch.from_numpy(gr.N).to(DEV)[None, :])
    feat = torch.cat([D.flatten(2), L.flatten(2), g.flatten(2)], 2)[real]
    mu = feat.mean(0)
    isd = 1.0 / (feat - mu).square().mean(0).sqrt().clamp(min=1e-6)
    ys = lam[real].square().mean().sqrt()
    nin, H = 2 * x * x + x, HIDDEN
    theta, m1, m2 = (torch.from_numpy(a).to(DEV, F64) for a in _training(case, seed, nin * H + H * H + 2 * H + H * x + x))
    theta.requires_grad_(True)
    W1, b1, W2, b2, W3, b3 = theta.split([nin * H, H, H * H, H, H * x, x])
    with torch.enable_grad():
        h = torch.nn.functional.gelu((feat - mu) * isd @ W1.view(nin, H) + b1)
        h = torch.nn.functional.gelu(h @ W2.view(H, H) + b2)
        y = ys * (h @ W3.view(H, x) + b3)
        e = torch.zeros_like(lam)
        e[real] = y[:, :, None]
        e = e - lam
        res = D @ e + L @ _shift(e) + _next(L).transpose(2, 3).contiguous() @ _next(e)
        loss = res[real].square().sum() / P
        loss.backward()
    grad = theta.grad
    m1, m2, t = 0.9 * m1 + 0.1 * grad, 0.999 * m2 + 0.001 * grad.square(), 101
    step = 1e-3 * (m1 / (1 - 0.9 ** t)) / ((m2 / (1 - 0.999 ** t)).sqrt() + 1e-8)
    return {"loss": loss.detach().reshape(1), "grad": grad, "theta": (theta - step).detach()}
