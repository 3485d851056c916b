"""Timing cases of the library: what a program that uses it has it do.

Every case goes through the Python binding (`Solver`, `Mlp`) as the README's example does:
the hierarchy, the network and their data are in hand (`prepare`), one pass (`run`) is the
call that such a program repeats.  Four kinds:

  vcycle   x = V b, the V-cycle as somebody else's preconditioner
  solve    A x = b to 1e-10 under refinement, CG or GMRES, for new right-hand sides
  setup    the cascade fit for new coefficients, with the fitted blocks read back on the
           device (as the collection of a training set does)
  net      the block-smoother network: prediction for a mesh, one epoch of training

The problem families and their sizes are those of `synth/`, the tests and `bench.py`.
"""
import functools

import numpy as np
import torch

from paper_2606_12577_amd.cascade import Solver
from paper_2606_12577_amd.learned import N_FEATURES, Mlp, fe_block_features
from synth import dg, fd, fe, stokes
from synth.batch import concatenate

DEV = "cuda"
RTOL = 1e-10


# ---------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------

def _solve(family, n, nrhs, precision, method, **more):
    return dict(kind="solve", family=family, n=n, nrhs=nrhs, precision=precision, method=method, **more)


def listed():
    return [
        # the smallest call in use: one V(2,2) of the 64^2 Poisson problem inside another
        # program's Krylov loop; launches and latency
        dict(name="vcycle poisson2d 64 fp64", kind="vcycle", family="poisson2d", n=64, nrhs=1),
        # a small solve, a time step's pressure equation say; launches and host round trips
        dict(name="solve poisson2d 64 fp64 ir", **_solve("poisson2d", 64, 1, "fp64", "ir")),
        # the headline workload: 2,097,152 unknowns, 8 right-hand sides, FP32 V-cycle in FP64
        # refinement; the largest
        dict(name="solve interface3d 128x8 fp32 ir", **_solve("interface3d", 128, 8, "fp32", "ir")),
        # one right-hand side, all in FP64, with the paper's own driver (left GMRES)
        dict(name="solve interface3d 96x1 fp64 gmres", **_solve("interface3d", 96, 1, "fp64", "gmres")),
        # new coefficients on a mesh: the depth-4 fit of 8 x 8 blocks (nonlinear and
        # time-dependent problems pay it for every operator)
        dict(name="setup interface3d 96", kind="setup", family="interface3d", n=96),
        # high-order DG: the multicoloured fit of 16 x 16 blocks with the ridge
        dict(name="setup sipg 64 ridge", kind="setup", family="sipg", n=64),
        # the same discretisation solved with BF16 blocks on the matrix cores
        dict(name="solve sipg 96x1 bf16 ir", **_solve("sipg", 96, 1, "bf16", "ir")),
        # many independent systems of ragged sizes at once
        dict(name="solve lognormal batch 16x4 fp32 cg", **_solve("lognormal", 16, 4, "fp32", "cg")),
        # an indefinite system: staggered-grid Stokes under flexible GMRES
        dict(name="solve stokes 128x1 fp32 fgmres", **_solve("stokes", 128, 1, "fp32", "fgmres")),
        # 27-point finite elements with general (trilinear) transfers, two right-hand sides
        dict(name="solve multiphase3d 48x2 fp64 cg", **_solve("multiphase3d", 48, 2, "fp64", "cg")),
        # the learned setup's prediction for a 96^3 mesh (110,592 blocks)
        dict(name="net forward 96", kind="net_forward", n=96),
        # an epoch of training over 16,384 blocks in batches of 1,024
        dict(name="net train 16384", kind="net_train", rows=16384),
    ]


# grid sizes that coarsen to a small bottom level
_SIZES_2D = (16, 24, 32, 40, 48, 64, 72, 80, 96, 112, 128, 144, 160, 176, 192, 224, 256, 288, 320, 384, 448, 512)
_SIZES_DG = (8, 10, 12, 14, 16, 18, 20, 22, 24, 28, 32, 36, 40, 44, 48, 56, 64, 72, 80, 88, 96)
_SIZES_3D = (8, 12, 16, 20, 24, 28, 32, 40, 44, 48, 56, 64, 72, 80, 88, 96, 104, 112, 128)


def _log_pick(rng, sizes, lo, hi):
    """A size between lo and hi, spread over its logarithm."""
    s = lo * (hi / lo) ** rng.random()
    return min((v for v in sizes if lo <= v <= hi), key=lambda v: abs(v - s))


def draw(rng):
    kind = rng.choice(["vcycle", "solve", "solve", "solve", "solve", "setup", "setup", "net_forward", "net_train"])
    nrhs = rng.choice([1, 2, 4, 8])
    if kind == "vcycle":
        if rng.random() < 0.5:
            return dict(kind=kind, family="poisson2d", n=_log_pick(rng, _SIZES_2D, 16, 256), nrhs=nrhs)
        return dict(kind=kind, family="interface3d", n=_log_pick(rng, _SIZES_3D, 8, 96), nrhs=nrhs)
    if kind == "setup":
        if rng.random() < 0.6:
            return dict(kind=kind, family="interface3d", n=_log_pick(rng, _SIZES_3D, 8, 96))
        return dict(kind=kind, family="sipg", n=_log_pick(rng, _SIZES_DG, 8, 64))
    if kind == "net_forward":
        return dict(kind=kind, n=2 * round(8 * 6 ** rng.random()))
    if kind == "net_train":
        return dict(kind=kind, rows=round(1000 * 16 ** rng.random()))
    family = rng.choice(["poisson2d", "interface3d", "interface3d", "sipg", "lognormal", "stokes", "multiphase3d"])
    if family == "poisson2d":
        return _solve(family, _log_pick(rng, _SIZES_2D, 16, 512), nrhs, rng.choice(["fp64", "fp32"]),
                      rng.choice(["ir", "cg", "gmres"]))
    if family == "interface3d":
        return _solve(family, _log_pick(rng, _SIZES_3D, 12, 112), nrhs, rng.choice(["fp64", "fp32"]),
                      rng.choice(["ir", "cg", "gmres", "fgmres"]))
    if family == "sipg":
        return _solve(family, _log_pick(rng, _SIZES_DG, 8, 96), 1, rng.choice(["bf16", "bf16", "fp32", "fp64"]),
                      rng.choice(["ir", "fgmres"]))
    if family == "lognormal":
        return _solve(family, rng.randint(4, 16), rng.choice([2, 4]), rng.choice(["fp64", "fp32"]), "cg")
    if family == "stokes":
        return _solve(family, rng.choice([16, 24, 32, 48, 64, 80, 96, 112]), 1, rng.choice(["fp64", "fp32"]),
                      rng.choice(["gmres", "fgmres"]))
    return _solve(family, rng.choice([8, 12, 16, 24, 32, 40, 48]), rng.choice([1, 2, 4]), "fp64", "cg")


# ---------------------------------------------------------------------------
# Problems
# ---------------------------------------------------------------------------

def _sphere(n, seed):
    """The interface problem's coefficients with the sphere's centre drawn from the seed."""
    centre = np.random.default_rng(seed).uniform(0.3, 0.7, size=3)
    return fd.fv_hierarchy(fd.sphere_mu(n, centre, 0.3, 1e4), bs=2)


@functools.lru_cache(maxsize=1)
def _fixed_levels(family, n):
    """Hierarchies whose coefficients do not change between right-hand sides."""
    return fd.poisson2d(n).levels if family == "poisson2d" else stokes.mac2d(n).levels


def _hierarchy(case, seed):
    """(levels, row offsets of independent systems or None)"""
    family, n = case["family"], case["n"]
    if family in ("poisson2d", "stokes"):
        return _fixed_levels(family, n), None
    if family == "interface3d":
        return _sphere(n, seed), None
    if family == "sipg":
        return dg.sipg_q3(n, seed_extra=seed).levels, None
    if family == "multiphase3d":
        return fe.multiphase3d(n, seed_extra=seed).levels, None
    sizes = fd.batch_sizes(n, 6.0, 7.5)     # n systems of 64 to 176 cells a side
    bt = concatenate([fd.lognormal2d(int(m), system=100 * seed + s) for s, m in enumerate(sizes)])
    return bt.levels, bt.sys_ptr


def _options(case):
    family = case["family"]
    if family == "poisson2d":
        return dict(depth=3, n_pre=2, n_post=2)
    if family == "interface3d":
        return dict(depth=4)
    if family == "sipg":
        return dict(depth=3, mode="multiplicative", order="FF", ridge=1e-3)
    if family == "stokes":
        return dict(depth=4, order="FF")
    return dict(depth=3) if family == "lognormal" else dict(depth=2)


def _rhs(case, levels, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    b = 2 * torch.rand((levels[0].n, case["nrhs"]), generator=g, device=DEV, dtype=torch.float64) - 1
    if case["family"] == "stokes":
        b[torch.as_tensor(levels[0].kind == 2, device=DEV)] = 0.0     # unused slots
    return b


def _log10mu(n, seed):
    """A two-phase coefficient field on n^3 hexes."""
    z = np.random.default_rng(seed).standard_normal((n // 2, n // 2, n // 2))
    return 3.0 * (np.kron(z, np.ones((2, 2, 2))) > 0.3)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "net_forward":
        net = Mlp()
        net.init_params(seed)
        rng = np.random.default_rng(seed)
        net.set_scaling(rng.normal(0, 0.2, net.n_out), rng.uniform(0.05, 0.5, net.n_out))
        return dict(kind=kind, net=net, X=fe_block_features(_log10mu(case["n"], seed)))
    if kind == "net_train":
        rows = case["rows"]
        X = fe_block_features(_log10mu(52, seed))
        net = Mlp()
        net.init_params(seed)
        p0 = net.get_params()
        g = torch.Generator(device=DEV).manual_seed(seed)
        mix = torch.randn((N_FEATURES, net.n_out), generator=g, device=DEV) / N_FEATURES ** 0.5
        T = torch.tanh(X @ mix) + 0.05 * torch.randn((X.shape[0], net.n_out), generator=g, device=DEV)
        order = torch.randperm(X.shape[0], generator=g, device=DEV)[:rows].to(torch.int32)[None, :]
        net.fit_scaling(T, order[0])
        return dict(kind=kind, net=net, X=X, T=T.contiguous(), order=order, p0=p0)
    levels, sys_ptr = _hierarchy(case, seed)
    s = Solver(levels)
    if sys_ptr is not None:
        s.set_systems(sys_ptr)
    opts = _options(case)
    if kind == "setup":
        return dict(kind=kind, solver=s, opts=dict(opts, precision="bf16" if case["family"] == "sipg" else "fp32"))
    s.setup(**opts, precision=case.get("precision", "fp64"))
    s.autotune(case["nrhs"])
    return dict(kind=kind, solver=s, b=_rhs(case, levels, seed), method=case.get("method"))


def run(state):
    kind = state["kind"]
    if kind == "vcycle":
        return state["solver"].vcycle(state["b"])
    if kind == "solve":
        return state["solver"].solve(state["b"], rtol=RTOL, maxit=500, method=state["method"])[0]
    if kind == "setup":
        state["solver"].setup(**state["opts"])
        return state["solver"].get_prescaled_blocks(0)
    if kind == "net_forward":
        return state["net"].forward(state["X"])
    net = state["net"]
    net.set_params(state["p0"])
    loss = net.train(state["X"], state["T"], state["order"], batch=1024)
    return dict(params=net.get_params(), loss=loss.astype(np.float32))


# ---------------------------------------------------------------------------
# Work that the path cannot do without
# ---------------------------------------------------------------------------

# stored entries per row, block size, coarsening factor per level, and a usual number of V-cycles
_SHAPE = dict(poisson2d=(5, 1, 4, 7), interface3d=(7, 8, 8, 20), sipg=(80, 16, 4, 40), lognormal=(5, 1, 4, 50),
              stokes=(9, 4, 4, 18), multiphase3d=(27, 8, 8, 30))


def _unknowns(case):
    family, n = case["family"], case["n"]
    if family == "lognormal":
        return int((fd.batch_sizes(n, 6.0, 7.5) ** 2).sum())
    return n ** 3 if family.endswith("3d") else n * n * {"sipg": 16, "stokes": 4}.get(family, 1)


def work(case):
    """Each input read once and each output written once: the matrices and smoothers of all
    levels, right-hand sides and solutions; the operations of the V-cycles, of the fit, or of
    the network's products."""
    kind = case["kind"]
    if kind.startswith("net"):
        rows = case["rows"] if kind == "net_train" else (case["n"] // 2) ** 3
        weights = N_FEATURES * 128 + 2 * 128 * 128
        passes = 3 if kind == "net_train" else 1
        return dict(bytes=4 * rows * (N_FEATURES + 128) + 4 * weights * passes, flops=2 * rows * weights * passes)
    z, nb, shrink, cycles = _SHAPE[case["family"]]
    n = _unknowns(case)
    total = n * shrink / (shrink - 1)            # unknowns of all levels
    depth = _options(case)["depth"]
    if kind == "setup":
        # blocks of the fitted residual's rows after 0, 1, ... steps
        k = [1, 7, 25, 63, 129] if case["family"] == "interface3d" else [1, 13, 41, 85]
        neighbours = 7 if case["family"] == "interface3d" else 5
        per_block = sum(neighbours * k[s] + 3 * k[s + 1] for s in range(depth)) * 2 * nb ** 3
        return dict(bytes=12 * z * total + 4 * depth * nb * n, flops=per_block * total / nb)
    es = 8 if case.get("precision", "fp64") == "fp64" else 4
    sweeps = depth * (4 if case["family"] == "poisson2d" else 2)
    flops = 2 * case["nrhs"] * total * (z * (sweeps + 1) + nb * sweeps)
    return dict(bytes=total * (z * (es + 4) + depth * nb * es) + 16 * n * case["nrhs"],
                flops=flops * (cycles if kind == "solve" else 1))


# ---------------------------------------------------------------------------
# The same values in 64 bits from plain torch
# ---------------------------------------------------------------------------

def _ell(A):
    """Row-padded columns and values of a CSR matrix, on the GPU."""
    A = A.tocsr()
    n, cnt = A.shape[0], np.diff(A.indptr)
    pos = np.arange(A.nnz) - np.repeat(A.indptr[:-1], cnt)
    row = np.repeat(np.arange(n), cnt)
    col, val = np.zeros((n, max(int(cnt.max()), 1)), np.int64), np.zeros((n, max(int(cnt.max()), 1)))
    col[row, pos], val[row, pos] = A.indices, A.data
    return torch.as_tensor(col, device=DEV), torch.as_tensor(val, device=DEV)


def _mul(ell, x, rows=slice(None)):
    col, val = ell[0][rows], ell[1][rows]
    y = torch.zeros((col.shape[0], x.shape[1]), dtype=torch.float64, device=DEV)
    for k in range(col.shape[1]):
        y += val[:, k, None] * x[col[:, k]]
    return y


def _fit(level, depth, colours=None, ridge=0.0):
    """Prescaled blocks [depth, B, nb, nb] of the cascade fit and the scaling w: the residual E
    held as a dense matrix, every block's normal equations formed and solved."""
    nb, n = level.block_size, level.n
    w = torch.as_tensor(1.0 / np.sqrt(level.A.diagonal()), device=DEV)
    col, val = _ell(level.A)
    at = col, val * w[:, None] * w[col]
    E = torch.eye(n, dtype=torch.float64, device=DEV)
    eye = torch.eye(nb, dtype=torch.float64, device=DEV)
    lam = torch.zeros((depth, n // nb, nb, nb), dtype=torch.float64, device=DEV)
    groups = [torch.arange(n // nb, device=DEV)] if colours is None else [
        torch.as_tensor(np.flatnonzero(colours == c), device=DEV) for c in range(int(colours.max()) + 1)]
    for step in range(depth):
        for blocks in groups:
            new = []
            for part in blocks.split(max(1, (1 << 28) // (n * nb))):
                rows = (part[:, None] * nb + torch.arange(nb, device=DEV)).reshape(-1)
                M = _mul(at, E, rows).reshape(len(part), nb, n)
                Mt = M.transpose(1, 2).contiguous()
                Ei = E[rows].reshape(len(part), nb, n)
                G, H = torch.matmul(M, Mt), torch.matmul(Ei, Mt)
                if ridge:
                    G = G + (ridge / nb) * G.diagonal(dim1=1, dim2=2).sum(1)[:, None, None] * eye
                lam[step, part] = torch.matmul(H, torch.linalg.pinv(G, rtol=1e-13, hermitian=True))
                new.append((rows, Ei - torch.matmul(lam[step, part], M)))
                if colours is not None or len(blocks) * nb < n:      # a colour's blocks do not see each other
                    E[rows] = new.pop()[1].reshape(-1, n)
            if new:
                E = torch.cat([v.reshape(-1, n) for _, v in new])
    return lam, w


def _exact_vcycle(case, seed):
    levels = _hierarchy(case, seed)[0]
    o = _options(case)
    data = []
    for lv in levels[:-1]:
        lam, w = _fit(lv, o["depth"])
        nb = lv.block_size
        lam = w.reshape(1, -1, nb, 1) * lam * w.reshape(1, -1, 1, nb)
        data.append((_ell(lv.A), lam, _ell(lv.P), _ell(lv.P.T.tocsr()), lv.r_scale, nb))
    bottom = torch.as_tensor(levels[-1].A.toarray(), device=DEV)

    def sweep(A, lam, nb, x, b):
        r = (_mul(A, x) - b).reshape(lam.shape[0], nb, -1)
        return x - torch.matmul(lam.contiguous(), r).reshape(x.shape)

    def cycle(l, b):
        if l == len(data):
            return torch.linalg.solve(bottom, b)
        A, lam, P, Pt, scale, nb = data[l]
        x = torch.zeros_like(b)
        for _ in range(o.get("n_pre", 1)):
            for k in reversed(range(o["depth"])):
                x = sweep(A, lam[k].transpose(1, 2), nb, x, b)
        x = x - _mul(P, cycle(l + 1, scale * _mul(Pt, _mul(A, x) - b)))
        for _ in range(o.get("n_post", 1)):
            for k in range(o["depth"]):
                x = sweep(A, lam[k], nb, x, b)
        return x

    return cycle(0, _rhs(case, levels, seed))


def _exact_solve(case, seed):
    levels = _hierarchy(case, seed)[0]
    b, A = _rhs(case, levels, seed), levels[0].A
    if A.shape[0] <= 8192:
        return torch.linalg.solve(torch.as_tensor(A.toarray(), device=DEV), b)
    if case["family"] == "stokes" or A.shape[0] * case["nrhs"] > 4_000_000:
        return None
    # conjugate gradients preconditioned by the diagonal blocks, until nothing is gained any more
    ell, nb = _ell(A), max(levels[0].block_size, 1)
    blocks = A.tobsr((nb, nb))
    row = np.repeat(np.arange(A.shape[0] // nb), np.diff(blocks.indptr))
    D = torch.as_tensor(blocks.data[row == blocks.indices], device=DEV)
    Di = torch.linalg.inv(D)
    pre = lambda r: torch.matmul(Di, r.reshape(Di.shape[0], nb, -1)).reshape(r.shape)  # noqa: E731
    x = torch.zeros_like(b)
    for _ in range(2):                       # restarted once from the true residual
        r = b - _mul(ell, x)
        z = pre(r)
        p, rz = z, (r * z).sum(0)
        for it in range(6000):
            q = _mul(ell, p)
            a = rz / (p * q).sum(0).clamp_min(1e-300)
            x, r = x + a * p, r - a * q
            if it % 50 == 0 and float((r.norm(dim=0) / b.norm(dim=0)).max()) < 1e-14:
                break
            z = pre(r)
            new = (r * z).sum(0)
            p, rz = z + (new / rz.clamp_min(1e-300)) * p, new
    if float(((b - _mul(ell, x)).norm(dim=0) / b.norm(dim=0)).max()) > 1e-11:
        return None
    return x


def _net(p, n_in, width, n_out):
    out, at = [], 0
    for i, o in ((n_in, width), (width, width), (width, n_out)):
        out += [p[at:at + i * o].reshape(o, i), p[at + i * o:at + i * o + o]]
        at += i * o + o
    return out


def _net_layers(P, X):
    z1 = X @ P[0].T + P[1]
    h1 = z1 * torch.sigmoid(z1)
    z2 = h1 @ P[2].T + P[3]
    h2 = z2 * torch.sigmoid(z2)
    return h2 @ P[4].T + P[5]


def _exact_train(case, seed):
    """Adam over the batches in their order, gradients by torch's reverse mode in 64 bits."""
    s = prepare(case, seed)
    net, order = s["net"], s["order"][0].long()
    X, T = s["X"].double(), s["T"].double()
    mean, std = (torch.as_tensor(v, device=DEV).double() for v in net.get_scaling())
    p = torch.as_tensor(s["p0"], device=DEV).double().requires_grad_()
    m, v, losses = torch.zeros_like(p), torch.zeros_like(p), []
    batches = order.split(1024)
    for k, rows in enumerate(batches):
        y = _net_layers(_net(p, net.n_in, net.width, net.n_out), X[rows])
        loss = ((y - (T[rows] - mean) / std) ** 2).mean()
        g, = torch.autograd.grad(loss, p)
        losses.append(float(loss))
        lr = 0.5e-3 * (1.0 + np.cos(np.pi * k / len(batches)))
        with torch.no_grad():
            m = 0.9 * m + 0.1 * g
            v = 0.999 * v + 0.001 * g * g
            p -= lr * (m / (1 - 0.9 ** (k + 1))) / ((v / (1 - 0.999 ** (k + 1))).sqrt() + 1e-8)
    return dict(params=p.detach(), loss=np.array([np.mean(losses)]))


def exact(case, seed):
    kind = case["kind"]
    if kind == "net_forward":
        s = prepare(case, seed)
        net = s["net"]
        mean, std = (torch.as_tensor(v, device=DEV).double() for v in net.get_scaling())
        p = torch.as_tensor(net.get_params(), device=DEV).double()
        return _net_layers(_net(p, net.n_in, net.width, net.n_out), s["X"].double()) * std + mean
    if kind == "net_train":
        return _exact_train(case, seed)
    n = _unknowns(case)
    if kind == "setup":
        if n > 33000:                        # the dense residual would take too long
            return None
        lv = _hierarchy(case, seed)[0][0]
        o = _options(case)
        lam, _ = _fit(lv, o["depth"], lv.colour if o.get("mode") == "multiplicative" else None, o.get("ridge", 0.0))
        return lam.transpose(0, 1).contiguous()
    if kind == "vcycle":
        return _exact_vcycle(case, seed) if n <= 33000 else None
    return _exact_solve(case, seed)
