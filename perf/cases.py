"""Performance cases of the library: the calls that a lattice program makes, over the sizes that it makes them at.

Each case is one public call (or the few that belong together) on Nrhs right-hand sides at once: the fine
Wilson-clover operator, its even-odd Schur complement, the transfers between the multigrid levels, the coarse stencil
and its minimal-residual solve, a Gram-Schmidt step, and a whole multigrid-preconditioned solve.  Lattices are given
as (Lx, Ly, Lz, Lt); inputs are Gaussian sources on Haar-random links, except for the solve, which runs on smooth
links at the bare mass -0.1.  `exact` evaluates the same definitions in complex128 with plain torch.
"""

import math
import os

import numpy as np
import torch

import paper_2211_13719_amd as mrhs

DEV = "cuda:0"
KAPPA, CSW = 0.13, 1.0
# smooth links U = exp(0.3 i H) at the bare mass m0 = -0.1: kappa = 1 / (2 (4 + m0))
KAPPA_SOLVE = 1 / 7.8
TUNE_CACHE = os.path.join(os.path.dirname(os.path.abspath(mrhs.__file__)), "tuning", "fine.txt")
CACHED = {(24, 24, 24, 24): (1, 6, 12, 24, 48, 64)}  # the lattices whose launch choices ship with the library


def listed():
    return [
        # a small lattice and one source: a call that is mostly launch latency
        dict(name="dwc_f32_8x8x8x8_n1", op="dwc", prec="f32", lx=8, ly=8, lz=8, lt=8, n=1, tuned=False),
        # the operator of a batched propagator calculation: 12 spin-colour sources on a production local volume
        dict(name="dwc_f32_24x24x24x24_n12", op="dwc", prec="f32", lx=24, ly=24, lz=24, lt=24, n=12, tuned=True),
        # the same at the largest batch the library takes
        dict(name="dwc_f32_24x24x24x24_n64", op="dwc", prec="f32", lx=24, ly=24, lz=24, lt=24, n=64, tuned=True),
        # a lattice whose extents share no power of two, an odd batch, and no tuning beforehand
        dict(name="dwc_f32_12x10x6x14_n7", op="dwc", prec="f32", lx=12, ly=10, lz=6, lt=14, n=7, tuned=False),
        # the true residual of an outer FP64 solver
        dict(name="dwc_f64_24x24x24x24_n12", op="dwc", prec="f64", lx=24, ly=24, lz=24, lt=24, n=12, tuned=True),
        # even-odd preconditioning: the Schur complement on the even sites, the smoother's operator
        dict(name="schur_f32_16x16x16x32_n24", op="schur", prec="f32", lx=16, ly=16, lz=16, lt=32, n=24, tuned=True),
        # down to the coarse lattice and back, in single precision
        dict(name="intergrid_f32_24x24x24x24_n24", op="intergrid", prec="f32", lx=24, ly=24, lz=24, lt=24, n=24, nv=16),
        # the same in the V-cycle's BF16 arithmetic, with 30 right-hand sides
        dict(name="intergrid_bf16_16x16x16x32_n30", op="intergrid", prec="bf16", lx=16, ly=16, lz=16, lt=32, n=30, nv=16),
        # the coarse operator of 24^4 with 4^4 aggregates
        dict(name="coarse_bf16_6x6x6x6_n48", op="coarse", prec="bf16", lx=6, ly=6, lz=6, lt=6, n=48),
        # the coarsest level's solve of 24^3 x 128: many small steps, each waiting for the one before
        dict(name="coarse_mr_bf16_3x3x3x16_n12", op="coarse_mr", prec="bf16", lx=3, ly=3, lz=3, lt=16, n=12, iters=64),
        # one Gram-Schmidt step of a user's own Krylov solver against six basis vectors
        dict(name="gram_schmidt_f32_24x24x24x24_n12", op="gram_schmidt", prec="f32", lx=24, ly=24, lz=24, lt=24, n=12, m=6),
        # twelve propagator columns to a true residual of 1e-11: FGMRES with the three-level V-cycle
        dict(name="solve_16x16x16x32_n12", op="solve", lx=16, ly=16, lz=16, lt=32, n=12),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: the operators at all precisions, lattices from 4^4 to 24^4 (odd extents
    among them where the call takes them), batches from 1 to 64."""
    op = rng.choice(["dwc", "dwc", "dwc", "schur", "intergrid", "intergrid", "coarse", "coarse", "coarse_mr",
                     "gram_schmidt"])
    if op in ("dwc", "schur", "gram_schmidt"):
        prec = rng.choice(["f32", "f32", "f64"])
        n = _log_int(rng, 1, 48 if prec == "f32" else 24)
        ext = [4, 6, 8, 10, 12, 14, 16, 18, 20, 24] + ([5, 7, 9, 11, 13, 15] if op != "schur" else [])
        c = dict(op=op, prec=prec, lx=rng.choice(ext), ly=rng.choice(ext), lz=rng.choice(ext), lt=rng.choice(ext), n=n)
        if op == "gram_schmidt":
            c["m"] = rng.randint(1, 8)
        else:
            c["tuned"] = rng.random() < 0.5
        return c
    n = _log_int(rng, 1, 64)
    if op == "intergrid":
        ext = [8, 12, 16, 20, 24]
        prec = rng.choice(["f32", "f32", "bf16", "bf16", "f64"])
        return dict(op=op, prec=prec, lx=rng.choice(ext), ly=rng.choice(ext), lz=rng.choice(ext), lt=rng.choice(ext),
                    n=max(1, n // 2) if prec == "f64" else n, nv=16 if prec == "bf16" else rng.choice([8, 16, 16]))
    if op == "coarse":
        return dict(op=op, prec=rng.choice(["f32", "bf16", "bf16", "f16"]), lx=rng.randint(2, 6), ly=rng.randint(2, 6),
                    lz=rng.randint(2, 6), lt=rng.randint(2, 16), n=n)
    return dict(op=op, prec=rng.choice(["f32", "bf16", "bf16"]), lx=rng.randint(2, 4), ly=rng.randint(2, 4),
                lz=rng.randint(2, 4), lt=rng.randint(2, 16), n=n, iters=rng.randint(16, 128))


# ---- inputs ---------------------------------------------------------------------------------------------------------
def _dims(c):
    return (c["lx"], c["ly"], c["lz"], c["lt"])


def _vol(c):
    return c["lx"] * c["ly"] * c["lz"] * c["lt"]


def _gen(seed, what):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 64 + what)
    return g


def _gauss(g, shape, dtype):
    real = torch.float64 if dtype == torch.complex128 else torch.float32
    return torch.view_as_complex(torch.randn(*shape, 2, generator=g, device=DEV, dtype=real))


def _mm(a, b):
    """Batched product of small matrices."""
    return (a.unsqueeze(-1) * b.unsqueeze(-3)).sum(-2)


def _dag(a):
    return a.transpose(-1, -2).conj()


def _haar_links(g, V):
    """Haar-random SU(3): two Gaussian rows orthonormalised, the third their conjugate cross product."""
    z = _gauss(g, (V, 4, 2, 3), torch.complex128)
    a = z[:, :, 0] / torch.linalg.vector_norm(z[:, :, 0], dim=-1, keepdim=True)
    b = z[:, :, 1] - (a.conj() * z[:, :, 1]).sum(-1, keepdim=True) * a
    b = b / torch.linalg.vector_norm(b, dim=-1, keepdim=True)
    return torch.stack([a, b, torch.linalg.cross(a, b, dim=-1).conj()], dim=2).contiguous()


def _smooth_links(g, V, eps=0.3):
    """exp(i eps H), H = sum_a h_a lambda_a / 2 with Gaussian h_a, by its Taylor series."""
    h = torch.randn(V, 4, 8, generator=g, device=DEV, dtype=torch.float64)
    H = torch.zeros(V, 4, 3, 3, device=DEV, dtype=torch.complex128)
    s3 = 1 / math.sqrt(3.0)
    for k, (i, j) in enumerate(((0, 1), (0, 2), (1, 2))):
        H[:, :, i, j] = torch.complex(h[:, :, 2 * k], -h[:, :, 2 * k + 1])
        H[:, :, j, i] = torch.complex(h[:, :, 2 * k], h[:, :, 2 * k + 1])
    H[:, :, 0, 0] = h[:, :, 6] + s3 * h[:, :, 7]
    H[:, :, 1, 1] = -h[:, :, 6] + s3 * h[:, :, 7]
    H[:, :, 2, 2] = -2 * s3 * h[:, :, 7]
    X = 0.5j * eps * H
    U = torch.eye(3, device=DEV, dtype=torch.complex128).expand(V, 4, 3, 3).clone()
    term = U.clone()
    for k in range(1, 25):
        term = _mm(term, X) / k
        U = U + term
    return U.contiguous()


def _dtype(c):
    return torch.complex128 if c.get("prec") == "f64" else torch.complex64


def _fine_inputs(c, seed):
    solve = c["op"] == "solve"
    U = (_smooth_links if solve else _haar_links)(_gen(seed, 1), _vol(c))
    sites = _vol(c) // 2 if c["op"] == "schur" else _vol(c)
    psi = _gauss(_gen(seed, 2), (sites, 12, c["n"]), torch.complex128 if solve else _dtype(c))
    return U, psi, KAPPA_SOLVE if solve else KAPPA


def _basis(c, seed):
    return _gauss(_gen(seed, 3), (_vol(c), c["nv"], 12), torch.complex128)


def _blocks(c, seed):
    """Stencil blocks like a Galerkin operator's: a dominant self block and smaller couplings."""
    B = 0.1 * _gauss(_gen(seed, 4), (_vol(c), 9, 32, 32), torch.complex128)
    B[:, 0] += 4 * torch.eye(32, device=DEV, dtype=torch.complex128)
    return B


def _coarse_vec(c, seed):
    return _gauss(_gen(seed, 5), (_vol(c), 32, c["n"]), torch.complex64)


def _context(c, U, kappa, tune):
    dims = _dims(c)
    ctx = mrhs.Context(dims, t_bc=-1)
    ctx.set_gauge(U)
    ctx.build_clover(CSW, kappa)
    if tune:
        ctx.tune([c["n"]], TUNE_CACHE if c["n"] in CACHED.get(dims, ()) else None)
    return ctx


def _hierarchy(dims, blocks, nv):
    """A hierarchy for the transfers or the coarse stencil alone: they need the lattice, not its links."""
    ctx = mrhs.Context(dims, t_bc=-1)
    return ctx, mrhs.Multigrid(ctx, blocks, nv)


def prepare(case, seed):
    op = case["op"]
    s = dict(case=case)
    if op in ("dwc", "schur"):
        U, psi, kappa = _fine_inputs(case, seed)
        s.update(ctx=_context(case, U, kappa, case["tuned"]), x=psi, out=torch.empty_like(psi))
        if op == "schur":
            s["ctx"].schur(s["out"], psi)  # builds the checkerboard tables and the inverse clover blocks
    elif op == "intergrid":
        ctx, mg = _hierarchy(_dims(case), [(4, 4, 4, 4)], [case["nv"]])
        mg.set_basis(0, _basis(case, seed))
        mg.block_orthonormalise(0)
        fine = _gauss(_gen(seed, 2), (mg.volume[0], 12, case["n"]), _dtype(case))
        coarse = _gauss(_gen(seed, 5), (mg.volume[1], mg.ncomp[1], case["n"]), _dtype(case))
        s.update(ctx=ctx, mg=mg, fine=fine, coarse=coarse, down=torch.empty_like(coarse), up=torch.empty_like(fine))
    elif op in ("coarse", "coarse_mr"):
        ctx, mg = _hierarchy(tuple(2 * d for d in _dims(case)), [(2, 2, 2, 2)], [16])
        mg.set_blocks(1, _blocks(case, seed))
        mg.tune([case["n"]])
        x = _coarse_vec(case, seed)
        s.update(ctx=ctx, mg=mg, x=x, out=torch.empty_like(x))
    elif op == "gram_schmidt":
        g = _gen(seed, 2)
        shape = (_vol(case), 12, case["n"])
        w = _gauss(g, shape, _dtype(case))
        # basis vectors of unit norm, as a Krylov solver keeps them
        vs = [_gauss(g, shape, _dtype(case)) / math.sqrt(2 * 12 * _vol(case)) for _ in range(case["m"])]
        s.update(ctx=mrhs.Context(_dims(case), t_bc=-1), w=w, vs=vs, work=torch.empty_like(w))
    elif op == "solve":
        U, b, kappa = _fine_inputs(case, seed)
        ctx = _context(case, U, kappa, True)
        mg = mrhs.Multigrid(ctx, [(4, 4, 4, 4), (2, 2, 2, 2)], [16, 16])
        g = _gen(seed, 3)
        for level in range(2):
            mg.set_basis(level, _gauss(g, (mg.volume[level], 16, mg.ncomp[level]), torch.complex128))
        mg.setup(setup_iters=4, smooth_steps=20, adapt_iters=0, coarse_prec="bf16", nu_pre=0, nu_post=4,
                 coarsest_iters=64)
        mg.tune([case["n"]])
        s.update(ctx=ctx, mg=mg, b=b, x=torch.zeros_like(b))
    else:
        raise ValueError(op)
    return s


def run(state):
    c = state["case"]
    op = c["op"]
    if op == "dwc":
        return state["ctx"].dwc(state["out"], state["x"])
    if op == "schur":
        return state["ctx"].schur(state["out"], state["x"])
    if op == "intergrid":
        prec = "bf16" if c["prec"] == "bf16" else None
        state["mg"].restrict(0, state["down"], state["fine"], prec)
        state["mg"].prolong(0, state["up"], state["coarse"], prec)
        return [state["down"], state["up"]]
    if op == "coarse":
        return state["mg"].coarse_apply(1, state["out"], state["x"], c["prec"])
    if op == "coarse_mr":
        return state["mg"].coarse_mr_solve(1, state["out"], state["x"], c["iters"], c["prec"])
    if op == "gram_schmidt":
        ctx, y = state["ctx"], state["work"]
        y.copy_(state["w"])
        h = ctx.multi_dot(state["vs"], y)
        for j, v in enumerate(state["vs"]):
            ctx.axpy(y, -h[j], v)
        return [h, ctx.norm2(y), y]
    x = state["x"]
    x.zero_()
    state["mg"].solve(x, state["b"], tol=1e-11, restart=5, max_iters=200, krylov_prec=mrhs.F32, coarse_prec="bf16",
                      nu_pre=0, nu_post=4, coarsest_iters=64, fine_eo=True, coarse_eo=True)
    return x


def work(case):
    """Bytes: inputs read once and outputs written once.  Flops: complex multiply-adds as 8."""
    V, n, op = _vol(case), case["n"], case["op"]
    z = 16 if case.get("prec") == "f64" else 8
    if op == "dwc":  # links and clover blocks (36 complex and 72 real numbers a site), one field in, one out
        return dict(bytes=V * (72 * z + 24 * z * n), flops=1920 * V * n)
    if op == "schur":  # every link; the clover blocks of the even sites and the inverses of the odd ones
        return dict(bytes=V * (72 * z + 12 * z * n), flops=(1320 + 552 + 24) * V * n)
    if op == "intergrid":
        nv = case["nv"]
        zb = 4 if case["prec"] == "bf16" else z
        return dict(bytes=V * 12 * nv * zb + 2 * z * n * (12 * V + 2 * nv * V // 256), flops=2 * 8 * 12 * nv * V * n)
    if op in ("coarse", "coarse_mr"):
        blocks = V * 9 * 1024 * (8 if case["prec"] == "f32" else 4)
        it = case.get("iters", 1)
        return dict(bytes=blocks + V * 32 * n * 16, flops=it * V * n * (8 * 9 * 1024 + (it > 1) * 32 * 32))
    if op == "gram_schmidt":
        return dict(bytes=12 * V * n * z * (case["m"] + 2), flops=12 * V * n * (16 * case["m"] + 4))
    # the solve: links, clover, sources and solutions once; ten preconditioned steps of ten operator applications
    return dict(bytes=V * (72 * 16 + 24 * 16 * n), flops=100 * 1920 * V * n)


# ---- the same in complex128 -----------------------------------------------------------------------------------------
_S = [np.array([[0, 1], [1, 0]], complex), np.array([[0, -1j], [1j, 0]]), np.array([[1, 0], [0, -1]], complex)]
_AXIS = (3, 2, 1, 0)


def _gammas():
    """Euclidean, Hermitian, chiral: gamma_k = [[0, -i s_k], [i s_k, 0]], gamma_4 = [[0, 1], [1, 0]]."""
    Z, one = np.zeros((2, 2)), np.eye(2)
    return [np.block([[Z, -1j * s], [1j * s, Z]]) for s in _S] + [np.block([[Z, one], [one, Z]]).astype(complex)]


def _lat(f, dims):
    return f.reshape(dims[3], dims[2], dims[1], dims[0], *f.shape[1:])


def _shift(f, mu, step):
    """f(x + step mu) on the (t, z, y, x, ...) view."""
    return torch.roll(f, -step, dims=_AXIS[mu])


def _spin(M, psi):
    """4 x 4 spin matrix on (..., 4, 3, N); its entries are 0, +-1 and +-i."""
    rows = []
    for s in range(4):
        row = 0
        for t in range(4):
            if M[s, t] != 0:
                row = row + complex(M[s, t]) * psi[..., t, :, :]
        rows.append(row)
    return torch.stack(rows, dim=-3)


def _colour(U, psi):
    """3 x 3 colour matrix per site on (..., 4, 3, N)."""
    rows = []
    for a in range(3):
        rows.append(sum(U[..., a, b, None, None] * psi[..., b, :] for b in range(3)))
    return torch.stack(rows, dim=-2)


def _hop(U, psi, dims):
    g = _gammas()
    Ul = _lat(U, dims)
    p = _lat(psi.reshape(psi.shape[0], 4, 3, psi.shape[-1]), dims)
    out = torch.zeros_like(p)
    for mu in range(4):
        f = _shift(p, mu, 1)
        b = _shift(_colour(_dag(Ul[..., mu, :, :]), p), mu, -1)
        if mu == 3:  # antiperiodic in time
            f[-1] *= -1
            b[0] *= -1
        out += _spin(np.eye(4) - g[mu], _colour(Ul[..., mu, :, :], f))
        out += _spin(np.eye(4) + g[mu], b)
    return out.reshape(psi.shape)


def _clover_dense(U, dims, kappa):
    """1 + i csw kappa sum_{mu<nu} sigma_{mu nu} (x) F_{mu nu} as two chiral 6 x 6 blocks a site, (V, 2, 6, 6)."""
    g, V = _gammas(), U.shape[0]
    A = torch.zeros(V, 2, 6, 6, device=U.device, dtype=U.dtype)
    Ul, s = _lat(U, dims), _shift
    for mu in range(4):
        for nu in range(mu + 1, 4):
            m, n = Ul[..., mu, :, :], Ul[..., nu, :, :]
            mb, nb = s(m, mu, -1), s(n, nu, -1)
            q = _mm(_mm(m, s(n, mu, 1)), _mm(_dag(s(m, nu, 1)), _dag(n)))
            q = q + _mm(_mm(n, _dag(s(mb, nu, 1))), _mm(_dag(s(n, mu, -1)), mb))
            q = q + _mm(_mm(_dag(mb), _dag(s(s(n, mu, -1), nu, -1))), _mm(s(mb, nu, -1), nb))
            q = q + _mm(_mm(_dag(nb), s(m, nu, -1)), _mm(s(nb, mu, 1), _dag(m)))
            F = ((q - _dag(q)) / 8).reshape(V, 3, 3)
            sig = 0.5j * (g[mu] @ g[nu] - g[nu] @ g[mu])
            for chi in range(2):
                for i in range(2):
                    for j in range(2):
                        z = complex(sig[2 * chi + i, 2 * chi + j])
                        if z != 0:
                            A[:, chi, 3 * i:3 * i + 3, 3 * j:3 * j + 3] += (1j * CSW * kappa * z) * F
    return A + torch.eye(6, device=U.device, dtype=U.dtype)


def _clover(A, psi):
    x = psi.reshape(psi.shape[0], 2, 6, psi.shape[-1])
    out = torch.empty_like(x)
    for i in range(6):
        out[:, :, i] = sum(A[:, :, i, j, None] * x[:, :, j] for j in range(6))
    return out.reshape(psi.shape)


def _parity_sites(dims, parity):
    """Lattice sites of one parity in checkerboard order: entry i is the one among 2i, 2i + 1."""
    s = torch.arange(dims[0] * dims[1] * dims[2] * dims[3], device=DEV)
    r, p = s, 0
    for L in dims:
        p = p + r % L
        r = r // L
    return s[p % 2 == parity]


def _columns(f, psi, width=8):
    return torch.cat([f(psi[..., k:k + width].to(torch.complex128).contiguous()) for k in range(0, psi.shape[-1], width)],
                     dim=-1)


def _agg_index(dims):
    """Sites of every 4^4 aggregate, (aggregates, 256), aggregates in lexicographic order."""
    s = torch.arange(dims[0] * dims[1] * dims[2] * dims[3], device=DEV)
    v = s.reshape(dims[3] // 4, 4, dims[2] // 4, 4, dims[1] // 4, 4, dims[0] // 4, 4)
    return v.permute(0, 2, 4, 6, 1, 3, 5, 7).reshape(-1, 256)


def _stencil(B, e, dims):
    el = _lat(e, dims)
    out = torch.matmul(B[:, 0], e)
    for mu in range(4):
        for k, step in enumerate((1, -1)):
            out = out + torch.matmul(B[:, 1 + 2 * mu + k], _shift(el, mu, step).reshape(e.shape).contiguous())
    return out


def _bicgstab(apply, b, tol, most):
    """Per-column BiCGStab; None if a column has not converged after `most` steps."""
    dot = lambda a, c: (a.conj() * c).sum((0, 1))  # noqa: E731
    x, r = torch.zeros_like(b), b.clone()
    r0, p = r.clone(), r.clone()
    rho, bn = dot(r0, r), torch.linalg.vector_norm(b, dim=(0, 1))
    for _ in range(most):
        v = apply(p)
        a = rho / dot(r0, v)
        sv = r - a * v
        t = apply(sv)
        w = dot(t, sv) / dot(t, t)
        x += a * p + w * sv
        r = sv - w * t
        if bool((torch.linalg.vector_norm(r, dim=(0, 1)) <= tol * bn).all()):
            return x
        new = dot(r0, r)
        p = r + (new / rho) * (a / w) * (p - w * v)
        rho = new
    return None


def exact(case, seed):
    op, dims = case["op"], _dims(case)
    if op in ("dwc", "schur", "solve"):
        U, psi, kappa = _fine_inputs(case, seed)
        A = _clover_dense(U, dims, kappa)
        if op == "dwc":
            return _columns(lambda p: _clover(A, p) - kappa * _hop(U, p, dims), psi)
        if op == "solve":
            return _bicgstab(lambda p: _clover(A, p) - kappa * _hop(U, p, dims), psi, 1e-12, 600)
        ev, od = _parity_sites(dims, 0), _parity_sites(dims, 1)
        Ai = torch.linalg.inv(A[od])

        def schur(p):
            full = torch.zeros(_vol(case), 12, p.shape[-1], device=DEV, dtype=p.dtype)
            full[ev] = p
            odd = _clover(Ai, _hop(U, full, dims)[od])
            full.zero_()
            full[od] = odd
            return _clover(A[ev], p) - kappa * kappa * _hop(U, full, dims)[ev]

        return _columns(schur, psi)
    if op == "intergrid":
        nv, idx = case["nv"], _agg_index(dims)
        W = _basis(case, seed)[idx].reshape(-1, 256, nv, 2, 6).permute(0, 3, 1, 4, 2).reshape(-1, 2, 1536, nv).contiguous()
        for _ in range(2):  # Q of the thin QR with a positive diagonal, by Cholesky of the Gram matrix, twice
            G = torch.matmul(_dag(W).contiguous(), W)
            Ri = torch.linalg.inv(_dag(torch.linalg.cholesky(G)))
            W = torch.matmul(W, Ri.contiguous())
        fine = _gauss(_gen(seed, 2), (_vol(case), 12, case["n"]), _dtype(case))
        coarse = _gauss(_gen(seed, 5), (idx.shape[0], 2 * nv, case["n"]), _dtype(case))

        def down(f):
            x = f[idx].reshape(-1, 256, 2, 6, f.shape[-1]).permute(0, 2, 1, 3, 4).reshape(-1, 2, 1536, f.shape[-1])
            return torch.matmul(_dag(W).contiguous(), x.contiguous()).reshape(-1, 2 * nv, f.shape[-1])

        def up(y):
            x = torch.matmul(W, y.reshape(-1, 2, nv, y.shape[-1]).contiguous())
            x = x.reshape(-1, 2, 256, 6, y.shape[-1]).permute(0, 2, 1, 3, 4).reshape(-1, 256, 12, y.shape[-1])
            out = torch.empty(_vol(case), 12, y.shape[-1], device=DEV, dtype=y.dtype)
            out[idx.reshape(-1)] = x.reshape(-1, 12, y.shape[-1])
            return out

        return [_columns(down, fine), _columns(up, coarse)]
    if op == "coarse":
        B = _blocks(case, seed)
        return _columns(lambda e: _stencil(B, e, dims), _coarse_vec(case, seed), 64)
    if op == "coarse_mr":
        B, r = _blocks(case, seed), _coarse_vec(case, seed).to(torch.complex128)
        x = torch.zeros_like(r)
        for _ in range(case["iters"]):
            p = _stencil(B, r, dims)
            pp = (p.abs() ** 2).sum((0, 1))
            if bool((pp < 1e-30).any()):
                break
            a = (p.conj() * r).sum((0, 1)) / pp
            x += a * r
            r -= a * p
        return x
    if op == "gram_schmidt":
        g = _gen(seed, 2)
        shape = (_vol(case), 12, case["n"])
        w = _gauss(g, shape, _dtype(case)).to(torch.complex128)
        y, h = w.clone(), []
        for _ in range(case["m"]):
            v = (_gauss(g, shape, _dtype(case)) / math.sqrt(2 * 12 * _vol(case))).to(torch.complex128)
            h.append((v.conj() * w).sum((0, 1)))
            y -= h[-1] * v
        return [torch.stack(h), (y.abs() ** 2).sum((0, 1)), y]
    raise ValueError(op)
