"""GPU parity of the multigrid pieces against the FP64 oracle: block
orthonormalisation, restriction / prolongation, block normalisation, the
coarse stencil (FP64, FP32, BF16 and FP16 matrix cores) and the Galerkin
construction of the coarse blocks.

Tolerances (relative L2 unless stated):
  FP64 paths      1e-12  (same operations as the oracle, other summation order)
  FP32 paths      1e-6   (unit roundoff 6e-8 times a short sum; expected ~1e-7)
  BF16/FP16 paths 2e-2 against the oracle on the original operands, and
                  1e-6 against the oracle on the same rounded operands (the
                  MFMA products are exact, only the FP32 accumulation rounds)
"""

import numpy as np
import pytest

import oracle as O
import synth

pytestmark = pytest.mark.gpu

KAPPA, CSW = 0.13, 1.0


def rel(a, b):
    a = np.asarray(a, dtype=np.complex128)
    b = np.asarray(b, dtype=np.complex128)
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def dev(a):
    import torch

    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    return t.cpu().numpy()


def make_mg(mrhs, dims, blocks, n_v, U=None, t_bc=-1):
    ctx = mrhs.Context(dims, t_bc=t_bc)
    if U is not None:
        ctx.set_gauge(U)
        ctx.build_clover(CSW, KAPPA)
    return ctx, mrhs.Multigrid(ctx, blocks, n_v)


# ---- basis and intergrid -------------------------------------------------------------

GEOMS = [
    # dims, block, n_v
    ((8, 8, 8, 8), (4, 4, 4, 4), 16),
    ((4, 8, 4, 6), (2, 4, 2, 3), 8),
    ((4, 4, 2, 2), (2, 2, 2, 1), 4),
]


@pytest.mark.parametrize("dims,block,nv", GEOMS)
def test_block_orthonormalise(gpu_lib, dims, block, nv):
    ctx, mg = make_mg(gpu_lib, dims, [block], [nv])
    V = synth.volume(dims)
    v = synth.gaussian_vectors(V, nv, 12, 31)
    mg.set_basis(0, v)
    np.testing.assert_array_equal(mg.get_basis(0), v)  # round trip through the internal layout
    mg.block_orthonormalise(0)
    got = mg.get_basis(0)
    want = O.block_orthonormalise(v, dims, block)
    assert np.max(np.abs(got - want)) < 1e-12


def test_block_orthonormalise_rank_deficient(gpu_lib):
    dims, block = (4, 4, 4, 4), (2, 2, 2, 2)
    ctx, mg = make_mg(gpu_lib, dims, [block], [4])
    v = synth.gaussian_vectors(synth.volume(dims), 4, 12, 5)
    v[:, 3] = v[:, 1]  # vector 3 repeats vector 1 everywhere
    mg.set_basis(0, v)
    with pytest.raises(gpu_lib.MrhsError, match="STATE"):
        mg.block_orthonormalise(0)


@pytest.mark.parametrize("dims,block,nv", GEOMS)
@pytest.mark.parametrize("nrhs", [1, 5, 24, 64])
@pytest.mark.parametrize("dt", [np.complex64, np.complex128])
def test_restrict_prolong(gpu_lib, dims, block, nv, nrhs, dt):
    import torch

    ctx, mg = make_mg(gpu_lib, dims, [block], [nv])
    V = synth.volume(dims)
    basis = O.block_orthonormalise(synth.gaussian_vectors(V, nv, 12, 3), dims, block)
    mg.set_basis(0, basis)
    b_used = basis.astype(dt).astype(np.complex128)  # the kernel's basis precision
    f = synth.spinor_source(dims, nrhs, 40, dt)
    Vc = mg.volume[1]
    y = torch.empty((Vc, 2 * nv, nrhs), dtype=torch.complex64 if dt == np.complex64 else torch.complex128,
                    device="cuda")
    mg.restrict(0, y, dev(f))
    tol = 1e-6 if dt == np.complex64 else 1e-12
    assert rel(host(y), O.restrict(b_used, f, dims, block)) < tol
    yc = synth.coarse_source(Vc, 2 * nv, nrhs, 70, dt)
    fo = torch.empty((V, 12, nrhs), dtype=y.dtype, device="cuda")
    mg.prolong(0, fo, dev(yc))
    assert rel(host(fo), O.prolong(b_used, yc, dims, block)) < tol


def test_restrict_prolong_coarse_level(gpu_lib):
    """Step 1 (coarse -> coarser) with 16 components per chirality, in FP64."""
    import torch

    dims = (4, 4, 4, 4)
    ctx, mg = make_mg(gpu_lib, dims, [(2, 2, 2, 2), (2, 1, 2, 1)], [16, 8])
    d1 = mg.dims[1]
    V1 = mg.volume[1]
    basis = O.block_orthonormalise(synth.gaussian_vectors(V1, 8, 32, 8), d1, (2, 1, 2, 1))
    mg.set_basis(1, basis)
    f = synth.coarse_source(V1, 32, 7, 9)
    y = torch.empty((mg.volume[2], 16, 7), dtype=torch.complex128, device="cuda")
    mg.restrict(1, y, dev(f))
    assert rel(host(y), O.restrict(basis, f, d1, (2, 1, 2, 1))) < 1e-12
    yc = synth.coarse_source(mg.volume[2], 16, 7, 10)
    fo = torch.empty((V1, 32, 7), dtype=torch.complex128, device="cuda")
    mg.prolong(1, fo, dev(yc))
    assert rel(host(fo), O.prolong(basis, yc, d1, (2, 1, 2, 1))) < 1e-12


@pytest.mark.parametrize("nrhs", [3, 4, 33])
def test_restrict_prolong_coarse_level_f32(gpu_lib, nrhs):
    """FP32 step 1 with n_v = 16 on 16-site aggregates (the matrix-core intergrid from 4 RHS on)."""
    import torch

    dims = (8, 8, 8, 8)
    blocks = [(2, 2, 2, 2), (2, 2, 2, 2)]
    ctx, mg = make_mg(gpu_lib, dims, blocks, [16, 16])
    d1 = mg.dims[1]
    V1 = mg.volume[1]
    basis = O.block_orthonormalise(synth.gaussian_vectors(V1, 16, 32, 12), d1, blocks[1])
    mg.set_basis(1, basis)
    b_used = basis.astype(np.complex64).astype(np.complex128)
    f = synth.coarse_source(V1, 32, nrhs, 13, np.complex64)
    y = torch.empty((mg.volume[2], 32, nrhs), dtype=torch.complex64, device="cuda")
    mg.restrict(1, y, dev(f))
    assert rel(host(y), O.restrict(b_used, f, d1, blocks[1])) < 1e-6
    yc = synth.coarse_source(mg.volume[2], 32, nrhs, 14, np.complex64)
    fo = torch.empty((V1, 32, nrhs), dtype=torch.complex64, device="cuda")
    mg.prolong(1, fo, dev(yc))
    assert rel(host(fo), O.prolong(b_used, yc, d1, blocks[1])) < 1e-6


@pytest.mark.parametrize("nrhs", [1, 7, 24, 33, 64])
def test_restrict_prolong_bf16(gpu_lib, nrhs):
    """Matrix-core BF16 restrict/prolong (FP32 fields, FP32 accumulation) on
    both steps of an 8^4 -> 2^4 -> 1^4 hierarchy: against the oracle on the
    same BF16-rounded operands (exact products, so only the FP32
    accumulation differs) and against the exact FP32-basis result within the
    BF16 bar.  Nrhs covers a partial 32-column tile, several tiles and a
    ragged tail."""
    import torch

    dims = (8, 8, 8, 8)
    blocks = [(4, 4, 4, 4), (2, 2, 2, 2)]
    ctx, mg = make_mg(gpu_lib, dims, blocks, [16, 16])
    for lev in (0, 1):
        d = mg.dims[lev]
        V = mg.volume[lev]
        nc = mg.ncomp[lev]
        basis = O.block_orthonormalise(synth.gaussian_vectors(V, 16, nc, 60 + lev), d, blocks[lev])
        mg.set_basis(lev, basis)
        b32 = basis.astype(np.complex64)
        f = synth.coarse_source(V, nc, nrhs, 61 + lev, np.complex64)
        y = torch.empty((mg.volume[lev + 1], 32, nrhs), dtype=torch.complex64, device="cuda")
        mg.restrict(lev, y, dev(f), prec="bf16")
        got = host(y)
        assert rel(got, O.restrict_lowprec(b32, f, d, blocks[lev])) < 2e-6
        assert rel(got, O.restrict(b32, f, d, blocks[lev])) < 2e-2
        yc = synth.coarse_source(mg.volume[lev + 1], 32, nrhs, 62 + lev, np.complex64)
        fo = torch.empty((V, nc, nrhs), dtype=torch.complex64, device="cuda")
        mg.prolong(lev, fo, dev(yc), prec="bf16")
        got = host(fo)
        assert rel(got, O.prolong_lowprec(b32, yc, d, blocks[lev])) < 2e-6
        assert rel(got, O.prolong(b32, yc, d, blocks[lev])) < 2e-2


@pytest.mark.parametrize("dims,block,level", [
    ((4, 4, 4, 4), (2, 2, 2, 2), 0),    # 16 sites: one tile, prolongation in one part
    ((4, 6, 4, 6), (4, 2, 2, 3), 0),    # 48 sites: an odd number of tiles, 12 aggregates over 8 XCDs
    ((12, 12, 8, 8), (4, 4, 4, 4), 0),  # 36 aggregates: every restriction staged
    ((4, 4, 6, 4), (2, 2, 2, 2), 1),    # step 1: 32 components of the 16-site aggregates of a coarse level
])
@pytest.mark.parametrize("nrhs", [1, 4, 16, 17, 31, 33, 63])
def test_restrict_prolong_tiles(gpu_lib, dims, block, level, nrhs):
    """The tiled matrix-core transfers at the edges of their tiles (sites per
    aggregate, odd column counts, one and two column tiles) and where they
    leave the shape to the other kernels; FP32 and BF16 as in the tests above."""
    import torch

    blocks = [block] if level == 0 else [(2, 2, 2, 2), block]
    fine = dims if level == 0 else tuple(2 * d for d in dims)
    ctx, mg = make_mg(gpu_lib, fine, blocks, [16] * len(blocks))
    V, nc = mg.volume[level], mg.ncomp[level]
    basis = synth.gaussian_vectors(V, 16, nc, 71) / np.sqrt(2.0 * nc * np.prod(block))
    mg.set_basis(level, basis)
    b32 = basis.astype(np.complex64)
    f = synth.coarse_source(V, nc, nrhs, 72, np.complex64)
    yc = synth.coarse_source(mg.volume[level + 1], 32, nrhs, 73, np.complex64)
    y = torch.empty((mg.volume[level + 1], 32, nrhs), dtype=torch.complex64, device="cuda")
    fo = torch.empty((V, nc, nrhs), dtype=torch.complex64, device="cuda")
    mg.restrict(level, y, dev(f))
    assert rel(host(y), O.restrict(b32.astype(np.complex128), f, dims, block)) < 1e-6
    mg.prolong(level, fo, dev(yc))
    assert rel(host(fo), O.prolong(b32.astype(np.complex128), yc, dims, block)) < 1e-6
    mg.restrict(level, y, dev(f), prec="bf16")
    assert rel(host(y), O.restrict_lowprec(b32, f, dims, block)) < 2e-6
    mg.prolong(level, fo, dev(yc), prec="bf16")
    assert rel(host(fo), O.prolong_lowprec(b32, yc, dims, block)) < 2e-6


@pytest.mark.parametrize("dims,block,level", [((12, 12, 12, 12), (4, 4, 4, 4), 0), ((10, 10, 6, 6), (2, 2, 2, 2), 1)])
@pytest.mark.parametrize("nrhs", [33, 50, 64])
def test_restrict_prolong_two_column_tiles(gpu_lib, dims, block, level, nrhs):
    """Two column tiles in one workgroup, on the aggregates (81 and 225) where
    these kernels are chosen: against the oracle with the bars of
    test_restrict_prolong_tiles."""
    from test_intergrid_rule_host import staged_leads

    for prec in ("f32", "bf16"):
        for prolong in (False, True):
            assert staged_leads(prec, prolong, dims, block, 6 if level == 0 else 16, nrhs)
    test_restrict_prolong_tiles(gpu_lib, dims, block, level, nrhs)


def test_restrict_prolong_bf16_unsupported(gpu_lib):
    """n_v = 8 has no matrix-core intergrid path: a clear UNSUPPORTED error."""
    import torch

    dims, block = (4, 4, 4, 4), (2, 2, 2, 2)
    ctx, mg = make_mg(gpu_lib, dims, [block], [8])
    mg.set_basis(0, O.block_orthonormalise(synth.gaussian_vectors(256, 8, 12, 1), dims, block))
    y = torch.empty((16, 16, 4), dtype=torch.complex64, device="cuda")
    f = torch.zeros((256, 12, 4), dtype=torch.complex64, device="cuda")
    with pytest.raises(gpu_lib.MrhsError, match="UNSUPPORTED"):
        mg.restrict(0, y, f, prec="bf16")


def test_intergrid_full_size(gpu_lib):
    """24^4 fine lattice, 4^4 aggregates, 16 Gaussian vectors block-orthonormalised
    in FP64 on the GPU, restrict / prolong / block-normalise of Nrhs = 24 FP32 fields."""
    import torch

    dims, block, nv, nrhs = (24, 24, 24, 24), (4, 4, 4, 4), 16, 24
    ctx, mg = make_mg(gpu_lib, dims, [block], [nv])
    V = synth.volume(dims)
    v = synth.gaussian_vectors(V, nv, 12, 2024)
    mg.set_basis(0, v)
    mg.block_orthonormalise(0)
    basis = O.block_orthonormalise(v, dims, block)
    assert np.max(np.abs(mg.get_basis(0) - basis)) < 1e-12
    b32 = basis.astype(np.complex64).astype(np.complex128)
    f = synth.spinor_source(dims, nrhs, 500, np.complex64)
    y = torch.empty((mg.volume[1], 32, nrhs), dtype=torch.complex64, device="cuda")
    tf = dev(f)
    mg.restrict(0, y, tf)
    assert rel(host(y), O.restrict(b32, f, dims, block)) < 1e-6
    fo = torch.empty_like(tf)
    mg.prolong(0, fo, y)
    assert rel(host(fo), O.prolong(b32, host(y), dims, block)) < 1e-6
    # the matrix-core BF16 path at the same size, against the rounded-operand oracle
    yb = torch.empty_like(y)
    mg.restrict(0, yb, tf, prec="bf16")
    assert rel(host(yb), O.restrict_lowprec(b32, f, dims, block)) < 2e-6
    fb = torch.empty_like(tf)
    mg.prolong(0, fb, y, prec="bf16")
    assert rel(host(fb), O.prolong_lowprec(b32, host(y), dims, block)) < 2e-6
    norms = torch.empty((mg.volume[1], 2, nrhs), dtype=torch.float64, device="cuda")
    mg.block_normalise(0, tf, norms)
    want, want_n = O.block_normalise(f, dims, block)
    assert rel(host(tf), want) < 1e-6
    np.testing.assert_allclose(host(norms), want_n, rtol=1e-12)


@pytest.mark.parametrize("dt", [np.complex64, np.complex128])
def test_block_normalise_small(gpu_lib, dt):
    import torch

    dims, block = (4, 8, 4, 6), (2, 4, 2, 3)
    ctx, mg = make_mg(gpu_lib, dims, [block], [8])
    f = synth.spinor_source(dims, 5, 1, dt)
    f[:32] = 0  # some all-zero blocks stay zero
    t = dev(f)
    norms = torch.empty((mg.volume[1], 2, 5), dtype=torch.float64, device="cuda")
    mg.block_normalise(0, t, norms)
    want, want_n = O.block_normalise(f, dims, block)
    assert rel(host(t), want) < (1e-6 if dt == np.complex64 else 1e-13)
    np.testing.assert_allclose(host(norms), want_n, rtol=1e-12, atol=0)


@pytest.mark.parametrize("nrhs", [2, 12, 24, 26, 28, 64])
def test_block_normalise_even_nrhs(gpu_lib, nrhs):
    """FP32, even Nrhs on 4^4 aggregates (1536 rows of 6 components): the single-pass
    kernel with the columns split into parts of 8 (24: three parts, 64: eight) or whole
    (2), the one with up to 20 rows per thread (12, and 26 with ragged last rows), the
    two-pass one beyond (28)."""
    import torch

    dims, block = (8, 8, 8, 8), (4, 4, 4, 4)
    ctx, mg = make_mg(gpu_lib, dims, [block], [4])
    f = synth.spinor_source(dims, nrhs, 77, np.complex64)
    f[:4] = 0  # sites 0..3 lie in aggregate 0: their rows are zero, the block is not
    f[synth.volume(dims) // 2:] = 0  # whole aggregates of zeros stay zero
    t = dev(f)
    norms = torch.empty((mg.volume[1], 2, nrhs), dtype=torch.float64, device="cuda")
    mg.block_normalise(0, t, norms)
    want, want_n = O.block_normalise(f, dims, block)
    assert rel(host(t), want) < 1e-6
    np.testing.assert_allclose(host(norms), want_n, rtol=1e-12, atol=0)


# ---- coarse stencil --------------------------------------------------------------------

def coarse_mg(mrhs, cdims, nb):
    """A hierarchy whose level 1 has lattice cdims and nb components (blocks set directly)."""
    fine = tuple(2 * c for c in cdims)
    return make_mg(mrhs, fine, [(2, 2, 2, 2)], [nb // 2])


@pytest.mark.parametrize("cdims", [(6, 6, 6, 6), (3, 3, 3, 3), (2, 3, 1, 2)])
@pytest.mark.parametrize("nrhs", [1, 12, 24, 48, 64])
def test_coarse_apply_all_precisions(gpu_lib, cdims, nrhs):
    import torch

    nb = 32
    ctx, mg = coarse_mg(gpu_lib, cdims, nb)
    Vc = synth.volume(cdims)
    B = synth.gaussian_blocks(Vc, nb, 7)
    mg.set_blocks(1, B)
    np.testing.assert_array_equal(mg.get_blocks(1), B)
    e64 = synth.coarse_source(Vc, nb, nrhs, 11)
    e32 = e64.astype(np.complex64)
    want64 = O.coarse_apply(B, e64, cdims)
    out = torch.empty((Vc, nb, nrhs), dtype=torch.complex128, device="cuda")
    mg.coarse_apply(1, out, dev(e64), "f64")
    assert rel(host(out), want64) < 1e-12
    B32 = B.astype(np.complex64)
    want32 = O.coarse_apply(B32, e32, cdims)
    o32 = torch.empty((Vc, nb, nrhs), dtype=torch.complex64, device="cuda")
    mg.coarse_apply(1, o32, dev(e32), "f32")
    assert rel(host(o32), want32) < 1e-6
    for fmt in ("bf16", "f16"):
        o = torch.empty_like(o32)
        mg.coarse_apply(1, o, dev(e32), fmt)
        got = host(o)
        assert rel(got, O.coarse_apply(B, e32, cdims)) < 2e-2, fmt
        assert rel(got, O.coarse_apply_lowprec(B, e32, cdims, fmt)) < 1e-6, fmt


@pytest.mark.parametrize("cdims", [(6, 6, 6, 6), (3, 3, 3, 3)])
def test_coarse_tune_keeps_parity(gpu_lib, cdims):
    """mrhs_mg_tune picks the FP32 stencil kernel per nrhs; whichever it picks matches
    the oracle on the FP32-rounded blocks (1e-6)."""
    import torch

    nb = 32
    ctx, mg = coarse_mg(gpu_lib, cdims, nb)
    Vc = synth.volume(cdims)
    B = synth.gaussian_blocks(Vc, nb, 17)
    mg.set_blocks(1, B)
    ns = [1, 12, 33]
    mg.tune(ns)
    B32 = B.astype(np.complex64)
    for n in ns:
        assert mg.get_tuning(1, n) in ("mfma", "valu")
        e32 = synth.coarse_source(Vc, nb, n, 19, np.complex64)
        o = torch.empty((Vc, nb, n), dtype=torch.complex64, device="cuda")
        mg.coarse_apply(1, o, dev(e32), "f32")
        assert rel(host(o), O.coarse_apply(B32, e32, cdims)) < 1e-6, (n, mg.get_tuning(1, n))


@pytest.mark.parametrize("cdims", [(6, 6, 6, 6), (3, 3, 3, 3), (2, 3, 1, 2)])
@pytest.mark.parametrize("cfg", [0, 1, 2, 3, 4, 5])
def test_coarse_lowp_launch_shapes(gpu_lib, cdims, cfg):
    """Every launch shape of the BF16/FP16 stencil (four or eight wavefronts per
    site, one or two 32-column tiles per workgroup, the two separate or as
    interleaved column pairs) against the oracle on the rounded operands (1e-6)
    and on the exact ones (2e-2), with ragged column counts (1, 33, 40) as well
    as full tiles (odd counts run the pair shapes as two separate tiles); per
    column the result equals the column applied alone (same shape)."""
    import torch

    nb = 32
    ctx, mg = coarse_mg(gpu_lib, cdims, nb)
    Vc = synth.volume(cdims)
    B = synth.gaussian_blocks(Vc, nb, 23)
    mg.set_blocks(1, B)
    for n in (1, 12, 33, 40, 64):
        mg.set_lowp_cfg(1, n, cfg)
        assert mg.get_lowp_tuning(1, n)["cfg"] == cfg
        e32 = synth.coarse_source(Vc, nb, n, 29, np.complex64)
        for fmt in ("bf16", "f16"):
            o = torch.empty((Vc, nb, n), dtype=torch.complex64, device="cuda")
            mg.coarse_apply(1, o, dev(e32), fmt)
            got = host(o)
            assert rel(got, O.coarse_apply_lowprec(B, e32, cdims, fmt)) < 1e-6, (n, fmt)
            assert rel(got, O.coarse_apply(B, e32, cdims)) < 2e-2, (n, fmt)
        if n == 40:
            mg.set_lowp_cfg(1, 1, cfg)
            for k in (0, 39):
                ok = torch.empty((Vc, nb, 1), dtype=torch.complex64, device="cuda")
                mg.coarse_apply(1, ok, dev(np.ascontiguousarray(e32[:, :, k:k + 1])), "bf16")
                o = torch.empty((Vc, nb, n), dtype=torch.complex64, device="cuda")
                mg.coarse_apply(1, o, dev(e32), "bf16")
                np.testing.assert_array_equal(host(ok)[:, :, 0], host(o)[:, :, k])


@pytest.mark.parametrize("cdims", [(6, 6, 6, 6), (3, 3, 3, 3)])
@pytest.mark.parametrize("cfg", [4, 5])
def test_coarse_lowp_pair_shapes_even_counts(gpu_lib, cdims, cfg):
    """The interleaved column-pair shapes at even column counts that leave
    the last pairs of a 64-column group empty (2, 30) or one pair short (62):
    against the rounded-operand oracle (1e-6), and each column equal to the
    column applied alone."""
    import torch

    nb = 32
    ctx, mg = coarse_mg(gpu_lib, cdims, nb)
    Vc = synth.volume(cdims)
    B = synth.gaussian_blocks(Vc, nb, 27)
    mg.set_blocks(1, B)
    for n in (2, 30, 62):
        mg.set_lowp_cfg(1, n, cfg)
        e32 = synth.coarse_source(Vc, nb, n, 31, np.complex64)
        for fmt in ("bf16", "f16"):
            o = torch.empty((Vc, nb, n), dtype=torch.complex64, device="cuda")
            mg.coarse_apply(1, o, dev(e32), fmt)
            assert rel(host(o), O.coarse_apply_lowprec(B, e32, cdims, fmt)) < 1e-6, (n, fmt)
        o = torch.empty((Vc, nb, n), dtype=torch.complex64, device="cuda")
        mg.coarse_apply(1, o, dev(e32), "bf16")
        mg.set_lowp_cfg(1, 1, cfg - 4)  # one column: the same wavefronts, one tile
        for k in (0, n - 1):
            ok = torch.empty((Vc, nb, 1), dtype=torch.complex64, device="cuda")
            mg.coarse_apply(1, ok, dev(np.ascontiguousarray(e32[:, :, k:k + 1])), "bf16")
            np.testing.assert_array_equal(host(ok)[:, :, 0], host(o)[:, :, k])


def test_coarse_tune_lowp_keeps_parity(gpu_lib):
    """mrhs_mg_tune also picks the BF16/FP16 launch shape per Nrhs; whichever
    it picks matches the rounded-operand oracle."""
    import torch

    cdims, nb = (3, 3, 3, 3), 32
    ctx, mg = coarse_mg(gpu_lib, cdims, nb)
    Vc = synth.volume(cdims)
    B = synth.gaussian_blocks(Vc, nb, 31)
    mg.set_blocks(1, B)
    ns = [12, 48, 64]
    mg.tune(ns)
    for n in ns:
        assert mg.get_lowp_tuning(1, n)["cfg"] in range(6)
        e32 = synth.coarse_source(Vc, nb, n, 37, np.complex64)
        for fmt in ("bf16", "f16"):
            o = torch.empty((Vc, nb, n), dtype=torch.complex64, device="cuda")
            mg.coarse_apply(1, o, dev(e32), fmt)
            assert rel(host(o), O.coarse_apply_lowprec(B, e32, cdims, fmt)) < 1e-6, (n, fmt)


def _mr_ref(B, b, cdims, iters, fmt):
    """iters minimal-residual steps from zero on the coarse stencil B, with the
    device's number formats: the stencil on BF16-rounded operands with exact
    products (fmt "bf16") or on FP32-rounded blocks (fmt "f32"); p, r and x kept
    in FP32; alpha = <p, r> / ||p||^2 per column in FP64, rounded to FP32 for
    the updates."""
    r = np.asarray(b, dtype=np.complex64)
    x = np.zeros_like(r)
    B32 = np.asarray(B).astype(np.complex64)
    for _ in range(iters):
        if fmt == "bf16":
            p = O.coarse_apply_lowprec(B, r, cdims, "bf16").astype(np.complex64)
        else:
            p = O.coarse_apply(B32, r, cdims).astype(np.complex64)
        p64, r64 = p.astype(np.complex128), r.astype(np.complex128)
        num = np.einsum("sck,sck->k", p64.conj(), r64)
        den = np.einsum("sck,sck->k", p64.conj(), p64).real
        a = np.where(den > 0, num / np.where(den > 0, den, 1.0), 0.0).astype(np.complex64).astype(np.complex128)
        x = (x.astype(np.complex128) + a * r64).astype(np.complex64)
        r = (r64 - a * p64).astype(np.complex64)
    return x


@pytest.mark.parametrize("cdims,cfg,prec", [
    ((3, 3, 3, 3), 0, "bf16"), ((3, 3, 3, 3), 1, "bf16"), ((3, 3, 3, 3), 2, "bf16"), ((3, 3, 3, 3), 3, "bf16"),
    ((3, 3, 3, 3), 5, "bf16"),
    ((3, 3, 3, 2), 0, "bf16"),
    ((6, 6, 6, 6), 0, "bf16"),
    ((3, 3, 3, 3), 0, "f32"),
])
def test_coarse_mr_solve_vs_emulation(gpu_lib, cdims, cfg, prec):
    """The coarsest-level MR solve: on levels of at most 1024 sites with BF16
    operands every step is one fused launch (stencil, per-site partial sums,
    update on the fly) and a small one that sums the partials into the step
    length; 6^4 (1296 sites) and FP32 take the separate kernels.  Against an FP64 emulation of the same
    iteration in the device's number formats, for 1, 12, 40 and 64 RHS: one
    step agrees to the FP32 accumulation order (1e-5); over 16 steps an FP32
    rounding difference can move an operand across a BF16 rounding boundary
    (one BF16 ulp, 2^-8), so the bar there is 2e-3 (FP32 path: 1e-5), and the
    residual reduction must match the emulation's."""
    import torch

    nb = 32
    ctx, mg = coarse_mg(gpu_lib, cdims, nb)
    Vc = synth.volume(cdims)
    B = synth.gaussian_blocks(Vc, nb, 41, shift=24.0)  # a shift that lets MR converge
    mg.set_blocks(1, B)
    for n in (1, 12, 40, 64):
        mg.set_lowp_cfg(1, n, cfg)
        b = synth.coarse_source(Vc, nb, n, 43, np.complex64)
        for iters, tol in ((1, 1e-5), (16, 2e-3 if prec == "bf16" else 1e-5)):
            x = torch.empty((Vc, nb, n), dtype=torch.complex64, device="cuda")
            mg.coarse_mr_solve(1, x, dev(b), iters, prec)
            want = _mr_ref(B, b, cdims, iters, prec)
            got = host(x)
            assert rel(got, want) < tol, (n, iters, rel(got, want))
            if iters == 16:
                res = np.linalg.norm(b - O.coarse_apply(B, got, cdims)) / np.linalg.norm(b)
                res_ref = np.linalg.norm(b - O.coarse_apply(B, want, cdims)) / np.linalg.norm(b)
                assert res < 0.5 and abs(res - res_ref) < 0.01 * res_ref, (n, res, res_ref)
                if n == 12:  # deterministic: a second call gives the same bits
                    x2 = torch.empty_like(x)
                    mg.coarse_mr_solve(1, x2, dev(b), iters, prec)
                    assert torch.equal(x, x2)


@pytest.mark.parametrize("cdims,nrhs", [
    ((1, 1, 1, 1), 1), ((2, 2, 1, 3), 16), ((2, 2, 1, 3), 17), ((3, 3, 3, 15), 1), ((3, 3, 3, 15), 15),
    ((3, 3, 3, 15), 20), ((3, 3, 3, 15), 33), ((4, 4, 4, 9), 16), ((4, 4, 4, 9), 18), ((4, 4, 4, 9), 33),
])
def test_coarse_mr_solve_step_forms(gpu_lib, cdims, nrhs):
    """The forms of the fused MR step at their edges: half-column loads up to 16
    RHS, one or two sites per workgroup (an odd count leaves half of the last
    one empty), the step length summed by the next launch (up to 256 rows of
    partial sums) or by one of its own.  Against the emulation of
    test_coarse_mr_solve_vs_emulation with its bars (one step 1e-5, more steps
    2e-3), for both wavefront counts, and bit for bit on a second call."""
    import torch

    nb = 32
    ctx, mg = coarse_mg(gpu_lib, cdims, nb)
    Vc = synth.volume(cdims)
    B = synth.gaussian_blocks(Vc, nb, 47, shift=24.0)
    mg.set_blocks(1, B)
    b = synth.coarse_source(Vc, nb, nrhs, 53, np.complex64)
    for iters, tol in ((1, 1e-5), (4, 2e-3)):
        want = _mr_ref(B, b, cdims, iters, "bf16")
        for cfg in (0, 1, 2, 3):
            mg.set_lowp_cfg(1, nrhs, cfg)
            x, x2 = (torch.empty((Vc, nb, nrhs), dtype=torch.complex64, device="cuda") for _ in range(2))
            mg.coarse_mr_solve(1, x, dev(b), iters, "bf16")
            mg.coarse_mr_solve(1, x2, dev(b), iters, "bf16")
            assert rel(host(x), want) < tol, (iters, cfg, rel(host(x), want))
            assert torch.equal(x, x2)


@pytest.mark.parametrize("nrhs", [1, 15, 16, 17])
@pytest.mark.parametrize("fmt", ["bf16", "f16"])
def test_coarse_half_column_loads(gpu_lib, nrhs, fmt):
    """Up to 16 RHS the BF16/FP16 stencil splits each column's rows over two
    lanes: full, hop and self modes against the oracle on the rounded operands
    (1e-6) around the switch, for both wavefront counts of the full stencil."""
    import torch

    cdims, nb = (2, 4, 2, 6), 32
    ctx, mg = coarse_mg(gpu_lib, cdims, nb)
    Vc = synth.volume(cdims)
    B = synth.gaussian_blocks(Vc, nb, 59)
    mg.set_blocks(1, B)
    e = synth.coarse_source(Vc, nb, nrhs, 61, np.complex64)
    want = O.coarse_apply_lowprec(B, e, cdims, fmt)
    for cfg in (0, 1):
        mg.set_lowp_cfg(1, nrhs, cfg)
        o = torch.empty((Vc, nb, nrhs), dtype=torch.complex64, device="cuda")
        mg.coarse_apply(1, o, dev(e), fmt)
        assert rel(host(o), want) < 1e-6, cfg
    # hop from parity 1 plus self on parity 0 of a field living on both: the full stencil's even rows
    site = np.arange(Vc)
    par, r = np.zeros(Vc, dtype=int), site.copy()
    for L in cdims:
        par += r % L
        r //= L
    par &= 1
    ev, od = np.flatnonzero(par == 0), np.flatnonzero(par == 1)
    hop, own = (torch.empty((Vc // 2, nb, nrhs), dtype=torch.complex64, device="cuda") for _ in range(2))
    mg.coarse_hop_eo(1, hop, dev(np.ascontiguousarray(e[od])), 0, fmt)
    mg.coarse_self_eo(1, own, dev(np.ascontiguousarray(e[ev])), 0, False, fmt)
    # FP16 scales are powers of two per field, so the operands round as in the full apply
    assert rel(host(hop) + host(own), want[ev]) < 1e-6


@pytest.mark.parametrize("nrhs", [5, 16, 24, 40])
def test_a_column_of_nan_and_infinity_stays_alone(gpu_lib, nrhs):
    """NaN and infinities in one right-hand side leave the bits of the others as
    they are without them: staged transfers, the coarse stencils with half and
    whole columns, the MR solve whose steps sum their own lengths."""
    import torch

    ctx, mg = make_mg(gpu_lib, (12, 12, 12, 12), [(4, 4, 4, 4)], [16])
    V, Vc, nc = mg.volume[0], mg.volume[1], mg.ncomp[0]
    mg.set_basis(0, synth.gaussian_vectors(V, 16, nc, 81) / np.sqrt(2.0 * nc * 256))
    mg.set_blocks(1, synth.gaussian_blocks(Vc, 32, 82, shift=24.0))
    fine = dev(synth.coarse_source(V, nc, nrhs, 83, np.complex64))
    coarse = dev(synth.coarse_source(Vc, 32, nrhs, 84, np.complex64))
    bad = nrhs - 2
    calls = {}
    for prec in ("f32", "bf16"):
        calls["restrict " + prec] = (lambda y, x, p=prec: mg.restrict(0, y, x, p), coarse, fine)
        calls["prolong " + prec] = (lambda y, x, p=prec: mg.prolong(0, y, x, p), fine, coarse)
    for prec in ("bf16", "f16"):
        calls["stencil " + prec] = (lambda y, x, p=prec: mg.coarse_apply(1, y, x, p), coarse, coarse)
    calls["mr"] = (lambda y, x: mg.coarse_mr_solve(1, y, x, 6, "bf16"), coarse, coarse)
    others = [k for k in range(nrhs) if k != bad]
    for name, (call, like, x) in calls.items():
        out = []
        for values in (None, (complex(np.nan, 1.0), complex(np.inf, -np.inf))):
            y, xx = torch.empty_like(like), x.clone()
            if values:
                xx[::2, :, bad], xx[1::2, :, bad] = values
            call(y, xx)
            out.append(y)
        torch.cuda.synchronize()
        assert not torch.isfinite(torch.view_as_real(out[1][:, :, bad])).all(), name
        assert torch.equal(out[0][:, :, others], out[1][:, :, others]), name


def test_coarse_apply_nb8_valu(gpu_lib):
    import torch

    cdims, nb = (2, 2, 4, 2), 8
    ctx, mg = coarse_mg(gpu_lib, cdims, nb)
    Vc = synth.volume(cdims)
    B = synth.gaussian_blocks(Vc, nb, 3)
    mg.set_blocks(1, B)
    e = synth.coarse_source(Vc, nb, 6, 1)
    out = torch.empty((Vc, nb, 6), dtype=torch.complex128, device="cuda")
    mg.coarse_apply(1, out, dev(e), "f64")
    assert rel(host(out), O.coarse_apply(B, e, cdims)) < 1e-12
    with pytest.raises(gpu_lib.MrhsError, match="UNSUPPORTED"):
        mg.coarse_apply(1, out.to(torch.complex64), dev(e.astype(np.complex64)), "bf16")


def test_coarse_mfma_mrhs_equals_columns(gpu_lib):
    """Within one tile configuration each column of a batched BF16 apply equals
    the column applied alone (the per-column arithmetic does not depend on N)."""
    import torch

    cdims, nb = (3, 3, 3, 3), 32
    ctx, mg = coarse_mg(gpu_lib, cdims, nb)
    Vc = synth.volume(cdims)
    mg.set_blocks(1, synth.gaussian_blocks(Vc, nb, 9))
    e = synth.coarse_source(Vc, nb, 24, 2, np.complex64)
    out = torch.empty((Vc, nb, 24), dtype=torch.complex64, device="cuda")
    mg.coarse_apply(1, out, dev(e), "bf16")
    for k in (0, 13, 23):
        ok = torch.empty((Vc, nb, 1), dtype=torch.complex64, device="cuda")
        mg.coarse_apply(1, ok, dev(e[:, :, k:k + 1]), "bf16")
        np.testing.assert_array_equal(host(ok)[:, :, 0], host(out)[:, :, k])


# ---- Galerkin construction -------------------------------------------------------------

def test_galerkin_two_levels_vs_oracle(gpu_lib):
    """8^4 Haar links -> 2^4 (4^4 aggregates, extent-2 aliasing) -> 1^4 (2^4
    aggregates, extent-1 aliasing), n_v = 16 at both steps, FP64."""
    dims = (8, 8, 8, 8)
    U = synth.gauge_haar(dims, 12)
    A = O.clover_packed(U, dims, CSW, KAPPA)
    ctx, mg = make_mg(gpu_lib, dims, [(4, 4, 4, 4), (2, 2, 2, 2)], [16, 16], U=U)
    V = synth.volume(dims)
    v0 = synth.gaussian_vectors(V, 16, 12, 100)
    mg.set_basis(0, v0)
    mg.block_orthonormalise(0)
    b0 = O.block_orthonormalise(v0, dims, (4, 4, 4, 4))
    mg.build_coarse(1)
    B1 = O.galerkin_fine(U, A, KAPPA, b0, dims, (4, 4, 4, 4))
    got1 = mg.get_blocks(1)
    assert rel(got1, B1) < 1e-12
    d1 = mg.dims[1]
    v1 = synth.gaussian_vectors(mg.volume[1], 16, 32, 200)
    mg.set_basis(1, v1)
    mg.block_orthonormalise(1)
    b1 = O.block_orthonormalise(v1, d1, (2, 2, 2, 2))
    mg.build_coarse(2)
    B2 = O.galerkin_coarse(B1, b1, d1, (2, 2, 2, 2))
    assert rel(mg.get_blocks(2), B2) < 1e-12


def test_galerkin_nonaliasing_vs_oracle(gpu_lib):
    """Coarse extent 3 (12^4 Haar links, 4^4 aggregates -> 3^4), where the +mu
    and -mu neighbours of an aggregate are different sites: every block of
    every direction equals the oracle's Galerkin product (FP64, n_v = 16)."""
    dims = (12, 12, 12, 12)
    U = synth.gauge_haar(dims, 13)
    A = O.clover_packed(U, dims, CSW, KAPPA)
    ctx, mg = make_mg(gpu_lib, dims, [(4, 4, 4, 4)], [16], U=U)
    v0 = synth.gaussian_vectors(synth.volume(dims), 16, 12, 110)
    mg.set_basis(0, v0)
    mg.block_orthonormalise(0)
    mg.build_coarse(1)
    assert mg.dims[1] == (3, 3, 3, 3)
    want = O.galerkin_fine(U, A, KAPPA, O.block_orthonormalise(v0, dims, (4, 4, 4, 4)), dims, (4, 4, 4, 4))
    assert rel(mg.get_blocks(1), want) < 1e-12


def test_galerkin_coarse_nonaliasing_vs_oracle(gpu_lib):
    """The coarse-to-coarser Galerkin product at coarse extent 3: Gaussian
    level-1 blocks (+4 I on the self block) on 6^4 with 2^4 aggregates -> 3^4,
    n_v = 16, against the oracle's P^dag D_c P (FP64)."""
    dims = (12, 12, 12, 12)
    ctx, mg = make_mg(gpu_lib, dims, [(2, 2, 2, 2), (2, 2, 2, 2)], [16, 16])
    d1 = mg.dims[1]
    B1 = synth.gaussian_blocks(mg.volume[1], 32, 77)
    mg.set_blocks(1, B1)
    v1 = synth.gaussian_vectors(mg.volume[1], 16, 32, 210)
    mg.set_basis(1, v1)
    mg.block_orthonormalise(1)
    mg.build_coarse(2)
    assert mg.dims[2] == (3, 3, 3, 3)
    want = O.galerkin_coarse(B1, O.block_orthonormalise(v1, d1, (2, 2, 2, 2)), d1, (2, 2, 2, 2))
    assert rel(mg.get_blocks(2), want) < 1e-12


def test_galerkin_nonsquare_periodic(gpu_lib):
    dims = (4, 2, 6, 4)
    U = synth.gauge_haar(dims, 5)
    A = O.clover_packed(U, dims, CSW, KAPPA)
    ctx = gpu_lib.Context(dims, t_bc=+1)
    ctx.set_gauge(U)
    ctx.build_clover(CSW, KAPPA)
    mg = gpu_lib.Multigrid(ctx, [(2, 2, 3, 2)], [4])
    v0 = synth.gaussian_vectors(synth.volume(dims), 4, 12, 1)
    mg.set_basis(0, v0)
    mg.block_orthonormalise(0)
    mg.build_coarse(1)
    b0 = O.block_orthonormalise(v0, dims, (2, 2, 3, 2))
    want = O.galerkin_fine(U, A, KAPPA, b0, dims, (2, 2, 3, 2), t_bc=1.0)
    assert rel(mg.get_blocks(1), want) < 1e-12


def test_galerkin_full_size(gpu_lib):
    """Galerkin blocks at full size: 24^4 Haar links (csw 1, kappa 0.13), 16
    Gaussian vectors -> 6^4, then 16 more -> 3^4.  Checked by what holds at
    any size: D_c e = P^dag D P e for the GPU's own P and D (FP64), and the
    coarse gamma_5-hermiticity B_{-mu}(A + mu) = G5 B_{+mu}(A)^dag G5,
    B_self = G5 B_self^dag G5."""
    import torch

    dims = (24, 24, 24, 24)
    U = synth.gauge_haar(dims, 2024)
    ctx, mg = make_mg(gpu_lib, dims, [(4, 4, 4, 4), (2, 2, 2, 2)], [16, 16], U=U)
    V = synth.volume(dims)
    mg.set_basis(0, synth.gaussian_vectors(V, 16, 12, 300))
    mg.block_orthonormalise(0)
    mg.build_coarse(1)
    mg.set_basis(1, synth.gaussian_vectors(mg.volume[1], 16, 32, 400))
    mg.block_orthonormalise(1)
    mg.build_coarse(2)
    for lev in (1, 2):
        n = 3
        e = synth.coarse_source(mg.volume[lev], 32, n, 50 + lev, np.complex128)
        te = dev(e)
        # P^dag D P e on the GPU
        finer = torch.empty((mg.volume[lev - 1], mg.ncomp[lev - 1], n), dtype=torch.complex128, device="cuda")
        mg.prolong(lev - 1, finer, te)
        applied = torch.empty_like(finer)
        if lev == 1:
            ctx.dwc(applied, finer)
        else:
            mg.coarse_apply(1, applied, finer, "f64")
        want = torch.empty_like(te)
        mg.restrict(lev - 1, want, applied)
        got = torch.empty_like(te)
        mg.coarse_apply(lev, got, te, "f64")
        assert rel(host(got), host(want)) < 1e-12, lev
        B = mg.get_blocks(lev)
        g5 = np.diag(np.r_[np.ones(16), -np.ones(16)])
        cd = mg.dims[lev]
        Vc = mg.volume[lev]
        s = np.arange(Vc)
        coord = np.stack([s % cd[0], (s // cd[0]) % cd[1], (s // (cd[0] * cd[1])) % cd[2],
                          s // (cd[0] * cd[1] * cd[2])], axis=1)
        stride = np.array([1, cd[0], cd[0] * cd[1], cd[0] * cd[1] * cd[2]])
        herm = g5 @ np.conj(np.swapaxes(B[:, 0], -1, -2)) @ g5
        assert np.max(np.abs(herm - B[:, 0])) < 1e-12 * np.max(np.abs(B[:, 0]))
        for mu in range(4):
            nbr = ((coord + np.eye(4, dtype=int)[mu]) % np.array(cd)) @ stride
            lhs = B[nbr, 2 + 2 * mu]
            rhs = g5 @ np.conj(np.swapaxes(B[:, 1 + 2 * mu], -1, -2)) @ g5
            assert np.max(np.abs(lhs - rhs)) < 1e-12 * np.max(np.abs(B[:, 1 + 2 * mu])), (lev, mu)
