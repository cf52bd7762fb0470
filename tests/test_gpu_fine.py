"""GPU parity of the fine Wilson-clover operator against the FP64 oracle.

Tolerances: the FP64 path must agree to 1e-12 relative L2 (rounding order
only); the FP32 path to 1e-6 relative L2 (FP32 rounding of ~40 terms per
output is ~1e-7).  The FP32 kernel is also required to give bit-identical
results for a column whether it is applied alone or inside a batch.
"""

import os
import shutil

import numpy as np
import pytest

import oracle as O
import synth
from test_walk_shapes_host import F64_LDS, FINE_LDS, UNTUNED_FINE, fine_default

pytestmark = pytest.mark.gpu

KAPPA, CSW = 0.13, 1.0


def rel_l2(a, b):
    a = np.asarray(a, dtype=np.complex128)
    b = np.asarray(b, dtype=np.complex128)
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def _ctx(mrhs, dims, U, t_bc=-1):
    ctx = mrhs.Context(dims, t_bc=t_bc)
    ctx.set_gauge(U)
    ctx.build_clover(CSW, KAPPA)
    return ctx


def _dev(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.fixture(scope="module")
def small(gpu_lib):
    """8^4, Haar links, csw = 1, kappa = 0.13, antiperiodic t."""
    dims = (8, 8, 8, 8)
    U = synth.gauge_haar(dims, 1001)
    A = O.clover_packed(U, dims, CSW, KAPPA)
    return dims, U, A, _ctx(gpu_lib, dims, U)


def test_clover_build_matches_oracle(small):
    dims, U, A, ctx = small
    got = ctx.get_clover()
    assert np.max(np.abs(got - A)) < 1e-14
    # the FP32 copy is the rounded FP64 one
    got32 = ctx.get_clover(1)
    np.testing.assert_array_equal(got32, A.astype(np.float32))


def test_clover_build_nonsquare(gpu_lib):
    dims = (4, 6, 2, 10)
    U = synth.gauge_haar(dims, 7)
    ctx = _ctx(gpu_lib, dims, U)
    np.testing.assert_allclose(ctx.get_clover(), O.clover_packed(U, dims, CSW, KAPPA), atol=1e-14)


def test_dwc_fp64_8888(small):
    import torch

    dims, U, A, ctx = small
    psi = synth.spinor_source(dims, 1, 2001)
    want = O.dwc(U, A, KAPPA, psi, dims)
    x = _dev(torch, psi)
    y = torch.empty_like(x)
    ctx.dwc(y, x)
    torch.cuda.synchronize()
    assert rel_l2(y.cpu().numpy(), want) < 1e-12


@pytest.mark.parametrize("op", ["dwc", "hop", "clover"])
@pytest.mark.parametrize("nrhs", [1, 2, 3, 6, 12, 64])
def test_fp32_vs_oracle_8444(small, op, nrhs):
    import torch

    dims, U, A, ctx = small
    psi = synth.spinor_source(dims, nrhs, 3000, np.complex64)
    if op == "dwc":
        want = O.dwc(U, A, KAPPA, psi, dims)
    elif op == "hop":
        want = O.hop(U, psi, dims)
    else:
        want = O.clover_apply(A, psi)
    x = _dev(torch, psi)
    y = torch.empty_like(x)
    getattr(ctx, op)(y, x)
    torch.cuda.synchronize()
    assert rel_l2(y.cpu().numpy(), want) < 1e-6


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_fp_odd_lattice_periodic(gpu_lib, prec):
    """Non-cubic lattice with extent 2 (x+mu and x-mu coincide) and periodic t."""
    import torch

    dims = (2, 6, 4, 2)
    U = synth.gauge_haar(dims, 5)
    ctx = _ctx(gpu_lib, dims, U, t_bc=+1)
    A = O.clover_packed(U, dims, CSW, KAPPA)
    dt = np.complex64 if prec == "f32" else np.complex128
    psi = synth.spinor_source(dims, 4, 9, dt)
    x = _dev(torch, psi)
    y = torch.empty_like(x)
    ctx.dwc(y, x)
    torch.cuda.synchronize()
    err = rel_l2(y.cpu().numpy(), O.dwc(U, A, KAPPA, psi, dims, t_bc=+1.0))
    assert err < (1e-6 if prec == "f32" else 1e-12)


def test_mrhs_equals_srhs_bitwise(small):
    """Each column of a batched apply is bit-identical to applying it alone."""
    import torch

    dims, U, A, ctx = small
    for nrhs in (6, 12, 64):
        psi = synth.spinor_source(dims, nrhs, 4000, np.complex64)
        x = _dev(torch, psi)
        y = torch.empty_like(x)
        ctx.dwc(y, x)
        batch = y.cpu().numpy()
        for k in (0, nrhs // 2, nrhs - 1):
            xk = _dev(torch, psi[:, :, k:k + 1])
            yk = torch.empty_like(xk)
            ctx.dwc(yk, xk)
            np.testing.assert_array_equal(batch[:, :, k:k + 1], yk.cpu().numpy())


def test_deterministic_repeat(small):
    import torch

    dims, U, A, ctx = small
    x = _dev(torch, synth.spinor_source(dims, 24, 5000, np.complex64))
    y1, y2 = torch.empty_like(x), torch.empty_like(x)
    ctx.dwc(y1, x)
    ctx.dwc(y2, x)
    assert torch.equal(y1, y2)


# ---- the benchmark's 24^4 FP32 workload, Nrhs in {1, 6, 12, 24, 48, 64} ----------

NRHS_BIG = (1, 6, 12, 24, 48, 64)
TUNE_CACHE = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2211_13719_amd",
                          "tuning", "fine.txt")


def _hip_runtime_version():
    """hipRuntimeGetVersion of the HIP runtime this process has loaded (the
    one the library runs on, which keys the autotuner cache)."""
    import ctypes

    libs = sorted({l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l})
    v = ctypes.c_int()
    assert libs and ctypes.CDLL(libs[0]).hipRuntimeGetVersion(ctypes.byref(v)) == 0
    return v.value


def _cached_lines(path, arch, dims):
    """The autotuner cache's configuration per Nrhs for this lattice and HIP
    runtime (the last matching line wins, as in the library)."""
    out = {}
    hv = _hip_runtime_version()
    for line in open(path):
        f = line.split()
        if len(f) != 18 or f[0] != arch or int(f[1]) != hv or tuple(map(int, f[2:6])) != tuple(dims):
            continue
        f = f[:1] + f[2:]  # drop the runtime version: the fields below as before
        n, R = int(f[5]), int(f[6])
        tile = tuple(map(int, f[7:11]))
        curve, occ, nt, chunks, cap = map(int, f[11:16])
        walk = curve == 2  # the t-walk kernel
        variant = (0 if walk else curve) + 2 * (occ == 4) + 4 * nt + 8 * {1: 0, 2: 1, 4: 2}[chunks] + 32 * cap
        out[n] = (R, tile, variant + 128 * walk)
    return out


@pytest.fixture(scope="module")
def big(gpu_lib, tmp_path_factory):
    """The 24^4 workload the benchmark times, in the launch configurations
    it times: the fine kernel's tuned configuration per Nrhs comes from the
    committed autotuner cache (read from a copy, so that nothing is appended
    to the committed file), exactly as bench.py loads it."""
    import torch

    dims = (24, 24, 24, 24)
    U = synth.gauge_haar(dims, 2024)
    A = O.clover_packed_direct(U, dims, CSW, KAPPA)
    ctx = _ctx(gpu_lib, dims, U)
    arch = torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]
    want = _cached_lines(TUNE_CACHE, arch, dims)
    assert set(NRHS_BIG) <= set(want), "the committed tuning cache lacks a 24^4 Nrhs"
    cache = tmp_path_factory.mktemp("tune") / "fine.txt"
    shutil.copyfile(TUNE_CACHE, cache)
    before = cache.read_text()
    ctx.tune(list(NRHS_BIG), str(cache))
    assert cache.read_text() == before, "a 24^4 configuration was tuned afresh instead of read from the cache"
    return dims, U, A, ctx, want


def test_clover_build_24(big):
    dims, U, A, ctx, _ = big
    assert np.max(np.abs(ctx.get_clover() - A)) < 1e-14


@pytest.mark.parametrize("nrhs", NRHS_BIG)
def test_fp32_24444_sampled(big, nrhs):
    """Full-size apply in the launch configuration the benchmark times (the
    cached tuned configuration of this Nrhs, asserted first), checked on a
    sample of sites (all boundary-wrapping directions included) against the
    per-site oracle; N = 1 is also checked on every site."""
    import torch

    dims, U, A, ctx, want = big
    R, tile, variant, _ = ctx.get_tuning(nrhs)
    assert (R, tuple(tile), variant) == want[nrhs]
    psi = synth.spinor_source(dims, nrhs, 100, np.complex64)
    x = _dev(torch, psi)
    y = torch.empty_like(x)
    ctx.dwc(y, x)
    torch.cuda.synchronize()
    got = y.cpu().numpy()
    V = synth.volume(dims)
    g = synth.rng(77 + nrhs)
    corners = np.array([0, 23, 24 * 23, 24**3 * 23, V - 1, V - 24, V // 2])
    sites = np.unique(np.concatenate([corners, g.integers(0, V, 1500)]))
    want = O.dwc_sites(U, A, KAPPA, psi, dims, sites)
    assert rel_l2(got[sites], want) < 1e-6
    if nrhs == 1:
        assert rel_l2(got, O.dwc(U, A, KAPPA, psi, dims)) < 1e-6


def test_autotune_bitwise_and_cache(small, tmp_path):
    """Tuned launch configurations give bit-identical results; the cache file
    is written and read back."""
    import torch

    dims, U, A, ctx = small
    outs = {}
    for n in (1, 6, 12):
        x = _dev(torch, synth.spinor_source(dims, n, 6000 + n, np.complex64))
        y = torch.empty_like(x)
        ctx.dwc(y, x)
        outs[n] = (x, y.clone())
    cache = str(tmp_path / "tune.txt")
    ctx.tune([1, 6, 12], cache)
    for n, (x, y0) in outs.items():
        R, tile, curve, us = ctx.get_tuning(n)
        assert R in (1, 2, 4) and n % R == 0 and us > 0 and 0 <= curve < 256
        assert all(t >= 1 and L % t == 0 for t, L in zip(tile, dims))
        y = torch.empty_like(x)
        ctx.dwc(y, x)
        assert torch.equal(y, y0)
    lines = open(cache).read().split("\n")
    assert sum(1 for l in lines if l.strip()) == 3
    ctx.tune([12], cache)  # served from the cache, no new line
    assert sum(1 for l in open(cache).read().split("\n") if l.strip()) == 3


@pytest.mark.parametrize(
    "R,tile,curve,occ,nt,chunks,cap",
    [
        (2, (2, 2, 2, 2), 0, 0, 0, 2, 0),
        (1, (4, 4, 4, 8), 1, 4, 1, 4, 0),
        (4, (8, 4, 4, 1), 0, 0, 0, 2, 2),
        (2, (2, 2, 2, 8), 1, 0, 1, 1, 1),
        (4, (1, 1, 1, 1), 0, 4, 0, 1, 2),
        # t-walk kernel (curve 2): spatial block, time slices per thread
        (1, (4, 4, 4, 8), 2, 0, 0, 1, 0),
        (2, (8, 8, 8, 2), 2, 4, 1, 2, 0),
        (1, (2, 4, 8, 1), 2, 0, 1, 4, 1),
        (2, (8, 2, 4, 4), 2, 4, 0, 1, 2),
    ],
)
def test_launch_configurations_bitwise(small, tmp_path, R, tile, curve, occ, nt, chunks, cap):
    """Every launch configuration the tuner can pick -- RHS per thread, tile and
    order, register budget, store kind, RHS chunks swept in turn, workgroups
    per CU -- gives the default launch's result bit for bit (set through a
    cache file, which the tuner reads without timing)."""
    import torch

    dims, U, A, ctx = small
    n = 24
    x = _dev(torch, synth.spinor_source(dims, n, 6100, np.complex64))
    y0 = torch.empty_like(x)
    ctx.dwc(y0, x)  # untuned default (or whatever an earlier test left): compare with FP32 oracle below
    arch = torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]
    cache = tmp_path / "cfg.txt"
    cache.write_text(f"{arch} {_hip_runtime_version()} {' '.join(map(str, dims))} {n} {R} {' '.join(map(str, tile))} "
                     f"{curve} {occ} {nt} {chunks} {cap} 1.0\n")
    ctx.tune([n], str(cache))
    got = ctx.get_tuning(n)
    assert got[0] == R and tuple(got[1]) == tile
    assert bool(got[2] & 128) == (curve == 2) and got[2] & 1 == curve % 2
    assert bool(got[2] & 2) == (occ == 4) and bool(got[2] & 4) == bool(nt)
    assert 1 << ((got[2] >> 3) & 3) == chunks
    y = torch.empty_like(x)
    ctx.dwc(y, x)
    assert torch.equal(y, y0)


@pytest.mark.parametrize("tile,R,chunks", [((2, 4, 2, 3), 1, 1), ((3, 2, 4, 2), 2, 2), ((6, 4, 8, 6), 1, 4)])
def test_walk_kernel_on_an_anisotropic_lattice(gpu_lib, tmp_path, tile, R, chunks):
    """The t-walk kernel on a lattice with four different extents (a mixed-up
    coordinate or stride shows), against the oracle and bit for bit against
    the tiled kernel; the runs of Ts slices wrap through the antiperiodic t
    boundary, and the last tile is one run over the whole t extent."""
    import torch

    dims = (6, 4, 8, 6)
    U = synth.gauge_haar(dims, 1301)
    A = O.clover_packed(U, dims, CSW, KAPPA)
    ctx = _ctx(gpu_lib, dims, U)
    n = 12
    psi = synth.spinor_source(dims, n, 1302, np.complex64)
    x = _dev(torch, psi)
    y0 = torch.empty_like(x)
    ctx.dwc(y0, x)
    arch = torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]
    cache = tmp_path / "walk.txt"
    cache.write_text(f"{arch} {_hip_runtime_version()} {' '.join(map(str, dims))} {n} {R} {' '.join(map(str, tile))} "
                     f"2 0 0 {chunks} 0 1.0\n")
    ctx.tune([n], str(cache))
    got = ctx.get_tuning(n)
    assert got[0] == R and tuple(got[1]) == tile and got[2] & 128
    y = torch.empty_like(x)
    ctx.dwc(y, x)
    torch.cuda.synchronize()
    assert torch.equal(y, y0)
    assert rel_l2(y.cpu().numpy(), O.dwc(U, A, KAPPA, psi, dims)) < 1e-6


@pytest.mark.parametrize("tile,variant", [((2, 4, 2, 3), 0), ((3, 2, 4, 2), 1), ((6, 4, 8, 6), 2), ((3, 4, 2, 1), 3)])
def test_f64_walk_kernel(gpu_lib, tile, variant):
    """The FP64 operator as a t-walk (one RHS per thread; non-temporal stores
    and the two-workgroup register budget by variant) on a lattice with four
    different extents: bit for bit the tiled FP64 kernel and within rounding
    of the FP64 oracle, for 1, 3 and 12 RHS; runs of Ts slices wrap through
    the antiperiodic t boundary (Ts = 1 to a whole t extent)."""
    import torch

    dims = (6, 4, 8, 6)
    U = synth.gauge_haar(dims, 1401)
    A = O.clover_packed(U, dims, CSW, KAPPA)
    ctx = _ctx(gpu_lib, dims, U)
    for n in (1, 3, 12):
        psi = synth.spinor_source(dims, n, 1402 + n)
        x = _dev(torch, psi)
        ctx.set_f64_walk(n, None)
        y0 = torch.empty_like(x)
        ctx.dwc(y0, x)
        ctx.set_f64_walk(n, tile, variant)
        on, t, v, _, _ = ctx.get_f64_walk(n)
        assert on and t == tile and v == variant
        y = torch.empty_like(x)
        ctx.dwc(y, x)
        torch.cuda.synchronize()
        assert torch.equal(y, y0), n
        assert rel_l2(y.cpu().numpy(), O.dwc(U, A, KAPPA, psi, dims)) < 1e-12


def test_f64_walk_rejects_and_tunes(gpu_lib):
    """A tile that does not divide the lattice is refused; mrhs_tune times the
    FP64 kernels and whichever it keeps gives the tiled kernel's bits."""
    import torch

    dims = (8, 8, 8, 8)
    U = synth.gauge_haar(dims, 1501)
    ctx = _ctx(gpu_lib, dims, U)
    with pytest.raises(Exception):
        ctx.set_f64_walk(4, (3, 8, 8, 8))
    psi = synth.spinor_source(dims, 4, 1502)
    x = _dev(torch, psi)
    y0 = torch.empty_like(x)
    ctx.dwc(y0, x)
    ctx.tune([4])
    on, tile, variant, us, us_tiled = ctx.get_f64_walk(4)
    assert us_tiled > 0 and us > 0 and us <= us_tiled
    y = torch.empty_like(x)
    ctx.dwc(y, x)
    torch.cuda.synchronize()
    assert torch.equal(y, y0)


def _set_walk(torch, ctx, dims, path, n, R, tile, curve, nt, chunks):
    arch = torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]
    path.write_text(f"{arch} {_hip_runtime_version()} {' '.join(map(str, dims))} {n} {R} {' '.join(map(str, tile))} "
                    f"{curve} 0 {nt} {chunks} 0 1.0\n")
    ctx.tune([n], str(path))


@pytest.mark.parametrize(
    "dims,n,R,tile,nt,chunks",
    [
        ((6, 10, 4, 6), 12, 2, (3, 5, 4, 3), 0, 1),  # a block that spans z; 360 of 384 threads
        ((6, 10, 4, 6), 24, 2, (2, 2, 2, 6), 1, 2),  # two chunks, one run over the whole t extent
        ((6, 10, 4, 6), 64, 2, (2, 2, 4, 1), 1, 1),  # 512 threads, runs of one slice
        ((6, 10, 4, 6), 7, 1, (6, 10, 1, 2), 0, 1),  # one site wide where the lattice is not: not kept in LDS
        ((6, 10, 4, 6), 7, 1, (3, 5, 4, 2), 1, 1),
        ((5, 3, 9, 4), 3, 1, (5, 3, 3, 2), 0, 1),  # odd extents, three threads per site: up to six link words each
        ((5, 3, 9, 4), 2, 1, (5, 3, 9, 4), 0, 1),  # the whole lattice in one block, up to nine
        ((4, 2, 2, 2), 1, 1, (2, 2, 2, 1), 0, 1),  # eight sites, one wavefront
        ((3, 3, 3, 5), 5, 1, (3, 3, 3, 5), 1, 1),
    ],
)
def test_walk_with_its_block_in_lds(gpu_lib, tmp_path, dims, n, R, tile, nt, chunks):
    """The t-walk whose workgroup keeps its block in LDS, over the edges of its
    shapes: blocks that span the lattice or meet it at a face, odd extents,
    partly filled workgroups, every count of staged links, chunks, short and
    full runs; bit for bit the tiled kernel, in FP32 and FP64."""
    import torch

    U = synth.gauge_haar(dims, 1601)
    A = O.clover_packed(U, dims, CSW, KAPPA)
    ctx = _ctx(gpu_lib, dims, U)
    psi = synth.spinor_source(dims, n, 1602, np.complex64)
    x = _dev(torch, psi)
    y0, y = torch.empty_like(x), torch.empty_like(x)
    _set_walk(torch, ctx, dims, tmp_path / "tiled.txt", n, 1, (1, 1, 1, 1), 0, 0, 1)
    ctx.dwc(y0, x)
    _set_walk(torch, ctx, dims, tmp_path / "walk.txt", n, R, tile, 2, nt, chunks)
    assert ctx.get_tuning(n)[0] == R and ctx.get_tuning(n)[1] == tile
    ctx.dwc(y, x)
    torch.cuda.synchronize()
    assert torch.equal(y, y0)
    assert rel_l2(y.cpu().numpy(), O.dwc(U, A, KAPPA, psi, dims)) < 1e-6
    x64 = x.to(torch.complex128)
    z0, z = torch.empty_like(x64), torch.empty_like(x64)
    ctx.set_f64_walk(n, None)
    ctx.dwc(z0, x64)
    ctx.set_f64_walk(n, tile, nt)
    ctx.dwc(z, x64)
    torch.cuda.synchronize()
    assert torch.equal(z, z0)
    assert rel_l2(z.cpu().numpy(), O.dwc(U, A, KAPPA, psi.astype(np.complex128), dims)) < 1e-12


@pytest.mark.parametrize("dims,n,R,tile,nt,chunks", FINE_LDS + F64_LDS)
def test_shapes_kept_in_lds(gpu_lib, tmp_path, dims, n, R, tile, nt, chunks):
    """Shapes that the rule keeps in LDS, at the edges of what it takes: bit for
    bit the tiled kernel, in FP32 and FP64."""
    import torch

    ctx = _ctx(gpu_lib, dims, synth.gauge_haar(dims, 1801))
    x = _dev(torch, synth.spinor_source(dims, n, 1802, np.complex64))
    out = []
    for i, (r, t, curve, c) in enumerate(((1, (1, 1, 1, 1), 0, 1), (R, tile, 2, chunks))):
        _set_walk(torch, ctx, dims, tmp_path / f"w{i}.txt", n, r, t, curve, nt, c)
        ctx.set_f64_walk(n, tile if curve == 2 else None, nt)
        out.append([torch.empty_like(x), torch.empty_like(x, dtype=torch.complex128)])
        ctx.dwc(out[i][0], x)
        ctx.dwc(out[i][1], x.to(torch.complex128))
    torch.cuda.synchronize()
    for a, b in zip(*out):
        assert torch.equal(a, b)


@pytest.mark.parametrize("dims", [(8, 8, 8, 8), (5, 3, 9, 4), (6, 10, 4, 6), (2, 2, 2, 2), (7, 7, 7, 11), (16, 2, 4, 6)])
def test_untuned_launch_is_the_tiled_result(gpu_lib, tmp_path, dims):
    """Without tuning the shape comes from an estimate: whatever it picks gives
    the tiled kernel's bits."""
    import torch

    U = synth.gauge_haar(dims, 1701)
    ctx = _ctx(gpu_lib, dims, U)
    for n in (1, 2, 3, 4, 5, 8, 12, 17, 30, 64):
        x = _dev(torch, synth.spinor_source(dims, n, 1702 + n, np.complex64))
        y0, y = torch.empty_like(x), torch.empty_like(x)
        assert ctx.get_tuning(n)[0] == 0
        ctx.dwc(y, x)
        _set_walk(torch, ctx, dims, tmp_path / f"tiled{n}.txt", n, 1, (1, 1, 1, 1), 0, 0, 1)
        ctx.dwc(y0, x)
        torch.cuda.synchronize()
        assert torch.equal(y, y0), n


def _random_gauge(torch, V, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.view_as_complex(0.4 * torch.randn(V, 4, 3, 3, 2, generator=g, device="cuda", dtype=torch.float64))


@pytest.mark.parametrize("dims,n,choice", UNTUNED_FINE)
def test_untuned_choice_is_the_tiled_result(gpu_lib, tmp_path, dims, n, choice):
    """Each kind of untuned launch -- the host tests say which one it is -- gives
    the tiled kernel's bits."""
    import torch

    assert fine_default(dims, n) == choice
    V = int(np.prod(dims))
    ctx = _ctx(gpu_lib, dims, _random_gauge(torch, V, 1901))
    g = torch.Generator(device="cuda").manual_seed(1902)
    x = torch.view_as_complex(torch.randn(V, 12, n, 2, generator=g, device="cuda"))
    y0, y = torch.empty_like(x), torch.empty_like(x)
    ctx.dwc(y, x)
    _set_walk(torch, ctx, dims, tmp_path / "tiled.txt", n, 1, (1, 1, 1, 1), 0, 0, 1)
    ctx.dwc(y0, x)
    torch.cuda.synchronize()
    assert torch.equal(y, y0)
    ctx.close()


def test_tuner_tries_one_rhs_per_thread_beside_a_walk(gpu_lib, tmp_path):
    """11x7x9x18 at two right-hand sides: a walk leads the tiled kernel with two
    per thread (17 against 18 us), and the tiled kernel with one (11 us among
    others) leads both; the tuned operator is within 1.2 of it."""
    import torch

    dims, n = (11, 7, 9, 18), 2
    V = int(np.prod(dims))
    ctx = _ctx(gpu_lib, dims, _random_gauge(torch, V, 2001))
    g = torch.Generator(device="cuda").manual_seed(2002)
    x = torch.view_as_complex(torch.randn(V, 12, n, 2, generator=g, device="cuda"))
    y = torch.empty_like(x)

    def us():
        start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        best = 1e9
        for _ in range(8):
            start.record()
            for _ in range(50):
                ctx.dwc(y, x)
            end.record()
            end.synchronize()
            best = min(best, start.elapsed_time(end) * 20)
        return best

    ctx.tune([n])
    tuned = us()
    _set_walk(torch, ctx, dims, tmp_path / "tiled.txt", n, 1, (1, 1, 1, 1), 0, 0, 1)
    assert tuned < 1.2 * us()
    ctx.close()
