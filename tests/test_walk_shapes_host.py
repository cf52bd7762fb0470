"""Which walk a launch shape runs: the rules of csrc/fine.hip, called in the
built library (host code only).  A shape whose block fits a workgroup keeps it
in LDS unless the walk without is expected to be faster."""

import ctypes as C

import pytest

from paper_2211_13719_amd._lib import lib


class Geom(C.Structure):
    _fields_ = [("L", C.c_int * 4), ("V", C.c_int), ("stride", C.c_int * 4), ("T", C.c_int * 4),
                ("order", C.c_void_p), ("nbr", C.c_void_p)]


def geom(dims):
    g = Geom()
    step = 1
    for m in range(4):
        g.L[m], g.stride[m] = dims[m], step
        step *= dims[m]
    g.V = step
    return g


def _fn(name, res, *args):
    f = lib[name]
    f.restype, f.argtypes = res, args
    return f


_walk_cost = _fn("_ZN4mrhs16staged_walk_costERKNS_4GeomEPKiiiib", C.c_double, C.POINTER(Geom), C.POINTER(C.c_int),
                 C.c_int, C.c_int, C.c_int, C.c_bool)
_eo_cost = _fn("_ZN4mrhs14staged_eo_costERKNS_4GeomEPKiii", C.c_double, C.POINTER(Geom), C.POINTER(C.c_int), C.c_int,
               C.c_int)
_walk_in_lds = _fn("_ZN4mrhs11walk_in_ldsERKNS_4GeomEPKiiiib", C.c_bool, C.POINTER(Geom), C.POINTER(C.c_int), C.c_int,
                   C.c_int, C.c_int, C.c_bool)
_eo_in_lds = _fn("_ZN4mrhs14eo_walk_in_ldsERKNS_4GeomEPKiii", C.c_bool, C.POINTER(Geom), C.POINTER(C.c_int), C.c_int,
                 C.c_int)


def fine_in_lds(dims, n, R, tile, chunks=1):
    return _walk_in_lds(C.byref(geom(dims)), (C.c_int * 4)(*tile), n, R, chunks, False)


def f64_in_lds(dims, n, tile):
    return _walk_in_lds(C.byref(geom(dims)), (C.c_int * 4)(*tile), n, 1, 1, True)


def eo_in_lds(dims, n, R, tile):
    return _eo_in_lds(C.byref(geom(dims)), (C.c_int * 4)(*tile), n, R)


# Shapes that keep their block in LDS, at the edges of what it takes; the GPU
# tests run them: (lattice, Nrhs, right-hand sides per thread, tile, ...)
FINE_LDS = [  # ..., non-temporal stores, chunks
    ((6, 10, 4, 40), 12, 2, (3, 5, 4, 1), 0, 1),  # a block that spans z; 360 of 384 threads
    ((6, 10, 4, 12), 24, 2, (2, 2, 2, 4), 1, 2),  # two chunks, runs of four slices
    ((8, 12, 8, 6), 24, 2, (2, 2, 2, 6), 0, 2),   # one run over the whole t extent
    ((6, 10, 4, 12), 64, 2, (2, 2, 4, 1), 1, 1),  # 512 threads, runs of one slice
]
F64_LDS = [
    ((6, 10, 4, 12), 12, 1, (3, 5, 4, 3), 0, 1),  # three chunks, 240 of 256 threads
    ((6, 10, 4, 12), 64, 1, (2, 2, 2, 12), 1, 1),  # two chunks, the whole t extent
]
FINE_LDS_RESIDUAL = [(12, 2, (2, 2, 2, 2), 0), (16, 2, (2, 4, 2, 1), 1)]  # on 8^4
EO_LDS = [
    ((8, 12, 8, 8), 48, 2, (2, 3, 4, 1)),   # two chunks, 288 of 320 threads, runs of one output site
    ((8, 12, 8, 8), 24, 2, (2, 4, 2, 4)),   # one run over the whole t extent
    ((8, 12, 8, 8), 6, 1, (2, 3, 4, 4)),    # more than three link words per thread, 144 of 192 threads
    ((8, 12, 8, 8), 13, 1, (4, 3, 2, 4)),
    ((8, 12, 8, 8), 24, 1, (2, 2, 8, 1)),   # a block that spans z, two chunks
    ((6, 12, 10, 16), 48, 1, (2, 4, 5, 4)),  # four chunks
    ((6, 12, 10, 16), 32, 2, (2, 2, 5, 2)),
]
EO_LDS_SMOOTHER = [((8, 8, 8, 8), 24, 2, (2, 4, 2, 4)), ((8, 12, 8, 8), 48, 2, (2, 3, 4, 1)),
                   ((8, 8, 8, 8), 6, 1, (4, 2, 2, 2)), ((8, 8, 8, 8), 48, 1, (2, 8, 2, 1))]


def test_shapes_of_the_lds_tests_run_there():
    for dims, n, R, tile, _, chunks in FINE_LDS:
        assert fine_in_lds(dims, n, R, tile, chunks), (dims, n)
    for dims, n, _, tile, _, _ in F64_LDS:
        assert f64_in_lds(dims, n, tile), (dims, n)
    for n, R, tile, _ in FINE_LDS_RESIDUAL:
        assert fine_in_lds((8, 8, 8, 8), n, R, tile), n
    for dims, n, R, tile in EO_LDS + EO_LDS_SMOOTHER:
        assert eo_in_lds(dims, n, R, tile), (dims, n)


@pytest.mark.parametrize("kind,dims,n,R,tile", [
    # (open, LDS) in us
    ("f32", (8, 8, 8, 8), 12, 2, (4, 4, 4, 1)),         # 13.3, 17.3
    ("f32", (16, 8, 8, 16), 12, 2, (4, 4, 4, 2)),       # 26.9, 30.9
    ("eo", (8, 8, 8, 8), 16, 1, (4, 4, 4, 1)),          # 25.0, 38.9
    ("eo", (16, 16, 16, 16), 24, 1, (4, 4, 4, 1)),      # 174, 293
    ("eo", (24, 24, 24, 24), 24, 1, (4, 4, 4, 3)),      # 1031, 1263
    ("f64", (8, 8, 8, 8), 12, 1, (4, 4, 4, 1)),         # 17.2, 19.8
    ("f64", (18, 4, 16, 8), 24, 1, (6, 4, 2, 4)),       # 47.6, 78.1
])
def test_shapes_faster_without_lds_stay_out(kind, dims, n, R, tile):
    """A stored or hand-set shape whose block fits LDS but was measured slower
    there runs the walk it was chosen for."""
    got = {"f32": lambda: fine_in_lds(dims, n, R, tile), "f64": lambda: f64_in_lds(dims, n, tile),
           "eo": lambda: eo_in_lds(dims, n, R, tile)}[kind]()
    assert not got


@pytest.mark.parametrize("kind,dims,n,R,tile", [
    ("f32", (24, 24, 24, 24), 12, 2, (3, 3, 8, 6)),     # 427, 320
    ("f32", (16, 16, 16, 32), 6, 1, (4, 4, 4, 4)),      # 129, 78
    ("eo", (24, 24, 24, 24), 6, 1, (4, 4, 4, 12)),      # 435, 287
    ("eo", (24, 24, 24, 24), 64, 2, (2, 3, 4, 6)),      # 1932, 1770
    ("f64", (16, 16, 16, 32), 4, 1, (4, 4, 4, 32)),     # 467, 313
])
def test_shapes_faster_in_lds_run_there(kind, dims, n, R, tile):
    got = {"f32": lambda: fine_in_lds(dims, n, R, tile), "f64": lambda: f64_in_lds(dims, n, tile),
           "eo": lambda: eo_in_lds(dims, n, R, tile)}[kind]()
    assert got


class FineCfg(C.Structure):
    _fields_ = [("R", C.c_int), ("T", C.c_int * 4), ("curve", C.c_int), ("walk", C.c_int), ("occ", C.c_int),
                ("nt", C.c_int), ("chunks", C.c_int), ("cap", C.c_int), ("lds", C.c_uint), ("order", C.c_void_p),
                ("us", C.c_float)]


class EoWalk(C.Structure):
    _fields_ = [("on", C.c_int), ("R", C.c_int), ("B", C.c_int * 3), ("Ts", C.c_int), ("us", C.c_float),
                ("us_tiled", C.c_float)]


_fine_default = _fn("_ZN4mrhs12fine_defaultERKNS_4GeomEi", FineCfg, C.POINTER(Geom), C.c_int)
_eo_default = _fn("_ZN4mrhs10eo_defaultERKNS_4GeomEi", EoWalk, C.POINTER(Geom), C.c_int)


def fine_default(dims, n):
    """(R, tile, chunks) of the untuned operator, None for the tiled kernel."""
    c = _fine_default(C.byref(geom(dims)), n)
    return (c.R, tuple(c.T), c.chunks) if c.R else None


def eo_default(dims, n):
    """(R, tile) of the untuned checkerboard hop, None for the tiled kernel."""
    c = _eo_default(C.byref(geom(dims)), n)
    return (c.R, (*c.B, c.Ts)) if c.on else None


def _divisors(n):
    return [d for d in range(1, n + 1) if n % d == 0]


def _tiles(dims, lt, smax):
    return [(x, y, z, t) for x in _divisors(dims[0]) for y in _divisors(dims[1]) for z in _divisors(dims[2])
            if x * y * z <= smax for t in _divisors(lt)]


@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (5, 3, 9, 4), (12, 10, 6, 14), (16, 16, 16, 32), (7, 7, 7, 11),
                                  (24, 24, 24, 24)])
def test_untuned_choice_is_that_of_the_full_search(dims):
    """The pruned search of the first apply finds what costing every shape does."""
    g = geom(dims)
    V = g.V
    for n in (1, 2, 3, 6, 7, 12, 24, 64):
        rows = V * n
        best, cost = None, 1e30
        for R in (1, 2):
            for chunks in (1, 2, 4):
                if n % chunks or (n // chunks) % R:
                    continue
                for T in _tiles(dims, dims[3], 512 * R * chunks // n):
                    c = _walk_cost(C.byref(g), (C.c_int * 4)(*T), n, R, chunks, False)
                    if 0 <= c < cost and fine_in_lds(dims, n, R, T, chunks):
                        best, cost = (R, T, chunks), c
        us, large = 3.8 * cost - 0.5, 2.5 * cost + 1.6 + 32e-6 * rows
        tiled = 1.9 + 90e-6 * rows + 359e-6 * V
        if best and best[2] > 1 and n // best[2] % 16:  # chunks that end within 128-byte lines
            tiled *= 0.75 if rows > 2.5e6 else 0.9
        if ((n == 1 and V < 1 << 17) or (n > 1 and n % 2 and us >= 0.9 * (6.6 + 96.4e-6 * rows + 159e-6 * V))
                or (n % 2 == 0 and n >= 8 and rows < 3e5 and us >= 0.75 * (9.0 + 62.7e-6 * rows + 358e-6 * V))
                or (n % 2 == 0 and n >= 8 and rows >= 3e5 and large >= tiled)):
            best = None
        assert fine_default(dims, n) == best, n
        best, cost = None, 1.55e-5 * rows
        if all(L % 2 == 0 for L in dims) and rows >= 1 << 20:
            for R in (1, 2):
                for T in _tiles(dims, dims[3] // 2, 2048 * R // n) if n % R == 0 else []:
                    c = _eo_cost(C.byref(g), (C.c_int * 4)(*T), n, R)
                    if 0 <= c < cost and eo_in_lds(dims, n, R, T):
                        best, cost = (R, T), c
        assert eo_default(dims, n) == best, n


def test_untuned_choice_costs_less_than_a_tenth_of_a_launch():
    """The first apply of a batch size makes the choice on the host: on
    24^3 x 128 at 12 right-hand sides in less than a tenth of the launch's
    1530 us (operator) and 1000 us (hop)."""
    import time

    g = geom((24, 24, 24, 128))
    for f, us in ((_fine_default, 153), (_eo_default, 100)):
        best = 1e9
        for _ in range(20):
            t = time.perf_counter()
            f(C.byref(g), 12)
            best = min(best, time.perf_counter() - t)
        assert best * 1e6 < us


# (lattice, Nrhs, the untuned choice), a case for each branch of the rules: the
# operator with one and two right-hand sides per thread, one and two chunks
# (16 right-hand sides and more a chunk store non-temporally), the odd and the
# small batches, one right-hand side; the hop with one and two per thread
UNTUNED_FINE = [
    ((8, 8, 8, 8), 1, None), ((16, 16, 16, 32), 1, (1, (2, 2, 4, 4), 1)),
    ((16, 16, 16, 16), 2, (1, (4, 4, 8, 2), 1)), ((16, 24, 20, 4), 6, (1, (4, 4, 4, 2), 1)),
    ((12, 10, 6, 14), 5, None), ((12, 12, 12, 24), 7, (1, (3, 3, 6, 3), 1)),
    ((12, 10, 6, 14), 12, None), ((8, 8, 8, 8), 12, (1, (2, 2, 4, 1), 1)),
    ((16, 16, 16, 16), 12, (2, (4, 4, 4, 4), 1)), ((14, 15, 12, 20), 16, (2, (2, 5, 4, 5), 1)),
    ((12, 10, 6, 14), 64, (1, (2, 2, 3, 7), 2)), ((12, 12, 12, 24), 64, (2, (3, 3, 3, 12), 2)),
]
UNTUNED_EO = [
    ((12, 4, 8, 16), 64, None), ((16, 16, 16, 16), 16, (1, (2, 4, 4, 4))), ((16, 16, 16, 16), 24, (2, (2, 4, 4, 4))),
    ((16, 16, 16, 32), 13, (1, (2, 4, 4, 8))), ((12, 12, 12, 24), 64, (1, (3, 3, 3, 12))),
]


def test_untuned_choices():
    for dims, n, want in UNTUNED_FINE:
        assert fine_default(dims, n) == want, (dims, n)
    for dims, n, want in UNTUNED_EO:
        assert eo_default(dims, n) == want, (dims, n)


class _Vector(C.Structure):  # std::vector of a trivially copyable type, never freed here
    _fields_ = [("begin", C.c_void_p), ("end", C.c_void_p), ("cap", C.c_void_p)]

    def of(self, cls):
        n = ((self.end or 0) - (self.begin or 0)) // C.sizeof(cls)
        return list((cls * n).from_address(self.begin)) if n else []


_staged_walks = _fn("_ZN4mrhs12staged_walksERKNS_4GeomEibm", _Vector, C.POINTER(Geom), C.c_int, C.c_bool, C.c_size_t)
_staged_eo_walks = _fn("_ZN4mrhs15staged_eo_walksERKNS_4GeomEim", _Vector, C.POINTER(Geom), C.c_int, C.c_size_t)


@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (8, 8, 8, 8), (12, 10, 6, 14), (5, 7, 9, 11), (16, 16, 16, 32)])
def test_tuner_times_only_shapes_near_the_best_estimate(dims):
    """The walks that fit LDS which the tuner times: in order of their estimate, at most
    as many as asked for, and none more than 1.25 times the first."""
    g = geom(dims)
    for n in (1, 6, 7, 12, 24, 64):
        for f64 in (False, True):
            costs = [_walk_cost(C.byref(g), w.T, n, w.R, w.chunks, f64)
                     for w in _staged_walks(C.byref(g), n, f64, 16).of(FineCfg)]
            assert len(costs) <= 16 and costs == sorted(costs)
            assert not costs or (0 <= costs[0] and costs[-1] <= 1.25 * costs[0])
        costs = [_eo_cost(C.byref(g), (C.c_int * 4)(*w.B, w.Ts), n, w.R)
                 for w in _staged_eo_walks(C.byref(g), n, 16).of(EoWalk)]
        assert len(costs) <= 16 and costs == sorted(costs)
        assert not costs or (0 <= costs[0] and costs[-1] <= 1.25 * costs[0])


@pytest.mark.parametrize("dims,n", [
    # us of the tiled kernel and of the walk of the least estimated time
    ((13, 10, 9, 13), 20),   # 33, 61
    ((8, 9, 17, 13), 20),    # 36, 55
    ((9, 19, 24, 11), 12),   # 72, 107
    ((24, 19, 20, 22), 48),  # 887, 1171
])
def test_large_fields_that_are_cut_badly_run_the_tiled_kernel(dims, n):
    assert fine_default(dims, n) is None
