// Restriction and prolongation on the matrix cores (paper Sec. 5, with
// n_v = 16 basis vectors per chirality): with Nrhs right-hand sides both are,
// per (aggregate A, chirality chi), complex GEMMs
//
//   restrict:  Y = W^dag F     (16 x R) = (16 x R_A)^dag (R_A x Nrhs)
//   prolong:   F = W Y         (R_A x Nrhs) = (R_A x 16) (16 x Nrhs)
//
// where R_A = (sites of A) x (h components of chi) and W holds the 16 basis
// vectors restricted to (A, chi).  They run as v_mfma_f32_32x32x16_bf16 with
// FP32 accumulation on the real form of the complex product:
//
//   restrict: rows 0..15 of the 32 x 32 output are Re y_i, rows 16..31 Im y_i,
//             A'[i][(r, re)] = Re w_ri, A'[i][(r, im)] = Im w_ri,
//             A'[16 + i][(r, re)] = -Im w_ri, A'[16 + i][(r, im)] = Re w_ri,
//             B'[(r, re|im)][k] = Re|Im f_rk;
//   prolong:  rows 0..15 are Re f_r, rows 16..31 Im f_r of 16 consecutive r,
//             A'[r][(i, re)] = Re w_ri, A'[r][(i, im)] = -Im w_ri,
//             A'[16 + r][(i, re)] = Im w_ri, A'[16 + r][(i, im)] = Re w_ri,
//             B'[(i, re|im)][k] = Re|Im y_ik.
//
// With the MFMA layouts A[l % 32][8 (l / 32) + q], B[8 (l / 32) + q][l % 32]
// and D[8 (p / 4) + 4 (l / 32) + p % 4][l % 32] (accumulator p), the real and
// imaginary part of one output sit in accumulators p and p + 8 of the same
// lane, so every store is one complex value and 32 lanes write 256
// contiguous bytes.  Rows r of (A, chi) are ordered component-major,
// r = c * (sites of A) + l, so a lane's consecutive rows are consecutive
// sites of one component.
//
// The basis is a BF16 copy of the FP32 basis (round to nearest even, one
// 32-bit word per complex value, re in the low half); the fine and coarse
// fields stay FP32 in memory and are rounded to BF16 on the fly by the
// hardware conversion (round to nearest even).  Products of BF16 values are
// exact in FP32, so the only other rounding is the FP32 accumulation.
//
// The FP32 variants use v_mfma_f32_32x32x2_f32 on the FP32 basis with the
// same real form: one contraction step is one row r (restrict) or one basis
// index i (prolong) with its real and imaginary part as the two k values,
// A[l % 32][k = l / 32], B[k = l / 32][l % 32].
#include <algorithm>

#include "agg.h"
#include "internal.h"
#include "rounding.h"

namespace mrhs {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(unsigned)))) unsigned u32x4;

constexpr int kNV = 16;

// The fine sites of aggregate A are computed once per workgroup into LDS:
// the site of an offset takes a chain of integer divisions by run-time
// extents, which per use would cost more vector instructions than the matrix
// products.  Aggregates of up to kAggTab sites (8^4) take these kernels.
constexpr int kAggTab = 4096;

struct AggSites {
  const int* tab;
  __device__ __forceinline__ int operator()(int l) const { return tab[l]; }
};

// Fills tab with the nsa sites from offset `first` (every thread of the
// workgroup takes part; ends with a barrier).
__device__ __forceinline__ AggSites agg_sites(const AggGeom& a, int A, int nsa, int* tab, int first = 0) {
  for (int l = threadIdx.x; l < nsa; l += blockDim.x) tab[l] = agg_site(a, A, first + l);
  __syncthreads();
  return AggSites{tab};
}

__device__ __forceinline__ bf16x8 to_bf16(const float (&x)[8]) {
  bf16x8 v;
#pragma unroll
  for (int q = 0; q < 8; ++q) v[q] = (__bf16)x[q];
  return v;
}

// One workgroup per (aggregate, chirality, 32-column tile); its four
// wavefronts take a quarter of the rows each and are summed through LDS in a
// fixed order.
__global__ __launch_bounds__(256) void restrict_bf16_kernel(AggGeom a, int h, int nrhs, int ntile,
                                                            const unsigned* __restrict__ W,
                                                            const float2* __restrict__ f, float2* __restrict__ y) {
  __shared__ float red[3][64][16];
  const int bid = blockIdx.x;
  const int tile = bid % ntile;
  const int chi = (bid / ntile) & 1;
  const int A = bid / ntile >> 1;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int m = lane & 31, g = lane >> 5;
  const int ncomp = 2 * h;
  const int nsa = a.b[0] * a.b[1] * a.b[2] * a.b[3];
  const int per_c = nsa / 8;  // MFMA steps per component
  const int steps = h * per_c;
  const int s0 = wave * steps / 4, s1 = (wave + 1) * steps / 4;
  const int k = tile * 32 + m;
  const bool kin = k < nrhs;
  const int i = m & 15;
  const bool imrow = m >= 16;
  __shared__ int stab[kAggTab];
  const AggSites site_of = agg_sites(a, A, nsa, stab);
  f32x16 acc = {};
  // four MFMA steps' loads in flight together, from clamped addresses with
  // the operands zeroed instead of branching (steps past the end and
  // columns past nrhs add zero products)
  constexpr int U = 4;
  const int kc = kin ? k : nrhs - 1;
  for (int s = s0; s < s1; s += U) {
    u32x4 av[U];
    float bv[U][8];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in = s + u < s1;
      const int su = in ? s + u : s0;
      const int c = su / per_c;
      const int l0 = (su - c * per_c) * 8 + 4 * g;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int site = site_of(l0 + j);
        const size_t row = (size_t)site * ncomp + chi * h + c;
        const unsigned w = W[row * kNV + i];
        const float2 v = f[row * nrhs + kc];
        const unsigned x = imrow ? (((w >> 16) ^ 0x8000u) | (w << 16)) : w;
        av[u][j] = in ? x : 0u;
        bv[u][2 * j] = (in && kin) ? v.x : 0.f;
        bv[u][2 * j + 1] = (in && kin) ? v.y : 0.f;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av[u]), to_bf16(bv[u]), acc, 0, 0, 0);
  }
  if (wave > 0) {
#pragma unroll
    for (int p = 0; p < 16; ++p) red[wave - 1][lane][p] = acc[p];
  }
  __syncthreads();
  if (wave == 0) {
#pragma unroll
    for (int w = 0; w < 3; ++w)
#pragma unroll
      for (int p = 0; p < 16; ++p) acc[p] += red[w][lane][p];
    if (kin) {
#pragma unroll
      for (int p = 0; p < 8; ++p) {
        const int row = 8 * (p / 4) + 4 * g + (p % 4);
        y[((size_t)A * 2 * kNV + chi * kNV + row) * nrhs + k] = make_float2(acc[p], acc[p + 8]);
      }
    }
  }
}

// One workgroup per (aggregate, chirality, 32-column tile); the coarse
// values are loaded once, and the four wavefronts walk the 16-row tiles of
// the aggregate in turn.
__global__ __launch_bounds__(256) void prolong_bf16_kernel(AggGeom a, int h, int nrhs, int ntile,
                                                           const unsigned* __restrict__ W,
                                                           const float2* __restrict__ y, float2* __restrict__ f) {
  const int bid = blockIdx.x;
  const int tile = bid % ntile;
  const int chi = (bid / ntile) & 1;
  const int A = bid / ntile >> 1;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int m = lane & 31, g = lane >> 5;
  const int ncomp = 2 * h;
  const int nsa = a.b[0] * a.b[1] * a.b[2] * a.b[3];
  const int k = tile * 32 + m;
  const bool kin = k < nrhs;
  const bool imrow = m >= 16;
  __shared__ int stab[kAggTab];
  const AggSites site_of = agg_sites(a, A, nsa, stab);
  bf16x8 B[2];
#pragma unroll
  for (int st = 0; st < 2; ++st) {
    float bv[8];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int i = st * 8 + 4 * g + j;
      // clamped column, zeroed past nrhs (no branch around the loads)
      const float2 v = y[((size_t)A * 2 * kNV + chi * kNV + i) * nrhs + (kin ? k : nrhs - 1)];
      bv[2 * j] = kin ? v.x : 0.f;
      bv[2 * j + 1] = kin ? v.y : 0.f;
    }
    B[st] = to_bf16(bv);
  }
  const int ntr = h * nsa / 16;
  // Software pipeline over the row tiles of the wavefront (t, t + 4, ...):
  // the basis loads of the next tile are issued before the matrix
  // instructions of the current one.  A tile past the end loads the first
  // tile's rows again and writes nothing.
  auto load = [&](int t, u32x4 (&wt)[2]) {
    const int tc = t < ntr ? t : wave;
    const int r0 = tc * 16;
    const int c = r0 / nsa;
    const int l0 = r0 - c * nsa;
    // A operand: row r0 + (m & 15)
    const size_t arow = (size_t)site_of(l0 + (m & 15)) * ncomp + chi * h + c;
#pragma unroll
    for (int st = 0; st < 2; ++st) wt[st] = *reinterpret_cast<const u32x4*>(W + arow * kNV + st * 8 + 4 * g);
  };
  auto row_tile = [&](int t, const u32x4 (&wt)[2]) {
    const int r0 = t * 16;
    const int c = r0 / nsa;
    const int l0 = r0 - c * nsa;
    f32x16 acc = {};
#pragma unroll
    for (int st = 0; st < 2; ++st) {
      u32x4 w = wt[st];
#pragma unroll
      for (int j = 0; j < 4; ++j) w[j] = imrow ? ((w[j] >> 16) | (w[j] << 16)) : (w[j] ^ 0x80000000u);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w), B[st], acc, 0, 0, 0);
    }
    if (kin && t < ntr) {
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        const int lb = l0 + 8 * half + 4 * g;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int site = site_of(lb + j);
          const int p = 4 * half + j;
          f[((size_t)site * ncomp + chi * h + c) * nrhs + k] = make_float2(acc[p], acc[p + 8]);
        }
      }
    }
  };
  u32x4 wA[2], wB[2];
  if (wave < ntr) load(wave, wA);
  for (int t = wave; t < ntr; t += 8) {
    load(t + 4, wB);
    row_tile(t, wA);
    load(t + 8, wA);
    row_tile(t + 4, wB);
  }
}

// FP32 restrict on the FP32 matrix cores; workgroup and wavefront split as
// in restrict_bf16_kernel, the rows of (A, chi) taken site by site (all h
// components of a site in turn).  H > 0 fixes h at compile time, so that the
// loads of a site are issued together (H = 0: any h).
template <int H>
__global__ __launch_bounds__(256) void restrict_f32_kernel(AggGeom a, int h, int nrhs, int ntile,
                                                           const float2* __restrict__ W,
                                                           const float2* __restrict__ f, float2* __restrict__ y) {
  __shared__ float red[3][64][16];
  const int bid = blockIdx.x;
  const int tile = bid % ntile;
  const int chi = (bid / ntile) & 1;
  const int A = bid / ntile >> 1;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int m = lane & 31, g = lane >> 5;
  const int ncomp = 2 * h;
  const int nsa = a.b[0] * a.b[1] * a.b[2] * a.b[3];
  const int l0 = wave * nsa / 4, l1 = (wave + 1) * nsa / 4;
  const int k = tile * 32 + m;
  const bool kin = k < nrhs;
  const int i = m & 15;
  const bool imrow = m >= 16;
  __shared__ int stab[kAggTab];
  const AggSites site_of = agg_sites(a, A, nsa, stab);
  f32x16 acc = {};
  if constexpr (H > 0) {
    // Software pipeline over the sites of the wavefront: the loads of the
    // next US sites are issued before the matrix instructions of the current
    // ones (the compiler does not unroll a loop around the matrix
    // instruction by itself).  Addresses are clamped to valid ones and the
    // operands zeroed instead of branching, so a site past the end and a
    // column past nrhs add zero products.
    constexpr int US = H <= 8 ? 2 : 1;
    const int kc = kin ? k : nrhs - 1;
    auto load = [&](int lb, float2 (&w)[US][H], float2 (&v)[US][H]) {
#pragma unroll
      for (int u = 0; u < US; ++u) {
        const size_t row0 = (size_t)site_of(lb + u < l1 ? lb + u : l0) * ncomp + chi * H;
#pragma unroll
        for (int c = 0; c < H; ++c) {
          w[u][c] = W[(row0 + c) * kNV + i];
          v[u][c] = f[(row0 + c) * nrhs + kc];
        }
      }
    };
    auto mma = [&](int lb, const float2 (&w)[US][H], const float2 (&v)[US][H]) {
#pragma unroll
      for (int u = 0; u < US; ++u) {
        const bool in = lb + u < l1;
#pragma unroll
        for (int c = 0; c < H; ++c) {
          // g = 0: coefficient of Re f, g = 1: of Im f
          const float x = imrow ? (g ? w[u][c].x : -w[u][c].y) : (g ? w[u][c].y : w[u][c].x);
          const float av = in ? x : 0.f;
          const float bv = (in && kin) ? (g ? v[u][c].y : v[u][c].x) : 0.f;
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av, bv, acc, 0, 0, 0);
        }
      }
    };
    float2 wA[US][H], vA[US][H], wB[US][H], vB[US][H];
    if (l0 < l1) load(l0, wA, vA);
    for (int l = l0; l < l1; l += 2 * US) {
      load(l + US, wB, vB);
      mma(l, wA, vA);
      load(l + 2 * US, wA, vA);
      mma(l + US, wB, vB);
    }
  } else {
    for (int l = l0; l < l1; ++l) {
      const size_t row0 = (size_t)site_of(l) * ncomp + chi * h;
      for (int c = 0; c < h; ++c) {
        const float2 wc = W[(row0 + c) * kNV + i];
        const float2 vc = kin ? f[(row0 + c) * nrhs + k] : make_float2(0.f, 0.f);
        const float av = imrow ? (g ? wc.x : -wc.y) : (g ? wc.y : wc.x);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av, g ? vc.y : vc.x, acc, 0, 0, 0);
      }
    }
  }
  if (wave > 0) {
#pragma unroll
    for (int p = 0; p < 16; ++p) red[wave - 1][lane][p] = acc[p];
  }
  __syncthreads();
  if (wave == 0) {
#pragma unroll
    for (int w = 0; w < 3; ++w)
#pragma unroll
      for (int p = 0; p < 16; ++p) acc[p] += red[w][lane][p];
    if (kin) {
#pragma unroll
      for (int p = 0; p < 8; ++p) {
        const int r = 8 * (p / 4) + 4 * g + (p % 4);
        y[((size_t)A * 2 * kNV + chi * kNV + r) * nrhs + k] = make_float2(acc[p], acc[p + 8]);
      }
    }
  }
}

// FP32 prolong on the FP32 matrix cores: as prolong_bf16_kernel, sixteen
// contraction steps (one per basis index) per 16-row tile.
__global__ __launch_bounds__(256) void prolong_f32_kernel(AggGeom a, int h, int nrhs, int ntile,
                                                          const float2* __restrict__ W,
                                                          const float2* __restrict__ y, float2* __restrict__ f) {
  const int bid = blockIdx.x;
  const int tile = bid % ntile;
  const int chi = (bid / ntile) & 1;
  const int A = bid / ntile >> 1;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int m = lane & 31, g = lane >> 5;
  const int ncomp = 2 * h;
  const int nsa = a.b[0] * a.b[1] * a.b[2] * a.b[3];
  const int k = tile * 32 + m;
  const bool kin = k < nrhs;
  const bool imrow = m >= 16;
  __shared__ int stab[kAggTab];
  const AggSites site_of = agg_sites(a, A, nsa, stab);
  float bv[kNV];
#pragma unroll
  for (int i = 0; i < kNV; ++i) {
    // a column past nrhs reads column nrhs - 1: B column k feeds only output
    // column k, which is not stored (and a select here would let the
    // compiler put each load behind a branch of its own)
    const float2 v = y[((size_t)A * 2 * kNV + chi * kNV + i) * nrhs + (kin ? k : nrhs - 1)];
    bv[i] = g ? v.y : v.x;
  }
  const int ntr = h * nsa / 16;
  // Software pipeline over the row tiles of the wavefront (t, t + 4, ...):
  // the basis loads of the next tile are issued before the matrix
  // instructions of the current one.  A tile past the end loads the first
  // tile's rows again and writes nothing.
  auto load = [&](int t, float4 (&wt)[kNV / 2]) {
    const int tc = t < ntr ? t : wave;
    const int r0 = tc * 16;
    const int c = r0 / nsa;
    const int lb0 = r0 - c * nsa;
    const size_t arow = (size_t)site_of(lb0 + (m & 15)) * ncomp + chi * h + c;
    const float4* wr = reinterpret_cast<const float4*>(W + arow * kNV);
#pragma unroll
    for (int q = 0; q < kNV / 2; ++q) wt[q] = wr[q];  // basis values i = 2q and 2q + 1
  };
  auto row_tile = [&](int t, const float4 (&wt)[kNV / 2]) {
    const int r0 = t * 16;
    const int c = r0 / nsa;
    const int lb0 = r0 - c * nsa;
    f32x16 acc = {};
#pragma unroll
    for (int q = 0; q < kNV / 2; ++q) {
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const float wre = e ? wt[q].z : wt[q].x, wim = e ? wt[q].w : wt[q].y;
        // g = 0: coefficient of Re y, g = 1: of Im y
        const float av = imrow ? (g ? wre : wim) : (g ? -wim : wre);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av, bv[2 * q + e], acc, 0, 0, 0);
      }
    }
    if (kin && t < ntr) {
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        const int lb = lb0 + 8 * half + 4 * g;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int site = site_of(lb + j);
          const int p = 4 * half + j;
          f[((size_t)site * ncomp + chi * h + c) * nrhs + k] = make_float2(acc[p], acc[p + 8]);
        }
      }
    }
  };
  float4 wA[kNV / 2], wB[kNV / 2];
  if (wave < ntr) load(wave, wA);
  for (int t = wave; t < ntr; t += 8) {
    load(t + 4, wB);
    row_tile(t, wA);
    load(t + 8, wA);
    row_tile(t + 4, wB);
  }
}

// ---- staged kernels (h = 6, the fine level, and h = 16, n_v = 16 below it) ----------
// A vector-memory instruction of a wavefront takes 16 cycles of its CU's
// address and cache pipeline however narrow its lanes are, so the kernels
// above, which load MFMA operands straight from memory (4 or 8 bytes a lane,
// most of them read by two or four lanes), are bound by the number of their
// instructions: 32 cycles per row of (A, chi) in the FP32 restriction, half of
// the 64-cycle matrix instruction it feeds on each of four SIMDs and not
// overlapped well with it.  Here the workgroup copies TS sites at a time, all
// rows and columns, as flat 16-byte words (a site's rows of one chirality are
// contiguous in the basis and in the field), keeps the next tile's words in
// registers while it works on the current one, and builds the operands from
// LDS.  Prolongation writes its tile to LDS too, so that whole rows go out as
// 16-byte words.  All column tiles of a site belong to one workgroup, so the
// basis is read once for up to 64 right-hand sides.
// 24^4 with 4^4 aggregates, restrict / prolong in us, each in a loop of its own
// (in turn a prolongation is up to an eighth faster and the restriction after it
// up to a fifth slower, which then waits for what the first left in the caches
// to be written back; pair by pair 516 and 412 at 24), before -> now:
//   FP32 at 12 RHS 362 / 332 -> 219 / 213, at 24 400 / 382 -> 245 / 265 (5.2 and
//   4.8 TB/s), at 48 710 / 612 -> 452 / 503;
//   BF16 at 12 RHS 180 / 249 -> 117 / 143, at 24 227 / 319 -> 187 / 208 (5.5 and
//   4.9 TB/s), at 48 373 / 458 -> 327 / 374.
// Sites per tile: 96 rows (H = 6) or 64 (H = 16); twice that for the BF16
// restriction of up to 16 right-hand sides.
template <int H>
constexpr int kTileSites = H == 6 ? 16 : 4;

// Workgroups are dealt round-robin to the eight XCDs; the two chiralities of
// an aggregate, whose rows alternate in memory, go to the same one in turn.
// An aggregate may be split into `parts` workgroups per chirality.
__device__ __forceinline__ bool staged_block(const AggGeom& a, int parts, int& A, int& chi, int& part) {
  const int j = blockIdx.x >> 3;
  chi = j & 1;
  part = (j >> 1) % parts;
  A = (j >> 1) / parts * 8 + (blockIdx.x & 7);
  return A < a.Vc;
}

__device__ __forceinline__ unsigned pack_bf16(float re, float im) {
  typedef __bf16 b2 __attribute__((ext_vector_type(2)));
  const b2 v = {(__bf16)re, (__bf16)im};
  return __builtin_bit_cast(unsigned, v);
}

// The flat copy of one tile: WPS 16-byte words per site, word p of the tile is
// word p % WPS of its site p / WPS; thread t takes p = t, t + THREADS, ....
// The word's site within the tile and its byte offset within the site's rows
// are the same for every tile.
template <int THREADS, int MAXW>
struct FlatTile {
  int site[MAXW];
  unsigned off[MAXW];
  int nw;  // words of a tile
  __device__ __forceinline__ FlatTile(int wps, int ts) : nw(wps * ts) {
#pragma unroll
    for (int j = 0; j < MAXW; ++j) {
      int p = (int)threadIdx.x + j * THREADS;
      if (p >= nw) p = nw - 1;
      site[j] = p / wps;
      off[j] = (unsigned)(p - site[j] * wps) * 16u;
    }
  }
  __device__ __forceinline__ bool has(int j) const { return (int)threadIdx.x + j * THREADS < nw; }
};

// restrict: per tile, wavefront w of four contracts the rows w RT / 4 ... of
// the tile; the four partial results are added in a fixed order at the end.
// MAXF bounds the words of the field a thread copies per tile.
template <int H, int TS, int NT, bool BF16, int MAXF>
__global__ __launch_bounds__(256) void restrict_staged_kernel(AggGeom a, int nrhs, const void* __restrict__ Wv,
                                                              const float2* __restrict__ f, float2* __restrict__ y) {
  constexpr int RT = TS * H, RW = RT / 4;
  constexpr int WROW = BF16 ? 20 : 32;               // 4-byte words per basis row in LDS
  constexpr int WPS = H * kNV * (BF16 ? 4 : 8) / 16;  // 16-byte words of a site's basis rows
  constexpr int MAXB = (TS * WPS + 255) / 256;
  extern __shared__ __attribute__((aligned(16))) unsigned lds[];
  int A, chi, part;
  if (!staged_block(a, 1, A, chi, part)) return;  // whole workgroup
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int m = lane & 31, g = lane >> 5, i = m & 15;
  const bool imrow = m >= 16;
  const int nsa = a.b[0] * a.b[1] * a.b[2] * a.b[3];
  unsigned* wl = lds;               // [RT][WROW]
  unsigned* fl = lds + RT * WROW;   // [RT][nrhs] complex (FP32, or BF16 packed)
  int* stab = reinterpret_cast<int*>(fl + RT * nrhs * (BF16 ? 1 : 2) + 64);
  const AggSites site_of = agg_sites(a, A, nsa, stab);
  const char* wb = static_cast<const char*>(Wv) + (size_t)chi * WPS * 16;
  const char* fb = reinterpret_cast<const char*>(f) + (size_t)chi * H * nrhs * 8;
  const size_t frow = (size_t)2 * H * nrhs * 8;
  const FlatTile<256, MAXB> tw(WPS, TS);
  const FlatTile<256, MAXF> tf(H * nrhs / 2, TS);
  u32x4 rw[MAXB], rf[MAXF];
  auto load = [&](int l0) {
#pragma unroll
    for (int j = 0; j < MAXB; ++j)
      rw[j] = *reinterpret_cast<const u32x4*>(wb + (size_t)site_of(l0 + tw.site[j]) * (2 * WPS * 16) + tw.off[j]);
#pragma unroll
    for (int j = 0; j < MAXF; ++j)
      rf[j] = *reinterpret_cast<const u32x4*>(fb + (size_t)site_of(l0 + tf.site[j]) * frow + tf.off[j]);
  };
  f32x16 acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = f32x16{};
  load(0);
  for (int l0 = 0; l0 < nsa; l0 += TS) {
    if (l0) __syncthreads();
#pragma unroll
    for (int j = 0; j < MAXB; ++j)
      if (tw.has(j)) {
        const int p = threadIdx.x + j * 256;
        if constexpr (BF16)
          *reinterpret_cast<u32x4*>(wl + (p >> 2) * WROW + (p & 3) * 4) = rw[j];
        else
          *reinterpret_cast<u32x4*>(wl + p * 4) = rw[j];
      }
#pragma unroll
    for (int j = 0; j < MAXF; ++j)
      if (tf.has(j)) {
        const int p = threadIdx.x + j * 256;
        if constexpr (BF16)
          *reinterpret_cast<uint2*>(fl + p * 2) =
              make_uint2(pack_bf16(__uint_as_float(rf[j][0]), __uint_as_float(rf[j][1])),
                         pack_bf16(__uint_as_float(rf[j][2]), __uint_as_float(rf[j][3])));
        else
          *reinterpret_cast<u32x4*>(fl + p * 4) = rf[j];
      }
    __syncthreads();
    if (l0 + TS < nsa) load(l0 + TS);
    __builtin_amdgcn_sched_barrier(0);
    // columns past nrhs read the next row's values: B column k feeds only
    // output column k, which is not stored
    if constexpr (BF16) {
#pragma unroll
      for (int q = 0; q < RW; q += 8) {
        const int r = wave * RW + q + 4 * g;
        u32x4 av;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const unsigned w = wl[(r + j) * WROW + i];
          av[j] = imrow ? (((w >> 16) ^ 0x8000u) | (w << 16)) : w;
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          u32x4 bv;
#pragma unroll
          for (int j = 0; j < 4; ++j) bv[j] = fl[(r + j) * nrhs + t * 32 + m];
          acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av),
                                                           __builtin_bit_cast(bf16x8, bv), acc[t], 0, 0, 0);
        }
      }
    } else {
      const int word = 2 * i + (imrow != (g != 0) ? 1 : 0);
      const unsigned sgn = imrow && !g ? 0x80000000u : 0u;
#pragma unroll
      for (int q = 0; q < RW; ++q) {
        const int r = wave * RW + q;
        const float av = __uint_as_float(wl[r * WROW + word] ^ sgn);
#pragma unroll
        for (int t = 0; t < NT; ++t)
          acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(av, __uint_as_float(fl[(r * nrhs + t * 32 + m) * 2 + g]),
                                                        acc[t], 0, 0, 0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  // sum over the wavefronts: [wavefront][quad of accumulators][lane], then
  // wavefront w = half + 2 (t % 2) adds and stores rows 8 half + 4 g ... of tile t
  typedef float f4 __attribute__((ext_vector_type(4)));
  f4* red = reinterpret_cast<f4*>(lds);
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q)
      red[(wave * 4 + q) * 64 + lane] = f4{acc[t][4 * q], acc[t][4 * q + 1], acc[t][4 * q + 2], acc[t][4 * q + 3]};
    __syncthreads();
    const int half = wave & 1, k = t * 32 + m;
    if ((wave >> 1) == t && k < nrhs) {
      f4 re = red[half * 64 + lane], im = red[(half + 2) * 64 + lane];
#pragma unroll
      for (int w = 1; w < 4; ++w) {
        re += red[(w * 4 + half) * 64 + lane];
        im += red[(w * 4 + half + 2) * 64 + lane];
      }
#pragma unroll
      for (int j = 0; j < 4; ++j)
        y[((size_t)A * 2 * kNV + chi * kNV + 8 * half + 4 * g + j) * nrhs + k] = make_float2(re[j], im[j]);
    }
  }
}

// prolong: the RT / 16 row tiles of a tile are dealt to the wavefronts (three
// for H = 6, four for H = 16), each with all NT column tiles.  On few
// aggregates each is split over `parts` workgroups by sites.
template <int H, int NT, bool BF16, int MAXF>
__global__ __launch_bounds__(H == 6 ? 192 : 256) void prolong_staged_kernel(AggGeom a, int nrhs, int parts,
                                                                            const void* __restrict__ Wv,
                                                                            const float2* __restrict__ y,
                                                                            float2* __restrict__ f) {
  constexpr int TS = kTileSites<H>, RT = TS * H, NW = H == 6 ? 3 : 4, TPB = 64 * NW;
  constexpr int WROW = BF16 ? 20 : 36;  // padded: 16 rows at one word offset fall into 16 bank groups
  constexpr int WW = BF16 ? 4 : 8;      // 16-byte words of a basis row
  constexpr int WPS = H * WW;
  constexpr int MAXB = (TS * WPS + TPB - 1) / TPB;
  extern __shared__ __attribute__((aligned(16))) unsigned lds[];
  int A, chi, part;
  if (!staged_block(a, parts, A, chi, part)) return;  // whole workgroup
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int m = lane & 31, g = lane >> 5;
  const bool imrow = m >= 16;
  const int nsa = a.b[0] * a.b[1] * a.b[2] * a.b[3] / parts;  // sites of this workgroup
  unsigned* wl = lds;                                         // [RT][WROW]
  float2* ol = reinterpret_cast<float2*>(lds + RT * WROW);    // [RT][nrhs]
  int* stab = reinterpret_cast<int*>(ol + RT * nrhs);
  const AggSites site_of = agg_sites(a, A, nsa, stab, part * nsa);
  const char* wb = static_cast<const char*>(Wv) + (size_t)chi * WPS * 16;
  char* fb = reinterpret_cast<char*>(f) + (size_t)chi * H * nrhs * 8;
  const size_t frow = (size_t)2 * H * nrhs * 8;
  const FlatTile<TPB, MAXB> tw(WPS, TS);
  const FlatTile<TPB, MAXF> tf(H * nrhs / 2, TS);
  u32x4 rw[MAXB];
  auto load = [&](int l0) {
#pragma unroll
    for (int j = 0; j < MAXB; ++j)
      rw[j] = *reinterpret_cast<const u32x4*>(wb + (size_t)site_of(l0 + tw.site[j]) * (2 * WPS * 16) + tw.off[j]);
  };
  load(0);
  // the coarse values (a column past nrhs reads column nrhs - 1 and is not stored)
  float bv[BF16 ? 1 : NT][BF16 ? 1 : kNV];
  bf16x8 bb[BF16 ? NT : 1][2];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int k = t * 32 + m < nrhs ? t * 32 + m : nrhs - 1;
    const float2* yb = y + ((size_t)A * 2 * kNV + chi * kNV) * nrhs + k;
    if constexpr (BF16) {
#pragma unroll
      for (int st = 0; st < 2; ++st) {
        float v[8];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float2 z = yb[(size_t)(st * 8 + 4 * g + j) * nrhs];
          v[2 * j] = z.x;
          v[2 * j + 1] = z.y;
        }
        bb[t][st] = to_bf16(v);
      }
    } else {
#pragma unroll
      for (int i = 0; i < kNV; ++i) {
        const float2 z = yb[(size_t)i * nrhs];
        bv[t][i] = g ? z.y : z.x;
      }
    }
  }
  for (int l0 = 0; l0 < nsa; l0 += TS) {
#pragma unroll
    for (int j = 0; j < MAXB; ++j)
      if (tw.has(j)) {
        const int p = threadIdx.x + j * TPB;
        *reinterpret_cast<u32x4*>(wl + (p / WW) * WROW + (p % WW) * 4) = rw[j];
      }
    __syncthreads();
    if (l0 + TS < nsa) load(l0 + TS);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int rt = wave; rt < RT / 16; rt += NW) {
      const int r0 = rt * 16;
      const unsigned* wr = wl + (r0 + (m & 15)) * WROW;
      f32x16 acc[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[t] = f32x16{};
      if constexpr (BF16) {
#pragma unroll
        for (int st = 0; st < 2; ++st) {
          u32x4 w = *reinterpret_cast<const u32x4*>(wr + st * 8 + 4 * g);
#pragma unroll
          for (int j = 0; j < 4; ++j) w[j] = imrow ? ((w[j] >> 16) | (w[j] << 16)) : (w[j] ^ 0x80000000u);
#pragma unroll
          for (int t = 0; t < NT; ++t)
            acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w), bb[t][st], acc[t], 0, 0, 0);
        }
      } else {
        const unsigned sgn = !imrow && g ? 0x80000000u : 0u;
        const unsigned* wi = wr + (imrow != (g != 0) ? 1 : 0);
#pragma unroll
        for (int i = 0; i < kNV; ++i) {
          const float av = __uint_as_float(wi[2 * i] ^ sgn);
#pragma unroll
          for (int t = 0; t < NT; ++t)
            acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(av, bv[t][i], acc[t], 0, 0, 0);
        }
      }
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int k = t * 32 + m;
        if (k < nrhs) {
#pragma unroll
          for (int p = 0; p < 8; ++p)
            ol[(r0 + 8 * (p >> 2) + 4 * g + (p & 3)) * nrhs + k] = make_float2(acc[t][p], acc[t][p + 8]);
        }
      }
    }
    __syncthreads();
    const u32x4* ow = reinterpret_cast<const u32x4*>(ol);
#pragma unroll
    for (int j = 0; j < MAXF; ++j)
      if (tf.has(j))
        *reinterpret_cast<u32x4*>(fb + (size_t)site_of(l0 + tf.site[j]) * frow + tf.off[j]) = ow[threadIdx.x + j * TPB];
  }
}

// LDS (bytes) of a staged kernel on a tile of RT rows: basis rows, field rows
// and the site table (the restriction's sum over the wavefronts reuses them).
size_t staged_lds(bool bf16, bool prolong, int RT, int nrhs, int nsa) {
  const size_t w = (size_t)RT * (bf16 ? 20 : (prolong ? 36 : 32)) * 4;
  const size_t fl = (size_t)RT * nrhs * (bf16 && !prolong ? 4 : 8) + 256;
  const size_t red = 16 * 1024;
  return std::max(w + fl, red) + (size_t)nsa * 4;
}

template <int H, int TS, int NT, bool BF16>
hipError_t launch_restrict_nt(const AggGeom& a, int nrhs, const void* W, const void* f, void* y, hipStream_t s) {
  constexpr int NMAX = TS > kTileSites<H> ? 16 : 32 * NT;
  constexpr int MAXF = (TS * H * NMAX / 2 + 255) / 256;
  const int nsa = a.b[0] * a.b[1] * a.b[2] * a.b[3];
  const unsigned lds = (unsigned)staged_lds(BF16, false, TS * H, nrhs, nsa);
  hipLaunchKernelGGL((restrict_staged_kernel<H, TS, NT, BF16, MAXF>), dim3((unsigned)((a.Vc + 7) / 8 * 16)), dim3(256),
                     lds, s, a, nrhs, W, static_cast<const float2*>(f), static_cast<float2*>(y));
  return hipGetLastError();
}

template <int H, bool BF16>
hipError_t launch_restrict_h(const AggGeom& a, int nrhs, const void* W, const void* f, void* y, hipStream_t s) {
  constexpr int TS = kTileSites<H>;
  const int nsa = a.b[0] * a.b[1] * a.b[2] * a.b[3];
  // tiles of twice the sites where the words per thread stay few: BF16 24^4 at
  // 4 RHS 74 against 85 us (12 RHS 117 / 119); in FP32 they cost a wavefront
  // per SIMD (213 against 197 us at 4 RHS)
  if constexpr (BF16)
    if (nrhs <= 16 && nsa % (2 * TS) == 0) return launch_restrict_nt<H, 2 * TS, 1, BF16>(a, nrhs, W, f, y, s);
  if (nrhs <= 32) return launch_restrict_nt<H, TS, 1, BF16>(a, nrhs, W, f, y, s);
  return launch_restrict_nt<H, TS, 2, BF16>(a, nrhs, W, f, y, s);
}

template <int H, int NT, bool BF16>
hipError_t launch_prolong_nt(const AggGeom& a, int nrhs, const void* W, const void* y, void* f, hipStream_t s) {
  constexpr int TPB = H == 6 ? 192 : 256, TS = kTileSites<H>;
  constexpr int MAXF = (TS * H * 32 * NT / 2 + TPB - 1) / TPB;
  const int nsa = a.b[0] * a.b[1] * a.b[2] * a.b[3];
  int parts = 1;
  while (nsa % (2 * parts * TS) == 0 && (long)a.Vc * 2 * parts < 512) parts *= 2;
  const unsigned lds = (unsigned)staged_lds(BF16, true, TS * H, nrhs, nsa / parts);
  hipLaunchKernelGGL((prolong_staged_kernel<H, NT, BF16, MAXF>), dim3((unsigned)((a.Vc + 7) / 8 * 16 * parts)),
                     dim3(TPB), lds, s, a, nrhs, parts, W, static_cast<const float2*>(y), static_cast<float2*>(f));
  return hipGetLastError();
}

// false (nothing launched): the shape is left to the kernels above
template <bool BF16, bool PROLONG>
bool staged(const AggGeom& a, int h, int nrhs, const void* W, const void* in, void* out, hipStream_t s, hipError_t* e) {
  const int nsa = a.b[0] * a.b[1] * a.b[2] * a.b[3];
  if (h != 6 && h != 16) return false;
  const int TS = h == 6 ? kTileSites<6> : kTileSites<16>;
  const int RT = TS * h * (BF16 && !PROLONG && nrhs <= 16 ? 2 : 1);
  if (nsa % TS || staged_lds(BF16, PROLONG, RT, nrhs, nsa) > 65536) return false;
  if (!intergrid_staged_leads(BF16, PROLONG, a, h, nrhs)) return false;
  if constexpr (PROLONG) {
    if (h == 6)
      *e = nrhs <= 32 ? launch_prolong_nt<6, 1, BF16>(a, nrhs, W, in, out, s)
                      : launch_prolong_nt<6, 2, BF16>(a, nrhs, W, in, out, s);
    else
      *e = nrhs <= 32 ? launch_prolong_nt<16, 1, BF16>(a, nrhs, W, in, out, s)
                      : launch_prolong_nt<16, 2, BF16>(a, nrhs, W, in, out, s);
  } else {
    *e = h == 6 ? launch_restrict_h<6, BF16>(a, nrhs, W, in, out, s) : launch_restrict_h<16, BF16>(a, nrhs, W, in, out, s);
  }
  return true;
}

// FP32 basis [site][ncomp][16] complex -> BF16 pairs (round to nearest even).
__global__ __launch_bounds__(256) void pack_basis_bf16_kernel(const float2* __restrict__ in, unsigned* __restrict__ out,
                                                              long n) {
  const long e = (long)blockIdx.x * 256 + threadIdx.x;
  if (e >= n) return;
  const float2 v = in[e];
  out[e] = (unsigned)bf16_rne_bits(__float_as_uint(v.x)) | ((unsigned)bf16_rne_bits(__float_as_uint(v.y)) << 16);
}

}  // namespace

// More than 32 right-hand sides are two column tiles, which one staged workgroup
// holds and two of the kernels above share: on few or short aggregates the
// latter fill the chip better.  Measured over aggregates of 16 to 512 sites, 1 to
// 512 of them, 33 to 64 right-hand sides, staged / other:
//   FP32 restriction: 1.13 to 1.43 up to 16384 rows (sites times components), 0.5
//   to 1.07 beyond, but 1.05 to 1.39 on up to 64 aggregates of at most 64 fine
//   sites;
//   BF16 restriction: 1.04 to 1.50 on 33 to 64 aggregates (the others have one
//   workgroup per CU there, 0.88 at the least), as fast below, 0.46 to 1.11 above,
//   with 48 and more right-hand sides on up to 128 aggregates of 64 fine sites
//   1.07 to 1.17;
//   aggregates of one tile (16 fine sites): restrictions 0.94 to 1.25, FP32
//   prolongation 1.14 to 1.27 up to 64 of them and 0.72 to 0.90 beyond, BF16 0.95
//   to 1.15; BF16 prolongation to up to 64 sites 0.98 to 1.21 on 64 to 144.
// Up to 32 right-hand sides the staged kernels lead (0.2 to 1.08); the BF16
// restriction of 17 to 32 on up to 32 aggregates is as fast either way.
bool intergrid_staged_leads(bool bf16, bool prolong, const AggGeom& a, int h, int nrhs) {
  const int nsa = a.b[0] * a.b[1] * a.b[2] * a.b[3];
  const bool one_tile = h == 6 && nsa == 16, few_tiles = h == 6 && nsa <= 64;
  if (nrhs <= 32) return !(bf16 && !prolong && nrhs > 16 && a.Vc <= 32);
  if (prolong) return bf16 ? !(one_tile || (few_tiles && a.Vc >= 64 && a.Vc <= 144)) : !(one_tile && a.Vc <= 64);
  if (one_tile || (few_tiles && a.Vc <= 64)) return false;
  return bf16 ? a.Vc > (few_tiles && nsa > 32 && nrhs >= 48 ? 128 : 64) : (long)a.Vc * nsa * h > 16384;
}

bool intergrid_mfma_supported(const AggGeom& a, int h, int nv) {
  const int nsa = a.b[0] * a.b[1] * a.b[2] * a.b[3];
  return nv == kNV && h >= 1 && nsa % 16 == 0 && nsa <= kAggTab;
}

hipError_t launch_pack_basis_bf16(const void* basis32, void* out, long ncomplex, hipStream_t s) {
  hipLaunchKernelGGL(pack_basis_bf16_kernel, dim3((unsigned)((ncomplex + 255) / 256)), dim3(256), 0, s,
                     static_cast<const float2*>(basis32), static_cast<unsigned*>(out), ncomplex);
  return hipGetLastError();
}

hipError_t launch_restrict_bf16(const AggGeom& a, int h, int nrhs, const void* Wbf16, const void* f, void* y,
                                hipStream_t s) {
  if (!intergrid_mfma_supported(a, h, kNV)) return hipErrorInvalidValue;
  hipError_t e;
  if (staged<true, false>(a, h, nrhs, Wbf16, f, y, s, &e)) return e;
  const int ntile = (nrhs + 31) / 32;
  hipLaunchKernelGGL(restrict_bf16_kernel, dim3((unsigned)(a.Vc * 2 * ntile)), dim3(256), 0, s, a, h, nrhs, ntile,
                     static_cast<const unsigned*>(Wbf16), static_cast<const float2*>(f), static_cast<float2*>(y));
  return hipGetLastError();
}

hipError_t launch_prolong_bf16(const AggGeom& a, int h, int nrhs, const void* Wbf16, const void* y, void* f,
                               hipStream_t s) {
  if (!intergrid_mfma_supported(a, h, kNV)) return hipErrorInvalidValue;
  hipError_t e;
  if (staged<true, true>(a, h, nrhs, Wbf16, y, f, s, &e)) return e;
  const int ntile = (nrhs + 31) / 32;
  hipLaunchKernelGGL(prolong_bf16_kernel, dim3((unsigned)(a.Vc * 2 * ntile)), dim3(256), 0, s, a, h, nrhs, ntile,
                     static_cast<const unsigned*>(Wbf16), static_cast<const float2*>(y), static_cast<float2*>(f));
  return hipGetLastError();
}

hipError_t launch_restrict_f32mfma(const AggGeom& a, int h, int nrhs, const void* W32, const void* f, void* y,
                                   hipStream_t s) {
  if (!intergrid_mfma_supported(a, h, kNV)) return hipErrorInvalidValue;
  hipError_t e;
  if (staged<false, false>(a, h, nrhs, W32, f, y, s, &e)) return e;
  const int ntile = (nrhs + 31) / 32;
  const dim3 grid((unsigned)(a.Vc * 2 * ntile));
  const auto* w = static_cast<const float2*>(W32);
  const auto* fi = static_cast<const float2*>(f);
  auto* yo = static_cast<float2*>(y);
  if (h == 6)
    hipLaunchKernelGGL(restrict_f32_kernel<6>, grid, dim3(256), 0, s, a, h, nrhs, ntile, w, fi, yo);
  else if (h == 16)
    hipLaunchKernelGGL(restrict_f32_kernel<16>, grid, dim3(256), 0, s, a, h, nrhs, ntile, w, fi, yo);
  else
    hipLaunchKernelGGL(restrict_f32_kernel<0>, grid, dim3(256), 0, s, a, h, nrhs, ntile, w, fi, yo);
  return hipGetLastError();
}

hipError_t launch_prolong_f32mfma(const AggGeom& a, int h, int nrhs, const void* W32, const void* y, void* f,
                                  hipStream_t s) {
  if (!intergrid_mfma_supported(a, h, kNV)) return hipErrorInvalidValue;
  hipError_t e;
  if (staged<false, true>(a, h, nrhs, W32, y, f, s, &e)) return e;
  const int ntile = (nrhs + 31) / 32;
  hipLaunchKernelGGL(prolong_f32_kernel, dim3((unsigned)(a.Vc * 2 * ntile)), dim3(256), 0, s, a, h, nrhs, ntile,
                     static_cast<const float2*>(W32), static_cast<const float2*>(y), static_cast<float2*>(f));
  return hipGetLastError();
}

}  // namespace mrhs
