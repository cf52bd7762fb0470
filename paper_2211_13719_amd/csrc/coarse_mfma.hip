// Coarse-level 9-point stencil on the matrix cores (paper Sec. 6), for
// Nb = 32 components per site: with many right-hand sides the coarse operator
// becomes, site by site, a sum of nine dense complex 32 x 32 by 32 x Nrhs
// products, which gfx950 runs as BF16 or FP16 MFMA with FP32 accumulation.
//
// Complex arithmetic is split into real products,
//   Re O += Re B Re E - Im B Im E,   Im O += Re B Im E + Im B Re E,
// four v_mfma_f32_32x32x16 per 16-wide slice of the contraction index j.
// One workgroup owns one site and one or two 32-column tiles of right-hand
// sides (two tiles either as columns c0.. and c0 + 32.., or interleaved, even
// columns in one tile and odd in the other, so that a lane reads a column pair
// with one 16-byte load).  The 18 units of work of a site (nine directions,
// two 16-wide slices of j) are dealt to its four or eight wavefronts in turn,
// and their partial sums are added through LDS in a fixed order, which gives
// the latency-bound small coarse lattices several wavefronts per site.  Rows
// of the 32 x 32 output are the 32 coarse components i, columns the
// right-hand sides.
//
// Operand layouts of v_mfma_f32_32x32x16_{bf16,f16} (lane l, 8 values each):
//   A (blocks):  A[i = l % 32][j = 8 (l / 32) + q], q = 0..7
//   B (vectors): B[j = 8 (l / 32) + q][col = l % 32]
//   D (output):  D[8 (r / 4) + 4 (l / 32) + r % 4][l % 32] in accumulator r = 0..15
// Blocks are pre-packed once per level in exactly the A order,
// [site][d][j-slice][re|im][lane][8], so every A load is one 16-byte load per
// lane and 1 KiB contiguous per wavefront.  Vectors stay FP32 in memory
// ([site][j][rhs]); each lane reads its eight values (256-byte contiguous runs
// across the wavefront) and rounds them from FP32 to BF16/FP16 on the fly
// (hardware conversion, round to nearest even; the one-time block pack,
// which starts from FP64, uses the explicit conversions of rounding.h).
// FP16 operands are first scaled per right-hand side by a power of two,
// 2^-E with max_k |x| = m 2^E, m in [0.5, 1), and the output is scaled back in
// FP32; the power of two keeps the scaling exact.
#include <type_traits>

#include "mg_internal.h"
#include "rounding.h"

namespace mrhs {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(8 * sizeof(_Float16)))) _Float16 f16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

constexpr int kNb = 32;
// Partial sums of an MR step that every workgroup of the next one sums itself,
// at most kMrMergedRows rows and kMrMergedBytes per column tile; above it a
// launch of its own does.  Per step (us, own sum / launch): 3^3 x 16 (216 rows)
// 11.5 / 13.5 at 12 RHS (62 KB), 15.5 / 16.2 at 24 (124 KB), 27.9 / 25.8 at 48
// (249 KB); 4^3 x 8 (256 rows) 12.9 / 14.7 at 16 (98 KB), 18.0 / 17.6 at 24
// (147 KB); 4^3 x 16 (512 rows) 24.0 / 19.6 at one RHS already (12 KB, but 16
// dependent loads per lane).
constexpr int kMrMergedRows = 256;
constexpr long kMrMergedBytes = 128 << 10;

__device__ __forceinline__ unsigned short bf16_rne(float f) { return bf16_rne_bits(__float_as_uint(f)); }
__device__ __forceinline__ unsigned short f16_rne(float f) { return f16_rne_bits(__float_as_uint(f)); }

template <bool F16>
struct Op;
template <>
struct Op<false> {
  using vec = bf16x8;
  static __device__ __forceinline__ f32x16 mma(vec a, vec b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
  // FP32 -> BF16 by the hardware conversion, which rounds to nearest even
  // (checked on exact ties; the parity tests compare with the emulation)
  static __device__ __forceinline__ vec cvt(const float (&x)[8]) {
    vec v;
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = (__bf16)x[q];
    return v;
  }
  static __device__ __forceinline__ uint2 cvt4(const float (&x)[4]) {
    typedef __bf16 h4 __attribute__((ext_vector_type(4)));
    const h4 v = {(__bf16)x[0], (__bf16)x[1], (__bf16)x[2], (__bf16)x[3]};
    return __builtin_bit_cast(uint2, v);
  }
};
template <>
struct Op<true> {
  using vec = f16x8;
  static __device__ __forceinline__ f32x16 mma(vec a, vec b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ vec cvt(const float (&x)[8]) {
    vec v;
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = (_Float16)x[q];
    return v;
  }
  static __device__ __forceinline__ uint2 cvt4(const float (&x)[4]) {
    typedef _Float16 h4 __attribute__((ext_vector_type(4)));
    const h4 v = {(_Float16)x[0], (_Float16)x[1], (_Float16)x[2], (_Float16)x[3]};
    return __builtin_bit_cast(uint2, v);
  }
};

// The eight operand values of lanes 0-15 (and 32-47) from four converted by
// each lane: lane c holds values 0-3 of column c, lane c + 16 values 4-7 of
// the same column.  Lanes 16-31 and 48-63 get copies (columns past nrhs).
template <class Vec>
__device__ __forceinline__ Vec join_halves(uint2 v) {
  const auto a = __builtin_amdgcn_permlane16_swap(v.x, v.x, false, false);
  const auto b = __builtin_amdgcn_permlane16_swap(v.y, v.y, false, false);
  return __builtin_bit_cast(Vec, make_uint4(a[0], b[0], a[1], b[1]));
}

// Workgroups are dealt round-robin to the 8 XCDs; remap so that every XCD
// works on one contiguous range of sites (and keeps their neighbours' vectors
// in its own L2).  The grid is a multiple of 8; surplus workgroups get an
// index past the end and exit.
__device__ __forceinline__ int xcd_block(int nblocks) {
  const int b = blockIdx.x;
  const int per = (nblocks + 7) >> 3;
  return (b & 7) * per + (b >> 3);
}

// Adds the partial accumulators of the four wavefronts as (0 + 2) + (1 + 3),
// through 16 KiB of LDS.  Returns false on the wavefronts that have nothing
// left to do.
__device__ __forceinline__ bool reduce_waves(f32x16& accR, f32x16& accI) {
  __shared__ float red[2][64][32];
  const int l = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (wv >= 2) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      red[wv - 2][l][r] = accR[r];
      red[wv - 2][l][16 + r] = accI[r];
    }
  }
  __syncthreads();
  if (wv < 2) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      accR[r] += red[wv][l][r];
      accI[r] += red[wv][l][16 + r];
    }
  }
  __syncthreads();
  if (wv == 1) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      red[0][l][r] = accR[r];
      red[0][l][16 + r] = accI[r];
    }
  }
  __syncthreads();
  if (wv != 0) return false;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    accR[r] += red[0][l][r];
    accI[r] += red[0][l][16 + r];
  }
  return true;
}

// Sum of the WV wavefronts' accumulators, scattered over them: wavefront wv
// gets the accumulator rows r = wv G + q, q < G = 16 / WV.  Every wavefront
// writes its 32 accumulators to buf once (WV x 2048 floats), as vectors of G
// that lie lane by lane, so neither the writes nor the reads conflict, and one
// barrier separates the two.  The partial sums are added as a halving tree
// (w + h added into w for h = WV / 2, ..., 1; for WV = 4 that is
// (0 + 2) + (1 + 3)).  Each wavefront then finishes and stores its own rows
// instead of leaving all of them to the first one (the tree through lane-major
// LDS rows with all stores by wavefront 0 before: 4^3 x 16 in BF16 11.6 us at
// 24 RHS and 18.4 at 48, now 10.0 and 13.8).  Every thread of the WV wavefronts
// must call it, and a barrier must come before buf is used again.
template <int WV>
__device__ __forceinline__ void reduce_scatter(const f32x16& accR, const f32x16& accI, float* buf, int wv,
                                               float (&oR)[16 / WV], float (&oI)[16 / WV]) {
  constexpr int G = 16 / WV;
  typedef float vecg __attribute__((ext_vector_type(G)));
  vecg* b = reinterpret_cast<vecg*>(buf);
  const int l = threadIdx.x & 63;
#pragma unroll
  for (int gr = 0; gr < WV; ++gr) {
    vecg vr, vi;
#pragma unroll
    for (int q = 0; q < G; ++q) {
      vr[q] = accR[gr * G + q];
      vi[q] = accI[gr * G + q];
    }
    b[((wv * WV + gr) * 2 + 0) * 64 + l] = vr;
    b[((wv * WV + gr) * 2 + 1) * 64 + l] = vi;
  }
  __syncthreads();
  vecg sr[WV], si[WV];
#pragma unroll
  for (int w = 0; w < WV; ++w) {
    sr[w] = b[((w * WV + wv) * 2 + 0) * 64 + l];
    si[w] = b[((w * WV + wv) * 2 + 1) * 64 + l];
  }
#pragma unroll
  for (int h = WV / 2; h >= 1; h >>= 1)
#pragma unroll
    for (int w = 0; w < h; ++w) {
      sr[w] += sr[w + h];
      si[w] += si[w + h];
    }
#pragma unroll
  for (int q = 0; q < G; ++q) {
    oR[q] = sr[0][q];
    oI[q] = si[0][q];
  }
}

// Component (row of the 32 x 32 output) of accumulator r on lane l.
__device__ __forceinline__ int acc_row(int r, int l) { return 8 * (r >> 2) + 4 * (l >> 5) + (r & 3); }

// Even-odd modes of the stencil kernels (all coarse extents even; a field on
// one parity is [V/2][Nb][nrhs], entry i the site of that parity among 2i,
// 2i + 1): EO = 1 applies the eight hop directions from parity 1 - p to p,
// EO = 2 the self blocks (or the packed blocks bstride = 1 of their
// inverses) on parity p.  EO = 0 is the full stencil.
__device__ __forceinline__ int cb_site(const Geom& g, int i, int p) {
  const int s2 = 2 * i;
  int r = s2;
  int sum = 0;
  for (int m = 0; m < 4; ++m) {
    sum += r % g.L[m];
    r /= g.L[m];
  }
  return (sum & 1) == p ? s2 : s2 + 1;
}

// Neighbour of site s (coordinates x) in direction d of the stencil
// (self, +x, -x, +y, -y, +z, -z, +t, -t), periodic.  Only constant indices
// into the geometry: indexed by a per-lane direction it is read from memory,
// and every such read waits for all loads issued before it, which would
// serialise the units of a wavefront.
__device__ __forceinline__ int stencil_nbr(const Geom& g, int s, const int (&x)[4], int d) {
  int off = 0;
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const int fw = x[m] + 1 < g.L[m] ? g.stride[m] : g.stride[m] * (1 - g.L[m]);
    const int bw = x[m] > 0 ? -g.stride[m] : g.stride[m] * (g.L[m] - 1);
    off = d == 2 * m + 1 ? fw : off;
    off = d == 2 * m + 2 ? bw : off;
  }
  return s + off;
}

// The stencil's work on one site, split into units (d, kc) = (direction,
// 16-wide slice of the contraction index): unit u = 2 d + kc.  Wavefront w of
// WV takes units u0 + w, u0 + w + WV, ... (balanced: 18 units over four
// wavefronts are 5, 5, 4, 4), each unit four v_mfma_f32_32x32x16 per
// 32-column tile of the NT tiles the workgroup covers, so a block slice is
// loaded once for all its right-hand sides.  A unit past the end is computed
// on a valid unit with zero operands (straight-line loads, no branch).
// fetch(row, e, t, d) returns what is loaded at row `row` (of the input field
// of direction d), element offset e = j nrhs + column, for tile t, as a Raw;
// operand(raw, t) turns it into the FP32 operand.  mid() runs once, between
// the loads of the first batch and their use.
// PAIR (with NT = 2): tile 0 holds the even and tile 1 the odd columns of a
// 64-column group, lane l columns c0 + 2 (l % 32) and the next, so each
// operand row is one 16-byte load fetch4(row, e, d) of the column pair at
// element offset e (colc[0] the even column) instead of two 8-byte loads.
// HALF (with NT = 1, at most 16 right-hand sides): the lanes whose column is
// 16 or more would read clamped duplicates; instead each column's rows are
// split over lanes c and c + 16 and the converted operands are joined by a
// row swap, so a wavefront issues half the loads and conversions (BF16 at 12
// RHS: 6^4 14.6 -> 11.6 us, 6^3 x 32 65.9 -> 51.0; at 24 RHS, with all loads,
// 73.6 -> 72.3).  colc[0] is then the column l % 16.
template <bool F16, int WV, int NT, bool PAIR, bool HALF, class Raw, class Fetch, class Fetch4, class Operand, class Mid>
__device__ __forceinline__ void stencil_units(const Geom& g, int s, int io, int EOmode, int nrhs, const uint4* Bp,
                                              int bstride, int wv, const int (&colc)[NT], const bool (&colok)[NT],
                                              const float (&sc)[NT], Fetch&& fetch, Fetch4&& fetch4, Operand&& operand,
                                              Mid&& mid, f32x16 (&accR)[NT], f32x16 (&accI)[NT]) {
  static_assert(!PAIR || NT == 2, "column pairs fill two tiles");
  static_assert(!HALF || NT == 1, "half columns are for one tile");
  constexpr int NQ = HALF ? 4 : 8;  // operand rows per lane and unit
  using O = Op<F16>;
  using vec = typename O::vec;
  // wv, the wavefront index within the site, and with it each unit's
  // direction is uniform (read with readfirstlane by the caller)
  const int l = threadIdx.x & 63;
  const int jh = 8 * (l >> 5) + (HALF ? 4 * ((l >> 4) & 1) : 0);
  int x[4];
  {
    int r = s;
    x[0] = r % g.L[0];
    r /= g.L[0];
    x[1] = r % g.L[1];
    r /= g.L[1];
    x[2] = r % g.L[2];
    x[3] = r / g.L[2];
  }
  const int u0 = EOmode == 1 ? 2 : 0, u1 = EOmode == 2 ? 2 : 18;
  constexpr int KMAX = (18 + WV - 1) / WV;
  // units are handled in batches: every load of a batch is issued before its
  // first matrix instruction, so a wavefront waits for memory once per batch
  // instead of once per unit (with one tile all of a wavefront's units form
  // one batch; with two tiles batches of three bound the registers, and for
  // column pairs smaller batches buy occupancy: one-unit batches on four
  // wavefronts measured fastest, 3 wavefronts per SIMD against 2).  Operands
  // made of two fields (the merged MR step) take twice the registers: batches of
  // three units with one tile (3^3 x 16 at 24 RHS 14.9 us per step, whole
  // batches 15.5) and of one with two (at 48 RHS 24.7 us, batches of three 31)
  constexpr int PB = (sizeof(Raw) > sizeof(float2) && !HALF) ? (NT == 1 ? 3 : 1) : NT == 1 ? KMAX : (PAIR ? (WV == 4 ? 1 : 2) : 3);
#pragma unroll
  for (int k0 = 0; k0 < KMAX; k0 += PB) {
    uint4 br[PB], bi[PB];
    Raw ev[PB][NT][NQ];
    bool live[PB];
#pragma unroll
    for (int kk = 0; kk < PB; ++kk) {
      const int u = u0 + wv + (k0 + kk) * WV;
      live[kk] = (k0 + kk < KMAX) && u < u1;
      const int uc = live[kk] ? u : u0;
      const int d = uc >> 1, kc = uc & 1;
      const int nbr = stencil_nbr(g, s, x, d);
      // input row: EO 1 the neighbour's checkerboard index, EO 2 the output
      // row, EO 3 both (self term on the output row, hops on the neighbours')
      const int ii = EOmode == 1 ? nbr / 2 : (EOmode == 2 ? io : (EOmode == 3 ? (d == 0 ? io : nbr / 2) : nbr));
      const uint4* bp = Bp + ((size_t)s * bstride + d) * 256;
      br[kk] = bp[(kc * 2 + 0) * 64 + l];
      bi[kk] = bp[(kc * 2 + 1) * 64 + l];
      if constexpr (PAIR) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const float4 v = fetch4(ii, (size_t)(kc * 16 + jh + q) * nrhs + colc[0], d);
          ev[kk][0][q] = make_float2(v.x, v.y);
          ev[kk][NT - 1][q] = make_float2(v.z, v.w);
        }
      } else {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int q = 0; q < NQ; ++q) ev[kk][t][q] = fetch(ii, (size_t)(kc * 16 + jh + q) * nrhs + colc[t], t, d);
      }
    }
    if (k0 == 0) mid();
#pragma unroll
    for (int kk = 0; kk < PB; ++kk) {
      const uint4 b_i = bi[kk];
      const uint4 nbi =
          make_uint4(b_i.x ^ 0x80008000u, b_i.y ^ 0x80008000u, b_i.z ^ 0x80008000u, b_i.w ^ 0x80008000u);
      const vec ar = __builtin_bit_cast(vec, br[kk]);
      const vec ai = __builtin_bit_cast(vec, b_i);
      const vec an = __builtin_bit_cast(vec, nbi);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        float er[NQ], ei[NQ];
        const bool on = live[kk] && (HALF || colok[t]);
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          const float2 v = operand(ev[kk][t][q], t);
          er[q] = on ? v.x * sc[t] : 0.f;
          ei[q] = on ? v.y * sc[t] : 0.f;
        }
        vec vr, vi;
        if constexpr (HALF) {
          vr = join_halves<vec>(O::cvt4(er));
          vi = join_halves<vec>(O::cvt4(ei));
        } else {
          vr = O::cvt(er);
          vi = O::cvt(ei);
        }
        accR[t] = O::mma(ar, vr, accR[t]);
        accR[t] = O::mma(an, vi, accR[t]);
        accI[t] = O::mma(ar, vi, accI[t]);
        accI[t] = O::mma(ai, vr, accI[t]);
      }
    }
  }
}

// One workgroup of WV wavefronts per (output site, group of NT 32-column
// tiles of right-hand sides).
// EO = 3 (the coarse Schur complement's outer product, all extents even):
// out = S_p in - H_{p,1-p} in2 on parity p, in on parity p, in2 on 1 - p.
template <bool F16, int EO, int WV, int NT, bool PAIR = false, bool HALF = false>
__global__ __launch_bounds__(64 * WV) void coarse_mfma_kernel(Geom g, int nrhs, const uint4* __restrict__ Bp,
                                                              const float2* __restrict__ in, float2* __restrict__ out,
                                                              const float* __restrict__ scale, int nblocks,
                                                              int parity, int bstride,
                                                              const float2* __restrict__ in2 = nullptr) {
  __shared__ __attribute__((aligned(16))) float red[WV * 2048];
  constexpr int G = 16 / WV;
  const int l = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ngroups = (nrhs + 32 * NT - 1) / (32 * NT);
  const long w = xcd_block(nblocks);
  const int nsite = EO ? g.V / 2 : g.V;
  if (w >= (long)nsite * ngroups) return;  // whole workgroup
  const int io = (int)(w / ngroups);  // output row
  const int s = EO ? cb_site(g, io, parity) : io;
  const int c0 = (int)(w % ngroups) * 32 * NT;
  int col[NT], colc[NT];
  bool colok[NT];
  float sc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    // PAIR: lane l owns the column pair c0 + 2 (l % 32), + 1 (nrhs even)
    col[t] = PAIR ? c0 + 2 * (l & 31) + t : c0 + 32 * t + (l & 31);
    colok[t] = col[t] < nrhs;
    colc[t] = colok[t] ? col[t] : (PAIR ? nrhs - 2 + t : nrhs - 1);
    if constexpr (HALF) colc[t] = (l & 15) < nrhs ? (l & 15) : nrhs - 1;
    sc[t] = (F16 && (HALF || colok[t])) ? scale[colc[t]] : 1.0f;
  }
  f32x16 accR[NT], accI[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    accR[t] = f32x16{};
    accI[t] = f32x16{};
  }
  stencil_units<F16, WV, NT, PAIR, HALF, float2>(
      g, s, io, EO, nrhs, Bp, bstride, wv, colc, colok, sc,
      // EO 3: minus the hop term, read from the second field (the field is
      // selected before the load, so no branch separates the loads)
      [&](int ii, size_t e, int, int d) {
        const bool hop = EO == 3 && d > 0;
        const float2 v = (hop ? in2 : in)[(size_t)ii * kNb * nrhs + e];
        return hop ? make_float2(-v.x, -v.y) : v;
      },
      [&](int ii, size_t e, int d) {
        const bool hop = EO == 3 && d > 0;
        const float4 v = *reinterpret_cast<const float4*>((hop ? in2 : in) + (size_t)ii * kNb * nrhs + e);
        return hop ? make_float4(-v.x, -v.y, -v.z, -v.w) : v;
      },
      [](float2 v, int) { return v; }, [] {}, accR, accI);
  float oR[NT][G], oI[NT][G];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    if (t) __syncthreads();
    reduce_scatter<WV>(accR[t], accI[t], red, wv, oR[t], oI[t]);
  }
  if constexpr (PAIR) {
    if (!colok[0]) return;
    const float inv0 = F16 ? 1.0f / sc[0] : 1.0f, inv1 = F16 ? 1.0f / sc[1] : 1.0f;
    float4* o = reinterpret_cast<float4*>(out + (size_t)io * kNb * nrhs + col[0]);
#pragma unroll
    for (int q = 0; q < G; ++q)
      o[(size_t)acc_row(wv * G + q, l) * nrhs / 2] =
          make_float4(oR[0][q] * inv0, oI[0][q] * inv0, oR[1][q] * inv1, oI[1][q] * inv1);
  } else {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (!colok[t]) continue;
      const float inv = F16 ? 1.0f / sc[t] : 1.0f;  // exact: sc is a power of two
      float2* o = out + (size_t)io * kNb * nrhs + col[t];
#pragma unroll
      for (int q = 0; q < G; ++q)
        o[(size_t)acc_row(wv * G + q, l) * nrhs] = make_float2(oR[t][q] * inv, oI[t][q] * inv);
    }
  }
}

// r_k - a_k p_k in FP32 with the rounding of the separate MR update kernel
// (a_k rounded to FP32 first).
__device__ __forceinline__ float2 mr_residual(float2 rv, float2 pv, float ar, float ai) {
  float2 rn;
  rn.x = fmaf(-ar, pv.x, fmaf(ai, pv.y, rv.x));
  rn.y = fmaf(-ar, pv.y, fmaf(-ai, pv.x, rv.y));
  return rn;
}

// One minimal-residual step on a coarse level with BF16 operands in one launch
// (paper Sec. 6: the coarsest level is latency-bound, so a step should be as
// few kernels as possible, not a stencil, two reductions and an update):
//   a_{i-1} = <p_{i-1}, r_{i-1}> / ||p_{i-1}||^2  summed by every workgroup from
//                                     the partial sums of the previous launch
//   r_i = r_{i-1} - a_{i-1} p_{i-1}   recomputed on the fly wherever the
//                                     stencil reads it, stored for the own site
//   x_i = x_{i-1} + a_{i-1} r_{i-1}   own site, in place
//   p_i = D r_i                       stored
//   per (workgroup, column): <p_i, r_i> and ||p_i||^2 over the Nb rows of its
//   NS sites (FP64), one row of `part`, read by the next launch (ppart, prows).
// All of it is a chain of memory latencies, so the loads that do not depend on
// each other are issued together: the first of the previous partial sums and
// the stencil's operands (the step length is summed while they arrive), and
// the own rows of r, p and x before the wavefronts' reduction, after which
// each wavefront updates and stores its share of the output rows.
// Summing the step length in every workgroup costs prows x 24 bytes per column
// and workgroup out of the L2; mr_step_plan() says up to which size that is
// cheaper than a launch of its own (mr_site_alpha_kernel; then, not MERGED,
// the length is read from aold).
// first: step 0, r_0 = rold as given, x untouched.  Fields [V][Nb][nrhs] FP32;
// rold / pold and rnew / pnew are different buffers (ping-pong across steps).
// The step is a template parameter: a run-time flag around the operand loads
// becomes a branch per load, each waiting for the loads before it.
// Measured per step of a 64-step solve, before (two launches, all loads of the
// epilogue and all stores on wavefront 0) and now, in us: 3^3 x 16 17.2 -> 11.1
// at 12 RHS, 17.5 -> 14.5 at 24, 25.3 -> 23.8 at 64; 2^3 x 4 12.5 -> 6.9 at 12;
// 4^3 x 16 29.3 -> 18.0 at 12.  What is left at 3^3 x 16 and 12 RHS: 7.3 us for
// a step without p and without a step length, 1.3 for reading p too, 2.5 for
// the step length.
struct MrRaw {
  float2 r, p;
};

// v + the value of the lane M = 16 or 32 away (the lane with that index bit
// flipped), the same sum on both, by a row swap in the vector ALU.
template <int M>
__device__ __forceinline__ double add_swapped(double v) {
  const uint2 w = __builtin_bit_cast(uint2, v);
  uint2 a, b;
  if constexpr (M == 16) {
    const auto x = __builtin_amdgcn_permlane16_swap(w.x, w.x, false, false);
    const auto y = __builtin_amdgcn_permlane16_swap(w.y, w.y, false, false);
    a = make_uint2(x[0], y[0]);
    b = make_uint2(x[1], y[1]);
  } else {
    const auto x = __builtin_amdgcn_permlane32_swap(w.x, w.x, false, false);
    const auto y = __builtin_amdgcn_permlane32_swap(w.y, w.y, false, false);
    a = make_uint2(x[0], y[0]);
    b = make_uint2(x[1], y[1]);
  }
  return __builtin_bit_cast(double, a) + __builtin_bit_cast(double, b);
}


// (two tiles on four wavefronts: a register budget of three wavefronts per
// SIMD, 42.8 us against 43.6 at 4^3 x 16 and 48 RHS)
template <int WV, int NT, int NS, bool HALF, bool MERGED, bool first>
__global__ __launch_bounds__(64 * WV * NS, (WV == 4 && NT == 2 && MERGED) ? 3 : 1) void coarse_mr_step_kernel(
    Geom g, int nrhs, const uint4* __restrict__ Bp, const float2* __restrict__ rold, const float2* __restrict__ pold,
    float2* __restrict__ rnew, float2* __restrict__ pnew, float2* __restrict__ x, const double2* __restrict__ aold,
    const double* __restrict__ ppart, int prows, double* __restrict__ part, int nblocks) {
  constexpr int G = 16 / WV, COLS = 32 * NT;
  __shared__ __attribute__((aligned(16))) float red[NS * WV * 2048];
  static_assert(sizeof(red) >= WV * NS * COLS * 24, "sums fit the buffer");
  const int l = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ns = wave / WV, wv = wave - ns * WV;
  const int ngroups = (nrhs + COLS - 1) / COLS;
  const long w = xcd_block(nblocks);
  const int nrow = (g.V + NS - 1) / NS;
  if (w >= (long)nrow * ngroups) return;  // whole workgroup
  const int row = (int)(w / ngroups);
  const bool site_ok = row * NS + ns < g.V;
  const int s = site_ok ? row * NS + ns : g.V - 1;
  const int c0 = (int)(w % ngroups) * COLS;
  int col[NT], colc[NT];
  bool colok[NT];
  float sc[NT], ar[NT], ai[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    col[t] = c0 + 32 * t + (l & 31);
    colok[t] = col[t] < nrhs;
    colc[t] = colok[t] ? col[t] : nrhs - 1;
    if constexpr (HALF) colc[t] = (l & 15) < nrhs ? (l & 15) : nrhs - 1;
    sc[t] = 1.0f;
    const double2 a = first || MERGED ? make_double2(0.0, 0.0) : aold[colc[t]];
    ar[t] = (float)a.x;
    ai[t] = (float)a.y;
  }
  // the previous step's partial sums: lane (sub, cu) of wavefront `wave` takes
  // the rows slot, slot + SLOTS, ... of column c0 + cu, slot = wave SUB + sub;
  // the first PA of them are loaded before anything else, the others PB at a
  // time
  constexpr int CW = HALF ? 16 : COLS, SUB = 64 / CW, SLOTS = WV * NS * SUB;
  constexpr int PA = HALF ? 7 : 2, PB = 6;
  const int ncol = nrhs - c0 < CW ? nrhs - c0 : CW;
  const int cu = l & (CW - 1), slot = wave * SUB + l / CW;
  const bool summing = !first && MERGED && cu < ncol;
  double pp[PA][3];
  if (summing) {
#pragma unroll
    for (int u = 0; u < PA; ++u) {
      const int rr = slot + u * SLOTS;
      const double* q = ppart + ((rr < prows ? rr : prows - 1) * nrhs + c0 + cu) * 3;
#pragma unroll
      for (int c = 0; c < 3; ++c) pp[u][c] = q[c];
    }
  }
  f32x16 accR[NT], accI[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    accR[t] = f32x16{};
    accI[t] = f32x16{};
  }
  // own rows (clamped column): with half columns there are registers to load
  // them before the matrix products, else before the wavefronts' reduction
  float2 rv[NT][G], pv[NT][G], xv[NT][G];
  auto own_rows = [&] {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int q = 0; q < G; ++q) {
        const size_t o = ((size_t)s * kNb + acc_row(wv * G + q, l)) * nrhs + colc[t];
        rv[t][q] = rold[o];
        if constexpr (!first) {
          pv[t][q] = pold[o];
          xv[t][q] = x[o];
        }
      }
  };
  auto step_length = [&] {
    if constexpr (first || !MERGED) return;
    double* sum = reinterpret_cast<double*>(red);  // [wavefront][column][3]
    double v[3] = {0.0, 0.0, 0.0};
    if (summing) {
#pragma unroll
      for (int u = 0; u < PA; ++u)
#pragma unroll
        for (int c = 0; c < 3; ++c) v[c] += slot + u * SLOTS < prows ? pp[u][c] : 0.0;
      for (int r0 = slot + PA * SLOTS; r0 < prows; r0 += PB * SLOTS) {
        double q[PB][3];
#pragma unroll
        for (int u = 0; u < PB; ++u) {
          const int rr = r0 + u * SLOTS;
          const double* e = ppart + ((rr < prows ? rr : prows - 1) * nrhs + c0 + cu) * 3;
#pragma unroll
          for (int c = 0; c < 3; ++c) q[u][c] = e[c];
        }
#pragma unroll
        for (int u = 0; u < PB; ++u)
#pragma unroll
          for (int c = 0; c < 3; ++c) v[c] += r0 + u * SLOTS < prows ? q[u][c] : 0.0;
      }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      if constexpr (CW <= 16) v[c] = add_swapped<16>(v[c]);
      if constexpr (CW <= 32) v[c] = add_swapped<32>(v[c]);
    }
    if (l < CW)
#pragma unroll
      for (int c = 0; c < 3; ++c) sum[(wave * CW + l) * 3 + c] = v[c];
    __syncthreads();
    // every lane adds the wavefronts' sums of its own columns
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      double w[WV * NS][3];
#pragma unroll
      for (int q = 0; q < WV * NS; ++q)
#pragma unroll
        for (int c = 0; c < 3; ++c) w[q][c] = sum[(q * CW + colc[t] - c0) * 3 + c];
#pragma unroll
      for (int h = WV * NS / 2; h >= 1; h >>= 1)
#pragma unroll
        for (int q = 0; q < h; ++q)
#pragma unroll
          for (int c = 0; c < 3; ++c) w[q][c] += w[q + h][c];
      ar[t] = w[0][2] > 0.0 ? (float)(w[0][0] / w[0][2]) : 0.f;
      ai[t] = w[0][2] > 0.0 ? (float)(w[0][1] / w[0][2]) : 0.f;
    }
    __syncthreads();  // red is the wavefronts' reduction buffer next
  };
  // with the step length at hand r_i is formed as its parts arrive, else both
  // are kept until mid() has it
  constexpr bool LATE = MERGED && !first;
  using Raw = std::conditional_t<LATE, MrRaw, float2>;
  stencil_units<false, WV, NT, false, HALF, Raw>(
      g, s, s, 0, nrhs, Bp, 9, wv, colc, colok, sc,
      [&](int ii, size_t e, int t, int) {
        const size_t o = (size_t)ii * kNb * nrhs + e;
        if constexpr (LATE)
          return MrRaw{rold[o], pold[o]};
        else if constexpr (first)
          return rold[o];
        else
          return mr_residual(rold[o], pold[o], ar[t], ai[t]);
      },
      [](int, size_t, int) { return make_float4(0.f, 0.f, 0.f, 0.f); },
      [&](const Raw& v, int t) {
        if constexpr (LATE)
          return mr_residual(v.r, v.p, ar[t], ai[t]);
        else
          return v;
      },
      [&] {
        if constexpr (HALF) own_rows();
        step_length();
      },
      accR, accI);
  // own rows of r_i, x_i, p_i and the partial sums
  if constexpr (!HALF) own_rows();
  double3 sums[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    float oR[G], oI[G];
    if (t) __syncthreads();
    reduce_scatter<WV>(accR[t], accI[t], red + ns * WV * 2048, wv, oR, oI);
    double sx = 0.0, sy = 0.0, sz = 0.0;
    if (colok[t] && site_ok) {
#pragma unroll
      for (int q = 0; q < G; ++q) {
        const size_t o = ((size_t)s * kNb + acc_row(wv * G + q, l)) * nrhs + colc[t];
        float2 ri = rv[t][q];
        if constexpr (!first) {
          ri = mr_residual(rv[t][q], pv[t][q], ar[t], ai[t]);
          float2 xn = xv[t][q];
          xn.x = fmaf(ar[t], rv[t][q].x, fmaf(-ai[t], rv[t][q].y, xn.x));
          xn.y = fmaf(ar[t], rv[t][q].y, fmaf(ai[t], rv[t][q].x, xn.y));
          x[o] = xn;
          rnew[o] = ri;
        }
        pnew[o] = make_float2(oR[q], oI[q]);
        const double px = oR[q], py = oI[q], rx = ri.x, ry = ri.y;
        sx = fma(px, rx, fma(py, ry, sx));
        sy = fma(px, ry, fma(-py, rx, sy));
        sz = fma(px, px, fma(py, py, sz));
      }
    }
    sums[t].x = sx;
    sums[t].y = sy;
    sums[t].z = sz;
  }
  // per column: the two row halves of a wavefront, then the wavefronts
  double* sum = reinterpret_cast<double*>(red);  // [wavefront][tile][column][3]
  __syncthreads();
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    sums[t].x = add_swapped<32>(sums[t].x);
    sums[t].y = add_swapped<32>(sums[t].y);
    sums[t].z = add_swapped<32>(sums[t].z);
    if (l < 32) {
      double* d = sum + ((wave * NT + t) * 32 + l) * 3;
      d[0] = sums[t].x;
      d[1] = sums[t].y;
      d[2] = sums[t].z;
    }
  }
  __syncthreads();
  if (threadIdx.x >= 32) return;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    double v[WV * NS][3];
#pragma unroll
    for (int q = 0; q < WV * NS; ++q)
#pragma unroll
      for (int c = 0; c < 3; ++c) v[q][c] = sum[((q * NT + t) * 32 + l) * 3 + c];
#pragma unroll
    for (int h = WV * NS / 2; h >= 1; h >>= 1)
#pragma unroll
      for (int q = 0; q < h; ++q)
#pragma unroll
        for (int c = 0; c < 3; ++c) v[q][c] += v[q + h][c];
    if (colok[t])
#pragma unroll
      for (int c = 0; c < 3; ++c) part[(row * nrhs + col[t]) * 3 + c] = v[0][c];
  }
}

// Step length of the fused MR step from its partial sums [rows][nrhs][3]: one
// workgroup per column sums the rows in a fixed order (strided by thread, then
// a tree) and writes a = <p, r> / ||p||^2.
__global__ __launch_bounds__(256) void mr_site_alpha_kernel(const double* __restrict__ part, int rows, int nrhs,
                                                            double2* __restrict__ anew) {
  __shared__ double red[3][256];
  const int k = blockIdx.x, t = threadIdx.x;
  double acc[3] = {0.0, 0.0, 0.0};
  for (int row = t; row < rows; row += 4 * 256) {
    double v[4][3];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int rr = row + u * 256 < rows ? row + u * 256 : row;
#pragma unroll
      for (int c = 0; c < 3; ++c) v[u][c] = part[(rr * nrhs + k) * 3 + c];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int c = 0; c < 3; ++c) acc[c] += row + u * 256 < rows ? v[u][c] : 0.0;
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) red[c][t] = acc[c];
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (t < w)
#pragma unroll
      for (int c = 0; c < 3; ++c) red[c][t] += red[c][t + w];
    __syncthreads();
  }
  if (t == 0) {
    const double z = red[2][0];
    anew[k] = z > 0.0 ? make_double2(red[0][0] / z, red[1][0] / z) : make_double2(0.0, 0.0);
  }
}

// After the last fused step: x += a r and, if rout is given, rout = r - a p
// (FP32, the separate update kernel's rounding).  rout may be r itself.
__global__ __launch_bounds__(256) void mr_finish_kernel(float2* __restrict__ x, const float2* r,
                                                        const float2* __restrict__ p, float2* rout,
                                                        const double2* __restrict__ alpha, long n, int nrhs) {
  const long e = (long)blockIdx.x * 256 + threadIdx.x;
  if (e >= n) return;
  const double2 a = alpha[e % nrhs];
  const float ar = (float)a.x, ai = (float)a.y;
  const float2 rv = r[e];
  float2 xv = x[e];
  xv.x = fmaf(ar, rv.x, fmaf(-ai, rv.y, xv.x));
  xv.y = fmaf(ar, rv.y, fmaf(ai, rv.x, xv.y));
  x[e] = xv;
  if (rout) rout[e] = mr_residual(rv, p[e], ar, ai);
}

// FP32 operands on v_mfma_f32_32x32x2_f32 (full-rate FP32 matrix cores):
//   A[i = l % 32][k = l / 32], B[k = l / 32][col = l % 32], D as above,
// so one instruction contracts two values of j.  Blocks are packed
// [site][d][re|im][lane][16] with element q of lane l holding
// B[i = l % 32][j = 2 q + l / 32]: four 16-byte loads per lane per part.
template <int EO>
__global__ __launch_bounds__(256) void coarse_mfma_f32_kernel(Geom g, int nrhs, const float4* __restrict__ Bp,
                                                              const float2* __restrict__ in,
                                                              float2* __restrict__ out, int nblocks, int parity,
                                                              int bstride) {
  const int l = threadIdx.x & 63;
  const int ntiles = (nrhs + 31) >> 5;
  const long w = xcd_block(nblocks);
  const int nsite = EO ? g.V / 2 : g.V;
  if (w >= (long)nsite * ntiles) return;  // whole workgroup
  const int io = (int)(w / ntiles);  // output row
  const int s = EO ? cb_site(g, io, parity) : io;
  const int col = (int)(w % ntiles) * 32 + (l & 31);
  const bool colok = col < nrhs;
  const int colc = colok ? col : nrhs - 1;
  const int jh = l >> 5;
  int x[4];
  {
    int r = s;
    x[0] = r % g.L[0];
    r /= g.L[0];
    x[1] = r % g.L[1];
    r /= g.L[1];
    x[2] = r % g.L[2];
    x[3] = r / g.L[2];
  }
  f32x16 accR = {}, accI = {};
  const int d0 = EO == 1 ? 1 : 0, d1 = EO == 2 ? 1 : 9;
  for (int d = d0 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); d < d1; d += 4) {
    const int nbr = stencil_nbr(g, s, x, d);
    const int ii = EO == 1 ? nbr / 2 : (EO == 2 ? io : nbr);  // input row
    const float4* bp = Bp + ((size_t)s * bstride + d) * 2 * 64 * 4;
    float br[16], bi[16];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 a = bp[(0 * 64 + l) * 4 + q], b = bp[(1 * 64 + l) * 4 + q];
      br[4 * q] = a.x;
      br[4 * q + 1] = a.y;
      br[4 * q + 2] = a.z;
      br[4 * q + 3] = a.w;
      bi[4 * q] = b.x;
      bi[4 * q + 1] = b.y;
      bi[4 * q + 2] = b.z;
      bi[4 * q + 3] = b.w;
    }
    // all vector loads first, from a clamped column (no branch around the
    // loads); columns past nrhs are zeroed and never stored
    const float2* e = in + (size_t)ii * kNb * nrhs + colc;
    float2 ev[16];
#pragma unroll
    for (int kc = 0; kc < 16; ++kc) ev[kc] = e[(size_t)(2 * kc + jh) * nrhs];
#pragma unroll
    for (int kc = 0; kc < 16; ++kc) {
      const float2 v = colok ? ev[kc] : make_float2(0.f, 0.f);
      accR = __builtin_amdgcn_mfma_f32_32x32x2f32(br[kc], v.x, accR, 0, 0, 0);
      accR = __builtin_amdgcn_mfma_f32_32x32x2f32(-bi[kc], v.y, accR, 0, 0, 0);
      accI = __builtin_amdgcn_mfma_f32_32x32x2f32(br[kc], v.y, accI, 0, 0, 0);
      accI = __builtin_amdgcn_mfma_f32_32x32x2f32(bi[kc], v.x, accI, 0, 0, 0);
    }
  }
  if (!reduce_waves(accR, accI) || !colok) return;
  float2* o = out + (size_t)io * kNb * nrhs + col;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int row = 8 * (r >> 2) + 4 * (l >> 5) + (r & 3);
    o[(size_t)row * nrhs] = make_float2(accR[r], accI[r]);
  }
}

__global__ void pack_f32_kernel(const double2* __restrict__ B, float* __restrict__ P, long nblk) {
  const long e = (long)blockIdx.x * 256 + threadIdx.x;
  if (e >= nblk * kNb * kNb) return;
  const long blk = e / (kNb * kNb);
  const int r = (int)(e % (kNb * kNb));
  const int i = r / kNb, j = r % kNb;
  const int lane = i + 32 * (j & 1), q = j >> 1;
  const double2 v = B[e];
  float* base = P + blk * (2 * 64 * 16);
  base[(0 * 64 + lane) * 16 + q] = (float)v.x;
  base[(1 * 64 + lane) * 16 + q] = (float)v.y;
}

// FP64 blocks [site][9][32][32] complex -> packed A-operand order; the value is
// rounded to FP32 first, then to BF16/FP16 (nearest even).
template <bool F16>
__global__ void pack_kernel(const double2* __restrict__ B, unsigned short* __restrict__ P, long nblk) {
  const long e = (long)blockIdx.x * 256 + threadIdx.x;  // one thread per packed element pair (re, im)
  if (e >= nblk * kNb * kNb) return;
  const long blk = e / (kNb * kNb);
  const int r = (int)(e % (kNb * kNb));
  const int i = r / kNb, j = r % kNb;
  const int kc = j / 16, jj = j % 16;
  const int lane = i + 32 * (jj / 8), q = jj % 8;
  const double2 v = B[e];
  const float fr = (float)v.x, fi = (float)v.y;
  unsigned short hr, hi;
  if constexpr (F16) {
    hr = f16_rne(fr);
    hi = f16_rne(fi);
  } else {
    hr = bf16_rne(fr);
    hi = bf16_rne(fi);
  }
  unsigned short* base = P + blk * (2 * 2 * 64 * 8);
  base[((kc * 2 + 0) * 64 + lane) * 8 + q] = hr;
  base[((kc * 2 + 1) * 64 + lane) * 8 + q] = hi;
}

// scale[k] = 2^-E with max over the column of |re|, |im| = m 2^E, m in [0.5, 1); 1 for a zero column.
__global__ void colmax_kernel(const float2* __restrict__ in, long rows, int nrhs, unsigned int* __restrict__ m) {
  const long e0 = (long)blockIdx.x * 256 + threadIdx.x;
  const long n = rows * nrhs;
  const long stride = (long)gridDim.x * 256;
  // the stride is a multiple of nrhs when launched as below, so the column is fixed
  const int k = (int)(e0 % nrhs);
  float mx = 0.f;
  // four loads in flight per thread; an index past the end reads this
  // thread's own first element (valid, as e0 < n inside the loop) and counts
  // zero, so no load sits in a branch
  constexpr int U = 4;
  for (long e = e0; e < n; e += U * stride) {
    float2 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = in[e + u * stride < n ? e + u * stride : e0];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float a = fmaxf(fabsf(v[u].x), fabsf(v[u].y));
      mx = fmaxf(mx, e + u * stride < n ? a : 0.f);
    }
  }
  // one atomic per (workgroup, column): thread j < nrhs combines the threads
  // t = j, j + nrhs, ... of the workgroup, which all hold column k(j)
  __shared__ float smax[256];
  smax[threadIdx.x] = mx;
  __syncthreads();
  if ((int)threadIdx.x < nrhs) {
    float c = 0.f;
    for (int t = threadIdx.x; t < 256; t += nrhs) c = fmaxf(c, smax[t]);
    atomicMax(m + k, __float_as_uint(c));  // non-negative floats order as their bit patterns
  }
}
// Also clears the reduction words, so that the next call starts from zero
// without a separate launch.
__global__ void colmax_to_scale(unsigned int* __restrict__ m, float* __restrict__ scale, int nrhs) {
  const int k = threadIdx.x;
  if (k >= nrhs) return;
  const float mx = __uint_as_float(m[k]);
  int E = 0;
  (void)frexpf(mx, &E);
  scale[k] = mx > 0.f ? ldexpf(1.0f, -E) : 1.0f;
  m[k] = 0u;
}

}  // namespace

bool mfma_supported(int nb) { return nb == kNb; }

size_t mfma_pack_bytes(long nsite) { return (size_t)nsite * 9 * kNb * kNb * 2 * 2; }

hipError_t launch_pack_blocks(int f16, const void* B64, void* packed, long nsite, hipStream_t s) {
  const long n = nsite * 9 * kNb * kNb;
  const int blocks = (int)((n + 255) / 256);
  if (f16)
    hipLaunchKernelGGL((pack_kernel<true>), dim3(blocks), dim3(256), 0, s, static_cast<const double2*>(B64),
                       static_cast<unsigned short*>(packed), nsite * 9);
  else
    hipLaunchKernelGGL((pack_kernel<false>), dim3(blocks), dim3(256), 0, s, static_cast<const double2*>(B64),
                       static_cast<unsigned short*>(packed), nsite * 9);
  return hipGetLastError();
}

// work: nrhs 32-bit words that are zero on entry (and are left zero).
hipError_t launch_column_scale(const void* in, long rows, int nrhs, void* work, float* scale, hipStream_t s) {
  unsigned int* m = static_cast<unsigned int*>(work);
  // workgroup stride must be a multiple of nrhs: use blocks of 256 threads and
  // a grid such that 256 * grid % nrhs == 0 (a few hundred workgroups: every
  // one ends in nrhs atomics on the same nrhs words)
  int grid = 256;
  while ((256L * grid) % nrhs) ++grid;
  hipLaunchKernelGGL(colmax_kernel, dim3(grid), dim3(256), 0, s, static_cast<const float2*>(in), rows, nrhs, m);
  hipLaunchKernelGGL(colmax_to_scale, dim3(1), dim3(64), 0, s, m, scale, nrhs);
  return hipGetLastError();
}

namespace {

template <bool F16, int WV, int NT, bool PAIR = false, bool HALF = false>
hipError_t launch_stencil_t(const Geom& g, int nrhs, const void* packed, const void* in, void* out, const float* scale,
                            hipStream_t s) {
  const int blocks = (int)((long)g.V * ((nrhs + 32 * NT - 1) / (32 * NT)));
  const int grid = ((blocks + 7) / 8) * 8;
  hipLaunchKernelGGL((coarse_mfma_kernel<F16, 0, WV, NT, PAIR, HALF>), dim3(grid), dim3(64 * WV), 0, s, g, nrhs,
                     static_cast<const uint4*>(packed), static_cast<const float2*>(in), static_cast<float2*>(out),
                     scale, blocks, 0, 9, nullptr);
  return hipGetLastError();
}

// How a fused MR step runs on V sites: NS sites per workgroup, one row of
// partial sums per workgroup, and whether the next launch sums those rows
// itself.  Two sites per workgroup where that still leaves about 200
// workgroups halve the rows (3^3 x 16 at 24 RHS 14.9 us per step, one site
// 16.8); with two column tiles a workgroup has enough to do with one (4^3 x 16
// at 48 RHS 42.8 us, two sites 44.5).
struct MrPlan {
  int ns, rows;
  bool merged;
};
MrPlan mr_step_plan(const Geom& g, int nrhs, int cfg) {
  const int wv = cfg & 1 ? 8 : 4, cols = cfg & 2 ? 64 : 32;
  const int ngroups = (nrhs + cols - 1) / cols;
  MrPlan p;
  p.ns = wv == 4 && cols == 32 && (g.V / 2) * ngroups >= 192 ? 2 : 1;
  p.rows = (g.V + p.ns - 1) / p.ns;
  p.merged = p.rows <= kMrMergedRows && (long)p.rows * (nrhs < cols ? nrhs : cols) * 3 * (long)sizeof(double) <= kMrMergedBytes;
  return p;
}

template <int WV, int NT, int NS, bool HALF, bool MERGED>
hipError_t launch_mr_k(const Geom& g, int nrhs, const MrPlan& pl, const void* packed, const void* rold, const void* pold,
                       void* rnew, void* pnew, void* x, const void* aold, const void* ppart, void* part, int first,
                       hipStream_t s) {
  const int blocks = (int)((long)pl.rows * ((nrhs + 32 * NT - 1) / (32 * NT)));
  const int grid = ((blocks + 7) / 8) * 8;
  auto k = first ? coarse_mr_step_kernel<WV, NT, NS, HALF, MERGED, true>
                 : coarse_mr_step_kernel<WV, NT, NS, HALF, MERGED, false>;
  hipLaunchKernelGGL(k, dim3(grid), dim3(64 * WV * NS), 0, s, g, nrhs, static_cast<const uint4*>(packed),
                     static_cast<const float2*>(rold), static_cast<const float2*>(pold), static_cast<float2*>(rnew),
                     static_cast<float2*>(pnew), static_cast<float2*>(x), static_cast<const double2*>(aold),
                     static_cast<const double*>(ppart), pl.rows, static_cast<double*>(part), blocks);
  return hipGetLastError();
}

template <int WV, int NT, int NS, bool HALF>
hipError_t launch_mr_t(const Geom& g, int nrhs, const MrPlan& pl, const void* packed, const void* rold, const void* pold,
                       void* rnew, void* pnew, void* x, const void* aold, const void* ppart, void* part, int first,
                       hipStream_t s) {
  auto l = pl.merged ? launch_mr_k<WV, NT, NS, HALF, true> : launch_mr_k<WV, NT, NS, HALF, false>;
  return l(g, nrhs, pl, packed, rold, pold, rnew, pnew, x, aold, ppart, part, first, s);
}

hipError_t launch_mr_alpha_rows(const void* part, int rows, int nrhs, void* anew, hipStream_t s) {
  hipLaunchKernelGGL(mr_site_alpha_kernel, dim3(nrhs), dim3(256), 0, s, static_cast<const double*>(part), rows, nrhs,
                     static_cast<double2*>(anew));
  return hipGetLastError();
}

}  // namespace

// cfg: launch shape of the BF16/FP16 stencil, bit 0 eight wavefronts per
// workgroup (else four); cfg >> 1 the column tiling: 0 one 32-column tile per
// workgroup, 1 two, 2 two tiles as interleaved column pairs read with 16-byte
// loads (fields are 16-byte aligned, which the entry points check).  The pair
// form needs an even nrhs; for an odd one cfg 4 / 5 run as cfg 2 / 3 (the same
// result).
hipError_t launch_coarse_mfma(int f16, const Geom& g, int nb, int nrhs, const void* packed, const void* in, void* out,
                              const float* scale, hipStream_t s, int cfg) {
  if (nb != kNb || cfg < 0 || cfg >= kLowpCfgs) return hipErrorInvalidValue;
  if (cfg >= 4 && (nrhs & 1)) cfg -= 2;
  if (nrhs <= 16) {  // one tile covers all columns: only the wavefront count is left of cfg
    if (f16)
      return cfg & 1 ? launch_stencil_t<true, 8, 1, false, true>(g, nrhs, packed, in, out, scale, s)
                     : launch_stencil_t<true, 4, 1, false, true>(g, nrhs, packed, in, out, scale, s);
    return cfg & 1 ? launch_stencil_t<false, 8, 1, false, true>(g, nrhs, packed, in, out, scale, s)
                   : launch_stencil_t<false, 4, 1, false, true>(g, nrhs, packed, in, out, scale, s);
  }
  if (f16) {
    switch (cfg) {
      case 0: return launch_stencil_t<true, 4, 1>(g, nrhs, packed, in, out, scale, s);
      case 1: return launch_stencil_t<true, 8, 1>(g, nrhs, packed, in, out, scale, s);
      case 2: return launch_stencil_t<true, 4, 2>(g, nrhs, packed, in, out, scale, s);
      case 3: return launch_stencil_t<true, 8, 2>(g, nrhs, packed, in, out, scale, s);
      case 4: return launch_stencil_t<true, 4, 2, true>(g, nrhs, packed, in, out, scale, s);
      default: return launch_stencil_t<true, 8, 2, true>(g, nrhs, packed, in, out, scale, s);
    }
  }
  switch (cfg) {
    case 0: return launch_stencil_t<false, 4, 1>(g, nrhs, packed, in, out, scale, s);
    case 1: return launch_stencil_t<false, 8, 1>(g, nrhs, packed, in, out, scale, s);
    case 2: return launch_stencil_t<false, 4, 2>(g, nrhs, packed, in, out, scale, s);
    case 3: return launch_stencil_t<false, 8, 2>(g, nrhs, packed, in, out, scale, s);
    case 4: return launch_stencil_t<false, 4, 2, true>(g, nrhs, packed, in, out, scale, s);
    default: return launch_stencil_t<false, 8, 2, true>(g, nrhs, packed, in, out, scale, s);
  }
}

// Two sets of partial sums: a step reads the previous one's and writes its own.
size_t coarse_mr_part_bytes(long nsite) { return 2 * (size_t)nsite * MRHS_MAX_NRHS * 3 * sizeof(double); }

hipError_t launch_coarse_mr_step(const Geom& g, int nb, int nrhs, const void* packed, const void* rold, const void* pold,
                                 void* rnew, void* pnew, void* x, void* alpha, void* part, int step, bool last, int cfg,
                                 hipStream_t s) {
  if (nb != kNb || cfg < 0 || cfg > 3 || nrhs < 1 || nrhs > MRHS_MAX_NRHS || step < 0) return hipErrorInvalidValue;
  const MrPlan pl = mr_step_plan(g, nrhs, cfg);
  const size_t half = coarse_mr_part_bytes(g.V) / 2;
  char* pc = static_cast<char*>(part) + (step & 1) * half;
  const char* pp = static_cast<const char*>(part) + ((step + 1) & 1) * half;
  const int first = step == 0;
  hipError_t e;
#define MRHS_MR(WV, NT, NS, HALF) \
  launch_mr_t<WV, NT, NS, HALF>(g, nrhs, pl, packed, rold, pold, rnew, pnew, x, alpha, pp, pc, first, s)
  if (nrhs <= 16)
    e = cfg & 1 ? MRHS_MR(8, 1, 1, true) : pl.ns == 2 ? MRHS_MR(4, 1, 2, true) : MRHS_MR(4, 1, 1, true);
  else if (cfg == 0)
    e = pl.ns == 2 ? MRHS_MR(4, 1, 2, false) : MRHS_MR(4, 1, 1, false);
  else if (cfg == 1)
    e = MRHS_MR(8, 1, 1, false);
  else if (cfg == 2)
    e = MRHS_MR(4, 2, 1, false);
  else
    e = MRHS_MR(8, 2, 1, false);
#undef MRHS_MR
  if (e == hipSuccess && (last || !pl.merged)) e = launch_mr_alpha_rows(pc, pl.rows, nrhs, alpha, s);
  return e;
}

hipError_t launch_mr_finish(void* x, const void* r, const void* p, void* rout, const void* alpha, long rows, int nrhs,
                            hipStream_t s) {
  const long n = rows * nrhs;
  hipLaunchKernelGGL(mr_finish_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, static_cast<float2*>(x),
                     static_cast<const float2*>(r), static_cast<const float2*>(p), static_cast<float2*>(rout),
                     static_cast<const double2*>(alpha), n, nrhs);
  return hipGetLastError();
}

// Even-odd modes (see cb_site): prec 0 FP32, 1 BF16, 2 FP16 (scale needed);
// eo 1 hop to parity p, eo 2 per-site blocks (bstride 9: the self blocks of
// the stencil pack, 1: a pack of single blocks per site).
hipError_t launch_coarse_mfma_eo(int prec, int eo, int parity, const Geom& g, int nb, int nrhs, const void* packed,
                                 int bstride, const void* in, void* out, const float* scale, hipStream_t s) {
  if (nb != kNb || (eo != 1 && eo != 2) || (parity != 0 && parity != 1)) return hipErrorInvalidValue;
  for (int m = 0; m < 4; ++m)
    if (g.L[m] % 2) return hipErrorInvalidValue;
  const int blocks = (int)((long)(g.V / 2) * ((nrhs + 31) / 32));
  const dim3 grid((unsigned)(((blocks + 7) / 8) * 8));
  const auto* x = static_cast<const float2*>(in);
  auto* y = static_cast<float2*>(out);
  if (prec == 0) {
    const auto* b = static_cast<const float4*>(packed);
    if (eo == 1)
      hipLaunchKernelGGL((coarse_mfma_f32_kernel<1>), grid, dim3(256), 0, s, g, nrhs, b, x, y, blocks, parity,
                         bstride);
    else
      hipLaunchKernelGGL((coarse_mfma_f32_kernel<2>), grid, dim3(256), 0, s, g, nrhs, b, x, y, blocks, parity,
                         bstride);
  } else {
    const auto* b = static_cast<const uint4*>(packed);
    // at most 16 columns: the half-column loads of stencil_units
    const bool half = nrhs <= 16;
    auto k = prec == 2 ? (eo == 1 ? (half ? coarse_mfma_kernel<true, 1, 4, 1, false, true> : coarse_mfma_kernel<true, 1, 4, 1>)
                                  : (half ? coarse_mfma_kernel<true, 2, 4, 1, false, true> : coarse_mfma_kernel<true, 2, 4, 1>))
                       : (eo == 1 ? (half ? coarse_mfma_kernel<false, 1, 4, 1, false, true> : coarse_mfma_kernel<false, 1, 4, 1>)
                                  : (half ? coarse_mfma_kernel<false, 2, 4, 1, false, true> : coarse_mfma_kernel<false, 2, 4, 1>));
    hipLaunchKernelGGL(k, grid, dim3(256), 0, s, g, nrhs, b, x, y, scale, blocks, parity, bstride, nullptr);
  }
  return hipGetLastError();
}

// The coarse Schur complement's outer product on parity p with BF16 operands:
// out = S_p in - H_{p,1-p} in2 (in, out on parity p; in2 on 1 - p).
hipError_t launch_coarse_schur(int parity, const Geom& g, int nb, int nrhs, const void* packed, const void* in,
                               const void* in2, void* out, hipStream_t s) {
  if (nb != kNb || (parity != 0 && parity != 1)) return hipErrorInvalidValue;
  for (int m = 0; m < 4; ++m)
    if (g.L[m] % 2) return hipErrorInvalidValue;
  const int blocks = (int)((long)(g.V / 2) * ((nrhs + 31) / 32));
  auto k = nrhs <= 16 ? coarse_mfma_kernel<false, 3, 4, 1, false, true> : coarse_mfma_kernel<false, 3, 4, 1>;
  hipLaunchKernelGGL(k, dim3((unsigned)(((blocks + 7) / 8) * 8)), dim3(256), 0, s, g, nrhs, static_cast<const uint4*>(packed), static_cast<const float2*>(in),
                     static_cast<float2*>(out), nullptr, blocks, parity, 9, static_cast<const float2*>(in2));
  return hipGetLastError();
}

// Rows of one parity between a full coarse field [V][Nb][nrhs] and a
// checkerboard one [V/2][Nb][nrhs] (entry i: the site of that parity among
// 2i, 2i + 1): half = full rows (gather), or full rows += half (scatter_add).
__global__ __launch_bounds__(256) void cb_rows_kernel(const Geom g, int parity, long rowlen, const float2* __restrict__ src,
                                                      float2* __restrict__ dst, int scatter_add) {
  const int i = blockIdx.y;
  const int s = cb_site(g, i, parity);
  for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < rowlen; e += (long)gridDim.x * 256) {
    if (scatter_add) {
      float2 v = dst[(size_t)s * rowlen + e];
      const float2 h = src[(size_t)i * rowlen + e];
      v.x += h.x;
      v.y += h.y;
      dst[(size_t)s * rowlen + e] = v;
    } else {
      dst[(size_t)i * rowlen + e] = src[(size_t)s * rowlen + e];
    }
  }
}

hipError_t launch_coarse_cb_rows(int parity, const Geom& g, int nb, int nrhs, const void* src, void* dst, int scatter_add,
                                 hipStream_t s) {
  if (g.V / 2 > 65535) return hipErrorInvalidValue;
  const long rowlen = (long)nb * nrhs;
  const dim3 grid((unsigned)((rowlen + 255) / 256), (unsigned)(g.V / 2));
  hipLaunchKernelGGL(cb_rows_kernel, grid, dim3(256), 0, s, g, parity, rowlen, static_cast<const float2*>(src),
                     static_cast<float2*>(dst), scatter_add);
  return hipGetLastError();
}

// Inverse of every Nb x Nb self block (FP64 Gauss-Jordan with partial
// pivoting, one workgroup per site, [M | 1] in LDS).  B64 is the stencil
// master [site][9][Nb][Nb]; out [site][Nb][Nb]; a vanishing pivot sets *flag.
__global__ __launch_bounds__(256) void self_invert_kernel(const double2* __restrict__ B64,
                                                          double2* __restrict__ out, int* __restrict__ flag) {
  __shared__ double2 M[kNb][2 * kNb];
  __shared__ int piv;
  const int site = blockIdx.x;
  const double2* b = B64 + (size_t)site * 9 * kNb * kNb;  // direction 0
  for (int e = threadIdx.x; e < kNb * 2 * kNb; e += 256) {
    const int r = e / (2 * kNb), c = e % (2 * kNb);
    M[r][c] = c < kNb ? b[r * kNb + c] : make_double2(c - kNb == r ? 1.0 : 0.0, 0.0);
  }
  __syncthreads();
  for (int k = 0; k < kNb; ++k) {
    if (threadIdx.x == 0) {
      int p = k;
      double best = -1.0;
      for (int r = k; r < kNb; ++r) {
        const double m = M[r][k].x * M[r][k].x + M[r][k].y * M[r][k].y;
        if (m > best) {
          best = m;
          p = r;
        }
      }
      piv = best > 0.0 ? p : -1;
    }
    __syncthreads();
    const int p = piv;
    if (p < 0) {
      if (threadIdx.x == 0) atomicOr(flag, 1);
      return;  // uniform across the workgroup
    }
    if (p != k && threadIdx.x < 2 * kNb) {
      const double2 t = M[k][threadIdx.x];
      M[k][threadIdx.x] = M[p][threadIdx.x];
      M[p][threadIdx.x] = t;
    }
    __syncthreads();
    const double2 a = M[k][k];
    const double n2 = a.x * a.x + a.y * a.y;
    const double2 ia = make_double2(a.x / n2, -a.y / n2);
    __syncthreads();
    if (threadIdx.x < 2 * kNb) {
      const double2 v = M[k][threadIdx.x];
      M[k][threadIdx.x] = make_double2(v.x * ia.x - v.y * ia.y, v.x * ia.y + v.y * ia.x);
    }
    __syncthreads();
    for (int e = threadIdx.x; e < kNb * 2 * kNb; e += 256) {
      const int r = e / (2 * kNb), c = e % (2 * kNb);
      if (r == k) continue;
      const double2 f = M[r][k], v = M[k][c];
      // M[r][k] itself is read by every column of row r: update it last
      if (c == k) continue;
      M[r][c] = make_double2(M[r][c].x - (f.x * v.x - f.y * v.y), M[r][c].y - (f.x * v.y + f.y * v.x));
    }
    __syncthreads();
    if (threadIdx.x < kNb && threadIdx.x != k) M[threadIdx.x][k] = make_double2(0.0, 0.0);
    __syncthreads();
  }
  double2* o = out + (size_t)site * kNb * kNb;
  for (int e = threadIdx.x; e < kNb * kNb; e += 256) o[e] = M[e / kNb][kNb + e % kNb];
}

hipError_t launch_self_invert(long nsite, const void* B64, void* out, int* flag, hipStream_t s) {
  hipLaunchKernelGGL(self_invert_kernel, dim3((unsigned)nsite), dim3(256), 0, s, static_cast<const double2*>(B64),
                     static_cast<double2*>(out), flag);
  return hipGetLastError();
}

// Packs nblk FP64 Nb x Nb blocks into the BF16 / FP16 (f16) or FP32 operand orders.
hipError_t launch_pack_block_list(int kind, const void* B64, void* packed, long nblk, hipStream_t s) {
  const long n = nblk * kNb * kNb;
  const int blocks = (int)((n + 255) / 256);
  if (kind == 0)
    hipLaunchKernelGGL(pack_f32_kernel, dim3(blocks), dim3(256), 0, s, static_cast<const double2*>(B64),
                       static_cast<float*>(packed), nblk);
  else if (kind == 2)
    hipLaunchKernelGGL((pack_kernel<true>), dim3(blocks), dim3(256), 0, s, static_cast<const double2*>(B64),
                       static_cast<unsigned short*>(packed), nblk);
  else
    hipLaunchKernelGGL((pack_kernel<false>), dim3(blocks), dim3(256), 0, s, static_cast<const double2*>(B64),
                       static_cast<unsigned short*>(packed), nblk);
  return hipGetLastError();
}

hipError_t launch_coarse_mfma_f32(const Geom& g, int nb, int nrhs, const void* packed, const void* in, void* out,
                                  hipStream_t s) {
  if (nb != kNb) return hipErrorInvalidValue;
  const int blocks = (int)((long)g.V * ((nrhs + 31) / 32));  // one workgroup per (site, 32-column tile)
  const int grid = ((blocks + 7) / 8) * 8;
  hipLaunchKernelGGL((coarse_mfma_f32_kernel<0>), dim3(grid), dim3(256), 0, s, g, nrhs,
                     static_cast<const float4*>(packed), static_cast<const float2*>(in), static_cast<float2*>(out),
                     blocks, 0, 9);
  return hipGetLastError();
}

// Packs both low-precision copies of a level's blocks from the FP64 master.
mrhs_status pack_blocks_mfma(mrhs_mg mg, int level) {
  LevelData& L = mg->lv[level];
  if (!mfma_supported(L.ncomp)) return MRHS_OK;
  mrhs_ctx ctx = mg->ctx;
  const size_t bytes = mfma_pack_bytes(L.g.V);
  mrhs_status st = ensure(ctx, L.Bbf16, bytes);
  if (st != MRHS_OK) return st;
  st = ensure(ctx, L.Bf16, bytes);
  if (st != MRHS_OK) return st;
  st = ensure(ctx, L.Bf32p, 2 * bytes);
  if (st != MRHS_OK) return st;
  MRHS_HIP(ctx, launch_pack_blocks(0, L.B64.p, L.Bbf16.p, L.g.V, ctx->stream));
  MRHS_HIP(ctx, launch_pack_blocks(1, L.B64.p, L.Bf16.p, L.g.V, ctx->stream));
  const long n = (long)L.g.V * 9 * kNb * kNb;
  hipLaunchKernelGGL(pack_f32_kernel, dim3((int)((n + 255) / 256)), dim3(256), 0, ctx->stream,
                     static_cast<const double2*>(L.B64.p), static_cast<float*>(L.Bf32p.p), (long)L.g.V * 9);
  MRHS_HIP(ctx, hipGetLastError());
  return MRHS_OK;
}

}  // namespace mrhs
