// Forward transform passes, the range kernel and the quantizer (worker side of Alg. 3).
#pragma once

#include "thc_device.hpp"
#include "thc_quant.hpp"

namespace thc {

// ---------------------------------------------------------------------------------------------
// Forward "lo" pass (Alg. 3: x = grad + e; ||x||; first part of R = RHT(x) with the diagonal D^r).
// grid = (tiles, n workers).  Writes the half-rotated tile to ws_x[worker] and one partial sum of
// squares per min(B, 8192) coordinates.
// ---------------------------------------------------------------------------------------------
struct FwdLoArgs {
  PtrArr grads;
  PtrArr efs;          // unused without error feedback
  float* ws_x;         // n * d floats
  double* partials;    // per worker `pstride` doubles, one per min(B, 8192) coordinates; or null: no norms wanted
  uint64_t pstride;
  uint64_t d;
  uint64_t j0;         // global coordinate of the vectors' first element (a multiple of B): indexes the diagonal
  uint32_t round, k0, k1;
  TileMap tm;          // where the bits of the tile index land; the tile shape is a template parameter
};

// Tile index -> offset inside the tile's span for the "lo" passes.  XO = false: 8192 consecutive
// coordinates.  XO = true: eight rows of 1024 consecutive coordinates, rows at offset bits 13..15 (the
// workgroup's XCD then stays on one value of offset bits 10..12 for reads and writes alike).
template <bool XO>
__device__ __forceinline__ uint32_t lo_map(uint32_t idx) {
  return XO ? ((idx & 1023u) | ((idx >> 10) << 13)) : idx;
}

template <bool BF16, Mem M = KEEP>
__device__ __forceinline__ float4 load_grad4(const void* g, uint64_t j) {
  if constexpr (BF16) {
    const Vec4<uint16_t>* const p = reinterpret_cast<const Vec4<uint16_t>*>(static_cast<const uint16_t*>(g) + j);
    const Vec4<uint16_t> h = M == STREAM ? __builtin_nontemporal_load(p) : *p;
    return make_float4(bf16_to_f32(h.x), bf16_to_f32(h.y), bf16_to_f32(h.z), bf16_to_f32(h.w));
  } else {
    return load_f4<M>(static_cast<const float*>(g) + j);
  }
}

// sum of squares in binary64 (a binary32 square is exact there)
__device__ __forceinline__ double sum_squares4(const float4 x) {
  const double p = (double)x.x, q = (double)x.y, r = (double)x.z, s = (double)x.w;
  return __builtin_fma(s, s, __builtin_fma(r, r, __builtin_fma(q, q, p * p)));
}

struct alignas(16) SmemLo {
  float lds[TILE_PAD];
  uint32_t sgn[TILE / 32];
  double wsum[4][NT / 64];
};

// One tile of the pass: tile index `tile` of vector `worker`; `dst` is where coordinate 0 of that vector's
// half-rotated image lives (the tile's results go to dst[offset in the vector]).  LOAD: how the vectors are read (stream_inputs,
// stream_norms), STORE: how the results are written (plain_first_pass); chosen by the launch, since a choice in the kernel took small
// calls with error feedback 2 to 4 % (13.0 us).
template <int L1, bool BF16, bool EF, bool XO, bool NORM_ONLY, Mem LOAD, Mem STORE, class A>
__device__ __forceinline__ void fwd_lo_tile(const A& a, uint32_t tile, uint32_t worker, float* dst_vec,
                                            SmemLo& sm) {
  static_assert(!XO || L1 == LOG_TILE, "the row-split tile needs blocks of at least 2^16");
  // Vectors are multiples of B, so only blocks shorter than a tile can leave the last tile partial.
  constexpr bool GUARD = L1 < LOG_TILE;
  float* const lds = sm.lds;
  uint32_t* const sgn = sm.sgn;
  double (*const wsum)[NT / 64] = sm.wsum;

  const int t = threadIdx.x;
  const void* grad = a.grads.p[worker];
  const float* ef = EF ? static_cast<const float*>(a.efs.p[worker]) : nullptr;
  const int wave = t >> 6, lane = t & 63;
  const uint64_t off = tm_base(a.tm, tile);   // coordinate of tile index 0

  // all loads of the tile are issued before anything waits on them
  float4 x[4], e[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint64_t j = off + lo_map<XO>(4u * (uint32_t)(i * NT + t));
    const bool ok = !GUARD || j < a.d;
    x[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    e[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (ok) {
      x[i] = load_grad4<BF16, LOAD>(grad, j);
      if constexpr (EF) e[i] = load_f4<LOAD>(ef + j);
    }
  }

  if (!NORM_ONLY && t < 64) {   // the tile's 8192 diagonal entries: 64 Philox calls of 128 bits
    const uint64_t q = (a.j0 + off + lo_map<XO>(128u * t)) >> 7;
    const uint4 r = philox4x32_10((uint32_t)q, (uint32_t)(q >> 32), a.round, SIGN_STREAM, a.k0, a.k1);
    *reinterpret_cast<uint4*>(&sgn[4 * t]) = r;
  }
  if constexpr (EF) {
#pragma unroll
    for (int i = 0; i < 4; ++i) { x[i].x += e[i].x; x[i].y += e[i].y; x[i].z += e[i].z; x[i].w += e[i].w; }
  }
  double acc[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) acc[i] = sum_squares4(x[i]);
  // a thread's four float4 sit 2048 coordinates apart: they share a block only if the block is that large
  if constexpr (L1 >= 13) {
    const double s = wave_sum((acc[0] + acc[1]) + (acc[2] + acc[3]));
    if (lane == 0) wsum[0][wave] = s;
  } else if constexpr (L1 == 12) {
    const double s0 = wave_sum(acc[0] + acc[1]), s1 = wave_sum(acc[2] + acc[3]);
    if (lane == 0) { wsum[0][wave] = s0; wsum[1][wave] = s1; }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const double s = wave_sum(acc[i]);
      if (lane == 0) wsum[i][wave] = s;
    }
  }
  __syncthreads();   // diagonal bits and wave sums visible

  // partial sums: one per block of 2^L1 coordinates inside the tile, combined in a fixed order
  constexpr int NBLK = TILE >> L1;
  if (t < NBLK) {
    double s = 0.0;
    if constexpr (L1 >= 13) {
#pragma unroll
      for (int w = 0; w < 8; ++w) s += wsum[0][w];
    } else if constexpr (L1 == 12 || L1 == 11) {
#pragma unroll
      for (int w = 0; w < 8; ++w) s += wsum[t][w];
    } else {   // L1 == 10: block = 2 * i + (wave >> 2)
#pragma unroll
      for (int w = 0; w < 4; ++w) s += wsum[t >> 1][4 * (t & 1) + w];
    }
    // one partial per tile (all of it in one block) or, for blocks below 8192, per block of the linear tile
    // the row-split tile is not contiguous: its number stands in (the same block either way); a contiguous tile
    // is numbered by where it lies
    const uint64_t pidx = XO ? (uint64_t)tile : (off >> L1) + t;
    if (a.partials && pidx < (a.d >> L1)) a.partials[(uint64_t)worker * a.pstride + pidx] = s;
  }
  if constexpr (NORM_ONLY) return;

  // diagonal, strides 1 and 2, then into LDS
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int idx = 4 * (i * NT + t);
    const uint32_t bits = sgn[idx >> 5] >> (idx & 31);
    x[i].x = flip(x[i].x, bits & 1u);
    x[i].y = flip(x[i].y, (bits >> 1) & 1u);
    x[i].z = flip(x[i].z, (bits >> 2) & 1u);
    x[i].w = flip(x[i].w, (bits >> 3) & 1u);
    bfly_f4(x[i]);
    *reinterpret_cast<float4*>(&lds[phys<PAD>(idx)]) = x[i];
  }

  float* dst = dst_vec + off;
  const uint64_t left = a.d - off;   // coordinates of this tile that exist (tail tile of a short vector)
  lds_stages<2, L1, true, PAD>(lds, t, [&](int base, int eoff, float v) {
    if (!GUARD || (uint64_t)(base + eoff) < left) store_f<STORE>(&dst[lo_map<XO>(base) + lo_map<XO>(eoff)], v);
  });
}

// What bounds it: bytes.  Stored through the L2, read non-temporally (see Mem, stream_inputs) and in groups of 2^27 coordinates it
// moves 7.0 TB/s between the L2s and memory (9 blocks of 2^20 x 16 vectors, 1.2 GB, 171 us), 6.1 with plain accesses in groups of 2^29.
// One workgroup per tile (grid = (tiles, n workers)): measured on MI355X this streams faster than a
// persistent grid with software prefetch, the hardware dispatcher keeps four workgroups per CU in flight.
// NORM_ONLY: stop after the partial sums of squares (the norm exchange of Alg. 3 on its own): same sums, same order.
template <int L1, bool BF16, bool EF, bool XO, bool NORM_ONLY, Mem LOAD, Mem STORE>
__global__ __launch_bounds__(NT) void k_fwd_lo(const FwdLoArgs a) {
  __shared__ SmemLo sm;
  fwd_lo_tile<L1, BF16, EF, XO, NORM_ONLY, LOAD, STORE>(a, blockIdx.x, blockIdx.y, a.ws_x + (uint64_t)blockIdx.y * a.d, sm);
}

// ---------------------------------------------------------------------------------------------
// Range (Sec. 5.3; Alg. 3: M = (t_p / sqrt(d)) * max_i ||x_i||, per block).
// ---------------------------------------------------------------------------------------------
struct RangeArgs {
  const double* partials;   // per worker `pstride` doubles
  float* range_M;           // K
  uint64_t pstride;
  uint64_t d;
  uint32_t n, L, L1;
  float t_p;
};

constexpr int RANGE_NT = NT;

__device__ __forceinline__ float range_from_sum(double smax, float t_p, uint32_t L) {
  return (float)(((double)t_p * __builtin_sqrt(smax)) / __builtin_sqrt((double)(1ull << L)));
}

// Blocks of at most 8 tiles (up to 2^16 coordinates): eight lanes per block, each of which adds the block's partial sums of
// every eighth worker in index order; they hold their largest up against each other.
constexpr int RANGE_SMALL_BLOCKS = 256 / 8;      // of a workgroup

__global__ __launch_bounds__(256) void k_range_small(const RangeArgs a) {
  const uint64_t k = (uint64_t)blockIdx.x * RANGE_SMALL_BLOCKS + (threadIdx.x >> 3);
  if (k >= (a.d >> a.L)) return;                 // all eight lanes or none
  const uint32_t ppb = 1u << (a.L - a.L1);
  double smax = 0.0;
  for (uint32_t i = threadIdx.x & 7; i < a.n; i += 8) {
    const double* p = a.partials + (uint64_t)i * a.pstride + k * ppb;
    double s = 0.0;
    for (uint32_t j = 0; j < ppb; ++j) s += p[j];
    smax = s > smax ? s : smax;
  }
#pragma unroll
  for (int m = 1; m < 8; m <<= 1) {
    const double o = __shfl_xor(smax, m, 64);
    smax = o > smax ? o : smax;
  }
  if ((threadIdx.x & 7) == 0) a.range_M[k] = range_from_sum(smax, a.t_p, a.L);
}

template <int TOTALS>     // totals of 64 partial sums a worker may have
struct SmemRange {
  double wsum[MAXW][TOTALS];
};

// largest sum over the lanes that hold one (NaN never wins, as in a loop of comparisons from 0)
__device__ __forceinline__ double wave_largest(double s) {
  double m = s > 0.0 ? s : 0.0;
#pragma unroll
  for (int k = 1; k < 64; k <<= 1) {
    const double o = __shfl_xor(m, k, 64);
    m = o > m ? o : m;
  }
  return m;
}

// The range of one block of at most 8 tiles by one wave, lane i on worker i: the same sums as in k_range_small.  In two
// steps, so that a tile's loads can be requested between them and neither waits for the other.
template <int PPB>
struct SmallRange {
  double p[PPB];
  __device__ __forceinline__ void request(const double* partials, uint64_t pstride, uint32_t n, uint64_t k) {
    const uint32_t lane = threadIdx.x & 63;
    const double* const q = partials + (uint64_t)(lane < n ? lane : 0u) * pstride + k * PPB;
#pragma unroll
    for (int j = 0; j < PPB; ++j) p[j] = q[j];
  }
  __device__ __forceinline__ float range(uint32_t n, float t_p, uint32_t L) const {
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < PPB; ++j) s += p[j];
    return range_from_sum(wave_largest((threadIdx.x & 63) < n ? s : 0.0), t_p, L);
  }
};

// Larger blocks: one workgroup of RANGE_NT threads per block k.  Sigma x^2 of every worker in a fixed summation
// order (partial sums strided by RANGE_NT, butterflies over each 64 of them, then those totals in sequence), the maximum
// over workers, and M, returned by the first wave (other threads return 0).  `partials` points at this call's first
// partial sum.  What bounds it is latency, so the (worker, 64 partial sums) pairs are dealt to the eight waves, four
// loads in flight each, and one lane per worker adds the totals up.  meanwhile() runs once in every wave, between the
// first loads and what waits for them.
template <int TOTALS, class Meanwhile>
__device__ __forceinline__ float block_range(const double* partials, uint64_t pstride, uint32_t n, uint32_t ppb,
                                             uint64_t k, float t_p, uint32_t L, SmemRange<TOTALS>& sm,
                                             Meanwhile&& meanwhile) {
  const uint32_t t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const uint32_t lc = ppb >= RANGE_NT ? 3 : ppb >= 256 ? 2 : ppb >= 128 ? 1 : 0;   // log2 of the totals per worker
  const uint32_t items = n << lc;
  uint32_t it = wave;
  do {
    double s[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {      // what does not exist is read from where something does, and not used
      const uint32_t item = it + u * (RANGE_NT / 64), i = item < items ? item : 0u;
      const uint32_t j = 64 * (i & ((1u << lc) - 1u)) + lane;
      s[u] = partials[(uint64_t)(i >> lc) * pstride + k * ppb + (j < ppb ? j : 0u)];
    }
    if (it == wave) meanwhile();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint32_t item = it + u * (RANGE_NT / 64), j = 64 * (item & ((1u << lc) - 1u)) + lane;
      if (item >= items || j >= ppb) s[u] = 0.0;
    }
    // blocks of more than 512 tiles, a power of two of them: up to 28 loads in flight
    for (uint32_t j0 = RANGE_NT; j0 < ppb; j0 += 7 * RANGE_NT) {
      double x[4][7];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t item = it + u * (RANGE_NT / 64), j = 64 * (item & 7u) + lane + j0;
        const double* const p = partials + (uint64_t)(item >> lc) * pstride + k * ppb;
#pragma unroll
        for (uint32_t c = 0; c < 7; ++c) x[u][c] = item < items && j + c * RANGE_NT < ppb ? p[j + c * RANGE_NT] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (uint32_t c = 0; c < 7; ++c) s[u] += x[u][c];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint32_t item = it + u * (RANGE_NT / 64);
      if (item >= items) break;
      s[u] = wave_sum(s[u]);
      if (lane == 0) sm.wsum[item >> lc][item & ((1u << lc) - 1u)] = s[u];
    }
    it += 4 * (RANGE_NT / 64);
  } while (it < items);
  __syncthreads();
  float M = 0.f;
  if (wave == 0) {
    double s = 0.0;
    if (lane < n)
      for (uint32_t w = 0; w < (1u << lc); ++w) s += sm.wsum[lane][w];
    M = range_from_sum(wave_largest(s), t_p, L);
  }
  return M;
}

__global__ __launch_bounds__(RANGE_NT) void k_range(const RangeArgs a) {
  __shared__ SmemRange<RANGE_NT / 64> sm;
  const float M = block_range(a.partials, a.pstride, a.n, 1u << (a.L - a.L1), blockIdx.x, a.t_p, a.L, sm, [] {});
  if (threadIdx.x == 0) a.range_M[blockIdx.x] = M;
}

// ---------------------------------------------------------------------------------------------
// Shared addressing of the strided passes: a tile of 2^R rows by W = 8192 >> R columns (see TileMap).
// ---------------------------------------------------------------------------------------------
template <int R>
struct HiGeom {
  static constexpr int LOGW = LOG_TILE - R;
  static constexpr int W = 1 << LOGW;
  const TileMap& m;
  uint64_t base;   // coordinate of (row 0, col 0)
  __device__ HiGeom(uint32_t tile, const TileMap& m_) : m(m_), base(tm_base(m_, tile)) {}
  // offset of a tile index from `base`: 32 bits are enough (blocks are at most 2^27 coordinates), so device
  // addresses can be formed as uniform 64-bit base + 32-bit per-lane offset
  __device__ uint32_t off(int idx) const { return tm_row(m, (uint32_t)idx >> LOGW) + (uint32_t)(idx & (W - 1)); }
  __device__ uint64_t coord(int idx) const { return base + off(idx); }
};

// Front half of a strided pass with R >= 2 row bits (no bounds checks: such tiles are always whole).
// Each thread loads four rows (4 rho + 0..3) of four consecutive columns, finishes row bits 0 and 1 in
// registers, parks the tile in LDS (row-major, no padding) and runs row bits [2, 2 + NB1) through LDS: one
// round of up to four bits for R <= 7, which leaves NB2 = R - 2 - NB1 (0 or 1) top bits for the caller's
// epilogue; two rounds and nothing left for R = 8 and 9 (rows of 128 and 64 bytes: blocks of 2^21 and 2^22
// coordinates then need no pass in between).
template <int R>
constexpr Mem hi_mem() { return R <= 8 ? STREAM : KEEP; }   // a row of the tile is a whole line; for its last reader

template <int R>
struct HiSplit {
  static constexpr int LOGW = LOG_TILE - R;
  static constexpr int W = 1 << LOGW;
  static constexpr int NB1 = R > 7 ? R - 2 : ((R - 2) < 4 ? (R - 2) : 4);
  static constexpr int NB2 = R - 2 - NB1;
  static_assert(R >= 2 && R <= 9 && NB2 <= 1, "strided pass handles 2..9 row bits");
};

template <int R, Mem M>
__device__ __forceinline__ void hi_issue_loads(const float* src, const HiGeom<R>& g, int t, float4 (&x)[4]) {
  using S = HiSplit<R>;
  const int cg = t & (S::W / 4 - 1), rho = t >> (S::LOGW - 2);
  const float* pb = src + g.base;
  const uint32_t o = tm_row(g.m, 4 * rho) + 4 * cg;
  const uint32_t p1 = tm_row(g.m, 1), p2 = tm_row(g.m, 2);   // rows 4 rho + {1, 2, 3}
  x[0] = load_f4<M>(pb + o);
  x[1] = load_f4<M>(pb + (o + p1));
  x[2] = load_f4<M>(pb + (o + p2));
  x[3] = load_f4<M>(pb + (o + p1 + p2));
}

// row bits 0 and 1 in registers, then the tile goes to LDS (row-major, no padding)
template <int R>
__device__ __forceinline__ void hi_r0_to_lds(float4 (&x)[4], float* lds, int t) {
  using S = HiSplit<R>;
  const int cg = t & (S::W / 4 - 1), rho = t >> (S::LOGW - 2);
  bf4(x[0], x[1]); bf4(x[2], x[3]);   // row bit 0
  bf4(x[0], x[2]); bf4(x[1], x[3]);   // row bit 1
  float* q = lds + (4 * rho) * S::W + 4 * cg;
  *reinterpret_cast<float4*>(q) = x[0];
  *reinterpret_cast<float4*>(q + S::W) = x[1];
  *reinterpret_cast<float4*>(q + 2 * S::W) = x[2];
  *reinterpret_cast<float4*>(q + 3 * S::W) = x[3];
}

// row bits [2, 2 + NB1)  <->  tile index bits [LOGW + 2, LOGW + 2 + NB1); ends with the tile readable
template <int R>
__device__ __forceinline__ void hi_round1(float* lds, int t) {
  using S = HiSplit<R>;
  lds_stages<S::LOGW + 2, S::LOGW + 2 + S::NB1, false, PLAIN>(lds, t, [](int, int, float) {});
  __syncthreads();
}

template <int R, Mem M>
__device__ __forceinline__ void hi_front(const float* src, const HiGeom<R>& g, float* lds, int t) {
  float4 x[4];
  hi_issue_loads<R, M>(src, g, t, x);
  hi_r0_to_lds<R>(x, lds, t);
  hi_round1<R>(lds, t);
}

// Two groups of eight consecutive coordinates per thread, with the last row bit (if any) applied:
// tile index of each group in idx[], values in v[][].
template <int R>
__device__ __forceinline__ void hi_back(const float* lds, int t, int (&idx)[2], float (&v)[2][8]) {
  using S = HiSplit<R>;
  idx[0] = 8 * t;
  idx[1] = 8 * (t + NT);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const float4 p0 = *reinterpret_cast<const float4*>(&lds[idx[h]]);
    const float4 p1 = *reinterpret_cast<const float4*>(&lds[idx[h] + 4]);
    v[h][0] = p0.x; v[h][1] = p0.y; v[h][2] = p0.z; v[h][3] = p0.w;
    v[h][4] = p1.x; v[h][5] = p1.y; v[h][6] = p1.z; v[h][7] = p1.w;
  }
  if constexpr (S::NB2 == 1) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float a = v[0][e], b = v[1][e];
      v[0][e] = a + b;
      v[1][e] = a - b;
    }
  }
}

// The same tile as four groups of four consecutive coordinates, group i at tile index 4 t + 4 NT i: a wave's access takes
// whole lines, where groups of eight take every other 16 bytes.
template <int R>
__device__ __forceinline__ void hi_back4(const float* lds, int t, float4 (&v)[4]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = *reinterpret_cast<const float4*>(&lds[4 * (t + NT * i)]);
  if constexpr (HiSplit<R>::NB2 == 1) { bf4(v[0], v[2]); bf4(v[1], v[3]); }
}

// R < 2: a thread's two groups of eight consecutive values (the two rows of the same columns where there are two) come
// straight from memory.  Coordinates past the vector's end belong to blocks of their own, whose results nobody takes:
// what is read for them does not matter, and loads that are requested in any case need not be waited for where an
// earlier one is wanted.
template <int R>
__device__ __forceinline__ void hi_direct_load(const float* src, const HiGeom<R>& g, uint64_t d, int t,
                                               float4 (&x)[2][2]) {
  static_assert(R < 2, "more rows go through LDS");
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint64_t j = g.coord(8 * (t + NT * h));
    const float4* const p = reinterpret_cast<const float4*>(src + (j < d ? j : 0));
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const float4 r = p[k];
      x[h][k] = make_float4(r.x, r.y, r.z, r.w);
    }
  }
}

template <int R>
__device__ __forceinline__ void hi_direct_stages(const float4 (&x)[2][2], float (&v)[2][8]) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      v[h][4 * k] = x[h][k].x; v[h][4 * k + 1] = x[h][k].y; v[h][4 * k + 2] = x[h][k].z; v[h][4 * k + 3] = x[h][k].w;
    }
  }
  if constexpr (R == 1) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float a = v[0][e], b = v[1][e];
      v[0][e] = a + b;
      v[1][e] = a - b;
    }
  }
}

// ---------------------------------------------------------------------------------------------
// "mid" pass: R more bits, in place.
// ---------------------------------------------------------------------------------------------
struct MidArgs {
  float* x;   // d floats per worker of the launch (grid.y = worker): half-rotated vectors
  uint64_t d;
  TileMap tm;
};

template <int R>
__global__ __launch_bounds__(NT) void k_mid(MidArgs a) {
  __shared__ __align__(16) float lds[TILE];
  const int t = threadIdx.x;
  const HiGeom<R> g(blockIdx.x, a.tm);
  a.x += (uint64_t)blockIdx.y * a.d;
  hi_front<R, KEEP>(a.x, g, lds, t);
  float4 v[4];
  hi_back4<R>(lds, t, v);
#pragma unroll
  for (int i = 0; i < 4; ++i) *reinterpret_cast<float4*>(a.x + g.coord(4 * (t + NT * i))) = v[i];
}

// ---------------------------------------------------------------------------------------------
// Forward "hi" pass + main stage, worker side (Alg. 3: R = RHT(x) finished; clamp to [-M, M];
// stochastic quantization onto the table's values (Sec. 4.1); Z = T^-1[Y] (Alg. 2); bit-pack).
//
// Per coordinate, in binary32:  v = h * c;  x' = med(v, m, M);  y = (x' - m) * scale;  k = floor(y);
// (lo, wd, z0) = LUT[k];  t = y - lo;  up iff u * wd < t with u = (half + 1/2) / 2^16;  z = z0 + up.
// Everything is carried scaled by 2^24, which moves exponents only: the cell is then the top byte of the converted
// integer, and the conversion saturates, so the clamp itself costs nothing (see quantize8).  When 1/sqrt(B) is a power
// of two (even log2 B) the multiplication by c is folded into m and the scale: again only exponents move.
// ---------------------------------------------------------------------------------------------
struct QuantArgs {
  const float* x;          // half-rotated vectors, d floats per worker of the launch (grid.y = worker)
  const float* range_M;    // K floats
  const float* range_m;    // K floats, or null: m = -M
  PtrArr packed;           // per worker of the launch: d*b/8 bytes, written
  uint64_t d;
  uint64_t j0;             // global coordinate of x[0] (a multiple of B): the random streams are indexed globally
  Walk walk;
  TileMap tm;
  uint32_t L;              // log2 B
  uint32_t b, g;
  uint32_t round, worker, k0, k1;   // worker: id of the launch's first worker (selects the rounding stream)
  float c;                 // 1/sqrt(B)
  uint32_t lut[256];       // per grid cell k: lo | wd << 8 | z0 << 16
  // only where the pass finds the range itself (FIND): what k_range would be given, and where M goes
  const double* partials;
  uint64_t pstride;
  float* range_out;
  uint32_t n;
  float t_p;
};

// float -> uint32, towards zero; below 0 gives 0 and above 2^32 - 1 gives 2^32 - 1 (a C++ cast leaves those undefined)
__device__ __forceinline__ uint32_t cvt_u32_sat(float y) {
  uint32_t k;
  asm("v_cvt_u32_f32 %0, %1" : "=v"(k) : "v"(y));
  return k;
}

// CAREFUL = false: no clamp.  Below m the position is negative, converts to cell 0 and never rounds up.  Above M it lies
// in or beyond the last cell: there quant_scalars has made sure that M itself, hence everything above it, ends in the
// top index for every draw.  Saves one of eleven instructions per coordinate, 16 a wave, of which the choice between the
// forms takes twelve back: 442 -> 438 a wave, and 472 -> 471 us for 64 blocks of 2^20 x 8 vectors.
// CAREFUL = true: the operations exactly as listed above, unscaled; for ranges so narrow that the scaled form would
// leave binary32, or grids so fine that a clamped coordinate may round down from the last cell: it takes three roundings
// to place M, which may leave it 3 g 2^-24 of a cell short, and a last cell w wide needs less than w 2^-17 (g up to 42 w
// never takes this form, g = 127 with w = 1 one time in six).
// Both forms take the same decisions: multiplying by a power of two commutes with every rounding involved.
template <bool MULC, bool CAREFUL = false>
__device__ __forceinline__ void quantize8(const float (&hv)[8], const uint4 rnd, const QuantScalars s,
                                          const uint4* lut, uint32_t (&z)[8]) {
  const uint32_t rw[4] = {rnd.x, rnd.y, rnd.z, rnd.w};
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float v = MULC ? hv[e] * s.c : hv[e];
    float y;
    uint4 ent;
    if constexpr (CAREFUL) {
      const float yu = (__builtin_amdgcn_fmed3f(v, s.lo, s.M) - s.lo) * s.sc;
      ent = lut[cvt_u32_sat(yu) & 255u];
      y = (yu - __uint_as_float(ent.x) * (1.0f / GRID_SCALE)) * GRID_SCALE;
    } else {
      y = (v - s.lo) * s.sc;
      ent = lut[cvt_u32_sat(y) >> 24];
      y -= __uint_as_float(ent.x);
    }
    const float hf = (float)((e & 1) ? (rw[e >> 1] >> 16) : (rw[e >> 1] & 0xFFFFu));
    const float prod = __builtin_fmaf(hf, __uint_as_float(ent.y), __uint_as_float(ent.z));
    z[e] = ent.w + (prod < y ? 1u : 0u);
  }
}

// eight B-bit fields, field 0 in the least significant bits
template <int B>
__device__ __forceinline__ uint32_t pack8(const uint32_t (&z)[8]) {
  uint32_t w = z[7];
#pragma unroll
  for (int e = 6; e >= 0; --e) w = (w << B) | z[e];
  return w;
}

// QUAD: aligned groups of four lanes hold 32 consecutive coordinates, all of them or none active.  3-bit indices then
// leave as dwords instead of bytes (the sweep's round of 2^20 coordinates, 10 workers, with k_aggregate_any: 63 to 46 us).
template <bool QUAD = true>
__device__ __forceinline__ void store_packed8(uint8_t* packed, uint64_t j, uint32_t b, const uint32_t (&z)[8]) {
  if (b == 4) {
    *reinterpret_cast<uint32_t*>(packed + (j >> 1)) = pack8<4>(z);
  } else if (b == 2) {
    *reinterpret_cast<uint16_t*>(packed + (j >> 2)) = (uint16_t)pack8<2>(z);
  } else if (b == 8) {
    const uint32_t w0 = z[0] | z[1] << 8 | z[2] << 16 | z[3] << 24;
    const uint32_t w1 = z[4] | z[5] << 8 | z[6] << 16 | z[7] << 24;
    *reinterpret_cast<uint2*>(packed + j) = make_uint2(w0, w1);
  } else if (b == 1) {
    packed[j >> 3] = (uint8_t)pack8<1>(z);
  } else if (QUAD && b == 3) {
    // four lanes hold three dwords: lane q < 3 takes the rest of its own 24 bits and the start of the next lane's
    const uint32_t w = pack8<3>(z), q = threadIdx.x & 3u;
    const uint32_t next = (uint32_t)__builtin_amdgcn_mov_dpp((int)w, 0x39, 0xF, 0xF, true);   // lanes 1, 2, 3, 0
    if (q < 3) *reinterpret_cast<uint32_t*>(packed + (j >> 3) * 3 + q) = w >> (8 * q) | next << (24 - 8 * q);
  } else {
    store_fields8(packed + (j >> 3) * b, z, b);
  }
}

// LDS entry of grid cell k: {lo * 2^24, wd * 2^8, wd * 2^7 (all binary32, exact), z0}; the comparison is
// (half + 1/2) * wd * 2^8 < y - lo * 2^24.  The top value (wd = 255 in the argument) never rounds up.
__device__ __forceinline__ uint4 quant_lut_entry(uint32_t ent) {
  const uint32_t wd = (ent >> 8) & 255u;
  const float w = wd == 255u && (ent & 255u) ? 0.f : (float)wd;
  const float half = wd == 255u && (ent & 255u) ? __builtin_inff() : 0.5f * (float)wd;
  return make_uint4(__float_as_uint((float)(ent & 255u) * GRID_SCALE), __float_as_uint(w * 256.0f),
                    __float_as_uint(half * 256.0f), ent >> 16);
}

__device__ __forceinline__ void build_quant_lut(uint32_t ent, uint4* lut, int t) {
  if (t < 256) lut[t] = quant_lut_entry(ent);
}

__device__ __forceinline__ float lower_of(const float* range_m, uint64_t blk, float M) {
  return range_m ? range_m[blk] : -M;
}

template <int R>
struct alignas(16) SmemQuant {
  float lds[R < 2 ? 4 : TILE];   // one or two rows need no exchange
  uint32_t lut[256][4];   // uint4 entries
  float sQ[8][4];         // QuantScalars
  int sCare[8];           // the block takes the careful form
};

// What FIND keeps of the partial sums: its blocks of up to 2^20 coordinates have at most 128 of them a worker.
using FindSmem = SmemRange<2>;

// One tile of the pass: tile index `tile` of the launch's vector `wk`, whose half-rotated image starts at xw.
// FIND: the range comes from the partial sums of squares, found again by every workgroup (see k_fwd_hi_quant).
// QUAD: see store_packed8; off where its registers would spill.
template <int R, bool CFOLD, bool FIND = false, bool QUAD = false, class A>
__device__ __forceinline__ void hi_quant_tile(const A& a, uint32_t tile, uint32_t wk, const float* xw,
                                              SmemQuant<R>& sm, FindSmem* smr = nullptr) {
  uint4* const lut = reinterpret_cast<uint4*>(sm.lut);
  QuantScalars* const sQ = reinterpret_cast<QuantScalars*>(sm.sQ);
  int* const sCare = sm.sCare;

  const int t = threadIdx.x;
  uint8_t* const packed = static_cast<uint8_t*>(const_cast<void*>(a.packed.p[wk]));
  const uint32_t stream = a.worker + wk;

  // Loads come back in the order of their requests: what the tables and the range need goes first, so that both are made
  // while the tile's own loads travel.
  const uint32_t ent = a.lut[t & 255];
  if constexpr (R >= 2) {
    const HiGeom<R> g(tile, a.tm);
    const uint64_t blk = g.base >> a.L;         // the whole tile lies in one block
    float4 x[4];
    float found = 0.f;
    if constexpr (FIND && R > 3) {
      found = block_range(a.partials, a.pstride, a.n, 1u << R, blk, a.t_p, a.L, *smr, [&] {
        __builtin_amdgcn_sched_barrier(0);
        hi_issue_loads<R, hi_mem<R>()>(xw, g, t, x);
        __builtin_amdgcn_sched_barrier(0);
      });
    } else if constexpr (FIND) {
      SmallRange<1 << R> r;
      if (t < 64) r.request(a.partials, a.pstride, a.n, blk);
      __builtin_amdgcn_sched_barrier(0);
      hi_issue_loads<R, hi_mem<R>()>(xw, g, t, x);
      __builtin_amdgcn_sched_barrier(0);
      if (t < 64) found = r.range(a.n, a.t_p, a.L);
    } else {
      __builtin_amdgcn_sched_barrier(0);
      hi_issue_loads<R, hi_mem<R>()>(xw, g, t, x);
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (FIND) {
      if (t == 0 && wk == 0 && g.base == blk << a.L) a.range_out[blk] = found;
    }
    if (t == 0) {
      const float M = FIND ? found : a.range_M[blk], m = FIND ? -M : lower_of(a.range_m, blk, M);
      bool careful;
      sQ[0] = quant_scalars(M, m, a.g, a.lut[a.g - 1], a.c, CFOLD, careful);
      sCare[0] = careful;
    }
    build_quant_lut(ent, lut, t);
    hi_r0_to_lds<R>(x, sm.lds, t);
    hi_round1<R>(sm.lds, t);
    int idx[2];
    float v[2][8];
    hi_back<R>(sm.lds, t, idx, v);
    const QuantScalars s = sQ[0];
    const bool careful = __builtin_amdgcn_readfirstlane(sCare[0]) != 0;   // uniform over the workgroup
    const uint64_t q0 = (a.j0 + g.base) >> 3;   // tiles start on multiples of 64 coordinates
    uint8_t* const pk0 = packed + (g.base >> 3) * a.b;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t o = g.off(idx[h]);
      const uint64_t q = q0 + (o >> 3);
      const uint4 rnd = philox4x32_10((uint32_t)q, (uint32_t)(q >> 32), a.round, stream, a.k0, a.k1);
      uint32_t z[8];
      if (!careful) quantize8<!CFOLD>(v[h], rnd, s, lut, z);
      else quantize8<true, true>(v[h], rnd, s, lut, z);
      store_packed8<QUAD && HiGeom<R>::W >= 32>(pk0, o, a.b, z);
    }
  } else {
    const HiGeom<R> g(tile, a.tm);
    // per-block scalars; a tile spans more than one block only when B < 8192 (then R == 0)
    const int nblk = a.L < LOG_TILE ? (TILE >> a.L) : 1;
    const int bt0 = FIND ? t >> 6 : t;          // FIND: a wave per block
    const uint64_t blk = (g.base >> a.L) + bt0;
    const bool mine = bt0 < nblk && blk < (a.d >> a.L);
    SmallRange<1 << R> r;                       // blocks of up to 2^13 have one partial sum a worker
    if constexpr (FIND) {
      if (mine) r.request(a.partials, a.pstride, a.n, blk);
    }
    float4 x[2][2];
    __builtin_amdgcn_sched_barrier(0);
    hi_direct_load<R>(xw, g, a.d, t, x);
    __builtin_amdgcn_sched_barrier(0);
    if (bt0 < nblk) {
      float M = 0.f, m = 0.f;
      if (mine) {
        if constexpr (FIND) {
          M = r.range(a.n, a.t_p, a.L);
          m = -M;
          if ((t & 63) == 0 && wk == 0 && (a.L < LOG_TILE || g.base == blk << a.L)) a.range_out[blk] = M;
        } else {
          M = a.range_M[blk];
          m = lower_of(a.range_m, blk, M);
        }
      }
      bool careful;
      const QuantScalars s = quant_scalars(M, m, a.g, a.lut[a.g - 1], a.c, false, careful);
      if (!FIND || (t & 63) == 0) {
        sQ[bt0] = s;
        sCare[bt0] = careful;
      }
    }
    build_quant_lut(ent, lut, t);
    __syncthreads();
    float v[2][8];
    hi_direct_stages<R>(x, v);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int idx = 8 * (t + NT * h);
      const uint64_t j = g.coord(idx);
      if (j >= a.d) continue;
      const int bt = a.L < LOG_TILE ? (idx >> a.L) : 0;
      const QuantScalars s = sQ[bt];
      const uint64_t q = (a.j0 + j) >> 3;
      const uint4 rnd = philox4x32_10((uint32_t)q, (uint32_t)(q >> 32), a.round, stream, a.k0, a.k1);
      uint32_t z[8];
      if (!sCare[bt]) quantize8<true>(v[h], rnd, s, lut, z);
      else quantize8<true, true>(v[h], rnd, s, lut, z);
      store_packed8<QUAD>(packed, j, a.b, z);
    }
  }
}

// FIND: the pass takes the place of the range kernel before it.  In a small call a launch of its own costs more than
// the work: the workgroups of a block all add up the block's partial sums, which the cache holds.  With the partial sums
// requested before the tile, room in LDS for the totals that occur here only and 64 registers, so that four workgroups
// share a compute unit as without it: 17.4 -> 15.4 us for one block of 2^20 x 10 vectors, 5.6 -> 4.9 us for two blocks of
// 2^14 x 4, and 67.1 -> 58.2 us (without FIND 58.3 -> 53.0) for 512 blocks of 2^14 x 8, whose tiles of one or two rows
// no longer go through LDS.
template <int R, bool CFOLD, bool FIND>
__global__ __launch_bounds__(NT, 8) void k_fwd_hi_quant(const QuantArgs a) {
  __shared__ SmemQuant<R> sm;
  // a launch that finds the range is too small to be walked backwards
  const uint32_t tile = FIND ? blockIdx.x : walk_x(a.walk), vec = FIND ? blockIdx.y : walk_y(a.walk);
  const float* const xw = a.x + (uint64_t)vec * a.d;
  if constexpr (FIND) {
    __shared__ FindSmem smr;
    hi_quant_tile<R, CFOLD, true, true>(a, tile, vec, xw, sm, &smr);
  } else {
    hi_quant_tile<R, CFOLD, false, true>(a, tile, vec, xw, sm);
  }
}

}  // namespace thc
