// Uniform THC (Alg. 1): min/max ranges and uniform stochastic quantization.
#pragma once

#include "thc_inverse.hpp"

namespace thc {

// ---------------------------------------------------------------------------------------------
// Uniform THC (Alg. 1).  Preliminary stage: every worker's minimum and maximum per block, then the
// global ones.  Main stage: uniform stochastic quantization = the same quantizer with the identity
// table, on the gradients themselves or (ablation of App. C) on their RHT.
// Partial minima / maxima: one per min(B, 8192) coordinates per worker, like the partial sums of squares.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ float wave_min(float v) {
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) v = __builtin_fminf(v, __shfl_xor(v, m, 64));
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) v = __builtin_fmaxf(v, __shfl_xor(v, m, 64));
  return v;
}

struct MinMaxArgs {
  PtrArr grads;
  PtrArr efs;
  float* pmin;       // n * (d >> L1)
  float* pmax;
  uint64_t d;
  uint32_t L1;       // log2 of min(B, 8192)
};

// LOAD: how the vectors are read, see stream_minmax.
template <bool BF16, bool EF, Mem LOAD>
__global__ __launch_bounds__(NT) void k_minmax(const MinMaxArgs a) {
  __shared__ float smin[32], smax[32];   // one per 256 consecutive coordinates of the tile
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
  const uint32_t worker = blockIdx.y;
  const uint64_t off = (uint64_t)xcd_tile(blockIdx.x, gridDim.x) << LOG_TILE;
  const float* ef = EF ? static_cast<const float*>(a.efs.p[worker]) : nullptr;
  // past the end: read from the tile's start, not used
  auto at = [&](int i) { const uint64_t j = off + 4u * (uint32_t)(i * NT + t); return j < a.d ? j : off; };
  float4 x[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (!EF) x[i] = load_grad4<BF16, LOAD>(a.grads.p[worker], at(i));
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if constexpr (EF) {                    // twice the loads: all of them at once are slower (bf16 by 4 %)
      x[i] = load_grad4<BF16, LOAD>(a.grads.p[worker], at(i));
      const float4 e = load_f4<LOAD>(ef + at(i));
      x[i].x += e.x; x[i].y += e.y; x[i].z += e.z; x[i].w += e.w;
    }
    float mn = __builtin_inff(), mx = -__builtin_inff();
    if (off + 4u * (uint32_t)(i * NT + t) < a.d) {
      mn = __builtin_fminf(__builtin_fminf(x[i].x, x[i].y), __builtin_fminf(x[i].z, x[i].w));
      mx = __builtin_fmaxf(__builtin_fmaxf(x[i].x, x[i].y), __builtin_fmaxf(x[i].z, x[i].w));
    }
    mn = wave_min(mn);
    mx = wave_max(mx);
    if (lane == 0) { smin[i * 8 + wave] = mn; smax[i * 8 + wave] = mx; }
  }
  __syncthreads();
  const int nblk = TILE >> a.L1, cpb = 32 / nblk;   // chunks of 256 per block inside the tile
  if (t < nblk) {
    float mn = __builtin_inff(), mx = -__builtin_inff();
    for (int c = 0; c < cpb; ++c) {
      mn = __builtin_fminf(mn, smin[t * cpb + c]);
      mx = __builtin_fmaxf(mx, smax[t * cpb + c]);
    }
    const uint64_t pidx = (off >> a.L1) + t;
    if (pidx < (a.d >> a.L1)) {
      a.pmin[(uint64_t)worker * (a.d >> a.L1) + pidx] = mn;
      a.pmax[(uint64_t)worker * (a.d >> a.L1) + pidx] = mx;
    }
  }
}

struct MinMaxFinalArgs {
  const float* pmin;
  const float* pmax;
  float* range_m;
  float* range_M;
  uint64_t d;
  uint32_t n, L, L1;
};

__global__ __launch_bounds__(64) void k_minmax_final(const MinMaxFinalArgs a) {
  const uint64_t k = blockIdx.x;
  const int lane = threadIdx.x;
  const uint32_t ppb = 1u << (a.L - a.L1);
  const uint64_t per_worker = a.d >> a.L1;
  float mn = __builtin_inff(), mx = -__builtin_inff();
  for (uint32_t i = 0; i < a.n; ++i) {
    const uint64_t base = (uint64_t)i * per_worker + k * ppb;
    for (uint32_t j = lane; j < ppb; j += 64) {
      mn = __builtin_fminf(mn, a.pmin[base + j]);
      mx = __builtin_fmaxf(mx, a.pmax[base + j]);
    }
  }
  mn = wave_min(mn);
  mx = wave_max(mx);
  if (lane == 0) { a.range_m[k] = mn; a.range_M[k] = mx; }
}

// Minimum and maximum of the rotated vectors: the last strided pass of the forward RHT, its results compared and
// dropped.  The quantizer goes through that pass again (k_fwd_hi_quant): writing the rotated vector and reading it back
// would cost twice the bytes of reading the half-rotated one a second time.
struct HiMinMaxArgs {
  const float* x;    // half-rotated vectors, d floats per worker of the launch (grid.y)
  float* pmin;       // partial minima, one per tile or smaller block: d >> min(L, 13) floats per worker
  float* pmax;
  uint64_t d;
  Walk walk;
  TileMap tm;
  uint32_t L;
  float c;
};
static_assert(sizeof(HiMinMaxArgs) <= 128, "a third cache line of arguments takes a small launch 0.2 us");

// LOAD: how they are read, see stream_rotated.
template <int R, Mem LOAD>
__global__ __launch_bounds__(NT) void k_fwd_hi_minmax(const HiMinMaxArgs a) {
  __shared__ __align__(16) float lds[R < 2 ? 4 : TILE];
  __shared__ float smin[16], smax[16];
  const uint32_t tile = walk_x(a.walk), vec = walk_y(a.walk);
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
  const HiGeom<R> g(tile, a.tm);
  const float* const x = a.x + (uint64_t)vec * a.d;
  const uint64_t part = (uint64_t)vec * (a.d >> (a.L < LOG_TILE ? a.L : LOG_TILE));
  float* const pmin = a.pmin + part;
  float* const pmax = a.pmax + part;
  if constexpr (R >= 2) {
    hi_front<R, LOAD>(x, g, lds, t);
    int idx[2];
    float v[2][8];
    hi_back<R>(lds, t, idx, v);
    float mn = __builtin_inff(), mx = -__builtin_inff();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        v[h][e] *= a.c;
        mn = __builtin_fminf(mn, v[h][e]);
        mx = __builtin_fmaxf(mx, v[h][e]);
      }
    }
    mn = wave_min(mn);
    mx = wave_max(mx);
    if (lane == 0) { smin[wave] = mn; smax[wave] = mx; }
    __syncthreads();
    if (t == 0) {   // the whole tile lies in one block: one partial per tile
      for (int w = 1; w < 8; ++w) { mn = __builtin_fminf(mn, smin[w]); mx = __builtin_fmaxf(mx, smax[w]); }
      pmin[tile] = mn;
      pmax[tile] = mx;
    }
  } else {
    float4 r[2][2];
    float v[2][8];
    hi_direct_load<R>(x, g, a.d, t, r);
    hi_direct_stages<R>(r, v);
    // thread owns tile indices [8(t + 512h), +8): a wave covers 512 consecutive values per h
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int idx = 8 * (t + NT * h);
      const uint64_t j = g.coord(idx);
      float mn = __builtin_inff(), mx = -__builtin_inff();
      if (j < a.d) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float q = v[h][e] * a.c;
          mn = __builtin_fminf(mn, q);
          mx = __builtin_fmaxf(mx, q);
        }
      }
      mn = wave_min(mn);
      mx = wave_max(mx);
      if (lane == 0) { smin[h * 8 + wave] = mn; smax[h * 8 + wave] = mx; }
    }
    __syncthreads();
    // blocks inside the tile (B < 8192) or the single one (then R rows of one block share the tile)
    const uint32_t L1 = a.L < LOG_TILE ? a.L : LOG_TILE;
    const int nblk = TILE >> L1, cpb = 16 / nblk;    // chunks of 512 per block inside the tile
    if (t < nblk) {
      float mn = __builtin_inff(), mx = -__builtin_inff();
      for (int c = 0; c < cpb; ++c) {
        mn = __builtin_fminf(mn, smin[t * cpb + c]);
        mx = __builtin_fmaxf(mx, smax[t * cpb + c]);
      }
      const uint64_t pidx = ((uint64_t)tile << (LOG_TILE - L1)) + t;
      if (pidx < (a.d >> L1)) { pmin[pidx] = mn; pmax[pidx] = mx; }
    }
  }
}

// Uniform stochastic quantization of one worker's vector: 4096 or 8192 consecutive coordinates per workgroup.
// Without rotation only, so that the error-feedback update e <- x - (m + z (M-m)/g) is done here.
struct UQuantArgs {
  const void* grad;
  float* ef;               // error feedback, read and written, or null
  const float* range_M;
  const float* range_m;
  uint8_t* packed;
  uint64_t d;
  uint32_t L, b, g;
  uint32_t round, worker, k0, k1;
  uint64_t j0;             // global coordinate of the first element
  uint32_t lut[256];
};

constexpr int LOG_UTILE = 12;   // coordinates of a workgroup, a group to a thread

// What bounds it: bytes (12.5 a coordinate with error feedback) and, in small calls, latency.  With one group of eight
// coordinates to a thread (G = 1) the workgroup asks for all it needs at once, the grid-cell table first, and prepares range
// and table while that travels; it fits 64 registers, hence four workgroups a compute unit.  With two groups (G = 2) tables
// serve twice as many coordinates, and the groups go one after the other (both requested at once spill 10 registers: 924
// us for eight vectors of 25 * 2^20 with error feedback, which take 61 us each, 5.3 TB/s).  Which call takes which:
// uniform_one_group.
template <bool BF16, bool EF, int G>
__global__ __launch_bounds__(NT, G == 1 ? 8 : 1) void k_uniform_quant(const UQuantArgs a) {
  constexpr int LOG = LOG_UTILE + G - 1, T = 1 << LOG;
  __shared__ uint4 lut[256];
  __shared__ QuantScalars sQ[T >> 10];
  __shared__ int sCare[T >> 10];
  __shared__ float sStep[T >> 10];
  const int t = threadIdx.x;
  const uint64_t off = (uint64_t)xcd_tile<5 - G>(blockIdx.x, gridDim.x) << LOG;
  float4 x[2], e[2];
  auto load = [&](uint64_t at) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      x[k] = load_grad4<BF16>(a.grad, at + 4 * k);
      if constexpr (EF) e[k] = *reinterpret_cast<const float4*>(a.ef + at + 4 * k);
    }
  };
  const uint64_t j = off + 8 * t, from = j < a.d ? j : off;   // past the end: read from the tile's own start, not used
  const uint32_t ent = a.lut[t & 255];
  if constexpr (G == 1) {
    __builtin_amdgcn_sched_barrier(0);
    load(from);
    __builtin_amdgcn_sched_barrier(0);
  }
  if (t < 256) lut[t] = quant_lut_entry(ent);
  const int nblk = a.L < LOG ? (T >> a.L) : 1;
  if (t < nblk) {
    const uint64_t blk = (off >> a.L) + t;
    float M = 0.f, m = 0.f;
    if (blk < (a.d >> a.L)) { M = a.range_M[blk]; m = lower_of(a.range_m, blk, M); }
    bool careful;
    sQ[t] = quant_scalars(M, m, a.g, a.lut[a.g - 1], 1.0f, false, careful);
    sCare[t] = careful;
    sStep[t] = (float)(((double)M - (double)m) / (double)a.g);
  }
  __syncthreads();
  auto group = [&](int idx, uint64_t j) {
    float hv[8];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      if constexpr (EF) { x[k].x += e[k].x; x[k].y += e[k].y; x[k].z += e[k].z; x[k].w += e[k].w; }
      hv[4 * k] = x[k].x; hv[4 * k + 1] = x[k].y; hv[4 * k + 2] = x[k].z; hv[4 * k + 3] = x[k].w;
    }
    const int bt = a.L < LOG ? (idx >> a.L) : 0;
    const QuantScalars s = sQ[bt];
    const uint64_t q = (a.j0 + j) >> 3;
    const uint4 rnd = philox4x32_10((uint32_t)q, (uint32_t)(q >> 32), a.round, a.worker, a.k0, a.k1);
    uint32_t z[8];
    if (!sCare[bt]) quantize8<false>(hv, rnd, s, lut, z);   // no scaling: the values are final (c = 1)
    else quantize8<false, true>(hv, rnd, s, lut, z);
    store_packed8(a.packed, j, a.b, z);
    if constexpr (EF) {
      const float step = sStep[bt], lo = s.lo;
      float r[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) r[k] = hv[k] - ((float)z[k] * step + lo);   // identity table: T[z] = z
      *reinterpret_cast<float4*>(a.ef + j) = make_float4(r[0], r[1], r[2], r[3]);
      *reinterpret_cast<float4*>(a.ef + j + 4) = make_float4(r[4], r[5], r[6], r[7]);
    }
  };
  if constexpr (G == 1) {
    if (j >= a.d) return;
    group(8 * t, j);
  } else {
#pragma unroll
    for (int h = 0; h < G; ++h) {
      const int idx = 8 * (t + NT * h);
      if (off + idx >= a.d) continue;
      load(off + idx);
      group(idx, off + idx);
    }
  }
}

// Alg. 1's estimate without rotation: out = m + X (M-m)/(g n), sixteen coordinates per thread.
struct UDequantArgs {
  const void* agg;
  const float* range_M;
  const float* range_m;
  float* out;
  uint64_t d;
  uint32_t L, agg_bits, divisor;
};

template <Mem OUT>
__global__ __launch_bounds__(256) void k_uniform_dequant(const UDequantArgs a) {
  if (a.agg_bits == 8 || a.agg_bits == 16) {
    // byte-aligned sums: four coordinates per thread and step, so that a wave writes 1 KB at a time
    const uint64_t base = (uint64_t)blockIdx.x * 4096;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint64_t j = base + 1024u * k + 4u * threadIdx.x;
      if (j >= a.d) return;
      uint32_t y[4];
      if (a.agg_bits == 8) {
        const uint32_t c = *reinterpret_cast<const uint32_t*>(static_cast<const uint8_t*>(a.agg) + j);
        y[0] = c & 255u; y[1] = (c >> 8) & 255u; y[2] = (c >> 16) & 255u; y[3] = c >> 24;
      } else {
        const uint2 c = *reinterpret_cast<const uint2*>(static_cast<const uint8_t*>(a.agg) + 2 * j);
        y[0] = c.x & 0xFFFFu; y[1] = c.x >> 16; y[2] = c.y & 0xFFFFu; y[3] = c.y >> 16;
      }
      const uint64_t blk = j >> a.L;
      const float M = a.range_M[blk], m = lower_of(a.range_m, blk, M);
      const float step = (float)(((double)M - (double)m) / (double)a.divisor);
      store_f4<OUT>(a.out + j, make_float4((float)y[0] * step + m, (float)y[1] * step + m, (float)y[2] * step + m,
                                           (float)y[3] * step + m));
    }
    return;
  }
  const uint64_t j = ((uint64_t)blockIdx.x * 256 + threadIdx.x) * 16;
  if (j >= a.d) return;
  uint32_t w[8] = {0, 0, 0, 0, 0, 0, 0, 0}, y[16];
  codes_load(static_cast<const uint8_t*>(a.agg), a.agg_bits, j, w, y);
  codes_decode(a.agg_bits, true, w, y);
  const uint64_t blk = j >> a.L;
  const float M = a.range_M[blk], m = lower_of(a.range_m, blk, M);
  const float step = (float)(((double)M - (double)m) / (double)a.divisor);
  float v[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) v[e] = (float)y[e] * step + m;
#pragma unroll
  for (int e = 0; e < 16; e += 4)
    *reinterpret_cast<float4*>(a.out + j + e) = make_float4(v[e], v[e + 1], v[e + 2], v[e + 3]);
}

}  // namespace thc
