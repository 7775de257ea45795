// Blocks of 2^10 to 2^14 coordinates: the worker side of a round (Alg. 3) in one launch.
//
// What bounds it: bytes and instructions alike.  A block fits one workgroup, so once its range is known nothing of it
// has to leave the compute unit: gradient (and buffer) in, indices (and buffer) out, 4.5 bytes a coordinate in binary32
// instead of the 12.5 of two passes through memory, with error feedback 12.5 instead of 29.  The range needs every
// worker's norm first: from thc_prepare_range, from a pass over the gradients that keeps the sums only (6.6 TB/s), or, in
// small calls without error feedback, from every workgroup adding up its block's squares of all workers itself (FIND).
// Which calls take which way, and what that measures: whole_route.  thc_compress at 2^28 coordinates in blocks of 2^10 / 2^13 /
// 2^14: 609 / 621 / 603 -> 264 / 289 / 308 us, with error feedback 1483 / 1453 / 1446 -> 612 / 682 / 878.
#pragma once

#include "thc_inverse.hpp"

namespace thc {

struct WholeArgs {
  PtrArr grads;
  PtrArr efs;              // error feedback, read and written
  PtrArr packed;
  float* range_M;          // K floats: read, or with FIND written
  uint64_t d;
  uint64_t j0;             // global coordinate of the vectors' first element
  uint32_t L, b, g;
  uint32_t round, worker, k0, k1;
  uint32_t n;              // FIND: vectors of the launch
  float c, t_p;
  uint32_t lut[256];
  uint8_t table[256];
};

template <int L>
struct WholeTile {
  static constexpr int LOG = L < LOG_TILE ? LOG_TILE : L;   // several blocks to a tile below 2^13
  static constexpr int N = 1 << (LOG - 4);                  // threads, 16 values each
  static constexpr int BLOCKS = 1 << (LOG - L);
};

template <int L, bool EF, bool FIND>
struct alignas(16) SmemWhole {
  float lds[padded(1 << WholeTile<L>::LOG)];
  uint32_t lut[256][4];
  uint32_t sgn[1 << (WholeTile<L>::LOG - 5)];
  float tabf[EF ? 256 : 4];
  float sQ[8][4];
  int sCare[8];
  float sLo[8], sStep[8];
  double wsum[FIND ? WHOLE_FIND_WORKERS : 1][FIND ? 32 : 1];
};

// Sums of squares of a thread's four groups of four values, in the order of the first pass: wsum[...] of one worker.
template <int L>
__device__ __forceinline__ void whole_squares(const float4 (&x)[4], double* wsum, int wave, int lane) {
  double acc[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) acc[i] = sum_squares4(x[i]);
  if constexpr (L >= 13) {
    const double s = wave_sum((acc[0] + acc[1]) + (acc[2] + acc[3]));
    if (lane == 0) wsum[wave] = s;
  } else if constexpr (L == 12) {
    const double s0 = wave_sum(acc[0] + acc[1]), s1 = wave_sum(acc[2] + acc[3]);
    if (lane == 0) { wsum[wave] = s0; wsum[8 + wave] = s1; }
  } else {
    const double s = wave_sum4(acc[0], acc[1], acc[2], acc[3]);
    if (lane < 4) wsum[8 * lane + wave] = s;
  }
}

// Sum of squares of block `k` of the tile out of a worker's wsum.
template <int L>
__device__ __forceinline__ double whole_block_sum(const double* wsum, int k) {
  if constexpr (L == 14) {
    double p = 0.0, q = 0.0;
#pragma unroll
    for (int w = 0; w < 8; ++w) { p += wsum[w]; q += wsum[8 + w]; }
    return p + q;
  } else {
    constexpr int W = L == 10 ? 4 : 8;
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < W; ++w) s += wsum[W * k + w];
    return s;
  }
}

// SPLIT: two workgroups to a tile, both of which transform all of it and quantize half (see whole_split).  LOAD: how the gradients
// are read (see stream_blocks).
template <int L, bool BF16, bool EF, bool FIND, bool SPLIT = false, Mem LOAD = KEEP>
__global__ __launch_bounds__(WholeTile<L>::N, FIND || EF ? 4 : 8) void k_whole(const WholeArgs a) {
  static_assert(!SPLIT || FIND, "small calls");
  static_assert(!(EF && FIND), "the buffers would be read by some workgroups while others write them");
  using T = WholeTile<L>;
  constexpr int N = T::N;
  constexpr bool CFOLD = (L & 1) == 0;
  __shared__ SmemWhole<L, EF, FIND> sm;
  float* const lds = sm.lds;
  uint4* const lut = reinterpret_cast<uint4*>(sm.lut);
  QuantScalars* const sQ = reinterpret_cast<QuantScalars*>(sm.sQ);
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
  const uint32_t vec = blockIdx.y;
  const uint32_t part = SPLIT ? blockIdx.x & 1u : 0u, tile = blockIdx.x >> SPLIT;
  const uint64_t off = (uint64_t)xcd_tile<L == 14 ? 2 : 3>(tile, gridDim.x >> SPLIT) << T::LOG;
  // the first pass's share of a thread, tile by tile of 8192
  const int first = (t >> 9) << 13 | 4 * (t & 511);

  const uint32_t ent = a.lut[t & 255], entry = a.table[t & 255];
  __builtin_amdgcn_sched_barrier(0);
  auto load = [&](uint32_t w, float4 (&x)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {              // past the end: read from the tile's start, not used
      const uint64_t j = off + first + 4 * 512 * i;
      x[i] = load_grad4<BF16, LOAD>(a.grads.p[w], j < a.d ? j : off);
    }
  };
  float4 x[4];
  load(vec, x);
  if constexpr (FIND) {                        // the other workers three at a time
    auto other = [&](uint32_t c) { return vec + c < a.n ? vec + c : vec + c - a.n; };
    for (uint32_t c = 1; c < a.n; c += 3) {
      float4 y[3][4];
#pragma unroll
      for (uint32_t u = 0; u < 3; ++u)
        if (c + u < a.n) load(other(c + u), y[u]);
#pragma unroll
      for (uint32_t u = 0; u < 3; ++u)
        if (c + u < a.n) whole_squares<L>(y[u], sm.wsum[other(c + u)], wave, lane);
    }
    whole_squares<L>(x, sm.wsum[vec], wave, lane);
  }
  float* const ef = EF ? static_cast<float*>(const_cast<void*>(a.efs.p[vec])) : nullptr;
  float4 own[4];
  if constexpr (EF) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint64_t j = off + first + 4 * 512 * i;
      own[i] = *reinterpret_cast<const float4*>(ef + (j < a.d ? j : off));
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  if (t < (1 << (T::LOG - 7))) {
    const uint64_t q = (a.j0 + off + 128u * t) >> 7;
    *reinterpret_cast<uint4*>(&sm.sgn[4 * t]) = philox4x32_10((uint32_t)q, (uint32_t)(q >> 32), a.round, SIGN_STREAM, a.k0, a.k1);
  }
  build_quant_lut(ent, lut, t);
  if (EF && t < 256) sm.tabf[t] = (float)entry;
  if constexpr (FIND) __syncthreads();         // the waves' sums
  const int bt = FIND ? wave : t;              // FIND: a wave per block
  if (bt < T::BLOCKS) {
    const uint64_t blk = (off >> L) + bt;
    float M = 0.f;
    if (blk < (a.d >> L)) {
      if constexpr (FIND) {
        const double s = (uint32_t)lane < a.n ? whole_block_sum<L>(sm.wsum[lane], bt) : 0.0;
        M = range_from_sum(wave_largest(s), a.t_p, L);
        if (lane == 0 && vec == 0 && part == 0) a.range_M[blk] = M;
      } else {
        M = a.range_M[blk];
      }
    }
    bool careful;
    const QuantScalars s = quant_scalars(M, -M, a.g, a.lut[a.g - 1], a.c, CFOLD, careful);
    if (!FIND || lane == 0) {
      sQ[bt] = s;
      sm.sCare[bt] = careful;
      sm.sLo[bt] = -M;
      sm.sStep[bt] = (float)(((double)M + (double)M) / (double)a.g);
    }
  }
  if constexpr (EF) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[i].x += own[i].x; x[i].y += own[i].y; x[i].z += own[i].z; x[i].w += own[i].w;
      own[i] = x[i];
    }
  }
  __syncthreads();                             // diagonal, tables and scalars
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int idx = first + 4 * 512 * i;
    const uint32_t bits = sm.sgn[idx >> 5] >> (idx & 31);
    x[i].x = flip(x[i].x, bits & 1u);
    x[i].y = flip(x[i].y, (bits >> 1) & 1u);
    x[i].z = flip(x[i].z, (bits >> 2) & 1u);
    x[i].w = flip(x[i].w, (bits >> 3) & 1u);
    bfly_f4(x[i]);
    *reinterpret_cast<float4*>(&lds[phys<PAD>(idx)]) = x[i];
  }
  lds_stages<2, L, false, PAD, N>(lds, t, [](int, int, float) {});
  __syncthreads();
#pragma unroll
  for (int h = 0; h < (SPLIT ? 1 : 2); ++h) {
    const int idx = 8 * (t + N * (SPLIT ? (int)part : h)), k = T::BLOCKS > 1 ? idx >> L : 0;
    const uint64_t j = off + idx;
    const float4 p0 = *reinterpret_cast<const float4*>(&lds[phys<PAD>(idx)]);
    const float4 p1 = *reinterpret_cast<const float4*>(&lds[phys<PAD>(idx + 4)]);
    const float hv[8] = {p0.x, p0.y, p0.z, p0.w, p1.x, p1.y, p1.z, p1.w};
    const QuantScalars s = sQ[k];
    const uint64_t q = (a.j0 + j) >> 3;
    const uint4 rnd = philox4x32_10((uint32_t)q, (uint32_t)(q >> 32), a.round, a.worker + vec, a.k0, a.k1);
    uint32_t z[8];
    if (!sm.sCare[k]) quantize8<!CFOLD>(hv, rnd, s, lut, z);
    else quantize8<true, true>(hv, rnd, s, lut, z);
    if (j < a.d) store_packed8(static_cast<uint8_t*>(const_cast<void*>(a.packed.p[vec])), j, a.b, z);
    if constexpr (EF) {                        // X_i = T[z] * step_g - M, and the first three stages of its inverse
      const float lo = sm.sLo[k], step = sm.sStep[k];
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = sm.tabf[z[e]] * step + lo;
      bfly<3>(v);
      *reinterpret_cast<float4*>(&lds[phys<PAD>(idx)]) = make_float4(v[0], v[1], v[2], v[3]);
      *reinterpret_cast<float4*>(&lds[phys<PAD>(idx + 4)]) = make_float4(v[4], v[5], v[6], v[7]);
      __builtin_amdgcn_sched_barrier(0);       // one group's draws at a time: both would not fit the registers
    }
  }
  if constexpr (EF) {                          // e <- (grad + e) - RHT^-1(X_i)
    lds_stages<3, L, false, PAD, N>(lds, t, [](int, int, float) {});
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int idx = first + 4 * 512 * i;
      const uint64_t j = off + idx;
      const uint32_t bits = sm.sgn[idx >> 5] >> (idx & 31);
      const float4 v = *reinterpret_cast<const float4*>(&lds[phys<PAD>(idx)]);
      if (j < a.d)
        *reinterpret_cast<float4*>(ef + j) =
            make_float4(own[i].x - flip(v.x * a.c, bits & 1u), own[i].y - flip(v.y * a.c, (bits >> 1) & 1u),
                        own[i].z - flip(v.z * a.c, (bits >> 2) & 1u), own[i].w - flip(v.w * a.c, (bits >> 3) & 1u));
    }
  }
}

}  // namespace thc
