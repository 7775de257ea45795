// Transform passes on tiles of 2^15 coordinates, 64 values per thread: blocks of 2^22 (large calls) to 2^25.
//
// What bounds it: bytes.  Every pass over a block reads and writes (or reads) each value once at what HBM takes, 5 to
// 6 TB/s here, so fewer passes is the gain: 15 + 10 stages make two passes of a 2^25-point block, where tiles of 8192
// (13 + 6 + 6) make three; and blocks of 2^22 get rows of 256 columns (1 KB) in the last pass instead of 16 (64 bytes,
// which over-fetches).  Measured, ResNet-50-shaped round (2^25, n = 8, error feedback): 3050 us with 8192-coordinate
// tiles, 2072 us with these; the EF chain of GPT-2-shaped blocks (2^22, n = 32): 15.1 ms and 12.8 ms.
//
// Why this shape.  64 values x 512 threads is what two workgroups per compute unit can keep in registers (128 each);
// the tile goes through LDS in two independent halves of 64 KB.  Four waves per SIMD are enough here because a wave
// has 32 to 64 loads in flight.  Blocks up to 2^21 are as fast or faster with the smaller tiles (first pass 740 us
// against 740 to 780 us at 64 blocks of 2^20 x 8 vectors), and small calls keep more compute units busy with them.
#pragma once

#include "thc_bigmap.hpp"
#include "thc_inverse.hpp"

namespace thc {

constexpr int BIG = 1 << LOG_BIG;

// ---------------------------------------------------------------------------------------------
// First pass.  A thread holds 64 values; the 15 stages run as 4 + 5 + 5 + 1: bits p0..p3 on the 16 consecutive
// values a thread loads, p4..p8 and p9..p13 after one exchange through LDS each, p14 between the two halves of the
// registers.  Both exchanges keep p14, so the tile goes through LDS in two halves of 64 KB and two workgroups share a
// compute unit.  LDS slots are padded so that every access is free of bank conflicts and the 32 addresses of a
// thread are one base plus constants.
// ---------------------------------------------------------------------------------------------
__host__ __device__ constexpr int bphys(int i) { return i + 4 * (i >> 6) + 16 * (i >> 10); }
constexpr int BIG_LDS = bphys(1 << 14);
constexpr int BIG_SIGN_WORDS = BIG / 32;

// fill(h, x): x[y][0..15] = values p = lane << 4 | wave << 10 | y << 13 | h << 14 + (0..15), before any stage;
// out(k, v): v belongs to processing index t | k << 9 (t = thread, k < 64, a constant).  P14 false: no stage p14.
template <bool P14 = true, class Fill, class Out>
__device__ __forceinline__ void big_lo_stages(float* lds, int t, Fill&& fill, Out&& out) {
  const int lane = t & 63, wave = t >> 6;
  float* const wp = lds + bphys(lane << 4 | wave << 10);
  float* const r1 = lds + bphys((lane & 15) | (lane >> 4) << 9 | wave << 11);
  const float* const r2 = lds + bphys(t);
  float u[2][32];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    float x[2][16];
    fill(h, x);
#pragma unroll
    for (int y = 0; y < 2; ++y) bfly<4>(x[y]);
    if (h) __syncthreads();                        // the first half has been read
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int e = 0; e < 16; e += 4)
        *reinterpret_cast<float4*>(wp + bphys(y << 13) + e) = make_float4(x[y][e], x[y][e + 1], x[y][e + 2], x[y][e + 3]);
    __syncthreads();
    float v[32];
#pragma unroll
    for (int e = 0; e < 32; ++e) v[e] = r1[bphys(e << 4)];
    bfly<5>(v);
#pragma unroll
    for (int e = 0; e < 32; ++e) r1[bphys(e << 4)] = v[e];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 32; ++e) u[h][e] = r2[bphys(e << 9)];
    bfly<5>(u[h]);
  }
#pragma unroll
  for (int e = 0; e < 32; ++e) {
    out(e, P14 ? u[0][e] + u[1][e] : u[0][e]);
    out(e | 32, P14 ? u[0][e] - u[1][e] : u[1][e]);
  }
}

struct alignas(16) SmemBigLo {
  float lds[BIG_LDS];
  uint32_t sgn[BIG_SIGN_WORDS];
  double wsum[BIG / TILE][NT / 64];
};

struct BigLoArgs {
  PtrArr grads;
  PtrArr efs;          // unused without error feedback
  float* ws_x;         // d floats per vector
  double* partials;    // per vector `pstride` doubles, one per 8192 coordinates; or null
  uint64_t pstride;
  uint64_t d;
  uint64_t j0;         // global coordinate of the vectors' first element
  uint32_t round, k0, k1;
};

template <bool BF16, Mem M = KEEP>
__device__ __forceinline__ void load_grad16(const void* g, uint64_t j, float (&v)[16]) {
  if constexpr (BF16) {
#pragma unroll
    for (int e = 0; e < 16; e += 8) {
      const uint4 r = load_u4<M>(static_cast<const uint16_t*>(g) + j + e);
      const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        v[e + 2 * k] = __uint_as_float(w[k] << 16);
        v[e + 2 * k + 1] = __uint_as_float(w[k] & 0xFFFF0000u);
      }
    }
  } else {
#pragma unroll
    for (int e = 0; e < 16; e += 4) {
      const float4 r = *reinterpret_cast<const float4*>(static_cast<const float*>(g) + j + e);
      v[e] = r.x; v[e + 1] = r.y; v[e + 2] = r.z; v[e + 3] = r.w;
    }
  }
}

// x with its sign bit flipped where bit k of `bits` is set: one shift and one three-input operation
__device__ __forceinline__ float flip_bit(float x, uint32_t bits, int k) {
  return __uint_as_float(__builtin_amdgcn_bitop3_b32(__float_as_uint(x), bits << (31 - k), 0x80000000u, 0x78));   // a ^ (b & c)
}

// grid = (tiles of a vector, vectors).
//
// The norms are added up exactly as fwd_lo_tile does, one partial sum per 8192 coordinates, so that M does not depend on
// which tile a call takes: a run of 16 values per thread and value of (p13, p14) is one of its tiles, whose thread holds
// four sums of four squares 2048 coordinates apart.  Those lie with other waves here and cross over through LDS, 32 KB a
// half, before the half's first stages need the space; the sums over a wave wait until the tile's stores are under way.
// What that costs against sums of 16 values in a row and one partial sum a tile: one block of 2^23, 2^24 or 2^25 34.1 us
// (32.5), 50.7 (49.3) and 92.6 (92.4) a call, eight vectors of 2^25 with error feedback 2041 us (2036).
//
// LOAD: how gradients are read, STREAM with bf16 and error feedback only, see stream_big_inputs.
template <bool BF16, bool EF, bool XO, Mem LOAD>
__global__ __launch_bounds__(NT, 4) void k_big_lo(const BigLoArgs a) {
  __shared__ SmemBigLo sm;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const uint32_t vec = blockIdx.y, tile = xcd_tile(blockIdx.x, gridDim.x);
  const uint64_t off = big_lo_base<XO>(tile);
  const char* const grad = static_cast<const char*>(a.grads.p[vec]) + off * (BF16 ? 2 : 4);
  const float* const ef = EF ? static_cast<const float*>(a.efs.p[vec]) + off : nullptr;
  const uint32_t tp = big_p<XO>(lane << 4 | wave << 10);

  float v[4][16], e[2][16];
  double acc[4];
  auto load = [&](int h) {   // operands of one half of the tile
#pragma unroll
    for (int y = 0; y < 2; ++y) {
      load_grad16<BF16, LOAD>(grad, tp + big_p<XO>((2 * h + y) << 13), v[2 * h + y]);
      if constexpr (EF) load_grad16<false>(ef, tp + big_p<XO>((2 * h + y) << 13), e[y]);
    }
  };
  double* const squares = reinterpret_cast<double*>(sm.lds);
  auto take = [&](int h) {   // x = grad + e and its squares in binary64 (a binary32 square is exact there)
    if constexpr (EF) {
#pragma unroll
      for (int y = 0; y < 2; ++y)
#pragma unroll
        for (int k = 0; k < 16; ++k) v[2 * h + y][k] += e[y][k];
    }
    if (!a.partials) return;
    if (h) __syncthreads();  // the first half has been read
#pragma unroll
    for (int y = 0; y < 2; ++y) {
      double2* const w = reinterpret_cast<double2*>(squares + (y << 11 | t << 2));
#pragma unroll
      for (int i = 0; i < 4; i += 2) {
        double c[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const float* const x = &v[2 * h + y][4 * (i + k)];
          c[k] = sum_squares4(make_float4(x[0], x[1], x[2], x[3]));
        }
        w[i >> 1] = make_double2(c[0], c[1]);
      }
    }
    __syncthreads();
#pragma unroll
    for (int y = 0; y < 2; ++y) {
      const double* const r = squares + (y << 11 | t);
      acc[2 * h + y] = (r[0] + r[NT]) + (r[2 * NT] + r[3 * NT]);
    }
    if (!h) __syncthreads();   // the second half has a barrier of its own before its first stages
  };

  load(0);
  if constexpr (!EF) load(1);
  if (t < BIG / 128) {   // the tile's diagonal: one Philox call per 128 coordinates
    const uint64_t q = (a.j0 + off + big_p<XO>(t << 7)) >> 7;
    *reinterpret_cast<uint4*>(&sm.sgn[4 * t]) =
        philox4x32_10((uint32_t)q, (uint32_t)(q >> 32), a.round, SIGN_STREAM, a.k0, a.k1);
  }
  __syncthreads();   // diagonal bits visible
  float* const dst = a.ws_x + (uint64_t)vec * a.d + off;
  big_lo_stages(
      sm.lds, t,
      [&](int h, float (&x)[2][16]) {
        take(h);
        if constexpr (EF) {
          if (h == 0) {      // the second half's operands travel while the first goes through its stages
            __builtin_amdgcn_sched_barrier(0);
            load(1);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
#pragma unroll
        for (int y = 0; y < 2; ++y) {
          const uint32_t bits = sm.sgn[lane >> 1 | wave << 5 | y << 8 | h << 9] >> ((lane & 1) << 4);
#pragma unroll
          for (int k = 0; k < 16; ++k) x[y][k] = flip_bit(v[2 * h + y][k], bits, k);
        }
      },
      [&](int k, float r) { store_f<THROUGH>(&dst[big_p<XO>(k << 9) + t], r); });
  if (a.partials) {          // the sums over a wave and over the waves, while the stores drain
    const double s = wave_sum4(acc[0], acc[1], acc[2], acc[3]);
    if (lane < 4) sm.wsum[lane][wave] = s;
    __syncthreads();
    if (t < BIG / TILE) {    // tiles 4 * tile + 0..3 of the smaller kind, in either stage order
      double r = 0.0;
#pragma unroll
      for (int w = 0; w < NT / 64; ++w) r += sm.wsum[t][w];
      a.partials[(uint64_t)vec * a.pstride + (uint64_t)tile * (BIG / TILE) + t] = r;
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Last pass: tiles of 2^R rows (stage bits q), 7 <= R <= 10, by 2^C columns, C = 15 - R.  A thread holds 8 consecutive
// columns (what one Philox call and one packed word cover) in eight slots.  Row bits q0..q2 start in the slot index,
// q3 and q4 on lane bits 4 and 5, from where a lane swap brings them into the slot index (half an instruction per
// value, no LDS, no barrier); q5..q7 take one exchange through LDS, in two halves of 64 KB, and q8 and q9 two more
// swaps.
// ---------------------------------------------------------------------------------------------
// LDS slot (16-byte units) of thread t's half of slot k before the exchange
__host__ __device__ constexpr int xphys(int k, int t) { return k * (NT + 4) + t; }
constexpr int BIG_XLDS = 8 * (NT + 4);   // 16-byte units: 66 KB

template <int BIT>
__device__ __forceinline__ void slot_stage(float (&v)[8][8]) {
#pragma unroll
  for (int k = 0; k < 8; ++k)
    if (!(k & (1 << BIT))) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float a = v[k][e], b = v[k | (1 << BIT)][e];
        v[k][e] = a + b;
        v[k | (1 << BIT)][e] = a - b;
      }
    }
}

// exchanges slot bit BIT with lane bit 4 (LANE32 = false) or 5
template <int BIT, bool LANE32>
__device__ __forceinline__ void slot_swap(float (&v)[8][8]) {
#pragma unroll
  for (int k = 0; k < 8; ++k)
    if (!(k & (1 << BIT))) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t a = __float_as_uint(v[k][e]), b = __float_as_uint(v[k | (1 << BIT)][e]);
        const auto r = LANE32 ? __builtin_amdgcn_permlane32_swap(a, b, false, false)
                              : __builtin_amdgcn_permlane16_swap(a, b, false, false);
        v[k][e] = __uint_as_float(r[0]);
        v[k | (1 << BIT)][e] = __uint_as_float(r[1]);
      }
    }
}

// Which tile bits select the XCD: 3 to 5, as for the first pass, but for two cases.  Tiles of 2^25-point blocks hold 128
// bytes of each of their rows, and an XCD that takes 64 of them in a row fetches whole pages: 2^28 worker-coordinates with
// error feedback 910 -> 867 us (ascending 928 -> 888), one vector 126 -> 117, the quantizer 287 -> 281.  The error-feedback
// update of 2^22-point blocks in the split order: 2^29 worker-coordinates in bf16 1432 -> 1402 us, in binary32 729 -> 718.
// For the other widths the choice is that of the first pass.  (R = 9: tile bits further up gain 2 to 9 % with error feedback
// and lose 3 % without; a choice by EF, as for R = 7, is not made there.)
template <int R, bool XO, bool EF>
__device__ __forceinline__ uint32_t big_hi_tile(const Walk& w) {
  return xcd_tile<R == 10 ? 6 : R == 7 && XO && EF ? 4 : 3>(walk_x(w), gridDim.x);
}

template <class H, bool XO, Mem M = KEEP>
__device__ __forceinline__ void big_hi_load(const float* src, int t, float (&v)[8][8]) {
  constexpr BigLayout m = H::first();
  const float* const p = src + H::template thread_off<XO, 0>(m, t);
#pragma unroll
  for (int k = 0; k < 8; ++k)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float4 r = load_f4<M>(p + H::template slot_off<XO>(m, k) + h * H::template half_off<XO>());
      v[k][4 * h] = r.x; v[k][4 * h + 1] = r.y; v[k][4 * h + 2] = r.z; v[k][4 * h + 3] = r.w;
    }
}

template <class H>
__device__ __forceinline__ void big_hi_stages(float4* lds, int t, float (&v)[8][8]) {
  slot_stage<0>(v);
  slot_stage<1>(v);
  slot_stage<2>(v);
  slot_swap<0, false>(v);
  slot_stage<0>(v);
  slot_swap<1, true>(v);
  slot_stage<1>(v);
  {
    constexpr BigLayout from = H::second(), to = H::third();
    // where the new thread bits find their data: thread bit i of the reader stands for to.thr[i], which the writer
    // had on a thread bit or in its slot index
    uint32_t rt = 0, rk = 0;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      const uint32_t bit = ((uint32_t)t >> i) & 1u;
      const int p = H::pos(from, to.thr[i]);
      if (p >= 0) rt |= bit << p;
      else
        for (int s = 0; s < 3; ++s)
          if (from.slot[s] == to.thr[i]) rk |= bit << s;
    }
    const int rbase = xphys((int)rk, (int)rt);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (h) __syncthreads();
#pragma unroll
      for (int k = 0; k < 8; ++k)
        lds[xphys(k, t)] = make_float4(v[k][4 * h], v[k][4 * h + 1], v[k][4 * h + 2], v[k][4 * h + 3]);
      __syncthreads();
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        int o = 0;                              // where the writer had slot bits 0..2 of the reader
        for (int s = 0; s < 3; ++s)
          if (k & (1 << s)) {
            const int p = H::pos(from, to.slot[s]);
            if (p >= 0) o += 1 << p;
            else
              for (int z = 0; z < 3; ++z)
                if (from.slot[z] == to.slot[s]) o += xphys(1 << z, 0);
          }
        const float4 r = lds[rbase + o];
        v[k][4 * h] = r.x; v[k][4 * h + 1] = r.y; v[k][4 * h + 2] = r.z; v[k][4 * h + 3] = r.w;
      }
    }
    slot_stage<0>(v);
    slot_stage<1>(v);
    if constexpr (H::E >= 3) slot_stage<2>(v);
    if constexpr (H::E >= 4) { slot_swap<0, false>(v); slot_stage<0>(v); }
    if constexpr (H::E >= 5) { slot_swap<1, true>(v); slot_stage<1>(v); }
  }
}

struct BigQuantArgs {
  const float* x;          // half-rotated vectors, d floats per vector of the launch (grid.y)
  const float* range_M;    // m = -M
  PtrArr packed;
  uint64_t d;
  uint64_t j0;
  Walk walk;
  uint32_t b, g;
  uint32_t round, worker, k0, k1;
  float c;
  uint32_t lut[256];
};

struct alignas(16) SmemBigHi {
  float4 x[BIG_XLDS];
  uint32_t lut[256][4];
  float sQ[4];
  int sCare;
};

template <int R, bool XO>
__global__ __launch_bounds__(NT, 4) void k_big_quant(const BigQuantArgs a) {
  constexpr bool CFOLD = ((LOG_BIG + R) & 1) == 0;
  __shared__ SmemBigHi sm;
  uint4* const lut = reinterpret_cast<uint4*>(sm.lut);
  const int t = threadIdx.x;
  const uint32_t vec = walk_y(a.walk), tile = big_hi_tile<R, XO, false>(a.walk);
  const uint64_t base = big_hi_base<R, XO>(tile);
  const uint32_t ent = a.lut[t & 255];   // requested before the tile, so that the table is made while that travels
  float v[8][8];
  __builtin_amdgcn_sched_barrier(0);
  big_hi_load<BigHi<R>, XO>(a.x + (uint64_t)vec * a.d + base, t, v);
  __builtin_amdgcn_sched_barrier(0);
  build_quant_lut(ent, lut, t);
  if (t == 0) {
    const uint32_t blk = tile >> R;
    const float M = a.range_M[blk];
    bool careful;
    *reinterpret_cast<QuantScalars*>(sm.sQ) = quant_scalars(M, -M, a.g, a.lut[a.g - 1], a.c, CFOLD, careful);
    sm.sCare = careful;
  }
  __syncthreads();
  big_hi_stages<BigHi<R>>(sm.x, t, v);
  const QuantScalars s = *reinterpret_cast<const QuantScalars*>(sm.sQ);
  const bool careful = __builtin_amdgcn_readfirstlane(sm.sCare) != 0;
  constexpr BigLayout m = BigHi<R>::last();
  const uint32_t to = BigHi<R>::template thread_off<XO, 0>(m, t);
  // the tile's base has no bits in common with the offsets inside it: both counter words come from one OR
  const uint64_t q0 = (a.j0 + base) >> 3;
  const uint32_t qlo = (uint32_t)q0 | (to >> 3), qhi = (uint32_t)(q0 >> 32);
  uint8_t* const packed = static_cast<uint8_t*>(const_cast<void*>(a.packed.p[vec])) + (base >> 3) * a.b;
  const uint32_t stream = a.worker + vec;
  auto step = [&](int k, auto mulc, auto care) {
    const uint32_t so = BigHi<R>::template slot_off<XO>(m, k);
    const uint4 rnd = philox4x32_10(qlo | (so >> 3), qhi, a.round, stream, a.k0, a.k1);
    uint32_t z[8];
    quantize8<mulc.value, care.value>(v[k], rnd, s, lut, z);
    store_packed8<false>(packed, to + so, a.b, z);
    __builtin_amdgcn_sched_barrier(0);   // one step's draws at a time: interleaved steps would not fit the registers
  };
  if (!careful) {
#pragma unroll
    for (int k = 0; k < 8; ++k) step(k, Const<!CFOLD>{}, Const<false>{});
  } else {
#pragma unroll
    for (int k = 0; k < 8; ++k) step(k, Const<true>{}, Const<true>{});
  }
}

// ---------------------------------------------------------------------------------------------
// Inverse first pass.  SB: bits per code where that is known at compile time (4, 8, 16), else 0.
// ---------------------------------------------------------------------------------------------
struct BigInvLoArgs {
  PtrArr src;
  const float* range_M;
  const float* range_m;    // or null: m = -M
  float* ws_x;
  uint64_t d;
  uint32_t L, src_bits, use_table, divisor;
  uint8_t table[256];
};

struct alignas(16) SmemBigInvLo {
  float lds[BIG_LDS];
  float tabf[256];
  float lo, step;
};

// sixteen W-bit fields from bit 16 * `half` of `first` on, reading only the dwords that hold them
template <int W>
__device__ __forceinline__ void cut16_global(const uint32_t* first, bool half, uint32_t (&y)[16]) {
  constexpr int NW = (16 * W + 31) / 32;
  uint32_t d[NW + 1];
#pragma unroll
  for (int k = 0; k < NW; ++k) d[k] = first[k];
  d[NW] = 0;
  if (half) {
#pragma unroll
    for (int k = 0; k < NW; ++k) d[k] = __builtin_amdgcn_alignbit(d[k + 1], d[k], 16);
  }
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    constexpr uint32_t mask = (1u << W) - 1u;
    const int k = (e * W) >> 5, sh = (e * W) & 31;
    uint32_t v = d[k] >> sh;
    if (sh + W > 32) v |= d[k + 1] << (32 - sh);
    y[e] = v & mask;
  }
}

// sixteen codes from coordinate j (a multiple of 16) on
__device__ __forceinline__ void codes16(const uint8_t* src, uint32_t bits, uint64_t j, uint32_t (&y)[16]) {
  if (codes_fast_width(bits)) {
    uint32_t w[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    codes_load(src, bits, j, w, y);
    codes_decode(bits, true, w, y);
    return;
  }
  const uint64_t bit = j * bits;
  const uint32_t* const first = reinterpret_cast<const uint32_t*>(src) + (bit >> 5);
  const bool half = (bit & 16u) != 0;
  switch (bits) {
#define THC_CUT(W) case W: cut16_global<W>(first, half, y); break;
    THC_CUT(3) THC_CUT(5) THC_CUT(6) THC_CUT(7) THC_CUT(9) THC_CUT(10) THC_CUT(11) THC_CUT(12) THC_CUT(13)
    THC_CUT(14) THC_CUT(15)
#undef THC_CUT
    default: break;
  }
}

// HOW the half-transformed vector is stored (see through_inverse).  With error feedback non-temporally at any size: 2^25 x 1
// 385 us against 383, 4 blocks of 2^23 of one vector 387 against 380.
template <int SB, bool TABLE, bool XO, Mem HOW>
__global__ __launch_bounds__(NT, 4) void k_big_inv_lo(const BigInvLoArgs a) {
  __shared__ SmemBigInvLo sm;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const uint32_t vec = blockIdx.y, tile = xcd_tile(blockIdx.x, gridDim.x);
  const uint64_t off = big_lo_base<XO>(tile);
  const uint32_t tp = big_p<XO>(lane << 4 | wave << 10);
  const uint32_t bits = SB ? SB : a.src_bits;
  const uint8_t* const src = static_cast<const uint8_t*>(a.src.p[vec]) + (off >> 3) * bits;
  // fast widths: the raw words of all four runs are requested before anything waits
  constexpr int NW = SB ? SB / 2 : 1;
  uint32_t w[4][NW];
  if constexpr (SB != 0) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const uint32_t* const p = reinterpret_cast<const uint32_t*>(src + ((tp + big_p<XO>(s << 13)) >> 3) * SB);
#pragma unroll
      for (int k = 0; k < NW; ++k) w[s][k] = p[k];
    }
  }
  const uint32_t blk = (uint32_t)(off >> a.L);
  const float M = a.range_M[blk], lo = lower_of(a.range_m, blk, M);
  const float step = (float)(((double)M - (double)lo) / (double)a.divisor);
  if constexpr (TABLE) {
    if (t < 256) sm.tabf[t] = (float)a.table[t] * step + lo;   // the table's values on the block's range
    __syncthreads();
  }
  float* const dst = a.ws_x + (uint64_t)vec * a.d + off;
  big_lo_stages(
      sm.lds, t,
      [&](int h, float (&x)[2][16]) {
#pragma unroll
        for (int y = 0; y < 2; ++y) {
          const int s = 2 * h + y;
          uint32_t c[16];
          if constexpr (SB != 0) {
#pragma unroll
            for (int e = 0; e < 16; ++e) c[e] = (w[s][e * SB / 32] >> (e * SB % 32)) & ((1u << SB) - 1u);
          } else {
            codes16(src, bits, tp + big_p<XO>(s << 13), c);
          }
#pragma unroll
          for (int e = 0; e < 16; ++e) x[y][e] = TABLE ? sm.tabf[c[e]] : (float)c[e] * step + lo;
        }
      },
      [&](int k, float r) { store_f<HOW>(&dst[big_p<XO>(k << 9) + t], r); });
}

// ---------------------------------------------------------------------------------------------
// Inverse last pass: finish H, scale, diagonal; EFM 0: out = result, 1 / 2: e <- (grad + e) - result with a binary32 /
// bf16 gradient.  Accesses of whole lines but for bf16 gradients at R = 9 (halves of 64 bytes; read plainly, 2 x 2^24 x 4 vectors
// take 1.00 to 1.01 of the time, 4 x 8 1.01), all of them non-temporal: rounds with error feedback 16 blocks of 2^22 x 32 in bf16
// 13.25 -> 12.87 ms, x 16 in binary32 7.53 -> 7.36, 2 of 2^24 x 4 1117 -> 1053 us, one worker of 4 blocks of 2^23 385 -> 339.
// ---------------------------------------------------------------------------------------------
struct BigInvHiArgs {
  const float* x;
  PtrArr out;
  PtrArr grad;
  uint64_t d;
  uint64_t j0;
  Walk walk;
  uint32_t round, k0, k1;
  float c;
};

struct alignas(16) SmemBigInvHi {
  float4 x[BIG_XLDS];
  uint32_t sgn[BIG_SIGN_WORDS];   // bit (u & 31) of word (row << (C - 5)) + (column >> 5)
};

template <int R, bool XO, int EFM, Mem OUT = R <= 9 ? STREAM : KEEP>
__global__ __launch_bounds__(NT, 4) void k_big_inv_hi(const BigInvHiArgs a) {
  // Rows of 32 columns (R = 10) are whole lines only over two accesses, in either layout.  They keep the eight neighbouring
  // columns, which measured best there; spread and streamed: 2^25 x 8 with error feedback 2077 -> 2203 us.
  constexpr bool LINES = R <= 9;
  constexpr Mem HOW = LINES ? STREAM : KEEP;
  using H = BigHi<R, LINES>;
  __shared__ SmemBigInvHi sm;
  const int t = threadIdx.x;
  const uint32_t vec = walk_y(a.walk), tile = big_hi_tile<R, XO, EFM != 0>(a.walk);
  const uint64_t base = big_hi_base<R, XO>(tile);
  float v[8][8];
  big_hi_load<H, XO, HOW>(a.x + (uint64_t)vec * a.d + base, t, v);
  // the diagonal while the loads travel: one Philox call covers 128 coordinates, or what of them the tile holds
  constexpr int PER = H::C >= 7 ? 4 : 1 << (H::C - 5);    // words of a call that belong to the tile
  for (int i = t; i < BIG_SIGN_WORDS / PER; i += NT) {
    const int word = i * PER, row = word >> (H::C - 5), col = (word & ((1 << (H::C - 5)) - 1)) << 5;
    const uint64_t j = a.j0 + base + big_q<XO>(row) + big_u<XO>(col);
    const uint4 r = philox4x32_10((uint32_t)(j >> 7), (uint32_t)(j >> 39), a.round, SIGN_STREAM, a.k0, a.k1);
    if constexpr (PER == 4) {
      *reinterpret_cast<uint4*>(&sm.sgn[word]) = r;
    } else if constexpr (PER == 2) {
      const bool up = (j >> 6) & 1u;
      sm.sgn[word] = up ? r.z : r.x;
      sm.sgn[word + 1] = up ? r.w : r.y;
    } else {
      const uint32_t sel = (uint32_t)(j >> 5) & 3u;
      sm.sgn[word] = sel == 0 ? r.x : sel == 1 ? r.y : sel == 2 ? r.z : r.w;
    }
  }
  __syncthreads();
  big_hi_stages<H>(sm.x, t, v);
  constexpr BigLayout m = H::last();
  const uint32_t to = H::template thread_off<XO, 0>(m, t);
  float* const out = static_cast<float*>(const_cast<void*>(a.out.p[vec])) + base;
  const char* const grad = EFM ? static_cast<const char*>(a.grad.p[vec]) + base * (EFM == 2 ? 2 : 4) : nullptr;
  // tile-local word and bit of the thread's eight columns
  uint32_t tword = 0, tbit = 0;
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    const uint32_t bit = ((uint32_t)t >> i) & 1u;
    const int what = m.thr[i];
    if (what >= 0) tword |= bit << (H::C - 5 + what);
    else if (-1 - what >= 5) tword |= bit << (-1 - what - 5);
    else tbit |= bit << (-1 - what);
  }
  // error feedback: the next eight values of the gradient and of the buffer are requested before this step's stores,
  // which the compiler must not move them across
  constexpr uint32_t half = H::template half_off<XO>();
  float4 g[2], e[2];
  auto operands = [&](uint32_t o, float4 (&gn)[2], float4 (&en)[2]) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      gn[h] = load_grad4<EFM == 2, HOW>(grad, o + h * half);
      en[h] = load_f4<HOW>(out + o + h * half);
    }
  };
  if constexpr (EFM != 0) operands(to, g, e);
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const uint32_t so = H::template slot_off<XO>(m, k);
    float4 gn[2], en[2];
    if constexpr (EFM != 0) {
      if (k < 7) operands(to + H::template slot_off<XO>(m, k + 1), gn, en);
    }
    uint32_t kw = 0;
    for (int s = 0; s < 3; ++s)
      if (k & (1 << s)) kw |= m.slot[s] >= 0 ? 1u << (H::C - 5 + m.slot[s]) : 1u << (-1 - m.slot[s] - 5);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      // the second half of the row lies in a word of its own, the second four neighbours in the same
      const uint32_t bits = sm.sgn[tword | kw | (LINES ? h << (LINES ? H::C - 6 : 0) : 0)] >> (tbit + (LINES ? 0 : 4 * h));
      float4 r = make_float4(flip_bit(v[k][4 * h] * a.c, bits, 0), flip_bit(v[k][4 * h + 1] * a.c, bits, 1),
                             flip_bit(v[k][4 * h + 2] * a.c, bits, 2), flip_bit(v[k][4 * h + 3] * a.c, bits, 3));
      if constexpr (EFM != 0)
        r = make_float4((g[h].x + e[h].x) - r.x, (g[h].y + e[h].y) - r.y, (g[h].z + e[h].z) - r.z, (g[h].w + e[h].w) - r.w);
      store_f4<OUT>(out + to + so + h * half, r);
    }
    if constexpr (EFM != 0) {
#pragma unroll
      for (int h = 0; h < 2; ++h) { g[h] = gn[h]; e[h] = en[h]; }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// The whole inverse transform of blocks of 2^14 (two to a tile) or 2^15 in one launch; see k_inv_whole.
// ---------------------------------------------------------------------------------------------
struct alignas(16) SmemBigWhole {
  float lds[BIG_LDS];
  uint32_t sgn[BIG_SIGN_WORDS];
  float tabf[2][256];
};

template <int L, int SB, int EFM, Mem OUT = STREAM>
__global__ __launch_bounds__(NT, 4) void k_big_inv_whole(const InvWholeArgs a) {
  static_assert(L == 14 || L == 15, "one or two blocks to a tile");
  constexpr bool TABLE = EFM != 0;               // error feedback starts from indices, decompression from sums
  __shared__ SmemBigWhole sm;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const uint32_t vec = blockIdx.y, tile = xcd_tile(blockIdx.x, gridDim.x);
  const uint64_t off = (uint64_t)tile << LOG_BIG;
  const uint32_t tp = lane << 4 | wave << 10;
  const uint32_t bits = SB ? SB : a.lo.src_bits;
  const bool two = L == 15 || a.lo.d - off >= BIG;      // false: an odd number of blocks, the last tile holds one
  const uint8_t* const src = static_cast<const uint8_t*>(a.lo.src.p[vec]) + (off >> 3) * bits;
  constexpr int NW = SB ? SB / 2 : 1;
  uint32_t w[4][NW];
  if constexpr (SB != 0) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const uint32_t* const p = reinterpret_cast<const uint32_t*>(src + ((tp + (s << 13)) >> 3) * SB);
#pragma unroll
      for (int k = 0; k < NW; ++k) w[s][k] = s < 2 || two ? p[k] : 0u;
    }
  }
  if (t < BIG / 128) {
    const uint64_t q = (a.j0 + off + 128u * t) >> 7;
    *reinterpret_cast<uint4*>(&sm.sgn[4 * t]) = philox4x32_10((uint32_t)q, (uint32_t)(q >> 32), a.round, SIGN_STREAM, a.k0, a.k1);
  }
  float lo[2], step[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint64_t blk = (off >> L) + (L == 14 && two ? h : 0);
    const float M = a.lo.range_M[blk];
    lo[h] = lower_of(a.lo.range_m, blk, M);
    step[h] = (float)(((double)M - (double)lo[h]) / (double)a.lo.divisor);
    if constexpr (TABLE) {
      if (t < 256) sm.tabf[h][t] = (float)a.lo.table[t] * step[h] + lo[h];
    }
  }
  __syncthreads();
  float v[8][8];
  big_lo_stages<L == 15>(
      sm.lds, t,
      [&](int h, float (&x)[2][16]) {
#pragma unroll
        for (int y = 0; y < 2; ++y) {
          const int s = 2 * h + y;
          uint32_t c[16];
          if constexpr (SB != 0) {
#pragma unroll
            for (int e = 0; e < 16; ++e) c[e] = (w[s][e * SB / 32] >> (e * SB % 32)) & ((1u << SB) - 1u);
          } else if (h == 0 || two) {
            codes16(src, bits, tp + (s << 13), c);
          } else {
#pragma unroll
            for (int e = 0; e < 16; ++e) c[e] = 0;
          }
#pragma unroll
          for (int e = 0; e < 16; ++e) x[y][e] = TABLE ? sm.tabf[h][c[e]] : (float)c[e] * step[h] + lo[h];
        }
      },
      [&](int k, float r) { v[k >> 3][k & 7] = r; });
  float* const out = static_cast<float*>(const_cast<void*>(a.out.p[vec])) + off + t;
  const char* const grad = EFM ? static_cast<const char*>(a.grad.p[vec]) + (off + t) * (EFM == 2 ? 2 : 4) : nullptr;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    if (k >= 4 && !two) break;
    finish_values<EFM, OUT>(v[k], a.c, out, grad, [&](int i) { return (uint32_t)(8 * k + i) << 9; },
                       [&](int i) { return (sm.sgn[(8 * k + i) << 4 | t >> 5] >> (t & 31)) & 1u; });
  }
}

}  // namespace thc
