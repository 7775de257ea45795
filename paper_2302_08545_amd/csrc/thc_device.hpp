// Device-side building blocks shared by the THC kernels (gfx950, wave64).
//
// Numeric contract: every butterfly is one binary32 add and one binary32 subtract, stages run in the order
// thc_params.stage_order fixes (the host hands each pass its bits as a TileMap), and nothing is contracted into a
// fused multiply-add unless written as __builtin_fmaf.  The file must be compiled with -ffp-contract=off.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "thc_tilemap.hpp"

namespace thc {

constexpr int TILE = 1 << LOG_TILE;   // coordinates one workgroup holds in LDS (32 KB of binary32)
constexpr int NT = 512;               // threads per workgroup: 16 coordinates each
constexpr int MAXW = 64;              // THC_MAX_WORKERS

struct PtrArr {
  const void* p[MAXW];
};

__device__ __forceinline__ uint64_t tm_base(const TileMap& m, uint32_t tile) {
  const uint32_t tib = tile & ((1u << m.nfixed) - 1u);
  uint32_t off = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) off |= ((tib >> m.fcum[i]) & m.fmask[i]) << m.fpos[i];
  return ((uint64_t)(tile >> m.nfixed) << m.L) | off;
}

// A pass that reads what the pass before it has just written, and more of it than the 256 MB memory-side cache holds, walks
// the launch's tiles and vectors last one first (see last_first): what was written last is still there, where a walk in the
// same order would find each line just dropped.  Where the walk starts and its step come as arguments, next to others that are
// read first: the grid's size lies behind all arguments, in a cache line that nothing else has asked for, and reading it there
// took 0.2 to 0.3 us of every launch (the quantizer on 32 tiles of blocks of 2^10 4.27 -> 3.75 us, of 2^17 4.57 -> 4.30;
// thc_compress_all on one block of 2^18 10.5 -> 10.2).  Each kernel's place for them is the one measured best: the quantizer
// 0.25 us ahead of the tiling, the inverse's last pass behind everything (8 blocks of 2^20 29.5 -> 28.3 us, from the grid's
// size 28.6).
struct Walk {
  uint32_t tile = 0, vec = 0;   // of the launch's first workgroup
  uint32_t step = 1;            // 1, or 2^32 - 1: backwards
};
__device__ __forceinline__ uint32_t walk_x(const Walk& w) { return w.tile + w.step * blockIdx.x; }
__device__ __forceinline__ uint32_t walk_y(const Walk& w) { return w.vec + w.step * blockIdx.y; }

// What an access leaves in the caches.
//   KEEP     the default.
//   STREAM   non-temporal: the line goes first.  For instructions that take whole 128-byte lines: where two instructions share a
//            line, the second finds it gone (rows of 64 bytes, a pass over blocks of 2^22: 435 -> 455 us).  Where it is used
//            all the same, the figures stand there.
//   THROUGH  a device-scope store: written through the XCD's L2 at once.  Plain stores fill the L2 with dirty lines, whose
//            eviction competes with the loads and whose rest is written back at the end of the kernel, before the next one starts.
enum Mem { KEEP, STREAM, THROUGH };

template <auto V>
struct Const { static constexpr auto value = V; };

template <class T>
using Vec4 = T __attribute__((ext_vector_type(4)));

template <Mem M>
__device__ __forceinline__ float4 load_f4(const float* p) {
  if constexpr (M == STREAM) {
    const Vec4<float> r = __builtin_nontemporal_load(reinterpret_cast<const Vec4<float>*>(p));
    return make_float4(r.x, r.y, r.z, r.w);
  } else {
    return *reinterpret_cast<const float4*>(p);
  }
}

template <Mem M>
__device__ __forceinline__ uint4 load_u4(const void* p) {
  if constexpr (M == STREAM) {
    const Vec4<uint32_t> r = __builtin_nontemporal_load(static_cast<const Vec4<uint32_t>*>(p));
    return make_uint4(r.x, r.y, r.z, r.w);
  } else {
    return *static_cast<const uint4*>(p);
  }
}

template <Mem M>
__device__ __forceinline__ void store_u4(void* p, uint4 v) {
  if constexpr (M == STREAM) {
    const Vec4<uint32_t> r = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(r, static_cast<Vec4<uint32_t>*>(p));
  } else {
    *static_cast<uint4*>(p) = v;
  }
}

template <Mem M>
__device__ __forceinline__ void store_f(float* p, float v) {
  if constexpr (M == STREAM) __builtin_nontemporal_store(v, p);
  else if constexpr (M == THROUGH) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else *p = v;
}

template <Mem M>
__device__ __forceinline__ void store_f4(float* p, float4 v) {
  static_assert(M != THROUGH, "no such store of 16 bytes");
  if constexpr (M == STREAM) {
    const Vec4<float> r = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(r, reinterpret_cast<Vec4<float>*>(p));
  } else {
    *reinterpret_cast<float4*>(p) = v;
  }
}

__device__ __forceinline__ uint32_t tm_row(const TileMap& m, uint32_t r) {
  return ((r & ((1u << m.n0) - 1u)) << m.sh0) | ((r >> m.n0) << m.sh1);
}

// ---------------------------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11).  One call yields 128 bits.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);   // three-input XOR in one instruction (truth table 0x96)
}

__device__ __forceinline__ uint4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                               uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
    const uint32_t n0 = xor3((uint32_t)(p1 >> 32), c1, k0);
    const uint32_t n1 = (uint32_t)p1;
    const uint32_t n2 = xor3((uint32_t)(p0 >> 32), c3, k1);
    const uint32_t n3 = (uint32_t)p0;
    c0 = n0; c1 = n1; c2 = n2; c3 = n3;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return make_uint4(c0, c1, c2, c3);
}

constexpr uint32_t SIGN_STREAM = 0x80000000u;

// Word `(j >> 5) & 3` of the sign stream call that covers coordinate j (j a multiple of 32).
__device__ __forceinline__ uint32_t sign_word(uint64_t j, uint32_t round, uint32_t k0, uint32_t k1) {
  const uint64_t q = j >> 7;
  const uint4 r = philox4x32_10((uint32_t)q, (uint32_t)(q >> 32), round, SIGN_STREAM, k0, k1);
  const uint32_t sel = (uint32_t)(j >> 5) & 3u;
  return sel == 0 ? r.x : sel == 1 ? r.y : sel == 2 ? r.z : r.w;
}

__device__ __forceinline__ float flip(float x, uint32_t bit /* 0 or 1 */) {
  return __uint_as_float(__float_as_uint(x) ^ (bit << 31));
}

// ---------------------------------------------------------------------------------------------
// In-register Walsh-Hadamard butterflies over 2^NB values, strides 1, 2, 4, ... in that order.
// ---------------------------------------------------------------------------------------------
template <int NB>
__device__ __forceinline__ void bfly(float (&v)[1 << NB]) {
#pragma unroll
  for (int s = 0; s < NB; ++s) {
    const int h = 1 << s;
#pragma unroll
    for (int j = 0; j < (1 << NB); ++j) {
      if ((j & h) == 0) {
        const float a = v[j], b = v[j + h];
        v[j] = a + b;
        v[j + h] = a - b;
      }
    }
  }
}

template <>
__device__ __forceinline__ void bfly<0>(float (&)[1]) {}

__device__ __forceinline__ void bfly_f4(float4& x) {   // strides 1 and 2 inside four consecutive values
  const float a = x.x + x.y, b = x.x - x.y, c = x.z + x.w, d = x.z - x.w;
  x.x = a + c; x.y = b + d; x.z = a - c; x.w = b - d;
}

// ---------------------------------------------------------------------------------------------
// LDS tile of TILE floats, three layouts (logical index -> physical slot):
//   PLAIN  identity.  Enough when every round reads 64 consecutive values per wave (P >= 6).
//   SWZ    bits 2..4 ^= bits 6..8: strided gathers of any round hit 32 distinct banks per half-wave.
//   PAD    four unused floats after every 64: the same property, and the 16 values a thread gathers in a
//          round sit at a constant physical stride, so their addresses are immediate offsets.
// All three keep four consecutive, 4-aligned values together as one 16-byte unit.
// ---------------------------------------------------------------------------------------------
enum Layout { PLAIN = 0, SWZ = 1, PAD = 2 };
constexpr int padded(int n) { return n + 4 * (n / 64); }
constexpr int TILE_PAD = padded(TILE);

__device__ __forceinline__ int swz(int i) { return i ^ (((i >> 6) & 7) << 2); }

template <Layout LY>
__device__ __forceinline__ int phys(int i) {
  if constexpr (LY == SWZ) return swz(i);
  else if constexpr (LY == PAD) return i + 4 * (i >> 6);
  else return i;
}

// One round: every thread gathers 16 values as (16 >> NB) groups of 2^NB values that differ in index
// bits [P, P+NB), runs the butterflies, and hands each result to sink(base, e << P, value): the value's
// tile index is base + (e << P), the two parts have no bits in common and the second is a constant.
template <int P, int NB, Layout LY, int N, class Sink>
__device__ __forceinline__ void lds_round(const float* lds, int t, Sink&& sink) {
  constexpr int E = 1 << NB;
  constexpr int G = 16 >> NB;
  // physical distance between consecutive gathered values (PLAIN / PAD only)
  constexpr int ESTR = (LY == PAD && P >= 6) ? (1 << P) + 4 * ((1 << P) >> 6) : (1 << P);
  static_assert(LY != PAD || P >= 6 || P + NB <= 6, "a padded gather must not straddle a 64-value group");
#pragma unroll
  for (int gi = 0; gi < G; ++gi) {
    const int vt = t + N * gi;
    const int base = (vt & ((1 << P) - 1)) | ((vt >> P) << (P + NB));
    const float* pb = lds + phys<LY>(base);
    float v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = (LY == SWZ) ? lds[swz(base + (e << P))] : pb[e * ESTR];
    bfly<NB>(v);
#pragma unroll
    for (int e = 0; e < E; ++e) sink(base, e << P, v[e]);
  }
}

// Stages for index bits [P, HI) on a tile resident in LDS, 16 values for each of the N threads.  When FUSE is set the last round hands its
// results to `sink` (typically a global store) instead of writing them back to LDS.
template <int P, int HI, bool FUSE, Layout LY, int N = NT, class Sink>
__device__ __forceinline__ void lds_stages(float* lds, int t, Sink&& sink) {
  constexpr int MAXB = LY == PAD && P < 6 ? (6 - P < 4 ? 6 - P : 4) : 4;   // a padded round stays inside 64 values or above
  constexpr int NB = (HI - P) < MAXB ? (HI - P) : MAXB;
  constexpr bool LAST = (P + NB == HI);
  __syncthreads();
  if constexpr (LAST && FUSE) {
    lds_round<P, NB, LY, N>(lds, t, sink);
  } else {
    if constexpr (NB > 0) {
      lds_round<P, NB, LY, N>(lds, t, [&](int base, int eoff, float v) { lds[phys<LY>(base + eoff)] = v; });
    }
    if constexpr (!LAST) lds_stages<P + NB, HI, FUSE, LY, N>(lds, t, sink);
  }
}

__device__ __forceinline__ void bf4(float4& a, float4& b) {   // (a, b) -> (a + b, a - b), four columns at once
  const float4 s = make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
  b = make_float4(a.x - b.x, a.y - b.y, a.z - b.z, a.w - b.w);
  a = s;
}

// fixed-order butterfly sum over the 64 lanes of a wave; every lane ends with the same total
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) v += __shfl_xor(v, m, 64);
  return v;
}

// The same totals of four values, that of the i-th in lane i: a lane hands over what it does not keep, so three
// exchanges take the place of eight (every sum has the same two operands as in wave_sum).
__device__ __forceinline__ double wave_sum4(double a, double b, double c, double d) {
  const int lane = threadIdx.x & 63;
  const bool odd = lane & 1, up = lane & 2;
  const double p = (odd ? b : a) + __shfl_xor(odd ? a : b, 1, 64);
  const double q = (odd ? d : c) + __shfl_xor(odd ? c : d, 1, 64);
  double v = (up ? q : p) + __shfl_xor(up ? p : q, 2, 64);
#pragma unroll
  for (int m = 4; m < 64; m <<= 1) v += __shfl_xor(v, m, 64);
  return v;
}

// ---------------------------------------------------------------------------------------------
// Bit streams of w-bit fields (w <= 16), least-significant bits first: eight consecutive fields occupy
// exactly w consecutive bytes.  Generic (byte-wise) codec for the widths without a dedicated fast path.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ void store_fields8(uint8_t* dst, const uint32_t (&z)[8], uint32_t w) {
  uint64_t lo = 0, hi = 0;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const uint32_t pos = w * e;
    if (pos < 64) {
      lo |= (uint64_t)z[e] << pos;
      if (pos + w > 64) hi |= (uint64_t)z[e] >> (64 - pos);
    } else {
      hi |= (uint64_t)z[e] << (pos - 64);
    }
  }
  for (uint32_t i = 0; i < w; ++i) dst[i] = (uint8_t)(i < 8 ? lo >> (8 * i) : hi >> (8 * (i - 8)));
}

__device__ __forceinline__ void load_fields8(const uint8_t* src, uint32_t w, uint32_t (&z)[8]) {
  uint64_t lo = 0, hi = 0;
  for (uint32_t i = 0; i < w; ++i) {
    const uint64_t byte = src[i];
    if (i < 8) lo |= byte << (8 * i); else hi |= byte << (8 * (i - 8));
  }
  const uint32_t mask = (1u << w) - 1u;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const uint32_t pos = w * e;
    uint64_t v;
    if (pos < 64) {
      v = lo >> pos;
      if (pos + w > 64) v |= hi << (64 - pos);
    } else {
      v = hi >> (pos - 64);
    }
    z[e] = (uint32_t)v & mask;
  }
}

__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

}  // namespace thc
