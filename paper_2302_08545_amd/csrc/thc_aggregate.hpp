// Aggregation in the compressed domain (PS side of Alg. 2).
#pragma once

#include "thc_device.hpp"

namespace thc {

// ---------------------------------------------------------------------------------------------
// What bounds it in large calls: reading n streams once.  There (from 80 MB on, stream_sums) M = STREAM: loads non-temporal (but for
// indices of 5 bits and more, whose loads share lines), the sums of 4-bit indices and those of other widths than 8 and 16 bits
// as whole lines by way of LDS and non-temporal as well; the others' are plain 16-byte stores.  16 streams of 33 * 2^20 4-bit indices to 9-bit sums 65.7 -> 55.5 us (5.8 TB/s), of 100 *
// 2^20 to 16-bit sums 200 -> 171 (6.1 TB/s), 8 of 40 * 2^20 to 8-bit sums 40.0 -> 36.2, 10 of 64 * 2^20 3-bit ones 64.4 -> 57.8.
// In small calls M = KEEP: the streams have just been written and are in the cache, and latency counts, so four workers'
// loads are in flight (16 streams of 4 * 2^20 to 16-bit sums 12.2 -> 9.4 us; in large calls the same takes 1 to 6 % more).
//
// Aggregation (Alg. 2: Y = sum_i T[Z_i]; the PS only looks up and adds).  Index widths without a kernel of their own
// below, sums of any width.
//
// One thread owns 32 coordinates: exactly B dwords of every stream, whatever B, read as dwords and in batches of four
// workers, because a small call has too few wavefronts to hide one load latency after another.  Up to 3 bits the table
// is two registers and four indices are looked up per byte permute, byte-wise sums widened every `chunk` = floor(255 / g)
// workers; wider tables sit in LDS.
// ---------------------------------------------------------------------------------------------
struct AggArgs {
  PtrArr packed;
  uint8_t* out;
  uint64_t nvec;    // d / 32
  uint32_t n, agg_bits, chunk;
  uint32_t tb[2];   // table bytes 0..7, little endian (B <= 3)
  uint8_t table[256];
};

// B bits at bit `pos` (a constant) of a thread's B dwords, with whatever follows them in the upper bits
template <int B>
__device__ __forceinline__ uint32_t bits_at(const uint32_t (&w)[B], int pos, int len) {
  const int k = pos >> 5, sh = pos & 31;
  return sh + len > 32 ? __builtin_amdgcn_alignbit(w[k + 1 < B ? k + 1 : k], w[k], sh) : w[k] >> sh;
}

// four consecutive fields of B <= 3 bits, one to a byte
template <int B>
__device__ __forceinline__ uint32_t spread4(uint32_t x) {
  constexpr uint32_t pair = ((1u << (2 * B)) - 1u) * 0x00010001u, one = ((1u << B) - 1u) * 0x01010101u;
  x &= (1u << (4 * B)) - 1u;
  x = (x | x << (16 - 2 * B)) & pair;
  return (x | x << (8 - B)) & one;
}

// Writes a thread's 32 sums, acc[m] = those of coordinates 2m (low half) and 2m + 1 (high half).  Widths other than 8
// and 16 go through LDS, `stage` holding 256 * 16 dwords, so that the workgroup writes consecutive 16-byte vectors; all of its
// threads take part, those with `own` false hold no coordinates.
template <Mem M>
__device__ __forceinline__ void store_sums32(const uint32_t (&acc)[16], uint32_t bits, uint8_t* out, uint64_t v0,
                                             uint64_t nvec, bool own, uint32_t* stage) {
  const uint32_t t = threadIdx.x;
  if (bits == 8 || bits == 16) {
    if (!own) return;
    uint4* const dst = reinterpret_cast<uint4*>(out + (v0 + t) * 4 * bits);
    if (bits == 16) {
#pragma unroll
      for (int k = 0; k < 4; ++k) dst[k] = make_uint4(acc[4 * k], acc[4 * k + 1], acc[4 * k + 2], acc[4 * k + 3]);
    } else {
      uint32_t o[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) o[k] = __builtin_amdgcn_perm(acc[2 * k + 1], acc[2 * k], 0x06040200u);
      dst[0] = make_uint4(o[0], o[1], o[2], o[3]);
      dst[1] = make_uint4(o[4], o[5], o[6], o[7]);
    }
    return;
  }
  uint64_t w = 0;
  uint32_t fill = 0, k = 0;                 // uniform: the fields' places do not depend on the thread
#pragma unroll
  for (int e = 0; e < 32; ++e) {
    const uint32_t f = (e & 1) ? acc[e >> 1] >> 16 : acc[e >> 1] & 0xFFFFu;
    w |= (uint64_t)f << fill;
    fill += bits;
    if (fill >= 32) {
      stage[t * bits + k] = (uint32_t)w;
      w >>= 32;
      fill -= 32;
      ++k;
    }
  }
  __syncthreads();
  const uint64_t left = nvec - v0;
  const uint32_t nvec4 = (uint32_t)(left < 256 ? left : 256) * bits / 4;   // whole: nvec is a multiple of 32
  uint4* const dst = reinterpret_cast<uint4*>(out + v0 * 4 * bits);
  for (uint32_t i = t; i < nvec4; i += 256) store_u4<M>(dst + i, reinterpret_cast<const uint4*>(stage)[i]);
}

template <int B, Mem M>
__global__ __launch_bounds__(256) void k_aggregate_any(const AggArgs a) {
  __shared__ __align__(16) uint32_t stage[256 * 16];
  __shared__ uint32_t tab[B > 3 ? 1 << B : 1];
  const uint32_t t = threadIdx.x;
  if constexpr (B > 3) {
    if (t < (1u << B)) tab[t] = a.table[t];
    __syncthreads();
  }
  const uint64_t v0 = (uint64_t)blockIdx.x * 256, v = v0 + t;
  const bool own = v < a.nvec;
  uint32_t acc[16];
#pragma unroll
  for (int m = 0; m < 16; ++m) acc[m] = 0;
  if (own) {
    uint32_t by[8];                         // B <= 3: sums of four consecutive coordinates to a register
    uint32_t run = 0;                       // workers in them
#pragma unroll
    for (int k = 0; k < 8; ++k) by[k] = 0;
    auto widen = [&] {
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        acc[2 * k] += __builtin_amdgcn_perm(0u, by[k], 0x0C010C00u);
        acc[2 * k + 1] += __builtin_amdgcn_perm(0u, by[k], 0x0C030C02u);
        by[k] = 0;
      }
      run = 0;
    };
    auto add = [&](const uint32_t (&w)[B]) {
      if constexpr (B <= 3) {
#pragma unroll
        for (int k = 0; k < 8; ++k)
          by[k] += __builtin_amdgcn_perm(a.tb[1], a.tb[0], spread4<B>(bits_at<B>(w, 4 * B * k, 4 * B)));
        if (++run == a.chunk) widen();
      } else {
#pragma unroll
        for (int m = 0; m < 16; ++m) {
          const uint32_t lo = tab[bits_at<B>(w, 2 * B * m, B) & ((1u << B) - 1u)];
          const uint32_t hi = tab[bits_at<B>(w, 2 * B * m + B, B) & ((1u << B) - 1u)];
          acc[m] += lo | hi << 16;
        }
      }
    };
    for (uint32_t i0 = 0; i0 < a.n; i0 += 4) {
      uint32_t w[4][B];
#pragma unroll
      for (uint32_t u = 0; u < 4; ++u) {
        const uint32_t i = i0 + u < a.n ? i0 + u : i0;          // past the end: a load that is not used
        const uint32_t* const p = static_cast<const uint32_t*>(a.packed.p[i]) + v * B;
#pragma unroll
        for (int k = 0; k < B; ++k) {
          if constexpr (M == STREAM && B <= 3) w[u][k] = __builtin_nontemporal_load(p + k);   // wider ones share lines
          else w[u][k] = p[k];
        }
      }
#pragma unroll
      for (uint32_t u = 0; u < 4; ++u)
        if (i0 + u < a.n) add(w[u]);
    }
    if constexpr (B <= 3) widen();
  }
  store_sums32<M>(acc, a.agg_bits, a.out, v0, a.nvec, own, stage);
}

// 4-bit indices -> 8-bit sums, the paper's prototype widths (Sec. 3).  One thread owns 32 coordinates
// (16 bytes of every stream); the 16-entry table sits in four registers and is applied to four
// nibbles at a time with byte permutes; sums of four coordinates share a register (no carry can
// cross a byte because g*n <= 255).
struct AggB4Args {
  PtrArr packed;
  uint8_t* out;
  uint64_t nvec;    // d / 32
  uint32_t n;
  uint32_t tb[4];   // table bytes 0..15, little endian
};

__device__ __forceinline__ uint32_t lut16x4(uint32_t sel, const uint32_t (&tb)[4]) {
  const uint32_t s7 = sel & 0x07070707u;
  const uint32_t lo = __builtin_amdgcn_perm(tb[1], tb[0], s7);
  const uint32_t hi = __builtin_amdgcn_perm(tb[3], tb[2], s7);
  const uint32_t m = ((sel & 0x08080808u) >> 3) * 0xFFu;
  return (hi & m) | (lo & ~m);
}

template <Mem M>
__global__ __launch_bounds__(256) void k_aggregate_b4w8(const AggB4Args a) {
  __shared__ uint4 stage[M == STREAM ? 512 : 1];
  const uint32_t t = threadIdx.x;
  const uint64_t v0 = (uint64_t)blockIdx.x * 256, v = v0 + t;
  if (M == KEEP && v >= a.nvec) return;
  const uint32_t tb[4] = {a.tb[0], a.tb[1], a.tb[2], a.tb[3]};
  uint32_t ev[4] = {0, 0, 0, 0}, od[4] = {0, 0, 0, 0};
  auto load = [&](uint32_t i) { return load_u4<M>(static_cast<const uint4*>(a.packed.p[i]) + v); };
  auto add = [&](const uint4 r) {
    const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      ev[k] += lut16x4(w[k] & 0x0F0F0F0Fu, tb);          // coordinates 8k + 0, 2, 4, 6
      od[k] += lut16x4((w[k] >> 4) & 0x0F0F0F0Fu, tb);   // coordinates 8k + 1, 3, 5, 7
    }
  };
  if (v < a.nvec) {
    uint32_t i = 0;
    for (; i + 4 <= a.n; i += 4) {         // four loads in flight: a small call has few wavefronts to hide them
      uint4 r[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) r[u] = load(i + u);
#pragma unroll
      for (int u = 0; u < 4; ++u) add(r[u]);
    }
    for (; i < a.n; ++i) add(load(i));
  }
  uint32_t o[8];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    o[2 * k] = __builtin_amdgcn_perm(od[k], ev[k], 0x05010400u);
    o[2 * k + 1] = __builtin_amdgcn_perm(od[k], ev[k], 0x07030602u);
  }
  uint4* const dst = reinterpret_cast<uint4*>(a.out + v0 * 32);
  uint4* const mine = (M == STREAM ? stage : dst) + 2 * t;
  mine[0] = make_uint4(o[0], o[1], o[2], o[3]);
  mine[1] = make_uint4(o[4], o[5], o[6], o[7]);
  if constexpr (M == STREAM) {             // a wave's stores as whole lines
    __syncthreads();
    const uint64_t left = a.nvec - v0;
    const uint32_t nvec4 = 2 * (uint32_t)(left < 256 ? left : 256);
#pragma unroll
    for (uint32_t i = t; i < 512; i += 256)
      if (i < nvec4) store_u4<STREAM>(dst + i, stage[i]);
  }
}

// 2-bit indices -> 8-bit sums.  One thread owns 64 coordinates (16 bytes of every stream); the four table
// values sit in one register; field f of every byte is looked up with one byte permute, so acc[k][f] holds the
// sums of coordinates 16k + 4*byte + f, and a 4x4 byte transpose restores coordinate order at the end.
struct AggB2Args {
  PtrArr packed;
  uint8_t* out;
  uint64_t nvec;    // d / 64
  uint32_t n;
  uint32_t tb;      // table bytes 0..3, little endian
};

template <Mem M>
__global__ __launch_bounds__(256) void k_aggregate_b2w8(const AggB2Args a) {
  const uint64_t v = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (v >= a.nvec) return;
  uint32_t acc[4][4];
#pragma unroll
  for (int k = 0; k < 4; ++k)
#pragma unroll
    for (int f = 0; f < 4; ++f) acc[k][f] = 0;
  for (uint32_t i = 0; i < a.n; ++i) {
    const uint4 r = load_u4<M>(static_cast<const uint4*>(a.packed.p[i]) + v);
    const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int f = 0; f < 4; ++f) acc[k][f] += __builtin_amdgcn_perm(0u, a.tb, (w[k] >> (2 * f)) & 0x03030303u);
  }
  uint4* dst = reinterpret_cast<uint4*>(a.out + v * 64);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t p0 = __builtin_amdgcn_perm(acc[k][1], acc[k][0], 0x05010400u);   // bytes 0, 1 of fields 0, 1
    const uint32_t p1 = __builtin_amdgcn_perm(acc[k][1], acc[k][0], 0x07030602u);   // bytes 2, 3
    const uint32_t q0 = __builtin_amdgcn_perm(acc[k][3], acc[k][2], 0x05010400u);
    const uint32_t q1 = __builtin_amdgcn_perm(acc[k][3], acc[k][2], 0x07030602u);
    dst[k] = make_uint4(__builtin_amdgcn_perm(q0, p0, 0x05040100u), __builtin_amdgcn_perm(q0, p0, 0x07060302u),
                        __builtin_amdgcn_perm(q1, p1, 0x05040100u), __builtin_amdgcn_perm(q1, p1, 0x07060302u));
  }
}

// 4-bit indices -> sums of any other width W: 16 bits (g*n above 255), or the exact width ceil(log2(g n + 1)) of Sec. 8.4,
// say.  Same lookups; workers are taken in runs of `chunk` = floor(255 / g), inside which the byte-wise sums cannot carry, and
// every run is then widened into 16-bit lanes.  A thread's 32 fields make exactly W dwords, which go through LDS so that the
// workgroup writes its 1024 * W bytes as consecutive 16-byte vectors.
struct AggB4WxArgs {
  PtrArr packed;
  uint8_t* out;
  uint64_t nvec;    // d / 32
  uint32_t n, chunk;
  uint32_t tb[4];
};

//
// FOUR: four workers' loads in flight, see sums_four_loads.
template <int W, Mem M, bool FOUR>
__global__ __launch_bounds__(256) void k_aggregate_b4wx(const AggB4WxArgs a) {
  __shared__ __align__(16) uint32_t stage[256 * W];
  const int t = threadIdx.x;
  const uint64_t v0 = (uint64_t)blockIdx.x * 256;
  const uint64_t v = v0 + t;
  if (v < a.nvec) {
    const uint32_t tb[4] = {a.tb[0], a.tb[1], a.tb[2], a.tb[3]};
    uint32_t acc[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0;
    for (uint32_t i0 = 0; i0 < a.n; i0 += a.chunk) {
      const uint32_t i1 = (i0 + a.chunk < a.n) ? i0 + a.chunk : a.n;
      uint32_t ev[4] = {0, 0, 0, 0}, od[4] = {0, 0, 0, 0};
      auto load = [&](uint32_t i) { return load_u4<M>(static_cast<const uint4*>(a.packed.p[i]) + v); };
      auto add = [&](const uint4 r) {
        const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          ev[k] += lut16x4(w[k] & 0x0F0F0F0Fu, tb);
          od[k] += lut16x4((w[k] >> 4) & 0x0F0F0F0Fu, tb);
        }
      };
      uint32_t i = i0;
      if constexpr (FOUR) {
        for (; i + 4 <= i1; i += 4) {
          uint4 r[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) r[u] = load(i + u);
#pragma unroll
          for (int u = 0; u < 4; ++u) add(r[u]);
        }
      }
      for (; i < i1; ++i) add(load(i));
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        acc[4 * k + 0] += __builtin_amdgcn_perm(od[k], ev[k], 0x0C040C00u);
        acc[4 * k + 1] += __builtin_amdgcn_perm(od[k], ev[k], 0x0C050C01u);
        acc[4 * k + 2] += __builtin_amdgcn_perm(od[k], ev[k], 0x0C060C02u);
        acc[4 * k + 3] += __builtin_amdgcn_perm(od[k], ev[k], 0x0C070C03u);
      }
    }
    // field e = coordinate e of the thread's 32: low or high half of acc[e / 2]; bits [e W, e W + W) of the output
    uint32_t out[W];
#pragma unroll
    for (int k = 0; k < W; ++k) out[k] = 0;
#pragma unroll
    for (int e = 0; e < 32; ++e) {
      const uint32_t f = (e & 1) ? acc[e >> 1] >> 16 : acc[e >> 1] & 0xFFFFu;
      const int pos = e * W, k = pos >> 5, sh = pos & 31;
      out[k] |= f << sh;
      if (sh + W > 32) out[k + 1] |= f >> (32 - sh);
    }
#pragma unroll
    for (int k = 0; k < W; ++k) stage[t * W + k] = out[k];
  }
  __syncthreads();
  const uint64_t left = a.nvec - v0;                       // threads of this workgroup that own coordinates
  const uint32_t nvec4 = (uint32_t)(left < 256 ? left : 256) * W / 4;   // a multiple of 8 W / 4: nvec is a multiple of 32
  uint4* dst = reinterpret_cast<uint4*>(a.out + v0 * 4 * W);
  const uint4* src = reinterpret_cast<const uint4*>(stage);
  for (uint32_t i = t; i < nvec4; i += 256) store_u4<M>(dst + i, src[i]);
}

}  // namespace thc
