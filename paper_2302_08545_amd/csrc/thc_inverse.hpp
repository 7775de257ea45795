// Inverse transform passes: decompression and the error-feedback update (Alg. 2 / Alg. 3).
#pragma once

#include "thc_forward.hpp"

namespace thc {

// ---------------------------------------------------------------------------------------------
// Sixteen consecutive codes (table indices or aggregated sums) of `bits` bits each, starting at
// coordinate j (a multiple of 16): codes_load fetches the raw words (for the widths with a fast path)
// or the decoded fields (any other width); codes_decode finishes the fast paths.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ void codes_load(const uint8_t* s8, uint32_t bits, uint64_t j, uint32_t (&w)[8],
                                           uint32_t (&y)[16]) {
  if (bits == 8) {
    const uint4 r = *reinterpret_cast<const uint4*>(s8 + j);
    w[0] = r.x; w[1] = r.y; w[2] = r.z; w[3] = r.w;
  } else if (bits == 16) {
    const uint4 r0 = *reinterpret_cast<const uint4*>(s8 + 2 * j);
    const uint4 r1 = *reinterpret_cast<const uint4*>(s8 + 2 * j + 16);
    w[0] = r0.x; w[1] = r0.y; w[2] = r0.z; w[3] = r0.w; w[4] = r1.x; w[5] = r1.y; w[6] = r1.z; w[7] = r1.w;
  } else if (bits == 4) {
    const uint2 r = *reinterpret_cast<const uint2*>(s8 + (j >> 1));
    w[0] = r.x; w[1] = r.y;
  } else if (bits == 2) {
    w[0] = *reinterpret_cast<const uint32_t*>(s8 + (j >> 2));
  } else if (bits == 1) {
    w[0] = *reinterpret_cast<const uint16_t*>(s8 + (j >> 3));
  } else {   // any other width: eight fields take `bits` bytes
    uint32_t z0[8], z1[8];
    load_fields8(s8 + (j >> 3) * bits, bits, z0);
    load_fields8(s8 + ((j >> 3) + 1) * bits, bits, z1);
#pragma unroll
    for (int e = 0; e < 8; ++e) { y[e] = z0[e]; y[8 + e] = z1[e]; }
  }
}

// Sixteen W-bit fields out of a staged bit stream: they start at `first`, or 16 bits into it (`half`).  W is a
// compile-time constant so that every field's word and shift are; one dword of slack is read past the fields.
template <int W>
__device__ __forceinline__ void cut16(const uint32_t* first, bool half, uint32_t (&y)[16]) {
  constexpr int NW = (16 * W + 31) / 32;          // dwords the fields span when they start on a boundary
  uint32_t d[NW + 1];
#pragma unroll
  for (int k = 0; k <= NW; ++k) d[k] = first[k];
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

// widths that codes_load / codes_decode take straight from global memory
__device__ __forceinline__ bool codes_fast_width(uint32_t bits) {
  return bits == 8 || bits == 16 || bits == 4 || bits == 2 || bits == 1;
}

__device__ __forceinline__ void codes_decode(uint32_t bits, bool ok, const uint32_t (&w)[8], uint32_t (&y)[16]) {
  if (bits == 8) {
#pragma unroll
    for (int e = 0; e < 16; ++e) y[e] = (w[e >> 2] >> (8 * (e & 3))) & 255u;
  } else if (bits == 16) {
#pragma unroll
    for (int e = 0; e < 16; ++e) y[e] = (w[e >> 1] >> (16 * (e & 1))) & 0xFFFFu;
  } else if (bits == 4) {
#pragma unroll
    for (int e = 0; e < 16; ++e) y[e] = (w[e >> 3] >> (4 * (e & 7))) & 15u;
  } else if (bits == 2) {
#pragma unroll
    for (int e = 0; e < 16; ++e) y[e] = (w[0] >> (2 * e)) & 3u;
  } else if (bits == 1) {
#pragma unroll
    for (int e = 0; e < 16; ++e) y[e] = (w[0] >> e) & 1u;
  } else if (!ok) {
#pragma unroll
    for (int e = 0; e < 16; ++e) y[e] = 0;
  }
}

// ---------------------------------------------------------------------------------------------
// Inverse "lo" pass.  Source is either the aggregated stream (decompression, Alg. 2:
// m + (Y/n)(M-m)/g = Y * step_n - M) or one worker's packed indices (error feedback, Alg. 3:
// X_i = m + T[z](M-m)/g = T[z] * step_g - M).  One thread loads 16 consecutive coordinates.
// ---------------------------------------------------------------------------------------------
struct InvLoArgs {
  PtrArr src;              // per vector of the launch (grid.y): aggregated stream or packed indices
  const float* range_M;
  const float* range_m;    // or null: m = -M
  float* ws_x;             // d floats per vector of the launch, written
  uint64_t d;
  uint32_t L;
  uint32_t src_bits;       // bits per coordinate in src
  uint32_t use_table;      // 1: src holds table indices; 0: src holds aggregated table values
  uint32_t divisor;        // g*n (aggregated) or g (indices)
  TileMap tm;
  uint8_t table[256];
};

template <int N = NT>          // threads, 16 values each
struct alignas(16) SmemInvLo {
  float lds[16 * N];
  float sM[8], sStep[8];
  float tabf[256];
};

// One tile of N threads: the one at coordinate `off` of the launch's vector `vec`; put(o, value) takes each result, o its
// offset from the tile's first coordinate.  TABLE: the codes are table indices, else sums.  SB is their width where the launch
// knows it, or 0: a.src_bits says.
template <int L1, bool XO, int SB, bool TABLE, int N = NT, class A, class Put>
__device__ __forceinline__ void inv_lo_stages(const A& a, uint64_t off, uint32_t vec, SmemInvLo<N>& sm, Put&& put) {
  static_assert(!XO || (L1 == LOG_TILE && N == NT), "the row-split tile needs blocks of at least 2^16");
  constexpr bool GUARD = (1 << L1) < 16 * N;
  float* const lds = sm.lds;
  float* const sM = sm.sM;
  float* const sStep = sm.sStep;
  float* const tabf = sm.tabf;

  const int t = threadIdx.x;
  const int idx = 16 * t;
  const uint64_t j = off + lo_map<XO>(idx);
  const bool ok = !GUARD || j < a.d;
  const uint8_t* const src = static_cast<const uint8_t*>(a.src.p[vec]);
  const uint32_t bits = SB ? SB : a.src_bits;

  // raw bits first, so the load is in flight while the block constants are prepared
  uint32_t entry = 0;
  if (TABLE && t < 256) entry = a.table[t];
  uint32_t w[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  uint32_t y[16];
  const bool staged = !codes_fast_width(bits);
  if (!staged) {
    if (ok) codes_load(src, bits, j, w, y);
  } else {
    // Any other width: the tile's runs of 1024 codes (128 * bits bytes each, dword aligned) are copied
    // into the still unused tile buffer with coalesced loads; every thread then cuts its sixteen fields out.
    uint32_t* stage = reinterpret_cast<uint32_t*>(lds);
    const uint32_t per_row = 32u * bits;                             // dwords per 1024 codes: fewer than NT
    if ((uint32_t)t < per_row) {
      constexpr uint32_t RUNS = 16 * N / 1024;
      uint32_t val[RUNS];
#pragma unroll
      for (uint32_t r = 0; r < RUNS; ++r) {
        const uint64_t jr = off + lo_map<XO>(1024u * r);             // first coordinate of the run
        val[r] = 0;
        if (!GUARD || jr < a.d)                                      // runs exist whole or not at all: 1024 divides d
          val[r] = reinterpret_cast<const uint32_t*>(src + (jr >> 3) * bits)[t];
      }
#pragma unroll
      for (uint32_t r = 0; r < RUNS; ++r) stage[r * per_row + t] = val[r];
    }
  }

  // A tile inside one block looks up values on the block's range; one of several blocks looks up the table's own values.
  constexpr bool SCALED = TABLE && !GUARD;
  const int nblk = GUARD ? (16 * N) >> a.L : 1;
  if (SCALED ? t < (SB ? 1 << SB : 256) : t < nblk) {
    const uint64_t blk = (off >> a.L) + (SCALED ? 0 : t);
    float M = 0.f, m = 0.f;
    if (blk < (a.d >> a.L)) { M = a.range_M[blk]; m = lower_of(a.range_m, blk, M); }
    const float step = (float)(((double)M - (double)m) / (double)a.divisor);
    if constexpr (SCALED) {
      tabf[t] = (float)entry * step + m;
    } else {
      sM[t] = m;                                                     // the affine map only needs the lower end
      sStep[t] = step;
    }
  }
  if (TABLE && !SCALED && t < 256) tabf[t] = (float)entry;
  __syncthreads();

  if (!staged) {
    codes_decode(bits, ok, w, y);
  } else {
    // sixteen fields start at bit 16 * (field number / 16) * bits of the run: on a dword boundary or in its middle
    const uint32_t* stage = reinterpret_cast<const uint32_t*>(lds);
    const uint32_t pos = (uint32_t)(idx & 1023) * bits;
    const uint32_t* first = stage + (uint32_t)(idx >> 10) * 32u * bits + (pos >> 5);
    switch (bits) {
#define THC_CUT(W) case W: cut16<W>(first, (pos & 16u) != 0, y); break;
      THC_CUT(3) THC_CUT(5) THC_CUT(6) THC_CUT(7) THC_CUT(9) THC_CUT(10) THC_CUT(11) THC_CUT(12) THC_CUT(13)
      THC_CUT(14) THC_CUT(15)
#undef THC_CUT
      default: break;
    }
    if (!ok) {
#pragma unroll
      for (int e = 0; e < 16; ++e) y[e] = 0;
    }
    __syncthreads();                                                 // every field is out before the tile is written
  }
  const int bt = GUARD ? (idx >> a.L) : 0;
  float lo = 0.f, step = 0.f;
  if constexpr (!SCALED) { lo = sM[bt]; step = sStep[bt]; }
  float v[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const float f = TABLE ? tabf[y[e]] : (float)y[e];
    v[e] = SCALED ? f : ok ? f * step + lo : 0.f;
  }
  bfly<4>(v);
#pragma unroll
  for (int e = 0; e < 16; e += 4)
    *reinterpret_cast<float4*>(&lds[swz(idx + e)]) = make_float4(v[e], v[e + 1], v[e + 2], v[e + 3]);

  lds_stages<4, L1, true, SWZ, N>(lds, t, [&](int base, int eoff, float val) { put(lo_map<XO>(base) + lo_map<XO>(eoff), val); });
}

template <bool XO, int SB, bool TABLE, Mem M, class A>
__device__ __forceinline__ void inv_lo_tile(const A& a, uint32_t tile, uint32_t vec, float* dst_vec, SmemInvLo<>& sm) {
  const uint64_t off = tm_base(a.tm, tile);
  float* const dst = dst_vec + off;
  inv_lo_stages<LOG_TILE, XO, SB, TABLE>(a, off, vec, sm, [&](uint32_t o, float val) { store_f<M>(&dst[o], val); });
}

// What bounds it: writing 4 bytes a coordinate (plain writes to HBM reach 5.7 TB/s here).  M: how they are stored, see
// through_inverse: 4 x 2^26 coordinates from 8-bit sums 210 us, where 2^28 in one launch with plain stores took 210 and left the next
// pass 410 instead of 324.  Decoding is a large part of its
// instructions, so the widths and sources that rounds use have instantiations of their own: 2^28 coordinates from 8-bit
// sums 251 -> 231 us, from 4-bit indices, whose values are looked up on the block's range, 268 -> 245 us; one block of
// 2^20 from 4-bit indices 5.4 -> 4.3 us.
template <bool XO, int SB, bool TABLE, Mem M>
__global__ __launch_bounds__(NT, 8) void k_inv_lo(const InvLoArgs a) {
  __shared__ SmemInvLo<> sm;
  inv_lo_tile<XO, SB, TABLE, M>(a, blockIdx.x, blockIdx.y, a.ws_x + (uint64_t)blockIdx.y * a.d, sm);
}

// ---------------------------------------------------------------------------------------------
// Inverse "hi" pass: finish H, scale by 1/sqrt(B), apply the diagonal (Sec. 5.1: RHT^-1 = D H / sqrt(d)).
// mode 0: out = result (Alg. 3, the global update);
// mode 1: e <- (grad + e) - result (Alg. 3, error-feedback update), out = ef buffer, read and written.
// ---------------------------------------------------------------------------------------------
struct InvHiArgs {
  const float* x;      // half-rotated vectors, d floats per vector of the launch (grid.y)
  PtrArr out;          // per vector: d floats
  PtrArr grad;         // per vector, mode 1 only
  uint64_t d;
  uint64_t j0;         // global coordinate of x[0] (a multiple of B), for the diagonal's random stream
  TileMap tm;
  uint32_t round, k0, k1;
  uint32_t mode, bf16;
  float c;
  Walk walk;           // the last of the arguments: see there
};

// scale by 1/sqrt(B) and apply the diagonal; mode 1: (x + e) - that
template <class A>
__device__ __forceinline__ float4 inv_finish4(float4 v, uint32_t bits, const A& a, float4 x, float4 e) {
  v.x = flip(v.x * a.c, bits & 1u);
  v.y = flip(v.y * a.c, (bits >> 1) & 1u);
  v.z = flip(v.z * a.c, (bits >> 2) & 1u);
  v.w = flip(v.w * a.c, (bits >> 3) & 1u);
  if (a.mode == 1) {
    x.x += e.x; x.y += e.y; x.z += e.z; x.w += e.w;
    v = make_float4(x.x - v.x, x.y - v.y, x.z - v.z, x.w - v.w);
  }
  return v;
}

struct alignas(16) SmemInvHi {
  float lds[TILE];
  uint32_t sgn[TILE / 32];
};

// One tile: tile index `tile` of the launch's vector `vec`, whose half-rotated image starts at xv.  OUT: how results are stored, see
// keep_estimate.
template <int R, Mem OUT, class A>
__device__ __forceinline__ void inv_hi_tile(const A& a, uint32_t tile, uint32_t vec, const float* xv,
                                            SmemInvHi& sm) {
  float* const lds = sm.lds;
  uint32_t* const sgn = sm.sgn;

  const int t = threadIdx.x;
  const HiGeom<R> g(tile, a.tm);
  float* const out = static_cast<float*>(const_cast<void*>(a.out.p[vec]));
  const void* const grad = a.grad.p[vec];

  float4 x[4];
  hi_issue_loads<R, hi_mem<R>()>(xv, g, t, x);
  // the diagonal's bits while the loads travel
  // 32 consecutive tile indices are 32 consecutive coordinates, or, with 16-wide rows, two aligned halves
  if (t < TILE / 32) {
    if constexpr (HiGeom<R>::W >= 32) {
      sgn[t] = sign_word(a.j0 + g.coord(32 * t), a.round, a.k0, a.k1);
    } else {
      const uint64_t j0 = a.j0 + g.coord(32 * t), j1 = a.j0 + g.coord(32 * t + 16);
      const uint32_t lo = sign_word(j0 & ~31ull, a.round, a.k0, a.k1) >> (j0 & 31);
      const uint32_t hi = sign_word(j1 & ~31ull, a.round, a.k0, a.k1) >> (j1 & 31);
      sgn[t] = (lo & 0xFFFFu) | (hi << 16);
    }
  }
  hi_r0_to_lds<R>(x, lds, t);
  hi_round1<R>(lds, t);
  // error-feedback update: the gradient and the buffer's old contents are all requested before anything is stored (the
  // stores go to that same buffer), and while the tile's last stage runs
  float4 gx[4], ex[4];
  if (a.mode == 1) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint64_t j = g.coord(4 * (t + NT * i));
      gx[i] = a.bf16 ? load_grad4<true>(grad, j) : load_grad4<false>(grad, j);
      ex[i] = *reinterpret_cast<const float4*>(out + j);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) gx[i] = ex[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  float4 v[4];
  hi_back4<R>(lds, t, v);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int idx = 4 * (t + NT * i);
    const uint32_t bits = sgn[idx >> 5] >> (idx & 31);
    store_f4<OUT>(out + g.coord(idx), inv_finish4(v[i], bits, a, gx[i], ex[i]));
  }
}

template <int R, Mem OUT>
__global__ __launch_bounds__(NT) void k_inv_hi(const InvHiArgs a) {
  __shared__ SmemInvHi sm;
  const uint32_t tile = walk_x(a.walk), vec = walk_y(a.walk);
  inv_hi_tile<R, OUT>(a, tile, vec, a.x + (uint64_t)vec * a.d, sm);
}

// ---------------------------------------------------------------------------------------------
// Blocks that fit one workgroup (2^10 to 2^14 here, 2^14 and 2^15 in thc_big.hpp): the whole inverse transform in one
// launch.  What bounds the two passes is bytes and, in small calls, launches: the intermediate's 8 bytes per
// coordinate and one launch go.  Rounds of 8 workers with error feedback: 4096 blocks of 2^13 2031 -> 1505 us, 512 blocks
// of 2^15 999 -> 764 us; one block of 2^14 without it 36 -> 25 us.  Calls back to back are faster at every size.  A call
// that is waited for is not with up to 16 blocks of 2^14 or 2^15, where one workgroup's chain is longer than two short
// launches of several (2^15: 20.5 -> 21.0 us, with error feedback 32.3 -> 33.5); from 32 blocks on it is (22.6 -> 21.5).
// ---------------------------------------------------------------------------------------------
// `N` results of a thread: scale, diagonal, and with EFM 1 / 2 (binary32 / bf16 gradient) e <- (grad + e) - that.  All
// operands are requested before the first store, which goes to the buffer some of them come from.
template <int EFM, Mem OUT, int N, class Off, class Bit>
__device__ __forceinline__ void finish_values(const float (&v)[N], float c, float* out, const void* grad, Off&& off,
                                              Bit&& bit) {
  float x[N], e[N];
  if constexpr (EFM != 0) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      x[i] = EFM == 2 ? bf16_to_f32(static_cast<const uint16_t*>(grad)[off(i)]) : static_cast<const float*>(grad)[off(i)];
      e[i] = out[off(i)];
    }
  }
#pragma unroll
  for (int i = 0; i < N; ++i) {
    float r = flip(v[i] * c, bit(i));
    if constexpr (EFM != 0) r = (x[i] + e[i]) - r;
    store_f<OUT>(&out[off(i)], r);
  }
}

struct InvWholeArgs {
  InvLoArgs lo;      // ws_x unused
  PtrArr out;        // per vector: d floats
  PtrArr grad;       // per vector, EFM only
  uint64_t j0;
  uint32_t round, k0, k1;
  float c;
};

constexpr int inv_whole_threads(int L) { return L <= LOG_TILE ? NT : 1 << (L - 4); }

// SB as for k_inv_lo: 2^28 coordinates in blocks of 2^13 from 8-bit sums 285 -> 260 us.
template <int L1, int SB, int EFM, Mem OUT = STREAM>
__global__ __launch_bounds__(inv_whole_threads(L1), EFM == 0 ? 8 : 4) void k_inv_whole(const InvWholeArgs a) {
  constexpr int N = inv_whole_threads(L1), T = 16 * N;
  constexpr bool PART = (1 << L1) < T;     // several blocks to a tile: the vector's last one may be partly empty
  __shared__ SmemInvLo<N> sm;
  __shared__ __align__(16) uint32_t sgn[T / 32];
  const int t = threadIdx.x;
  const uint32_t vec = blockIdx.y, tile = blockIdx.x;
  const uint64_t off = N == NT ? tm_base(a.lo.tm, tile) : (uint64_t)xcd_tile<2>(tile, gridDim.x) * T;
  if (t < T / 128) {
    const uint64_t q = (a.j0 + off + 128u * t) >> 7;
    *reinterpret_cast<uint4*>(&sgn[4 * t]) = philox4x32_10((uint32_t)q, (uint32_t)(q >> 32), a.round, SIGN_STREAM, a.k0, a.k1);
  }
  float v[16];
  uint32_t at[16];
  int c = 0;
  inv_lo_stages<L1, false, SB, EFM != 0, N>(a.lo, off, vec, sm, [&](uint32_t o, float val) { v[c] = val; at[c] = o; ++c; });
  float* const out = static_cast<float*>(const_cast<void*>(a.out.p[vec])) + off;
  const char* const grad = EFM ? static_cast<const char*>(a.grad.p[vec]) + off * (EFM == 2 ? 2 : 4) : nullptr;
  const uint64_t left = a.lo.d - off;
  auto bit = [&](uint32_t o) { return (sgn[o >> 5] >> (o & 31)) & 1u; };
  if (!PART || left >= T) {
    finish_values<EFM, OUT>(v, a.c, out, grad, [&](int i) { return at[i]; }, [&](int i) { return bit(at[i]); });
  } else {           // the last tile of a vector of short blocks
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (at[i] >= left) continue;
      const float one[1] = {v[i]};
      finish_values<EFM, OUT>(one, a.c, out, grad, [&](int) { return at[i]; }, [&](int) { return bit(at[i]); });
    }
  }
}

}  // namespace thc
