// Device-side helpers of libbct: 16-byte vector access, storage-dtype
// conversion and wavefront (64-lane) reductions for gfx950.
#ifndef BCT_DEVICE_H
#define BCT_DEVICE_H

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bct {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

struct F32 {
  typedef float elem;
  static constexpr int kElemsPerVec = 4;  // elements in one 16-byte vector
};
struct BF16 {
  typedef uint16_t elem;
  static constexpr int kElemsPerVec = 8;
};

// 16 bytes of storage -> E floats (exact widening).
template <typename DT>
__device__ __forceinline__ void unpack16(const u32x4 v, float* f);

template <>
__device__ __forceinline__ void unpack16<F32>(const u32x4 v, float* f) {
  f[0] = __uint_as_float(v.x);
  f[1] = __uint_as_float(v.y);
  f[2] = __uint_as_float(v.z);
  f[3] = __uint_as_float(v.w);
}
template <>
__device__ __forceinline__ void unpack16<BF16>(const u32x4 v, float* f) {
  f[0] = __uint_as_float(v.x << 16);
  f[1] = __uint_as_float(v.x & 0xFFFF0000u);
  f[2] = __uint_as_float(v.y << 16);
  f[3] = __uint_as_float(v.y & 0xFFFF0000u);
  f[4] = __uint_as_float(v.z << 16);
  f[5] = __uint_as_float(v.z & 0xFFFF0000u);
  f[6] = __uint_as_float(v.w << 16);
  f[7] = __uint_as_float(v.w & 0xFFFF0000u);
}

// Two floats -> two bf16 in one word, round-to-nearest-even (the hardware
// conversion of gfx950: v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  bf16x2 r;
  r.x = (__bf16)lo;
  r.y = (__bf16)hi;
  return __builtin_bit_cast(uint32_t, r);
}

// E floats -> 16 bytes of storage, rounding to the storage dtype; the floats
// are overwritten with the stored (rounded) values so that a later read uses
// exactly what the cache now holds.
template <typename DT>
__device__ __forceinline__ u32x4 pack16_round(float* f);

template <>
__device__ __forceinline__ u32x4 pack16_round<F32>(float* f) {
  u32x4 v;
  v.x = __float_as_uint(f[0]);
  v.y = __float_as_uint(f[1]);
  v.z = __float_as_uint(f[2]);
  v.w = __float_as_uint(f[3]);
  return v;
}
template <>
__device__ __forceinline__ u32x4 pack16_round<BF16>(float* f) {
  u32x4 v;
  v.x = pack_bf16x2(f[0], f[1]);
  v.y = pack_bf16x2(f[2], f[3]);
  v.z = pack_bf16x2(f[4], f[5]);
  v.w = pack_bf16x2(f[6], f[7]);
  unpack16<BF16>(v, f);
  return v;
}

// One float -> storage element (used by the small epilogues).
__device__ __forceinline__ void store_elem(float* p, size_t i, float v) { p[i] = v; }
__device__ __forceinline__ void store_elem(uint16_t* p, size_t i, float v) {
  p[i] = __builtin_bit_cast(uint16_t, (__bf16)v);
}
__device__ __forceinline__ float load_elem(const float* p, size_t i) { return p[i]; }
__device__ __forceinline__ float load_elem(const uint16_t* p, size_t i) {
  return __uint_as_float((uint32_t)p[i] << 16);
}

// 16 bytes per lane from memory (an address per lane) to LDS at lds + 16 * lane, lds the same in every lane; no trip
// through registers.  Counts as an outstanding vector-memory operation until the bytes are in LDS.
__device__ __forceinline__ void load_to_lds(const void* g, void* lds) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)g,
                                   (__attribute__((address_space(3))) void*)lds, 16, 0, 0);
}
// BYTES (16 or 4) per lane to LDS at lds + BYTES * lane, lds the same in every lane: from base, the same in every lane, +
// offset bytes; or from an address per lane.  Written out because the compiler takes its own instruction for an access to
// LDS in flight and answers it with a wait for all LDS reads before the next use of one, and adds the offset to a 64-bit
// address in vector registers.  It counts as an outstanding vector-memory operation, which the compiler does not know:
// whoever requests waits for it (wait_vm); the compiler's own waits only become stricter by it.  The LDS address is an
// operand bound to m0, so the compiler sets it.  Nor does the compiler know the distances that the load needs: 1 wait
// state from a write of m0, 5 from a vector instruction that writes its scalar base (v_readfirstlane, a spilled register's
// v_readlane).  So the load takes a copy of the base, made here by the scalar unit, which needs no distance on either
// side and is the one instruction after m0 as well.  (s_nop 4 instead: write-only chunk of B = 32, H = 32, M = 4096, T = 512
// 2200 us against 2180.)
template <int BYTES = 16>
__device__ __forceinline__ void lds_request(const void* base, uint32_t offset, void* lds) {
  static_assert(BYTES == 16 || BYTES == 4, "one of two instructions");
  const uint32_t to = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds;
  const void* from;
  if constexpr (BYTES == 4)
    asm volatile("s_mov_b64 %0, %2\n\tglobal_load_lds_dword %1, %0" : "=&s"(from) : "v"(offset), "s"(base), "{m0}"(to) : "memory");
  else
    asm volatile("s_mov_b64 %0, %2\n\tglobal_load_lds_dwordx4 %1, %0" : "=&s"(from) : "v"(offset), "s"(base), "{m0}"(to) : "memory");
}
__device__ __forceinline__ void lds_request(const void* lane_address, void* lds) {
  const uint32_t to = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds;
  asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(lane_address), "{m0}"(to) : "memory");
}
// A barrier that waits for nothing else: requests into LDS stay in flight across it.
__device__ __forceinline__ void bare_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
}
// s_waitcnt operands: at most n vector-memory operations outstanding / no LDS operation outstanding.  The counter has six
// bits: a wavefront keeps at most kMostVm operations outstanding.
constexpr int kMostVm = 63;
constexpr int wait_vm(int n) { return (n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14); }
constexpr int kWaitLds = 15 | (7 << 4) | (0 << 8) | (3 << 14);

// The workgroup's LDS writes so far are there for all its wavefronts; vector-memory operations stay in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_s_waitcnt(kWaitLds);
  bare_barrier();
}

template <int I>
struct Int {
  static constexpr int v = I;
};

// The memory a workgroup of a unit_grid launch works on (see bct_internal.h).
__device__ __forceinline__ uint32_t block_unit() { return blockIdx.z * 32768u + blockIdx.y; }

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Butterfly reductions over the lanes whose ids differ in the bits of `mask`
// (a contiguous range of bits given as lowest and highest xor distance).
// The butterfly visits partners in a fixed order, so results are reproducible.
//
// A butterfly that starts at distance 1 takes its partners at distances 1, 2, 4 and 8 through the
// data-parallel-primitive path of the vector ALU (no trip through the LDS crossbar that a general
// lane exchange makes): distances 1 and 2 are quad permutations; at distance 4 every quad already
// holds one value, so the lane 7 - i of the half row (row_half_mirror) holds what lane i ^ 4 holds,
// and at distance 8 the lane 15 - i of the row (row_mirror) holds what lane i ^ 8 holds.  Same
// operands in the same order as the plain butterfly, so the same bits.
template <int CTRL>
__device__ __forceinline__ float dpp_partner(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
template <int LO, int O>
__device__ __forceinline__ float xor_partner(float v) {
  if constexpr (LO == 1 && O == 1) return dpp_partner<0xB1>(v);        // quad_perm [1, 0, 3, 2]
  else if constexpr (LO == 1 && O == 2) return dpp_partner<0x4E>(v);   // quad_perm [2, 3, 0, 1]
  else if constexpr (LO == 1 && O == 4) return dpp_partner<0x141>(v);  // row_half_mirror
  else if constexpr (LO == 1 && O == 8) return dpp_partner<0x140>(v);  // row_mirror
  else return __shfl_xor(v, O, 64);
}
template <int LO, int HI>
__device__ __forceinline__ float xor_sum(float v) {
  v += xor_partner<LO, LO>(v);
  if constexpr (2 * LO <= HI) v += xor_partner<LO, 2 * LO>(v);
  if constexpr (4 * LO <= HI) v += xor_partner<LO, 4 * LO>(v);
  if constexpr (8 * LO <= HI) v += xor_partner<LO, 8 * LO>(v);
  if constexpr (16 * LO <= HI) v += xor_partner<LO, 16 * LO>(v);
  if constexpr (32 * LO <= HI) v += xor_partner<LO, 32 * LO>(v);
  return v;
}
template <int LO, int HI>
__device__ __forceinline__ float xor_max(float v) {
  v = fmaxf(v, xor_partner<LO, LO>(v));
  if constexpr (2 * LO <= HI) v = fmaxf(v, xor_partner<LO, 2 * LO>(v));
  if constexpr (4 * LO <= HI) v = fmaxf(v, xor_partner<LO, 4 * LO>(v));
  if constexpr (8 * LO <= HI) v = fmaxf(v, xor_partner<LO, 8 * LO>(v));
  if constexpr (16 * LO <= HI) v = fmaxf(v, xor_partner<LO, 16 * LO>(v));
  if constexpr (32 * LO <= HI) v = fmaxf(v, xor_partner<LO, 32 * LO>(v));
  return v;
}

// The value that lane L of this lane's row of 16 holds (a data-parallel-primitive move, no LDS crossbar).
template <int L>
__device__ __forceinline__ float row_lane(float v) {
  return dpp_partner<0x150 + L>(v);   // row_newbcast
}

// Scores of 16 key rows against up to 16 query rows on v_mfma_f32_16x16x32_bf16, D the head dimension.  key: this
// lane's key row (row l % 16 of the 16), query: this lane's query row (column l % 16), both already advanced
// to the lane's 8 inputs at 8 * (l / 16).  Element v of the result: key row 4 * (l / 16) + v, query row l % 16.
// The statistics pass and the MV pass both call this, so a score has the same bits in both.
template <int D>
__device__ __forceinline__ f32x4 score16(const u32x4* key, const u32x4* query) {
  f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < D / 32; ++ks)
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, key[ks]), __builtin_bit_cast(bf16x8, query[ks]),
                                                c, 0, 0, 0);
  return c;
}

// out[g][column] += sum over slots of weight[g][slot] * MV[slot][column] on v_mfma_f32_16x16x32_bf16, for eight slots of
// every lane.  raw: the lane's 16-byte chunk (8 columns) of its eight consecutive slots.  Lane l is row / column c = l % 16 of
// the operands and their eight entries 8 * (l / 16) of the contraction.
// LPS = 16 lanes to a slot row: the contraction runs over the wavefront's 32 slots; operand e, a transposition in the lane,
// is element e of chunk c.  acc[e], element v of a lane: query head 4 * (l / 16) + v, column 8 c + e.
// LPS = 8: lanes l and l ^ 8 hold the same chunk of different slots.  They exchange halves, so that lanes c < 8 have
// elements 0 to 3 and lanes c >= 8 elements 4 to 7 of both groups of slots: two contractions over 32 slots, part j the
// slots of lanes with l / 8 % 2 = j.  acc[e]: column 8 (c % 8) + 4 (c / 8) + e.
// w: per part the weights of head c for the slots 8 * (l / 16) .. of the part, as N bf16 addends (split_weights).
template <int LPS>
struct ReadShape {
  static constexpr int kParts = 16 / LPS, kProducts = LPS / 2;
  static __device__ __forceinline__ uint32_t column(uint32_t c) { return LPS == 16 ? 8 * c : 8 * (c % 8) + 4 * (c / 8); }
};
template <int N>
__device__ __forceinline__ f32x4 mfma_addends(const u32x4* w, u32x4 b, f32x4 c) {
#pragma unroll
  for (int n = 0; n < N; ++n)
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[n]), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  return c;
}
template <int LPS, int N>
__device__ __forceinline__ void mfma_read(const u32x4* raw, const u32x4 (*w)[N], f32x4* acc) {
  // element e % 2 of word w of the eight slots
  auto operand = [](const uint32_t* x, int odd) -> u32x4 {
    u32x4 t;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      t[i] = odd ? ((x[2 * i] >> 16) | (x[2 * i + 1] & 0xFFFF0000u)) : ((x[2 * i] & 0xFFFFu) | (x[2 * i + 1] << 16));
    return t;
  };
  if constexpr (LPS == 16) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      uint32_t x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] = raw[u][e / 2];
      acc[e] = mfma_addends<N>(w[0], operand(x, e % 2), acc[e]);
    }
  } else {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      // row_ror:8 is the lane l ^ 8; the bank mask names the lanes that take from it, the others keep their own word
      uint32_t a[8], b[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        a[u] = (uint32_t)__builtin_amdgcn_update_dpp((int)raw[u][k], (int)raw[u][2 + k], 0x128, 0xF, 0xC, false);
        b[u] = (uint32_t)__builtin_amdgcn_update_dpp((int)raw[u][2 + k], (int)raw[u][k], 0x128, 0xF, 0x3, false);
      }
#pragma unroll
      for (int o = 0; o < 2; ++o) {
        acc[2 * k + o] = mfma_addends<N>(w[0], operand(a, o), acc[2 * k + o]);
        acc[2 * k + o] = mfma_addends<N>(w[1], operand(b, o), acc[2 * k + o]);
      }
    }
  }
}
// Eight fp32 weights as N bf16 operands that add up to them.  N = 2: the weights' roundings and what those left, rounded: 16 to
// 17 bits.  N = 3: the upper, middle and lower eight bits, cut off, so nothing is lost: a product of them is the fp32 product before
// its rounding.  There no addend of a weight is zero (2^-30 of it at least), so that an infinity in MV is read as one, not as 0 * inf.
template <int N>
__device__ __forceinline__ void split_weights(const float* w, u32x4* out) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float a = w[2 * i], b = w[2 * i + 1];
    if constexpr (N == 2) {
      const uint32_t h = pack_bf16x2(a, b);
      out[0][i] = h;
      out[1][i] = pack_bf16x2(a - __uint_as_float(h << 16), b - __uint_as_float(h & 0xFFFF0000u));
    } else {
      auto top = [](float x) -> float { return __uint_as_float(__float_as_uint(x) & 0xFFFF0000u); };
      auto pack = [](float x, float y) -> uint32_t { return (__float_as_uint(x) >> 16) | (__float_as_uint(y) & 0xFFFF0000u); };
      constexpr float kLeast = 1.0f / (1 << 30);
      const float la = a * kLeast, lb = b * kLeast, ra = a - top(a), rb = b - top(b);
      const float ma = top(fmaxf(ra, la)), mb = top(fmaxf(rb, lb));
      out[0][i] = pack(a, b);
      out[1][i] = pack(ma, mb);
      out[2][i] = pack(fmaxf(ra - ma, la), fmaxf(rb - mb, lb));
    }
  }
}

// One wavefront merges the per-tile (max, sum of exp2(score - max)) pairs of a row, up to 128 of them (lane l
// takes tiles l and l + 64), into the row's (max, sum).  The operations and their order are those of
// normalise_kernel, so both give the same bits.
struct TileStats {
  float2 a, c;
};
__device__ __forceinline__ TileStats load_tile_stats(const float2* st, uint32_t n_tiles, uint32_t lane) {
  TileStats t = {make_float2(-INFINITY, 0.f), make_float2(-INFINITY, 0.f)};
  if (lane < n_tiles) t.a = st[lane];
  if (lane + 64 < n_tiles) t.c = st[lane + 64];
  return t;
}
__device__ __forceinline__ float2 merge_tile_stats(const TileStats& t) {
  const float mx = xor_max<1, 32>(fmaxf(t.a.x, t.c.x));
  float sm = t.a.y * fast_exp2(t.a.x - mx);
  sm += t.c.y * fast_exp2(t.c.x - mx);
  return make_float2(mx, xor_sum<1, 32>(sm));
}
__device__ __forceinline__ float2 merge_tile_stats(const float2* st, uint32_t n_tiles, uint32_t lane) {
  return merge_tile_stats(load_tile_stats(st, n_tiles, lane));
}
constexpr uint32_t kMaxMergedTiles = 128;

}  // namespace bct

#endif
