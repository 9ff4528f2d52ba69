// Chunked prefill of libbct for bf16 caches (gfx950, MFMA).
//
// A chunk of T tokens is T decode steps in token order with MV carried in fp32
// through the chunk.  Because MK is static, the write weights ww_t do not
// depend on MV, so the recurrence unrolls into dense contractions (section 3.5,
// "Optimized for Parallelism": the per-token updates are independent and can be
// accumulated concurrently):
//     WW = softmax_rows(write_scale * WQ . MK^T)   [T x M]
//     RW = softmax_rows(read_scale  * Q  . MK^T)   [T*G x M]
//     MV_end   = round(MV_start + WW^T . WV)                       (section 3.4 eq., summed over t)
//     out_t    = RW_t . (MV_start + sum_{s<=t} ww_s^T wv_s)         (read after the token's own write)
// A chunk of few tokens is one pass over MK and MV (prefill_pass_kernel).  Otherwise tokens are grouped in sub-chunks of 128.
// For sub-chunk c,
//     out_c = RW_c . MV_c + tril(RW_c . WW_c^T) . WV_c,   MV_c = MV at the start of the sub-chunk,
// where the state kernel, which walks the sub-chunks in order with its MV tile
// in fp32 registers, leaves MV_c (rounded to bf16, as an MFMA operand has to be)
// in the workspace.  Launches: transpose (WV) -> stats (write rows) -> state -> read (all
// sub-chunks, the read rows normalised on the fly); a chunk that only reads: transpose (MV) -> stats
// (read rows) -> read.
//
// All matrix products use v_mfma_f32_32x32x16_bf16, whose operands are rows along the contraction index
// (C[i][j] += sum_k A[i][k] B[j][k]); the accumulator of lane l holds column j = l % 32 and rows
// i = 8*(v/4) + 4*(l/32) + v%4.  Operands that are contracted the other way than they lie in memory (MV over slots, WV
// over tokens) are kept in the workspace as operand tiles (below), in the order in which a lane's accumulator
// registers become the next product's operand.  Tiles come to LDS by lds_request, one or two tiles ahead,
// and LDS reads are issued a region ahead of the products that use them.
//
// Precision: scores in fp32 from exact bf16 products; softmax weights are
// rounded to bf16 as MFMA operands for the reads; for the state they are split
// into hi + lo bf16 parts (two MFMAs), 16 to 17 bits, so that the stored MV is within one rounding of the
// decode step's.
#include "bct_device.h"
#include "bct_internal.h"

namespace bct {

namespace {

constexpr int kTC = 128;          // tokens per sub-chunk = rows per tile
constexpr float kNegBig = -1e30f;  // stands in for -inf in running maxima
constexpr uint32_t kMaxStatsSplit = 8;  // shares of the keys in a statistics launch
constexpr float kNoRow = 1e30f;    // shift of a row that does not exist: exp2(score - kNoRow) = 0

__device__ __forceinline__ f32x16 mfma_bf16(const bf16x8 a, const bf16x8 b, const f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ bf16x8 frag(const uint16_t* tile, int ld, int row, int k) {
  return *(const bf16x8*)(tile + row * ld + k);
}
__device__ __forceinline__ f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int v = 0; v < 16; ++v) z[v] = 0.f;
  return z;
}
__device__ __forceinline__ uint16_t bf16_bits(float x) { return __builtin_bit_cast(uint16_t, (__bf16)x); }
__device__ __forceinline__ float bf16_val(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// Global -> LDS tile copies in two halves, so that the loads of the next tile
// can be in flight while the current one is used: fetch() issues all of a
// thread's 16-byte loads into registers, put() writes them to LDS.
// A tile is NROWS rows of NCOLS bf16; thread t handles 16-byte chunk t % CPR of
// rows t / CPR, t / CPR + RPP, ... of a workgroup of NT threads
template <int NROWS, int NCOLS, int NT = 256>
struct Tile {
  static constexpr int CPR = NCOLS / 8, RPP = NT / CPR, N = NROWS / RPP;
  static_assert(NROWS % RPP == 0, "whole passes");
  u32x4 v[N];
  uint32_t missing = 0;  // bit i: row i of this thread is a zero row

  // rowptr(r): address of row r, or nullptr for a zero row.  A missing row is a
  // load from `safe` (any valid 16-byte aligned address) whose result put()
  // replaces by zeros: the loads carry no branches, and nothing touches the
  // loaded registers until put(), so the loads stay in flight across the
  // products of the current tile.
  template <typename F>
  __device__ __forceinline__ void fetch_rows(const uint16_t* safe, F rowptr) {
    const int ch = threadIdx.x % CPR, r0 = threadIdx.x / CPR;
    missing = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const uint16_t* src = rowptr(r0 + i * RPP);
      const bool ok = src != nullptr;
      v[i] = *(const u32x4*)((ok ? src : safe) + (ok ? ch * 8 : 0));
      missing |= ok ? 0u : (1u << i);
    }
  }
  // rows at src + r * src_ld, all present
  __device__ __forceinline__ void fetch_block(const uint16_t* src, size_t src_ld) {
    const int ch = threadIdx.x % CPR, r0 = threadIdx.x / CPR;
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = *(const u32x4*)(src + (size_t)(r0 + i * RPP) * src_ld + ch * 8);
    missing = 0;
  }
  __device__ __forceinline__ void put(uint16_t* dst, int ld) const {
    const int ch = threadIdx.x % CPR, r0 = threadIdx.x / CPR;
#pragma unroll
    for (int i = 0; i < N; ++i)
      *(u32x4*)(dst + (r0 + i * RPP) * ld + ch * 8) = ((missing >> i) & 1u) ? (u32x4){0u, 0u, 0u, 0u} : v[i];
  }
};
__device__ __forceinline__ void store4_bf16(uint16_t* dst, float a, float b, float c, float d) {
  uint2 w;
  w.x = pack_bf16x2(a, b);
  w.y = pack_bf16x2(c, d);
  *(uint2*)dst = w;
}

__device__ __forceinline__ void merge_stat(float& m, float& s, float mo, float so) {
  const float mn = fmaxf(m, mo);
  s = s * fast_exp2(m - mn) + so * fast_exp2(mo - mn);
  m = mn;
}

}  // namespace

// ------------------------------------------------------------------ operand tiles and key tiles

// A matrix contracted over its ROWS (slots of MV, tokens of WV), stored as tiles of 16 rows x 32 columns in the order
// a lane of v_mfma_f32_32x32x16_bf16 holds them, with the rows in the order in which a product's accumulator
// hands its own rows on: lane l = column l % 32, half h = l / 32, its 8 elements are the rows
// 4 h + {0, 1, 2, 3} and 8 + 4 h + {0, 1, 2, 3} of the 16.  A lane's accumulator registers 8 j .. 8 j + 7 (rows
// 8 (v / 4) + 4 h + v % 4), packed to bf16, then ARE an operand of the next product: weights and states go
// from product to product without leaving the registers or through LDS as whole 16-byte chunks.
// Chunk index of (row group of 16, column group of 32, lane) in a matrix of D columns.
template <int D>
__device__ __forceinline__ size_t operand_chunk(uint32_t g16, uint32_t c32, uint32_t lane) {
  return ((size_t)g16 * (D / 32) + c32) * 64 + lane;
}
__device__ __forceinline__ bf16x8 pack8(const f32x16& a, int j) {
  return __builtin_bit_cast(bf16x8, (u32x4){pack_bf16x2(a[8 * j + 0], a[8 * j + 1]), pack_bf16x2(a[8 * j + 2], a[8 * j + 3]),
                                            pack_bf16x2(a[8 * j + 4], a[8 * j + 5]), pack_bf16x2(a[8 * j + 6], a[8 * j + 7])});
}

// Rows contracted along their own elements (keys, write queries), and MV on its way in and out, lie in LDS row after
// row, the 16-byte chunk c of row r at position c ^ swizzle(r) of the row.  So a load instruction brings whole rows (4 of
// 256 bytes): neighbouring lanes ask for neighbouring chunks.  The address unit takes four such lanes a cycle, 64 bytes;
// of lanes that ask in the order of an operand, each for another row, one: a 64-slot tile of keys took 1024 cycles of it, a
// third of what the read kernel needs for the tile, and 256 in whole rows.
template <int D>
__device__ __forceinline__ int swizzle(int r) {
  return D == 128 ? r % 16 : (r / 2) % 8;
}
// Instructions are not moved across.
__device__ __forceinline__ void region() { __builtin_amdgcn_sched_barrier(0); }

template <int D>
struct RowTile {
  static constexpr int CPR = D / 8;        // chunks per row
  static constexpr int RPL = 64 / CPR;     // rows per load instruction
  // load instruction n of a tile: this lane's row and chunk
  static __device__ __forceinline__ int row(int n, int lane) { return n * RPL + lane / CPR; }
  static __device__ __forceinline__ int chunk(int n, int lane) { return (lane % CPR) ^ swizzle<D>(row(n, lane)); }
  // byte offset of that chunk from the instruction's first row, rows in memory one after another
  static __device__ __forceinline__ uint32_t source(int n, int lane) { return (uint32_t)((lane / CPR) * D * 2 + chunk(n, lane) * 16); }
  // this lane's operand ks (row lane % 32 of 32, elements 16 ks + 8 (lane / 32) ..) of 32 rows at `rows`: 16 lanes
  // read 16 different chunk columns, no two in one bank.  at: operand_at(lane).  The exclusive or is opaque: the compiler
  // would keep its D / 16 results in registers.
  static __device__ __forceinline__ uint32_t operand_at(int lane) {
    return (uint32_t)((lane % 32) * D * 2 + ((lane / 32) ^ swizzle<D>(lane % 32)) * 16);
  }
  static __device__ __forceinline__ bf16x8 operand(const uint16_t* rows, int ks, uint32_t at) {
    uint32_t a = at;
    if (ks) asm volatile("v_xor_b32 %0, %1, %2" : "=v"(a) : "n"(32 * ks), "v"(at));
    return *(const bf16x8*)((const char*)rows + a);
  }
};

// max over the two lanes l, l ^ 32 (v_permlane32_swap: no LDS crossbar)
__device__ __forceinline__ float max_of_halves(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// ------------------------------------------------------------------ transposes

// MFMA operands must run along the contraction index, and two of them do not in memory: WV [token][column] is
// contracted over tokens and MV [slot][column] over slots.  Once per chunk:
//   which = 0:  WVt[unit], WV as operand tiles (see operand_chunk; tokens >= T zero-filled up to Tpad)
//   which = 1:  snap[0][unit][column][slot] = MV, for a chunk that only reads
// One workgroup transposes 64 rows through LDS.
template <int D>
__global__ __launch_bounds__(256) void prefill_transpose_kernel(const PrefillParams p, int which) {
  constexpr int LD = D + 8;
  __shared__ __attribute__((aligned(16))) uint16_t sT[64 * LD];
  const uint32_t unit = block_unit();
  if (unit >= p.B * p.Hkv) return;
  const uint32_t b = unit / p.Hkv, h = unit % p.Hkv;
  const uint32_t r0 = blockIdx.x * 64;
  const uint32_t rows = which == 0 ? p.Tpad : p.M;
  {
    Tile<64, D> t;
    t.fetch_rows(p.mv, [&](int r) -> const uint16_t* {
      if (which == 0) return r0 + r < p.T ? p.wv + (((size_t)b * p.T + r0 + r) * p.Hkv + h) * D : nullptr;
      return p.mv + ((size_t)unit * p.M + r0 + r) * D;
    });
    if (which == 0 && p.gate) {
      // A negative step size eta_t (section 3.5 reading: MV += eta_t ww^T wv) flips the sign of token t's row of
      // WV here, which is exact; the statistics kernel folds |eta_t| into the token's shift.
#pragma unroll
      for (int i = 0; i < Tile<64, D>::N; ++i) {
        const uint32_t tk = r0 + threadIdx.x / Tile<64, D>::CPR + i * Tile<64, D>::RPP;
        const uint32_t flip = tk < p.T && p.gate[((size_t)b * p.T + tk) * p.Hkv + h] < 0.f ? 0x80008000u : 0u;
        t.v[i] ^= (u32x4){flip, flip, flip, flip};
      }
    }
    t.put(sT, LD);
  }
  __syncthreads();
  if (which == 0) {
    uint16_t* dst = p.wvt + ((size_t)unit * rows + r0) * D;
    // thread -> (column j, the 8 tokens of an operand lane)
    for (int i = threadIdx.x; i < D * 8; i += 256) {
      const int lane = i % 64, tile = i / 64, half = lane / 32;
      const int j = 32 * (tile % (D / 32)) + lane % 32, t8 = 16 * (tile / (D / 32)) + 4 * half;
      uint32_t e[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) e[k] = sT[(t8 + (k / 4) * 8 + k % 4) * LD + j];
      *(u32x4*)(dst + (size_t)i * 8) = (u32x4){e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16)};
    }
    return;
  }
  uint16_t* dst = p.snap + (size_t)unit * D * rows + r0;
  // thread -> (column j, 8 consecutive rows)
  for (int i = threadIdx.x; i < D * 8; i += 256) {
    const int j = i / 8, rr = (i % 8) * 8;
    u32x4 v;
    v.x = (uint32_t)sT[(rr + 0) * LD + j] | ((uint32_t)sT[(rr + 1) * LD + j] << 16);
    v.y = (uint32_t)sT[(rr + 2) * LD + j] | ((uint32_t)sT[(rr + 3) * LD + j] << 16);
    v.z = (uint32_t)sT[(rr + 4) * LD + j] | ((uint32_t)sT[(rr + 5) * LD + j] << 16);
    v.w = (uint32_t)sT[(rr + 6) * LD + j] | ((uint32_t)sT[(rr + 7) * LD + j] << 16);
    *(u32x4*)(dst + (size_t)j * rows + rr) = v;
  }
}

// ------------------------------------------------------------------ stats

// Row statistics of the score matrix: for each write row (token t) and read
// row (token t, query head g) of a memory, the shift max + log2(sum of
// exp2(score - max)) over all M slots, so that a weight is exp2(score - shift)
// with no further multiplication (rows that do not exist use kNoRow, which makes every weight zero).
// One workgroup = 128 rows; it walks its share of the keys 128 slots at a time; each of its eight wavefronts
// scores 32 slots of the tile against 64 of the rows.  Bound by the vector work for the exponentials (32 per lane
// and tile against 16 matrix instructions); the products of a tile are issued in between the exponentials of
// the one before, and the keys are requested into LDS two tiles ahead.
// A launch with few rows splits the keys over p.stats_split workgroups and leaves their (max, sum) pairs in
// p.stats_part for prefill_stats_merge_kernel.
__device__ __forceinline__ void store_shift(const PrefillParams& p, uint32_t unit, uint32_t b, uint32_t h, uint32_t nw,
                                            uint32_t nr, uint32_t row, float m, float s) {
  if (row < nw) {
    // a step size eta scales the token's write weights: exp2(score - shift) * |eta|
    // = exp2(score - (shift - log2 |eta|)); eta = 0 gives shift = +inf and weights 0
    // (|eta| here; the sign of eta rides on the token's row of WV^T, see prefill_transpose_kernel)
    const float le = p.gate ? __log2f(fabsf(p.gate[((size_t)b * p.T + row) * p.Hkv + h])) : 0.f;
    p.norm_w[(size_t)unit * p.T + row] = m + __log2f(s) - le;
  } else if (row - nw < nr) {
    p.norm_r[(size_t)unit * p.T * p.G + (row - nw)] = m + __log2f(s);
  }
}

template <int D>
__global__ __launch_bounds__(512, 2) void prefill_stats_kernel(const PrefillParams p) {
  typedef RowTile<D> RT;
  constexpr int KS = D / 16;
  constexpr int kTile = 128 * D;           // elements of a key tile
  constexpr int NL = kTile / 512 / 8;      // its load instructions per wavefront
  __shared__ __attribute__((aligned(16))) uint16_t sK0[kTile], sK1[kTile], sK2[kTile];
  __shared__ float2 sRed[4][kTC];

  // launch order: all sequences of one KV head, then the next head, so that the workgroups in flight
  // share one head's keys (1 MB at M = 4096) in each XCD's L2 instead of cycling through all heads
  const uint32_t uy = block_unit();
  if (uy >= p.B * p.Hkv) return;
  const uint32_t h = uy / p.B, b = uy % p.B, unit = b * p.Hkv + h;
  const uint32_t nw = p.has_write ? p.T : 0u, nr = (p.has_read && p.stats_read) ? p.T * p.G : 0u;
  const uint32_t row0 = blockIdx.x / p.stats_split * kTC, part = blockIdx.x % p.stats_split;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64, col = lane % 32, half = lane / 32;
  // wavefront = (32 slots sg of the key tile, 64 rows rh of the row tile)
  const int sg = wave & 3, rh = wave >> 2;
  // this workgroup's slots: whole tiles but for the last share, whose end may cut a tile in half
  const uint32_t tiles = (p.M + 127) / 128, tile0 = (uint32_t)((uint64_t)tiles * part / p.stats_split),
                 tile1 = (uint32_t)((uint64_t)tiles * (part + 1) / p.stats_split), n = tile1 - tile0;
  const uint16_t* mk = p.mk + (size_t)(p.mk_per_seq ? unit : h) * p.M * D;

  auto stage = [&](auto i) -> uint16_t* {
    if constexpr (decltype(i)::v % 3 == 0) return sK0;
    else if constexpr (decltype(i)::v % 3 == 1) return sK1;
    else return sK2;
  };
  // slots past the end of the memory (the second half of a last tile; M is a multiple of 64): its last 32 again
  auto request = [&](auto i, uint32_t t) {
    const uint32_t m0 = (tile0 + min(t, n - 1)) * 128;
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      const int ld = wave * NL + j, row = ld * RT::RPL;
      const uint32_t slot = min(m0 + row / 32 * 32, p.M - 32) + row % 32;
      lds_request(mk + (size_t)slot * D, RT::source(ld, lane), stage(i) + ld * 512);
    }
  };
  // The query rows come the same way, once per workgroup, through the stage that the keys need last (the wavefronts'
  // own loads of them, four times over and before the keys' requests: 91 us on 1890 workgroups of three tiles, so 72;
  // B = 32, H = 32, M = 4096, T = 512 755 against 720).  They do not change over the loop: their operand fragments stay
  // in registers.  Rows past the end: the last row again, never stored.
  const uint32_t nrows = nw + nr;
#pragma unroll
  for (int j = 0; j < NL; ++j) {
    const int ld = wave * NL + j;
    const uint32_t row = min(row0 + (uint32_t)RT::row(ld, lane), nrows - 1), rr = row - nw;
    const uint16_t* src = row < nw ? p.wq + (((size_t)b * p.T + row) * p.Hkv + h) * D
                                   : p.q + (((size_t)b * p.T + rr / p.G) * p.Hq + h * p.G + rr % p.G) * D;
    lds_request(src + RT::chunk(ld, lane) * 8, sK2 + ld * 512);
  }
  // the waits count requests from the last one back: rows, first keys, second keys stay in this order
  region();
  request(Int<0>{}, 0);
  region();
  request(Int<1>{}, 1);
  region();
  __builtin_amdgcn_s_waitcnt(wait_vm(2 * NL));
  bare_barrier();
  // A negative scale is moved into the row itself (negating bf16 is exact), so that below the
  // largest raw score is also the largest scaled one and the scaling can ride in the exponent's fma.
  const uint32_t at = RT::operand_at(lane);
  float scale[2], m[2], s[2];
  bf16x8 xb[2][KS];
#pragma unroll
  for (int jt = 0; jt < 2; ++jt) {
    scale[jt] = row0 + 64 * rh + 32 * jt + col < nw ? p.wscale_l2e : p.rscale_l2e;
    m[jt] = kNegBig;
    s[jt] = 0.f;
    const uint32_t flip = scale[jt] < 0.f ? 0x80008000u : 0u;
    scale[jt] = fabsf(scale[jt]);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      xb[jt][ks] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, RT::operand(sK2 + (2 * rh + jt) * 32 * D, ks, at)) ^
                                                  (u32x4){flip, flip, flip, flip});
  }
  __builtin_amdgcn_s_waitcnt(kWaitLds);
  f32x16 acc[2][2];   // [tile parity][row group]
  // The products of a tile, and between them the exponentials of the tile before (from its maximum on: m is already
  // what it has to be).  OLD: there is a tile before.
  auto tile = [&](auto i, auto par, auto old, uint32_t t) {
    constexpr int P = decltype(par)::v;
    request(Int<decltype(i)::v + 2>{}, t + 2);
    bf16x8 f[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) f[ks] = RT::operand(stage(i) + sg * 32 * D, ks, at);
    acc[P][0] = zero16();
    acc[P][1] = zero16();
    float add[2] = {0.f, 0.f};
    region();
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
      for (int jt = 0; jt < 2; ++jt) acc[P][jt] = mfma_bf16(f[ks], xb[jt][ks], acc[P][jt]);
      if constexpr (decltype(old)::v != 0) {
#pragma unroll
        for (int v = ks * (16 / KS); v < (ks + 1) * (16 / KS); ++v)
#pragma unroll
          for (int jt = 0; jt < 2; ++jt) add[jt] += fast_exp2(__builtin_fmaf(acc[1 - P][jt][v], scale[jt], -m[jt]));
      }
      region();
    }
#pragma unroll
    for (int jt = 0; jt < 2; ++jt) {
      s[jt] += add[jt];
      float tmax = acc[P][jt][0];
#pragma unroll
      for (int v = 1; v < 16; ++v) tmax = fmaxf(tmax, acc[P][jt][v]);
      const float mn = fmaxf(m[jt], tmax * scale[jt]);   // of slots that come twice as well: the same maximum
      s[jt] *= fast_exp2(m[jt] - mn);
      m[jt] = mn;
    }
    __builtin_amdgcn_s_waitcnt(kWaitLds);
    __builtin_amdgcn_s_waitcnt(wait_vm(NL));   // the next tile has arrived, the one after it is in flight
    bare_barrier();
  };
  __builtin_amdgcn_s_waitcnt(wait_vm(NL));   // the first keys have arrived; every wavefront has its rows
  bare_barrier();
  tile(Int<0>{}, Int<0>{}, Int<0>{}, 0);
  uint32_t t = 1;
  for (; t + 6 <= n; t += 6) {
    tile(Int<1>{}, Int<1>{}, Int<1>{}, t);
    tile(Int<2>{}, Int<0>{}, Int<1>{}, t + 1);
    tile(Int<0>{}, Int<1>{}, Int<1>{}, t + 2);
    tile(Int<1>{}, Int<0>{}, Int<1>{}, t + 3);
    tile(Int<2>{}, Int<1>{}, Int<1>{}, t + 4);
    tile(Int<0>{}, Int<0>{}, Int<1>{}, t + 5);
  }
  if (t < n) tile(Int<1>{}, Int<1>{}, Int<1>{}, t);
  if (t + 1 < n) tile(Int<2>{}, Int<0>{}, Int<1>{}, t + 1);
  if (t + 2 < n) tile(Int<0>{}, Int<1>{}, Int<1>{}, t + 2);
  if (t + 3 < n) tile(Int<1>{}, Int<0>{}, Int<1>{}, t + 3);
  if (t + 4 < n) tile(Int<2>{}, Int<1>{}, Int<1>{}, t + 4);
  // the exponentials of the last tile (parity (n - 1) % 2); a wavefront whose slots of it lie outside has none
  if ((tile1 - 1) * 128 + 32 * sg < p.M) {
#pragma unroll
    for (int jt = 0; jt < 2; ++jt)
#pragma unroll
      for (int v = 0; v < 16; ++v)
        s[jt] += fast_exp2(__builtin_fmaf((n & 1) ? acc[0][jt][v] : acc[1][jt][v], scale[jt], -m[jt]));
  }
  __builtin_amdgcn_s_waitcnt(wait_vm(0));
#pragma unroll
  for (int jt = 0; jt < 2; ++jt) {
    merge_stat(m[jt], s[jt], __shfl_xor(m[jt], 32, 64), __shfl_xor(s[jt], 32, 64));
    if (half == 0) sRed[sg][64 * rh + 32 * jt + col] = make_float2(m[jt], s[jt]);
  }
  __syncthreads();
  if (threadIdx.x < kTC) {
    float mm = sRed[0][threadIdx.x].x, ss = sRed[0][threadIdx.x].y;
#pragma unroll
    for (int w = 1; w < 4; ++w) merge_stat(mm, ss, sRed[w][threadIdx.x].x, sRed[w][threadIdx.x].y);
    const uint32_t row = row0 + threadIdx.x;
    if (p.stats_split == 1) store_shift(p, unit, b, h, nw, nr, row, mm, ss);
    else if (row < nw + nr) p.stats_part[((size_t)unit * p.stats_split + part) * (nw + nr) + row] = make_float2(mm, ss);
  }
}

// The same for few slots and many workgroups: one key tile at a time through registers, which leaves room for two
// workgroups per compute unit, one of which starts or ends while the other multiplies (see launch_prefill_bf16).
template <int D>
__global__ __launch_bounds__(512, 4) void prefill_stats_short_kernel(const PrefillParams p) {
  constexpr int LD = D + 8, KS = D / 16, NT = 512;
  // the query tile is only read into registers before the loop: the key tiles reuse its memory
  __shared__ __attribute__((aligned(16))) uint16_t sTile[128 * LD];
  __shared__ float2 sRed[4][kTC];
  uint16_t* const sX = sTile;
  uint16_t* const sK = sTile;

  const uint32_t uy = block_unit();
  if (uy >= p.B * p.Hkv) return;
  const uint32_t h = uy / p.B, b = uy % p.B, unit = b * p.Hkv + h;
  const uint32_t nw = p.has_write ? p.T : 0u, nr = (p.has_read && p.stats_read) ? p.T * p.G : 0u;
  const uint32_t row0 = blockIdx.x * kTC;
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, col = lane % 32, half = lane / 32;
  // wavefront = (32 slots sg of the key tile, 64 rows rh of the row tile)
  const int sg = wave & 3, rh = wave >> 2;

  {
    Tile<kTC, D, NT> t;
    t.fetch_rows(p.mk, [&](int r) -> const uint16_t* {
      uint32_t row = row0 + r;
      if (row < nw) return p.wq + (((size_t)b * p.T + row) * p.Hkv + h) * D;
      row -= nw;
      if (row < nr) return p.q + (((size_t)b * p.T + row / p.G) * p.Hq + h * p.G + row % p.G) * D;
      return nullptr;
    });
    t.put(sX, LD);
  }
  const uint16_t* mk = p.mk + (size_t)(p.mk_per_seq ? unit : h) * p.M * D;

  float scale[2], m[2], s[2];
#pragma unroll
  for (int jt = 0; jt < 2; ++jt) {
    scale[jt] = (row0 + 64 * rh + 32 * jt + col < nw) ? p.wscale_l2e : p.rscale_l2e;
    m[jt] = kNegBig;
    s[jt] = 0.f;
  }
  // the query rows do not change over the loop: keep their operand fragments in registers.
  // A negative scale is moved into the row itself (negating bf16 is exact), so that below the
  // largest raw score is also the largest scaled one and the scaling can ride in the exponent's fma.
  __syncthreads();
  bf16x8 xb[2][KS];
#pragma unroll
  for (int jt = 0; jt < 2; ++jt) {
    const uint32_t flip = scale[jt] < 0.f ? 0x80008000u : 0u;
    scale[jt] = fabsf(scale[jt]);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      u32x4 v = __builtin_bit_cast(u32x4, frag(sX, LD, 64 * rh + 32 * jt + col, ks * 16 + half * 8));
      v ^= (u32x4){flip, flip, flip, flip};
      xb[jt][ks] = __builtin_bit_cast(bf16x8, v);
    }
  }
  Tile<128, D, NT> tk;
  auto fetch_keys = [&](uint32_t m0) {
    tk.fetch_rows(p.mk, [&](int r) -> const uint16_t* { return (m0 + r < p.M) ? mk + (size_t)(m0 + r) * D : nullptr; });
  };
  fetch_keys(0);
  for (uint32_t m0 = 0; m0 < p.M; m0 += 128) {
    __syncthreads();
    tk.put(sK, LD);
    if (m0 + 128 < p.M) fetch_keys(m0 + 128);  // in flight during this tile's products
    __syncthreads();
    if (m0 + 32 * sg < p.M) {  // M is a multiple of 64: a wavefront's 32 slots are all in or all out
      f32x16 acc[2];
#pragma unroll
      for (int jt = 0; jt < 2; ++jt) acc[jt] = zero16();
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const bf16x8 a = frag(sK, LD, 32 * sg + col, ks * 16 + half * 8);
#pragma unroll
        for (int jt = 0; jt < 2; ++jt) acc[jt] = mfma_bf16(a, xb[jt][ks], acc[jt]);
      }
#pragma unroll
      for (int jt = 0; jt < 2; ++jt) {
        float tmax = acc[jt][0];
#pragma unroll
        for (int v = 1; v < 16; ++v) tmax = fmaxf(tmax, acc[jt][v]);
        const float mn = fmaxf(m[jt], tmax * scale[jt]);
        float add = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) add += fast_exp2(__builtin_fmaf(acc[jt][v], scale[jt], -mn));
        s[jt] = s[jt] * fast_exp2(m[jt] - mn) + add;
        m[jt] = mn;
      }
    }
  }
#pragma unroll
  for (int jt = 0; jt < 2; ++jt) {
    merge_stat(m[jt], s[jt], __shfl_xor(m[jt], 32, 64), __shfl_xor(s[jt], 32, 64));
    if (half == 0) sRed[sg][64 * rh + 32 * jt + col] = make_float2(m[jt], s[jt]);
  }
  __syncthreads();
  if (threadIdx.x < kTC) {
    float mm = sRed[0][threadIdx.x].x, ss = sRed[0][threadIdx.x].y;
#pragma unroll
    for (int w = 1; w < 4; ++w) merge_stat(mm, ss, sRed[w][threadIdx.x].x, sRed[w][threadIdx.x].y);
    store_shift(p, unit, b, h, nw, nr, row0 + threadIdx.x, mm, ss);
  }
}

// The shares of a split statistics launch, merged in their order.
__global__ __launch_bounds__(256) void prefill_stats_merge_kernel(const PrefillParams p) {
  const uint32_t unit = block_unit();
  if (unit >= p.B * p.Hkv) return;
  const uint32_t nw = p.has_write ? p.T : 0u, nr = (p.has_read && p.stats_read) ? p.T * p.G : 0u;
  const uint32_t row = blockIdx.x * 256 + threadIdx.x;
  if (row >= nw + nr) return;
  const float2* part = p.stats_part + (size_t)unit * p.stats_split * (nw + nr) + row;
  float2 v[kMaxStatsSplit];   // requested together
#pragma unroll
  for (uint32_t k = 0; k < kMaxStatsSplit; ++k) v[k] = part[(size_t)min(k, p.stats_split - 1) * (nw + nr)];
  float m = v[0].x, s = v[0].y;
#pragma unroll
  for (uint32_t k = 1; k < kMaxStatsSplit; ++k)
    if (k < p.stats_split) merge_stat(m, s, v[k].x, v[k].y);
  store_shift(p, unit, unit / p.Hkv, unit % p.Hkv, nw, nr, row, m, s);
}

// ------------------------------------------------------------------ read of a chunk that does not write

// Output rows of one tile of 128 read rows (row rho of the tile = token rho / G, query head rho % G)
// when MV does not change over the chunk:  out = RW . MV,  with the rows' shifts from the statistics
// kernel.  The workgroup walks the M slots 64 at a time, recomputing the score tiles.  Eight wavefronts:
// for the scores each takes 32 rows x 32 slots of the tile, for the product 32 output rows x d/2 value
// columns.
template <int D>
__global__ __launch_bounds__(512) void prefill_read_only_kernel(const PrefillParams p) {
  constexpr int NT = 512;
  constexpr int LD = D + 8, KS = D / 16;
  constexpr int LP = 64 + 8;    // row length of tiles contracted over 64 slots
  __shared__ __attribute__((aligned(16))) uint16_t sXr[kTC * LD];
  __shared__ __attribute__((aligned(16))) uint16_t sBuf[64 * LD + D * LP + kTC * LP];
  uint16_t* const sK = sBuf;
  uint16_t* const sVt = sK + 64 * LD;
  uint16_t* const sPr = sVt + D * LP;

  // launch order: all sequences of one KV head, then the next head, so that the workgroups in flight
  // share one head's keys (1 MB at M = 4096) in each XCD's L2 instead of cycling through all heads
  const uint32_t uy = block_unit();
  if (uy >= p.B * p.Hkv) return;
  const uint32_t h = uy / p.B, b = uy % p.B, unit = b * p.Hkv + h;
  const uint32_t G = p.G, T = p.T;
  const uint32_t c = p.c_begin + blockIdx.x / G, gp = blockIdx.x % G;
  const uint32_t t0 = c * kTC, rho0 = gp * kTC;
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, col = lane % 32, half = lane / 32;

  {
    Tile<kTC, D, NT> t;
    t.fetch_rows(p.mk, [&](int r) -> const uint16_t* {
      const uint32_t rho = rho0 + r, tk = t0 + rho / G;
      return tk < T ? p.q + (((size_t)b * T + tk) * p.Hq + h * G + rho % G) * D : nullptr;
    });
    t.put(sXr, LD);
  }
  const uint16_t* mk = p.mk + (size_t)(p.mk_per_seq ? unit : h) * p.M * D;
  const uint16_t* mvt = p.snap + (size_t)unit * p.M * D;   // MV, transposed: [column][slot]

  // score step: wavefront = (slot half si, row group rj of 32); lane column = row
  const int si = wave & 1, rj = wave >> 1;
  float nrm_r;
  {
    const uint32_t rho = rho0 + 32 * rj + col, t = t0 + rho / G;
    nrm_r = t < T ? p.norm_r[(size_t)unit * T * G + (size_t)t * G + rho % G] : kNoRow;
  }
  // product step: wavefront = (32 output rows, half of the value columns)
  constexpr int NOC = D / 64;                      // 32-column tiles per wavefront in the output product
  const int orow = 32 * (wave & 3), ocol = 32 * NOC * (wave >> 2);
  f32x16 oacc[NOC];
#pragma unroll
  for (int jt = 0; jt < NOC; ++jt) oacc[jt] = zero16();

  // the query rows do not change over the loop: keep their operand fragments in registers
  __syncthreads();
  bf16x8 xr[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) xr[ks] = frag(sXr, LD, 32 * rj + col, ks * 16 + half * 8);
  Tile<64, D, NT> tk;
  Tile<D, 64, NT> tv;
  tk.fetch_block(mk, D);
  tv.fetch_block(mvt, p.M);
  for (uint32_t m0 = 0; m0 < p.M; m0 += 64) {
    __syncthreads();
    tk.put(sK, LD);
    tv.put(sVt, LP);
    if (m0 + 64 < p.M) {  // next tiles, in flight during this tile's products
      tk.fetch_block(mk + (size_t)(m0 + 64) * D, D);
      tv.fetch_block(mvt + m0 + 64, p.M);
    }
    __syncthreads();
    {
      f32x16 sr = zero16();
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) sr = mfma_bf16(frag(sK, LD, 32 * si + col, ks * 16 + half * 8), xr[ks], sr);
      const int r = 32 * rj + col;
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        float e[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) e[i] = fast_exp2(sr[4 * q4 + i] * p.rscale_l2e - nrm_r);
        store4_bf16(sPr + r * LP + 32 * si + 8 * q4 + 4 * half, e[0], e[1], e[2], e[3]);
      }
    }
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const int k = ks * 16 + half * 8;
      const bf16x8 a = frag(sPr, LP, orow + col, k);
#pragma unroll
      for (int jt = 0; jt < NOC; ++jt) oacc[jt] = mfma_bf16(a, frag(sVt, LP, ocol + 32 * jt + col, k), oacc[jt]);
    }
  }

#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const uint32_t r = orow + 8 * (v / 4) + 4 * half + (v % 4);
    const uint32_t rho = rho0 + r, t = t0 + rho / G;
    if (t < T) {
      uint16_t* o = p.out + (((size_t)b * T + t) * p.Hq + h * G + rho % G) * D;
#pragma unroll
      for (int jt = 0; jt < NOC; ++jt) o[ocol + 32 * jt + col] = bf16_bits(oacc[jt][v]);
    }
  }
}

// ------------------------------------------------------------------ read of a chunk that writes

// The read of a chunk that also writes, without a statistics pass over the read rows: the softmax of a
// read row is normalised at the end, out = (sum_m e_m MV_c[m] + sum_s A'[s] wv_s) / sum_m e_m with
// e_m = exp2(score_m - shift), and the shift follows the row's running maximum lazily - it moves only
// when a tile's maximum exceeds it by more than kTau (the weights then reach at most 2^kTau, far inside
// bf16 and fp32 range), which after the first tile is rare, so rescaling what has been accumulated is a
// seldom-taken branch of one wavefront.  The write rows keep their shifts from the statistics kernel
// (the state kernel needs those before it can add anything to MV).
// Output rows of one tile of 128 read rows of sub-chunk c:
//     out = RW . MV_c  +  mask(RW . WW_c^T) . WV_c ,  mask: write token s <= the row's token.
// The workgroup walks the M slots 64 at a time.  Of its eight wavefronts four are readers and four writers, one of
// each on a SIMD.  A writer owns 32 write tokens: it scores them against the tile and leaves their weights in
// LDS as operand tiles.  A reader owns 32 read rows: every product has its rows as the columns (lane = read
// row), so its weights pass from the score product to the next ones in registers, a row's shift, sum and rescaling
// factor are the lane's own, and what is accumulated (32 rows x d columns and 32 rows x 128 tokens) never
// needs another wavefront.  The writers are one tile ahead; one barrier per tile.  Keys and MV_c come through LDS,
// requested two tiles ahead without a trip through registers.
// What bounds it: the SIMD that has most to multiply (d = 128: a writer 16 products a tile, a reader 32 and 4 for each group of
// 32 tokens it can read, so 52, 56, 60 and 64 for G = 1; the barrier waits for the 64), and that a reader and a writer share
// its issue slots.  A tile of 64 slots is up to 2048 cycles of matrix instructions
// beside 1300 cycles of vector instructions, and the older wavefront always goes first; it takes 3050 cycles at
// 1.65 GHz (B = 32, H = 32, M = 4096, T = 512: 2100 us) and as many at 2.1 GHz (192 workgroups of one round, 33 tiles: 59).  A
// reader alone takes 2700.  Before, keys came as operand tiles (see RowTile), every wavefront requested its share, a
// reader kept one operand in scratch and the sum's terms until after the products: 3300 cycles, 2270 us, 67.  The
// requests are the writers' because the address unit takes a request in 16 cycles and holds up whoever asks (which of them:
// see `idle`).  Built, right
// and not kept, us for the two sizes: a block's weights between the next 32 slots' score products 2220, 65; operands from
// LDS a region earlier 2180, 65; writers with a higher priority 3720 cycles a tile; requests after the scores 3940.
// The rows leave whole (see the end): 8-byte pieces of 32 rows a store and a token group's operands when they were needed took
// 1.5 us more of a workgroup (B = 45, Hkv = 21, M = 320, T = 166, five tiles: 296 us for the chunk, now 286).
template <int D>
__global__ __launch_bounds__(512, 2) void prefill_read_online_kernel(const PrefillParams p) {
  typedef RowTile<D> RT;
  constexpr int KS = D / 16, NC = D / 32;
  constexpr float kTau = 8.f;
  constexpr int kTile = 64 * D;                 // elements of a 64-slot tile
  constexpr int NL = kTile / 512 / 4;           // its load instructions per writer
  // three stages each; separate arrays, so that the compiler knows what a request into one does not touch
  __shared__ __attribute__((aligned(16))) uint16_t sK0[kTile], sK1[kTile], sK2[kTile];
  __shared__ __attribute__((aligned(16))) uint16_t sV0[kTile], sV1[kTile], sV2[kTile];
  __shared__ __attribute__((aligned(16))) bf16x8 sW[2 * 4 * 4 * 64];   // [tile parity][token group][16 slots][lane]

  // launch order: all sequences of one KV head, then the next head (shared keys stay in L2)
  const uint32_t uy = block_unit();
  if (uy >= p.B * p.Hkv) return;
  const uint32_t h = uy / p.B, b = uy % p.B, unit = b * p.Hkv + h;
  const uint32_t G = p.G, T = p.T, n = p.M / 64;
  const uint32_t c = p.c_begin + blockIdx.x / G, gp = blockIdx.x % G;
  const uint32_t t0 = c * kTC, rho0 = gp * kTC;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64, col = lane % 32, half = lane / 32;
  const size_t units = (size_t)p.B * p.Hkv;
  const uint16_t* mk = p.mk + (size_t)(p.mk_per_seq ? unit : h) * p.M * D;
  const uint16_t* mvc = p.snap + ((size_t)c * units + unit) * p.M * D;   // MV_c as operand tiles

  auto stage_k = [&](auto i) __attribute__((always_inline)) -> uint16_t* {
    if constexpr (decltype(i)::v % 3 == 0) return sK0;
    else if constexpr (decltype(i)::v % 3 == 1) return sK1;
    else return sK2;
  };
  auto stage_v = [&](auto i) __attribute__((always_inline)) -> uint16_t* {
    if constexpr (decltype(i)::v % 3 == 0) return sV0;
    else if constexpr (decltype(i)::v % 3 == 1) return sV1;
    else return sV2;
  };
  // nl of the tile's 4 NL load instructions of either matrix, `first` and the ones after it
  auto request = [&](auto nl, auto i, uint32_t tile, int first) __attribute__((always_inline)) {
    const uint32_t t = min(tile, n - 1);   // past the end: the last tile again, never used
    const uint16_t *k = mk + (size_t)t * kTile, *v = mvc + (size_t)t * kTile;
#pragma unroll
    for (int j = 0; j < decltype(nl)::v; ++j) {
      const int ld = first + j;
      lds_request(k + ld * 512, RT::source(ld, lane), stage_k(i) + ld * 512);
    }
    __builtin_amdgcn_sched_barrier(0);   // the keys are needed a tile before the values: see tile_end
#pragma unroll
    for (int j = 0; j < decltype(nl)::v; ++j) {
      const int ld = first + j;
      lds_request(v + ld * 512, (uint32_t)lane * 16u, stage_v(i) + ld * 512);
    }
  };
  // 32 slots of the tile (blk = 0, 1) against this wavefront's 32 rows: lane = row, register v = slot
  // 8 (v / 4) + 4 half + v % 4 of the 32
  // LDS operands are requested a region ahead of the products that use them (region(): the scheduler keeps its
  // order; left to itself it waits out an LDS latency before every second product).
  const uint32_t at = RT::operand_at(lane);
  auto scores = [&](const uint16_t* k, const bf16x8* x, f32x16* s) __attribute__((always_inline)) {
    bf16x8 f[2][4];
    auto load = [&](int bt) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < 4; ++i) f[bt & 1][i] = RT::operand(k + (i & 1) * 32 * D, 2 * bt + i / 2, at);
    };
    s[0] = zero16();
    s[1] = zero16();
    load(0);
    region();
#pragma unroll
    for (int bt = 0; bt < KS / 2; ++bt) {
      if (bt + 1 < KS / 2) load(bt + 1);
#pragma unroll
      for (int i = 0; i < 4; ++i) s[i & 1] = mfma_bf16(f[bt & 1][i], x[2 * bt + i / 2], s[i & 1]);
      region();
    }
  };
  // End of tile i: this wavefront's LDS accesses are done; of its requests the values of tile i + 2 may still be on
  // their way, the keys of i + 2 (for the writers) and the values of i + 1 have arrived
  auto tile_end = [&](auto nl) __attribute__((always_inline)) {
    __builtin_amdgcn_s_waitcnt(kWaitLds);
    __builtin_amdgcn_s_waitcnt(wait_vm(decltype(nl)::v));
    bare_barrier();
  };

  const bool reader = wave < 4;
  const int rg = wave & 3, srow = 32 * rg + col;
  // A row's own token and the earlier ones of the sub-chunk are all it can read: of the four groups of 32 write
  // tokens a reader needs the first nsb (none: its rows are all past the chunk's end), the workgroup those
  // whose writer is asked
  auto groups = [&](uint32_t first_row, uint32_t last_row) __attribute__((always_inline)) -> int {
    const uint32_t left = T - t0;   // tokens of the sub-chunk, at least one
    return (rho0 + first_row) / G >= left ? 0 : (int)(min((rho0 + last_row) / G, left - 1) / 32 + 1);
  };
  const int nsb = groups(32 * rg, 32 * rg + 31);
  const int nasked = groups(0, kTC - 1);
  const bool asked = rg < nasked;
  // Who requests (every workgroup has a row, so at least one writer is asked): every writer a quarter of a tile; where some
  // writers have no weights to make (96 tokens or fewer to read) two of those half each or the only one all of it, so that
  // nobody who computes waits for the address unit.  Us, with quarters
  // always and so: B = 40, H = 37, M = 7680, d = 64, 4 tokens 1820 and 1702 (the read 720 and 602); B = 8, H = 8, M = 4096, d = 128, 20 tokens
  // 141.9 and 134.4; B = 1, H = 7, M = 9216, d = 64, 90 tokens 170.0 and 152.7; B = 4, H = 8, M = 4096, d = 128, 80 tokens 127.8 and 124.7.
  const int idle = 4 - nasked;
  // Outstanding: two tiles here, then three matrices' requests (the values of a tile and all of the one after the next).
  // One idle writer at d = 128 starts with 64, more than the counter holds: it waits for the first.
  static_assert(3 * 4 * NL <= kMostVm, "a lone requester's tiles in flight");
  auto begin = [&](auto nl, int first) __attribute__((always_inline)) {
    constexpr int kAll = 4 * decltype(nl)::v;
    request(nl, Int<0>{}, 0, first);
    if constexpr (kAll > kMostVm) __builtin_amdgcn_s_waitcnt(wait_vm(kMostVm - kAll / 2));
    request(nl, Int<1>{}, 1, first);
  };
  if (!reader) {
    if (idle == 0) begin(Int<NL>{}, rg * NL);
    else if (idle == 1 && rg == 3) begin(Int<4 * NL>{}, 0);
    else if (idle >= 2 && rg >= 2) begin(Int<2 * NL>{}, (rg - 2) * 2 * NL);
  }
  // this wavefront's rows as operand fragments, kept in registers.  A negative read scale moves into the
  // row (negating bf16 is exact), so that the largest raw score is also the largest scaled one.
  float cs = reader ? p.rscale_l2e : p.wscale_l2e;   // scale of this wavefront's rows (log2 domain)
  const uint32_t rtok = reader ? t0 + (rho0 + srow) / G : t0 + srow;   // the row's token
  const bool present = rtok < T;
  bf16x8 x[KS];
  {
    const uint32_t flip = reader && cs < 0.f ? 0x80008000u : 0u;
    if (reader) cs = fabsf(cs);
    const uint16_t* src = reader ? p.q + (((size_t)b * T + rtok) * p.Hq + h * G + (rho0 + srow) % G) * D
                                 : p.wq + (((size_t)b * T + rtok) * p.Hkv + h) * D;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      u32x4 v = {0u, 0u, 0u, 0u};
      if (present) v = *(const u32x4*)(src + ks * 16 + half * 8);
      x[ks] = __builtin_bit_cast(bf16x8, v ^ (u32x4){flip, flip, flip, flip});
    }
  }
  if (idle == 1) tile_end(Int<4 * NL>{});
  else if (idle >= 2) tile_end(Int<2 * NL>{});
  else tile_end(Int<NL>{});

  if (!reader) {
    const float shift = present ? p.norm_w[(size_t)unit * T + rtok] : kNoRow;
    auto weights = [&](auto i, uint32_t it) __attribute__((always_inline)) {
      f32x16 s[2];
      scores(stage_k(i), x, s);
#pragma unroll
      for (int k = 0; k < 2; ++k) {
#pragma unroll
        for (int v = 0; v < 16; ++v) s[k][v] = fast_exp2(__builtin_fmaf(s[k][v], cs, -shift));
#pragma unroll
        for (int j = 0; j < 2; ++j) sW[(((it & 1) * 4 + rg) * 4 + 2 * k + j) * 64 + lane] = pack8(s[k], j);
      }
    };
    // nl: the writer's requests of either matrix and tile, none (then all of them are others')
    auto walk = [&](auto nl, auto weighs, int first) __attribute__((always_inline)) {
      auto tile = [&](auto i, uint32_t it) __attribute__((always_inline)) {
        if constexpr (decltype(nl)::v > 0) request(nl, Int<decltype(i)::v + 2>{}, it + 2, first);
        if (decltype(weighs)::v && asked) weights(Int<decltype(i)::v + 1>{}, it + 1);   // past the end: of whatever tile is there, never used
        tile_end(nl);
      };
      if (decltype(weighs)::v && asked) weights(Int<0>{}, 0);
      tile_end(nl);
      uint32_t it = 0;
      for (; it + 3 <= n; it += 3) {
        tile(Int<0>{}, it);
        tile(Int<1>{}, it + 1);
        tile(Int<2>{}, it + 2);
      }
      if (it < n) tile(Int<0>{}, it);
      if (it + 1 < n) tile(Int<1>{}, it + 1);
    };
    if (idle == 0) walk(Int<NL>{}, Int<1>{}, rg * NL);
    else if (idle == 1 && rg == 3) walk(Int<4 * NL>{}, Int<0>{}, 0);
    else if (idle >= 2 && rg >= 2) walk(Int<2 * NL>{}, Int<0>{}, (rg - 2) * 2 * NL);
    else walk(Int<0>{}, Int<1>{}, 0);
    __builtin_amdgcn_s_waitcnt(wait_vm(0));
    return;   // no barrier follows
  }

  f32x16 oacc[NC], aacc[4];   // [columns][row], [write tokens][row]: lane = this wavefront's row
#pragma unroll
  for (int jt = 0; jt < NC; ++jt) oacc[jt] = zero16();
#pragma unroll
  for (int sb = 0; sb < 4; ++sb) aacc[sb] = zero16();
  float shift = kNegBig, zsum = 0.f;
  auto tile = [&](auto i, uint32_t it) __attribute__((always_inline)) {
    f32x16 s[2];
    scores(stage_k(i), x, s);
    float tm = fmaxf(s[0][0], s[1][0]);
#pragma unroll
    for (int v = 1; v < 16; ++v) tm = fmaxf(fmaxf(tm, s[0][v]), s[1][v]);
    tm = max_of_halves(tm) * cs;
    const bool moves = tm > shift + kTau;        // also the first tile (shift = kNegBig, nothing accumulated yet)
    if (__builtin_amdgcn_ballot_w64(moves)) {    // bring what has been accumulated to the new shifts
      const float f = moves ? fast_exp2(shift - tm) : 1.f;
      shift = moves ? tm : shift;
      zsum *= f;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
#pragma unroll
        for (int jt = 0; jt < NC; ++jt) oacc[jt][v] *= f;
#pragma unroll
        for (int sb = 0; sb < 4; ++sb) aacc[sb][v] *= f;
      }
    }
    // regions of: the next operands from LDS, the products of the last, the weights of the next 16 slots
    const bf16x8* mvt = (const bf16x8*)stage_v(i) + lane;
    const bf16x8* ww = sW + (it & 1) * 1024 + lane;
    constexpr int NF = NC > 4 ? NC : 4;
    bf16x8 f[2][NF], pw[4];     // pw: the row's weights, 16 slots each
    float add = 0.f;
    auto weights = [&](int j) __attribute__((always_inline)) {
#pragma unroll
      for (int v = 8 * (j & 1); v < 8 * (j & 1) + 8; ++v) {
        s[j / 2][v] = fast_exp2(__builtin_fmaf(s[j / 2][v], cs, -shift));
        add += s[j / 2][v];
      }
      asm volatile("" : "+v"(add));   // added here: moved behind the products, the terms take 32 registers
      pw[j] = pack8(s[j / 2], j & 1);
    };
#pragma unroll
    for (int jt = 0; jt < NC; ++jt) f[0][jt] = mvt[jt * 64];
    weights(0);
    region();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (j < 3) {
#pragma unroll
        for (int jt = 0; jt < NC; ++jt) f[(j + 1) & 1][jt] = mvt[((j + 1) * NC + jt) * 64];
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) f[0][k] = ww[k * 64];
      }
#pragma unroll
      for (int jt = 0; jt < NC; ++jt) oacc[jt] = mfma_bf16(f[j & 1][jt], pw[j], oacc[jt]);
      if (j < 3) weights(j + 1);
      region();
    }
    zsum += add;
#pragma unroll
    for (int sb = 0; sb < 4; ++sb)
      if (sb < nsb) {
        if (sb < 3) {
#pragma unroll
          for (int k = 0; k < 4; ++k) f[(sb + 1) & 1][k] = ww[((sb + 1) * 4 + k) * 64];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) aacc[sb] = mfma_bf16(f[sb & 1][k], pw[k], aacc[sb]);
        region();
      }
  };
  auto step = [&](auto i, uint32_t it) __attribute__((always_inline)) {
    if (nsb > 0) tile(i, it);
    tile_end(Int<NL>{});
  };
  tile_end(Int<NL>{});   // the writers' first tile
  uint32_t it = 0;
  for (; it + 3 <= n; it += 3) {
    step(Int<0>{}, it);
    step(Int<1>{}, it + 1);
    step(Int<2>{}, it + 2);
  }
  if (it < n) step(Int<0>{}, it);
  if (it + 1 < n) step(Int<1>{}, it + 1);
  __builtin_amdgcn_s_waitcnt(wait_vm(0));

  // A'[s] = (s <= token of the row) ? sum_m e[row][m] ww[s][m] : 0, and with it the tokens of the sub-chunk itself
  const int tl = (int)((rho0 + srow) / G);  // the row's token within the sub-chunk
  const bf16x8* wvt = (const bf16x8*)(p.wvt + ((size_t)unit * p.Tpad + t0) * D);
  bf16x8 wf[2][2 * NC];   // operands of 32 tokens, requested while the 32 before are multiplied
  auto tokens = [&](int sb) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < 2 * NC; ++k) wf[sb & 1][k] = wvt[operand_chunk<D>(2 * sb + k / NC, k % NC, lane)];
  };
  tokens(0);
#pragma unroll
  for (int sb = 0; sb < 4; ++sb) {   // a group that was not multiplied holds zeros
    if (sb < 3) tokens(sb + 1);
    region();
#pragma unroll
    for (int v = 0; v < 16; ++v)
      if (32 * sb + 8 * (v / 4) + 4 * half + v % 4 > tl) aacc[sb][v] = 0.f;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const bf16x8 a = pack8(aacc[sb], j);
#pragma unroll
      for (int jt = 0; jt < NC; ++jt) oacc[jt] = mfma_bf16(wf[sb & 1][j * NC + jt], a, oacc[jt]);
    }
    region();
  }
  const float z = zsum + __shfl_xor(zsum, 32, 64), inv = 1.0f / z;   // the normaliser of everything accumulated
  // A lane has pieces of 8 bytes of its row; the rows leave whole, through this wavefront's 32 rows of LDS.  The key stages are
  // free: the requests that the writers may still have in flight are for values.
  uint16_t* const strip = (rg < 2 ? sK0 : sK1) + (rg % 2) * 32 * D;
#pragma unroll
  for (int jt = 0; jt < NC; ++jt)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4)
      store4_bf16(strip + col * D + ((4 * jt + q4) ^ swizzle<D>(col)) * 8 + 4 * half, oacc[jt][4 * q4 + 0] * inv,
                  oacc[jt][4 * q4 + 1] * inv, oacc[jt][4 * q4 + 2] * inv, oacc[jt][4 * q4 + 3] * inv);
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int i = 0; i < D / 16; ++i) {
    const uint32_t rho = rho0 + 32 * rg + RT::row(i, lane), tk = t0 + rho / G;
    if (tk < T)
      *(u32x4*)(p.out + (((size_t)b * T + tk) * p.Hq + h * G + rho % G) * D + RT::chunk(i, lane) * 8) =
          *(const u32x4*)(strip + (i * 64 + lane) * 8);
  }
}

// ------------------------------------------------------------------ state

// MV tile of 128 slots: acc = MV_start; tokens are walked 32 at a time; at the
// start of every sub-chunk c (if reads follow) round(acc) is left as MV_c;
// acc += WW^T . WV; finally MV = round(acc).  The write weights are recomputed
// per token tile and never leave the registers: a wavefront owns 32 slots and
// all d value columns.  Its score product has rows = tokens, columns = slots, so a lane's accumulator registers are
// the A operand (row = slot) of the state product with WV^T as operand tiles.  MV_c leaves in operand tiles
// too: a lane's accumulator registers, rounded, are its 16-byte chunks of them, and a wavefront stores whole
// kilobytes without a detour through LDS.  The token tiles (write queries, WV^T) are requested into LDS a tile
// ahead; one barrier per tile, between which the wavefronts run on their own.  The key fragments of a
// wavefront's slots stay in registers.
// With reads the kernel is partly bound by memory (MV in and out and a copy of MV per sub-chunk: 6.4 GB of the 8.4 a
// chunk moves at B = 32, H = 32, M = 4096, T = 512), without by its matrix and vector work.  A token tile of 32 keeps
// a workgroup within 168 registers and 34 KB, so that three of them (three wavefronts per SIMD) hide each
// other's barriers and stores; two: 2250 us against 1950 at that size, four (registers spilled): 2680.  Row-major
// token tiles of 64 with padded rows, where a third of the LDS cycles were bank conflicts, took 2170.  With write queries as operand
// tiles (see RowTile) 1950 to 1970, in whole rows 1870.  The wait that ends a
// tile is for all requests; in every fourth tile that includes the snapshot's stores, issued after them.
// FAR: a token tile's write queries lie further apart than a lane's 32-bit byte offset reaches (see
// launch_prefill_bf16), so their addresses are 64-bit.  Not for every chunk: 64-bit addresses spill 62 registers of
// the d = 128 kernel, the 32-bit offsets none.
template <int D, bool FAR>
__global__ __launch_bounds__(256, 3) void prefill_state_kernel(const PrefillParams p) {
  constexpr int KS = D / 16, NC = D / 32;
  constexpr int TT = 32;            // tokens per tile
  constexpr int kTile = TT * D;     // elements of a token tile of either matrix = of a wavefront's 32 slots
  constexpr int NI = kTile / 512;   // load instructions of a tile
  constexpr int NL = NI / 4;        // of them per wavefront
  typedef RowTile<D> RT;
  // two stages of write queries, WV^T and shifts (a copy per wavefront); before and after the token loop the first
  // four arrays hold the four wavefronts' slots on their way in and out, as a RowTile each
  __shared__ __attribute__((aligned(16))) uint16_t sX0[kTile], sX1[kTile], sT0[kTile], sT1[kTile];
  __shared__ __attribute__((aligned(16))) float sN0[4 * 64], sN1[4 * 64];

  const uint32_t unit = block_unit();
  if (unit >= p.B * p.Hkv) return;
  const uint32_t b = unit / p.Hkv, h = unit % p.Hkv;
  const uint32_t m0 = blockIdx.x * 128, T = p.T;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64, col = lane % 32, half = lane / 32;
  const size_t units = (size_t)p.B * p.Hkv;
  // M is a multiple of 64, so a wavefront's 32 slots are all inside the memory or all outside
  const uint32_t slot0 = m0 + 32 * wave;
  const bool live = slot0 < p.M;
  const uint16_t* mk = p.mk + ((size_t)(p.mk_per_seq ? unit : h) * p.M + slot0) * D;
  uint16_t* mv = p.mv + ((size_t)unit * p.M + slot0) * D;
  uint16_t* const strip = wave == 0 ? sX0 : wave == 1 ? sX1 : wave == 2 ? sT0 : sT1;

  if (live) {
#pragma unroll
    for (int i = 0; i < NI; ++i) lds_request(mv, RT::row(i, lane) * D * 2 + RT::chunk(i, lane) * 16, strip + i * 512);
  }
  bf16x8 kb[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    u32x4 v = {0u, 0u, 0u, 0u};
    if (live) v = *(const u32x4*)(mk + (size_t)col * D + ks * 16 + half * 8);
    kb[ks] = __builtin_bit_cast(bf16x8, v);
  }
  // state product: lane = value column, accumulator rows = slots.  Element (slot row, column) of the strip:
  auto cell = [&](int r, int jt) { return r * D + (((4 * jt + col / 8) ^ swizzle<D>(r)) * 8) + col % 8; };
  f32x16 macc[NC];
#pragma unroll
  for (int jt = 0; jt < NC; ++jt) macc[jt] = zero16();
  __builtin_amdgcn_s_waitcnt(wait_vm(0));
  if (live) {
#pragma unroll
    for (int jt = 0; jt < NC; ++jt)
#pragma unroll
      for (int v = 0; v < 16; ++v) macc[jt][v] = bf16_val(strip[cell(8 * (v / 4) + 4 * half + v % 4, jt)]);
  }
  __syncthreads();

  const uint32_t ntile = (T + TT - 1) / TT, at = RT::operand_at(lane);
  auto pick = [](auto i, auto* a, auto* c) {
    if constexpr (decltype(i)::v % 2 == 0) return a;
    else return c;
  };
  // Tokens past the end of the chunk load the last token instead: their WV^T columns are zero, so whatever
  // finite weights they get change nothing.  Past the last tile: the last one again, never used.
  const uint32_t xstride = p.Hkv * D, lastrow = (T - 1) % TT;
  const uint16_t* wq = p.wq + ((size_t)b * T * p.Hkv + h) * D;
  const uint16_t* wvt = p.wvt + (size_t)unit * p.Tpad * D;
  auto request = [&](auto i, uint32_t tile) {
    const uint32_t tl = min(tile, ntile - 1), over = tl == ntile - 1 ? lastrow : (uint32_t)TT - 1;
    uint16_t *sx = pick(i, sX0, sX1), *st = pick(i, sT0, sT1);
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      const int ld = wave * NL + j;
      const uint32_t row = min((uint32_t)RT::row(ld, lane), over), ch = (uint32_t)RT::chunk(ld, lane) * 8u;
      if constexpr (FAR) lds_request(wq + ((size_t)(tl * TT + row) * xstride + ch), sx + ld * 512);
      else lds_request(wq + (size_t)tl * TT * xstride, (row * xstride + ch) * 2u, sx + ld * 512);
      lds_request(wvt + (size_t)tl * kTile + ld * 512, (uint32_t)lane * 16u, st + ld * 512);
    }
    lds_request<4>(p.norm_w + (size_t)unit * T + tl * TT, min((uint32_t)col, over) * 4u, pick(i, sN0, sN1) + 64 * wave);
  };
  auto tile = [&](auto i, uint32_t tt) {
    request(Int<decltype(i)::v + 1>{}, tt + 1);
    if (p.has_read && live && tt % (kTC / TT) == 0) {
      // MV at the start of sub-chunk c
      u32x4* sn = (u32x4*)(p.snap + ((size_t)(tt / (kTC / TT)) * units + unit) * p.M * D);
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int jt = 0; jt < NC; ++jt)
          __builtin_nontemporal_store(__builtin_bit_cast(u32x4, pack8(macc[jt], j)), sn + operand_chunk<D>(slot0 / 16 + j, jt, lane));
    }
    const uint16_t *sx = pick(i, sX0, sX1), *st = pick(i, sT0, sT1);
    const float* sn = pick(i, sN0, sN1) + 64 * wave;
    // Regions, as in the read kernel: the next operands from LDS beside the products of the last.
    // Scores: rows = tokens, columns = this wavefront's 32 slots
    f32x16 sc = zero16();
    bf16x8 f[2][4];
    f32x4 sh[4];   // shifts of the lane's tokens
    const bf16x8* wt = (const bf16x8*)st + lane;
#pragma unroll
    for (int k = 0; k < 4; ++k) f[0][k] = RT::operand(sx, k, at);
    region();
#pragma unroll
    for (int bt = 0; bt < KS / 4; ++bt) {
      if (bt + 1 < KS / 4) {
#pragma unroll
        for (int k = 0; k < 4; ++k) f[(bt + 1) & 1][k] = RT::operand(sx, 4 * (bt + 1) + k, at);
      } else {
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) sh[q4] = *(const f32x4*)(sn + 8 * q4 + 4 * half);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) sc = mfma_bf16(f[bt & 1][k], kb[4 * bt + k], sc);
      region();
    }
    // weights of 16 tokens, and what bf16 leaves of them
    bf16x8 wh[2], wl[2];
    auto weights = [&](int j) {
      f32x16 lo;
#pragma unroll
      for (int v = 8 * j; v < 8 * j + 8; ++v) sc[v] = fast_exp2(sc[v] * p.wscale_l2e - sh[v / 4][v % 4]);
      wh[j] = pack8(sc, j);
      const u32x4 hw = __builtin_bit_cast(u32x4, wh[j]);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        lo[8 * j + 2 * k] = sc[8 * j + 2 * k] - __uint_as_float(hw[k] << 16);
        lo[8 * j + 2 * k + 1] = sc[8 * j + 2 * k + 1] - __uint_as_float(hw[k] & 0xFFFF0000u);
      }
      wl[j] = pack8(lo, j);
    };
    // state product over the tile's 32 tokens, 16 per MFMA.  All hi products of a token group before its lo
    // products: no product waits for its predecessor.
    bf16x8 bv[2][NC];
#pragma unroll
    for (int jt = 0; jt < NC; ++jt) bv[0][jt] = wt[jt * 64];
    weights(0);
    region();
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if (j == 0) {
#pragma unroll
        for (int jt = 0; jt < NC; ++jt) bv[1][jt] = wt[(NC + jt) * 64];
      }
#pragma unroll
      for (int jt = 0; jt < NC; ++jt) macc[jt] = mfma_bf16(wh[j], bv[j][jt], macc[jt]);
#pragma unroll
      for (int jt = 0; jt < NC; ++jt) macc[jt] = mfma_bf16(wl[j], bv[j][jt], macc[jt]);
      if (j == 0) weights(1);
      region();
    }
    __builtin_amdgcn_s_waitcnt(kWaitLds);
    __builtin_amdgcn_s_waitcnt(wait_vm(0));   // the next tile has arrived
    bare_barrier();
  };
  request(Int<0>{}, 0);
  __builtin_amdgcn_s_waitcnt(wait_vm(0));
  bare_barrier();
  uint32_t tt = 0;
  for (; tt + 2 <= ntile; tt += 2) {
    tile(Int<0>{}, tt);
    tile(Int<1>{}, tt + 1);
  }
  if (tt < ntile) tile(Int<0>{}, tt);
  __builtin_amdgcn_s_waitcnt(wait_vm(0));
  __syncthreads();   // everyone's last requests have arrived: the arrays are free
  if (live) {
#pragma unroll
    for (int jt = 0; jt < NC; ++jt)
#pragma unroll
      for (int v = 0; v < 16; ++v) strip[cell(8 * (v / 4) + 4 * half + v % 4, jt)] = bf16_bits(macc[jt][v]);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < NI; ++i)
      __builtin_nontemporal_store(*(const u32x4*)(strip + (i * 64 + lane) * 8), (u32x4*)(mv + (size_t)RT::row(i, lane) * D + RT::chunk(i, lane) * 8));
  }
}

// ------------------------------------------------------------------ chunks of few tokens

// With one sub-chunk MV_c is MV itself, and with few tokens the products are small beside the bytes: one pass over MK and
// MV does the read and the update (prefill_pass_kernel).  Before it, one launch makes the statistics of the write rows and puts
// the operands of the chunk's rows in order, since every workgroup of the pass wants them (prefill_begin_kernel); after
// it, the outputs of the slot ranges are added (prefill_pass_merge_kernel), if there are several.
//
// Operand tiles of the write queries and of the read rows: tile (group of 32 rows, 16 inputs ks), lane l: row l % 32, inputs
// 16 ks + 8 (l / 32) ..; rows that do not exist are zero.  A negative read scale moves into the read rows.  WV as in
// prefill_transpose_kernel, 32 NT tokens.
struct PassParams {
  PrefillParams c;
  uint16_t *wvt, *wqt, *qt;   // [units][..]
  float2* pairs;              // [units][shares][T] (max, sum) of a token's write scores over a share of the slots
  float* part;                // [units][splits][rows][d] outputs of a range of slots, not normalised
  float2* mz;                 // [units][splits][rows] their shift and sum of weights
  uint32_t rows;              // T G
  uint32_t shares, share_tiles;   // of 128 slots
  uint32_t splits;            // of 128 slots
};

template <int D, int NT, int NR>
__global__ __launch_bounds__(256) void prefill_begin_kernel(const PassParams q) {
  constexpr int LD = D + 8, KS = D / 16, kRows = 32 * D, NI = kRows / 512;
  typedef RowTile<D> RT;
  __shared__ __attribute__((aligned(16))) uint16_t sT[4 * kRows];   // a wavefront's 32 key rows each, or 64 rows of WV
  __shared__ float2 sPair[NT][4][32];
  static_assert(64 * LD <= 4 * kRows, "WV");
  const PrefillParams& p = q.c;
  const uint32_t unit = block_unit();
  if (unit >= p.B * p.Hkv) return;
  const uint32_t b = unit / p.Hkv, h = unit % p.Hkv, T = p.T;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64, col = lane % 32, half = lane / 32;
  if (blockIdx.x < q.shares) {
    // statistics of a share: a wavefront takes every fourth 32 slots of it; lane = token, register = slot
    bf16x8 x[NT][KS];
#pragma unroll
    for (int g = 0; g < NT; ++g)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        u32x4 v = {0u, 0u, 0u, 0u};
        if ((uint32_t)(32 * g + col) < T) v = *(const u32x4*)(p.wq + (((size_t)b * T + 32 * g + col) * p.Hkv + h) * D + ks * 16 + half * 8);
        x[g][ks] = __builtin_bit_cast(bf16x8, v);
      }
    const uint16_t* mk = p.mk + (size_t)(p.mk_per_seq ? unit : h) * p.M * D;
    const uint32_t first = blockIdx.x * q.share_tiles * 128 + 32 * wave, end = min((blockIdx.x + 1) * q.share_tiles * 128, p.M);
    float m[NT], sum[NT];
#pragma unroll
    for (int g = 0; g < NT; ++g) {
      m[g] = kNegBig;
      sum[g] = 0.f;
    }
    uint16_t* const strip = sT + wave * kRows;
    const uint32_t at = RT::operand_at(lane);
    auto request = [&](uint32_t slot) {
#pragma unroll
      for (int i = 0; i < NI; ++i) lds_request(mk + (size_t)slot * D + i * 512, RT::source(i, lane), strip + i * 512);
    };
    if (first < end) request(first);
    for (uint32_t slot = first; slot < end; slot += 128) {
      __builtin_amdgcn_s_waitcnt(wait_vm(0));
      asm volatile("" ::: "memory");
      region();
      bf16x8 kb[KS];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) kb[ks] = RT::operand(strip, ks, at);
      __builtin_amdgcn_s_waitcnt(kWaitLds);   // the rows have been read: the next ones may come
      asm volatile("" ::: "memory");
      region();
      if (slot + 128 < end) request(slot + 128);
#pragma unroll
      for (int g = 0; g < NT; ++g) {
        f32x16 s = zero16();
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) s = mfma_bf16(kb[ks], x[g][ks], s);
        float t = kNegBig, add = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          s[v] *= p.wscale_l2e;
          t = fmaxf(t, s[v]);
        }
        t = fmaxf(m[g], t);
#pragma unroll
        for (int v = 0; v < 16; ++v) add += fast_exp2(s[v] - t);
        sum[g] = sum[g] * fast_exp2(m[g] - t) + add;
        m[g] = t;
      }
    }
#pragma unroll
    for (int g = 0; g < NT; ++g) {
      merge_stat(m[g], sum[g], __shfl_xor(m[g], 32, 64), __shfl_xor(sum[g], 32, 64));
      if (half == 0) sPair[g][wave][col] = make_float2(m[g], sum[g]);
    }
    __syncthreads();
    if (threadIdx.x < T) {
      const int g = threadIdx.x / 32, c = threadIdx.x % 32;
      float2 r = sPair[g][0][c];
#pragma unroll
      for (int w = 1; w < 4; ++w) merge_stat(r.x, r.y, sPair[g][w][c].x, sPair[g][w][c].y);
      q.pairs[((size_t)unit * q.shares + blockIdx.x) * T + threadIdx.x] = r;
    }
    return;
  }
  Tile<64, D> t;
  t.fetch_rows(p.wv, [&](int r) -> const uint16_t* { return r < (int)T ? p.wv + (((size_t)b * T + r) * p.Hkv + h) * D : nullptr; });
  if (p.gate) {   // the sign of a step size: see prefill_transpose_kernel
#pragma unroll
    for (int i = 0; i < Tile<64, D>::N; ++i) {
      const uint32_t tk = threadIdx.x / Tile<64, D>::CPR + i * Tile<64, D>::RPP;
      const uint32_t flip = tk < T && p.gate[((size_t)b * T + tk) * p.Hkv + h] < 0.f ? 0x80008000u : 0u;
      t.v[i] ^= (u32x4){flip, flip, flip, flip};
    }
  }
  t.put(sT, LD);
  const uint32_t rflip = p.rscale_l2e < 0.f ? 0x80008000u : 0u;
  for (int i = threadIdx.x; i < (NT + NR) * KS * 64; i += 256) {
    const int l = i % 64, ks = i / 64 % KS, g = i / 64 / KS;   // row group: the write queries', then the read rows'
    const bool wr = g < NT;
    const uint32_t row = (wr ? g : g - NT) * 32 + l % 32, k = ks * 16 + l / 32 * 8;
    u32x4 v = {0u, 0u, 0u, 0u};
    if (wr && row < T) v = *(const u32x4*)(p.wq + (((size_t)b * T + row) * p.Hkv + h) * D + k);
    if (!wr && row < q.rows)
      v = *(const u32x4*)(p.q + (((size_t)b * T + row / p.G) * p.Hq + h * p.G + row % p.G) * D + k) ^ (u32x4){rflip, rflip, rflip, rflip};
    u32x4* to = wr ? (u32x4*)q.wqt + (size_t)unit * NT * KS * 64 + i : (u32x4*)q.qt + (size_t)unit * NR * KS * 64 + (i - NT * KS * 64);
    *to = v;
  }
  __syncthreads();
  u32x4* dst = (u32x4*)q.wvt + (size_t)unit * NT * 32 * D / 8;
  for (int i = threadIdx.x; i < NT * 32 * D / 8; i += 256) {
    const int l = i % 64, tile = i / 64, hf = l / 32;
    const int j = 32 * (tile % (D / 32)) + l % 32, t8 = 16 * (tile / (D / 32)) + 4 * hf;
    uint32_t e[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) e[k] = sT[(t8 + (k / 4) * 8 + k % 4) * LD + j];
    dst[i] = (u32x4){e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16)};
  }
}

// One workgroup walks its range of slots 128 at a time, a wavefront 32 of them: keys as operands in registers, MV through
// LDS in whole rows and back as operand tiles.  Up to 32 NT tokens and 32 NR read rows.
//   1. scores of the read rows against this wavefront's slots (lane = row, register = slot); a row's largest of the 128
//      moves its shift; weights of the write tokens (lane = token);
//   2. weights, sums and MV of all wavefronts meet in LDS as operand tiles;
//   3. a wavefront makes 32 columns of 32 read rows: += RW . MV + mask(RW . WW^T) . WV;
//   4. the state, as in prefill_state_kernel: the same products in the same order, so from equal shifts MV has the same bits.  (The
//      shifts come from other sums: prefill_begin_kernel's, of every fourth 32 slots and up to eight shares, not prefill_stats_kernel's;
//      so a chunk that only writes, which takes that one, may leave MV an ulp from this one's here and there.)
// A workgroup is one chain of these steps, 6 us alone and 10 beside another one, and two fit a compute unit (d = 64: three, 10 %
// faster than two): 3456 of them (B = 3, H = 36, M = 4096, T = 10) take 74 us, 4.6 TB/s.  Keys in operand order from memory instead of
// in whole rows: 78; the operands of the rows from memory where they are used, not staged: 92; walking several tiles in a
// workgroup with the next one's loads in flight: spills.
template <int D, int NT, int NR>
__global__ __launch_bounds__(256, D == 64 && NR == 1 ? 3 : D == 64 || NR == 1 ? 2 : 1) void prefill_pass_kernel(const PassParams q) {
  constexpr int KS = D / 16, NC = D / 32;
  constexpr int kRows = 32 * D;       // elements of a wavefront's slots
  constexpr int NI = kRows / 512;     // load instructions of them
  constexpr int NK = (NR * NC + 3) / 4;   // blocks of 32 rows x 32 columns of a wavefront
  typedef RowTile<D> RT;
  __shared__ __attribute__((aligned(16))) uint16_t sMV[4 * kRows];   // rows on the way in and out, operand tiles between
  __shared__ __attribute__((aligned(16))) bf16x8 sW[NT * 4 * 2 * 64], sP[NR * 4 * 2 * 64];   // [group][wavefront][16 slots][lane]
  __shared__ __attribute__((aligned(16))) u32x4 sX[NT * KS * 64], sQ[NR * KS * 64], sV[NT * 2 * NC * 64];
  __shared__ float sMax[NR][4][32], sSum[NR][4][32];
  __shared__ __attribute__((aligned(16))) float sShift[NT * 32];
  const PrefillParams& p = q.c;
  const uint32_t unit = block_unit();
  if (unit >= p.B * p.Hkv) return;
  const uint32_t b = unit / p.Hkv, h = unit % p.Hkv, split = blockIdx.x, T = p.T;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64, col = lane % 32, half = lane / 32;
  const uint32_t first = split * 128, end = min(first + 128, p.M);
  const uint16_t* mk = p.mk + (size_t)(p.mk_per_seq ? unit : h) * p.M * D;
  uint16_t* mv = p.mv + (size_t)unit * p.M * D;
  uint16_t* const strip = sMV + wave * kRows;

  // the rows' operands, a quarter of the tiles a wavefront: older than the loads below, so they are there when those are
#pragma unroll
  for (int i = 0; i < (NT + NR) * KS / 4 + NT * NC / 2; ++i) {
    const int k = i * 4 + wave;
    const char* from = k < NT * KS         ? (const char*)q.wqt + ((size_t)unit * NT * KS + k) * 1024
                       : k < (NT + NR) * KS ? (const char*)q.qt + ((size_t)unit * NR * KS + (k - NT * KS)) * 1024
                                            : (const char*)q.wvt + ((size_t)unit * NT * 2 * NC + (k - (NT + NR) * KS)) * 1024;
    u32x4* to = k < NT * KS ? sX + k * 64 : k < (NT + NR) * KS ? sQ + (k - NT * KS) * 64 : sV + (k - (NT + NR) * KS) * 64;
    lds_request(from, (uint32_t)lane * 16u, to);
  }
  // M is a multiple of 64, so a wavefront's 32 slots are all inside the memory or all outside.  Keys in whole rows through
  // the strip, then MV through registers: it is needed later.
  const uint32_t slot0 = first + 32 * wave;
  const bool live = slot0 < end;
  if (live) {
#pragma unroll
    for (int i = 0; i < NI; ++i) lds_request(mk + (size_t)slot0 * D + i * 512, RT::source(i, lane), strip + i * 512);
  }
  float2 pair[kMaxStatsSplit];   // requested together; past the end the last share again, not counted
  if (threadIdx.x < T) {
#pragma unroll
    for (uint32_t k = 0; k < kMaxStatsSplit; ++k) pair[k] = q.pairs[((size_t)unit * q.shares + min(k, q.shares - 1)) * T + threadIdx.x];
  }
  asm volatile("" ::: "memory");
  u32x4 mn[NI];
  if (live) {
#pragma unroll
    for (int i = 0; i < NI; ++i) mn[i] = __builtin_nontemporal_load((const u32x4*)(mv + (size_t)slot0 * D + i * 512) + lane);
  }
  asm volatile("" ::: "memory");
  // a token's shift, from the pairs of all shares: max + log2(sum) - log2 |step size| (see store_shift)
  if (threadIdx.x < NT * 32) {
    float s = kNoRow;
    if (threadIdx.x < T) {
      float m = kNegBig, sum = 0.f;
#pragma unroll
      for (uint32_t k = 0; k < kMaxStatsSplit; ++k)
        if (k < q.shares) merge_stat(m, sum, pair[k].x, pair[k].y);
      const float le = p.gate ? __log2f(fabsf(p.gate[((size_t)b * T + threadIdx.x) * p.Hkv + h])) : 0.f;
      s = m + __log2f(sum) - le;
    }
    sShift[threadIdx.x] = s;
  }
  if (live) __builtin_amdgcn_s_waitcnt(wait_vm(NI));   // all but MV
  else __builtin_amdgcn_s_waitcnt(wait_vm(0));
  lds_barrier();

  const float cs = fabsf(p.rscale_l2e);
  auto against = [&](const u32x4* rows, const bf16x8* kb) -> f32x16 {   // lane = row, register v = slot 8 (v / 4) + 4 half + v % 4
    f32x16 s = zero16();
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) s = mfma_bf16(kb[ks], __builtin_bit_cast(bf16x8, rows[ks * 64 + lane]), s);
    return s;
  };
  f32x16 oacc[NK];
  float shift[NR], zsum[NR];
#pragma unroll
  for (int k = 0; k < NK; ++k) oacc[k] = zero16();
#pragma unroll
  for (int g = 0; g < NR; ++g) {
    shift[g] = kNegBig;
    zsum[g] = 0.f;
  }

  {
    // element (slot row, this lane's column of the 32 of jt) of the strip
    auto cell = [&](int r, int jt) { return r * D + (((4 * jt + col / 8) ^ swizzle<D>(r)) * 8) + col % 8; };
    // 1
    bf16x8 kb[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8 v = RT::operand(strip, ks, RT::operand_at(lane));
      kb[ks] = live ? v : __builtin_bit_cast(bf16x8, (u32x4){0u, 0u, 0u, 0u});
    }
    f32x16 s[NR];
#pragma unroll
    for (int g = 0; g < NR; ++g) {
      s[g] = against(sQ + g * KS * 64, kb);
      float tm = s[g][0];
#pragma unroll
      for (int v = 1; v < 16; ++v) tm = fmaxf(tm, s[g][v]);
      tm = max_of_halves(tm);
      // a tile whose scores all overflowed to -inf still has a finite shift: its weights are zero
      if (half == 0) sMax[g][wave][col] = live ? fmaxf(tm * cs, kNegBig) : kNegBig;
    }
#pragma unroll
    for (int g = 0; g < NT; ++g) {
      f32x16 w = against(sX + g * KS * 64, kb);
      const float sh = sShift[32 * g + col];
#pragma unroll
      for (int v = 0; v < 16; ++v) w[v] = live ? fast_exp2(__builtin_fmaf(w[v], p.wscale_l2e, -sh)) : 0.f;
#pragma unroll
      for (int j = 0; j < 2; ++j) sW[((g * 4 + wave) * 2 + j) * 64 + lane] = pack8(w, j);
    }
    __builtin_amdgcn_s_waitcnt(kWaitLds);   // the keys have been read
    asm volatile("" ::: "memory");
    // 2: MV to the strip in whole rows, and out of it as operand tiles (rows = columns of MV, contracted over slots)
#pragma unroll
    for (int i = 0; i < NI; ++i)
      *(u32x4*)(strip + RT::row(i, lane) * D + RT::chunk(i, lane) * 8) = live ? mn[i] : (u32x4){0u, 0u, 0u, 0u};
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    u32x4 mo[NC][2];
#pragma unroll
    for (int jt = 0; jt < NC; ++jt)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        uint32_t e[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) e[k] = strip[cell(16 * j + 8 * (k / 4) + 4 * half + k % 4, jt)];
#pragma unroll
        for (int k = 0; k < 4; ++k) mo[jt][j][k] = e[2 * k] | (e[2 * k + 1] << 16);
      }
    __builtin_amdgcn_s_waitcnt(kWaitLds);
    asm volatile("" ::: "memory");
#pragma unroll
    for (int jt = 0; jt < NC; ++jt)
#pragma unroll
      for (int j = 0; j < 2; ++j) *(u32x4*)(strip + ((jt * 2 + j) * 64 + lane) * 8) = mo[jt][j];
    lds_barrier();
#pragma unroll
    for (int g = 0; g < NR; ++g) {
      const float to = fmaxf(fmaxf(sMax[g][0][col], sMax[g][1][col]), fmaxf(sMax[g][2][col], sMax[g][3][col]));
      shift[g] = to;
      float sum = 0.f;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        s[g][v] = live ? fast_exp2(__builtin_fmaf(s[g][v], cs, -to)) : 0.f;
        sum += s[g][v];
      }
      sum += __shfl_xor(sum, 32, 64);
      if (half == 0) sSum[g][wave][col] = sum;
#pragma unroll
      for (int j = 0; j < 2; ++j) sP[((g * 4 + wave) * 2 + j) * 64 + lane] = pack8(s[g], j);
    }
    lds_barrier();
    // 3
#pragma unroll
    for (int g = 0; g < NR; ++g) zsum[g] = (sSum[g][0][col] + sSum[g][1][col]) + (sSum[g][2][col] + sSum[g][3][col]);
#pragma unroll
    for (int k0 = 0; k0 < NK; ++k0) {
      const int k = k0 * 4 + wave, g = k / NC, jt = k % NC;
      if (k < NR * NC && 32u * g < q.rows) {
        const bf16x8* pw = sP + g * 4 * 2 * 64 + lane;
        f32x16 o = zero16();
#pragma unroll
        for (int w = 0; w < 4; ++w)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            o = mfma_bf16(*(const bf16x8*)(sMV + w * kRows + ((jt * 2 + j) * 64 + lane) * 8), pw[(w * 2 + j) * 64], o);
        const int tl = (int)((32 * g + col) / p.G);   // the row's token
#pragma unroll
        for (int tg = 0; tg < NT; ++tg) {
          const bf16x8* ww = sW + tg * 4 * 2 * 64 + lane;
          f32x16 a = zero16();
#pragma unroll
          for (int w = 0; w < 8; ++w) a = mfma_bf16(ww[w * 64], pw[w * 64], a);
#pragma unroll
          for (int v = 0; v < 16; ++v)
            if (32 * tg + 8 * (v / 4) + 4 * half + v % 4 > tl) a[v] = 0.f;
#pragma unroll
          for (int j = 0; j < 2; ++j)
            o = mfma_bf16(__builtin_bit_cast(bf16x8, sV[operand_chunk<D>(2 * tg + j, jt, lane)]), pack8(a, j), o);
        }
        oacc[k0] = o;
      }
    }
    // 4
    f32x16 macc[NC];
#pragma unroll
    for (int jt = 0; jt < NC; ++jt)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const uint32_t w = mo[jt][v / 8][v % 8 / 2];
        macc[jt][v] = __uint_as_float(v % 2 ? w & 0xFFFF0000u : w << 16);
      }
#pragma unroll
    for (int tg = 0; tg < NT; ++tg) {
      f32x16 sc = zero16();
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) sc = mfma_bf16(__builtin_bit_cast(bf16x8, sX[(tg * KS + ks) * 64 + lane]), kb[ks], sc);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        f32x16 lo;
#pragma unroll
        for (int q4 = 2 * j; q4 < 2 * j + 2; ++q4) {
          const f32x4 sh = *(const f32x4*)(sShift + 32 * tg + 8 * q4 + 4 * half);
#pragma unroll
          for (int v = 0; v < 4; ++v) sc[4 * q4 + v] = fast_exp2(sc[4 * q4 + v] * p.wscale_l2e - sh[v]);
        }
        const bf16x8 wh = pack8(sc, j);
        const u32x4 hw = __builtin_bit_cast(u32x4, wh);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          lo[8 * j + 2 * k] = sc[8 * j + 2 * k] - __uint_as_float(hw[k] << 16);
          lo[8 * j + 2 * k + 1] = sc[8 * j + 2 * k + 1] - __uint_as_float(hw[k] & 0xFFFF0000u);
        }
        const bf16x8 wl = pack8(lo, j);
        bf16x8 bv[NC];
#pragma unroll
        for (int jt = 0; jt < NC; ++jt) bv[jt] = __builtin_bit_cast(bf16x8, sV[operand_chunk<D>(2 * tg + j, jt, lane)]);
#pragma unroll
        for (int jt = 0; jt < NC; ++jt) macc[jt] = mfma_bf16(wh, bv[jt], macc[jt]);
#pragma unroll
        for (int jt = 0; jt < NC; ++jt) macc[jt] = mfma_bf16(wl, bv[jt], macc[jt]);
      }
    }
    lds_barrier();   // the operand tiles have been read
    if (live) {
#pragma unroll
      for (int jt = 0; jt < NC; ++jt)
#pragma unroll
        for (int v = 0; v < 16; ++v) strip[cell(8 * (v / 4) + 4 * half + v % 4, jt)] = bf16_bits(macc[jt][v]);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int i = 0; i < NI; ++i)
        __builtin_nontemporal_store(*(const u32x4*)(strip + RT::row(i, lane) * D + RT::chunk(i, lane) * 8), (u32x4*)(mv + (size_t)slot0 * D + i * 512) + lane);
      __builtin_amdgcn_s_waitcnt(kWaitLds);   // the strip has been read
      asm volatile("" ::: "memory");
    }
  }

#pragma unroll
  for (int k0 = 0; k0 < NK; ++k0) {
    const int k = k0 * 4 + wave, g = k / NC, jt = k % NC;
    const uint32_t rho = 32 * g + col;
    if (k < NR * NC && rho < q.rows) {
      const f32x16 o = oacc[k0];
      const float sh = NR == 2 && g ? shift[NR - 1] : shift[0], z = NR == 2 && g ? zsum[NR - 1] : zsum[0];
      if (q.splits == 1) {
        const float inv = 1.0f / z;
        uint16_t* to = p.out + (((size_t)b * T + rho / p.G) * p.Hq + h * p.G + rho % p.G) * D + 32 * jt + 4 * half;
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) store4_bf16(to + 8 * q4, o[4 * q4] * inv, o[4 * q4 + 1] * inv, o[4 * q4 + 2] * inv, o[4 * q4 + 3] * inv);
      } else {
        const size_t at = ((size_t)unit * q.splits + split) * q.rows + rho;
        float* to = q.part + at * D + 32 * jt + 4 * half;
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) *(f32x4*)(to + 8 * q4) = (f32x4){o[4 * q4], o[4 * q4 + 1], o[4 * q4 + 2], o[4 * q4 + 3]};
        if (jt == 0 && half == 0) q.mz[at] = make_float2(sh, z);
      }
    }
  }
}

// out[row] = sum over the slot tiles of exp2(shift_s - shift) part_s / sum of the same of their sums, shift the largest.  One
// workgroup = one row; group k of D / 4 lanes takes the tiles k, k + groups, ..; the groups are added in order.
template <int D>
__global__ __launch_bounds__(256) void prefill_pass_merge_kernel(const PassParams q) {
  constexpr int L = D / 4, NG = 256 / L;
  __shared__ f32x4 sO[NG][L];
  __shared__ float sZ[NG], sM[4];
  const PrefillParams& p = q.c;
  const uint32_t unit = block_unit(), rho = blockIdx.x;
  if (unit >= p.B * p.Hkv) return;
  const uint32_t b = unit / p.Hkv, h = unit % p.Hkv;
  const int tid = threadIdx.x, g = tid / L, l = tid % L;
  const float2* mz = q.mz + (size_t)unit * q.splits * q.rows + rho;
  float m = kNegBig;
  for (uint32_t s = tid; s < q.splits; s += 256) m = fmaxf(m, mz[(size_t)s * q.rows].x);
  m = xor_max<1, 32>(m);
  if (tid % 64 == 0) sM[tid / 64] = m;
  __syncthreads();
  m = fmaxf(fmaxf(sM[0], sM[1]), fmaxf(sM[2], sM[3]));
  f32x4 o = {0.f, 0.f, 0.f, 0.f};
  float z = 0.f;
#pragma unroll 4
  for (uint32_t s = g; s < q.splits; s += NG) {
    const float2 v = mz[(size_t)s * q.rows];
    const float f = fast_exp2(v.x - m);
    z = __builtin_fmaf(v.y, f, z);
    o += *(const f32x4*)(q.part + (((size_t)unit * q.splits + s) * q.rows + rho) * D + 4 * l) * f;
  }
  sO[g][l] = o;
  if (l == 0) sZ[g] = z;
  __syncthreads();
  if (g == 0) {
#pragma unroll
    for (int k = 1; k < NG; ++k) {
      o += sO[k][l];
      z += sZ[k];
    }
    const float inv = 1.0f / z;
    store4_bf16(p.out + (((size_t)b * p.T + rho / p.G) * p.Hq + h * p.G + rho % p.G) * D + 4 * l, o[0] * inv, o[1] * inv, o[2] * inv, o[3] * inv);
  }
}

// ------------------------------------------------------------------ host side

// The shifts of the write rows, or of the read rows of a chunk that only reads (p.stats_read).
static hipError_t launch_stats(PrefillParams& p, hipStream_t s) {
  const uint32_t units = p.B * p.Hkv;
  const uint32_t rows = (p.has_write ? p.T : 0u) + (p.stats_read ? p.T * p.G : 0u);
  const bool d128 = p.d == 128;
  // Few rows of few memories leave compute units without a statistics workgroup (one fits each): split the keys, at
  // least 256 slots a share and at most 8 shares, and merge the shares' pairs in a launch of 5 us: 3 memories x 8 heads,
  // T = 333, M = 2112 (72 workgroups): 36 us in one share, 15 in three.  From 1024 slots on: 128 slots are 1.3 us of a
  // share's time, so below that the merge (5 us, and its launch) costs what the split gives.
  const uint64_t wgs = (uint64_t)((rows + kTC - 1) / kTC) * units;
  uint32_t most = p.has_write ? kMaxStatsSplit : 2 * p.d / 8 / p.G;
  if (most > kMaxStatsSplit) most = kMaxStatsSplit;
  p.stats_split = 1;
  while (p.M >= 1024 && p.stats_split < most && wgs * (p.stats_split + 1) <= 256 && p.M / (p.stats_split + 1) >= 256)
    ++p.stats_split;
  const dim3 gs = unit_grid((rows + kTC - 1) / kTC * p.stats_split, units);
  // Few slots: the kernel that fits two workgroups on a compute unit, where a workgroup's start and end are much of its
  // time, or where its own start (one key tile, not three) is most of the launch.  us, this kernel against the other:
  // d = 128, 1890 workgroups: M = 320 46 | 68, 1280 143 | 154, 2048 199 | 196, 3072 285 | 266; 512 workgroups: 640 22 | 26,
  // 1280 37 | 37, 2048 57 | 53; 256: 640 14.4 | 13.7, 2048 37 | 26; 24: 128 6.4 | 7.8, 384 9.3 | 9.9.  d = 64, 1890: 320
  // 31 | 46, 1280 81 | 93, 3072 178 | 187; 256: 640 9.1 | 9.6, 2048 22 | 19.
  // One round of workgroups, whole read-only chunk: d = 64, 32 workgroups: 512 19.6 | 20.2, 768 25.1 | 25.3, 896 27.7 | 26.7;
  // 255: 512 28.6 | 29.6, 768 33.4 | 34.6, 896 36.8 | 36.6; d = 128, 32: 384 23.8 | 24.2, 448 26.7 | 26.8, 576 31.9 | 31.3; 255:
  // 320 32.9 | 33.0, 384 35.3 | 35.0, 448 39.2 | 38.5.
  const bool brief =
      p.stats_split == 1 && (p.M <= (d128 ? 384u : 768u) || (wgs > 256 && p.M <= (d128 ? 1280u : 3072u)));
  if (brief && d128) hipLaunchKernelGGL(prefill_stats_short_kernel<128>, gs, dim3(512), 0, s, p);
  else if (brief) hipLaunchKernelGGL(prefill_stats_short_kernel<64>, gs, dim3(512), 0, s, p);
  else if (d128) hipLaunchKernelGGL(prefill_stats_kernel<128>, gs, dim3(512), 0, s, p);
  else hipLaunchKernelGGL(prefill_stats_kernel<64>, gs, dim3(512), 0, s, p);
  if (p.stats_split == 1) return hipGetLastError();
  {
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(prefill_stats_merge_kernel, unit_grid((rows + 255) / 256, units), dim3(256), 0, s, p);
  return hipGetLastError();
}

template <int D, int NT, int NR>
static hipError_t launch_pass(const PassParams& q, hipStream_t s) {
  const uint32_t units = q.c.B * q.c.Hkv;
  hipLaunchKernelGGL((prefill_begin_kernel<D, NT, NR>), unit_grid(q.shares + 1, units), dim3(256), 0, s, q);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((prefill_pass_kernel<D, NT, NR>), unit_grid(q.splits, units), dim3(256), 0, s, q);
  if ((e = hipGetLastError()) != hipSuccess || q.splits == 1) return e;
  hipLaunchKernelGGL((prefill_pass_merge_kernel<D>), unit_grid(q.rows, units), dim3(256), 0, s, q);
  return hipGetLastError();
}

// A chunk of few tokens in one pass: up to 32 read rows of a memory always; up to 64 rows (and tokens), whose workgroups are
// alone on a compute unit with d = 128, where a memory is one workgroup or the memories are few, so that the others' chains over
// a whole memory leave the chip idle, and the scratch holds them (below).  us a chunk, transpose, statistics, state and read launches | begin, pass and merge (430
// shapes): d = 128, G = 1: 3 memories of 192 slots, T = 5 24.6 | 13.6; 44 of 12864, T = 6 343 | 122; 108 of 4096, T = 10 176 | 98; 512
// of 4096, T = 32 564 | 426; d = 64: 234 of 3904, G = 4, T = 4 161 | 100, 1024 of 192, T = 32 68.7 | 64.5 (the smallest gain up to 32 rows).
// Up to 64 rows: d = 128, 6 of 12800, T = 55 255 | 60; 28 of 1088, T = 38 49 | 27; 1024 of 128, G = 4, T = 16 93 | 67; but 208 of 1152,
// T = 41 104 | 141; 128 of 6976, G = 3, T = 19 323 | 387; 66 of 576, T = 47 41.6 | 40.2; d = 64, 232 of 1088, T = 45 64.5 | 68.2.
// Its scratch lies where the other launches keep WV and the copies of MV, which are one after another: of a chunk of up to
// 128 tokens 2 d (128 + M) bytes per memory.  32 rows always fit, and 64 in one tile of
// slots, but none of 33 to 64 tokens at M = 64.  In several tiles: up to 32 tokens 60 rows, where 128 does not divide M 45 (M = 192), 51 (320)
// to 60; 33 tokens or more none at M = 192, 40 (320), 45 (256), 52 (512) to 61 (from 4096 on).
static bool pass_params(const PrefillParams& p, PassParams& q, int& nt, int& nr) {
  if (!p.has_write || !p.has_read || p.T > 64 || p.T * p.G > 64) return false;
  const uint64_t units = (uint64_t)p.B * p.Hkv, D = p.d;
  const uint32_t tiles = (p.M + 127) / 128;
  q.c = p;
  q.rows = p.T * p.G;
  if (q.rows > 32 && tiles > 1 && units > 64) return false;
  nt = p.T > 32 ? 2 : 1;
  nr = q.rows > 32 ? 2 : 1;
  q.splits = tiles;
  q.share_tiles = (tiles + kMaxStatsSplit - 1) / kMaxStatsSplit;
  q.shares = (tiles + q.share_tiles - 1) / q.share_tiles;
  const uint64_t wvt = units * nt * 32 * D * 2, qt = units * nr * 32 * D * 2, pairs = units * q.shares * p.T * 8;
  const uint64_t part = q.splits > 1 ? units * q.splits * q.rows : 0;
  if (2 * wvt + qt + pairs + part * (4 * D + 8) > units * (128 + p.M) * D * 2) return false;
  q.wvt = p.wvt;
  q.wqt = q.wvt + wvt / 2;
  q.qt = q.wqt + wvt / 2;
  q.part = (float*)(q.qt + qt / 2);
  q.mz = (float2*)(q.part + part * D);
  q.pairs = q.mz + part;
  return true;
}

bool prefill_one_pass(const PrefillParams& p) {
  PassParams q;
  int nt, nr;
  return pass_params(p, q, nt, nr);
}

hipError_t launch_prefill_bf16(const PrefillParams& p0, hipStream_t s) {
  {
    PassParams q;
    int nt, nr;
    if (pass_params(p0, q, nt, nr)) {
      if (p0.d == 128) return nt == 2 ? launch_pass<128, 2, 2>(q, s) : nr == 2 ? launch_pass<128, 1, 2>(q, s) : launch_pass<128, 1, 1>(q, s);
      return nt == 2 ? launch_pass<64, 2, 2>(q, s) : nr == 2 ? launch_pass<64, 1, 2>(q, s) : launch_pass<64, 1, 1>(q, s);
    }
  }
  PrefillParams p = p0;
  const uint32_t units = p.B * p.Hkv;
  // a chunk that writes normalises its read rows on the fly (prefill_read_online_kernel): statistics of
  // the write rows only
  p.stats_read = (p.has_read && !p.has_write) ? 1u : 0u;
  const uint32_t nb = (p.T + kTC - 1) / kTC;
  const bool d128 = p.d == 128;
  const dim3 block(256);
  hipError_t e;
  p.Tpad = nb * kTC;
  auto transpose = [&](int which) -> hipError_t {
    const dim3 g = unit_grid((which == 0 ? p.Tpad : p.M) / 64, units);
    if (d128) hipLaunchKernelGGL(prefill_transpose_kernel<128>, g, block, 0, s, p, which);
    else hipLaunchKernelGGL(prefill_transpose_kernel<64>, g, block, 0, s, p, which);
    return hipGetLastError();
  };
  if (p.has_write && (e = transpose(0)) != hipSuccess) return e;
  // with a write, the state kernel leaves MV_0 as the first snapshot on its way through
  if (p.has_read && !p.has_write && (e = transpose(1)) != hipSuccess) return e;

  // the pairs of a split launch (8 bytes a row and share) lie where a later launch of the chunk writes first: in the
  // snapshots (at least 8 KB per memory and sub-chunk) or, for a chunk that only reads, in the space of WV^T (2 d bytes a
  // token, G rows a token)
  p.stats_part = (float2*)(p.has_write ? p.snap : p.wvt);
  if ((e = launch_stats(p, s)) != hipSuccess) return e;

  // Row tiles of 128 read rows (T * G rows): G of each whole sub-chunk, as many as have a row of the last one.  All G of a
  // last sub-chunk of few tokens would be workgroups that walk the whole memory for nothing: us a chunk, all G | those
  // with a row: G = 8, Hkv = 8, M = 4096, d = 128: B = 8, T = 4 203 | 130, B = 32, T = 130 1631 | 1229 (a chunk that only reads
  // 174 | 106, 1534 | 1106); B = 32, M = 2048, d = 64, T = 10 296 | 89.  (Workgroups that return at once do not help: with G = 8 one
  // in eight has a row, and workgroups go to the eight XCDs in turn, so that one XCD would do all the work: 205.)
  auto read = [&]() -> hipError_t {
    p.c_begin = 0;
    const uint32_t left = p.T - (nb - 1) * kTC;
    const dim3 g = unit_grid((nb - 1) * p.G + (left * p.G + kTC - 1) / kTC, units);
    const dim3 rblock(512);
    if (p.has_write) {
      if (d128) hipLaunchKernelGGL((prefill_read_online_kernel<128>), g, rblock, 0, s, p);
      else hipLaunchKernelGGL((prefill_read_online_kernel<64>), g, rblock, 0, s, p);
    } else {
      if (d128) hipLaunchKernelGGL((prefill_read_only_kernel<128>), g, rblock, 0, s, p);
      else hipLaunchKernelGGL((prefill_read_only_kernel<64>), g, rblock, 0, s, p);
    }
    return hipGetLastError();
  };
  if (p.has_write) {
    const dim3 g = unit_grid((p.M + 127) / 128, units);
    // byte offset of the last lane's 16 bytes in 32 tokens' write queries: past 32 bits from 541201 heads of 128
    // (1082402 of 64) on
    const bool far = (31 * (uint64_t)p.Hkv * p.d + p.d - 8) * 2 > 0xFFFFFFFFu;
    if (d128 && far) hipLaunchKernelGGL((prefill_state_kernel<128, true>), g, dim3(256), 0, s, p);
    else if (far) hipLaunchKernelGGL((prefill_state_kernel<64, true>), g, dim3(256), 0, s, p);
    else if (d128) hipLaunchKernelGGL((prefill_state_kernel<128, false>), g, dim3(256), 0, s, p);
    else hipLaunchKernelGGL((prefill_state_kernel<64, false>), g, dim3(256), 0, s, p);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  // every sub-chunk reads its starting state from a copy of MV in the workspace (with a write: copy c, in operand
  // tiles, is what the state kernel left when it reached sub-chunk c, MV_0 for c = 0; without a write: the one
  // transposed copy made above serves all of them), so one launch serves all sub-chunks
  if (p.has_read && (e = read()) != hipSuccess) return e;
  return hipSuccess;
}

}  // namespace bct
