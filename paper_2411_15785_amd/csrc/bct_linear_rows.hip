// The projections of the decoder stack for MANY token rows (a prompt chunk: batch x T rows; gfx950), where the
// product is a dense contraction bound by the matrix cores and no longer by streaming the weights.
//
// Both operands are already stored in MFMA operand order (packed weights, tiled activations), so a K step of 32
// inputs is a set of 1 KB tiles that go from memory to LDS unchanged (global_load_lds: 16 bytes per lane, no
// trip through registers) and are read back by the wavefronts as v_mfma_f32_16x16x32_bf16 operands with linear
// 16-byte LDS reads (no bank conflicts).  Row-major activations take the same path with one row of 64 bytes
// per 16 lanes.
//
// What bounds it: the matrix cores, once loads and LDS reads are out of their way.  Three things do that:
//   - four LDS stages, so that a tile is requested three K steps before it is used.  A wavefront waits only for
//     its own requests of the next stage (vmcnt leaves the two later stages in flight); the barrier that
//     follows makes the stage the workgroup's.  Each stage is a __shared__ array of its own: the compiler
//     then knows that reading one stage does not depend on requests into another and adds no wait.
//   - two wavefronts per SIMD that take turns ("ping"): while one issues the K step's products, the other
//     reads its operands of the next one from LDS and requests tiles; two barriers per K step keep them
//     half a step apart, and s_setprio lets the products go first.
//   - workgroup ids mapped so that the workgroups resident on one XCD cover 4 row tiles x consecutive
//     feature tiles: each operand panel enters that XCD's L2 once per four uses.
// With one stage ahead held in registers, one barrier per K step and no turns, the same 256 x 256 tile took
// 1353 us at 16384 rows x 11008 -> 4096 (1.09 PFLOP/s); this form takes 955 us (1.55 PFLOP/s); four stages
// without turns 1131 us; bands of 8 instead of 4 row tiles 1033 us.
//
// Where 256 x 256 tiles are too few for 256 compute units, smaller tiles follow; and where even 128 x 128 tiles
// leave every compute unit at most one workgroup of four wavefronts, two groups of wavefronts share a
// tile, each with half of the inputs, and are the two that take turns on a SIMD (see rows_shape for the choice
// and the measurements).  128 x 512 fills rounds where 256 wastes rows.
#include "bct_device.h"
#include "bct_linear.h"

namespace bct {

namespace {

// KS groups of WR x WC wavefronts; a wavefront owns 16 * MI token rows x 16 * NJ B-tile columns (SwiGLU: gate and
// up tiles alternate, so half as many output features); group g sums the K steps [KT * g / KS, ...).
// PAIR (row-major activations): the two K steps of a line are requested together, see request_rows.
template <bool SWIGLU, bool XT, bool PAIR, int MI, int NJ, int WR, int WC, int KS>
__global__ __launch_bounds__(64 * WR * WC * KS, 2) void linear_rows_kernel(
    const uint16_t* __restrict__ x, const u32x4* __restrict__ w, const u32x4* __restrict__ w2, const uint16_t* residual,
    LinearOut dst, uint32_t rows, uint32_t K, uint32_t NT, uint32_t out_tiled) {
  constexpr int NW = WR * WC;                      // wavefronts of a group
  constexpr int TA = MI * WR, TB = NJ * WC, TT = TA + TB;  // 1 KB tiles of a K step: activations, weights
  constexpr int ND = TT / NW, NA = TA / NW, NB = TB / NW;  // of them per wavefront
  static_assert(TA % NW == 0 && TB % NW == 0, "tiles must divide among the wavefronts");
  static_assert(!PAIR || !XT, "tiled activations have no half lines");
  constexpr int S = 4;                             // LDS stages
  constexpr bool PING = NW * KS == 8;              // two wavefronts per SIMD that take turns
  constexpr uint32_t HB = 4;                       // row tiles of a band
  constexpr uint32_t BM = 16 * MI * WR;            // token rows of a workgroup
  constexpr uint32_t CW = 16 * NJ;                 // B columns of a wavefront
  constexpr uint32_t BNF = CW * WC / (SWIGLU ? 2 : 1);  // output features of a workgroup
  __shared__ __attribute__((aligned(16))) u32x4 st0[KS * TT * 64];
  __shared__ __attribute__((aligned(16))) u32x4 st1[KS * TT * 64];
  __shared__ __attribute__((aligned(16))) u32x4 st2[KS * TT * 64];
  __shared__ __attribute__((aligned(16))) u32x4 st3[KS * TT * 64];

  const uint32_t RT = (rows + BM - 1) / BM, total = RT * NT, per = (total + 7) / 8;
  const uint32_t vid = (blockIdx.x % 8) * per + blockIdx.x / 8;
  if (vid >= total) return;   // the grid is 8 * per workgroups: every id below total comes up once
  // The last band takes the remainder as well (HB to 2 * HB - 1 row tiles): a band of one row tile of its own would read
  // every weight for that row tile alone.  us, own band | this: 320 rows, 11008 -> 4096 89.5 | 82.5, 4096 -> 12288 73 | 67,
  // 640 rows 107 | 102; 330 shapes 0.95 to 1.2, in the mean 1.004 to 1.02 for each tile (64 x 64: 434, 6464 -> 2176 35.6 |
  // 37.6, 283, 10752 -> 6016 125 | 106).  Not where two workgroups share a compute
  // unit (no turns): the two are 32 ids of their XCD apart, so in bands of HB they have the same row tile and its activations
  // from L1, in others not.  1060 rows, 928 -> 4480 21.0 | 24.3, 1598, 4000 -> 3456 56.2 | 62.6, 515, 10464 -> 7296 132 | 151 (but
  // 616, 8704 -> 6784 131 | 110).
  const uint32_t nfull = !PING ? RT / HB : RT < 2 * HB ? 0u : RT / HB - 1;
  uint32_t rt, nt;
  if (vid < nfull * HB * NT) {
    const uint32_t band = vid / (HB * NT), rem = vid % (HB * NT);
    nt = rem / HB;
    rt = band * HB + rem % HB;
  } else {
    const uint32_t rem = vid - nfull * HB * NT, cnt = RT - nfull * HB;
    nt = rem / cnt;
    rt = nfull * HB + rem % cnt;
  }
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64, jl = lane % 16, kg = lane / 16;
  const int grp = KS > 1 ? wv / NW : 0, wave = wv % NW, wr = wave / WC, wc = wave % WC;
  const uint32_t r0 = rt * BM, KT = K / 32;
  const uint32_t kfirst = grp ? (KT + 1) / 2 : 0u;                       // this group's K steps
  const uint32_t kcount = KS > 1 ? (grp ? KT / 2 : (KT + 1) / 2) : KT;
  const uint32_t kboth = KS > 1 ? KT / 2 : KT, kmost = KS > 1 ? (KT + 1) / 2 : KT;  // steps all groups / some group have

  // this lane's 16 bytes of the tiles wave, wave + NW, ... of a K step
  const char* src[ND];
  uint32_t step[ND];
#pragma unroll
  for (int j = 0; j < ND; ++j) {
    const uint32_t tile = wave + NW * j;
    if (tile < (uint32_t)TA) {
      if (XT) {
        const uint32_t g = min(r0 / 32 + tile / 2, (rows + 31) / 32 - 1);   // row groups past the end: a valid one
        src[j] = (const char*)(x + (((size_t)g * KT * 2 + tile % 2) * 64 + lane) * 8);
        step[j] = 2048;
      } else {
        const uint32_t r = min(r0 + tile * 16 + jl, rows - 1);
        src[j] = (const char*)(x + (size_t)r * K + kg * 8);
        step[j] = 64;
      }
    } else {
      // features past the end: the last ones again, not stored
      const uint32_t bt = tile - TA, most = dst.start[3] / 16 - 1;
      if (SWIGLU) src[j] = (const char*)(((bt % 2) ? w2 : w) + (size_t)min(nt * (TB / 2) + bt / 2, most) * KT * 64 + lane);
      else src[j] = (const char*)(w + (size_t)min(nt * TB + bt, most) * KT * 64 + lane);
      step[j] = 1024;
    }
  }

  f32x4 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  auto stage = [&](auto c) -> u32x4* {
    if constexpr (decltype(c)::v % S == 0) return st0;
    else if constexpr (decltype(c)::v % S == 1) return st1;
    else if constexpr (decltype(c)::v % S == 2) return st2;
    else return st3;
  };
  // one index into the stage each: the compiler loses track of which array an access belongs to when the
  // address is a long chain
  const int put0 = (grp * TT + wave) * 64, geta = (grp * TT + MI * wr) * 64 + lane, getb = (grp * TT + TA + NJ * wc) * 64 + lane;
  auto at = [&](uint32_t kt) { return min(kfirst + kt, KT - 1); };   // past the end: the last step again, never multiplied
  auto request = [&](auto c, uint32_t kt, auto first, auto last) {   // loads first .. last - 1 of step kt
    u32x4* s = stage(c);
    const uint32_t k = at(kt);
#pragma unroll
    for (int j = decltype(first)::v; j < decltype(last)::v; ++j) load_to_lds(src[j] + (size_t)k * step[j], s + put0 + NW * 64 * j);
  };
  // PAIR: a row's 64 bytes of a K step are half a line; the two steps of a line are requested together, before its other
  // half is evicted.
  auto request_rows = [&](auto c, uint32_t kt) {
    u32x4 *s0 = stage(c), *s1 = stage(Int<decltype(c)::v + 1>{});
    const uint32_t k0 = at(kt), k1 = at(kt + 1);
#pragma unroll
    for (int j = 0; j < NA; ++j) {
      load_to_lds(src[j] + (size_t)k0 * step[j], s0 + put0 + NW * 64 * j);
      load_to_lds(src[j] + (size_t)k1 * step[j], s1 + put0 + NW * 64 * j);
    }
    __builtin_amdgcn_sched_barrier(0);   // before the weights that are requested next: the waits count on it
  };
  // K step kt from stage c; requests step kt + S - 1 (PAIR: of the activations, in even steps, kt + 2 and kt + 3) into
  // stages whose reads all wavefronts have finished (they waited for them before the barrier that ended their step
  // kt - 1).  Left in flight at the end: what steps kt + 2 and kt + 3 need (PAIR: after an odd step only their weights,
  // as the activations of kt + 1 came with those of kt + 2).
  auto k_step = [&](auto c, uint32_t kt, auto last) {
    u32x4* s = stage(c);
    bf16x8 a[MI], b[NJ];
#pragma unroll
    for (int i = 0; i < NJ; ++i) b[i] = __builtin_bit_cast(bf16x8, s[getb + 64 * i]);
#pragma unroll
    for (int i = 0; i < MI; ++i) a[i] = __builtin_bit_cast(bf16x8, s[geta + 64 * i]);
    constexpr bool even = decltype(c)::v % 2 == 0;   // of kt as well
    constexpr int left = (S - 2) * (PAIR && !even ? NB : ND);
    if constexpr (PAIR && even) request_rows(Int<decltype(c)::v + 2>{}, kt + 2);
    request(Int<decltype(c)::v + S - 1>{}, kt + S - 1, Int<PAIR ? NA : 0>{}, Int<ND>{});
    if constexpr (PING) {
      __builtin_amdgcn_s_waitcnt(kWaitLds);
      __builtin_amdgcn_s_waitcnt(wait_vm(left));
      bare_barrier();
    }
    auto products = [&] {
      if constexpr (PING) __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
      if constexpr (PING) __builtin_amdgcn_s_setprio(0);
    };
    if constexpr (decltype(last)::v == 0) products();
    else if (kt < kcount) products();   // the second group of an odd number of steps has one fewer
    if constexpr (!PING) {
      // the operands have been read: a wavefront's products wait for them and come before the barrier
      __builtin_amdgcn_s_waitcnt(kWaitLds);
      __builtin_amdgcn_s_waitcnt(wait_vm(left));
    }
    bare_barrier();
  };

  // The wait counts requests from the last one back, here and in the loop, so the stages' order has to stand: nothing
  // is moved across the scheduling barriers (in the loop, bare_barrier has them).
  if constexpr (PAIR) request_rows(Int<0>{}, 0);
  request(Int<0>{}, 0, Int<PAIR ? NA : 0>{}, Int<ND>{});
  __builtin_amdgcn_sched_barrier(0);
  request(Int<1>{}, 1, Int<PAIR ? NA : 0>{}, Int<ND>{});
  __builtin_amdgcn_sched_barrier(0);
  request(Int<2>{}, 2, Int<PAIR ? NA : 0>{}, Int<ND>{});
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(wait_vm((S - 2) * (PAIR ? NB : ND)));
  bare_barrier();
  const bool second = PING && wv >= 4;   // the wavefront of a SIMD that is half a step behind
  if (second) bare_barrier();
  uint32_t kt = 0;
  for (; kt + S <= kboth; kt += S) {
    k_step(Int<0>{}, kt, Int<0>{});
    k_step(Int<1>{}, kt + 1, Int<0>{});
    k_step(Int<2>{}, kt + 2, Int<0>{});
    k_step(Int<3>{}, kt + 3, Int<0>{});
  }
  if (kt < kmost) k_step(Int<0>{}, kt, Int<1>{});
  if (kt + 1 < kmost) k_step(Int<1>{}, kt + 1, Int<1>{});
  if (kt + 2 < kmost) k_step(Int<2>{}, kt + 2, Int<1>{});
  if (KS > 1 && kt + 3 < kmost) k_step(Int<3>{}, kt + 3, Int<1>{});
  if (PING && !second) bare_barrier();   // every wavefront passes the same number of barriers
  __builtin_amdgcn_s_waitcnt(wait_vm(0));   // the stages are free once the last requests have arrived
  __syncthreads();

  // the row tiles this wavefront writes out: with two groups, the first half is summed and written by group 0,
  // the second by group 1
  constexpr int MO = MI / KS;
  f32x4 res[MO][NJ];
  if constexpr (KS > 1) {
    f32x4* ex = (f32x4*)(wave % 2 ? st1 : st0) + (wave / 2) * (2 * MO * NJ * 64);   // [for group][tile][lane]
#pragma unroll
    for (int i = 0; i < MO; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const f32x4 lo = acc[i][j], hi = acc[MO + i][j];
        f32x4 other;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          other[v] = grp ? lo[v] : hi[v];
          res[i][j][v] = grp ? hi[v] : lo[v];
        }
        ex[((1 - grp) * MO * NJ + i * NJ + j) * 64 + lane] = other;
      }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < MO; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const f32x4 o = ex[(grp * MO * NJ + i * NJ + j) * 64 + lane];
#pragma unroll
        for (int v = 0; v < 4; ++v) res[i][j][v] += o[v];   // group 0's sum + group 1's, either way round
      }
    __syncthreads();
  } else {
#pragma unroll
    for (int i = 0; i < MO; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) res[i][j] = acc[i][j];
  }

  // Output, one row tile of every wavefront at a time, through an LDS strip of the wavefront's own (so no
  // barriers).  Accumulator element v of a lane: token row 4 * kg + v of the row tile, column jl of B tile j.  Staging
  // columns: plain, B tile j at 16 * j; SwiGLU, B tile j = 2 * f + matrix at CW / 2 * matrix + 16 * f.
  constexpr int ES = CW + 4;                       // floats per staged row
  constexpr int CPR = (SWIGLU ? CW / 2 : CW) / 8;  // 16-byte output chunks per row
  constexpr int RPP = 64 / CPR < 16 ? 64 / CPR : 16;   // rows per pass
  static_assert((NW * KS + 1) / 2 * 16 * ES * 4 <= KS * TT * 1024, "the strips of four wavefronts fit a stage");
  float(*e)[ES] = (float(*)[ES])((wv % 2 ? (char*)st1 : (char*)st0) + (wv / 2) * (16 * ES * 4));
#pragma unroll
  for (int i = 0; i < MO; ++i) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int col = SWIGLU ? (int)(CW / 2) * (j % 2) + 16 * (j / 2) + jl : 16 * j + jl;
#pragma unroll
      for (int v = 0; v < 4; ++v) e[4 * kg + v][col] = res[i][j][v];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int cc = lane % CPR;
#pragma unroll
    for (int ps = 0; ps < 16 / RPP; ++ps) {
      const int rr = ps * RPP + lane / CPR;
      const uint32_t row = r0 + wr * (16 * MI) + (grp * MO + i) * 16 + rr;
      const uint32_t n = nt * BNF + wc * (BNF / WC) + 8 * cc;
      if (rr < 16 && row < rows && n < dst.start[3]) {
        float y[8];
        *(f32x4*)&y[0] = *(const f32x4*)&e[rr][8 * cc];
        *(f32x4*)&y[4] = *(const f32x4*)&e[rr][8 * cc + 4];
        const int which = n >= dst.start[2] ? 2 : n >= dst.start[1] ? 1 : 0;
        const uint32_t width = dst.start[which + 1] - dst.start[which], col = n - dst.start[which];
        const size_t oo = (size_t)row * width + col;
        if (SWIGLU) {
          float u[8];
          *(f32x4*)&u[0] = *(const f32x4*)&e[rr][CW / 2 + 8 * cc];
          *(f32x4*)&u[4] = *(const f32x4*)&e[rr][CW / 2 + 8 * cc + 4];
#pragma unroll
          for (int k = 0; k < 8; ++k) y[k] = y[k] / (1.0f + __expf(-y[k])) * u[k];
        } else if (residual) {
          float rv[8];
          unpack16<BF16>(*(const u32x4*)(residual + oo), rv);
#pragma unroll
          for (int k = 0; k < 8; ++k) y[k] += rv[k];
        }
        const u32x4 o = pack16_round<BF16>(y);
        if (out_tiled) ((u32x4*)dst.ptr[which])[tiled_chunk(row, col, width)] = o;
        else *(u32x4*)(dst.ptr[which] + oo) = o;
      }
    }
  }
}

// The tile of a shape.  It decides in how many parts K is summed as well, so a result's last bits depend on the
// row and feature counts (bctm_linear_tile tells).  The time of a launch is the number of rounds its workgroups take on 256 compute units
// times the K steps times what a step of a resident workgroup takes; measured us per K step at 640 and 16384
// rows, K = 11008 / 4096, one set of weights again and again, so out of the caches:
//   256 x 256             one workgroup per compute unit  0.46 (few) - 0.69 (chip full)
//   128 x 512             one                             0.80
//   128 x 256             one                             0.34 - 0.44
//   128 x 128             two of four wavefronts          0.26 alone on its compute unit, 0.46 for a pair
//   128 x 128, K in two   one                             0.19 - 0.25
//   128 x 64, K in two    one                             0.16
//   64 x 64, K in two     two                             0.11 alone, 0.19 for a pair
// so 256 x 256 wins where the chip is full (4 rounds of it against 16 of 128 x 128), the others where its
// workgroups are few: 640 rows x 11008 -> 4096 takes 157 us in 256 x 256, 117, 88, 67, 94 in the last four (with weights from
// memory, as a stack of layers has them, the 67 are 96).
// A compute unit gets 50 to 60 GB/s of operands then, however many stages are in flight (5 or 8 stages instead of 4:
// the same times), so the fewest bytes per compute unit win among the shapes that have one round of workgroups, and 128 x 64 is
// for where 64 x 64 would be pairs and 128 x 128 would leave compute units idle.  us, weights from memory, without | with it: 320
// rows, 11008 -> 4096 82.9 | 62.4, 4096 -> 4096 30.9 | 25.9, 5120 -> 5120 41.7 | 37.9; 384 85.2 | 70.4, 31.8 | 28.3, 42.4 | 36.3; 512
// 86.9 | 73.6, 33.5 | 29.8; 192, 2048 -> 6144 18.6 | 16.4; 1024, 2048 -> 2048 17.6 | 16.5; 700, 2048 -> 2048 15.3 | 15.6.
// 128 x 512 has the work of 256 x 256 and 5 / 4 of its loads; it is there for row counts that 256 wastes, where it saves
// a round of workgroups.  With weights from memory, us without | with it, tiled x: against 128 x 256 838 rows, 4096 -> 53248
// 367 | 326, 384, 8192 -> 37376 242 | 212; against 128 x 128 526, 4096 -> 66560 366 | 314, 319, 4096 -> 69632 239 | 216 (a predicted 2 %:
// the price of many pairs is low).  Against 256 x 256 it depends on K: up to 4096 885, 4096 -> 66560 426 | 414, 3690, 2048 ->
// 22528 280 | 269, 1057, 512 -> 68608 111 | 102 (44 shapes, 0.986 to 1.12 times as fast); from 5120 on a step of 256 x 256 takes 0.62 to
// 0.68, of 128 x 512 0.78 to 0.83, and where it saves one round of six or seven it loses: 1658, 8192 -> 24576 SwiGLU 1019 | 1070,
// 4654, 11008 -> 20992 1626 | 1676 (15 shapes, 0.95 to 1.015; on another card 0.96 to 1.0), hence 83 there, which leaves it one of
// five: 2135, 11008 -> 14592 SwiGLU 1103 | 1071 (7 shapes, 0.98 to 1.045).  A row-major x waits longer for its rows, and the wider
// tile wins in all 37 shapes: 4654, 11008 -> 20992 2105 | 1841, 1911, 1024 -> 50176 218 | 212.
// A count of columns that 128 does not divide leaves the last tile of every row of tiles partly used, in any shape: all of them
// are open to it, at what their whole tiles cost.
enum RowsShape { kTile256, kTile128x512, kTile128x256, kTile128, kTile128K2, kTile128x64K2, kTile64K2 };

RowsShape rows_shape(uint32_t rows, uint32_t bcols, uint32_t K, bool x_tiled) {
  auto tiles = [&](uint32_t bm, uint32_t bn) { return (uint64_t)((rows + bm - 1) / bm) * ((bcols + bn - 1) / bn); };
  // hundredths of a us per K step: one workgroup per compute unit at a time; two, a last one may have it alone
  auto one = [](uint64_t t, uint64_t cost) { return (t + 255) / 256 * cost; };
  auto two = [](uint64_t t, uint64_t alone, uint64_t pair) {
    const uint64_t rem = t % 512;
    return t / 512 * pair + (rem > 256 ? pair : rem ? alone : 0);
  };
  RowsShape best = kTile128;
  uint64_t cost = two(tiles(128, 128), 26, 46);
  auto take = [&](RowsShape s, uint64_t c) {
    if (c < cost) {
      cost = c;
      best = s;
    }
  };
  take(kTile128K2, one(tiles(128, 128), 25));
  take(kTile128x64K2, one(tiles(128, 64), 16));
  take(kTile64K2, two(tiles(64, 64), 11, 19));
  const bool ragged = bcols % 128 != 0;
  if (bcols % 256 == 0 || ragged) {
    take(kTile128x256, one(tiles(128, 256), 44));
    take(kTile256, one(tiles(256, 256), 69));
  }
  // (dear only against 256 x 256, which sums K in one part as well: the parts do not depend on x's order)
  if (bcols % 512 == 0 || ragged) take(kTile128x512, one(tiles(128, 512), best == kTile256 && x_tiled && K > 4096 ? 83 : 80));
  return best;
}

template <bool SWIGLU, bool XT, int MI, int NJ, int WR, int WC, int KS, bool PAIR = false>
void launch_shape(const void* x, const void* w, const void* w2, const void* residual, const LinearOut& dst, uint32_t rows,
                  uint32_t K, uint32_t bcols, bool out_tiled, hipStream_t s) {
  const uint32_t NT = (bcols + 16 * NJ * WC - 1) / (16 * NJ * WC), RT = (rows + 16 * MI * WR - 1) / (16 * MI * WR);
  hipLaunchKernelGGL((linear_rows_kernel<SWIGLU, XT, PAIR, MI, NJ, WR, WC, KS>), dim3(8 * ((RT * NT + 7) / 8)),
                     dim3(64 * WR * WC * KS), 0, s, (const uint16_t*)x, (const u32x4*)w, (const u32x4*)w2,
                     (const uint16_t*)residual, dst, rows, K, NT, out_tiled ? 1u : 0u);
}

template <bool SWIGLU, bool XT>
void launch_rows(const void* x, const void* w, const void* w2, const void* residual, const LinearOut& dst, uint32_t rows,
                 uint32_t K, uint32_t N, bool out_tiled, hipStream_t s) {
  const uint32_t bcols = SWIGLU ? 2 * N : N;
  const RowsShape shape = rows_shape(rows, bcols, K, XT);
  if constexpr (!SWIGLU && !XT) {
    // Row-major activations under 128 x 128 tiles (feature counts that 256 does not divide), many of them, and weights
    // that the last-level cache does not keep: in pairs.  us, in pairs | step by step, 70 shapes: 2894 rows, 10400 -> 11904
    // 872 | 972; 7647, 9120 -> 13184 2217 | 2411; 1172, 9792 -> 23936 794 | 839; 3463, 4416 -> 27520 1109 | 1205; 781, 5440 ->
    // 22912 300 | 298.  Fewer weights: 2236, 4288 -> 17280 415 | 390; K below 4000 up to 13 % slower.  Fewer
    // tiles (the activations of odd steps come later): 677, 10688 -> 11392 328 | 301.
    const uint64_t tiles = (uint64_t)((rows + 127) / 128) * ((N + 127) / 128);
    if (shape == kTile128 && (uint64_t)K * N >= (100u << 20) && tiles >= 850)
      return launch_shape<false, false, 4, 4, 2, 2, 1, true>(x, w, w2, residual, dst, rows, K, bcols, out_tiled, s);
  }
  switch (shape) {
    case kTile256: return launch_shape<SWIGLU, XT, 8, 4, 2, 4, 1>(x, w, w2, residual, dst, rows, K, bcols, out_tiled, s);
    case kTile128x512: return launch_shape<SWIGLU, XT, 4, 8, 2, 4, 1>(x, w, w2, residual, dst, rows, K, bcols, out_tiled, s);
    case kTile128x256: return launch_shape<SWIGLU, XT, 4, 4, 2, 4, 1>(x, w, w2, residual, dst, rows, K, bcols, out_tiled, s);
    case kTile128: return launch_shape<SWIGLU, XT, 4, 4, 2, 2, 1>(x, w, w2, residual, dst, rows, K, bcols, out_tiled, s);
    case kTile128K2: return launch_shape<SWIGLU, XT, 4, 4, 2, 2, 2>(x, w, w2, residual, dst, rows, K, bcols, out_tiled, s);
    case kTile128x64K2: return launch_shape<SWIGLU, XT, 2, 4, 4, 1, 2>(x, w, w2, residual, dst, rows, K, bcols, out_tiled, s);
    case kTile64K2: return launch_shape<SWIGLU, XT, 2, 2, 2, 2, 2>(x, w, w2, residual, dst, rows, K, bcols, out_tiled, s);
  }
}

}  // namespace

LinearTile linear_rows_tile(uint32_t rows, uint32_t K, uint32_t N, bool swiglu, bool x_tiled) {
  const uint32_t per = swiglu ? 2 : 1;   // B columns of a feature
  switch (rows_shape(rows, per * N, K, x_tiled)) {
    case kTile256: return {256, 256 / per, 1};
    case kTile128x512: return {128, 512 / per, 1};
    case kTile128x256: return {128, 256 / per, 1};
    case kTile128: return {128, 128 / per, 1};
    case kTile128K2: return {128, 128 / per, 2};
    case kTile128x64K2: return {128, 64 / per, 2};
    case kTile64K2: return {64, 64 / per, 2};
  }
  return {0, 0, 0};
}

hipError_t launch_linear_rows(const void* x, const void* w, const void* w2, const void* residual, const LinearOut& dst,
                              uint32_t rows, uint32_t K, uint32_t N, bool x_tiled, bool out_tiled, hipStream_t s) {
  if (w2) {
    if (x_tiled) launch_rows<true, true>(x, w, w2, residual, dst, rows, K, N, out_tiled, s);
    else launch_rows<true, false>(x, w, w2, residual, dst, rows, K, N, out_tiled, s);
  } else {
    if (x_tiled) launch_rows<false, true>(x, w, w2, residual, dst, rows, K, N, out_tiled, s);
    else launch_rows<false, false>(x, w, w2, residual, dst, rows, K, N, out_tiled, s);
  }
  return hipGetLastError();
}

}  // namespace bct
