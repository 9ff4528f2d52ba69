// The MV pass for several query heads per KV head (bf16, G > 2; gfx950).
//
// The update of MV is the same read-modify-write stream as in bct_mv_pass.hip.
// What changes is the read: with G query heads the output is
//     out[g,:] = sum_m rw[g][m] * MV_new[m,:]          (G x M) . (M x d)
// and on the vector ALU that is G FMAs per element of MV: at G = 4 the pass is
// bound by those FMAs (and by every one of the 16 lanes of a slot row computing
// all G softmax weights again), not by memory.  Here the contraction over the
// wavefront's 32 slots runs on v_mfma_f32_16x16x32_bf16:
//   B operand = MV_new (exactly the bf16 values just stored), A operand = the softmax weights: mfma_read.  A lane computes
//     the weights of ONE query head (row l % 16; rows >= G hold zeros), as bf16 addends, a product each: d = 128 two (16 to 17
//     bits), d = 64 three (all 24), as this pass took the place of fp32 products there.  Share of bf16 outputs that are not the rounding
//     of the exact read: two 2.0e-3 to 2.9e-3, three and fp32 products 1e-4 to 3e-4; three cost 0 to 3 % of a step (G = 4, 32 memories of
//     2048 slots 14.75 -> 15.1 us, G = 8, 256 of 8192 the same).
// The products also sum over the lane groups, so no lane exchange of sums is needed.  d = 64, G = 8, 256 memories of 8192
// slots: 146 us the step against 305 with the read on the vector ALU.
//
// RESCORE (d = 128, keys shared by the batch): the scores are not read from memory but computed again from the
// workgroup's 16 KB of keys (from L2: every sequence's workgroups read the same table): two v_mfma_f32_16x16x32_bf16 per 32 inputs,
// key row 4 a + c of group n = slot 8 a + 4 n + c, column g = query head g, column 15 = the write row.  Lane
// (sub, sl) then holds, in the two groups, exactly the scores of head g = sub for its 8 slots, the A
// operand above; the write weights reach the 16 lanes of a slot row by a row broadcast from column 15.
// For large grids only (plan_mv_pass has the measurements); those take their normalisers from the launch.  What is left beside
// MV are the partial outputs, 512 G bytes a workgroup that the merge reads again (B = 64, Hkv = 8, G = 4, M = 8192: 134 MB both
// ways), so a workgroup takes two tiles of slots, one after the other.  180 registers, two wavefronts a SIMD; held to three:
// 395 us of that step against 391.
#include "bct_device.h"
#include "bct_internal.h"

namespace bct {

namespace {

template <bool WRITE, int BS, bool NORM, int U, bool RESCORE, int D, bool TILES>
__global__ __launch_bounds__(BS) void mv_pass_gqa_kernel(const DecodeParams p) {
  constexpr int LPS = D / 8, SPI = 64 / LPS, PARTS = ReadShape<LPS>::kParts;   // lanes per slot row, slots per load instruction
  constexpr int NB = U / 8, NW = BS / 64, SPB = NW * SPI * U;
  constexpr uint32_t W = WRITE ? 1u : 0u;
  constexpr int ADD = D == 64 ? 3 : 2;   // bf16 addends of a weight
  __shared__ float s_red[NW * kMaxG * D];

  static_assert(!RESCORE || (U == 8 && PARTS == 1), "a lane's slots are two MFMA groups of four");
  static_assert(PARTS == 1 || NB == 1, "a part's slots are eight, one block of loads");
  const uint32_t split = blockIdx.x, unit = block_unit();
  if (unit >= p.B * p.Hkv) return;
  const uint32_t b = unit / p.Hkv, h = unit % p.Hkv;
  const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64;
  const int sub = lane % LPS, sl = lane / LPS;   // 16-byte chunk of a slot row, group of U slots
  const int col = lane % 16, kg = lane / 16;     // query head (row of A), group of eight entries of the contraction
  const uint32_t R = p.R, G = p.G, M = p.M;

  u32x4 xq[4];   // RESCORE: this lane's query row (column sub)
  const bool wcol = WRITE && col == 15;
  if (RESCORE) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) xq[ks] = (u32x4){0u, 0u, 0u, 0u};
    if ((uint32_t)sub < G || wcol) {
      const uint16_t* x = wcol ? (const uint16_t*)p.wq + (size_t)b * p.kv_bstride + (size_t)h * D
                               : (const uint16_t*)p.q + (size_t)b * p.q_bstride + (size_t)(h * G + sub) * D;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) xq[ks] = *(const u32x4*)(x + ks * 32 + sl * 8);
    }
  }
  constexpr int NP = ReadShape<LPS>::kProducts;
  f32x4 acc[NP];
#pragma unroll
  for (int e = 0; e < NP; ++e) acc[e] = (f32x4){0.f, 0.f, 0.f, 0.f};
  // TILES: as many tiles of SPB slots as the plan's splits leave a workgroup (perhaps none the last), otherwise one
  const uint32_t n_tiles = (M + SPB - 1) / SPB, per = TILES ? (n_tiles + p.S - 1) / p.S : 1u, first = split * per;
  const uint32_t end = TILES ? min(first + per, n_tiles) : first + 1;
  float2 nw = make_float2(0.f, 0.f), nr = make_float2(0.f, 0.f);
  // stored scores: a tile's MV is requested while the one before is worked on
  constexpr bool AHEAD = TILES && !RESCORE;
  u32x4 next[AHEAD ? U : 1];
  auto request = [&](uint32_t tile) __attribute__((always_inline)) {
    const uint32_t slot = tile * SPB + wave * (SPI * U) + sl * U;
    const uint16_t* from = (const uint16_t*)p.mv + ((size_t)unit * M + slot) * D + sub * 8;
    if constexpr (AHEAD) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        next[u] = slot < M ? __builtin_nontemporal_load((const u32x4*)(from + (size_t)u * D)) : (u32x4){0u, 0u, 0u, 0u};
    }
  };
  if (AHEAD && first < end) request(first);
  for (uint32_t tile = first; tile < end; ++tile) {
    // M is a multiple of 64: the SPI * U (32 or 64) slots of a wavefront are all inside the memory or all outside
    const uint32_t slot0 = tile * SPB + wave * (SPI * U) + sl * U;
    const bool active = slot0 < M;
    uint16_t* mv = (uint16_t*)p.mv + ((size_t)unit * M + slot0) * D + sub * 8;

    // RESCORE: the keys, requested before MV
    u32x4 kf[RESCORE ? 2 : 1][4];
    if (RESCORE) {
      if (active) {
        const uint16_t* mk = (const uint16_t*)p.mk + ((size_t)h * M + tile * SPB + wave * (4 * U)) * D + sl * 8;
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
          for (int ks = 0; ks < 4; ++ks)
            kf[RESCORE ? n : 0][ks] = *(const u32x4*)(mk + (size_t)(8 * (sub / 4) + 4 * n + sub % 4) * D + ks * 32);
      }
    }
    u32x4 raw[U];
#pragma unroll
    for (int u = 0; u < U; ++u) raw[u] = AHEAD ? next[AHEAD ? u : 0] : (u32x4){0u, 0u, 0u, 0u};
    if (AHEAD) {
      if (tile + 1 < end) request(tile + 1);
    } else if (active) {
#pragma unroll
      for (int u = 0; u < U; ++u) raw[u] = __builtin_nontemporal_load((const u32x4*)(mv + (size_t)u * D));
    }

    if (tile == first) {
      // (max, 1/sum) of the write row and of this lane's read row (query head g = col)
      if (NORM) {
        // all rows' pairs are requested before the first is reduced (rows past R repeat row 0 and are dropped)
        TileStats ts[kMaxRows];
#pragma unroll
        for (uint32_t r = 0; r < kMaxRows; ++r)
          ts[r] = load_tile_stats(p.stats + ((size_t)unit * R + (r < R ? r : 0u)) * p.n_tiles, p.n_tiles, lane);
#pragma unroll
        for (uint32_t r = 0; r < kMaxRows; ++r) {
          if (r < R) {
            const float2 ms = merge_tile_stats(ts[r]);
            const float mx = ms.x;
            float inv = 1.0f / ms.y;
            if (WRITE && r == 0) {
              if (p.gate) inv *= p.gate[(size_t)b * p.gate_bstride + h];
              nw = make_float2(mx, inv);
            }
            if (r == W + (uint32_t)col && r >= W) nr = make_float2(mx, inv);
          }
        }
      } else {
        if (WRITE) nw = p.norm[(size_t)unit * R];
        if ((uint32_t)col < G) nr = p.norm[(size_t)unit * R + W + col];
      }
    }
    // rw: the lane's weights as an A operand (zero in lanes without a query head); ww: the write weights of its slots, with
    // stored scores only where they are used (here as well, the pass takes 1-2 % longer)
    const float* sc = p.scores + (size_t)unit * R * M + slot0;  // row r at sc + r * M
    float rw[PARTS][U], ww[U];
#pragma unroll
    for (int j = 0; j < PARTS; ++j)
#pragma unroll
      for (int u = 0; u < U; ++u) rw[j][u] = 0.f;
    if (RESCORE) {
#pragma unroll
      for (int u = 0; u < U; ++u) ww[u] = 0.f;
      if (active) {
        const float scale = wcol ? p.wscale_l2e : p.rscale_l2e;
        const float2 n2 = wcol ? nw : nr;
#pragma unroll
        for (int n = 0; n < 2; ++n) {
          const f32x4 c = score16<D>(kf[RESCORE ? n : 0], xq);
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const float e = fast_exp2(c[v] * scale - n2.x) * n2.y;
            if (WRITE) ww[4 * n + v] = row_lane<15>(e);
            rw[0][4 * n + v] = (uint32_t)col < G ? e : 0.f;
          }
        }
      }
    } else {
      if (active && (uint32_t)col < G) {
        // this lane's entries of the contraction: its own slots with one part, with two those of both groups
        const float* from = PARTS == 1 ? sc : p.scores + (size_t)unit * R * M + tile * SPB + wave * (SPI * U) + kg * (PARTS * U);
#pragma unroll
        for (int j = 0; j < PARTS; ++j)
#pragma unroll
          for (int k = 0; k < U / 4; ++k) {
            const f32x4 a = *(const f32x4*)(from + (size_t)(W + col) * M + j * U + 4 * k);
#pragma unroll
            for (int i = 0; i < 4; ++i) rw[j][4 * k + i] = fast_exp2(a[i] - nr.x) * nr.y;
          }
      }
    }
    // the lane's weights as bf16 addends, 8 slots per block: the A operands
    u32x4 aw[NB][PARTS][ADD];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int j = 0; j < PARTS; ++j) split_weights<ADD>(&rw[j][8 * nb], aw[nb][j]);

    if (WRITE && active) {
      if (!RESCORE) {
#pragma unroll
        for (int k = 0; k < U / 4; ++k) {
          const f32x4 a = *(const f32x4*)(sc + 4 * k);
#pragma unroll
          for (int i = 0; i < 4; ++i) ww[4 * k + i] = fast_exp2(a[i] - nw.x) * nw.y;
        }
      }
      float wvf[8];
      const uint16_t* wv = (const uint16_t*)p.wv + (size_t)b * p.kv_bstride + (size_t)h * D;
      unpack16<BF16>(*(const u32x4*)(wv + sub * 8), wvf);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float x[8];
        unpack16<BF16>(raw[u], x);
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = __builtin_fmaf(ww[u], wvf[e], x[e]);
        raw[u] = pack16_round<BF16>(x);
        __builtin_nontemporal_store(raw[u], (u32x4*)(mv + (size_t)u * D));
      }
    }

#pragma unroll
    for (int nb = 0; nb < NB; ++nb) mfma_read<LPS, ADD>(raw + 8 * nb, aw[nb], acc);
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const uint32_t g = 4 * kg + v;
    if (g < G) {
#pragma unroll
      for (int e = 0; e < NP; ++e) s_red[(wave * kMaxG + g) * D + ReadShape<LPS>::column(col) + e] = acc[e][v];
    }
  }
  __syncthreads();
  for (uint32_t i = tid; i < G * D; i += BS) {
    const uint32_t g = i / D, j = i % D;
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) v += s_red[(w * kMaxG + g) * D + j];
    const uint32_t hq = h * G + g;
    if (p.S == 1) {
      store_elem((uint16_t*)p.out, (size_t)b * p.q_bstride + (size_t)hq * D + j, v);
    } else {
      p.partial[(((size_t)split * p.B + b) * p.Hq + hq) * D + j] = v;
    }
  }
}

}  // namespace

template <int BS, int U, int D>
static void launch_gqa_bs(const DecodeParams& p, hipStream_t s) {
  const dim3 grid = unit_grid(p.S, (uint64_t)p.B * p.Hkv), block(BS);
  if constexpr (D == 128) {
    if (p.rescore) {
      // one tile a workgroup (an odd number of them, or keys out of reach) without the loop over tiles, which leaves a SIMD two
      // wavefronts where this has three: us a step, loop | this: G = 6, 1295 memories of 54 tiles 494 | 482, G = 3, 1950 of 45 548 | 535
      const bool one = (uint64_t)p.S * (BS * U * 16 / 256) >= p.M;
      if (p.has_write && one) hipLaunchKernelGGL((mv_pass_gqa_kernel<true, BS, false, U, true, D, false>), grid, block, 0, s, p);
      else if (p.has_write) hipLaunchKernelGGL((mv_pass_gqa_kernel<true, BS, false, U, true, D, true>), grid, block, 0, s, p);
      else if (one) hipLaunchKernelGGL((mv_pass_gqa_kernel<false, BS, false, U, true, D, false>), grid, block, 0, s, p);
      else hipLaunchKernelGGL((mv_pass_gqa_kernel<false, BS, false, U, true, D, true>), grid, block, 0, s, p);
      return;
    }
  }
  if constexpr (D == 64) {
    if ((uint64_t)p.S * 128 < p.M) {
      if (p.has_write && p.fuse_norm) hipLaunchKernelGGL((mv_pass_gqa_kernel<true, BS, true, U, false, D, true>), grid, block, 0, s, p);
      else if (p.has_write) hipLaunchKernelGGL((mv_pass_gqa_kernel<true, BS, false, U, false, D, true>), grid, block, 0, s, p);
      else if (p.fuse_norm) hipLaunchKernelGGL((mv_pass_gqa_kernel<false, BS, true, U, false, D, true>), grid, block, 0, s, p);
      else hipLaunchKernelGGL((mv_pass_gqa_kernel<false, BS, false, U, false, D, true>), grid, block, 0, s, p);
      return;
    }
  }
  if (p.has_write) {
    if (p.fuse_norm) hipLaunchKernelGGL((mv_pass_gqa_kernel<true, BS, true, U, false, D, false>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((mv_pass_gqa_kernel<true, BS, false, U, false, D, false>), grid, block, 0, s, p);
  } else {
    if (p.fuse_norm) hipLaunchKernelGGL((mv_pass_gqa_kernel<false, BS, true, U, false, D, false>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((mv_pass_gqa_kernel<false, BS, false, U, false, D, false>), grid, block, 0, s, p);
  }
}

// bf16, G > 2, a step with a read.  The launch shape is the plan's: 128 threads, 8 loads per lane
// (with d = 128 the kernel is written for any multiple of 8 loads; 16 measured slower, see plan_mv_pass).
hipError_t launch_stream_gqa(const DecodeParams& p, hipStream_t s) {
  if (p.G <= 2 || p.G > kMaxG || !p.has_read) return hipErrorInvalidConfiguration;
  if (p.mv_bs != 128 || p.mv_u != 8) return hipErrorInvalidConfiguration;
  if (p.rescore && (p.fuse_norm || p.d != 128 || p.mk_per_seq)) return hipErrorInvalidConfiguration;
  // with stored scores and d = 128 a workgroup has one tile of slots: the splits have to cover the memory
  if (!p.rescore && p.d == 128 && (uint64_t)p.S * 64 < p.M) return hipErrorInvalidConfiguration;
  if (p.d == 128) launch_gqa_bs<128, 8, 128>(p, s);
  else launch_gqa_bs<128, 8, 64>(p, s);
  return hipGetLastError();
}

}  // namespace bct
