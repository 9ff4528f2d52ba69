// The decode step of a mid-size cache as one launch (gfx950).
//
// The streaming step is three launches (scores, MV pass, merge), each of one round of workgroups or less at these
// sizes: their ramps, drains and gaps cost as much as the bytes.  Here one workgroup takes CW = d / CS columns of one
// memory (b, h) through the whole step.  It scores ALL M slots itself, so that the normaliser of section 3.2 step 2 is a
// workgroup barrier and no output has to be summed over workgroups:
//   A. scores of the write query and the G read queries against the M keys on the matrix cores (16 slots by 16 query rows,
//      1 + G of them used), to LDS as fp32.  Keys come to LDS in whole rows (lds_request), two tiles
//      ahead per wavefront, the 16-byte chunks of a row exchanged so that operand reads have no bank conflicts;
//   B. per row max of the scaled scores, then exp2(score * scale - max) in place, one rounding before the exponential, and its sum;
//   C. the columns of MV: load, fma(ww[m], wv, MV[m,:]), round, store, rw[g][m] times the value just stored;
//   D. the G output rows summed over lanes and wavefronts in a fixed order;
//   E. a step that writes keys: the same update of the memory's own keys, with the weights they gave.
// Sums over wavefronts are taken in halves and a score is rounded once on its way into the exponential, so the step is no further
// from 64 bits than the launches it takes the place of (fp32, root mean square of the output: 1.27e-7 at 4 memories of 64 slots with 64
// columns, where the one-workgroup launch has 1.33e-7; 1.55e-7 | 1.58e-7 streaming at 128 of 512; in a chain over the wavefronts and with
// scaled scores 1.38e-7 and 1.66e-7, and 0.05 us less a step).
// What bounds it: at few memories the chain of a workgroup (keys at about 64 bytes a cycle, one compute unit's share of L2),
// at many the bytes.  A quarter of a lane's MV loads are requested before the first score and the others as soon as the
// last keys are, so that MV streams while the keys come from the XCD's L2: workgroups are numbered so that those of one
// head, which read the same keys if the batch shares them, are on one XCD.  MV is read and written once whatever CS is; the
// keys are read CS times per memory.
#include "bct_device.h"
#include "bct_internal.h"

namespace bct {

namespace {

// Lanes 0 to 31 get the sum of a over the two halves of the wavefront, lanes 32 to 63 that of b.
__device__ __forceinline__ float half_sums(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// Rows of 16 lanes in pairs: the even row gets the sum of a over the two, the odd row that of b.
__device__ __forceinline__ float row_sums(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// The sum of term(0) .. term(N - 1), N a power of two, in halves: log2(N) roundings deep.
template <int N, typename F>
__device__ __forceinline__ float sum_of(F term) {
  float t[N];
#pragma unroll
  for (int i = 0; i < N; ++i) t[i] = term(i);
#pragma unroll
  for (int n = N / 2; n > 0; n /= 2)
#pragma unroll
    for (int i = 0; i < n; ++i) t[i] += t[i + n];
  return t[0];
}

// 16 key rows by up to 16 query rows; chunk ks of a lane: 16 bytes of its row (row l % 16) at 16 * (4 ks + l / 16).
// Element v of the result: key row 4 * (l / 16) + v, query row l % 16.
template <typename DT, int D>
__device__ __forceinline__ f32x4 score_tile(const u32x4* key, const u32x4* query) {
  if constexpr (DT::kElemsPerVec == 8) {
    return score16<D>(key, query);
  } else {
    // four inputs a product, then pairs, as the streaming launches add (4 inputs a lane, then pairs of lanes): one chain of
    // products over all of d rounds more often (out against 64 bits, d = 64, M = 64: 1.4e-7 where those have 1.2e-7)
    constexpr int N = D / 16;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    auto two = [&](int ks, int j) -> f32x4 {
      return __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(key[ks][j]), __uint_as_float(query[ks][j]), zero, 0, 0, 0) +
             __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(key[ks][j + 1]), __uint_as_float(query[ks][j + 1]), zero, 0, 0, 0);
    };
    f32x4 c[N];
#pragma unroll
    for (int ks = 0; ks < N; ++ks) {
      c[ks] = two(ks, 0);
      c[ks] += two(ks, 2);
      if (ks % 2) c[ks - 1] += c[ks];
      if (ks % 4 == 3) c[ks - 3] += c[ks - 1];
    }
    if (N == 8) c[0] += c[4];
    return c[0];
  }
}

template <typename DT, int D, int GT, int U, int CS, int BS>
__global__ __launch_bounds__(BS) void decode_whole_kernel(const DecodeParams p, const KeyWrite kw, uint32_t per_xcd) {
  typedef typename DT::elem elem;
  constexpr int E = DT::kElemsPerVec;
  constexpr int RB = D * (int)sizeof(elem);   // bytes of a slot row
  constexpr int NW = BS / 64;
  constexpr int CW = D / CS;             // columns of MV this workgroup updates and reads
  constexpr int LPS = CW / E;            // lanes per slot row
  constexpr int SPI = 64 / LPS;          // slots per load instruction of a wavefront
  constexpr int KS = RB / 64;            // 16-byte chunks of a row per lane
  constexpr int TILE = 16 * RB;          // bytes of a key tile
  constexpr int REQ = TILE / 1024;       // requests per tile (1 KB each)
  constexpr int LPR = RB / 16, RPR = 64 / LPR;   // lanes per key row and key rows of a request
  constexpr int EARLY = U / 4;           // MV loads requested before the first score
  // bf16, GT > 2: the read runs on the matrix cores as well (step C)
  constexpr bool MF = E == 8 && GT > 2;
  static_assert((E == 8 && (LPS == 8 || LPS == 16)) || (E == 4 && (LPS == 16 || LPS == 32)), "lane layouts of steps C and D");
  static_assert(!MF || U % 8 == 0, "a lane's slots are groups of eight");
  static_assert(2 * REQ + U <= kMostVm, "the counter of outstanding operations");

  extern __shared__ __attribute__((aligned(16))) char s_mem[];
  char* ring = s_mem;                                      // [NW][2][TILE]
  float* s_w = (float*)(s_mem + NW * 2 * TILE);            // [R][M]
  const uint32_t R = p.R, G = p.G, M = p.M, W = p.has_write;
  float* s_stat = s_w + (size_t)R * M;                     // [2][NW][16]

  // head-major order, a contiguous part of it for each XCD
  const uint32_t n = blockIdx.x % 8 * per_xcd + blockIdx.x / 8;
  if (n >= p.B * p.Hkv * CS) return;
  const uint32_t cs = n % CS, h = n / CS / p.B, b = n / CS % p.B, unit = b * p.Hkv + h;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64;
  const int col = lane % 16, kg = lane / 16;               // scoring: query row / key row, chunk of four
  const int sub = lane % LPS, sl = lane / LPS;             // MV: 16-byte chunk of the columns, slot of the load

  u32x4 xq[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) xq[ks] = (u32x4){0u, 0u, 0u, 0u};
  const bool wrow = W && col == 0;
  if ((uint32_t)col < R) {
    const elem* x = wrow ? (const elem*)p.wq + (size_t)b * p.kv_bstride + (size_t)h * D
                         : (const elem*)p.q + (size_t)b * p.q_bstride + (size_t)(h * G + (col - W)) * D;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) xq[ks] = *(const u32x4*)((const char*)x + (ks * 4 + kg) * 16);
  }

  // ---- A
  const char* mk = (const char*)p.mk + (size_t)(p.mk_per_seq ? unit : h) * M * RB;
  const uint32_t tiles = M / 16, rounds = (tiles + NW - 1) / NW;
  // LDS row r of a tile holds the key row's chunk c at c ^ swap(r): the 16 rows of an operand read, all at chunk c, then
  // cover the 16 chunks of 256 bytes once
  auto swap = [](int r) -> int { return RB == 128 ? r / 2 : r; };
  const uint32_t off0 = (lane / LPR) * RB + ((lane % LPR) ^ swap(lane / LPR)) * 16;
  auto request = [&](uint32_t i) {
    const uint32_t t = min(i * NW + wave, tiles - 1);      // past the end: the last tile again, not counted
    const char* from = mk + (size_t)t * TILE;
    char* to = ring + (wave * 2 + (i & 1)) * TILE;
#pragma unroll
    for (int q = 0; q < REQ; ++q) lds_request(from, (off0 ^ (swap(q * RPR) * 16)) + q * 1024, to + q * 1024);
  };
  char* mv = (char*)p.mv + (size_t)unit * M * RB + cs * CW * sizeof(elem) + sub * 16;
  u32x4 raw[U];
  // The slots of load u: first of the wavefront's (M is a multiple of 64: they are all inside the memory or all
  // outside), this lane's.  MF: a lane's slots of 8 loads are consecutive.
  auto first_slot = [&](int u) -> uint32_t { return MF ? (u / 8 * NW + wave) * (8 * SPI) : (u * NW + wave) * SPI; };
  auto slot_of = [&](int u) -> uint32_t { return first_slot(u) + (MF ? sl * 8 + u % 8 : sl); };
  auto load_mv = [&](int u) {
    if (first_slot(u) < M) raw[u] = __builtin_nontemporal_load((const u32x4*)(mv + (size_t)slot_of(u) * RB));
  };
  const float scale = wrow ? p.wscale_l2e : p.rscale_l2e;
  float mx = -INFINITY;
  auto score = [&](uint32_t i) {
    const char* from = ring + (wave * 2 + (i & 1)) * TILE;
    u32x4 kf[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) kf[ks] = *(const u32x4*)(from + col * RB + ((ks * 4 + kg) ^ swap(col)) * 16);
    f32x4 c = score_tile<DT, D>(kf, xq);
    const uint32_t t = i * NW + wave;
    if (t < tiles) {
#pragma unroll
      for (int v = 0; v < 4; ++v) mx = fmaxf(mx, c[v] * scale);
      if ((uint32_t)col < R) *(f32x4*)(s_w + (size_t)col * M + t * 16 + kg * 4) = c;
    }
  };
  // Memory operations of a wavefront complete in order, so tile i is there once no more are outstanding than were issued
  // after its requests: `younger` of them, rounded down to a multiple of four.
  auto arrived = [&](uint32_t younger) {
    if (younger >= 20) __builtin_amdgcn_s_waitcnt(wait_vm(20));
    else if (younger >= 16) __builtin_amdgcn_s_waitcnt(wait_vm(16));
    else if (younger >= 12) __builtin_amdgcn_s_waitcnt(wait_vm(12));
    else if (younger >= 8) __builtin_amdgcn_s_waitcnt(wait_vm(8));
    else if (younger >= 4) __builtin_amdgcn_s_waitcnt(wait_vm(4));
    else __builtin_amdgcn_s_waitcnt(wait_vm(0));
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  uint32_t loads = 0;
#pragma unroll
  for (int u = 0; u < U; ++u) loads += first_slot(u) < M ? 1u : 0u;
  const uint32_t early = min(loads, (uint32_t)EARLY), late = loads - early;
  request(0);
  if (rounds > 1) request(1);
#pragma unroll
  for (int u = 0; u < EARLY; ++u) load_mv(u);
  uint32_t i = 0;
  for (; i + 2 < rounds; ++i) {
    arrived(REQ + (i < 2 ? early : 0u));
    score(i);
    __builtin_amdgcn_s_waitcnt(kWaitLds);                  // the stage has been read
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    request(i + 2);
  }
#pragma unroll
  for (int u = EARLY; u < U; ++u) load_mv(u);
  asm volatile("" ::: "memory");
  for (; i < rounds; ++i) {
    arrived((i + 1 < rounds ? REQ : 0u) + late + (i < 2 ? early : 0u));
    score(i);
  }

  // ---- B: the lanes of a query row hold its scores at kg * 4 .. + 3 of their tiles
  const size_t row0 = (size_t)min((uint32_t)col, R - 1) * M;
  mx = xor_max<16, 32>(mx);
  if (kg == 0) s_stat[wave * 16 + col] = mx;
  lds_barrier();
#pragma unroll
  for (int w = 0; w < NW; ++w) mx = fmaxf(mx, s_stat[w * 16 + col]);
  float sm = 0.f;
  for (i = 0; i < rounds; ++i) {
    const uint32_t t = i * NW + wave;
    if (t < tiles && (uint32_t)col < R) {
      f32x4* at = (f32x4*)(s_w + row0 + t * 16 + kg * 4);
      f32x4 e = *at;
#pragma unroll
      for (int v = 0; v < 4; ++v) e[v] = fast_exp2(__builtin_fmaf(e[v], scale, -mx));
      sm += (e[0] + e[1]) + (e[2] + e[3]);
      *at = e;
    }
  }
  sm = xor_sum<16, 32>(sm);
  if (kg == 0) s_stat[NW * 16 + wave * 16 + col] = sm;
  lds_barrier();
  sm = sum_of<NW>([&](int w) { return s_stat[NW * 16 + w * 16 + col]; });
  // lane r of the wavefront has row r's normaliser; a step size scales the write row's
  const float inv = 1.0f / sm;
  const float inv0 = __shfl(inv, 0, 64), invw = W && p.gate ? inv0 * p.gate[(size_t)b * p.gate_bstride + h] : inv0;

  // ---- C
  float wvf[E];
#pragma unroll
  for (int e = 0; e < E; ++e) wvf[e] = 0.f;
  if (W) unpack16<DT>(*(const u32x4*)((const elem*)p.wv + (size_t)b * p.kv_bstride + (size_t)h * D + cs * CW + sub * E), wvf);
  float* s_red = (float*)ring;   // [NW][GT][CW]; every key tile has been read
  if constexpr (!MF) {
    float invr[GT], acc[GT][E];
#pragma unroll
    for (int g = 0; g < GT; ++g) {
      invr[g] = __shfl(inv, (int)W + g, 64);
#pragma unroll
      for (int e = 0; e < E; ++e) acc[g][e] = 0.f;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (first_slot(u) < M) {
        const uint32_t slot = slot_of(u);
        float x[E];
        unpack16<DT>(raw[u], x);
        if (W) {
          const float ww = s_w[slot] * invw;
#pragma unroll
          for (int e = 0; e < E; ++e) x[e] = __builtin_fmaf(ww, wvf[e], x[e]);
          __builtin_nontemporal_store(pack16_round<DT>(x), (u32x4*)(mv + (size_t)slot * RB));
        }
        if (p.has_read) {
#pragma unroll
          for (int g = 0; g < GT; ++g) {
            if ((uint32_t)g < G) {
              const float rw = s_w[(size_t)(W + g) * M + slot] * invr[g];
#pragma unroll
              for (int e = 0; e < E; ++e) acc[g][e] = __builtin_fmaf(rw, x[e], acc[g][e]);
            }
          }
        }
      }
    }
    // sum over the lanes of a column chunk: swaps of half wavefronts, then of neighbouring rows of 16, leave every lane
    // E / 2 and then E / 4 of its chunk's columns
    if (p.has_read) {
#pragma unroll
      for (int g = 0; g < GT; ++g) {
        float r[E / 2];
#pragma unroll
        for (int e = 0; e < E / 2; ++e) r[e] = half_sums(acc[g][e], acc[g][e + E / 2]);
        float* to = s_red + (wave * GT + g) * CW + sub * E;
        if constexpr (E == 4 && LPS == 32) {
          *(float2*)(to + 2 * (lane / 32)) = make_float2(r[0], r[1]);
        } else if constexpr (E == 4) {
          to[kg] = row_sums(r[0], r[1]);
        } else {
          const float r0 = row_sums(r[0], r[2]), r1 = row_sums(r[1], r[3]);
          if constexpr (LPS == 16) {
            *(float2*)(to + 2 * kg) = make_float2(r0, r1);
          } else {   // lanes l and l ^ 8 hold the same chunk
            const float t0 = r0 + dpp_partner<0x128>(r0), t1 = r1 + dpp_partner<0x128>(r1);   // row_ror:8
            to[2 * kg + lane / 8 % 2] = lane / 8 % 2 ? t1 : t0;
          }
        }
      }
    }
  } else {
    // as the MV pass for several query heads: weights of 32 slots times the values just stored.  Three bf16 addends a weight (see
    // split_weights): with two, 20 of every 10000 outputs were not the rounding of the exact read, in M <= 128 and d = 64 where fp32
    // products were used before; the third costs 0.1 to 0.3 us of a step (G = 4, 32 memories of 64 slots 4.85 -> 5.15).
    constexpr int PARTS = ReadShape<LPS>::kParts, NP = ReadShape<LPS>::kProducts;
    const float invr = __shfl(inv, (int)min(W + (uint32_t)col, R - 1), 64);
    const size_t rrow = (size_t)min(W + (uint32_t)col, R - 1) * M;
    f32x4 acc[NP];
#pragma unroll
    for (int e = 0; e < NP; ++e) acc[e] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ub = 0; ub < U / 8; ++ub) {
      if (first_slot(ub * 8) < M) {
        const uint32_t first = first_slot(ub * 8), own = slot_of(ub * 8);
        if (W) {
          float ww[8];
          *(f32x4*)&ww[0] = *(const f32x4*)(s_w + own);
          *(f32x4*)&ww[4] = *(const f32x4*)(s_w + own + 4);
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            float x[8];
            unpack16<BF16>(raw[ub * 8 + u], x);
            const float w = ww[u] * invw;
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = __builtin_fmaf(w, wvf[e], x[e]);
            raw[ub * 8 + u] = pack16_round<BF16>(x);
            __builtin_nontemporal_store(raw[ub * 8 + u], (u32x4*)(mv + (size_t)(own + u) * RB));
          }
        }
        if (p.has_read) {
          u32x4 aw[PARTS][3];
#pragma unroll
          for (int j = 0; j < PARTS; ++j) {
            float rw[8];
            const float* from = s_w + rrow + first + (kg * PARTS + j) * 8;
            *(f32x4*)&rw[0] = *(const f32x4*)from;
            *(f32x4*)&rw[4] = *(const f32x4*)(from + 4);
#pragma unroll
            for (int u = 0; u < 8; ++u) rw[u] = (uint32_t)col < G ? rw[u] * invr : 0.f;
            split_weights<3>(rw, aw[j]);
          }
          mfma_read<LPS, 3>(raw + ub * 8, aw, acc);
        }
      }
    }
    if (p.has_read) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const uint32_t g = 4 * kg + v;
        if (g < G) {
          float* to = s_red + ((size_t)wave * GT + g) * CW + ReadShape<LPS>::column(col);
#pragma unroll
          for (int e = 0; e < NP; e += 4) *(f32x4*)(to + e) = (f32x4){acc[e][v], acc[e + 1][v], acc[e + 2][v], acc[e + 3][v]};
        }
      }
    }
  }

  // ---- E: MK += kappa * ww^T wk on this memory's own keys (CS = 1: nobody else reads them)
  if (CS == 1 && kw.wk) {
    char* keys = (char*)kw.mk + (size_t)unit * M * RB + sub * 16;
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (first_slot(u) < M) raw[u] = *(const u32x4*)(keys + (size_t)slot_of(u) * RB);
    const float invk = kw.gate ? inv0 * kw.gate[(size_t)b * p.gate_bstride + h] : inv0;
    unpack16<DT>(*(const u32x4*)((const elem*)kw.wk + (size_t)b * p.kv_bstride + (size_t)h * D + sub * E), wvf);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (first_slot(u) < M) {
        const uint32_t slot = slot_of(u);
        float x[E];
        unpack16<DT>(raw[u], x);
        const float ww = s_w[slot] * invk;
#pragma unroll
        for (int e = 0; e < E; ++e) x[e] = __builtin_fmaf(ww, wvf[e], x[e]);
        __builtin_nontemporal_store(pack16_round<DT>(x), (u32x4*)(keys + (size_t)slot * RB));
      }
    }
  }

  // ---- D
  if (p.has_read) {
    lds_barrier();
    for (uint32_t k = tid; k < G * CW; k += BS) {
      const uint32_t g = k / CW, j = k % CW;
      const float v = sum_of<NW>([&](int w) { return s_red[(w * GT + g) * CW + j]; });
      store_elem((elem*)p.out, (size_t)b * p.q_bstride + (size_t)(h * G + g) * D + cs * CW + j, v);
    }
  }
}

template <typename DT, int D, int GT, int U, int CS, int BS>
hipError_t launch(const DecodeParams& p, const KeyWrite& kw, hipStream_t s) {
  const uint32_t wgs = p.B * p.Hkv * CS, per_xcd = (wgs + 7) / 8;
  const size_t lds = whole_lds_bytes(BS, D * sizeof(typename DT::elem), p.R, p.M);
  hipLaunchKernelGGL((decode_whole_kernel<DT, D, GT, U, CS, BS>), dim3(8 * per_xcd), dim3(BS), lds, s, p, kw, per_xcd);
  return hipGetLastError();
}

// 1024 threads only where 512 cannot hold the memory's columns with the most loads a lane has
template <typename DT, int D, int GT, int CS>
hipError_t launch_u(const DecodeParams& p, const WholePlan& w, const KeyWrite& kw, hipStream_t s) {
  constexpr bool MF = DT::kElemsPerVec == 8 && GT > 2;
  const uint32_t u = whole_loads(w.threads, D / CS * sizeof(typename DT::elem), p.M);
  if (w.threads == 1024) {
    // 128 registers a lane: the matrix-core read's accumulators or fp32 scores beside 16 loads do not fit
    if constexpr (DT::kElemsPerVec == 8 && !MF)
      if (u <= 16) return launch<DT, D, GT, 16, CS, 1024>(p, kw, s);
    return hipErrorInvalidConfiguration;
  }
  if constexpr (!MF)
    if (u <= 4) return launch<DT, D, GT, 4, CS, 512>(p, kw, s);
  if (u <= 8) return launch<DT, D, GT, 8, CS, 512>(p, kw, s);
  if (u <= 16) return launch<DT, D, GT, 16, CS, 512>(p, kw, s);
  return hipErrorInvalidConfiguration;
}

template <typename DT, int D>
hipError_t launch_g(const DecodeParams& p, const WholePlan& w, const KeyWrite& kw, hipStream_t s) {
  constexpr int G4 = DT::kElemsPerVec == 8 ? (int)kMaxG : 4;   // bf16: one instantiation for more than two query heads
  if constexpr (D == 128)
    if (w.workgroups == 2)
      return p.G == 1 ? launch_u<DT, D, 1, 2>(p, w, kw, s) : p.G == 2 ? launch_u<DT, D, 2, 2>(p, w, kw, s)
             : p.G <= 4 ? launch_u<DT, D, G4, 2>(p, w, kw, s) : launch_u<DT, D, (int)kMaxG, 2>(p, w, kw, s);
  return p.G == 1 ? launch_u<DT, D, 1, 1>(p, w, kw, s) : p.G == 2 ? launch_u<DT, D, 2, 1>(p, w, kw, s)
         : p.G <= 4 ? launch_u<DT, D, G4, 1>(p, w, kw, s) : launch_u<DT, D, (int)kMaxG, 1>(p, w, kw, s);
}

}  // namespace

// Which steps are one launch.  us of a step inside a HIP graph, caches with workspaces of their own taking turns: streaming
// launches (for M <= 128 the one-launch step of bct_fused.hip) / this kernel, n memories.
//   bf16, d = 128, G = 1: M = 64: n = 4 5.5 / 3.9, 256 6.2 / 4.7, 1024 11.0 / 11.7; M = 256: 64 9.5 / 6.3, 256 12.5 / 9.1,
//     1024 28.7 / 28.7; M = 512: 128 14.0 / 10.3, 256 17.1 / 15.7, 512 29.0 / 30.9; M = 1024: 4 9.5 / 12.9, 64 14.4 / 15.4,
//     128 19.2 / 17.2, 256 29.2 / 30.7
//   G = 2: M = 256, n = 256 16.4 / 9.9; M = 512, 1024 65.7 / 59.6; G = 8: M = 256, 256 20.6 / 9.7; M = 512, 1024 80 / 60
//   d = 64, G = 8: M = 512, n = 64 13 / 8.8, 1024 58 / 32; fp32, d = 128, G = 1: M = 128, n = 4 11.8 / 5.8, M = 320, 24 10.7 / 11.4
//   fp32, d = 64, G = 4: M = 128, n = 64 11.5 / 6.0, M = 512, 256 26.5 / 17.4
//   keys per sequence that move: d = 64, G = 1, M = 256, n = 256 26.1 / 13.9
// Two workgroups per memory while they still are one round of a workgroup per compute unit (the keys are then read twice:
// only keys shared by the batch, which stay in L2), 512 threads while the columns of M slots fit 16 loads a lane: 1024 are up
// to 6 % faster at 512 slots, 30 % slower at 64.  The borders, as the ratio of the streaming launches' time to this kernel's at n
// memories (3300 shapes, 3045 of them taken: 0.96 at the least, 1.42 in the geometric mean):
//   few memories: the chain of a workgroup over its keys is the step, streaming splits M over workgroups.  Ratio by KB of values a
//     memory, one workgroup: G = 1 bf16 64 KB 1.3, 80 1.05, 96 0.92, f32 80 1.01, 96 0.94; G = 2 bf16 88 1.05, 96 0.98 to 1.04, 104 0.95,
//     128 0.84, f32 96 1.03, 112 0.93, 128 0.84; G > 2 up to 128 1.0 to 1.7.  Two workgroups: G = 1 128 1.1, 160 0.96; G > 1 160 1.0 to
//     1.4.  32 memories and more, which streaming feels: G = 1, two workgroups 160 KB 1.08, f32 96 1.05 to 1.2, keys per sequence 96 1.08 to
//     1.26; G = 2 104 1.04 to 1.13, keys per sequence 128 1.04 to 1.18.  fp32, G = 1, whose dot products cost streaming least, up to 127
//     memories (96 KB at 64 of them 1.12);
//   two workgroups of more than 128 memories, a second round: n = 129 costs what 256 do.  bf16 G = 3 n = 129 0.81 to 0.94, 160 0.90 to
//     0.98, 192 1.0 to 1.05, 224 1.02 to 1.12; f32 G = 2 160 0.91 to 0.95, 208 1.05 to 1.08; from more heads on it gains at once (f32 G = 5
//     n = 129 1.20, bf16 G = 8 0.98 to 1.0).  Beyond, streaming runs at the rate of memory: bf16 G = 5, n = 900, 144 KB 1.03, 256 KB
//     0.91; G = 8 n = 1024 1.01 to 1.06, 2048 0.95; f32 G = 8 4096 1.5;
//   G <= 2, 64 to 127 memories: one round of long chains.  n = 64, G = 1: M = 1088 1.0, 1408 0.91, 2048 0.76; G = 2: 1.08, 0.94 to 0.99,
//     0.79 to 0.96; n = 80 M = 1088 1.02 to 1.11, 1408 0.95 to 1.02; n = 100, one workgroup, M = 1408 1.03 to 1.1, 2048 0.85 to
//     0.93; keys per sequence of 64 memories 192 KB 1.01 to 1.05, 256 KB 0.89 to 0.96;
//   G = 1: streaming runs at the rate of memory once the chip is full.  n = 200, d = 128 192 KB 1.03, 240 KB 0.96 to 1.0; 128, d = 64 192 KB
//     1.0, 256 KB 0.91; fp32 beyond one round of workgroups only where there are nearly two: n = 320 0.96, 512 1.02 to 1.05, 640 0.89;
//   G = 2 beyond 256 memories: 208 KB 0.99 to 1.17, 256 KB 0.91 to 1.04; 1024 threads, alone on a compute unit, n = 264 0.92 to 0.97, 304
//     1.0 to 1.03, 520 0.97 to 1.01; at most the rounds that were measured;
//   G > 2: streaming writes 1 + G scores a slot and its partial outputs, this kernel neither, so it stays ahead at every n that was
//     measured; M <= 128 fills lanes only partly.
WholePlan plan_whole(const DecodeParams& p, int dtype, bool two_allowed) {
  const uint32_t row = p.d * (dtype == 0 ? 4u : 2u), G = p.G, M = p.M;
  const uint64_t n = (uint64_t)p.B * p.Hkv, mem = (uint64_t)M * row, KB = 1024;
  const bool f32 = dtype == 0, mf = !f32 && G > 2, two = two_allowed && p.d == 128 && !p.mk_per_seq;
  const WholePlan none = {0u, 0u};
  WholePlan w = none;
  auto fits = [&](uint32_t threads, uint32_t workgroups) {
    if (threads == 1024 && (mf || f32)) return false;   // see launch_u
    if (whole_loads(threads, row / workgroups, M) > kWholeMaxLoads || whole_lds_bytes(threads, row, 1 + G, M) > kLdsBytes)
      return false;
    w = WholePlan{workgroups, threads};
    return true;
  };
  if (two && n <= 128) {
    if (!fits(512, 2) && !fits(1024, 2)) return none;
  } else if (!fits(512, 1) && !fits(1024, 1)) {
    if (!two || !fits(512, 2)) return none;
  }
  const bool pair = w.workgroups == 2, own = p.mk_per_seq;
  const uint64_t kb = mem / KB;
  bool take;
  if (n < (f32 && G == 1 ? 128 : 64)) {
    uint32_t most;
    if (pair) most = G == 1 && (f32 || n < 32) ? 128 : 160;
    else if (G > 2) most = 128;
    else if (n < 32) most = G == 1 ? 80 : 96;
    else if (G == 1) most = own || f32 ? 96 : 80;
    else most = own ? 128 : 104;
    take = kb <= most;
  } else if (pair && n > 128) {
    take = f32 ? (G > 4 ? n <= 4096 : G > 1 && n >= (G == 2 ? 208 : 192) && n <= 256)
               : (G > 6 ? n <= 1024 : n >= 192 && (n <= 256 || (G > 4 && n <= 1024 && kb <= 160)));
  } else if (G <= 2) {
    if (n < 96) take = M <= (own ? 1408 : 8 * n + 576) && (pair || kb <= 192);
    else take = pair || own || n > 128 || M <= (G == 1 && n > 96 ? 1536 : 16 * n);
    if (G == 2 && w.threads == 1024 && n > 256 && n < 304) take = false;
    else if (G == 2) take = take && (n <= 256 || (n <= (f32 ? 512 : 1024) && (kb <= 216 || (n >= 448 && n <= 512))));
    else if (n <= 256) take = take && (pair || own || n < 192 || kb <= 208) && n * kb <= (kb < 256 ? 62 : 48) * KB;
    else take = kb <= 64 && (f32 ? M > 128 && n >= 448 && n <= 512 : n <= 640);
  } else {
    take = n <= (f32 || M <= 128 ? 1024 : 4096);
  }
  return take ? w : none;
}

hipError_t launch_whole(const DecodeParams& p, const WholePlan& w, const KeyWrite& kw, int dtype, hipStream_t s) {
  if (dtype == 0) return p.d == 128 ? launch_g<F32, 128>(p, w, kw, s) : launch_g<F32, 64>(p, w, kw, s);
  return p.d == 128 ? launch_g<BF16, 128>(p, w, kw, s) : launch_g<BF16, 64>(p, w, kw, s);
}

}  // namespace bct
