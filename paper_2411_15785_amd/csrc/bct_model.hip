// The dense glue of a Llama-shaped stack around the bounded-cache attention
// layer (gfx950): embedding lookup, RMS normalisation, skinny projections
// (the paper's W_wq and W_wv of section 3.2 step 1 among them), the SwiGLU MLP
// and the greedy arg-max, with their C entry points (include/bct_model.h).
//
// The projections multiply a handful of token rows (the decode batch) by a
// large weight matrix, so they are bound by streaming the weights from HBM
// once.  The weights are repacked once, when they are loaded, into 1 KB tiles
// in MFMA operand order, so that every wavefront load instruction reads one
// contiguous tile.  A workgroup owns 16 output features and all K inputs: its
// wavefronts split K, each keeps two 16 x 16 fp32 accumulators
// (v_mfma_f32_16x16x32_bf16; rows = token rows, columns = output features) for
// 32 token rows and reads the activations straight from memory (they stay in
// L2); the partial accumulators are summed through LDS in a fixed order.
#include "../../include/bct_model.h"

#include <stdio.h>

#include "bct_device.h"
#include "bct_linear.h"

namespace bct {

namespace {

// Workgroup shapes of the projections (wavefronts that split K, weight tiles a wavefront has in flight,
// feature tiles per workgroup) are template parameters chosen where the kernels are launched.

__device__ __forceinline__ float bf16f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
__device__ __forceinline__ uint16_t f2bf16(float x) { return __builtin_bit_cast(uint16_t, (__bf16)x); }

// Row-major w [N][K] -> tiles of 16 features x 32 inputs, 1 KB each, tile (n / 16, k / 32) at index
// (n / 16) * (K / 32) + k / 32.  Inside a tile the 16 bytes of lane l = 16 * ((k % 32) / 8) + n % 16 hold
// the 8 consecutive inputs k % 8 = 0..7: the B operand of v_mfma_f32_16x16x32_bf16, so that one wavefront
// load instruction reads one whole tile, contiguously.
__global__ __launch_bounds__(256) void pack_weight_kernel(const uint16_t* __restrict__ w, u32x4* __restrict__ packed,
                                                          uint32_t N, uint32_t K) {
  const size_t c = (size_t)blockIdx.x * 256 + threadIdx.x;  // 16-byte chunk of the packed array
  if (c >= (size_t)N * K / 8) return;
  const uint32_t KT = K / 32, l = (uint32_t)(c % 64);
  const size_t tile = c / 64;
  const uint32_t nt = (uint32_t)(tile / KT), kt = (uint32_t)(tile % KT);
  const uint32_t n = nt * 16 + l % 16, k = kt * 32 + (l / 16) * 8;
  packed[c] = *(const u32x4*)(w + (size_t)n * K + k);
}

// In the order of the output, so that it is written in whole lines (in the order of the rows, every line came from
// many workgroups, on several XCDs); a workgroup reads 128 bytes of each of 32 rows.  16384 rows x 4096: 52 us against
// 122 (268 MB: 5.2 TB/s, what a copy reaches), 2048 rows 9.4 against 15.5.
__global__ __launch_bounds__(256) void pack_rows_kernel(const uint16_t* __restrict__ x, u32x4* __restrict__ packed,
                                                        uint32_t rows, uint32_t K) {
  const size_t c = (size_t)blockIdx.x * 256 + threadIdx.x, tile = c / 64;   // 16-byte chunk of the tiled array
  const uint32_t lane = c % 64, group = (uint32_t)(tile / 2 / (K / 32)), kt = (uint32_t)(tile / 2 % (K / 32));
  const uint32_t r = group * 32 + (uint32_t)(tile % 2) * 16 + lane % 16, k = kt * 32 + lane / 16 * 8;
  if (r >= rows) return;
  packed[c] = *(const u32x4*)(x + (size_t)r * K + k);
}

// FT: feature tiles (of 16) per workgroup.  Every wavefront streams FT (x 2 for SwiGLU) weight tiles against
// each activation fragment it loads: the activations come from L2, where all workgroups ask for the same
// lines at the same time, and with one weight tile per fragment that traffic (2 KB per KB of weights)
// bounds the kernel at about 4 TB/s of weights; two tiles per fragment reach about 5.
// RT: row tiles (of 16) per workgroup.  Up to 16 rows need one, and with it half of that traffic: at 4 rows against
// two row tiles, 11008 -> 4096 17.6 us (21.5), 4096 -> 4096 11.9 (12.7), 4096 -> 32000 47.9 (50.1), SwiGLU
// 4096 -> 11008 30.0 (32.2); at 16 rows 23.1 (25.8), 11.7 (12.7), 50.2 (52.2), 33.8 (34.2).  4096 -> 12288 (three feature
// tiles): see streaming_row_tiles.
template <bool SWIGLU, bool XT, int WAVES, int U, int FT, int RT>
__global__ __launch_bounds__(64 * WAVES) void linear_kernel(const uint16_t* __restrict__ x,
                                                            const u32x4* __restrict__ w,
                                                            const u32x4* __restrict__ w2, const uint16_t* residual,
                                                            LinearOut dst, uint32_t rows, uint32_t K,
                                                            uint32_t out_tiled) {
  constexpr int NW2 = SWIGLU ? 2 : 1;   // weight matrices
  constexpr int NS = FT * NW2;          // weight streams of a wavefront: stream s = feature tile s / NW2 of matrix s % NW2
  constexpr int NTHR = 64 * WAVES;
  constexpr int ROWS = 16 * RT;
  __shared__ float sC[WAVES][ROWS][17];
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, jl = lane % 16, kg = lane / 16;
  const uint32_t nt0 = blockIdx.x * FT, r0 = blockIdx.y * ROWS, KT = K / 32;
  // this wavefront's share of the K tiles
  const uint32_t kt0 = (uint32_t)((uint64_t)wave * KT / WAVES), kt1 = (uint32_t)((uint64_t)(wave + 1) * KT / WAVES);
  const u32x4* wt[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) wt[s] = ((s % NW2) ? w2 : w) + ((size_t)(nt0 + s / NW2) * KT + kt0) * 64 + lane;
  // A operand: lane holds token row jl (+16 for the second row tile), inputs 8 * kg .. + 8 of the K tile.
  // Rows past the end load a valid row instead; their results are never stored.
  // Tiled activations: the two operands of K tile kt are the consecutive 1 KB tiles 2 * kt, 2 * kt + 1
  // of this row group (rows past the end are allocated, their content is never stored).
  // xstep: distance in bf16 elements between a lane's chunks of consecutive K tiles.
  const uint16_t* xr[RT];
#pragma unroll
  for (int j = 0; j < RT; ++j)
    xr[j] = XT ? x + (((size_t)(r0 / 32) * KT + kt0) * 128 + j * 64 + lane) * 8
               : x + (size_t)min(r0 + 16 * j + jl, rows - 1) * K + (size_t)kt0 * 32 + kg * 8;
  constexpr size_t xstep = XT ? 128 * 8 : 32;
  f32x4 acc[NS][RT];
#pragma unroll
  for (int s = 0; s < NS; ++s)
#pragma unroll
    for (int j = 0; j < RT; ++j) acc[s][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const uint32_t n_t = kt1 - kt0;
  // Rounds of U tiles: all loads of a round are issued before its first MFMA, so a round costs one memory
  // latency.  The last, partial round loads its missing tiles from the share's last tile (in bounds) and
  // zeroes their weights, which removes them from the sum.
  for (uint32_t t = 0; t < n_t; t += U) {
    const bool whole = t + U <= n_t;
    u32x4 b[U][NS], a[U][RT];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const size_t i = whole ? t + u : min(t + u, n_t - 1);
#pragma unroll
      for (int s = 0; s < NS; ++s) b[u][s] = __builtin_nontemporal_load(wt[s] + i * 64);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const size_t i = whole ? t + u : min(t + u, n_t - 1);
#pragma unroll
      for (int j = 0; j < RT; ++j) a[u][j] = *(const u32x4*)(xr[j] + i * xstep);
    }
    if (!whole) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (t + u >= n_t) {
#pragma unroll
          for (int s = 0; s < NS; ++s) b[u][s] = u32x4{0u, 0u, 0u, 0u};
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int j = 0; j < RT; ++j)
          acc[s][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[u][j]),
                                                              __builtin_bit_cast(bf16x8, b[u][s]), acc[s][j], 0, 0, 0);
    }
  }
  // accumulator element v of a lane: token row 4 * kg + v of the row tile, feature jl.  Per feature tile
  // the partials of all wavefronts go through LDS (one matrix at a time through the same buffer) and
  // every thread adds them in wave order for the outputs it owns (ROWS x 16 per tile).
  constexpr int OPT = (ROWS * 16 + NTHR - 1) / NTHR;   // outputs per thread and tile
#pragma unroll
  for (int f = 0; f < FT; ++f) {
    float sum[NW2][OPT];
#pragma unroll
    for (int pass = 0; pass < NW2; ++pass) {
      if (f || pass) __syncthreads();
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int v = 0; v < 4; ++v) sC[wave][16 * rt + 4 * kg + v][jl] = acc[f * NW2 + pass][rt][v];
      __syncthreads();
#pragma unroll
      for (int q = 0; q < OPT; ++q) {
        const uint32_t o = (threadIdx.x + q * NTHR) % (ROWS * 16), oi = o / 16, oj = o % 16;
        float a = 0.f;
#pragma unroll
        for (int k = 0; k < WAVES; ++k) a += sC[k][oi][oj];
        sum[pass][q] = a;
      }
    }
#pragma unroll
    for (int q = 0; q < OPT; ++q) {
      const uint32_t o = threadIdx.x + q * NTHR, oi = (o % (ROWS * 16)) / 16, oj = o % 16;
      if (o < ROWS * 16 && r0 + oi < rows) {
        const uint32_t n = (nt0 + f) * 16 + oj;
        const int which = n >= dst.start[2] ? 2 : n >= dst.start[1] ? 1 : 0;
        const uint32_t width = dst.start[which + 1] - dst.start[which], col = n - dst.start[which];
        const size_t oo = (size_t)(r0 + oi) * width + col;
        const float g = sum[0][q];
        float y;
        if (SWIGLU) y = g / (1.0f + __expf(-g)) * sum[NW2 - 1][q];
        else y = residual ? g + bf16f(residual[oo]) : g;
        // a tiled output is the input of a projection whose K is this output's width
        dst.ptr[which][out_tiled ? tiled_chunk(r0 + oi, col, width) * 8 + col % 8 : oo] = f2bf16(y);
      }
    }
  }
}

// The row of a workgroup.  Workgroups go to the eight XCDs in turn; a 128-byte line of the tiled order holds 8 inputs
// of 8 consecutive rows, and rows in launch order would leave parts of every line in eight L2s.  So 16 consecutive
// rows (1 KB tiles) are those of one XCD, for as many whole groups of 128 rows as there are.  16384 rows x 4096:
// 80 us against 139 (8 rows per workgroup: 110), 2048 rows 10.3 against 16.3.  That is 3.4 TB/s, not the rate of memory: the
// same 268 MB take pack_rows_kernel 52 us.  A workgroup here holds one row of 8 KB and waits for it and for the sum.
__device__ __forceinline__ uint32_t tiled_row(uint32_t block, uint32_t rows) {
  if (block >= rows / 128 * 128) return block;
  return (block / 128 * 8 + block % 8) * 16 + block / 8 % 16;
}

// One workgroup per row; a thread keeps its NV 16-byte chunks of the row in registers between the sum of squares and the
// scaling.  When the gains and the chunks are requested depends on the size (rmsnorm_form):
//   kGainsWithRow   all at once, so that a workgroup waits for memory once.  us, this | gains after the sum | after it and
//                   eight chunks a thread for every width: 4 x 4096 2.5 | 2.6 | 2.9, 640 x 4096 4.5 | 4.7 | 5.1, 4096 x 8192 39 |
//                   44 | 46, 16384 x 12288 259 | 283 | 296
//   kGainsLate      the gains after the sum: less in flight
//   kChunkByChunk   as that, and a chunk is requested when the one before has arrived: the workgroups of 16 rows that write one
//                   line of the tiled order stay closer together, and fewer lines leave the L2 in parts (16384 x 4096, 134 MB
//                   of output: 168 MB written, with the gains late 212)
enum RmsForm { kGainsWithRow, kGainsLate, kChunkByChunk };

template <int NV, RmsForm FORM>
__global__ __launch_bounds__(256) void rmsnorm_kernel(const uint16_t* x, const uint16_t* gain, uint16_t* out,
                                                      uint32_t rows, uint32_t dim, float eps, uint32_t out_tiled) {
  __shared__ float s_part[4];
  const uint32_t row = out_tiled ? tiled_row(blockIdx.x, rows) : blockIdx.x;
  const uint16_t* xr = x + (size_t)row * dim;
  u32x4 v[NV], gv[NV];
  if constexpr (FORM != kChunkByChunk) {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      // chunks past the end: the first one again, not counted and not stored
      const uint32_t c = (threadIdx.x + i * 256) * 8, from = c < dim ? c : 0u;
      v[i] = *(const u32x4*)(xr + from);
      if (FORM == kGainsWithRow) gv[i] = *(const u32x4*)(gain + from);
    }
  }
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const uint32_t c = (threadIdx.x + i * 256) * 8;
    if (c < dim) {
      if constexpr (FORM == kChunkByChunk) v[i] = *(const u32x4*)(xr + c);
      float f[8];
      unpack16<BF16>(v[i], f);
#pragma unroll
      for (int e = 0; e < 8; ++e) ss = __builtin_fmaf(f[e], f[e], ss);
    }
  }
  ss = xor_sum<1, 32>(ss);
  if (threadIdx.x % 64 == 0) s_part[threadIdx.x / 64] = ss;
  __syncthreads();
  ss = (s_part[0] + s_part[1]) + (s_part[2] + s_part[3]);
  const float r = 1.0f / sqrtf(ss / (float)dim + eps);
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const uint32_t c = (threadIdx.x + i * 256) * 8;
    if (c < dim) {
      float f[8], g[8];
      unpack16<BF16>(v[i], f);
      unpack16<BF16>(FORM == kGainsWithRow ? gv[i] : *(const u32x4*)(gain + c), g);
#pragma unroll
      for (int e = 0; e < 8; ++e) f[e] = f[e] * r * g[e];
      const u32x4 o = pack16_round<BF16>(f);
      if (out_tiled) ((u32x4*)out)[tiled_chunk(row, c, dim)] = o;
      else *(u32x4*)(out + (size_t)row * dim + c) = o;
    }
  }
}

__global__ __launch_bounds__(256) void embed_kernel(const int32_t* ids, const uint16_t* table, uint16_t* out,
                                                    uint32_t rows, uint32_t vocab, uint32_t dim) {
  const uint32_t cpr = dim / 8;
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (size_t)rows * cpr) return;
  const uint32_t r = (uint32_t)(i / cpr), c = (uint32_t)(i % cpr);
  const int32_t id = ids[r];
  u32x4 v = {0u, 0u, 0u, 0u};
  if (id >= 0 && (uint32_t)id < vocab) v = *(const u32x4*)(table + (size_t)id * dim + c * 8);
  *(u32x4*)(out + (size_t)r * dim + c * 8) = v;
}

__global__ __launch_bounds__(256) void argmax_kernel(const uint16_t* logits, int32_t* ids, uint32_t N) {
  __shared__ float sv[256];
  __shared__ uint32_t si[256];
  const uint16_t* row = logits + (size_t)blockIdx.x * N;
  float best = -INFINITY;
  uint32_t bi = 0xFFFFFFFFu;
  auto take = [&](float v, uint32_t j) {
    if (v > best || bi == 0xFFFFFFFFu) {  // ascending j: a later equal value never replaces an earlier one
      best = v;
      bi = j;
    }
  };
  // 16-byte vectors (8 logits), four in flight per thread; rows start 16-byte aligned when N is a multiple of 8
  const uint32_t nvec = (N % 8 == 0) ? N / 8 : 0u;
  for (uint32_t v0 = threadIdx.x; v0 < nvec; v0 += 4 * 256) {
    u32x4 raw[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (v0 + u * 256 < nvec) raw[u] = *(const u32x4*)(row + (size_t)(v0 + u * 256) * 8);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (v0 + u * 256 < nvec) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t j = (v0 + u * 256) * 8 + 2 * e;
          take(__uint_as_float(raw[u][e] << 16), j);
          take(__uint_as_float(raw[u][e] & 0xFFFF0000u), j + 1);
        }
      }
    }
  }
  for (uint32_t j = nvec * 8 + threadIdx.x; j < N; j += 256) take(bf16f(row[j]), j);
  sv[threadIdx.x] = best;
  si[threadIdx.x] = bi;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      const float ov = sv[threadIdx.x + s];
      const uint32_t oi = si[threadIdx.x + s];
      if (oi != 0xFFFFFFFFu && (si[threadIdx.x] == 0xFFFFFFFFu || ov > sv[threadIdx.x] ||
                                (ov == sv[threadIdx.x] && oi < si[threadIdx.x]))) {
        sv[threadIdx.x] = ov;
        si[threadIdx.x] = oi;
      }
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) ids[blockIdx.x] = (int32_t)si[0];
}

thread_local char g_merr[256] = "";

bct_status mfail(bct_status s, const char* msg) {
  snprintf(g_merr, sizeof(g_merr), "%s", msg);
  return s;
}
bct_status launched(const char* what, hipError_t e = hipGetLastError()) {
  if (e == hipSuccess) return BCT_OK;
  snprintf(g_merr, sizeof(g_merr), "%s launch failed: %s", what, hipGetErrorString(e));
  return BCT_ERR_HIP;
}
// The form of a size, by what it measured: us, kGainsWithRow | kGainsLate | kChunkByChunk, the same buffers again and again
// (x and out in the last-level cache where they fit) / buffers from memory.
// Row-major outputs: 4096 x 4096 11.5 | 12.0 | 12.2 / 14.1 | 14.6 | 14.8; 16384 x 2048 20.8 | 21.3 | - / 24.2 | 25.2 | -; 16384 x
// 4096 38.7 | 38.9 | 38.9 / 46.0 | 47.2 | 46.6; 32768 x 5120 116 | 115 | 118 / 115 | 115 | 117; 16384 x 12288 139 | 141 | 154.
// Tiled outputs, from 8 M elements on.  Up to 4096 wide: 1024 x 4096 5.83 | 5.93 | 6.02 / 6.50 | 6.99 | 7.11; 2048 9.27 | 9.40 | 9.60
// / 11.9 | 10.6 | 10.7; 6144 21.8 | 22.0 | 23.0 / 34.3 | 31.1 | 32.6; 9000 x 3584 26.6 | 26.0 | 27.9 / 42.8 | 38.2 | 39.3; 16384 - | 52.7
// | 50.5 / - | 81.9 | 79.7; 32768 - | 164 | 157 / - | 166 | 154; but 32768 x 3584 - | 128 | 135 / - | 129 | 135 (the border lies at 4000:
// 24000 rows 108 | 112 / 113 | 113, 50000 236 | 234 / 237 | 233); 8192 x 1024 8.8 | 9.3 | 9.3 / 12.5 | 11.8 | 11.7, 12000 12.3 | 12.3 | 12.1
// / 19.0 | 17.7 | 17.4, 32768 x 2048 - | 47.7 | 47.5 / - | 72.4 | 73.8.
// Wider: 9000 x 4224 33.7 | 34.8 | 34.8 / 52.1 | 51.3 | 50.9; 14000 x 5120 89.7 | 93.5 | 84.1 / 88.2 | 91.2 | 86.9; 50000 x 5120 351 | 343
// | 312; 16384 x 6144 116 | 132 | 120 / 118 | 136 | 120; 24000 180 | 206 | 174 / 181 | 205 | 175; 50000 425 | 442 | 363; 32768 x 7168 295 |
// 344 | 298; 32768 x 8192 338 | 410 | 354.  Not chosen by: 2048 rows of 8192 or 12288 from memory, 21.8 | 22.8 | 20.3, from the
// cache 16.6 | 17.9 | 19.4.
RmsForm rmsnorm_form(uint32_t rows, uint32_t dim, bool out_tiled) {
  const uint64_t n = (uint64_t)rows * dim, M = 1u << 20;
  if (!out_tiled) return kGainsWithRow;
  if (dim <= 4000 || (dim <= 4096 && n < 48 * M)) return n >= (dim > 2048 ? 8 : 10) * M ? kGainsLate : kGainsWithRow;
  return dim <= 6144 && n >= (dim <= 5120 ? 48 : 128) * M ? kChunkByChunk : kGainsWithRow;
}

bool al16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

bct_status check_linear(const void* x, const void* w, const void* out, uint32_t rows, uint32_t K, uint32_t N) {
  if (!x || !w || !out || rows == 0 || K == 0 || N == 0) return mfail(BCT_ERR_INVALID_ARG, "NULL pointer or zero size");
  if (K % 32 != 0 || N % 16 != 0) return mfail(BCT_ERR_UNSUPPORTED, "K must be a multiple of 32 and N of 16");
  if (!al16(x) || !al16(w) || !al16(out)) return mfail(BCT_ERR_MISALIGNED, "pointers must be 16-byte aligned");
  return BCT_OK;
}

}  // namespace
}  // namespace bct

using namespace bct;

template <int WV, int UN, int FT, int RT>
static void launch_linear_rt(const void* x, const void* w, const void* residual, const LinearOut& dst, uint32_t rows,
                             uint32_t K, uint32_t N, uint32_t flags, void* hip_stream) {
  const dim3 grid(N / (16 * FT), (rows + 16 * RT - 1) / (16 * RT)), block(64 * WV);
  if (flags & BCTM_X_TILED)
    hipLaunchKernelGGL((linear_kernel<false, true, WV, UN, FT, RT>), grid, block, 0, (hipStream_t)hip_stream,
                       (const uint16_t*)x, (const u32x4*)w, (const u32x4*)nullptr, (const uint16_t*)residual, dst, rows,
                       K, 0u);
  else
    hipLaunchKernelGGL((linear_kernel<false, false, WV, UN, FT, RT>), grid, block, 0, (hipStream_t)hip_stream,
                       (const uint16_t*)x, (const u32x4*)w, (const u32x4*)nullptr, (const uint16_t*)residual, dst, rows,
                       K, 0u);
}
// Row tiles of a streaming launch with FT feature tiles a workgroup.
static uint32_t streaming_row_tiles(uint32_t FT, uint32_t rows, uint32_t N, uint32_t flags) {
  // One row tile up to 16 rows, but for row-major activations of more than 8 rows under three feature tiles on one
  // workgroup per compute unit: there half as many row loads in flight cost more than their traffic.  us, one row tile |
  // two: 12288 features, 16 row-major rows, K = 4096 19.5 | 19.1, K = 8192 34.8 | 34.4, K = 2048 11.9 | 11.9; 8 rows 18.9 |
  // 18.8, 34.3 | 34.3, 11.2 | 11.4; tiled, 16 rows 18.9 | 19.1, 33.6 | 34.2, 11.2 | 11.7.  More workgroups: 14400 features,
  // K = 4096, 16 row-major rows 29.0 | 29.9, tiled 26.9 | 29.5.
  const bool two = FT == 3 && !(flags & BCTM_X_TILED) && rows > 8 && N / (16 * FT) <= 256;
  return rows <= 16 && !two ? 1 : 2;
}
template <int WV, int UN, int FT>
static void launch_linear_w(const void* x, const void* w, const void* residual, const LinearOut& dst, uint32_t rows,
                            uint32_t K, uint32_t N, uint32_t flags, void* hip_stream) {
  if (streaming_row_tiles(FT, rows, N, flags) == 1)
    launch_linear_rt<WV, UN, FT, 1>(x, w, residual, dst, rows, K, N, flags, hip_stream);
  else launch_linear_rt<WV, UN, FT, 2>(x, w, residual, dst, rows, K, N, flags, hip_stream);
}

// The kernel of a projection shape.  Many rows (from 128 on): the matrix-core kernel (bct_linear_rows.hip); its two values
// name ranges of shapes, the tile inside it is linear_rows_tile's choice.  Feature counts that no tile divides take it as
// well, with a last tile that is partly used, once the streaming kernel, which reads the weights again for every 32 rows, has
// more than one round of workgroups (of inputs beyond 3072: two; SwiGLU, whose weights are twice as many, one).  us, streaming | matrix-core, weights from memory:
//   709 rows, 11264 -> 2912 332 | 94; 2381, 1664 -> 1344 142 | 20; 4096, 4096 -> 4128 959 | 157; 8192, 5088 -> 5088 3679 | 361;
//   SwiGLU 1500, 4000 -> 1504 188 | 54; 640, 1024 -> 2848 42 | 14; 256, 1024 -> 736 (368 workgroups) 11.8 | 6.9; 700, 3072
//   -> 320 (440) 13.3 | 12.6; 516, 10976 -> 576 (612) 50.4 | 44.6; 256, 11008 -> 1504 (752) 67 | 45; SwiGLU 256, 5120 -> 736 27 | 24, 167,
//   8992 -> 720 (270) 45.7 | 43.6.  One to two rounds of more than 3072 inputs, where few tiles are one long chain each, either way:
//   145, 4032 -> 1200 (375) 15.9 | 19.3; 360, 7072 -> 448 (336) 23.4 | 27.9; 700, 4096 -> 320 14.5 | 15.7; but 700, 4096 -> 272 17.4 | 15.7.
//   Up to one round: 200, 5120 -> 480 (210) 12.9 | 19.0, SwiGLU 15.8 | 20.8
// Not below 128 features, where no tile is half used, and not beyond 16384.
// Few rows: the streaming kernel; measured at 32 rows (weights in TB/s): K = 4096, N = 4096 / 12288: 16
// wavefronts, one feature tile 3.6 / 4.0 against 2.8 / 3.8 for two tiles (too few workgroups); N = 32000:
// two tiles 5.0 against 4.3.
static uint32_t linear_kernel_of(uint32_t rows, uint32_t K, uint32_t N, bool swiglu) {
  const bool ragged = N >= 128 && N <= 16384 && (uint64_t)(N / 16) * ((rows + 31) / 32) > (!swiglu && K > 3072 ? 512u : 256u);
  if (rows >= 128 && (N % (swiglu ? 64u : 128u) == 0 || ragged))
    return (rows >= 1024 && N % (swiglu ? 128u : 256u) == 0) ? BCTM_KERNEL_TILE256 : BCTM_KERNEL_TILE128;
  if (!swiglu && N >= 16384 && N % 32 == 0) return BCTM_KERNEL_STREAMING_WIDE;
  // three feature tiles per workgroup when that still leaves a workgroup for every compute unit: 12288
  // features (W_q | W_wq | W_wv at 4096 each) are exactly 256 workgroups, 19.5 us against 24.3
  if (!swiglu && N % 48 == 0 && N / 48 >= 256) return BCTM_KERNEL_STREAMING_TRIPLE;
  return BCTM_KERNEL_STREAMING;
}

// What the launches below and above give a workgroup; the wavefronts of a workgroup share K.
static LinearTile streaming_tile(uint32_t kernel, uint32_t rows, uint32_t N, bool swiglu, uint32_t flags) {
  const uint32_t ft = kernel == BCTM_KERNEL_STREAMING_TRIPLE ? 3 : kernel == BCTM_KERNEL_STREAMING_WIDE ? 2 : 1;
  return {16 * streaming_row_tiles(ft, rows, N, flags), 16 * ft, swiglu ? 4u : ft > 1 ? 8u : 16u};
}

template <int WV, int UN, int FT, int RT>
static void launch_swiglu_w(const void* x, const void* wg, const void* wu, const LinearOut& dst, uint32_t rows,
                            uint32_t K, uint32_t N, uint32_t flags, void* hip_stream) {
  const dim3 grid(N / (16 * FT), (rows + 16 * RT - 1) / (16 * RT)), block(64 * WV);
  const uint32_t ot = flags & BCTM_OUT_TILED ? 1u : 0u;
  if (flags & BCTM_X_TILED)
    hipLaunchKernelGGL((linear_kernel<true, true, WV, UN, FT, RT>), grid, block, 0, (hipStream_t)hip_stream,
                       (const uint16_t*)x, (const u32x4*)wg, (const u32x4*)wu, (const uint16_t*)nullptr, dst, rows, K, ot);
  else
    hipLaunchKernelGGL((linear_kernel<true, false, WV, UN, FT, RT>), grid, block, 0, (hipStream_t)hip_stream,
                       (const uint16_t*)x, (const u32x4*)wg, (const u32x4*)wu, (const uint16_t*)nullptr, dst, rows, K, ot);
}

extern "C" {

bct_status bctm_embed(const int32_t* ids, const void* table, void* out, uint32_t rows, uint32_t vocab, uint32_t dim,
                      void* hip_stream) {
  if (!ids || !table || !out || rows == 0 || vocab == 0 || dim == 0)
    return mfail(BCT_ERR_INVALID_ARG, "NULL pointer or zero size");
  if (dim % 8 != 0) return mfail(BCT_ERR_UNSUPPORTED, "dim must be a multiple of 8");
  if (!al16(table) || !al16(out)) return mfail(BCT_ERR_MISALIGNED, "pointers must be 16-byte aligned");
  const size_t n = (size_t)rows * (dim / 8);
  hipLaunchKernelGGL(embed_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)hip_stream, ids,
                     (const uint16_t*)table, (uint16_t*)out, rows, vocab, dim);
  return launched("embed");
}

bct_status bctm_rmsnorm(const void* x, const void* gain, void* out, uint32_t rows, uint32_t dim, float eps,
                        uint32_t flags, void* hip_stream) {
  if (!x || !gain || !out || rows == 0 || dim == 0) return mfail(BCT_ERR_INVALID_ARG, "NULL pointer or zero size");
  if (flags & ~BCTM_OUT_TILED) return mfail(BCT_ERR_INVALID_ARG, "rmsnorm takes only BCTM_OUT_TILED");
  if (dim % 8 != 0 || dim > 16384) return mfail(BCT_ERR_UNSUPPORTED, "dim must be a multiple of 8, at most 16384");
  if ((flags & BCTM_OUT_TILED) && dim % 32 != 0)
    return mfail(BCT_ERR_UNSUPPORTED, "tiled activations need a multiple of 32 columns");
  if ((flags & BCTM_OUT_TILED) && x == out) return mfail(BCT_ERR_INVALID_ARG, "a tiled output cannot overwrite x");
  if (!al16(x) || !al16(gain) || !al16(out)) return mfail(BCT_ERR_MISALIGNED, "pointers must be 16-byte aligned");
  const RmsForm form = rmsnorm_form(rows, dim, (flags & BCTM_OUT_TILED) != 0);
  const auto kernel = dim <= 2048   ? (form == kGainsLate ? rmsnorm_kernel<1, kGainsLate> : rmsnorm_kernel<1, kGainsWithRow>)
                      : dim <= 4096 ? (form == kChunkByChunk ? rmsnorm_kernel<2, kChunkByChunk>
                                       : form == kGainsLate  ? rmsnorm_kernel<2, kGainsLate>
                                                             : rmsnorm_kernel<2, kGainsWithRow>)
                      : dim <= 8192 ? (form == kChunkByChunk ? rmsnorm_kernel<4, kChunkByChunk> : rmsnorm_kernel<4, kGainsWithRow>)
                                    : rmsnorm_kernel<8, kGainsWithRow>;
  hipLaunchKernelGGL(kernel, dim3(rows), dim3(256), 0, (hipStream_t)hip_stream, (const uint16_t*)x, (const uint16_t*)gain,
                     (uint16_t*)out, rows, dim, eps, flags & BCTM_OUT_TILED);
  return launched("rmsnorm");
}

bct_status bctm_pack_rows(const void* x, void* tiled, uint32_t rows, uint32_t K, void* hip_stream) {
  if (!x || !tiled || rows == 0 || K == 0) return mfail(BCT_ERR_INVALID_ARG, "NULL pointer or zero size");
  if (x == tiled) return mfail(BCT_ERR_INVALID_ARG, "packing in place is not possible");
  if (K % 32 != 0) return mfail(BCT_ERR_UNSUPPORTED, "tiled activations need a multiple of 32 columns");
  if (!al16(x) || !al16(tiled)) return mfail(BCT_ERR_MISALIGNED, "pointers must be 16-byte aligned");
  const size_t chunks = (size_t)rows * K / 8;
  if ((chunks + 255) / 256 > 0x7FFFFFFFu) return mfail(BCT_ERR_UNSUPPORTED, "matrix too large");
  const size_t grid = ((size_t)((rows + 31) / 32) * 32 * K / 8 + 255) / 256;   // whole groups of 32 rows
  hipLaunchKernelGGL(pack_rows_kernel, dim3((unsigned)grid), dim3(256), 0, (hipStream_t)hip_stream,
                     (const uint16_t*)x, (u32x4*)tiled, rows, K);
  return launched("pack_rows");
}

bct_status bctm_pack_weight(const void* w, void* packed, uint32_t N, uint32_t K, void* hip_stream) {
  if (!w || !packed || N == 0 || K == 0) return mfail(BCT_ERR_INVALID_ARG, "NULL pointer or zero size");
  if (w == packed) return mfail(BCT_ERR_INVALID_ARG, "packing in place is not possible");
  if (K % 32 != 0 || N % 16 != 0) return mfail(BCT_ERR_UNSUPPORTED, "K must be a multiple of 32 and N of 16");
  if (!al16(w) || !al16(packed)) return mfail(BCT_ERR_MISALIGNED, "pointers must be 16-byte aligned");
  const size_t chunks = (size_t)N * K / 8;
  if ((chunks + 255) / 256 > 0x7FFFFFFFu) return mfail(BCT_ERR_UNSUPPORTED, "matrix too large");
  hipLaunchKernelGGL(pack_weight_kernel, dim3((unsigned)((chunks + 255) / 256)), dim3(256), 0, (hipStream_t)hip_stream,
                     (const uint16_t*)w, (u32x4*)packed, N, K);
  return launched("pack_weight");
}

static bct_status launch_linear(const void* x, const void* w, const void* residual, const LinearOut& dst,
                                uint32_t rows, uint32_t K, uint32_t N, uint32_t flags, void* hip_stream) {
  const uint32_t kernel = linear_kernel_of(rows, K, N, false);
  if (kernel == BCTM_KERNEL_TILE128 || kernel == BCTM_KERNEL_TILE256)
    return launched("linear", launch_linear_rows(x, w, nullptr, residual, dst, rows, K, N, flags & BCTM_X_TILED, false,
                                                 (hipStream_t)hip_stream));
  if (kernel == BCTM_KERNEL_STREAMING_WIDE) launch_linear_w<8, 4, 2>(x, w, residual, dst, rows, K, N, flags, hip_stream);
  else if (kernel == BCTM_KERNEL_STREAMING_TRIPLE) launch_linear_w<8, 4, 3>(x, w, residual, dst, rows, K, N, flags, hip_stream);
  else launch_linear_w<16, 8, 1>(x, w, residual, dst, rows, K, N, flags, hip_stream);
  return launched("linear");
}

bct_status bctm_linear(const void* x, const void* w, const void* residual, void* out, uint32_t rows, uint32_t K,
                       uint32_t N, uint32_t flags, void* hip_stream) {
  const bct_status st = check_linear(x, w, out, rows, K, N);
  if (st != BCT_OK) return st;
  if (flags & ~BCTM_X_TILED) return mfail(BCT_ERR_INVALID_ARG, "linear takes only BCTM_X_TILED");
  if (x == out) return mfail(BCT_ERR_INVALID_ARG, "out must not be x");
  if (!al16(residual)) return mfail(BCT_ERR_MISALIGNED, "pointers must be 16-byte aligned");
  const LinearOut dst = {{(uint16_t*)out, nullptr, nullptr}, {0u, N, N, N}};
  return launch_linear(x, w, residual, dst, rows, K, N, flags, hip_stream);
}

bct_status bctm_linear_split(const void* x, const void* w, void* out0, uint32_t N0, void* out1, uint32_t N1,
                             void* out2, uint32_t N2, uint32_t rows, uint32_t K, uint32_t flags, void* hip_stream) {
  if (N0 == 0 || N1 == 0) return mfail(BCT_ERR_INVALID_ARG, "the first two outputs must not be empty");
  if ((uint64_t)N0 + N1 + N2 > 0xFFFFFFF0ull) return mfail(BCT_ERR_UNSUPPORTED, "too many features");
  const uint32_t N = N0 + N1 + N2;
  const bct_status st = check_linear(x, w, out0, rows, K, N);
  if (st != BCT_OK) return st;
  if (flags & ~BCTM_X_TILED) return mfail(BCT_ERR_INVALID_ARG, "linear takes only BCTM_X_TILED");
  if (!out1 || (N2 && !out2)) return mfail(BCT_ERR_INVALID_ARG, "NULL pointer or zero size");
  if (N0 % 16 != 0 || N1 % 16 != 0 || N2 % 16 != 0)
    return mfail(BCT_ERR_UNSUPPORTED, "every output width must be a multiple of 16");
  if (x == out0 || x == out1 || x == out2) return mfail(BCT_ERR_INVALID_ARG, "out must not be x");
  if (!al16(out1) || !al16(out2)) return mfail(BCT_ERR_MISALIGNED, "pointers must be 16-byte aligned");
  const LinearOut dst = {{(uint16_t*)out0, (uint16_t*)out1, (uint16_t*)out2}, {0u, N0, N0 + N1, N}};
  return launch_linear(x, w, nullptr, dst, rows, K, N, flags, hip_stream);
}

bct_status bctm_swiglu(const void* x, const void* w_gate, const void* w_up, void* out, uint32_t rows, uint32_t K,
                       uint32_t N, uint32_t flags, void* hip_stream) {
  const bct_status st = check_linear(x, w_gate, out, rows, K, N);
  if (st != BCT_OK) return st;
  if (flags & ~(BCTM_X_TILED | BCTM_OUT_TILED)) return mfail(BCT_ERR_INVALID_ARG, "unknown flag");
  if (!w_up) return mfail(BCT_ERR_INVALID_ARG, "NULL pointer or zero size");
  if (x == out) return mfail(BCT_ERR_INVALID_ARG, "out must not be x");
  if ((flags & BCTM_OUT_TILED) && N % 32 != 0)
    return mfail(BCT_ERR_UNSUPPORTED, "tiled activations need a multiple of 32 columns");
  if (!al16(w_up)) return mfail(BCT_ERR_MISALIGNED, "pointers must be 16-byte aligned");
  const LinearOut dst = {{(uint16_t*)out, nullptr, nullptr}, {0u, N, N, N}};
  const uint32_t kernel = linear_kernel_of(rows, K, N, true);
  if (kernel == BCTM_KERNEL_TILE128 || kernel == BCTM_KERNEL_TILE256)
    return launched("swiglu", launch_linear_rows(x, w_gate, w_up, nullptr, dst, rows, K, N, flags & BCTM_X_TILED,
                                                 flags & BCTM_OUT_TILED, (hipStream_t)hip_stream));
  // 36 us at 32 rows, 4096 -> 11008 (8 wavefronts: 38)
  if (streaming_row_tiles(1, rows, N, flags) == 1) launch_swiglu_w<4, 8, 1, 1>(x, w_gate, w_up, dst, rows, K, N, flags, hip_stream);
  else launch_swiglu_w<4, 8, 1, 2>(x, w_gate, w_up, dst, rows, K, N, flags, hip_stream);
  return launched("swiglu");
}

bct_status bctm_linear_plan(uint32_t rows, uint32_t K, uint32_t N, uint32_t swiglu, uint32_t* kernel) {
  if (!kernel || rows == 0 || K == 0 || N == 0) return mfail(BCT_ERR_INVALID_ARG, "NULL pointer or zero size");
  if (K % 32 != 0 || N % 16 != 0) return mfail(BCT_ERR_UNSUPPORTED, "K must be a multiple of 32 and N of 16");
  *kernel = linear_kernel_of(rows, K, N, swiglu != 0);
  return BCT_OK;
}

bct_status bctm_linear_tile(uint32_t rows, uint32_t K, uint32_t N, uint32_t swiglu, uint32_t flags, uint32_t* tile_rows,
                            uint32_t* tile_features, uint32_t* k_parts) {
  if (!tile_rows || !tile_features || !k_parts || rows == 0 || K == 0 || N == 0)
    return mfail(BCT_ERR_INVALID_ARG, "NULL pointer or zero size");
  if (K % 32 != 0 || N % 16 != 0) return mfail(BCT_ERR_UNSUPPORTED, "K must be a multiple of 32 and N of 16");
  const uint32_t kernel = linear_kernel_of(rows, K, N, swiglu != 0);
  const LinearTile t = kernel == BCTM_KERNEL_TILE128 || kernel == BCTM_KERNEL_TILE256
                           ? linear_rows_tile(rows, K, N, swiglu != 0, (flags & BCTM_X_TILED) != 0)
                           : streaming_tile(kernel, rows, N, swiglu != 0, flags);
  *tile_rows = t.rows;
  *tile_features = t.features;
  *k_parts = t.k_parts;
  return BCT_OK;
}

bct_status bctm_argmax(const void* logits, int32_t* ids, uint32_t rows, uint32_t N, void* hip_stream) {
  if (!logits || !ids || rows == 0 || N == 0) return mfail(BCT_ERR_INVALID_ARG, "NULL pointer or zero size");
  hipLaunchKernelGGL(argmax_kernel, dim3(rows), dim3(256), 0, (hipStream_t)hip_stream, (const uint16_t*)logits, ids, N);
  return launched("argmax");
}

const char* bctm_last_error(void) { return g_merr; }

}  // extern "C"
