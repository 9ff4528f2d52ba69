// Host-side plan and launcher declarations shared by the C ABI layer and the
// kernel files of libbct.  Nothing here is visible to callers of the library.
#ifndef BCT_INTERNAL_H
#define BCT_INTERNAL_H

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace bct {

constexpr uint32_t kMaxG = 8;          // query heads per KV head
constexpr uint32_t kMaxRows = 1 + kMaxG;  // score rows per memory: write + G reads
constexpr uint32_t kMinStatTile = 32;  // smallest slot tile with its own (max, sum) partial
// decode_fused_kernel, one workgroup per memory: up to this many slots and this many memories (one resident round of
// workgroups).  Beyond 128 slots a workgroup of 256 threads has too few loads in flight (M = 256: 15-21 us against 9-23 us
// for the streaming launches); plan_whole says which of these steps decode_whole_kernel takes.
constexpr uint32_t kFusedMaxM = 128;
constexpr uint32_t kFusedMaxUnits = 512;

// decode_whole_kernel with `threads` a workgroup: MV loads per lane for columns of col_bytes of M slots (at most
// kWholeMaxLoads), bytes of LDS (at most kLdsBytes): two key tiles of 16 rows per wavefront, R fp32 weights a slot, statistics.
constexpr uint32_t kWholeMaxLoads = 16, kLdsBytes = 160u << 10;
inline uint32_t whole_loads(uint32_t threads, uint32_t col_bytes, uint32_t M) {
  const uint32_t slots = threads * 16 / col_bytes;
  return (M + slots - 1) / slots;
}
inline size_t whole_lds_bytes(uint32_t threads, uint32_t row_bytes, uint32_t R, uint32_t M) {
  return (size_t)threads / 64 * 32 * row_bytes + ((size_t)R * M + threads / 64 * 32) * sizeof(float);
}

// One decode step of one layer: everything its launches need.
struct DecodeParams {
  const void* mk;   // [Hkv][M][d] or [B][Hkv][M][d]
  void* mv;         // [B][Hkv][M][d], updated in place
  const void* q;    // [B][Hq][d] or null
  const void* wq;   // [B][Hkv][d] or null
  const void* wv;   // [B][Hkv][d] or null
  void* out;        // [B][Hq][d] or null
  float* scores;    // [B*Hkv][R][M], log2-domain scaled scores
  float2* stats;    // [B*Hkv][R][n_tiles] (max, sum of exp2(score - max)) per slot tile
  float2* norm;     // [B*Hkv][R] (max, 1 / sum of exp2(score - max)) per row
  float* partial;   // [S][B][Hq][d] split-M partial outputs
  uint32_t B, Hq, Hkv, G, M, d;
  uint32_t R;        // rows per memory this step: has_write + (has_read ? G : 0)
  uint32_t has_write, has_read;
  uint32_t mk_per_seq;
  uint32_t stat_tile;  // slots per (max, sum) partial
  uint32_t n_tiles;    // M / stat_tile
  uint32_t S;          // split-M factor of the MV pass: workgroups per memory
  uint32_t mv_bs;      // threads per workgroup of the MV pass
  uint32_t mv_u;       // 16-byte loads per lane of the MV pass
  uint32_t fused;      // 1: the whole step is one launch of decode_fused_kernel
  uint32_t fuse_norm;  // 1: the MV pass merges the per-tile statistics itself, no normaliser launch
  float rscale_l2e, wscale_l2e;  // scale * log2(e)
  // strides (in elements) between consecutive batch entries of q/out and wq/wv;
  // [B][H][d] inputs use H*d, a token t of a [B][T][H][d] chunk uses T*H*d.
  uint64_t q_bstride, kv_bstride;
  // optional step size per memory (section 3.5, learning-rate adaptation): eta of memory (b, h) at
  // gate[b * gate_bstride + h]; null = 1.  Scales the write weights.
  const float* gate;
  uint64_t gate_bstride;
  // last, so that the kernels that do not use it load the fields above as before
  uint32_t rescore;    // 1: the MV pass of a step that reads scores its slots again; no scores in memory
};

// The scratch of a decode step: byte offsets of its parts, and their end.
struct DecodeScratch {
  size_t scores, stats, norm, partial, bytes;
};
inline DecodeScratch decode_scratch(const DecodeParams& p) {
  auto up = [](size_t x) { return (x + 255) / 256 * 256; };
  const size_t rows = (size_t)p.B * p.Hkv * (1 + p.G);
  DecodeScratch z;
  z.scores = 0;
  z.stats = z.scores + up(rows * p.M * sizeof(float));
  z.norm = z.stats + up(rows * (p.M / kMinStatTile) * sizeof(float2));
  z.partial = z.norm + up(rows * sizeof(float2));
  // (two splits where a step whose output lies in its inputs may need two of one)
  const size_t splits = p.rescore && p.S == 1 && p.M > 64 ? 2 : p.S;
  z.bytes = z.partial + up(splits * p.B * p.Hq * p.d * sizeof(float));
  return z;
}
constexpr size_t kStaticScratchBytes = 8u << 20;   // of bct_decode_step_static

// One prefill chunk of a bf16 cache: everything its launches need.
struct PrefillParams {
  const uint16_t* mk;  // [Hkv][M][d] or [B][Hkv][M][d]
  uint16_t* mv;        // [B][Hkv][M][d], updated in place
  const uint16_t* q;   // [B][T][Hq][d] or null
  const uint16_t* wq;  // [B][T][Hkv][d] or null
  const uint16_t* wv;  // [B][T][Hkv][d] or null
  uint16_t* out;       // [B][T][Hq][d] or null
  float* norm_w;       // [B*Hkv][T]   shift of each write row: max + log2(sum of exp2(score - max))
  float* norm_r;       // [B*Hkv][T*G] the same of each read row, for a chunk that only reads
  uint16_t* snap;      // [ceil(T/128)][B*Hkv] MV at the start of each sub-chunk as operand tiles (M x d); a chunk that
                       // only reads: one copy of MV as [B*Hkv][d][M]
  uint16_t* wvt;       // [B*Hkv] WV as operand tiles (Tpad x d), zero beyond T
  uint32_t Tpad;       // T rounded up to whole sub-chunks
  uint32_t B, Hq, Hkv, G, M, d, T;
  uint32_t has_write, has_read, mk_per_seq;
  float rscale_l2e, wscale_l2e;
  uint32_t c_begin;    // first sub-chunk of a read launch
  uint32_t stats_read; // the statistics kernel also covers the read rows (chunks that only read)
  uint32_t stats_split;  // workgroups of the statistics kernel that share a row tile's keys
  float2* stats_part;    // [B*Hkv][stats_split][rows] their (max, sum) pairs, if more than one
  const float* gate;   // [B][T][Hkv] step sizes (any sign) or null
};
constexpr uint32_t kPrefillSubChunk = 128;
hipError_t launch_prefill_bf16(const PrefillParams& p, hipStream_t s);
bool prefill_one_pass(const PrefillParams& p);   // a chunk of few tokens that is one pass over keys and values

// dtype: 0 = fp32, 1 = bf16 (the ABI's bct_dtype values).
hipError_t launch_scores(const DecodeParams& p, int dtype, hipStream_t s);
hipError_t launch_normalise(const DecodeParams& p, hipStream_t s);
hipError_t launch_stream(const DecodeParams& p, int dtype, hipStream_t s);
hipError_t launch_stream_gqa(const DecodeParams& p, hipStream_t s);   // bf16, G > 2, with a read
hipError_t launch_merge(const DecodeParams& p, int dtype, hipStream_t s);
hipError_t launch_fused(const DecodeParams& p, hipStream_t s);   // fp32, G = 1
// A step that is one launch of decode_whole_kernel: `workgroups` (0: it is not) of `threads` threads per memory.
struct WholePlan {
  uint32_t workgroups, threads;
};
// Of a step that writes keys in that launch: the keys, the key write vectors [B][Hkv][d] (null: none), their step sizes
// [B][Hkv] (strides of the gate) or null.
struct KeyWrite {
  void* mk;
  const void* wk;
  const float* gate;
};
// two_allowed: a memory may be two workgroups', which read its inputs while the other one stores
WholePlan plan_whole(const DecodeParams& p, int dtype, bool two_allowed);
hipError_t launch_whole(const DecodeParams& p, const WholePlan& w, const KeyWrite& kw, int dtype, hipStream_t s);
hipError_t launch_fill_zero(void* dst, size_t n_bytes, hipStream_t s);
hipError_t launch_copy(void* dst, const void* src, size_t n_bytes, hipStream_t s);
hipError_t launch_randomize(void* dst, size_t n_bytes, int dtype, uint64_t seed, float amplitude, hipStream_t s);

// Launches indexed by memory (unit = b * Hkv + h) put the unit on grid.y and, beyond the 65535 that a grid
// dimension other than x holds, on grid.z as well: unit = blockIdx.z * kUnitsPerZ + blockIdx.y.  A workgroup
// whose unit is past the end returns at once (the test is uniform over the workgroup).
constexpr uint32_t kUnitsPerZ = 32768;
inline dim3 unit_grid(uint32_t x, uint64_t units) {
  return dim3(x, (unsigned)(units < kUnitsPerZ ? units : kUnitsPerZ), (unsigned)((units + kUnitsPerZ - 1) / kUnitsPerZ));
}

// Chooses stat_tile / n_tiles (scores pass) and the MV pass shape (mv_bs, mv_u, S).
void plan_decode(DecodeParams& p, int dtype);
void plan_mv_pass(DecodeParams& p, int dtype);

}  // namespace bct

#endif
