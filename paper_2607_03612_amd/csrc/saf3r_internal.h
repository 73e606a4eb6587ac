// Internal declarations shared by the gfx950 kernels and the C ABI layer.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace saf3r {

constexpr int kHeadDim = 64;
constexpr int kBlock = 64;
constexpr int kMaxHeads = 256;
constexpr int kMaxBlocks = 16384;  // select keeps one score row per query block in LDS

enum Pattern : int32_t {
  kDense = 0,
  kFrameLocal = 1,
  kTopK = 2,
  kAnchor = 3,
  kStride = 4,
  kGlobalProbe = 5,
  kCosineTopK = 6
};

constexpr int kMaxCosineDim = 4096;   // feature width accepted by the cosine selection
constexpr int kMaxCosinePerFrame = 64;  // key blocks kept per frame by a cosine head
constexpr int kNmseParts = 128;         // NMSE partial sums per head (workspace pairs)
// Device array of saf3r_nmse_noalloc's partial sums: every head count the
// library accepts (one float64 pair per part).
constexpr int64_t kNmseScratchBytes = (int64_t)kMaxHeads * kNmseParts * 16;

// ---------------------------------------------------------------- launches

struct PoolArgs {
  int64_t n;            // tokens per head
  int32_t nb;           // blocks per head
  int32_t n_heads;      // heads to pool (the Top-K heads)
  int16_t head[kMaxHeads];
};

// The Top-K heads, and after them in head[] the static and the global-probe
// heads whose lists the same launch writes.
struct TopKArgs {
  int64_t n;
  int32_t nb;
  int32_t cap;
  int32_t tokens_per_frame;
  int32_t rows_per_group;  // query blocks scored together by one workgroup
  int32_t n_heads;         // Top-K heads
  int32_t n_static;
  int32_t n_global;        // only where nb <= kGlobalFusedBlocks
  int16_t head[kMaxHeads];
  int32_t topk[kMaxHeads];   // Top-K, global: blocks kept; static: the class parameter
  int8_t pattern[kMaxHeads];  // of the static heads
};
// Global-probe heads of layers up to this size go with the Top-K launch: their
// one workgroup per head takes 6 KB + 12 bytes per block of LDS and writes
// every row itself, so only up to so many list entries of a head (nb * cap) for
// each turn of the chip that the Top-K rows beside it take, twice as many in one
// launch without a workspace, which takes longer. us for 4 Top-K heads and two
// such, with the Top-K launch / in launches of their own: 10 / 23 at 128 blocks,
// 51 / 55 at 651 and 53 k entries, 50 / 51 at 105 k, 61 / 53 at 211 k, 69 / 65 at
// 1024 and 131 k, 155 / 75 at 1049 k; without a workspace 46 / 50 at 651 and 211
// k, 55 / 59 at 1024 and 262 k, 60 / 53 at 800 and 320 k. Beside 10 Top-K heads
// (three turns) 94 / 105 at 1024 and 262 k, 109 / 101 at 912 and 415 k; without a
// workspace 80 / 110 at 1024 and 524 k, 127 / 122 at 1049 k.
constexpr int kCus = 256;
constexpr int kGlobalFusedBlocks = 1024;
constexpr int64_t kGlobalFusedEntries = 1 << 17;
// Top-K rows of layers up to kOneLaunchBlocks are scored and selected in one
// launch with or without a workspace, four rows to a workgroup, as long as that
// makes at most two workgroups per CU: a third one's turn costs more than the
// second launch (each workgroup reads every pooled key). us, one launch / two
// (with a workspace): 10 Top-K heads beside 6 static ones 7.0 / 10.8 at 17
// blocks, 13.8 / 15.4 at 172 (430 workgroups), 18.1 / 16.5 at 220 (550); 16
// heads 12.2 / 14.3 at 128 (512), 16.8 / 15.7 at 172 (688), 27.6 / 18.8 at 256;
// 40 heads 13.9 / 14.2 at 64 (640), 34.4 / 26.7 at 172. (Sixteen rows to a
// workgroup of 8 or 16 waves: 13 and 20 us at 17 blocks; two rows to one of two
// waves: 18 us at 172.)
constexpr int kOneLaunchBlocks = 256;
constexpr int kOneLaunchGroups = 512;

struct StaticArgs {
  int64_t n;
  int32_t nb;
  int32_t cap;
  int32_t tokens_per_frame;
  int32_t n_heads;
  int16_t head[kMaxHeads];
  int8_t pattern[kMaxHeads];
  int32_t param[kMaxHeads];  // ANCHOR: anchor frame; STRIDE: key stride
};

// Paper-literal query probe: one probe per head over all N queries.
struct GlobalArgs {
  int64_t n;
  int32_t nb;
  int32_t cap;
  int32_t n_heads;
  int16_t head[kMaxHeads];
  int32_t topk[kMaxHeads];
};

// Key-range split of long lists: on a layer of at least kSplitMinExtent key
// blocks, a list head whose list can hold kSplitMinBlocks or more key blocks
// runs as kSplitChunks work items per query block, item c walking the list
// entries in key blocks [c nb / C, (c + 1) nb / C). The waves that run together on an XCD then
// read K and V from one key range instead of the head's whole extent. Each
// item writes its unnormalised output and softmax statistics to a workspace
// and a merge launch combines the chunks in a fixed order.
constexpr int kSplitMinBlocks = 384;
constexpr int kSplitMinExtent = 4096;
constexpr int kSplitChunks = 4;
// Load balance: a list or dense head whose items walk at least
// kBalanceMinBlocks (bf16) or kBalanceMinBlocksF32 key blocks is also split
// when one item is longer than twice the layer's work spread over the chip's
// wave slots (256 CUs x 4 SIMDs x 2 waves), i.e. when its rows, not the total
// work, would set the launch's length. The workspace is sized by that rule; a
// launch splits fewer heads, because the four waves of a workgroup can share a
// row (fp32: always; bf16: where that shortens the launch) and the merge
// launch costs about 10 us: rows of kSplitMinWalk (bf16) or kSplitMinWalkF32
// or more blocks whose quarter outlasts twice the layer's work per wave slot
// (fp32 attention, unsplit / split: 16 heads, one or four of them dense, 1044
// tokens 33 / 45 us, 5496 tokens 156 / 185, 10992 tokens 415 / 428; one dense
// head of 5496 tokens 119 / 68, 8 heads of 10992 tokens with one 246 / 202).
constexpr int kBalanceMinBlocks = 32;
constexpr int kBalanceMinBlocksF32 = 8;
constexpr int kSplitMinWalk = 128;
constexpr int kSplitMinWalkF32 = 64;
// Shared rows in bf16 (shared_rows_cost in api.cpp): the start and end of a
// wave, and of one that shares a row, in key blocks' time, and the gain from
// which rows are shared. On 2244 random tables (16 to 900 key blocks, 1 to 24
// heads, no workspace) the launch so chosen takes 1.018 times the best of its
// forms, always one wave a row 1.32 times; 14 tables are more than 4% slower than
// with one wave a row. (Without a look at whole turns 171, by up to half: 653
// equal rows of 8 blocks take 20 us shared, 15 not; of 48 blocks 48 and 54; 130
// rows of 8 blocks 8.6 and 12.)
constexpr int kItemOverhead = 3;
constexpr int kSharedOverhead = 4;
constexpr double kFirstTurn = 0.7;
constexpr double kShareGain = 0.95;
constexpr int kShareMinBlocks = 8;  // shorter rows are not worth four waves
constexpr int64_t kWaveSlots = 2048;
constexpr int64_t kSplitItemBytes = (int64_t)kBlock * kHeadDim * 4 + (int64_t)kBlock * 2 * 4;

struct AttnArgs {
  int64_t n;
  int32_t nb;
  int32_t cap;
  int32_t heads;          // heads in this launch (entries of order[])
  int32_t slab;           // query blocks of one head handled by one XCD: ceil(nb / 8)
  int32_t slab4;          // groups of four of them: ceil(ceil(nb / 4) / 8)
  int32_t waves;          // bf16: waves per workgroup, 1 or 4
  int32_t mode;           // 0: lists or dense per head; 1: every head dense; 2: STRIDE heads
  int32_t splits;         // key ranges of a split head (kSplitChunks)
  float scale_log2;       // log2(e) / sqrt(64)
  float* part_o;          // split items' O^T accumulators, 64 x 64 fp32 each
  float* part_ml;         // split items' (running max, row sum) per query
  int16_t order[kMaxHeads];        // heads of this launch, longest work item first
  int16_t split_pos[kMaxHeads];    // by order position: index among split heads, or -1
  int32_t unit_start[kMaxHeads + 1];  // by order position: first work unit (slab units a key range)
  int16_t shared_before[kMaxHeads + 1];  // four waves: key ranges of heads before it whose rows they share
  int8_t dense[kMaxHeads];    // by head index: 1 = iterate all key blocks
  int32_t stride[kMaxHeads];  // by head index: key stride of a STRIDE head
};

static_assert(sizeof(AttnArgs) <= 4096 - 64, "kernel arguments: 4 KB with the pointers beside it");

// The first work unit of an order position for workgroups of four waves: a
// key range is slab units where they share its rows, slab4 where they do not.
__host__ __device__ inline int unit4_start(const AttnArgs& a, int pos) {
  return a.unit_start[pos] / a.slab * a.slab4 + a.shared_before[pos] * (a.slab - a.slab4);
}

// What workgroup `group` of an attention launch does.
struct Work {
  int h, i;
  int chunk;  // key range of a split head's item, or -1
  int item;   // split item index (partials), or -1
  bool shared;  // bf16: the workgroup's waves share the row
  bool valid;
};

// The last order position whose first unit start(pos) is at most u.
template <typename Start>
__host__ __device__ inline int order_position(const AttnArgs& a, int u, Start start) {
  int lo = 0, hi = a.heads;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (start(mid) <= u) lo = mid;
    else hi = mid;
  }
  return lo;
}

// Work unit u = b / 8 of order position hh covers unit_start[hh] <= u <
// unit_start[hh + 1]: slab units per key range, key ranges in order, so the
// items that run together on an XCD share one key range of one head.
__host__ __device__ inline Work work_item(const AttnArgs& a, uint32_t group) {
  const int xcd = group & 7;
  const int u = group >> 3;
  Work w;
  w.valid = u < a.unit_start[a.heads];
  if (!w.valid) return w;
  const int lo = order_position(a, u, [&](int p) { return a.unit_start[p]; });
  const int r = u - a.unit_start[lo];
  const int chunk = r / a.slab;
  const int i = xcd * a.slab + (r - chunk * a.slab);
  w.valid = i < a.nb;
  w.h = a.order[lo];
  w.i = i;
  const int sp = a.split_pos[lo];
  w.chunk = sp >= 0 ? chunk : -1;
  w.item = sp >= 0 ? (sp * a.splits + chunk) * a.nb + i : -1;
  return w;
}

// The same for workgroups of four waves (bf16): a unit is four neighbouring
// query blocks, one a wave, or, for a head whose rows are shared, one query
// block for all four. Slabs start one XCD further on from head to head, so
// that the short last slab is not always the same XCD's.
__host__ __device__ inline Work work_item4(const AttnArgs& a, uint32_t group, int wave) {
  const int u = group >> 3;
  Work w;
  w.valid = u < unit4_start(a, a.heads);
  if (!w.valid) return w;
  const int lo = order_position(a, u, [&](int p) { return unit4_start(a, p); });
  w.shared = a.shared_before[lo + 1] > a.shared_before[lo];
  const int slab = w.shared ? a.slab : a.slab4;
  const int r = u - unit4_start(a, lo);
  const int chunk = r / slab;
  const int unit = (int)((group + lo) & 7) * slab + (r - chunk * slab);
  const int i = w.shared ? unit : 4 * unit + wave;
  w.valid = i < a.nb;
  w.h = a.order[lo];
  w.i = i;
  const int sp = a.split_pos[lo];
  w.chunk = sp >= 0 ? chunk : -1;
  w.item = sp >= 0 ? (sp * a.splits + chunk) * a.nb + i : -1;
  return w;
}

// The merge of split heads: one wave per (split head, query block).
struct MergeArgs {
  int64_t n;
  int32_t nb;
  int32_t splits;
  int32_t n_split;
  int32_t dtype;  // of the output rows: 1 bf16, 0 fp32
  int16_t head[kMaxHeads];  // by split index: head
};

// Block-wise DINO Top-K on caller-supplied per-token features.
struct CosineArgs {
  int64_t n;
  int32_t nb;
  int32_t cap;
  int32_t dim;  // feature width
  int32_t tokens_per_frame;
  int32_t n_groups;                     // cosine heads grouped by per-frame count
  int32_t group_k[kMaxHeads];           // key blocks kept per frame by group g
  int16_t group_start[kMaxHeads + 1];   // group g: head[group_start[g] .. group_start[g + 1])
  int16_t head[kMaxHeads];
};

// List check of the listed heads: one wave per (head, query block).
struct ValidateArgs {
  int32_t nb;
  int32_t cap;
  int32_t n_heads;
  int16_t head[kMaxHeads];
  int32_t expect[kMaxHeads];  // by slot: the exact count a row must hold, or -1 (any)
};

hipError_t launch_pool(int dtype, const void* q, const void* k, double* qp, double* kp,
                       const PoolArgs& a, hipStream_t s);
hipError_t launch_select_topk(const double* qp, const double* kpT, int32_t* idx, int32_t* cnt,
                              double* scores, const TopKArgs& a, size_t lds_bytes, hipStream_t s);
hipError_t launch_select_static(int32_t* idx, int32_t* cnt, const StaticArgs& a, hipStream_t s);
// The list check on `s`, then its result copied to the host and the stream
// waited for: out[0] = rows that fail, out[1] = the lowest failing row
// (h * nb + i). `result` is the caller's 8-byte device workspace.
hipError_t run_validate_index(const int32_t* idx, const int32_t* cnt, int32_t* result,
                              const ValidateArgs& a, int32_t out[2], hipStream_t s);
hipError_t launch_select_global(const double* qp, const double* kpT, int32_t* idx, int32_t* cnt,
                                double* scores, const GlobalArgs& a, hipStream_t s);
hipError_t launch_cosine(int dtype, const void* f, double* fb, double* sim, int32_t* idx,
                         int32_t* cnt, const CosineArgs& a, hipStream_t s);
hipError_t launch_nmse(int dtype, const void* ref, const void* test, void* workspace, double* out,
                       int heads, int64_t n, hipStream_t s);
// Device address of the current device's NMSE scratch array (resolved on the
// first call on that device).
hipError_t nmse_scratch(void** ptr);
hipError_t launch_attention(int dtype, const void* q, const void* k, const void* v,
                            const int32_t* idx, const int32_t* cnt, void* out, float* lse,
                            const AttnArgs& a, hipStream_t s);
hipError_t launch_attention_merge(const float* part_o, const float* part_ml, void* out,
                                  float* lse, const MergeArgs& a, hipStream_t s);

// Top-K selection sizes, shared by the kernels and the host layer. Key
// slots per lane for a row of nb blocks: ceil(nb / 64) rounded up to a
// multiple of 4; a row occupies 64 * row_chunk(nb) words (LDS or workspace).
__host__ __device__ constexpr int row_chunk(int nb) { return ((nb + 63) / 64 + 3) & ~3; }
// LDS entries after the last row, so that every lane may read its C slots
// rounded up to a multiple of 8 unconditionally.
constexpr int kRowPad = 128;
// Bytes of LDS the single-launch Top-K selection needs for `rows` query blocks.
inline size_t topk_lds_bytes(int rows, int nb) {
  return ((size_t)rows * 64 * row_chunk(nb) + kRowPad) * sizeof(uint32_t);
}
// Threads per workgroup of the single-launch Top-K selection for `rows` query blocks.
inline int topk_threads(int rows) { return rows >= 16 ? 512 : 256; }
// Workspace path of the Top-K selection: bytes of one query block's key row.
inline size_t topk_ws_row_bytes(int nb) { return (size_t)64 * row_chunk(nb) * sizeof(uint32_t); }
// The workspace path's two launches (scores into `keys`, then one wave per row).
hipError_t launch_select_topk_ws(const double* qp, const double* kpT, uint32_t* keys, int32_t* idx,
                                 int32_t* cnt, double* scores, const TopKArgs& a, hipStream_t s);

}  // namespace saf3r
