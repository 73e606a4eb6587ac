// Block-sparse attention over the kept key blocks (Sec. 4.1: the Top-K and
// static kernels compute only the scores between the queries and the
// selected keys, and the softmax is renormalised over that set), with the
// dense ("Full") case as the same loop over every key block.
//
// One wave owns one (head, 64-query block) and walks its kept-block list in
// half tiles of 32 keys with an online softmax:
//   S^T = K Q^T      (keys x queries) on MFMA, so a lane owns one query
//                    column and the row sum stays inside the lane pair
//                    (lane, lane ^ 32);
//   O^T += V^T P^T   (head dim x queries) on MFMA, P^T taken straight from
//                    the S^T accumulators, V^T read from LDS with the gfx950
//                    transposing LDS read so V is never transposed in memory.
// The half-tile steps are software-pipelined: step t issues S^T of half t+1
// and the P V product of half t-1 on the matrix cores while the VALU runs
// the softmax of half t, and the scheduler is told to interleave the two
// streams. Q sits in registers for the whole loop; K and V half tiles are
// staged in LDS by the direct buffer-to-LDS load two steps ahead. Every
// global access of Q, K, V and O is a buffer instruction whose range-checked
// offsets (vector and immediate, never the unchecked scalar offset) are
// bounded by the head's extent, so a partial last block reads zeros and a
// corrupt index list cannot touch memory outside the head.
//
// Launch order: workgroup b runs on XCD b % 8; each XCD takes a contiguous
// slab of query blocks of every head (neighbouring query blocks share kept
// key blocks, which then hit in that XCD's L2), longest work items first.
//
// Long lists can run split into key ranges: a work item is then (head, key
// range c of splits, query block) and walks only its list's entries inside
// range c (a dense head's item walks every block of the range), ranges in
// order within a head, so the waves that run together on an XCD read K and V
// from one range rather than the head's whole extent, and no item of a small
// layer is much longer than the others.
// Such an item stores its unnormalised O^T and (running max, row sum) per
// query in a workspace; attn_merge_kernel combines the ranges of each query
// block in range order.
//
// Where one wave per row would leave a launch waiting for its longest rows, it
// runs attn_bf16_rows4_kernel: workgroups of four waves with the same walk,
// which take four query blocks or share one row and combine in LDS.
//
// A launch in which every head is dense runs attn_bf16_dense_kernel: four
// waves take four neighbouring query blocks of one head, and since all four
// walk every key block in order, each K and V half tile is staged in LDS
// once for the four (one barrier per half-tile step).
#include <type_traits>

#include "saf3r_internal.h"

namespace saf3r {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
typedef __attribute__((address_space(3))) f32x4 lds_f32x4;

constexpr uint32_t kRsrcWord3 = 0x00020000u;  // gfx9 buffer descriptor: 32-bit raw data
constexpr float kNegInf = -__builtin_inff();
constexpr float kLn2 = 0.6931471805599453f;

__device__ inline __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes,
                                           (int)kRsrcWord3);
}

__device__ inline bf16x8 load_b128(__amdgpu_buffer_rsrc_t r, uint32_t byte_off) {
  return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, (int)byte_off, 0, 0));
}

__device__ inline float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// A split item's share of its row: key blocks [c nb / splits, (c + 1) nb /
// splits) of range c. A dense head's item walks every block of the range
// (from dense_lo); a list head's item keeps its list's entries inside the
// range: in an ascending list, the entries after those below jlo and before
// the first at or above jhi (any other list still yields a sub-range of the
// row, read within it).
__device__ inline void split_range(const Work& w, const AttnArgs& a, bool dense,
                                   const int32_t*& list, int& count, int& dense_lo, int lane) {
  const int nb = a.nb;
  const int jlo = (int)(((int64_t)w.chunk * nb) / a.splits);
  const int jhi = (int)(((int64_t)(w.chunk + 1) * nb) / a.splits);
  if (dense) {
    dense_lo = jlo;
    count = jhi - jlo;
    return;
  }
  int below_lo = 0, below_hi = 0;
  for (int base = 0; base < count; base += 64) {
    const int p = base + lane;
    const int j = p < count ? list[p] : 0x7fffffff;
    below_lo += __popcll(__ballot(j < jlo));
    below_hi += __popcll(__ballot(j < jhi));
  }
  list += below_lo;
  count = max(below_hi - below_lo, 0);
}

typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

// A split item's result: its O^T accumulators as they stand, relative to its
// own running max (register-major: 16 stores of 64 lanes x 16 B), and the
// (running max, row sum) of each query. An empty range writes only the
// statistics (-inf, 0), and the merge never reads its accumulators.
template <typename Acc>
__device__ inline void store_partials(const Acc (&o)[2][2], const float (&m)[2], const float (&lt)[2],
                                      const AttnArgs& a, int64_t item, bool empty, int lane) {
  const int l32 = lane & 31;
  if (!empty) {
    float* const po = a.part_o + item * (kBlock * kHeadDim);
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int tq = 0; tq < 2; ++tq)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *(f32x4_t*)(po + (((c * 2 + tq) * 4 + g) * 64 + lane) * 4) =
              f32x4_t{o[c][tq][4 * g], o[c][tq][4 * g + 1], o[c][tq][4 * g + 2], o[c][tq][4 * g + 3]};
  }
  if ((lane >> 5) == 0) {
#pragma unroll
    for (int tq = 0; tq < 2; ++tq)
      *(f32x2_t*)(a.part_ml + (item * kBlock + 32 * tq + l32) * 2) =
          empty ? f32x2_t{-__builtin_inff(), 0.f} : f32x2_t{m[tq], lt[tq]};
  }
}

// fp32 output of one query block from the O^T accumulators (register e of
// tile [c][tq] of lane (l32, hf) is head dim 32c + 8(e/4) + 4hf + e%4 of
// query 32tq + l32), scaled by inv; lse_row, if not null, is the head's LSE
// row (natural log).
template <typename Acc>
__device__ inline void write_out_tile_f32(const Acc (&o)[2][2], const float (&inv)[2],
                                          const float (&lse_val)[2], __amdgpu_buffer_rsrc_t ro,
                                          float* lse_row, int i, int64_t n, int lane) {
  const int l32 = lane & 31;
  const int hf = lane >> 5;
#pragma unroll
  for (int tq = 0; tq < 2; ++tq) {
    const int query = i * kBlock + 32 * tq + l32;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        f32x4_t ov;
#pragma unroll
        for (int r = 0; r < 4; ++r) ov[r] = o[c][tq][4 * g + r] * inv[tq];
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(i32x4, ov), ro,
                                               (query * kHeadDim + 32 * c + 8 * g + 4 * hf) * 4, 0, 0);
      }
    if (lse_row && hf == 0 && query < n) lse_row[query] = lse_val[tq];
  }
}

// ------------------------------------------------------------------ bf16

typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) char lds_char;
typedef __attribute__((address_space(3))) const bf16x8 lds_bf16x8;

// LDS tiles: rows of 128 B; 16-byte chunk c of row r is stored at slot
// c ^ f(r), f(r) = (bit2(r), bit1(r), bit0(r) ^ bit1(r) ^ bit3(r)). With it
// the MFMA operand reads (16 rows at one chunk) and the transposing reads
// (4 rows x 2 chunks per 16 lanes, 4 x 4 per 32) touch every bank once,
// whether the LDS serves 128 or 256 bytes per clock.
__device__ inline int swz_f(int r) {
  return ((r >> 2) & 1) | (r & 2) | (((r ^ (r >> 1) ^ (r >> 3)) & 1) << 2);
}
__device__ inline int swz(int r, int c) { return r * 128 + ((c ^ swz_f(r)) << 4); }

// Direct buffer-to-LDS loads of 8-row groups: instruction n fills LDS bytes
// [1024n, 1024n + 1024), lane l its 16 bytes at 16l, i.e. row 8n + l/8,
// slot l%8, which must hold chunk (l%8) ^ f(8n + l/8) = (l%8) ^ f(l/8) ^ (4
// if n is odd). The lane's byte offset inside its 8-row group depends only
// on the parity of n; the group offset 1024n is the instruction's immediate
// offset, which the hardware adds to both the memory and the LDS address.
struct DmaLaneOffsets {
  int even, odd;
};
__device__ inline DmaLaneOffsets dma_lane_offset(int lane) {
  const int r = lane >> 3;
  const int c = (lane & 7) ^ swz_f(r);
  return {(r * kHeadDim + c * 8) * 2, (r * kHeadDim + (c ^ 4) * 8) * 2};
}
// max / sum of a value over the lane pair (l, l ^ 32) that shares a query
__device__ inline float pair_max(float x) {
  const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(s[0]), __uint_as_float(s[1]));
}
__device__ inline float pair_sum(float x) {
  const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}

constexpr bf16x2 kOnes = {(__bf16)1.0f, (__bf16)1.0f};

// Waits expressed as s_waitcnt immediates (gfx9 encoding: vmcnt in bits 3:0
// and 15:14, expcnt 6:4, lgkmcnt 11:8).
constexpr int kWaitVm8 = 0x0F78;   // vmcnt(8)
constexpr int kWaitVm0 = 0x0F70;   // vmcnt(0)
constexpr int kWaitLgkm0 = 0xC07F; // lgkmcnt(0)

// One 32-row half tile (rows 64j + 32h .. of the head) into an LDS half
// buffer with the direct buffer-to-LDS load: four 1 KB instructions. The
// tile's offset goes into the base and extent of a descriptor built for this
// tile in scalar registers, and the scalar offset operand stays 0: the
// hardware range-checks the vector and immediate offsets against the extent
// but not the scalar offset. So rows past the head's last token (a partial
// last block) read zeros, and a block index outside [0, nb) reads a tile of
// zeros instead of memory outside the head.
// head_bytes - t, or 0 when t is at or past the end, on the scalar unit: as
// plain C the compiler lowers this saturating subtract of two scalars to a
// copy, a clamped vector subtract and a readfirstlane, three VALU
// instructions per tile load in the loop. The borrow of s_sub_u32 sets SCC.
__device__ inline uint32_t rem_bytes(uint32_t head_bytes, uint32_t t) {
  uint32_t r;
  asm("s_sub_u32 %0, %1, %2\n\ts_cselect_b32 %0, 0, %0" : "=&s"(r) : "s"(head_bytes), "s"(t) : "scc");
  return r;
}

__device__ inline void dma_half(const uint16_t* head, uint32_t head_bytes, int nb, int j, int h,
                                lds_char* buf, DmaLaneOffsets off) {
  const uint32_t t = __builtin_amdgcn_readfirstlane(
      (uint32_t)j < (uint32_t)nb ? ((uint32_t)j * kBlock + 32u * h) * (kHeadDim * 2) : head_bytes);
  const uint32_t rem = rem_bytes(head_bytes, t);
  const __amdgpu_buffer_rsrc_t r = make_rsrc(reinterpret_cast<const char*>(head) + t, rem);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)buf, 16, off.even, 0, 0, 0);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)buf, 16, off.odd, 0, 1024, 0);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)buf, 16, off.even, 0, 2048, 0);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)buf, 16, off.odd, 0, 3072, 0);
}

// Key sets a launch walks: per-head lists or all blocks (kLists), every block
// of every head (kAllDense), or the keys 0, s, 2s, ... of STRIDE heads taken
// 64 at a time as virtual blocks (kStrided).
enum AttnMode { kLists = 0, kAllDense = 1, kStrided = 2 };

// One 32-row half of virtual key block j of a STRIDE head: key rows
// (64j + 32h + r) * stride, r < 32, into an LDS half buffer (same slot layout
// as dma_half). As there the half's first row goes into the descriptor, on the
// scalar unit, and a lane's four offsets inside it are the same for every half
// (StrideLaneOffsets), so a load takes no VALU instruction; rows at or past
// token n lie past the extent and load as zeros. With per-load 64-bit row
// arithmetic instead, every head at stride 7 took 1.47 ms at 43968 tokens and
// 12.3 at 137400, 1.31 and 11.1 so.
struct StrideLaneOffsets {
  int group[4];  // rows 8g .. 8g + 7
};
__device__ inline StrideLaneOffsets stride_lane_offsets(int lane, uint32_t stride) {
  const int rr = lane >> 3;
  const int c = (lane & 7) ^ swz_f(rr);
  StrideLaneOffsets o;
#pragma unroll
  for (int g = 0; g < 4; ++g)  // a row past any head's end (at most 2^20 rows) stays past it
    o.group[g] = (int)(min((uint32_t)(8 * g + rr) * stride, 1u << 21) * (kHeadDim * 2)) + ((g & 1) ? (c ^ 4) : c) * 16;
  return o;
}
__device__ inline void dma_half_strided(const uint16_t* head, uint32_t n, uint32_t stride, int j, int h, lds_char* buf,
                                        const StrideLaneOffsets& off) {
  const uint32_t tok = __builtin_amdgcn_readfirstlane(min(((uint32_t)j * kBlock + 32u * h) * stride, n));
  const __amdgpu_buffer_rsrc_t r = make_rsrc(head + (size_t)tok * kHeadDim, (n - tok) * (kHeadDim * 2));
#pragma unroll
  for (int g = 0; g < 4; ++g)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)(buf + 1024 * g), 16, off.group[g], 0, 0, 0);
}

// Output of one query block from the O^T accumulators (register e of tile
// [c][tq] of lane (l32, hf) holds head dim 32c + 8(e/4) + 4hf + e%4 of query
// 32tq + l32): scaled by inv, rounded to bf16 into two idle LDS half buffers
// (query rows 0..31 in b0, 32..63 in b1, same swizzle as the K tiles), then
// stored as full 128-byte rows, eight 1 KB stores. lse_row, if not null, is
// the head's LSE row; lse_val is in natural log.
__device__ inline void write_out_tile(const f32x16 (&o)[2][2], const float (&inv)[2],
                                      const float (&lse_val)[2], lds_char* b0, lds_char* b1,
                                      __amdgpu_buffer_rsrc_t ro, float* lse_row, int i, int64_t n,
                                      int lane) {
  const int l32 = lane & 31;
  const int hf = lane >> 5;
#pragma unroll
  for (int tq = 0; tq < 2; ++tq) {
    const int query = i * kBlock + 32 * tq + l32;
    lds_char* const ob = tq ? b1 : b0;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        bf16x4 ov;
#pragma unroll
        for (int r = 0; r < 4; ++r) ov[r] = (__bf16)(o[c][tq][4 * g + r] * inv[tq]);
        *(lds_bf16x4*)(ob + swz(l32, 4 * c + g) + 8 * hf) = ov;
      }
    if (lse_row && hf == 0 && query < n) lse_row[query] = lse_val[tq];
  }
#pragma unroll
  for (int nn = 0; nn < 8; ++nn) {
    const int row = 8 * nn + (lane >> 3);
    const int chunk = lane & 7;
    lds_char* const ob = row >= 32 ? b1 : b0;
    const bf16x8 val = *(lds_bf16x8*)(ob + swz(row & 31, chunk));
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(i32x4, val), ro,
                                           (int)(((i * kBlock + row) * kHeadDim + 8 * chunk) * 2), 0, 0);
  }
}

// Per-wave state and building blocks of the bf16 walk over one 64-query
// block: Q^T in registers, the O^T accumulators, the running max and row-sum
// share of each query half, and the lane's LDS operand offsets.
template <bool kPin>
struct Bf16Walk {
  bf16x8 qB[2][4];  // Q^T as the B operand: qB[tq][s] = Q[64i + 32tq + l32][16s + 8hf + (0..7)]
  f32x16 o[2][2];   // O^T tiles [head-dim half c][query half tq]
  float nm[2];      // minus the running max of the log2-scaled scores (the fma's addend)
  float l[2];       // this lane's share of the running row sum
  float sc;
  int l32, hf;
  int tr_row, tr_col;  // transposing-read position of this lane in a 4-row x 16-column group
  // Lane parts of the LDS operand addresses: the K read of chunk pair st (row
  // l32), and the transposing V reads of column half c, rows +0 / +8 of a
  // 16-row group (the 16-row group's 2 KB is an immediate offset). With kPin
  // an empty asm redefines a part at each use, so the buffer's base also
  // goes into the immediate offset instead of one hoisted address register
  // per (buffer, part): eight registers in all for a ring of eight buffers.
  // With two buffers per tensor the hoisted addresses measured faster.
  int kpart[4];
  int vpart[2][2];

  __device__ __forceinline__ void init(__amdgpu_buffer_rsrc_t rq, int i, int lane, float scale, int lds_off = 0) {
    l32 = lane & 31;
    hf = lane >> 5;
    sc = scale;
#pragma unroll
    for (int tq = 0; tq < 2; ++tq)
#pragma unroll
      for (int s = 0; s < 4; ++s)
        qB[tq][s] = load_b128(
            rq, (uint32_t)(((i * kBlock + 32 * tq + l32) * kHeadDim + 16 * s + 8 * hf) * 2));
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int tq = 0; tq < 2; ++tq)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[c][tq][e] = 0.f;
    nm[0] = nm[1] = -kNegInf;
    l[0] = l[1] = 0.f;
    tr_row = 4 * hf + ((lane & 15) >> 2);
    tr_col = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
#pragma unroll
    for (int st = 0; st < 4; ++st) kpart[st] = swz(l32, 2 * st + hf) + lds_off;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int r8 = 0; r8 < 2; ++r8)
        vpart[c][r8] = swz(tr_row + 8 * r8, (32 * c + tr_col) >> 3) + (tr_col & 7) * 2 + lds_off;
  }

  // S^T of a key half (32 keys x 64 queries) from an LDS K half buffer
  __device__ __forceinline__ void read_k(lds_char* kb, bf16x8 (&kA)[4]) {
#pragma unroll
    for (int st = 0; st < 4; ++st) {
      if constexpr (kPin) asm volatile("" : "+v"(kpart[st]));
      kA[st] = *(lds_bf16x8*)(kb + kpart[st]);
    }
  }
  __device__ __forceinline__ void read_v(lds_char* vb, bf16x8 (&vA)[2][2]) {
    if constexpr (kPin) {
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int r8 = 0; r8 < 2; ++r8) asm volatile("" : "+v"(vpart[c][r8]));
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(vb + 2048 * u + vpart[c][0]));
        const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(vb + 2048 * u + vpart[c][1]));
        vA[u][c] = bf16x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      }
  }
  __device__ __forceinline__ void mfma_s(const bf16x8 (&kA)[4], f32x16 (&s)[2]) {
    f32x16 acc0 = {}, acc1 = {};
#pragma unroll
    for (int st = 0; st < 4; ++st) {
      acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kA[st], qB[0][st], acc0, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kA[st], qB[1][st], acc1, 0, 0, 0);
    }
    s[0] = acc0;
    s[1] = acc1;
  }
  __device__ __forceinline__ void mfma_pv(const bf16x8 (&vA)[2][2], const bf16x8 (&p)[2][2]) {
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int tq = 0; tq < 2; ++tq)
          o[c][tq] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vA[u][c], p[u][tq], o[c][tq], 0, 0, 0);
  }
  // Online-softmax step over one key half. P = exp2(s*sc - m) is taken with
  // the running max as it stands and rounded to bf16; the row sum adds the
  // rounded values (one bf16 dot with (1, 1) per pair), so the normaliser
  // matches the weights the P V product uses. Only when some lane's share of
  // the row sum leaves [0, 2^12] (a new larger max, or the first half where
  // the max is still -inf and the sum is inf or NaN) is the half's max taken:
  // the running max moves to it, O and l are rescaled (after the P V of the
  // previous half, which is already issued) and P is recomputed. Keys at or
  // past `valid` (a partial last block) get P = 0.
  __device__ __forceinline__ void probs(const f32x16 (&s)[2], bf16x8 (&p)[2][2], float (&rs)[2]) {
#pragma unroll
    for (int tq = 0; tq < 2; ++tq) {
      const float nmcur = nm[tq];
      float r = 0.f;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        bf16x2 pr[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const f32x2 pf = {fast_exp2(fmaf(s[tq][8 * u + 2 * e], sc, nmcur)),
                            fast_exp2(fmaf(s[tq][8 * u + 2 * e + 1], sc, nmcur))};
          pr[e] = __builtin_convertvector(pf, bf16x2);
          r = __builtin_amdgcn_fdot2_f32_bf16(pr[e], kOnes, r, false);
        }
        p[u][tq] = bf16x8{pr[0][0], pr[0][1], pr[1][0], pr[1][1],
                          pr[2][0], pr[2][1], pr[3][0], pr[3][1]};
      }
      rs[tq] = r;
    }
  }
  __device__ __forceinline__ void mask_keys(f32x16 (&s)[2], int valid) {
    if (valid < 32) {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int key = 8 * (e >> 2) + 4 * hf + (e & 3);
        if (key >= valid) {
          s[0][e] = kNegInf;
          s[1][e] = kNegInf;
        }
      }
    }
  }
  __device__ __forceinline__ void fixup(f32x16 (&s)[2], bf16x8 (&p)[2][2], float (&rs)[2]) {
    // 0x45800000 is 2^12; inf and NaN compare above it as unsigned bits
    if (__ballot(__float_as_uint(rs[0]) > 0x45800000u || __float_as_uint(rs[1]) > 0x45800000u)) {
#pragma unroll
      for (int tq = 0; tq < 2; ++tq) {
        float mx = fmaxf(fmaxf(s[tq][0], s[tq][1]), s[tq][2]);
#pragma unroll
        for (int e = 3; e < 15; e += 2) mx = fmaxf(fmaxf(mx, s[tq][e]), s[tq][e + 1]);
        mx = fmaxf(mx, s[tq][15]);
        // -max(x, m) = min(-x, -m) and (-m) - (-m') = m' - m, exactly
        const float nmnew = fminf(-(pair_max(mx) * sc), nm[tq]);
        const float alpha = fast_exp2(nmnew - nm[tq]);
        nm[tq] = nmnew;
        l[tq] *= alpha;
#pragma unroll
        for (int c = 0; c < 2; ++c) o[c][tq] *= alpha;
      }
      probs(s, p, rs);
    }
    l[0] += rs[0];
    l[1] += rs[1];
  }

  // One half-tile step t: Sᵀ of half t+1 (from kb, if kNext) and O += Vᵀ Pᵀ
  // of half t-1 (from vb) on the matrix cores while the VALU runs the softmax
  // of half t (s_cur, keys past `valid` masked); then s_cur and p_prev move
  // on by one half. Both are issued in one scheduling region: the 12 LDS
  // operand reads first (mask 0x100), ten softmax VALU ops (0x002) while they
  // land, then each of the 16 MFMAs (0x008) followed by four VALU ops, so the
  // matrix cores and the VALU work on independent data side by side.
  template <bool kNext>
  __device__ __forceinline__ void step(lds_char* kb, lds_char* vb, int valid, f32x16 (&s_cur)[2],
                       bf16x8 (&p_prev)[2][2]) {
    bf16x8 kA[4];
    bf16x8 vA[2][2];
    if constexpr (kNext) read_k(kb, kA);
    read_v(vb, vA);
    f32x16 s_next[2];
    if constexpr (kNext) mfma_s(kA, s_next);
    mfma_pv(vA, p_prev);
    bf16x8 p_new[2][2];
    mask_keys(s_cur, valid);
    float rs[2];
    probs(s_cur, p_new, rs);
    __builtin_amdgcn_sched_group_barrier(0x100, 12, 0);
    __builtin_amdgcn_sched_group_barrier(0x002, 10, 0);
#pragma unroll
    for (int g = 0; g < 16; ++g) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
    }
    fixup(s_cur, p_new, rs);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int tq = 0; tq < 2; ++tq) p_prev[u][tq] = p_new[u][tq];
    if constexpr (kNext) {
      s_cur[0] = s_next[0];
      s_cur[1] = s_next[1];
    }
  }
  // The last step: no half t+1; O += Vᵀ Pᵀ of half t-1, the softmax of half
  // t, then the P V of half t itself.
  __device__ __forceinline__ void last_step(lds_char* vb_prev, lds_char* vb_cur, int valid, f32x16 (&s_cur)[2],
                            const bf16x8 (&p_prev)[2][2]) {
    bf16x8 vA[2][2];
    read_v(vb_prev, vA);
    mfma_pv(vA, p_prev);
    bf16x8 p_new[2][2];
    mask_keys(s_cur, valid);
    float rs[2];
    probs(s_cur, p_new, rs);
    fixup(s_cur, p_new, rs);
    read_v(vb_cur, vA);
    mfma_pv(vA, p_new);
  }
  __device__ __forceinline__ void running_max(float (&m)[2]) const {
    m[0] = -nm[0];
    m[1] = -nm[1];
  }
  // the row sums of the two query halves (the lane pair's shares added)
  __device__ __forceinline__ void row_sums(float (&lt)[2]) const {
    lt[0] = pair_sum(l[0]);
    lt[1] = pair_sum(l[1]);
  }
};

constexpr int kHalfBytes = 32 * 128;

// kWaves = 1: a workgroup is one wave and one item. kWaves = 4: four waves
// take four neighbouring query blocks, or share one row where a.shared says
// so: wave w walks list entries w, w + 4, ... with its own running max, row
// sum and O^T, and the four meet in LDS. With one wave per item a layer that
// does not fill the chip lasts as long as its longest row; a launch uses this
// form when sharing shortens it (4 frames of 1374 tokens, 16 heads: the layer
// 79 -> 61 us; 20 frames of 1001, 12 heads, three of them dense: 640 -> 522
// us) and the one-wave form, whose items start and end on their own, when not
// (137400 tokens: 4.57 ms, 4.64 with four).
template <int kMode, int kWaves>
__device__ __forceinline__ void attn_bf16_items(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
                                               const uint16_t* __restrict__ v, const int32_t* __restrict__ idx,
                                               const int32_t* __restrict__ cnt, uint16_t* __restrict__ out,
                                               float* __restrict__ lse, const AttnArgs& a) {
  // Four LDS half tiles of 32 rows per wave: K half 0 / 1 and V half 0 / 1 of
  // the tiles in flight. Separate objects, so the compiler sees which DMA
  // writes can alias which reads; a wave's part of each goes into its lane
  // offsets (wk.init), so reads need no more registers than with one wave.
  __shared__ __attribute__((aligned(1024))) char k0_buf[kWaves][kHalfBytes];
  __shared__ __attribute__((aligned(1024))) char k1_buf[kWaves][kHalfBytes];
  __shared__ __attribute__((aligned(1024))) char v0_buf[kWaves][kHalfBytes];
  __shared__ __attribute__((aligned(1024))) char v1_buf[kWaves][kHalfBytes];
  __shared__ float2 ml[kWaves > 1 ? kWaves : 1][kBlock];  // shared rows: (running max, row sum) of each wave
  lds_char* const kbuf0 = (lds_char*)k0_buf;
  lds_char* const kbuf1 = (lds_char*)k1_buf;
  lds_char* const vbuf0 = (lds_char*)v0_buf;
  lds_char* const vbuf1 = (lds_char*)v1_buf;

  const int wave = kWaves == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lds_off = wave * kHalfBytes;
  Work w;
  if constexpr (kWaves == 1) w = work_item(a, blockIdx.x);
  else w = work_item4(a, blockIdx.x, wave);
  if (!w.valid) return;  // a wave on its own, or all four of a shared row
  const bool shared = kWaves > 1 && w.shared;
  // (not threadIdx.x & 63: with the mask the walk spills, and its matrix and
  // VALU instructions no longer interleave, 10% slower)
  const int lane = kWaves == 1 ? threadIdx.x : __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0));
  const int l32 = lane & 31;
  const int hf = lane >> 5;
  const int nb = a.nb;
  const bool dense = kMode != kLists || a.dense[w.h] != 0;
  const int32_t* list = idx + ((int64_t)w.h * nb + w.i) * a.cap;
  // STRIDE heads: nkeys sampled keys in count virtual blocks of 64
  const int64_t stride = kMode == kStrided ? a.stride[w.h] : 1;
  const int64_t nkeys = kMode == kStrided ? (a.n + stride - 1) / stride : a.n;
  int count = kMode == kStrided ? (int)((nkeys + kBlock - 1) / kBlock) : nb;
  if (!dense) count = min(max(cnt[(int64_t)w.h * nb + w.i], 0), a.cap);
  int dense_lo = 0;  // first key block of a dense head's item
  if constexpr (kMode == kLists) {
    if (w.chunk >= 0) split_range(w, a, dense, list, count, dense_lo, lane);
  }

  // of a shared row, this wave takes every fourth list entry
  const int step_tiles = shared ? kWaves : 1;
  const int first_tile = shared ? wave : 0;
  if (shared) count = (count - wave + kWaves - 1) / kWaves;

  const int64_t head_off = (int64_t)w.h * a.n * kHeadDim;
  const uint32_t head_bytes = (uint32_t)(a.n * kHeadDim * 2);
  const __amdgpu_buffer_rsrc_t ro = make_rsrc(out + head_off, head_bytes);
  const uint16_t* const kh = k + head_off;
  const uint16_t* const vh = v + head_off;
  StrideLaneOffsets stride_off = {};
  if constexpr (kMode == kStrided) stride_off = stride_lane_offsets(lane, (uint32_t)stride);
  auto load_half = [&](bool is_v, int j, int h, lds_char* buf, DmaLaneOffsets off) {
    if constexpr (kMode == kStrided)
      dma_half_strided(is_v ? vh : kh, (uint32_t)a.n, (uint32_t)stride, j, h, buf + lds_off, stride_off);
    else
      dma_half(is_v ? vh : kh, head_bytes, nb, j, h, buf + lds_off, off);
  };

  Bf16Walk<false> wk;
  wk.init(make_rsrc(q + head_off, head_bytes), w.i, lane, a.scale_log2, lds_off);

  const DmaLaneOffsets dma_off = dma_lane_offset(lane);
  // tile of list position it, clamped to the last kept tile: loads past the
  // end of the list refetch that tile into a buffer no later step reads
  auto tile_at = [&](int it) -> int {
    const int c = first_tile + step_tiles * min(it, count - 1);
    return dense ? dense_lo + c : list[c];
  };

  if (count <= 0 && !shared) {  // an empty list: no keys, zero output, LSE -inf
    if constexpr (kMode == kLists) {
      if (w.chunk >= 0) {  // an empty key range: statistics only, the merge skips it
        float m[2];
        wk.running_max(m);
        store_partials(wk.o, m, wk.l, a, w.item, true, lane);
        return;
      }
    }
#pragma unroll
    for (int tq = 0; tq < 2; ++tq) {
      const int query = w.i * kBlock + 32 * tq + l32;
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          __builtin_amdgcn_raw_buffer_store_b64(i32x2{0, 0}, ro,
              (int)((query * kHeadDim + 32 * c + 8 * g + 4 * hf) * 2), 0, 0);
      if (lse && hf == 0 && query < a.n) lse[(int64_t)w.h * a.n + query] = kNegInf;
    }
    return;
  }

  // the last (virtual) key block may hold fewer than 64 keys
  const int last_block = kMode == kStrided ? (int)((nkeys + kBlock - 1) / kBlock) - 1 : nb - 1;
  const bool tail = (nkeys % kBlock) != 0;
  const int valid_last = (int)(nkeys - (int64_t)last_block * kBlock);

  // ---- pipeline
  // Half-tile steps t = 2j + h (tile j of the list, key half h). Step t
  // reads K half t+1 and V half t-1, then refills the buffers it read: K
  // half t+3 (same parity as t+1) and V half t+1 (parity of t-1). Every step
  // issues eight DMA loads, so at the start of a step the loads of the step
  // before last, which it reads, are done after vmcnt(8).
  f32x16 s_cur[2];
  bf16x8 p_prev[2][2];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int tq = 0; tq < 2; ++tq) p_prev[u][tq] = bf16x8{};  // P of half -1: nothing

  if (count > 0) {
  int j0 = tile_at(0), j1 = tile_at(1), j2 = tile_at(2);
  {
    // prologue: S^T of half 0, then the loads steps -2 and -1 would issue
    load_half(false, j0, 0, kbuf0, dma_off);
    __builtin_amdgcn_s_waitcnt(kWaitVm0);
    bf16x8 kA[4];
    wk.read_k(kbuf0, kA);
    wk.mfma_s(kA, s_cur);
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
    load_half(false, j0, 1, kbuf1, dma_off);   // K half 1 (tile 0)
    load_half(true, j0, 1, vbuf1, dma_off);   // V of half -1: any tile (its P is 0)
    load_half(false, j1, 0, kbuf0, dma_off);   // K half 2 (tile 1)
    load_half(true, j0, 0, vbuf0, dma_off);   // V half 0 (tile 0)
  }

  // kNext: there is a half t+1; kMask: half t may be the partial last block
  auto step = [&](auto h_c, auto next_c, auto mask_c, int jcur, int jkn, int jvn) {
    constexpr int h = decltype(h_c)::value;
    constexpr bool kNext = decltype(next_c)::value;
    constexpr bool kMask = decltype(mask_c)::value;
    lds_char* const kb = h == 0 ? kbuf1 : kbuf0;  // K half t+1
    lds_char* const vb = h == 0 ? vbuf1 : vbuf0;  // V half t-1
    __builtin_amdgcn_s_waitcnt(kWaitVm8);
    int valid = 32;
    if constexpr (kMask) {
      if (tail && jcur == last_block) valid = valid_last - 32 * h;
    }
    wk.template step<kNext>(kb, vb, valid, s_cur, p_prev);
    // refill the two buffers this step read
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
    if constexpr (kNext) {
      load_half(false, jkn, h ^ 1, kb, dma_off);
      load_half(true, jvn, h ^ 1, vb, dma_off);
    }
  };

  using F = std::false_type;
  using T = std::true_type;
  using H0 = std::integral_constant<int, 0>;
  using H1 = std::integral_constant<int, 1>;
  for (int it = 0; it + 1 < count; ++it) {
    // tiles it (j0), it+1 (j1), it+2 (j2)
    const int j3 = tile_at(it + 3);
    step(H0{}, T{}, F{}, j0, j1, j0);  // half 2it:   loads K(it+1,1), V(it,1)
    step(H1{}, T{}, F{}, j0, j2, j1);  // half 2it+1: loads K(it+2,0), V(it+1,0)
    j0 = j1;
    j1 = j2;
    j2 = j3;
  }
  // last tile: its halves may hold the partial last block
  step(H0{}, T{}, T{}, j0, j1, j0);
  __builtin_amdgcn_s_waitcnt(kWaitVm0);
  wk.last_step(vbuf0, vbuf1, tail && j0 == last_block ? valid_last - 32 : 32, s_cur, p_prev);
  }

  float lt[2], m[2];
  wk.row_sums(lt);
  wk.running_max(m);
  float* const lse_row = lse ? lse + (int64_t)w.h * a.n : nullptr;
  if (shared) {
    // the four waves' O^T (own 16 KB, the idle half tiles) and statistics meet
    // in LDS; wave 2c + tq sums and writes tile [c][tq]
    lds_char* const own[4] = {kbuf0 + lds_off, kbuf1 + lds_off, vbuf0 + lds_off, vbuf1 + lds_off};
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int tq = 0; tq < 2; ++tq)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *(lds_f32x4*)(own[2 * c + tq] + (g * 64 + lane) * 16) =
              f32x4{wk.o[c][tq][4 * g], wk.o[c][tq][4 * g + 1], wk.o[c][tq][4 * g + 2], wk.o[c][tq][4 * g + 3]};
    if (hf == 0) {
#pragma unroll
      for (int tq = 0; tq < 2; ++tq) ml[wave][32 * tq + l32] = float2{m[tq], lt[tq]};
    }
    __syncthreads();
    const int c = wave >> 1, tq = wave & 1;
    lds_char* const tile = wave == 0 ? kbuf0 : wave == 1 ? kbuf1 : wave == 2 ? vbuf0 : vbuf1;
    float2 x[kWaves];
    float mx = kNegInf, sum = 0.f;
#pragma unroll
    for (int u = 0; u < kWaves; ++u) {
      x[u] = ml[u][32 * tq + l32];
      mx = fmaxf(mx, x[u].x);
    }
#pragma unroll
    for (int u = 0; u < kWaves; ++u) {
      x[u].x = x[u].x == kNegInf ? 0.f : fast_exp2(x[u].x - mx);
      sum = fmaf(x[u].x, x[u].y, sum);
    }
    const bool part = kMode == kLists && w.chunk >= 0;  // of a split row: the merge combines the ranges
    // an empty list (no keys) gives a zero output and LSE -inf
    const float inv = sum == 0.f ? 0.f : 1.0f / sum;
    const int query = w.i * kBlock + 32 * tq + l32;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      f32x4 ov = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int u = 0; u < kWaves; ++u) {
        const f32x4 y = *(lds_f32x4*)(tile + u * kHalfBytes + (g * 64 + lane) * 16);
#pragma unroll
        for (int r = 0; r < 4; ++r) ov[r] = fmaf(x[u].x, y[r], ov[r]);
      }
      if (part) {
        *(f32x4*)(a.part_o + (int64_t)w.item * (kBlock * kHeadDim) + (((c * 2 + tq) * 4 + g) * 64 + lane) * 4) = ov;
      } else {
        bf16x4 ob;
#pragma unroll
        for (int r = 0; r < 4; ++r) ob[r] = (__bf16)(ov[r] * inv);
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(i32x2, ob), ro,
                                              (int)((query * kHeadDim + 32 * c + 8 * g + 4 * hf) * 2), 0, 0);
      }
    }
    if (c == 0 && hf == 0) {
      if (part) *(f32x2*)(a.part_ml + ((int64_t)w.item * kBlock + 32 * tq + l32) * 2) = f32x2{mx, sum};
      else if (lse_row && query < a.n) lse_row[query] = sum == 0.f ? kNegInf : (mx + __log2f(sum)) * kLn2;
    }
    return;
  }
  if constexpr (kMode == kLists) {
    if (w.chunk >= 0) {  // a split item: the merge combines the ranges
      store_partials(wk.o, m, lt, a, w.item, false, lane);
      return;
    }
  }
  const float inv[2] = {1.0f / lt[0], 1.0f / lt[1]};
  const float lse_val[2] = {(m[0] + __log2f(lt[0])) * kLn2, (m[1] + __log2f(lt[1])) * kLn2};
  write_out_tile(wk.o, inv, lse_val, kbuf0 + lds_off, kbuf1 + lds_off, ro, lse_row, w.i, a.n, lane);
}

template <int kMode>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_bf16_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const int32_t* __restrict__ idx, const int32_t* __restrict__ cnt, uint16_t* __restrict__ out,
    float* __restrict__ lse, AttnArgs a) {
  attn_bf16_items<kMode, 1>(q, k, v, idx, cnt, out, lse, a);
}

template <int kMode>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_bf16_rows4_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const int32_t* __restrict__ idx, const int32_t* __restrict__ cnt, uint16_t* __restrict__ out,
    float* __restrict__ lse, AttnArgs a) {
  attn_bf16_items<kMode, 4>(q, k, v, idx, cnt, out, lse, a);
}

// ---- every head dense: kDenseWaves waves per workgroup sharing the K / V tiles
//
// A workgroup takes kDenseWaves neighbouring query blocks of one head, and
// since every one of them walks every key block in order, each K and V half
// tile is staged in LDS once for all of them. Wave w owns query block
// kDenseWaves * group + w; a block past the head's last one runs the last
// block again and stores nothing, so every wave meets every barrier. The K and
// V half tiles go into a ring of four LDS buffers per tensor (K half x in
// kring[x % 4], V half x in vring[x % 4]). Step t reads K half t+1 and V half
// t-1; right after the step's barrier the waves refill the buffers step t-1
// read (K half t+4, V half t+2), each wave issuing its share of the eight 1 KB
// DMA instructions, three steps before those buffers are read. Before the
// barrier each wave waits for its own loads of three steps back, so after it
// every wave's loads for the step have landed, and every wave has finished
// the reads of step t-1.
constexpr int kDenseWaves = 4;

// Group g (rows 8g .. 8g+7) of the 32-row half h of block j into buf: one 1 KB
// DMA instruction. The descriptor starts at the group and extends over what
// is left of the head, so rows past the head, and any j outside [0, nb),
// read zeros.
__device__ inline void dma_group(const uint16_t* head, uint32_t head_bytes, int nb, int j, int h,
                                 int g, lds_char* buf, int lane_off) {
  const uint32_t t = __builtin_amdgcn_readfirstlane(
      (uint32_t)j < (uint32_t)nb ? ((uint32_t)j * kBlock + 32u * h + 8u * g) * (kHeadDim * 2)
                                 : head_bytes);
  const uint32_t rem = rem_bytes(head_bytes, t);
  const __amdgpu_buffer_rsrc_t r = make_rsrc(reinterpret_cast<const char*>(head) + t, rem);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)(buf + 1024 * g), 16, lane_off, 0, 0, 0);
}

__global__ __launch_bounds__(64 * kDenseWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_bf16_dense_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    uint16_t* __restrict__ out, float* __restrict__ lse, AttnArgs a) {
  __shared__ __attribute__((aligned(1024))) char kr0[32 * 128];
  __shared__ __attribute__((aligned(1024))) char kr1[32 * 128];
  __shared__ __attribute__((aligned(1024))) char kr2[32 * 128];
  __shared__ __attribute__((aligned(1024))) char kr3[32 * 128];
  __shared__ __attribute__((aligned(1024))) char vr0[32 * 128];
  __shared__ __attribute__((aligned(1024))) char vr1[32 * 128];
  __shared__ __attribute__((aligned(1024))) char vr2[32 * 128];
  __shared__ __attribute__((aligned(1024))) char vr3[32 * 128];
  lds_char* const kring[4] = {(lds_char*)kr0, (lds_char*)kr1, (lds_char*)kr2, (lds_char*)kr3};
  lds_char* const vring[4] = {(lds_char*)vr0, (lds_char*)vr1, (lds_char*)vr2, (lds_char*)vr3};
  constexpr int kW = kDenseWaves;

  // workgroup b runs on XCD b % 8; each XCD takes a contiguous run of the
  // (head, group) units, so the workgroups it runs at once walk one head
  const int nb = a.nb;
  const int groups = (nb + kW - 1) / kW;
  const int total = a.heads * groups;
  const int per_xcd = (total + 7) / 8;
  const int unit = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (unit >= total) return;  // the whole workgroup
  const int hpos = unit / groups;
  const int hidx = a.order[hpos];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int l32 = lane & 31;
  const int hf = lane >> 5;
  const int i_own = (unit - hpos * groups) * kW + wave;
  const bool valid_block = i_own < nb;

  const int64_t head_off = (int64_t)hidx * a.n * kHeadDim;
  const uint32_t head_bytes = (uint32_t)(a.n * kHeadDim * 2);
  const uint16_t* const kh = k + head_off;
  const uint16_t* const vh = v + head_off;

  Bf16Walk<true> wk;
  wk.init(make_rsrc(q + head_off, head_bytes), valid_block ? i_own : nb - 1, lane, a.scale_log2);

  // this wave's share of a step's eight DMA instructions n = wave, wave + kW,
  // ... (n < 4: K group n, else V group n - 4); its group is wave % 4 either way
  const DmaLaneOffsets dma_off = dma_lane_offset(lane);
  const int dma_g = wave & 3;
  const int dma_lane = (dma_g & 1) ? dma_off.odd : dma_off.even;
  auto issue = [&](int jk, int hk, lds_char* kb, int jv, int hv, lds_char* vb) {
#pragma unroll
    for (int n0 = 0; n0 < 8; n0 += kW) {
      if (n0 + wave < 4) dma_group(kh, head_bytes, nb, jk, hk, dma_g, kb, dma_lane);
      else dma_group(vh, head_bytes, nb, jv, hv, dma_g, vb, dma_lane);
    }
  };
  // this wave's loads up to `pending` instructions back have landed and its
  // LDS reads are done; then the workgroup meets (the asm's memory clobber
  // keeps LDS accesses on their side of the barrier)
  auto sync = [&](auto pending_c) {
    constexpr int pending = decltype(pending_c)::value;
    __builtin_amdgcn_s_waitcnt((0x0F70 | pending) & kWaitLgkm0);
    asm volatile("s_barrier" ::: "memory");
  };
  constexpr int kPending = 2 * (8 / kW);  // two steps of this wave's loads

  const bool tail = (a.n % kBlock) != 0;
  const int valid_last = (int)(a.n - (int64_t)(nb - 1) * kBlock);

  f32x16 s_cur[2];
  bf16x8 p_prev[2][2];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int tq = 0; tq < 2; ++tq) p_prev[u][tq] = bf16x8{};  // P of half -1: nothing

  // prologue: K halves 0-3 into kring[0..3]; V half -1 (any data, its P is 0:
  // V half 1) into vring[3], V halves 0 and 1 into vring[0] and vring[1]
  issue(0, 0, kring[0], 0, 1, vring[3]);
  issue(0, 1, kring[1], 0, 0, vring[0]);
  issue(1, 0, kring[2], 0, 1, vring[1]);
  issue(1, 1, kring[3], 0, 1, vring[1]);
  sync(std::integral_constant<int, 0>{});
  {
    bf16x8 kA[4];
    wk.read_k(kring[0], kA);
    wk.mfma_s(kA, s_cur);
  }

  // step t = 2j + h with P = t % 4 (the ring slots are then fixed)
  auto step = [&](auto p_c, auto mask_c, int j) {
    constexpr int P = decltype(p_c)::value;
    constexpr int h = P & 1;
    constexpr bool kMask = decltype(mask_c)::value;
    sync(std::integral_constant<int, kPending>{});
    // refill what step t-1 read: K half t+4 (block j+2, half h), V half t+2 (block j+1, half h)
    issue(j + 2, h, kring[P], j + 1, h, vring[(P + 2) & 3]);
    const int valid = kMask && tail ? valid_last - 32 * h : 32;
    wk.template step<true>(kring[(P + 1) & 3], vring[(P + 3) & 3], valid, s_cur, p_prev);
  };
  // the last step t = 2nb - 1, P = t % 4
  auto last = [&](auto p_c) {
    constexpr int P = decltype(p_c)::value;
    sync(std::integral_constant<int, 0>{});
    wk.last_step(vring[(P + 3) & 3], vring[P], tail ? valid_last - 32 : 32, s_cur, p_prev);
  };

  using F = std::false_type;
  using T = std::true_type;
  using P0 = std::integral_constant<int, 0>;
  using P1 = std::integral_constant<int, 1>;
  using P2 = std::integral_constant<int, 2>;
  using P3 = std::integral_constant<int, 3>;
  int it = 0;  // tiles it and it + 1 per iteration, it even
  for (; it + 2 < nb; it += 2) {
    step(P0{}, F{}, it);
    step(P1{}, F{}, it);
    step(P2{}, F{}, it + 1);
    step(P3{}, F{}, it + 1);
  }
  if (nb - it == 2) {
    step(P0{}, F{}, it);
    step(P1{}, F{}, it);
    step(P2{}, T{}, it + 1);
    last(P3{});
  } else {
    step(P0{}, T{}, it);
    last(P1{});
  }

  if (!valid_block) return;
  float lt[2];
  wk.row_sums(lt);
  const __amdgpu_buffer_rsrc_t ro = make_rsrc(out + head_off, head_bytes);
  float* const lse_row = lse ? lse + (int64_t)hidx * a.n : nullptr;
  // straight from the registers: 8-byte stores, once per walk of nb blocks
#pragma unroll
  for (int tq = 0; tq < 2; ++tq) {
    const int query = i_own * kBlock + 32 * tq + l32;
    const float inv = 1.0f / lt[tq];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        bf16x4 ov;
#pragma unroll
        for (int r = 0; r < 4; ++r) ov[r] = (__bf16)(wk.o[c][tq][4 * g + r] * inv);
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(i32x2, ov), ro,
                                              (int)((query * kHeadDim + 32 * c + 8 * g + 4 * hf) * 2), 0, 0);
      }
    if (lse_row && hf == 0 && query < a.n) lse_row[query] = (__log2f(lt[tq]) - wk.nm[tq]) * kLn2;
  }
}

// Combines the key ranges of split heads: per query, M = max of the ranges'
// running maxima, weights 2^(m_c - M), O = sum_c w_c O_c / sum_c w_c l_c, in
// range order; rows written in the layer's dtype. One wave per (split head,
// query block).
template <bool kBf16>
__global__ __launch_bounds__(64) void attn_merge_kernel(const float* __restrict__ part_o,
                                                       const float* __restrict__ part_ml,
                                                       void* __restrict__ out,
                                                       float* __restrict__ lse, MergeArgs a) {
  __shared__ __attribute__((aligned(1024))) char b0[32 * 128];
  __shared__ __attribute__((aligned(1024))) char b1[32 * 128];
  const int sp = blockIdx.x / a.nb;
  const int i = blockIdx.x - sp * a.nb;
  if (sp >= a.n_split) return;
  const int h = a.head[sp];
  const int lane = threadIdx.x;
  const int l32 = lane & 31;
  auto ml_at = [&](int c, int tq) -> f32x2 {
    const int64_t item = (int64_t)(sp * a.splits + c) * a.nb + i;
    return *(const f32x2*)(part_ml + (item * kBlock + 32 * tq + l32) * 2);
  };
  float mx[2] = {kNegInf, kNegInf};
  for (int c = 0; c < a.splits; ++c)
#pragma unroll
    for (int tq = 0; tq < 2; ++tq) mx[tq] = fmaxf(mx[tq], ml_at(c, tq)[0]);
  float lt[2] = {0.f, 0.f};
  f32x16 o[2][2];
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int tq = 0; tq < 2; ++tq)
#pragma unroll
      for (int e = 0; e < 16; ++e) o[c][tq][e] = 0.f;
  for (int c = 0; c < a.splits; ++c) {
    float wgt[2];
#pragma unroll
    for (int tq = 0; tq < 2; ++tq) {
      const f32x2 ml = ml_at(c, tq);
      wgt[tq] = ml[0] == kNegInf ? 0.f : fast_exp2(ml[0] - mx[tq]);
      lt[tq] = fmaf(wgt[tq], ml[1], lt[tq]);
    }
    // an empty range (every query's max is -inf) wrote no accumulators
    if (!__ballot(wgt[0] != 0.f || wgt[1] != 0.f)) continue;
    const float* const po = part_o + ((int64_t)(sp * a.splits + c) * a.nb + i) * (kBlock * kHeadDim);
#pragma unroll
    for (int c2 = 0; c2 < 2; ++c2)
#pragma unroll
      for (int tq = 0; tq < 2; ++tq)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x4 val = *(const f32x4*)(po + (((c2 * 2 + tq) * 4 + g) * 64 + lane) * 4);
#pragma unroll
          for (int r = 0; r < 4; ++r) o[c2][tq][4 * g + r] = fmaf(wgt[tq], val[r], o[c2][tq][4 * g + r]);
        }
  }
  float inv[2], lse_val[2];
#pragma unroll
  for (int tq = 0; tq < 2; ++tq) {
    inv[tq] = lt[tq] > 0.f ? 1.0f / lt[tq] : 0.f;
    lse_val[tq] = lt[tq] > 0.f ? (mx[tq] + __log2f(lt[tq])) * kLn2 : kNegInf;
  }
  const int64_t head_off = (int64_t)h * a.n * kHeadDim;
  float* const lse_row = lse ? lse + (int64_t)h * a.n : nullptr;
  if constexpr (kBf16) {
    const __amdgpu_buffer_rsrc_t ro =
        make_rsrc(static_cast<uint16_t*>(out) + head_off, (uint32_t)(a.n * kHeadDim * 2));
    write_out_tile(o, inv, lse_val, (lds_char*)b0, (lds_char*)b1, ro, lse_row, i, a.n, lane);
  } else {
    const __amdgpu_buffer_rsrc_t ro =
        make_rsrc(static_cast<float*>(out) + head_off, (uint32_t)(a.n * kHeadDim * 4));
    write_out_tile_f32(o, inv, lse_val, ro, lse_row, i, a.n, lane);
  }
}

// ------------------------------------------------------------------ fp32

// fp32 inputs on the bf16 matrix cores, at fp32 accuracy. Every operand x is
// taken as three bf16 values, hi = bf16(x), mid = bf16(x - hi) and lo =
// x - hi - mid, which hold its 24 bits exactly and have fp32's exponent range,
// so there is no scale and no range to leave; a product is hi hi + hi mid +
// mid hi + mid mid + hi lo + lo hi, six matrix instructions with fp32
// accumulation (the dropped mid lo, lo mid and lo lo are at most 2^-25 of it
// together, below the rounding of one fp32 addition). The weights P are split
// the same way, and the row sum adds the fp32 weights.
//
// Not exact in that form: values whose parts fall below bf16's normal range
// (|x| < 2^-102: up to 2^-126 of them is lost), and those at the top that
// round to an infinity. So a workgroup with a Q value in 0 < |q| < 2^-100 or
// from 2^90 on, and a wave whose O or row sum is not finite at the end or
// whose outputs are not 0 but below 2^-100 (all that V's lost parts could
// matter to: with Q below 2^90, K's move no score by more than 2^-33), walks
// its half tiles once more on the fp32 matrix instructions
// (v_mfma_f32_32x32x2_f32) and the values as they are. So do walks over
// infinite or NaN inputs. Weights below 2^-102 of the largest keep an absolute
// 2^-126 of it.
//
// A workgroup of four waves owns one (head, 64-query block) or one key range
// of it. Wave w walks the half tiles w, w + 4, ... of the list with its own
// running max, row sum and O^T, and the four are combined through LDS at the
// end, so an item is a quarter as long as with one wave and needs no
// workspace to be. Split Q^T (the same for all four) sits in LDS in operand
// order, its hi part in registers too. Each wave's K half tile comes by the
// direct buffer-to-LDS load: read straight into the operand layout, a K load
// would touch 32 rows per instruction, and the L1's tag lookups would be the
// bound. A lane's V column (the A operand of O^T = V^T P^T) is contiguous
// across lanes as it stands and goes straight to registers.
//
// Bound by the matrix cores (a half tile: 96 matrix instructions, 3072 cycles)
// beside VALU issue (most of it the splits of K, V and P). Every head dense at
// 10992 tokens, 16 heads: 5.02 ms (99 TFLOP/s) with one wave per item on the
// fp32 matrix instructions, 2.45 ms (202 TFLOP/s) so, relative error against 64
// bits 1.5e-6 before, 4.9e-7 now; with every walk made twice, 5.7 ms. (Pairs of
// scaled f16 values, three products, take 1.5 ms, but hold a value to an
// absolute 2^-35 of the largest that shares its scale, and weights likewise.)
struct SplitBf16 {
  bf16x8 part[3];  // hi, mid, lo
};
// The empty asm keeps the compiler from converting each half of a packed pair
// once more on its own.
__device__ __forceinline__ SplitBf16 split_bf16(const float (&x)[8]) {
  SplitBf16 r;
#pragma unroll
  for (int e = 0; e < 8; e += 2) {
    f32x2 rest = {x[e], x[e + 1]};
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      uint32_t b = __builtin_bit_cast(uint32_t, __builtin_convertvector(rest, bf16x2));
      asm("" : "+v"(b));
      const bf16x2 y = __builtin_bit_cast(bf16x2, b);
      r.part[t][e] = y[0];
      r.part[t][e + 1] = y[1];
      if (t < 2) rest = f32x2{rest[0] - __uint_as_float(b << 16), rest[1] - __uint_as_float(b & 0xffff0000u)};
    }
  }
  return r;
}
// The six products by the parts of their factors, the smallest first.
constexpr int kProducts = 6;
constexpr int kPartA[kProducts] = {2, 0, 1, 1, 0, 0};
constexpr int kPartB[kProducts] = {0, 2, 1, 0, 1, 0};

// A descriptor over rows [tok, n) of a head of 256-byte fp32 rows (empty for tok outside [0, n)).
__device__ inline __amdgpu_buffer_rsrc_t rows_from(const float* head, uint32_t tok, uint32_t n) {
  const uint32_t t = tok < n ? tok : n;
  return make_rsrc(head + (size_t)t * kHeadDim, (n - t) * (kHeadDim * 4));
}

// Sixteen 256-byte rows into LDS by four buffer-to-LDS loads, lane offsets
// off[g]. With kRows the immediate offset takes instruction g four rows (1 KB)
// on in memory and in LDS; otherwise off[g] holds the whole memory offset.
template <bool kRows>
__device__ __forceinline__ void dma_rows16(__amdgpu_buffer_rsrc_t r, lds_char* b, const int (&off)[4]) {
  if constexpr (kRows) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)b, 16, off[0], 0, 0, 0);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)b, 16, off[1], 0, 1024, 0);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)b, 16, off[2], 0, 2048, 0);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)b, 16, off[3], 0, 3072, 0);
  } else {
#pragma unroll
    for (int g = 0; g < 4; ++g)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)(b + 1024 * g), 16, off[g], 0, 0, 0);
  }
}

constexpr int kF32Waves = 4;

template <int kMode>
__global__ __launch_bounds__(64 * kF32Waves) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
    const int32_t* __restrict__ idx, const int32_t* __restrict__ cnt, float* __restrict__ out,
    float* __restrict__ lse, AttnArgs a) {
  // split Q^T in B-operand order: [hi, mid, lo][dims 16s ..][query half][lane] 16 bytes
  __shared__ __attribute__((aligned(16))) bf16x8 qs[3][4][2][64];
  __shared__ int q_odd[kF32Waves];  // a wave's part of Q leaves the split form's range
  // per wave a K half tile: 32 rows of 256 B, 16-byte chunk c of row r at slot
  // c ^ (r & 15), which spreads a chunk's reads over the banks
  __shared__ __attribute__((aligned(1024))) char kbuf[kF32Waves][32 * 256];

  const Work w = work_item(a, blockIdx.x);
  if (!w.valid) return;  // the whole workgroup
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31;
  const int hf = lane >> 5;
  const int nb = a.nb;
  const bool dense = kMode != kLists || a.dense[w.h] != 0;
  const int32_t* list = idx + ((int64_t)w.h * nb + w.i) * a.cap;
  const uint32_t n = (uint32_t)a.n;  // at most 2^20, and so is a stride
  const uint32_t stride = kMode == kStrided ? (uint32_t)a.stride[w.h] : 1u;
  const int nkeys = (int)(kMode == kStrided ? (n + stride - 1) / stride : n);
  int count = kMode == kStrided ? (nkeys + kBlock - 1) / kBlock : nb;
  if (!dense) count = min(max(cnt[(int64_t)w.h * nb + w.i], 0), a.cap);
  int dense_lo = 0;  // first key block of a dense head's item
  if constexpr (kMode == kLists) {
    if (w.chunk >= 0) split_range(w, a, dense, list, count, dense_lo, lane);
  }
  const int last_block = kMode == kStrided ? count - 1 : nb - 1;
  const int blocks = kMode == kStrided ? count : nb;

  const int64_t head_off = (int64_t)w.h * a.n * kHeadDim;
  const uint32_t head_bytes = n * kHeadDim * 4;
  const float* const kh = k + head_off;
  const float* const vh = v + head_off;
  const __amdgpu_buffer_rsrc_t rq = make_rsrc(q + head_off, head_bytes);

  // Q: wave s splits dims 16s ..; lane (l32, hf) dims 16s + 8hf .. of queries l32 and 32 + l32
  {
    uint32_t large = 0, small = ~0u;  // largest and smallest nonzero magnitude, as bits << 1
#pragma unroll
    for (int tq = 0; tq < 2; ++tq) {
      float x[8];
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const f32x4 y = __builtin_bit_cast(
            f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                       rq, ((w.i * kBlock + 32 * tq + l32) * kHeadDim + 16 * wave + 8 * hf + 4 * c) * 4, 0, 0));
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          x[4 * c + e] = y[e];
          const uint32_t mag = __float_as_uint(y[e]) << 1;
          large = max(large, mag);
          small = min(small, mag - 1);  // 0 wraps to the largest
        }
      }
      const SplitBf16 p = split_bf16(x);
#pragma unroll
      for (int t = 0; t < 3; ++t) qs[t][wave][tq][lane] = p.part[t];
    }
    const bool odd = large >= (127u + 90) << 24 || small < ((127u - 100) << 24) - 1;
    const bool any_odd = __ballot(odd) != 0;
    if (lane == 0) q_odd[wave] = any_odd ? 1 : 0;
  }

  f32x16 o[2][2];
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int tq = 0; tq < 2; ++tq)
#pragma unroll
      for (int e = 0; e < 16; ++e) o[c][tq][e] = 0.f;
  float nm[2] = {-kNegInf, -kNegInf};  // minus the running max of the log2-scaled scores
  float l[2] = {0.f, 0.f};
  const bool tail = (nkeys % kBlock) != 0;
  const float sc = a.scale_log2;

  // This wave's half tiles: half h = wave & 1 of list entries wave / 2, wave / 2 + 2, ...
  const int h = wave & 1;
  auto block_at = [&](int it) -> int {
    const int c = min(it, count - 1);
    return __builtin_amdgcn_readfirstlane(dense ? dense_lo + c : list[c]);
  };
  auto first_token = [&](int j) -> uint32_t {
    return (uint32_t)j < (uint32_t)blocks ? ((uint32_t)j * kBlock + 32 * h) * stride : n;
  };
  // byte offset of key row r of a half tile; a strided row past the head stays past it
  auto row_off = [&](int r) -> int {
    return kMode == kStrided ? (int)(min((uint32_t)r * stride, 1u << 22) * (kHeadDim * 4)) : r * (kHeadDim * 4);
  };
  // K by DMA: instruction g fills rows 4g .. 4g + 3, lane l its 16 bytes at
  // 16 l: row 4g + l / 16, slot l % 16, which holds chunk (l % 16) ^ (row % 16)
  lds_char* const kb = (lds_char*)kbuf[wave];
  int k_dma[4];  // by g % 4; 16 rows further on the chunks repeat
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int r = 4 * g + (lane >> 4);
    k_dma[g] = (kMode == kStrided ? 0 : (lane >> 4) * (kHeadDim * 4)) + (((lane & 15) ^ r) << 4);
  }
  auto load_k = [&](int j) {
    const uint32_t tok = first_token(j);
#pragma unroll
    for (int u = 0; u < 2; ++u) {  // rows 16u .. 16u + 15
      int off[4];
#pragma unroll
      for (int g = 0; g < 4; ++g) off[g] = k_dma[g] + (kMode == kStrided ? row_off(4 * g + (lane >> 4)) : 0);
      dma_rows16<kMode != kStrided>(rows_from(kh, tok + 16 * u * stride, n), kb + 4096 * u, off);
    }
    __builtin_amdgcn_sched_barrier(0);  // before the V loads that the wait below counts
  };
  // V column 32c + l32 at the keys of P's registers, 16u + 8b + 4hf + r
  // (a descriptor per u, so that the rest of an offset fits the instruction)
  // (each call's own copy, so that no sum of it is hoisted into a register)
  int v_off = 4 * hf * (kHeadDim * 4) + 4 * l32;
  auto load_v = [&](int j, int u, float (&x)[2][8]) {
    asm volatile("" : "+v"(v_off));
    const __amdgpu_buffer_rsrc_t r = rows_from(vh, first_token(j) + 16 * u * stride, n);
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int c = 0; c < 2; ++c)
        x[c][e] = __uint_as_float((uint32_t)__builtin_amdgcn_raw_buffer_load_b32(
            r,
            kMode == kStrided ? row_off(8 * (e >> 2) + (e & 3) + 4 * hf) + 4 * l32 + 128 * c
                              : v_off + (8 * (e >> 2) + (e & 3)) * (kHeadDim * 4) + 128 * c,
            0, 0));
  };

  float vx[2][2][8];
  int j = 0, jn = 0;  // key block of this step and of the next
  int it = wave >> 1;
  if (it < count) {
    j = block_at(it);
    jn = block_at(it + 2);
    load_k(j);
#pragma unroll
    for (int u = 0; u < 2; ++u) load_v(j, u, vx[u]);
  }
  __syncthreads();  // Q's parts of all waves
  const bool odd = __builtin_amdgcn_readfirstlane(q_odd[0] | q_odd[1] | q_odd[2] | q_odd[3]) != 0;
  // K of this step from LDS: row l32, dims 16s + 8hf + (0..7). Its loads have
  // landed when only the 32 V loads issued after them are in flight.
  auto read_k = [&](float (&x)[4][8]) {
    asm volatile("s_waitcnt vmcnt(32)" ::: "memory");
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const f32x4 y = *(lds_f32x4*)(kb + 256 * l32 + (((4 * s + 2 * hf + c) ^ (l32 & 15)) << 4));
#pragma unroll
        for (int e = 0; e < 4; ++e) x[s][4 * c + e] = y[e];
      }
  };
  bf16x8 qh[2][4];
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int tq = 0; tq < 2; ++tq) qh[tq][s] = qs[0][s][tq][lane];
  int q_pos = lane;
  for (; it < count && !odd; it += 2) {
    const int j2 = block_at(it + 4);
    // ---- S^T = K Q^T
    f32x16 s_acc[2] = {};
    {
      float kx[4][8];
      read_k(kx);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // read: the buffer may be filled again
      load_k(jn);
      // the small products of all 64 dims first: the sum then rounds at its
      // full size in the four hi hi instructions alone
      bf16x8 kh[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const SplitBf16 kp = split_bf16(kx[s]);
        kh[s] = kp.part[0];
        // read again in every half tile: hoisted, they would take 64 registers more
        asm volatile("" : "+v"(q_pos));
        const bf16x8 qp[3][2] = {{qh[0][s], qh[1][s]},
                                 {qs[1][s][0][q_pos], qs[1][s][1][q_pos]},
                                 {qs[2][s][0][q_pos], qs[2][s][1][q_pos]}};
#pragma unroll
        for (int t = 0; t + 1 < kProducts; ++t)
#pragma unroll
          for (int tq = 0; tq < 2; ++tq)
            s_acc[tq] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kp.part[kPartA[t]], qp[kPartB[t]][tq], s_acc[tq], 0, 0, 0);
      }
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int tq = 0; tq < 2; ++tq)
          s_acc[tq] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kh[s], qh[tq][s], s_acc[tq], 0, 0, 0);
    }
    float add[2] = {nm[0], nm[1]};
    if (tail && j == last_block) {
      asm volatile("");  // a branch, not 32 selects in every half tile
      const int valid = nkeys - j * kBlock - 32 * h;
      if (valid <= 0) {  // no key at all (its rows read as zeros): P = 0 and the max stays
        add[0] = add[1] = kNegInf;
      } else {
#pragma unroll
        for (int e = 0; e < 16; ++e)
          if (8 * (e >> 2) + 4 * hf + (e & 3) >= valid) s_acc[0][e] = s_acc[1][e] = kNegInf;
      }
    }

    // ---- online softmax
    float p[2][2][8];
    float rs[2];
    auto probs = [&]() {
#pragma unroll
      for (int tq = 0; tq < 2; ++tq) {
        rs[tq] = 0.f;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          p[e >> 3][tq][e & 7] = fast_exp2(fmaf(s_acc[tq][e], sc, add[tq]));
          rs[tq] += p[e >> 3][tq][e & 7];
        }
      }
    };
    probs();
    // a lane's share above 2^12 (as unsigned bits, so also inf and NaN): the max moves
    if (__ballot(__float_as_uint(rs[0]) > 0x45800000u || __float_as_uint(rs[1]) > 0x45800000u)) {
#pragma unroll
      for (int tq = 0; tq < 2; ++tq) {
        float mx = s_acc[tq][0];
#pragma unroll
        for (int e = 1; e < 16; ++e) mx = fmaxf(mx, s_acc[tq][e]);
        const float nmnew = fminf(-(pair_max(mx) * sc), nm[tq]);
        const float alpha = fast_exp2(nmnew - nm[tq]);
        nm[tq] = add[tq] = nmnew;
        l[tq] *= alpha;
#pragma unroll
        for (int c = 0; c < 2; ++c) o[c][tq] *= alpha;
      }
      probs();
    }
    l[0] += rs[0];
    l[1] += rs[1];

    // ---- O^T += V^T P^T
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const SplitBf16 vp[2] = {split_bf16(vx[u][0]), split_bf16(vx[u][1])};
      load_v(jn, u, vx[u]);
      const SplitBf16 pp[2] = {split_bf16(p[u][0]), split_bf16(p[u][1])};
#pragma unroll
      for (int t = 0; t < kProducts; ++t)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
          for (int tq = 0; tq < 2; ++tq)
            o[c][tq] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vp[c].part[kPartA[t]], pp[tq].part[kPartB[t]], o[c][tq],
                                                               0, 0, 0);
    }
    j = jn;
    jn = j2;
  }

  // ---- outside the split form (see above): once more on the fp32 matrix instructions
  float bad = l[0] * 0.f + l[1] * 0.f;
  uint32_t small[2] = {~0u, ~0u};  // smallest nonzero |O| of the lane's queries, as bits << 1, less 1
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        bad = fmaf(o[c][t][e], 0.f, bad);
        small[t] = min(small[t], (__float_as_uint(o[c][t][e]) << 1) - 1);
      }
  bool again = odd || bad != 0.f;
#pragma unroll
  for (int t = 0; t < 2; ++t)  // |O| / l < 2^-100, l the whole row sum of this wave
    again = again || small[t] < __float_as_uint(pair_sum(l[t]) * 0x1p-100f) << 1;
  if (__ballot(again)) {
    __builtin_amdgcn_s_waitcnt(kWaitVm0);
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int t = 0; t < 2; ++t) o[c][t] = f32x16{};
    float m[2] = {kNegInf, kNegInf};
    l[0] = l[1] = 0.f;
    for (it = wave >> 1; it < count; it += 2) {
      j = block_at(it);
      const int valid = min(nkeys - j * kBlock - 32 * h, 32);
      if (j == last_block && valid <= 0) continue;
      const __amdgpu_buffer_rsrc_t rk = rows_from(kh, first_token(j), n);
      f32x16 s_acc[2] = {};
#pragma unroll 1
      for (int d = 0; d < kHeadDim; d += 4) {  // k-steps of 2 dims: d + hf, then d + 2 + hf
        const f32x4 x = __builtin_bit_cast(
            f32x4, __builtin_amdgcn_raw_buffer_load_b128(rk, row_off(l32) + 4 * d, 0, 0));
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const f32x4 y = __builtin_bit_cast(
              f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                         rq, ((w.i * kBlock + 32 * t + l32) * kHeadDim + d) * 4, 0, 0));
          s_acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(hf ? x[1] : x[0], hf ? y[1] : y[0], s_acc[t], 0, 0, 0);
          s_acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(hf ? x[3] : x[2], hf ? y[3] : y[2], s_acc[t], 0, 0, 0);
        }
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) load_v(j, u, vx[u]);
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        float mx = kNegInf;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          if (j == last_block && 8 * (e >> 2) + 4 * hf + (e & 3) >= valid) s_acc[t][e] = kNegInf;
          mx = fmaxf(mx, s_acc[t][e]);
        }
        const float mnew = fmaxf(m[t], pair_max(mx) * sc);
        const float alpha = fast_exp2(m[t] - mnew);
        m[t] = mnew;
        l[t] *= alpha;
#pragma unroll
        for (int c = 0; c < 2; ++c) o[c][t] *= alpha;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          s_acc[t][e] = fast_exp2(fmaf(s_acc[t][e], sc, -mnew));
          l[t] += s_acc[t][e];
        }
      }
      // k-step e pairs key 8 (e / 4) + e % 4 (lane half 0) with the one 4 further on (lane half 1)
#pragma unroll
      for (int e = 0; e < 16; ++e)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
          for (int t = 0; t < 2; ++t)
            o[c][t] = __builtin_amdgcn_mfma_f32_32x32x2f32(vx[e >> 3][c][e & 7], s_acc[t][e], o[c][t], 0, 0, 0);
    }
    nm[0] = -m[0];
    nm[1] = -m[1];
  }

  // ---- the four waves' parts: weights 2^(m_w - M) on O^T, through LDS:
  // (running max, row sum) per wave and query into Q's array, O^T in two
  // rounds (head-dim halves) into the K buffers, 8 KB a wave
  const float lt[2] = {pair_sum(l[0]), pair_sum(l[1])};
  __builtin_amdgcn_s_waitcnt(kWaitVm0);  // the last prefetch into the K buffer
  __syncthreads();                       // every wave is done with Q
  f32x2* const ml = (f32x2*)qs;          // [wave][64] (max, sum)
  if (hf == 0) {
#pragma unroll
    for (int tq = 0; tq < 2; ++tq) ml[wave * 64 + 32 * tq + l32] = f32x2{-nm[tq], lt[tq]};
  }
  // this wave sums query half tq, 16-byte groups g2, g2 + 1 of the registers
  const int tq = wave & 1, g2 = 2 * (wave >> 1);
  float m = kNegInf, sum = 0.f, inv = 1.0f, f[kF32Waves];
  const int query = w.i * kBlock + 32 * tq + l32;
  const __amdgpu_buffer_rsrc_t ro = make_rsrc(out + head_off, head_bytes);
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    if (c) __syncthreads();  // the first round's reads
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *(lds_f32x4*)(kb + ((t * 4 + g) * 64 + lane) * 16) =
            f32x4{o[c][t][4 * g], o[c][t][4 * g + 1], o[c][t][4 * g + 2], o[c][t][4 * g + 3]};
    __syncthreads();
    if (c == 0) {
      f32x2 x[kF32Waves];
#pragma unroll
      for (int u = 0; u < kF32Waves; ++u) {
        x[u] = ml[u * 64 + 32 * tq + l32];
        m = fmaxf(m, x[u][0]);
      }
#pragma unroll
      for (int u = 0; u < kF32Waves; ++u) {
        f[u] = x[u][0] == kNegInf ? 0.f : fast_exp2(x[u][0] - m);
        sum = fmaf(f[u], x[u][1], sum);
      }
      const bool part = kMode == kLists && w.chunk >= 0;  // a split item: the merge combines the ranges
      // an empty list (no keys) gives a zero output and LSE -inf
      if (!part) inv = sum > 0.f ? 1.0f / sum : 0.f;
      if (g2 == 0 && hf == 0) {
        if (part)
          *(f32x2*)(a.part_ml + ((int64_t)w.item * kBlock + 32 * tq + l32) * 2) = f32x2{m, sum};
        else if (lse && query < (int)n)
          lse[(int64_t)w.h * a.n + query] = sum > 0.f ? (m + log2f(sum)) * kLn2 : kNegInf;
      }
    }
#pragma unroll
    for (int g = g2; g < g2 + 2; ++g) {
      f32x4 ov = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int u = 0; u < kF32Waves; ++u) {
        const f32x4 y = *(lds_f32x4*)((lds_char*)kbuf[u] + ((tq * 4 + g) * 64 + lane) * 16);
#pragma unroll
        for (int r = 0; r < 4; ++r) ov[r] = fmaf(f[u], y[r], ov[r]);
      }
      if (kMode == kLists && w.chunk >= 0)
        *(f32x4*)(a.part_o + (int64_t)w.item * (kBlock * kHeadDim) + (((c * 2 + tq) * 4 + g) * 64 + lane) * 4) = ov;
      else
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(i32x4, ov * inv), ro,
                                               (query * kHeadDim + 32 * c + 8 * g + 4 * hf) * 4, 0, 0);
    }
  }
}

}  // namespace

hipError_t launch_attention(int dtype, const void* q, const void* k, const void* v,
                            const int32_t* idx, const int32_t* cnt, void* out, float* lse,
                            const AttnArgs& a, hipStream_t s) {
  const int64_t groups = 8LL * a.unit_start[a.heads];
  if (groups == 0) return hipSuccess;
  const dim3 grid((unsigned)groups);
  if (dtype == 1) {
    if (a.mode == kAllDense) {
      const int64_t units = (int64_t)a.heads * ((a.nb + kDenseWaves - 1) / kDenseWaves);
      hipLaunchKernelGGL(attn_bf16_dense_kernel, dim3((unsigned)(8 * ((units + 7) / 8))),
                         dim3(64 * kDenseWaves), 0, s, static_cast<const uint16_t*>(q),
                         static_cast<const uint16_t*>(k), static_cast<const uint16_t*>(v),
                         static_cast<uint16_t*>(out), lse, a);
      return hipGetLastError();
    }
    const dim3 grid4((unsigned)(8LL * unit4_start(a, a.heads)));
    auto kern = a.waves == 1 ? (a.mode == kStrided ? attn_bf16_kernel<kStrided> : attn_bf16_kernel<kLists>)
                             : (a.mode == kStrided ? attn_bf16_rows4_kernel<kStrided> : attn_bf16_rows4_kernel<kLists>);
    hipLaunchKernelGGL(kern, a.waves == 1 ? grid : grid4, dim3(64 * a.waves), 0, s, static_cast<const uint16_t*>(q),
                       static_cast<const uint16_t*>(k), static_cast<const uint16_t*>(v), idx, cnt,
                       static_cast<uint16_t*>(out), lse, a);
  } else {
    auto kern = a.mode == kStrided ? attn_f32_kernel<kStrided> : attn_f32_kernel<kLists>;
    hipLaunchKernelGGL(kern, grid, dim3(64 * kF32Waves), 0, s, static_cast<const float*>(q),
                       static_cast<const float*>(k), static_cast<const float*>(v), idx, cnt,
                       static_cast<float*>(out), lse, a);
  }
  return hipGetLastError();
}

hipError_t launch_attention_merge(const float* part_o, const float* part_ml, void* out,
                                  float* lse, const MergeArgs& a, hipStream_t s) {
  const int64_t groups = (int64_t)a.n_split * a.nb;
  if (groups == 0) return hipSuccess;
  if (a.dtype == 1)
    hipLaunchKernelGGL(attn_merge_kernel<true>, dim3((unsigned)groups), dim3(64), 0, s, part_o,
                       part_ml, out, lse, a);
  else
    hipLaunchKernelGGL(attn_merge_kernel<false>, dim3((unsigned)groups), dim3(64), 0, s, part_o,
                       part_ml, out, lse, a);
  return hipGetLastError();
}

}  // namespace saf3r
