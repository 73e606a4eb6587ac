// Launch stand-ins for the host-layer sanitizer build: the C ABI layer
// (csrc/api.cpp) compiled by g++ with AddressSanitizer and
// UndefinedBehaviorSanitizer and linked against these functions instead of
// the HIP kernels, so every validation, sizing and launch-ordering path of
// the ABI runs on the CPU. Each stand-in checks the arguments the host layer
// built for its kernel (counts inside their arrays, heads in range and
// distinct, ordered prefix sums, workspace offsets inside the workspace the
// caller declared) and returns hipErrorInvalidValue when one is off, which
// the ABI reports as SAF3R_ERR_HIP. Nothing here touches a GPU.
#include <stdint.h>

#include <vector>

#include "../../paper_2607_03612_amd/csrc/saf3r_internal.h"

namespace saf3r {
namespace {

bool heads_ok(const int16_t* head, int n, int limit) {
  if (n < 0 || n > kMaxHeads) return false;
  std::vector<char> seen(kMaxHeads, 0);
  for (int i = 0; i < n; ++i) {
    if (head[i] < 0 || head[i] >= limit || seen[head[i]]) return false;
    seen[head[i]] = 1;
  }
  return true;
}

// The Top-K heads and, after them, the static and the global-probe heads whose
// lists the same launch writes.
bool topk_heads_ok(const TopKArgs& a) {
  if (a.n_heads < 0 || a.n_static < 0 || a.n_global < 0) return false;
  if (a.n_global > 0 && a.nb > kGlobalFusedBlocks) return false;
  if (a.n_static > 0 && a.tokens_per_frame < 1) return false;
  if (!heads_ok(a.head, a.n_heads + a.n_static + a.n_global, kMaxHeads)) return false;
  for (int i = 0; i < a.n_heads + a.n_static + a.n_global; ++i) {
    const bool is_static = i >= a.n_heads && i < a.n_heads + a.n_static;
    if (is_static ? a.pattern[i] != kDense && a.pattern[i] != kFrameLocal && a.pattern[i] != kAnchor && a.pattern[i] != kStride
                  : a.topk[i] < 1 || a.topk[i] > a.nb || a.topk[i] > a.cap)
      return false;
  }
  return true;
}

bool blocks_ok(int64_t n, int nb) { return n >= 1 && nb == (int)((n + kBlock - 1) / kBlock); }

hipError_t launch_status(bool ok) { return ok ? hipSuccess : hipErrorInvalidValue; }

int attention_launches[2] = {0, 0};  // of one wave and of four waves to a workgroup
int topk_rows_per_group = 0;         // of the last Top-K launch; 0 for the pair with a workspace
int topk_global = 0;                 // global-probe heads beside it

// The workgroups of a list or strided launch take every (head, key range,
// query block) exactly once: one wave each, or all four waves of a workgroup
// where the head's rows are shared. With the kernels' own work_item functions.
bool covers_every_item(const AttnArgs& a) {
  const bool four = a.waves == 4;
  std::vector<int> pos_of(kMaxHeads, -1);
  for (int p = 0; p < a.heads; ++p) pos_of[a.order[p]] = p;
  std::vector<int> first(a.heads + 1, 0);  // of a head's items
  for (int p = 0; p < a.heads; ++p) first[p + 1] = first[p] + a.nb * (a.split_pos[p] >= 0 ? a.splits : 1);
  std::vector<int> taken(first[a.heads], 0);
  const int groups = 8 * (four ? unit4_start(a, a.heads) : a.unit_start[a.heads]);
  for (int g = 0; g < groups; ++g) {
    int shared_item = -1;
    for (int wave = 0; wave < a.waves; ++wave) {
      const Work w = four ? work_item4(a, g, wave) : work_item(a, g);
      if (!w.valid) continue;
      const int p = w.h >= 0 && w.h < kMaxHeads ? pos_of[w.h] : -1;
      if (p < 0 || w.i < 0 || w.i >= a.nb) return false;
      const bool split = a.split_pos[p] >= 0;
      if (split ? w.chunk < 0 || w.chunk >= a.splits : w.chunk != -1) return false;
      if (w.item != (split ? (a.split_pos[p] * a.splits + w.chunk) * a.nb + w.i : -1)) return false;
      const int item = first[p] + (split ? w.chunk : 0) * a.nb + w.i;
      if (four && w.shared) {
        if (wave > 0 && shared_item != item) return false;  // the four waves meet at barriers
        if (wave == 0) ++taken[item];
        shared_item = item;
      } else {
        if (shared_item >= 0) return false;
        ++taken[item];
      }
    }
  }
  for (int t : taken)
    if (t != 1) return false;
  return true;
}

}  // namespace

extern "C" int saf3r_stub_topk_rows_per_group() { return topk_rows_per_group; }
extern "C" int saf3r_stub_topk_global() { return topk_global; }
extern "C" int saf3r_stub_attention_launches(int waves) { return attention_launches[waves == 4 ? 1 : 0]; }

hipError_t launch_pool(int dtype, const void* q, const void* k, double* qp, double* kp,
                       const PoolArgs& a, hipStream_t) {
  return launch_status((dtype == 0 || dtype == 1) && q && k && qp && kp && blocks_ok(a.n, a.nb) &&
                 heads_ok(a.head, a.n_heads, kMaxHeads));
}

hipError_t launch_select_topk(const double* qp, const double* kpT, int32_t* idx, int32_t* cnt,
                              double*, const TopKArgs& a, size_t lds_bytes, hipStream_t) {
  bool ok = qp && kpT && idx && cnt && blocks_ok(a.n, a.nb) && topk_heads_ok(a);
  ok = ok && (a.rows_per_group == 1 || a.rows_per_group == 2 || a.rows_per_group == 4 ||
              a.rows_per_group == 8 || a.rows_per_group == 16);
  ok = ok && lds_bytes == topk_lds_bytes(a.rows_per_group, a.nb) && lds_bytes <= 160 * 1024;
  topk_rows_per_group = a.rows_per_group;
  topk_global = a.n_global;
  for (int i = 0; ok && i < a.n_heads; ++i) ok = a.topk[i] >= 1 && a.topk[i] <= a.nb && a.topk[i] <= a.cap;
  return launch_status(ok);
}

hipError_t launch_select_topk_ws(const double* qp, const double* kpT, uint32_t* keys, int32_t* idx,
                                 int32_t* cnt, double*, const TopKArgs& a, hipStream_t) {
  bool ok = qp && kpT && keys && idx && cnt && blocks_ok(a.n, a.nb) && topk_heads_ok(a) && a.n_heads >= 1;
  topk_rows_per_group = 0;
  topk_global = a.n_global;
  for (int i = 0; ok && i < a.n_heads; ++i) ok = a.topk[i] >= 1 && a.topk[i] <= a.nb && a.topk[i] <= a.cap;
  return launch_status(ok);
}

hipError_t launch_select_static(int32_t* idx, int32_t* cnt, const StaticArgs& a, hipStream_t) {
  bool ok = idx && cnt && blocks_ok(a.n, a.nb) && heads_ok(a.head, a.n_heads, kMaxHeads) &&
            a.tokens_per_frame >= 1;
  for (int i = 0; ok && i < a.n_heads; ++i)
    ok = a.pattern[i] == kDense || a.pattern[i] == kFrameLocal || a.pattern[i] == kAnchor ||
         a.pattern[i] == kStride;
  return launch_status(ok);
}

hipError_t launch_select_global(const double* qp, const double* kpT, int32_t* idx, int32_t* cnt,
                                double*, const GlobalArgs& a, hipStream_t) {
  bool ok = qp && kpT && idx && cnt && blocks_ok(a.n, a.nb) && heads_ok(a.head, a.n_heads, kMaxHeads);
  for (int i = 0; ok && i < a.n_heads; ++i) ok = a.topk[i] >= 1 && a.topk[i] <= a.nb && a.topk[i] <= a.cap;
  return launch_status(ok);
}

hipError_t launch_cosine(int dtype, const void* f, double* fb, double* sim, int32_t* idx,
                         int32_t* cnt, const CosineArgs& a, hipStream_t) {
  bool ok = (dtype == 0 || dtype == 1) && f && fb && idx && cnt && blocks_ok(a.n, a.nb) &&
            a.dim >= 1 && a.dim <= kMaxCosineDim && sim == fb + (int64_t)a.dim * a.nb &&
            a.n_groups >= 0 && a.n_groups <= kMaxHeads && a.group_start[0] == 0;
  for (int g = 0; ok && g < a.n_groups; ++g)
    ok = a.group_start[g + 1] > a.group_start[g] && a.group_k[g] >= 1 &&
         a.group_k[g] <= kMaxCosinePerFrame && (g == 0 || a.group_k[g] > a.group_k[g - 1]);
  ok = ok && heads_ok(a.head, a.group_start[a.n_groups], kMaxHeads);
  return launch_status(ok);
}

hipError_t launch_nmse(int dtype, const void* ref, const void* test, void* workspace, double* out,
                       int heads, int64_t n, hipStream_t) {
  return launch_status((dtype == 0 || dtype == 1) && ref && test && workspace && out && heads >= 1 &&
                 heads <= kMaxHeads && n >= 1);
}

hipError_t nmse_scratch(void** ptr) {
  static double2 fake[kMaxHeads * kNmseParts];  // host stand-in, never written
  *ptr = fake;
  return hipSuccess;
}

hipError_t launch_attention(int dtype, const void* q, const void* k, const void* v,
                            const int32_t*, const int32_t*, void* out, float*, const AttnArgs& a,
                            hipStream_t) {
  bool ok = (dtype == 0 || dtype == 1) && q && k && v && out && blocks_ok(a.n, a.nb) &&
            a.slab == (a.nb + 7) / 8 && a.slab4 == ((a.nb + 3) / 4 + 7) / 8 && a.splits == kSplitChunks &&
            a.mode >= 0 && a.mode <= 2 && (a.waves == 1 || (a.waves == 4 && dtype == 1 && a.mode != 1)) &&
            heads_ok(a.order, a.heads, kMaxHeads) && a.unit_start[0] == 0 && a.shared_before[0] == 0;
  bool any_shared = false;
  int n_split = 0;
  for (int i = 0; ok && i < a.heads; ++i) {
    const bool split = a.split_pos[i] >= 0;
    ok = a.unit_start[i + 1] == a.unit_start[i] + a.slab * (split ? a.splits : 1) &&
         a.split_pos[i] >= -1 && a.split_pos[i] < kMaxHeads && (!split || a.part_o);
    const int shared = a.shared_before[i + 1] - a.shared_before[i];
    ok = ok && (shared == 0 || (shared == (split ? a.splits : 1) && a.waves == 4));
    any_shared = any_shared || shared != 0;
    if (split) {
      ok = ok && a.split_pos[i] == n_split && a.mode == 0;
      ++n_split;
    }
    if (a.mode == 2) ok = ok && a.stride[a.order[i]] >= 1 && a.stride[a.order[i]] <= a.n;
  }
  // the partials of split items start after the O accumulators
  if (ok && n_split > 0)
    ok = a.part_ml == a.part_o + (int64_t)n_split * a.splits * a.nb * kBlock * kHeadDim;
  ok = ok && any_shared == (a.waves == 4);
  if (ok && a.mode != 1) ok = covers_every_item(a);
  if (ok && a.heads > 0) ++attention_launches[a.waves == 4 ? 1 : 0];
  return launch_status(ok);
}

// the check's result as the device would report it for lists that pass
hipError_t run_validate_index(const int32_t* idx, const int32_t* cnt, int32_t* result,
                              const ValidateArgs& a, int32_t out[2], hipStream_t) {
  bool ok = idx && cnt && result && out && a.nb >= 1 && a.nb <= kMaxBlocks && a.cap >= 1 &&
            a.n_heads >= 1 && heads_ok(a.head, a.n_heads, kMaxHeads);
  for (int i = 0; ok && i < a.n_heads; ++i) ok = a.expect[i] == -1 || (a.expect[i] >= 1 && a.expect[i] <= a.nb);
  out[0] = 0;
  out[1] = 0x7fffffff;
  return launch_status(ok);
}

hipError_t launch_attention_merge(const float* part_o, const float* part_ml, void* out, float*,
                                  const MergeArgs& a, hipStream_t) {
  return launch_status(part_o && part_ml && out && blocks_ok(a.n, a.nb) && a.splits == kSplitChunks &&
                 (a.dtype == 0 || a.dtype == 1) &&
                 heads_ok(a.head, a.n_split, kMaxHeads) && a.n_split >= 1 &&
                 part_ml == part_o + (int64_t)a.n_split * a.splits * a.nb * kBlock * kHeadDim);
}

}  // namespace saf3r
