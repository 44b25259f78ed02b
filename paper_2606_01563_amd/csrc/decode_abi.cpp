// C ABI of the corrected decode: argument checks, launch shape, workspace layout and the
// launches.  Nothing here allocates, frees or synchronises.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>

#include "../../include/momentkv.h"
#include "mkv_abi.h"
#include "mkv_decode.h"

using namespace mkv::abi;

namespace {

constexpr int64_t kDecodeWaves = 768;      // target slice count of an automatic decode split
constexpr int64_t kMaxDecodeWaves = 1 << 24;  // decode grid limit (single-wave workgroups)
// Automatic shape (n_split = 0).  Measured with G = 4, d = 128, bf16, the prepared summary,
// calls replayed back to back, us per call (one workgroup per head / slices / groups):
//   8 heads    256 rows  8.7 /  8.2 /  8.8    512 rows 12.1 / 10.1 /  8.8
//             1024 rows 19.0 / 14.5 /  9.6   2048 rows   -  / 23.5 / 10.4
//   16 heads  1024 rows 19.5 / 18.8 / 10.6   4096 rows   -  / 25.8 / 14.9
//   32 heads   512 rows 12.7 / 13.3 /  9.6   2048 rows   -  / 19.2 / 14.4
//   64 heads   384 rows 11.4 / 14.8 / 10.3   1024 rows 20.0 / 17.2 / 14.0
//             2048 rows   -  / 21.6 / 19.7   4096 rows   -  / 29.6 / 33.8
//   128 heads  512 rows 13.4 / 16.6 / 16.4   1024 rows 20.5 / 21.3 / 21.4
//   256 heads  512 rows 17.3 / 21.0 / 22.5   1024 rows 26.7 / 29.9 / 35.8
//   288 heads  384 rows 21.2 / 20.7 / 25.4    512 rows 25.7 / 24.1 / 30.0
// and with lengths spread over a quarter to all of max_len (one workgroup / slices / groups):
//   48 heads  1020 rows 19.6 / 14.7 / 12.2   1500 rows   -  / 14.7 / 13.8
//   64 heads  1020 rows 19.0 / 13.8 / 13.5   1500 rows   -  / 14.8 / 15.9
//   96 heads   450 rows 12.1 / 13.1 / 15.4   1020 rows 19.5 / 15.0 / 19.2
//   128 heads  600 rows 14.2 / 15.8 / 18.2   1020 rows 19.6 / 17.0 / 20.0
//   192 heads  600 rows 14.4 / 17.3 / 23.6   1020 rows 19.7 / 19.9 / 31.1
// Other types, head dims, groups and orders (G q heads; one workgroup / slices / groups):
//   bf16 d 64, G 4      8 heads  300 rows  5.8 /  7.7 /  7.3    96 heads 640 rows  8.7 / 10.4 /  -
//   bf16 d 64, G 16    64 heads  384 rows  9.2 / 20.7 / 12.6
//   bf16 d 128, G 8    64 heads  257 rows 10.6 / 16.7 / 11.3    64 heads 384 rows 12.4 / 20.0 / 12.0
//   bf16 d 128, G 16   64 heads  300 rows 13.6 / 25.9 / 14.6
//   bf16 d 128, G 1     2 heads  450 rows 11.2 /  8.6 /  8.7    96 heads 640 rows 14.2 / 13.0 /  -
//   bf16, order 0       8 heads  300 rows  7.7 /  8.7 /  9.1
//   bf16, raw summary  32 heads  257 rows 11.0 / 10.5 / 10.1    96 heads 640 rows 17.2 / 15.3 /  -
//   fp32 d 128, G 4    64 heads  300 rows 20.9 / 17.0 / 13.5     2 heads 450 rows 26.0 / 11.1 / 12.2
//                      64 heads  450 rows 27.7 / 18.0 / 18.7    32 heads 1500 rows  -  / 24.4 / 20.2
//                      32 heads 4096 rows   -  / 37.0 / 39.1    96 heads 640 rows 34.1 / 23.9 /  -
//                     160 heads  640 rows 34.8 / 32.4 /  -     256 heads 640 rows 40.4 / 46.8 /  -
//   fp32 d 128, G 8     8 heads  640 rows   -  / 18.5 / 15.2    32 heads 1500 rows  -  / 30.4 / 22.6
//   fp32 d 128, G 16  128 heads  512 rows 33.8 / 39.2 /  -
// (in fp32 a block's products take a wave several times as long: one workgroup per head or
// two blocks per wave of a group lose to slices earlier; at d = 64, or without the summary's
// product, a short cache is too little work to hand over.)
// Up to 256 rows every head runs in one workgroup.  Longer caches of few heads: the
// smallest group length (a multiple of 128 rows) that keeps the launch at kGroupWgs token
// workgroups and, from 8 waves each (one workgroup per CU), with the heads' S_tilde q
// workgroups at the CUs, so that each starts at once; longer groups than kGroupMaxLen lose
// to slices where the lengths differ, except with so few heads that slices are many per
// head.  groups_pay() leaves out what the lines above show.  Otherwise one workgroup per
// head, which needs no hand-off, while the caches are short for how far the heads fill the
// CUs (fused_max_len()); else slices.
constexpr int kCUs = 256;
constexpr int kFusedMaxLen = 256;
constexpr int kFusedMaxLenMany = 384;   // any number of heads
constexpr int kGroupWgs = 192, kGroupMaxLen = 384;
constexpr int kGroupVeryFewHeads = 32, kGroupMaxLenVeryFew = 768;

bool groups_pay(const mkv_decode_params* p, int64_t heads, int group_len) {
  const bool f32 = p->dtype == MKV_F32, d64 = p->head_dim == 64;
  const int rows = p->max_len, G = p->n_q_heads / p->n_kv_heads;
  if (rows <= kFusedMaxLenMany) {  // against one workgroup per head
    if (f32) return d64 ? G <= 8 && heads <= 64 && rows > 288 : heads <= 64 || rows > 288;
    const bool raw = p->summary == 0 || p->summary == 3;
    return !d64 && p->order >= 1 && G <= 8 && (raw || (heads <= 64 && rows > 288));
  }
  if (!f32 || G > 4) return true;  // against slices
  if (group_len == 128) return heads >= 8 || rows > 640;
  return d64 ? rows >= 640 : heads <= 64 && rows > 640 && group_len <= 512;
}

// Longest cache for which one workgroup per head beats slices (with too many heads, or too
// few rows, for groups).
int fused_max_len(const mkv_decode_params* p, int64_t heads) {
  const bool f32 = p->dtype == MKV_F32, d64 = p->head_dim == 64, wide = p->n_q_heads / p->n_kv_heads > 4;
  if (heads > kCUs || 3 * heads <= kCUs) return kFusedMaxLenMany;
  if (heads > 160) return 1024;
  if (f32 && !d64) {
    const bool wider = p->n_q_heads / p->n_kv_heads > 8;
    return heads > 128 ? (wider ? 1024 : 512) : (wider ? 512 : kFusedMaxLenMany);
  }
  if (heads > 128) return 1024;
  return heads == 128 || wide || (d64 && !f32) ? 640 : 512;
}
static_assert(kGroupWgs / 2 <= mkv::kMaxGroupHeads, "at least two groups per head");

// ----------------------------------------------------------------------- decode
// Token slices per KV head of the slices shape.  With n_split = 0: about kDecodeWaves
// single-wave slices in the whole grid (three per CU), at least 32 rows each.  Measured on a
// 288-head stack, longer slices (fewer partials to merge) beat finer splits once every CU
// holds a few slices.  Rows per slice are a multiple of the 32-row block.
void slice_split(const mkv_decode_params* p, int* split_len, int* nsplit) {
  const int64_t heads = (int64_t)p->batch * p->n_kv_heads;
  const int want = p->n_split > 0 ? p->n_split
                                  : (int)std::min<int64_t>(std::max<int64_t>((kDecodeWaves + heads - 1) / heads, 1), 1 << 20);
  const int sl = ceil_div(p->max_len, want);
  *split_len = std::max(32, ceil_div(sl, 32) * 32);
  *nsplit = ceil_div(p->max_len, *split_len);
}

mkv::DecodeShape decode_shape(const mkv_decode_params* p, int* split_len, int* nsplit) {
  const int64_t heads = (int64_t)p->batch * p->n_kv_heads;
  if (p->n_split == 0 && p->max_len > kFusedMaxLen) {
    const int gl_max = heads <= kGroupVeryFewHeads ? kGroupMaxLenVeryFew : kGroupMaxLen;
    for (int gl = 128; gl <= gl_max; gl += 128) {
      const int n = ceil_div(p->max_len, gl);
      if (n > 1 && n <= mkv::kMaxGroups && heads * n <= kGroupWgs &&
          (gl < mkv::kGroupWideLen || heads * (n + 1) <= kCUs)) {
        if (!groups_pay(p, heads, gl)) break;
        *split_len = gl;
        *nsplit = n;
        return mkv::kDecodeGroup;
      }
    }
  }
  slice_split(p, split_len, nsplit);
  if (p->n_split == 1) return mkv::kDecodeFused;
  if (p->n_split == 0 && p->max_len <= fused_max_len(p, heads)) return mkv::kDecodeFused;
  return mkv::kDecodeSlices;
}

}  // namespace

namespace mkv {
namespace abi {

mkv_status check_decode_params(const mkv_decode_params* p) {
  if (!p) return MKV_ERR_NULL;
  if (p->dtype != MKV_F32 && p->dtype != MKV_BF16) return MKV_ERR_DTYPE;
  if (p->batch < 1 || p->n_q_heads < 1 || p->n_kv_heads < 1 || p->head_dim < 1 || p->cap < 1)
    return MKV_ERR_SHAPE;
  if (p->n_q_heads % p->n_kv_heads) return MKV_ERR_SHAPE;
  if (p->order < -1 || p->order > 1) return MKV_ERR_SHAPE;
  if (!(p->scale >= 0.f) || !std::isfinite(p->scale) || !(p->tau >= 0.f) || !std::isfinite(p->tau))
    return MKV_ERR_SHAPE;
  if (p->head_dim != 64 && p->head_dim != 128) return MKV_ERR_UNSUPPORTED;
  if (p->n_q_heads / p->n_kv_heads > 16) return MKV_ERR_UNSUPPORTED;
  if (p->n_split < 0) return MKV_ERR_SHAPE;
  if (p->summary < 0 || p->summary > 3) return MKV_ERR_SHAPE;
  if (p->summary == 2 && p->dtype != MKV_BF16) return MKV_ERR_SHAPE;  // half precision: bf16 only
  if (p->max_len < 1 || p->max_len > p->cap) return MKV_ERR_CAPACITY;
  // grid of single-wave workgroups: B * Hkv * (slices + covariance waves)
  int split_len = 0, nsplit = 0;
  decode_shape(p, &split_len, &nsplit);
  const int64_t waves = (int64_t)p->batch * p->n_kv_heads * (nsplit + p->head_dim / 32);
  if (waves > kMaxDecodeWaves) return MKV_ERR_UNSUPPORTED;
  return MKV_OK;
}

mkv::DecodeArgs decode_layout(const mkv_decode_params* p, void* ws, size_t* total,
                              size_t cnt_slots) {
  mkv::DecodeArgs a;
  std::memset(&a, 0, sizeof a);
  a.n_heads = p->batch * p->n_kv_heads;
  a.G = p->n_q_heads / p->n_kv_heads;
  a.n_pairs = p->batch * p->n_q_heads;
  a.Hkv = p->n_kv_heads;
  a.cap = p->cap;
  a.order = p->order;
  a.scale = p->scale > 0.f ? p->scale : 1.0f / std::sqrt((float)p->head_dim);
  a.tau = p->tau;
  a.shape = decode_shape(p, &a.split_len, &a.nsplit);
  a.nsq = p->order >= 1 ? p->head_dim / 32 : 0;
  a.summary = p->summary;
  const size_t H = a.n_heads, D = p->head_dim, G = a.G;
  // Every shape reserves the partials of the slices shape (a group launch has fewer, one
  // workgroup per head none), so that the bytes grow with max_len as they would without the
  // choice of a shape: a workspace sized for long caches serves the calls on shorter ones.
  int slice_len = 0, slices = 0;
  slice_split(p, &slice_len, &slices);
  const size_t parts = std::max(slices, a.nsplit);
  Carver c;
  c.base = static_cast<char*>(ws);
  // The leading bytes (the flag and the group launch's counters in its block, then one
  // arrival counter per head) are zero-filled by the caller before first use; every call
  // leaves the counters at zero.
  a.flag = c.take<int32_t>(sizeof(int32_t));
  a.cnt = c.take<int32_t>(std::max<size_t>(cnt_slots, H) * sizeof(int32_t));
  auto take_parts = [&](size_t n) {
    a.part_o = c.take<float>(H * n * G * D * sizeof(float));
    a.part_ml = c.take<float>(H * n * G * 2 * sizeof(float));
    a.sq = c.take<float>(H * G * D * sizeof(float));
  };
  const size_t first = c.off;
  take_parts(parts);
  if (a.shape == kDecodeGroup) {
    // The group launch's few partials at the end of the reservation: away from the leading
    // bytes, where a call with more heads on the same workspace has its counters.
    if (a.flag) a.cnt = a.flag + 1;
    const size_t end = c.off;
    c.off = first;
    take_parts(a.nsplit);
    c.off = first + (end - c.off);
    take_parts(a.nsplit);
  }
  *total = c.off;
  return a;
}

mkv_status check_decode_buffers(const mkv_decode_params* p, const void* q, const void* k_cache,
                                const void* v_cache, const int32_t* lens, const void* k_new,
                                const void* v_new, const int32_t* n_e, const float* s_k,
                                const float* s_v, const void* S, const void* out) {
  if (!q || !k_cache || !v_cache || !lens || !n_e || !s_k || !s_v || !S || !out) return MKV_ERR_NULL;
  if ((k_new == nullptr) != (v_new == nullptr)) return MKV_ERR_NULL;
  const size_t es = elem_size(p->dtype);
  const size_t cache_bytes = (size_t)p->batch * p->n_kv_heads * p->cap * p->head_dim * es;
  const size_t out_bytes = (size_t)p->batch * p->n_q_heads * p->head_dim * es;
  if (ranges_overlap(out, out_bytes, k_cache, cache_bytes) ||
      ranges_overlap(out, out_bytes, v_cache, cache_bytes) ||
      ranges_overlap(out, out_bytes, q, out_bytes) ||
      ranges_overlap(k_cache, cache_bytes, v_cache, cache_bytes))
    return MKV_ERR_ALIAS;
  return MKV_OK;
}

bool decode_overlaps(const mkv_decode_params* p, const void* buf, size_t bytes,
                     const void* k_cache, const void* v_cache, const void* out) {
  const size_t es = elem_size(p->dtype);
  const size_t cache_bytes = (size_t)p->batch * p->n_kv_heads * p->cap * p->head_dim * es;
  const size_t out_bytes = (size_t)p->batch * p->n_q_heads * p->head_dim * es;
  return ranges_overlap(buf, bytes, k_cache, cache_bytes) ||
         ranges_overlap(buf, bytes, v_cache, cache_bytes) || ranges_overlap(buf, bytes, out, out_bytes);
}

void set_decode_buffers(DecodeArgs& a, const void* q, void* k_cache, void* v_cache, int32_t* lens,
                        const void* k_new, const void* v_new, const int32_t* n_e, const float* s_k,
                        const float* s_v, const void* S, void* out, float* lse_out,
                        float* w_r_out) {
  a.q = q;
  a.k_cache = k_cache;
  a.v_cache = v_cache;
  a.lens = lens;
  a.k_new = k_new;
  a.v_new = v_new;
  a.n_e = n_e;
  a.s_k = s_k;
  a.s_v = s_v;
  a.S = static_cast<const float*>(S);
  a.out = out;
  a.lse_out = lse_out;
  a.w_r_out = w_r_out;
}

}  // namespace abi
}  // namespace mkv

extern "C" {

size_t momentkv_decode_workspace_size(const mkv_decode_params* p) {
  if (check_decode_params(p) != MKV_OK) return 0;
  size_t total = 0;
  decode_layout(p, nullptr, &total, 0);
  return total;
}

size_t momentkv_decode_workspace_bytes(const mkv_decode_params* p) {
  return momentkv_decode_workspace_size(p);
}

size_t momentkv_decode_workspace_zero_bytes(const mkv_decode_params* p) {
  if (check_decode_params(p) != MKV_OK) return 0;
  const size_t heads = (size_t)p->batch * p->n_kv_heads;
  return align_up(sizeof(int32_t)) + align_up(heads * sizeof(int32_t));
}

size_t momentkv_prepared_summary_size(const mkv_decode_params* p) {
  if (check_decode_params(p) != MKV_OK || p->summary == 3) return 0;
  return (size_t)p->batch * p->n_kv_heads * p->head_dim * p->head_dim * (p->summary == 2 ? 2 : 4);
}

mkv_status momentkv_prepare_summary(const mkv_decode_params* p, const int32_t* n_e,
                                    const float* s_k, const float* s_v, const float* S,
                                    void* prepared, void* stream) {
  mkv_status st = check_decode_params(p);
  if (st != MKV_OK) return st;
  if (p->summary == 3) return MKV_ERR_SHAPE;  // the raw bf16 form has no prepared form
  if (!n_e || !s_k || !s_v || !S || !prepared) return MKV_ERR_NULL;
  if (reinterpret_cast<uintptr_t>(prepared) % 16) return MKV_ERR_SHAPE;
  const size_t heads = (size_t)p->batch * p->n_kv_heads, d = p->head_dim;
  const size_t out_bytes = heads * d * d * (p->summary == 2 ? 2 : 4);
  if (ranges_overlap(prepared, out_bytes, S, heads * d * d * 4) ||
      ranges_overlap(prepared, out_bytes, s_k, heads * d * 4) ||
      ranges_overlap(prepared, out_bytes, s_v, heads * d * 4) ||
      ranges_overlap(prepared, out_bytes, n_e, heads * 4))
    return MKV_ERR_ALIAS;
  size_t total = 0;
  mkv::DecodeArgs a = decode_layout(p, nullptr, &total, 0);
  a.n_e = n_e;
  a.s_k = s_k;
  a.s_v = s_v;
  a.S = S;
  hipError_t e = mkv::launch_prepare_summary(a, prepared, p->dtype == MKV_BF16, p->head_dim,
                                             static_cast<hipStream_t>(stream));
  return e == hipSuccess ? MKV_OK : MKV_ERR_HIP;
}

mkv_status momentkv_decode_attn(const mkv_decode_params* p, const void* q, void* k_cache,
                                void* v_cache, int32_t* lens, const void* k_new,
                                const void* v_new, const int32_t* n_e, const float* s_k,
                                const float* s_v, const void* S, void* out, float* lse_out,
                                float* w_r_out, void* workspace, size_t workspace_bytes,
                                void* stream) {
  mkv_status st = check_decode_params(p);
  if (st != MKV_OK) return st;
  st = check_decode_buffers(p, q, k_cache, v_cache, lens, k_new, v_new, n_e, s_k, s_v, S, out);
  if (st != MKV_OK) return st;
  size_t need = 0;
  decode_layout(p, nullptr, &need, 0);
  if (!workspace || workspace_bytes < need) return MKV_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(workspace) % kAlign) return MKV_ERR_WORKSPACE;
  if (decode_overlaps(p, workspace, need, k_cache, v_cache, out)) return MKV_ERR_ALIAS;
  size_t total = 0;
  mkv::DecodeArgs a = decode_layout(p, workspace, &total, 0);
  set_decode_buffers(a, q, k_cache, v_cache, lens, k_new, v_new, n_e, s_k, s_v, S, out, lse_out,
                     w_r_out);
  hipError_t e = mkv::launch_decode(a, p->dtype == MKV_BF16, p->head_dim,
                                    static_cast<hipStream_t>(stream));
  return e == hipSuccess ? MKV_OK : MKV_ERR_HIP;
}

}  // extern "C"
