// C ABI of the decode step with eviction: argument checks, workspace layout and the
// launches.  Nothing here allocates, frees or synchronises.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdint>
#include <cstring>

#include "../../include/momentkv.h"
#include "mkv_abi.h"
#include "mkv_evict.h"

using namespace mkv::abi;

namespace {

// ------------------------------------------------------------------ decode + eviction
// Two launch shapes.  Fused (one read of the cache; where one_read() says, or whenever
// n_split > 0): the scoring launch has one workgroup per CU of the target (kCUs; n_split
// per head when n_split > 0), each taking an equal contiguous share of the flattened
// (head, 32-row block) range, so that a head has at most maxslots partial states (at most
// evict_max_slices(); fewer workgroups otherwise); a finishing launch follows.  Short
// caches: one launch with one workgroup per head (two per CU) that scores, selects,
// updates and then attends to the new cache itself (a second read of a short cache,
// mostly from L2); a fused workgroup holds one head's summary and V tiles alone on its
// CU, which there costs more than that second read.
// Workspace: the flag first, then the score records and the per-block running maxima, then
// the heads' partial states (fused).
constexpr int kCUs = 256;
// Where the one-read shape runs.  Measured per call, every head evicting, short against
// one-read shape, us (fp32 swept over 33 numbers of heads, bf16 over 17, 8 to 12 lengths and
// 1 to 16 queries per KV head; 320 rows and more do not fit the short launch's records):
//   bf16 d 128, G 4     8 heads 256 rows 23.1 / 20.5    32 heads 256 rows 23.3 / 24.2
//                      32 heads 288 rows 25.9 / 24.3    48 heads 288 rows 26.2 / 31.2
//                      64 heads 288 rows 26.3 / 26.1
//   bf16 d 128, G 16   32 heads 288 rows 38.6 / 38.7    d 64, G 4  8 heads 256 rows 13.3 / 14.9
//   fp32 d 128, G 4     8 heads 112 rows 37.2 / 29.1    64 heads 112 rows 37.9 / 33.9
//                      96 heads 128 rows 41.6 / 50.3    96 heads 160 rows 54.1 / 50.2
//                     128 heads 112 rows 42.5 / 36.8   192 heads 128 rows 45.2 / 52.1
//                     192 heads 160 rows 57.6 / 56.5   256 heads 112 rows 47.5 / 35.0
//                     288 heads 128 rows 65.1 / 62.3   400 heads 192 rows 89.2 / 91.6
//   fp32 d 128, G 8    32 heads 112 rows 36.4 / 36.1    96 heads 128 rows 37.5 / 56.7
//                      48 heads 160 rows 46.4 / 37.5    48 heads 256 rows 52.0 / 55.0
//   fp32 d 128, G 16    8 heads 112 rows 43.4 / 43.7    32 heads 160 rows 53.8 / 46.1
//   fp32 d 64, G 4     64 heads 112 rows 19.0 / 18.1    96 heads 160 rows 23.7 / 24.7
//                     192 heads 192 rows 25.5 / 27.5   288 heads 224 rows 38.4 / 33.5
//   fp32 d 64, G 8    128 heads 112 rows 21.9 / 21.8   160 heads 224 rows 30.4 / 34.0
//   fp32 d 64, G 16     8 heads 128 rows 26.0 / 26.5     8 heads 160 rows 30.9 / 26.6
// Few heads leave CUs idle that the one-read shape shares out, and in fp32 a block's products
// take the one workgroup of a head several times as long.  Once a workgroup's share is more
// than a block it crosses heads (a second setup and partial state) unless the heads divide the
// CUs; above 256 heads the short launch runs in two rounds.  The lines are drawn where no
// evicting call is more than 3% slower than with the short launch.  (Where no head evicts, the
// second launch makes the call longer: bf16, 8 heads 288 rows 14.1 / 15.3.)
constexpr int kFusedMinLen = 320, kFusedMinLenF32 = 112;

bool one_read(const mkv_decode_params* p) {
  if (p->n_split > 0 || p->max_len >= kFusedMinLen) return true;
  const int64_t heads = (int64_t)p->batch * p->n_kv_heads;
  const int G = p->n_q_heads / p->n_kv_heads, wide = G <= 4 ? 0 : G <= 8 ? 1 : 2;
  if (p->dtype != MKV_F32)
    return p->head_dim == 128 && G <= 8 && heads <= 32 && p->max_len >= (heads <= 16 ? 256 : 257);
  if (p->max_len < kFusedMinLenF32) return false;
  // fp32: the least number of 32-row blocks, by heads (rows) and d = 64, 128 with up to 4, 8
  // and 16 queries per head; 11 blocks are never short
  static constexpr int kBlocks[9][2][3] = {
      {{4, 4, 5}, {4, 4, 5}},      // up to 32 heads, or a block per workgroup at most
      {{5, 6, 8}, {5, 9, 9}},      // up to 63
      {{5, 5, 5}, {5, 5, 5}},      // 64
      {{6, 7, 9}, {5, 10, 10}},    // up to 127
      {{4, 4, 6}, {4, 7, 7}},      // 128
      {{7, 8, 10}, {5, 11, 11}},   // up to 255
      {{4, 6, 8}, {4, 11, 11}},    // 256
      {{6, 10, 10}, {4, 10, 10}},  // up to 320
      {{8, 11, 11}, {7, 11, 11}},  // more
  };
  const int blocks = ceil_div(p->max_len, 32);
  const int row = heads <= 32 || heads * blocks <= kCUs ? 0
                  : heads < 64                          ? 1
                  : heads == 64                         ? 2
                  : heads < 128                         ? 3
                  : heads == 128                        ? 4
                  : heads < 256                         ? 5
                  : heads == 256                        ? 6
                  : heads <= 320                        ? 7
                                                        : 8;
  const bool d128 = p->head_dim == 128;
  if (row == 0 && d128 && wide == 1 && heads > 32) return blocks >= 5;
  return blocks >= kBlocks[row][d128][wide];
}

mkv::EvictArgs evict_layout(const mkv_decode_params* p, int32_t budget, void* ws, size_t* total) {
  mkv::EvictArgs e;
  std::memset(&e, 0, sizeof e);
  e.n_heads = p->batch * p->n_kv_heads;
  e.G = p->n_q_heads / p->n_kv_heads;
  e.cap = p->cap;
  e.max_len = p->max_len;
  e.budget = budget;
  e.order = p->order;
  e.scale = p->scale > 0.f ? p->scale : 1.0f / std::sqrt((float)p->head_dim);
  e.tau = p->tau;
  e.hblocks = ceil_div(p->max_len, 32);
  e.rec_len = 32 * e.hblocks;
  e.fused = one_read(p) ? 1 : 0;
  const size_t H = e.n_heads, G = e.G, D = p->head_dim;
  Carver c;
  c.base = static_cast<char*>(ws);
  const int64_t want = p->n_split > 0 ? (int64_t)p->n_split * e.n_heads : kCUs;
  if (e.fused) {
    const int64_t T = (int64_t)e.n_heads * e.hblocks;
    int64_t nwg = std::max<int64_t>(1, std::min(want, T));
    auto slots = [&](int64_t n) {
      const int64_t per = std::max<int64_t>(1, T / n);  // the fewest blocks a workgroup takes
      return std::min<int64_t>(n, (e.hblocks + per - 1) / per + 1);
    };
    while (nwg > 1 && slots(nwg) > mkv::evict_max_slices()) --nwg;
    e.nwg = (int)nwg;
    e.maxslots = (int)slots(nwg);
  }
  e.flag = c.take<int32_t>(sizeof(int32_t));  // zero-filled once by the caller
  e.rec = c.take<float>(H * (G + 2) * e.rec_len * sizeof(float));
  e.blkm = c.take<float>(H * (G + 1) * e.hblocks * sizeof(float));
  // Partial states are reserved for both shapes, by a bound on H * maxslots that grows with
  // the rows and with the heads (slots() is at most hblocks + 1, and at most
  // ceil(2 want / H) + 1 since a workgroup takes at least T / (2 want) blocks): a workspace
  // sized for long caches or many heads serves the calls with less of either, whichever
  // shape they take.
  const size_t parts = std::min({H * (e.hblocks + 1), (size_t)(2 * want) + 2 * H, H * mkv::evict_max_slices()});
  e.part_o = c.take<float>(parts * G * D * sizeof(float));
  e.part_ml = c.take<float>(parts * G * 2 * sizeof(float));
  *total = c.off;
  return e;
}

mkv_status check_evict_params(const mkv_decode_params* p, int32_t budget) {
  mkv_status st = check_decode_params(p);
  if (st != MKV_OK) return st;
  if (p->summary != 0) return MKV_ERR_SHAPE;
  if (budget < 1) return MKV_ERR_BUDGET;
  return MKV_OK;
}

}  // namespace

extern "C" {

size_t momentkv_decode_evict_workspace_size(const mkv_decode_params* p) {
  if (check_evict_params(p, 1) != MKV_OK) return 0;
  size_t total = 0;
  evict_layout(p, 1, nullptr, &total);
  return total;
}

size_t momentkv_decode_evict_workspace_bytes(const mkv_decode_params* p) {
  return momentkv_decode_evict_workspace_size(p);
}

mkv_status momentkv_decode_evict(const mkv_decode_params* p, int32_t budget, const void* q,
                                 void* k_cache, void* v_cache, int32_t* lens,
                                 const void* k_new, const void* v_new, int32_t* n_e,
                                 float* s_k, float* s_v, float* S, void* out, float* lse_out,
                                 float* w_r_out, int32_t* evicted_out, void* workspace,
                                 size_t workspace_bytes, void* stream) {
  mkv_status st = check_evict_params(p, budget);
  if (st != MKV_OK) return st;
  if (!q || !k_cache || !v_cache || !lens || !k_new || !v_new || !n_e || !s_k || !s_v || !S || !out)
    return MKV_ERR_NULL;
  size_t need = 0;
  evict_layout(p, budget, nullptr, &need);
  if (!workspace || workspace_bytes < need) return MKV_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(workspace) % kAlign) return MKV_ERR_WORKSPACE;
  const size_t es = elem_size(p->dtype);
  const size_t heads = (size_t)p->batch * p->n_kv_heads, d = p->head_dim;
  const size_t cache_bytes = heads * p->cap * d * es;
  const size_t out_bytes = (size_t)p->batch * p->n_q_heads * d * es;
  const size_t s_bytes = heads * d * d * 4, vec_bytes = heads * d * 4;
  const void* outs[] = {k_cache, v_cache, out, S, s_k, s_v, workspace};
  const size_t outn[] = {cache_bytes, cache_bytes, out_bytes, s_bytes, vec_bytes, vec_bytes, need};
  for (int i = 0; i < 7; ++i)
    for (int j = i + 1; j < 7; ++j)
      if (ranges_overlap(outs[i], outn[i], outs[j], outn[j])) return MKV_ERR_ALIAS;
  if (ranges_overlap(out, out_bytes, q, out_bytes)) return MKV_ERR_ALIAS;
  size_t total = 0;
  mkv::EvictArgs e = evict_layout(p, budget, workspace, &total);
  e.q = q;
  e.k_cache = k_cache;
  e.v_cache = v_cache;
  e.lens = lens;
  e.k_new = k_new;
  e.v_new = v_new;
  e.n_e = n_e;
  e.s_k = s_k;
  e.s_v = s_v;
  e.S = S;
  e.evicted = evicted_out;
  e.out = out;
  e.lse_out = lse_out;
  e.w_r_out = w_r_out;
  const hipStream_t hs = static_cast<hipStream_t>(stream);
  return mkv::launch_evict(e, p->dtype == MKV_BF16, p->head_dim, hs) == hipSuccess ? MKV_OK : MKV_ERR_HIP;
}

}  // extern "C"
