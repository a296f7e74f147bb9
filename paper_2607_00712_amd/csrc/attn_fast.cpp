// Host side of the hand-scheduled head_dim-128 attention kernel.
//
// The kernel itself is gfx950 assembly generated by attn_fast_gen.py and
// assembled at build time into a code object that this file embeds; it is
// loaded once per device with hipModuleLoadData and launched with its
// arguments packed in one by-value block (AttnFastArgs, whose layout the
// generator reads at fixed offsets). It computes what attn_chunk_kernel<128>
// computes (same work items, split segments and partial-result layout, so the
// same merge kernel completes a split launch); see the generator for the
// schedule.
#include <limits.h>
#include <mutex>
#include <stdlib.h>
#include <string.h>

#include "ispa_internal.h"

namespace ispa {
namespace {

const unsigned char kAttnFastImage[] = {
#include "attn_fast_hsaco.inc"
};

// Kernel arguments; the byte offsets are those of the generator's A_* names.
struct AttnFastArgs {
  const void* q;          // 0
  const void* k;          // 8
  const void* v;          // 16
  float* out;             // 24
  float* lse;             // 32
  float* out_local;       // 40
  float* lse_local;       // 48
  float* part_o;          // 56
  float* part_lse;        // 64
  uint32_t units;         // 72
  int32_t ld;             // 76
  int32_t n_q;            // 80
  int32_t q_tiles;        // 84
  int32_t n_tiles;        // 88
  int32_t n_tiles_local;  // 92
  int32_t n_seg;          // 96
  int32_t max_pieces;     // 100
  int32_t per_xcd;        // 104
  int32_t n_log;          // 108
  int32_t b0, e0, b1, e1, b2, e2;  // 112 .. 132
  int32_t tb1, tb2;       // 136, 140
  float scale;            // 144
  float scale_log2;       // 148
  float lazy;             // 152
  int32_t dual;           // 156
  float neg_scale_log2;   // 160
  int32_t ld2;            // 164
  int32_t ld4;            // 168
  int32_t pad0;           // 172
  uint32_t* ctr;          // 176: split fold counters (null: the merge kernel completes the split)
  int32_t pad1[2];        // 184 .. 191
};
static_assert(sizeof(AttnFastArgs) == 192, "argument block size");
static_assert(offsetof(AttnFastArgs, units) == 72 && offsetof(AttnFastArgs, b0) == 112 &&
                  offsetof(AttnFastArgs, scale) == 144 && offsetof(AttnFastArgs, ld4) == 168 &&
                  offsetof(AttnFastArgs, ctr) == 176,
              "argument offsets");

constexpr int kMaxDevices = 64;
std::mutex g_mu;
hipFunction_t g_fn[kMaxDevices];

hipFunction_t fast_function() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_mu);
  if (g_fn[dev] == nullptr) {
    hipModule_t mod = nullptr;
    if (hipModuleLoadData(&mod, kAttnFastImage) != hipSuccess) return nullptr;
    hipFunction_t fn = nullptr;
    if (hipModuleGetFunction(&fn, mod, "ispa_attn_fast_d128") != hipSuccess) return nullptr;
    g_fn[dev] = fn;
  }
  return g_fn[dev];
}

}  // namespace

bool attn_fast_eligible(const AttnArgs& a, int head_dim) {
  if (head_dim != 128) return false;
  const char* env = getenv("ISPA_ATTN_LEGACY");
  if (env != nullptr && env[0] == '1') return false;
  int n_local = 0;
  const int T = attn_tiles(a.r, &n_local);
  const int64_t q_tiles = (a.n_q + kAttnBq - 1) / kAttnBq;
  const int64_t n_work = q_tiles * a.n_heads;
  // the kernel's work-decomposition arithmetic is 32-bit
  if ((int64_t)T * n_work >= ((int64_t)1 << 31)) return false;
  if (a.split.n_seg > 0 && (double)a.split.units * (double)(a.split.n_seg + 1) >= 4294967295.0) return false;
  if ((int64_t)a.n_heads * a.n_q >= ((int64_t)1 << 31)) return false;
  if (a.ld * 4 >= ((int64_t)1 << 24)) return false;
  for (int i = 0; i < a.r.n_total; ++i)
    if (a.r.end[i] >= ((int64_t)1 << 31)) return false;
  return fast_function() != nullptr;
}

hipError_t launch_attn_fast(const AttnArgs& a, bool fold, hipStream_t stream) {
  hipFunction_t fn = fast_function();
  if (fn == nullptr) return hipErrorNotFound;
  int n_local = 0;
  const int T = attn_tiles(a.r, &n_local);
  const int q_tiles = (a.n_q + kAttnBq - 1) / kAttnBq;
  const int n_work = q_tiles * a.n_heads;
  const int n_log = a.split.n_seg > 0 ? a.split.n_seg : n_work;
  const int per_xcd = (n_log + 7) / 8;
  AttnFastArgs p;
  memset(&p, 0, sizeof(p));
  p.q = a.q;
  p.k = a.k;
  p.v = a.v;
  p.out = a.out;
  p.lse = a.lse;
  p.out_local = a.out_local;
  p.lse_local = a.lse_local;
  p.part_o = a.split.part_o;
  p.part_lse = a.split.part_lse;
  p.units = (uint32_t)a.split.units;
  p.ld = (int32_t)a.ld;
  p.n_q = a.n_q;
  p.q_tiles = q_tiles;
  p.n_tiles = T;
  p.n_tiles_local = n_local;
  p.n_seg = a.split.n_seg;
  p.max_pieces = a.split.max_pieces;
  p.per_xcd = per_xcd;
  p.n_log = n_log;
  const int nt0 = (int)((a.r.end[0] - a.r.begin[0] + 63) / 64);
  const int nt1 = a.r.n_total > 1 ? (int)((a.r.end[1] - a.r.begin[1] + 63) / 64) : 0;
  p.b0 = (int32_t)a.r.begin[0];
  p.e0 = (int32_t)a.r.end[0];
  p.b1 = a.r.n_total > 1 ? (int32_t)a.r.begin[1] : 0;
  p.e1 = a.r.n_total > 1 ? (int32_t)a.r.end[1] : 0;
  p.b2 = a.r.n_total > 2 ? (int32_t)a.r.begin[2] : 0;
  p.e2 = a.r.n_total > 2 ? (int32_t)a.r.end[2] : 0;
  p.tb1 = a.r.n_total > 1 ? nt0 : INT_MAX;
  p.tb2 = a.r.n_total > 2 ? nt0 + nt1 : INT_MAX;
  p.scale = a.scale;
  p.scale_log2 = a.scale_log2;
  p.lazy = 8.0f / a.scale_log2;
  p.dual = a.out_local != nullptr ? 1 : 0;
  p.neg_scale_log2 = -a.scale_log2;
  p.ld2 = (int32_t)(a.ld * 2);
  p.ld4 = (int32_t)(a.ld * 4);
  p.ctr = fold ? a.split.ctr : nullptr;
  size_t size = sizeof(p);
  void* config[] = {HIP_LAUNCH_PARAM_BUFFER_POINTER, &p, HIP_LAUNCH_PARAM_BUFFER_SIZE, &size, HIP_LAUNCH_PARAM_END};
  return hipModuleLaunchKernel(fn, (unsigned)(per_xcd * 8), 1, 1, 256, 1, 1, 0, stream, nullptr, config);
}

}  // namespace ispa
