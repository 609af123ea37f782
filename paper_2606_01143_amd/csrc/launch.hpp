// Host-side launchers of the gfx950 kernels and the per-kernel event timer.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "common.hpp"

namespace spr {

// --- per-kernel timing (enabled through spr_profile_enable) -------------
bool profile_enabled(const char* kernel);
void profile_record(const char* kernel, hipEvent_t begin, hipEvent_t end);
hipEvent_t profile_event();  // from a pool owned by the profiler

// Brackets one kernel launch with two events on `stream` while profiling
// is enabled; a no-op otherwise.
class ProfileScope {
 public:
  ProfileScope(const char* kernel, hipStream_t stream) : kernel_(kernel), stream_(stream) {
    if (profile_enabled(kernel)) {
      begin_ = profile_event();
      end_ = profile_event();
      if (begin_ && end_) hipEventRecord(begin_, stream_);
    }
  }
  ~ProfileScope() {
    if (begin_ && end_) {
      hipEventRecord(end_, stream_);
      profile_record(kernel_, begin_, end_);
    }
  }
  ProfileScope(const ProfileScope&) = delete;
  ProfileScope& operator=(const ProfileScope&) = delete;

 private:
  const char* kernel_;
  hipStream_t stream_;
  hipEvent_t begin_ = nullptr;
  hipEvent_t end_ = nullptr;
};

// --- fp32 storage path (kernels_f32.hip) --------------------------------
hipError_t launch_fwd_f32(const AttnArgs& a, int head_dim, int n_z, hipStream_t st);
hipError_t launch_bwd_f32(const AttnArgs& a, int head_dim, int n_qz, hipStream_t st);

// --- bf16 storage path, MFMA (kernels_bf16_fwd.hip, kernels_bf16_bwd.hip) --
hipError_t launch_fwd_bf16(const AttnArgs& a, int head_dim, int n_z, hipStream_t st);
hipError_t launch_fwd_bf16_wide(const AttnArgs& a, int head_dim, int n_z, hipStream_t st);
int fwd_bf16_wide_block_q();
hipError_t launch_fwd_bf16_pack(const AttnArgs& a, int head_dim, int n_z, hipStream_t st);
hipError_t launch_bwd_bf16(const AttnArgs& a, int head_dim, int n_qz, bool deterministic,
                           hipStream_t st);
// Row-tile sizes the launchers expect in AttnArgs (q tiles / k tiles).
int fwd_bf16_block_q();
// key splits of the bf16 suffix forward for n_row_blocks (row tile, q head,
// suffix) blocks and a prefix of prefix_len keys
int fwd_bf16_split(int n_row_blocks, int prefix_len);
// row tiles per suffix and kv head of the suffix forward's packed-row form,
// taken where that is at most 3/4 of the one-head form's (short suffixes, or
// lengths just past a multiple of 128); 0: the one-head form
long fwd_bf16_pack_tiles(int hq, int hkv, int max_len);
// its key splits: 1, or the prefix key ranges plus one for the suffixes' own;
// 0: the one-head form is the faster one
int fwd_bf16_pack_split(int hq, int hkv, int n_mb, int max_len, int prefix_len);
int bwd_bf16_block_k();
// key-outer role alone with six wave pairs (192 keys) per workgroup, one
// workgroup per CU, for the prefix backward of long prefixes (default mode)
hipError_t launch_bwd_bf16_kv_wide(const AttnArgs& a, int head_dim, hipStream_t st);
int bwd_bf16_kv_wide_block_k();
int bwd_bf16_kv_wide_slots();
// key splits of the bf16 suffix backward's query-outer role for
// n_row_blocks (row tile, q head, suffix) blocks that each sweep
// n_key_tiles key tiles
int bwd_bf16_qsplit(int n_row_blocks, int n_key_tiles);
int bwd_bf16_kvsplit(long kv_tiles, long max_tiles, bool kv_alone, int slots = 512);
int bwd_bf16_block_q();

// The suffix backward's key-outer-only launch with filled rounds (the prefix
// tiles' row shares first, whole suffix tiles after them), for sizes the host
// knows; whether it pays depends on the microbatch's rows in all, which the
// host knows of packed suffixes only.
constexpr long kKvWideMinSteps = 32768;                    // see kv_wide
constexpr long kWideShareSteps = 128, kWideTileCost = 8;  // steps; a tile's prologue and epilogue
struct FillRule {
  long prefix_tiles, group, hkv;  // prefix key tiles over all kv heads, q heads per kv head, kv heads
  long n, max_len, causal;        // suffixes, the longest, its key tiles' steps of one kv head
  long shares, slots;             // row shares of a prefix tile, workgroups resident at once
  long head_dim;
};
// The launch's time, in steps per CU: the rounds of shares; suffix tiles in
// the slots the last round leaves and after it; never less than the longest
// suffix tile begun after the full rounds, nor than the even spread plus
// half of it.  Against the even spread of the useful work it may take 1.25 times
// that; 1.44 times on up to 13 prefix tiles per kv head (2496 keys), 1.6 times on
// up to 6 and 1.8 times at d = 64, where the shared launch is slower by as much,
// and 1.6 times for suffixes of equal length (all 77 measured gained, 1.02 to
// 1.8).  Shares of fewer than 100 steps do not pay.  Integers only: host and
// device agree.
__host__ __device__ inline bool fill_pays(const FillRule& r, long rows) {
  const long steps = r.group * ((rows + 31) / 32), whole = steps / r.shares;
  const long share = (steps + r.shares - 1) / r.shares + kWideTileCost, tiles = r.prefix_tiles * r.shares;
  const long longest = r.group * ((r.max_len + 31) / 32);
  const long suffix = r.causal * (256 * rows / r.max_len) / 256 * r.hkv;
  const long work = suffix + (rows / 192 + r.n) * r.hkv * kWideTileCost;
  const long full = tiles / r.slots * share, last = tiles % r.slots;
  const long rest = (last * share + work) / r.slots, after = full + longest + kWideTileCost;
  const long spread = (tiles * share + work) / r.slots + (longest + kWideTileCost) / 2;
  long t = full + (last > 0 && rest < share ? share : rest);
  if (t < after) t = after;
  if (t < spread) t = spread;
  const long useful = r.prefix_tiles * steps + suffix;
  const long limit = rows == r.n * r.max_len        ? 160
                     : r.head_dim == 64             ? 180
                     : r.prefix_tiles <= 6 * r.hkv  ? 160
                     : r.prefix_tiles <= 13 * r.hkv ? 144
                                                    : 125;
  return whole >= 100 && 100 * t * r.slots <= limit * useful;
}
// where the rows are known on the device only: *out = fill_pays(rule, rows) as
// 0 or 1, written by the launch that adds up the lengths (null: not asked for)
struct FillGate {
  FillRule rule;
  int32_t* out;
};

int f32_block_q();
int f32_block_k();
// row shares of Phase C's key-outer role in fp32 storage (1 + group / 2 at most)
int f32_kvsplit(long kv_tiles, long max_tiles, int group);

// --- auxiliary kernels (kernels_aux.hip) ----------------------------------
// dd[row * hq + h] = sum_d dO[row,h,d] * O[row,h,d] and
// lse2[row * hq + h] = lse[row * hq + h] * log2(e) for rows [0, rows), or,
// when cu != nullptr, for the rows cu[seq] .. cu[seq+1]-1 of one packed
// suffix (rows then bounds their count, total_rows is the buffers' row
// count the offsets are clamped to); dO == nullptr gives dd = 0.
hipError_t launch_row_dot(int dtype, const void* dO, const void* O, int rows, int total_rows,
                          const int32_t* cu, int seq, int hq, int head_dim, float* dd,
                          const float* lse, float* lse2, hipStream_t st);
hipError_t launch_fill_zero(float* p, size_t n, hipStream_t st);
hipError_t launch_fill_zero2(float* p, float* q, size_t n, hipStream_t st);
// out = acc * scale (+ add when add != nullptr), converted to `dtype`
hipError_t launch_convert(int dtype, const float* acc, float scale, const float* add,
                          void* out, size_t n, hipStream_t st);
// dst += src
hipError_t launch_accumulate(float* dst, const float* src, size_t n, hipStream_t st);
// padded suffix layout: cu/lens_c from device lengths, and row gather
// (padded -> packed) or scatter (packed -> padded, padding rows zeroed)
hipError_t launch_seq_offsets(const int32_t* lens, int n, int s_max, int32_t* cu, int32_t* lens_c,
                              hipStream_t st, const FillGate& gate = {});
constexpr int kMaxRowMoves = 6;
struct RowMove {
  const void* src;
  void* dst;
  size_t row_bytes;  // a multiple of 4
};
// few suffixes: the move kernels derive the offsets (and a gather's gate) from
// `lens` themselves; many: they must come from launch_seq_offsets first
bool rows_move_needs_offsets(int n);
hipError_t launch_rows_move(bool gather, const RowMove* moves, int count, const int32_t* lens,
                            const int32_t* cu, const int32_t* lens_c, int n, int s_max, hipStream_t st,
                            const FillGate& gate = {});

// decoder-layer token-wise operations (kernels_layer.hip)
hipError_t launch_rmsnorm_fwd(int rows, int width, float eps, const void* x, void* y, float* rstd,
                              hipStream_t st);
hipError_t launch_rmsnorm_bwd(int rows, int width, const void* x, const float* rstd, const void* dy,
                              const void* add, void* dx, hipStream_t st);
hipError_t launch_rope(int tokens, int heads, int d, int pos0, double theta, const void* x, void* y,
                       bool inverse, hipStream_t st);
hipError_t launch_swiglu_fwd(long n, const void* g, const void* u, void* m, hipStream_t st);
hipError_t launch_swiglu_bwd(long n, const void* g, const void* u, const void* dm, void* dg, void* du,
                             hipStream_t st);

hipError_t launch_grad_accumulate(long n, const void* src, float* dst, bool overwrite, hipStream_t st);

// MoE router aux-loss accounting (kernels_moe.hip).  Statistics layout:
// int64 count[E], double mass[E], int64 total, int64 invalid.
int moe_blocks(int n_tokens);
size_t moe_workspace_bytes(int E, int n_tokens);
hipError_t launch_moe_accumulate(const float* p, const int* r, int n, int E, int k, int mult,
                                 const int* mu, void* stats, void* ws, hipStream_t st);
hipError_t launch_moe_loss(const void* stats, int E, int k, double coef, double* f, double* pe,
                           double* loss, hipStream_t st);
hipError_t launch_moe_grad(const void* stats, int E, int k, double scale, int n, int mult,
                           const int* mu, float* dp, hipStream_t st);

}  // namespace spr
