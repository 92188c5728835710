// Internal declarations shared by the translation units of libkvra (not installed).
#ifndef KVRA_INTERNAL_H
#define KVRA_INTERNAL_H

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "kvra.h"

namespace kvra {

int launch_append_kv(const void* k_in, const void* v_in, void* q_inout, void* k_cache, void* v_cache,
                     int64_t prefix_len, int64_t chunk_len, int n_q_heads, int n_kv_heads, int head_dim,
                     float rope_base, hipStream_t stream);

// base^(-2i/d), i < d/2, in fp64 (64 entries; zeros before the first base > 0): the calling thread's, until its next call.
const double* rope_frequencies(float rope_base, int head_dim);

// The kernel for few rows (kvra_attn_rows.hip), `splits` workgroups per slice of 32 virtual rows.  splits > 1 needs scratch:
// attn_rows_slot_bytes(head_dim) and, zero between launches, one counter per slice (times splits for the slots).
int launch_attn_rows(const void* q, const void* k_cache, const void* v_cache, int64_t prefix_len, int64_t chunk_len,
                     int n_q_heads, int n_kv_heads, int head_dim, float scale, void* out, int splits, float* scratch,
                     int* counters, hipStream_t stream);
int64_t attn_rows_slot_bytes(int head_dim);
int64_t attn_static_scratch_bytes();   // size of the fixed scratch array kvra_chunk_attn_noalloc uses

// Launch shape of kvra_chunk_attn for a device with `cus` compute units (pure host arithmetic).
//
// Units.  A unit is one kv head x one tile of rows_per_tile query rows walked over the key tiles it can
// see (`steps` of them).  The kv heads are dealt to `groups` groups (8 = one per XCD when the head count
// and the CU count allow, else 1); every group has the same list of units, longest first, and `slots`
// persistent workgroups, one per CU.
//
// Schedule of a slot.  Round 0: slot c runs unit c - only its first head_steps key tiles if it is one of
// the `cut` longest units (cutting is considered while there are fewer than two complete rounds).  Rounds
// 1 .. rounds-1: whole units (round k, slot c: unit k * slots + c, every second round in reverse slot order
// so that long and short units add up alike).  What is left over - the tails of the cut units, then the
// units beyond the complete rounds - forms `segments` key ranges laid end to end; slot c takes the part of
// that line from (fill_seg[c], fill_off[c]) to (fill_seg[c+1], fill_off[c+1]), chosen so that all slots
// finish together.  A piece that is not a whole unit leaves its un-normalised result in the scratch; the
// piece of a unit that finishes last merges them.
constexpr int kMaxSlots = 256;
struct AttnPlan {
  int row_tiles;       // row tiles per kv head
  int rows_per_tile;   // virtual rows (token * group + head in group) per workgroup, <= 256
  int key_tile;        // keys per tile step
  int groups;
  int slots;           // per group, <= kMaxSlots
  int units;           // per group
  int rounds;
  int head_steps;      // 0 = no unit is cut
  int cut;             // units 0 .. cut-1 of the first round stop after head_steps key tiles
  int segments;
  int gangs;           // gang mode: gangs of filler slots per group (0: the line of segments is shared out evenly)
  int gang_heads;      // gang mode: heads per gang slot
  int steps_per_slot;  // planned tile steps (plus the per-piece allowance) of the busiest slot
  int partial_pieces;  // pieces (all groups) that go through the scratch
  int scratch_slots;   // partial-result slots the launch may touch (all groups)
  unsigned fill_seg[kMaxSlots + 1];
  unsigned fill_off[kMaxSlots + 1];
};
// Scratch that a launch meets through: partial results, and counters that are zero between launches (put back by whoever counts).
struct SharedScratch {
  float* data = nullptr;
  int64_t bytes = 0;
  int* counters = nullptr;
  int n_counters = 0;
};
// A kvra_chunk_attn launch, decided (and allowed, its scratch allocated) but not yet enqueued.
struct AttnLaunch {
  AttnPlan plan;
  int splits;              // 0: the tiled kernel with `plan`; else the one for few rows with so many workgroups per slice
  SharedScratch scratch;   // null if the launch does not use any; where it does, so may what the same call enqueues around it
};
int prepare_chunk_attn(int64_t prefix_len, int64_t chunk_len, int n_q_heads, int n_kv_heads, int head_dim, hipStream_t stream,
                       bool static_scratch_only, AttnLaunch* launch);
int launch_chunk_attn(const AttnLaunch& launch, const void* q, const void* k_cache, const void* v_cache,
                      int64_t prefix_len, int64_t chunk_len, int n_q_heads, int n_kv_heads, int head_dim,
                      float scale, void* out, hipStream_t stream);
int64_t attn_partial_bytes(int head_dim);   // scratch bytes per partial-result slot
int64_t attn_counter_bytes();               // scratch bytes of the merge counters, behind the slots
int plan_chunk_attn(int64_t prefix_len, int64_t chunk_len, int n_q_heads, int n_kv_heads, int head_dim,
                    int cus, bool scratch_available, AttnPlan* plan);
// Which kernel the launch gets: 0 = the tiled one with that plan, else the one for few rows with so many workgroups per slice.
int attn_row_splits(int64_t prefix_len, int64_t chunk_len, int n_q_heads, int n_kv_heads, int head_dim, int cus, int* splits);
// Every piece of the launch as kPieceRecordInts ints: workgroup, kv head, row tile, first key tile, end key
// tile, key tiles of the unit, partial-result slot (-1: whole unit), pieces the merge of its unit reads,
// whether its own slot is among them, merge counter (-1: none).
constexpr int kPieceRecordInts = 10;
int list_chunk_attn_pieces(int64_t prefix_len, int64_t chunk_len, int n_q_heads, int n_kv_heads, int head_dim,
                           int cus, int32_t* records, int64_t capacity, int64_t* count_out);

// out[m, n_out] = x[m, k] . w[n_out, k]^T (+ residual), or silu(x . w^T) * (x . w2^T) when w2 is given.
// With `shared`, launches of few tiles may share out k over workgroups that meet through that scratch.
// The n_out output columns are split over n_seg (1..3) dense matrices of seg_cols[s] columns each.
int launch_linear(const void* x, const void* w, const void* w2, const void* residual,
                  void* const* out, const int* seg_cols, int n_seg,
                  int64_t m, int64_t n_out, int64_t k, hipStream_t stream, const SharedScratch* shared = nullptr);
// The first half of a layer's attention block: norm, projection onto `out` (Q, rows of the K cache, rows of the V cache), Q and
// K rotated (rope_base > 0) for positions from `position` on.  h [m, k] and angles [m][head_dim] (cos of a token's head_dim / 2
// angles, then their sin) are workspace that may or may not be used.
int launch_norm_qkv_append(const void* x, const void* gain, float eps, void* h, float* angles, const void* wqkv, void* const* out,
                           const int* seg_cols, int64_t position, float rope_base, int head_dim, int64_t m, int64_t k,
                           hipStream_t stream);
// Norm, then silu(. w_gate^T) * (. w_up^T); h [m, k] as above.
int launch_norm_swiglu(const void* x, const void* gain, float eps, void* h, const void* w_gate, const void* w_up, void* out,
                       int64_t m, int64_t n_out, int64_t k, hipStream_t stream);

// Which kernel and tile such a launch gets (dual: with w2): weight rows (dual: of both weights) x tokens of a workgroup's tile,
// depth of a k stage (0: the direct kernel for few tokens, which has none), tiles the busiest workgroup walks.
struct LinearPlan {
  int tile_rows, tile_tokens, tile_k, rounds;
};
int linear_plan(int64_t m, int64_t n_out, int64_t k, bool dual, LinearPlan* plan);

int launch_rms_norm(const void* x, const void* gain, void* y, int64_t rows, int hidden, float eps,
                    hipStream_t stream);
// The same, and the rotary angles of the rows' tokens (positions from `position` on) as launch_norm_qkv_append has them.
int launch_rms_norm_angles(const void* x, const void* gain, void* y, int64_t rows, int hidden, float eps, int64_t position,
                           int head_dim, float rope_base, float* angles, hipStream_t stream);
int rms_norm_max_hidden();

// More than 64 KiB of dynamic LDS has to be granted per kernel and device.  A thread remembers what it has asked for (the
// request goes through the runtime's locks: 0.3 of a 3.5 us call).
inline bool grant_lds(const void* kernel, unsigned bytes) {
  struct Grant {
    const void* kernel;
    int device;
    unsigned bytes;
  };
  constexpr int kGrants = 64;   // more than there are such kernels
  static thread_local Grant grants[kGrants] = {};
  static thread_local int next = 0;
  int device = 0;
  if (hipGetDevice(&device) != hipSuccess) return false;
  for (const Grant& g : grants)
    if (g.kernel == kernel && g.device == device && g.bytes >= bytes) return true;
  if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(bytes)) != hipSuccess) return false;
  grants[next] = Grant{kernel, device, bytes};
  next = (next + 1) % kGrants;
  return true;
}

// Launch with the runtime's own status as the result.  (hipGetLastError would also pick up
// stale, unrelated codes that other users of the runtime in this thread left behind.)
template <typename Args>
inline int launch_kernel(void (*kernel)(Args), dim3 grid, dim3 block, Args& args, hipStream_t stream,
                         unsigned dynamic_lds_bytes = 0) {
  if (dynamic_lds_bytes > 64 * 1024 && !grant_lds(reinterpret_cast<const void*>(kernel), dynamic_lds_bytes)) return KVRA_ELAUNCH;
  void* params[] = {static_cast<void*>(&args)};
  const hipError_t e = hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, params,
                                       dynamic_lds_bytes, stream);
  return e == hipSuccess ? KVRA_OK : KVRA_ELAUNCH;
}

}  // namespace kvra

#endif
