// Linear layers of the decoder layer a KV-Runahead process runs around its attention block
// (App. C listing: q/k/v projections before, output projection after the attention; the SwiGLU MLP
// of the LLaMA models of Sec. 5) for gfx950:  out[m, n] = sum_k x[m, k] * w[n, k], bf16 in, fp32
// accumulate, bf16 out, with four fused epilogues (plain / + residual / silu(gate) * up / rotary embedding of Q and K).
//
// Orientation.  Both operands are contiguous along k, which is exactly what the two register
// operands of v_mfma_f32_16x16x32_bf16 want (lane (r, kg) holds 8 consecutive k of row r).  The
// weight rows go to the A side and the token rows to the B side, i.e. the kernel forms the
// TRANSPOSED tile out^T[n, m]: in the 16x16 accumulator layout a lane then owns one token and
// 4 consecutive n.  (The 32x32x16 form of the same work holds a 10 % lower rate on this power-managed chip: a loop of nothing
// but MFMAs on N(0,1) operands, all CUs, 1821 against 2028 TFLOP/s - half as deep, it writes its sums twice as often.)
//
// Pipeline of a workgroup.  Both operand tiles come by LDS-direct loads into a ring of k stages, a stage 64 deep (a whole
// 128-byte line of every row: with 32-deep stages each line came in two halves, -10 %); the ring is refilled as the waves
// walk through it, across tiles when a workgroup has more than one.  Everything that is not an MFMA is placed between
// MFMAs: operand reads one step ahead, the loads of the stage that replaces the one just read (2 to 8 per wave and stage;
// in a burst they block the wave that issues them for hundreds of cycles), and the one barrier per stage sits inside the
// MFMA stream, where every wave already holds the operands of the next few MFMAs.
// 8192^3: 974 -> 777 us (1416 TFLOP/s), 11584 x 12288 x 4096: 1010 -> 912 us; what remains is power: with the loads and
// operand reads taken out the same loop is 20 % faster at the same MFMA count.
#include "kvra_rope_device.h"

#include <algorithm>
#include <type_traits>

namespace kvra {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void;

struct OutSegment {
  __bf16* ptr;   // dense [m, width] matrix that receives output columns [first, end)
  int end;       // one past the last output column of this segment
  int first;
  int ld;        // row stride of ptr in elements
};

struct GemmArgs {
  const __bf16* x;     // [m, k]
  const __bf16* w;     // [rows, k]
  const __bf16* w2;    // dual mode: second weight [rows, k]; else null
  const __bf16* res;   // residual [m, seg[0].ld] or null (single segment only)
  OutSegment seg[3];
  int n_seg;
  int m;
  int n;               // weight rows walked: rows, or 2 * rows in dual mode (blocks of GemmTile::DUAL_ROWS alternate w / w2)
  int k;
  int tiles_n, tiles_m;
  int dual;
  // Q/K/V projection that also rotates and appends (segments: Q, cache rows of K, cache rows of V): head size, else 0.  The
  // weight rows are walked in blocks of GemmTile::ROPE_ROWS alternating between the lower and the upper half of a head.
  int rope;
  int rotated;             // output columns [0, rotated) are rotated (those of Q and K; 0: none)
  const float* angles;     // [m][rope]: cos of a token's rope / 2 angles, then their sin
  // Launches whose tiles leave CUs idle: `splits` workgroups share the k of a tile and meet through the scratch.
  int stagger;             // stages between the starts of neighbouring weight tiles (0: all start at the first)
  int splits;
  float* scratch;          // a tile's sums per workgroup
  int* counters;           // pieces counted so far, one per tile; all zero between launches
};

// Tile of a workgroup: TN weight rows x TM tokens, k in stages of TK through a ring of ST LDS slots;
// WN x WM waves over the tile, WK waves over the k of a stage (their sums meet in LDS at the end).
template <int TN_, int TM_, int TK_, int ST_, int WN_, int WM_, int WK_, int PER_SIMD_, bool WHOLE_ = false>
struct GemmTile {
  static constexpr int TN = TN_, TM = TM_, TK = TK_, ST = ST_, WN = WN_, WM = WM_, WK = WK_;
  static constexpr bool WHOLE = WHOLE_;                    // operands of a whole stage are read ahead (see the kernel)
  static constexpr int DUAL_ROWS = TN / WN >= 64 ? 32 : 16;   // dual mode: rows of a weight that sit side by side in the tile
  static constexpr int ROPE_ROWS = TN / WN % 64 == 0 ? 32 : 16;   // rope mode: rows of a half that sit side by side
  static constexpr int NW = WN * WM * WK, THREADS = 64 * NW;
  static constexpr int PER_SIMD = PER_SIMD_;               // waves per SIMD the register budget is cut for
  static constexpr int NB = TN / WN / 16, MB = TM / WM / 16;   // 16 x 16 blocks of a wave
  static constexpr int PR = TK / 8;                        // 16-byte pieces per LDS row
  static constexpr int RPL = 64 / PR;                      // rows one wave load moves
  static constexpr int WLOADS = TN / RPL, LOADS = (TN + TM) / RPL;
  static constexpr int L = (LOADS + NW - 1) / NW;          // wave loads per stage and wave (the last may repeat one)
  static constexpr int STAGE = (TN + TM) * TK * 2;
  static constexpr int KPW = TK / 32 / WK;                 // 32-deep contraction steps of a wave per stage
  static constexpr int REDUCE = (WK - 1) * WN * WM * NB * MB * 4 * 64 * 4;
  static constexpr int LDS = ST * STAGE + REDUCE;
  static_assert(WHOLE || (KPW % 2 == 0 && KPW >= 2), "two fragment sets alternate");
  static_assert(TN % (32 * WN) == 0 && TM % (16 * WM) == 0 && LDS <= 160 * 1024 && (ST - 1) * L < 64, "");
};

// 64 lanes x 16 bytes -> 1 KiB of consecutive LDS (lane l lands at +16 l); inline assembly so that completion can be
// awaited by hand with s_waitcnt vmcnt(n) instead of a full drain per load.  With on_mask = 0 no lane is enabled and
// nothing moves: no branch around it, so that it can sit between MFMAs.  Between a vector instruction that writes a scalar
// register (a spilled address coming back) and a memory instruction that reads it five wait states have to lie, and the compiler
// does not see that one stands in here: two scalar moves and s_nop 2 make them up (no slower: 8192^3 777 and 767 us).
__device__ __forceinline__ void gemm_lds_dma16_if(unsigned long long on_mask, const void* uniform_base,
                                                  unsigned lane_byte_off, unsigned lds_byte_addr) {
  unsigned long long saved;
  asm volatile("s_mov_b32 m0, %3\n\ts_and_saveexec_b64 %0, %4\n\ts_nop 2\n\tglobal_load_lds_dwordx4 %1, %2\n\ts_mov_b64 exec, %0"
               : "=&s"(saved)
               : "v"(lane_byte_off), "s"(uniform_base), "s"(lds_byte_addr), "s"(on_mask)
               : "memory", "m0", "scc");
}

template <int N>
__device__ __forceinline__ void wait_loads() {   // at most N vector-memory operations of this wave outstanding
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);
}

// Two accumulator blocks of 16 columns each: a lane holds, for token lane % 16, columns 4 g .. 4 g + 3 of both (g = its
// 16-lane row).  Trading registers between odd and even rows leaves 8 consecutive columns of the 32 in a lane, from
// 16 (g % 2) + 8 (g / 2): a store then covers 16 tokens x 64 consecutive bytes in pieces of 16.
__device__ __forceinline__ void gather_columns(const f32x4& lo, const f32x4& hi, float (&v)[8]) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(lo[e]), __float_as_uint(hi[e]), false, false);
    v[e] = __uint_as_float(r[0]);
    v[4 + e] = __uint_as_float(r[1]);
  }
}

template <class T, bool ROPE, bool SPLIT, bool STAGGER>
__global__ __launch_bounds__(T::THREADS, T::PER_SIMD) void linear_kernel(GemmArgs a) {
  static_assert(!SPLIT || T::WK == 1, "either the waves of a workgroup share k or workgroups do");
  constexpr int NB = T::NB, MB = T::MB, L = T::L, ST = T::ST, TK = T::TK, KPW = T::KPW, PR = T::PR;
  extern __shared__ u32x4 smem[];
  char* const lds = reinterpret_cast<char*>(smem);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, kg = lane >> 4;
  const int wn = wave % T::WN, wm = (wave / T::WN) % T::WM, wk = wave / (T::WN * T::WM);

  // Workgroup -> tiles.  Workgroup ids go round-robin over the 8 XCDs; each XCD takes a contiguous
  // run of the tile order "bands of 4 weight tiles, token tiles inside a band, weight tile
  // fastest", so that the workgroups an XCD runs together share few weight and token tiles in its L2.
  // (Split: the run goes over all tiles of the first share of k, then of the second, ..., and a workgroup has one piece.)
  const int tiles = a.tiles_n * a.tiles_m;
  const int total = SPLIT ? tiles * a.splits : tiles;
  const int per = (total + 7) >> 3;
  const int t_step = gridDim.x >> 3;
  const int t_mine = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  const int t_last = min(((blockIdx.x & 7) + 1) * per, total);
  if (t_mine >= t_last) return;   // whole workgroup leaves before any barrier
  const int share = SPLIT ? t_mine / tiles : 0;
  const int t_first = SPLIT ? t_mine - share * tiles : t_mine, t_end = SPLIT ? t_first + 1 : t_last;
  auto place = [&](int t, int* n0, int* m0) {
    const int band = t / (4 * a.tiles_m);
    const int width = min(4, a.tiles_n - 4 * band);
    const int within = t - band * 4 * a.tiles_m;
    *m0 = (within / width) * T::TM;
    *n0 = (4 * band + within % width) * T::TN;
  };
  const int KT_all = a.k / TK;
  const int kt_first = SPLIT ? static_cast<int>(static_cast<long long>(KT_all) * share / a.splits) : 0;
  const int KT = SPLIT ? static_cast<int>(static_cast<long long>(KT_all) * (share + 1) / a.splits) - kt_first : KT_all;
  int stages_left = ((t_end - t_first + t_step - 1) / t_step) * KT;   // not yet computed
  int loads_left = stages_left;                                       // not yet sent for

  // ---- global -> LDS staging -----------------------------------------------------------------
  // A stage is the weight rows, then the token rows, PR pieces of 16 bytes each.  The lane that owns (row, slot)
  // fetches column piece slot ^ f(row), f(row) = row / (16 / PR) mod PR, so that the operand reads below (16 rows
  // of one column piece per quarter wave) spread over all banks.  Rows past the end of a matrix repeat its last row.
  const int ld_row = lane / PR;
  const int ld_piece = (lane % PR) ^ (((wave * T::RPL + ld_row) / (16 / PR)) % PR);
  constexpr int PERIOD = 16 / PR * PR;   // rows after which f repeats
  static_assert(T::NW * T::RPL % PERIOD == 0 && T::TN % PERIOD == 0 && (T::RPL % PERIOD == 0 || T::LOADS % T::NW == 0),
                "f(row) must not depend on which of a wave's loads it is");
  unsigned off[L];
  const __bf16* src[L];
  // Rope mode with three units of 32 rows (16 of a lower half, 16 of an upper) to a wave: the second wave takes its last two
  // units first, so that either has two that are neighbours in a head, and then one.
  auto rope_unit = [](int u) -> int { return u < 3 ? u : u == 5 ? 3 : u + 1; };
  auto aim = [&](int t) {
    int n0, m0;
    place(t, &n0, &m0);
#pragma unroll
    for (int i = 0; i < L; ++i) {
      const int idx = T::LOADS % T::NW == 0 ? i * T::NW + wave : min(i * T::NW + wave, T::LOADS - 1);
      int row;
      if (T::WLOADS % T::NW == 0 ? i * T::NW < T::WLOADS : idx < T::WLOADS) {
        const int first = min(n0 + idx * T::RPL, a.n - 1);   // uniform
        row = min(n0 + idx * T::RPL + ld_row, a.n - 1);
        src[i] = a.w;
        if (ROPE) {                                          // blocks of rows alternate between the halves of a head
          constexpr int RR = T::ROPE_ROWS;
          if constexpr (NB == 6) row = min(n0 + rope_unit(idx * T::RPL / 32) * 32 + idx * T::RPL % 32 + ld_row, a.n - 1);
          const int in_head = row & (a.rope - 1);
          row += (in_head / (2 * RR) * RR + (in_head / RR % 2) * (a.rope / 2) + in_head % RR) - in_head;
        } else if (a.dual) {                                 // or between the two weights
          constexpr int DR = T::DUAL_ROWS;
          if ((first / DR) & 1) src[i] = a.w2;
          row = row / (2 * DR) * DR + row % DR;
        }
      } else {
        row = min(m0 + (idx - T::WLOADS) * T::RPL + ld_row, a.m - 1);
        src[i] = a.x;
      }
      off[i] = 2u * (static_cast<unsigned>(row) * static_cast<unsigned>(a.k) + 8u * ld_piece);
    }
  };
  const unsigned lds0 = static_cast<unsigned>(reinterpret_cast<uintptr_t>((lds_void*)smem));
  // STAGGER: the walk along k starts somewhere else for every weight tile and wraps around (a form of its own: the two extra scalar
  // values cost the others 0.3 %)
  auto k_start = [&](int t) __attribute__((always_inline)) -> int {
    if constexpr (!STAGGER) return 0;
    int n0, m0;
    place(t, &n0, &m0);
    return n0 / T::TN * a.stagger % KT;
  };
  int load_t = t_first, load_from = k_start(t_first), load_kt = load_from, load_end = KT;
  auto send = [&](int i, unsigned slot_base, unsigned long long on) __attribute__((always_inline)) {
    const int idx = T::LOADS % T::NW == 0 ? i * T::NW + wave : min(i * T::NW + wave, T::LOADS - 1);
    gemm_lds_dma16_if(on, src[i] + static_cast<long long>(SPLIT ? kt_first + load_kt : load_kt) * TK, off[i], slot_base + idx * 1024);
  };
  auto sent = [&]() {   // the stage under load_t / load_kt is on its way: on to the next one
    --loads_left;
    if (++load_kt == (STAGGER ? load_end : KT)) {
      if (STAGGER && load_end == KT && load_from != 0) {   // wraps around
        load_kt = 0;
        load_end = load_from;
      } else {
        load_kt = 0;
        load_t += t_step;
        if (load_t < t_end) {
          aim(load_t);
          load_from = load_kt = k_start(load_t);
          load_end = KT;
        }
      }
    }
  };

  // ---- operand reads -------------------------------------------------------------------------
  const int sw = (r16 / (16 / PR)) % PR;   // f(row) of the rows this lane reads (multiples of 16 apart)
  static_assert(16 % PERIOD == 0, "blocks of 16 rows share the swizzle");
  unsigned wofs[KPW], xofs[KPW];
#pragma unroll
  for (int j = 0; j < KPW; ++j) {
    const unsigned piece = static_cast<unsigned>((4 * (wk * KPW + j) + kg) ^ sw);
    wofs[j] = static_cast<unsigned>(wn * (T::TN / T::WN) + r16) * (TK * 2) + piece * 16;
    xofs[j] = static_cast<unsigned>(T::TN + wm * (T::TM / T::WM) + r16) * (TK * 2) + piece * 16;
  }
  constexpr int N = NB * MB, R = NB + MB;   // MFMAs and operand reads of a step; MFMA i: mb = i / NB, nb = i % NB
  // The weight fragments of a contraction step serve all its MFMAs and are double-buffered.  A token fragment serves NB
  // consecutive ones; in a long step it is replaced by the next step's as soon as they are issued, in a short one,
  // where that would be too late for the next step, it is double-buffered too.
  constexpr int XSETS = N <= 16 ? 2 : 1;
  bf16x8 fw[T::WHOLE ? 1 : 2][NB], fx[T::WHOLE ? 1 : XSETS][MB];
  // Small tiles have too few MFMAs in a step to cover the way to LDS and back; there the operands of a whole stage are
  // read, right after the barrier, while the MFMAs of the stage before run from registers.
  bf16x8 gw[T::WHOLE ? 2 : 1][KPW][NB], gx[T::WHOLE ? 2 : 1][KPW][MB];
  // operand read r of contraction step j, in the order the MFMAs want them: w0 x0 w1 .. x1 x2 ..
  auto fetch = [&](auto set_tag, unsigned slot_ofs, int j, int r) __attribute__((always_inline)) {
    constexpr int S = decltype(set_tag)::value;
    if (r == 0 || (r >= 2 && r <= NB)) {
      const int b = r == 0 ? 0 : r - 1;
      fw[S][b] = *reinterpret_cast<const bf16x8*>(lds + slot_ofs + wofs[j] + b * 16 * TK * 2);
    } else {
      const int b = r == 1 ? 0 : r - NB;
      fx[S % XSETS][b] = *reinterpret_cast<const bf16x8*>(lds + slot_ofs + xofs[j] + b * 16 * TK * 2);
    }
  };
  // the MFMA after which read r of the next step is issued, spread over those from `first` on
  auto fetch_at = [](int r, int first) constexpr -> int {
    const int spread = first + r * (N - first) / R;
    if (XSETS == 2 || r == 0 || (r >= 2 && r <= NB)) return spread;
    const int free_at = ((r == 1 ? 0 : r - NB) + 1) * NB - 1;   // the register is still an operand until then
    return spread > free_at ? spread : free_at;
  };
  constexpr int BAR = N * 3 / 8;   // MFMA of a stage's last step before which the waves meet

  f32x4 acc[NB][MB];

  // ---- pipeline ------------------------------------------------------------------------------
  aim(t_first);
#pragma unroll
  for (int s = 0; s < ST; ++s)
    if (loads_left > 0) {
#pragma unroll
      for (int i = 0; i < L; ++i) send(i, lds0 + s * T::STAGE, ~0ull);
      sent();
    }
  if (stages_left >= ST) wait_loads<(ST - 1) * L>();
  else wait_loads<0>();
  __syncthreads();
  unsigned slot = 0;   // byte offset of the slot the current stage sits in
  unsigned send_slot = 0;
  unsigned long long on = 0;
  auto fetch_whole = [&](auto set_tag, unsigned slot_ofs, int q) __attribute__((always_inline)) {   // read q of R * KPW
    constexpr int S = decltype(set_tag)::value;
    const int j = q / R, r = q % R;
    if (r < NB) gw[S][j][r] = *reinterpret_cast<const bf16x8*>(lds + slot_ofs + wofs[j] + r * 16 * TK * 2);
    else gx[S][j][r - NB] = *reinterpret_cast<const bf16x8*>(lds + slot_ofs + xofs[j] + (r - NB) * 16 * TK * 2);
  };
  if constexpr (T::WHOLE) {
#pragma unroll
    for (int q = 0; q < R * KPW; ++q) fetch_whole(std::integral_constant<int, 0>{}, 0, q);
  } else {
#pragma unroll
    for (int r = 0; r < R; ++r) fetch(std::integral_constant<int, 0>{}, 0, 0, r);
  }
  // one stage of the whole-stage form: its operands are in set S (or on their way there)
  auto whole_stage = [&](auto set_tag) __attribute__((always_inline)) {
    constexpr int S = decltype(set_tag)::value;
    --stages_left;
    const unsigned next = slot + T::STAGE == ST * T::STAGE ? 0 : slot + T::STAGE;
    if (stages_left >= ST - 1) wait_loads<(ST - 2) * L>();
    else wait_loads<0>();
    __syncthreads();   // the next stage has landed, and this one's slot has been read
    on = __builtin_amdgcn_ballot_w64(loads_left > 0);
    __builtin_amdgcn_sched_barrier(0);
    constexpr int M = N * KPW, Q = R * KPW;
#pragma unroll
    for (int i = 0; i < M; ++i) {
      const int j = i / N, mb = i % N / NB, nb = i % NB;
      if constexpr (T::WHOLE)
        acc[nb][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(gw[S][j][nb], gx[S][j][mb], acc[nb][mb], 0, 0, 0);
      asm volatile("" : "+v"(acc[nb][mb]));
#pragma unroll
      for (int q = 0; q < Q; ++q)
        if (q * M / Q == i) fetch_whole(std::integral_constant<int, 1 - S>{}, next, q);
#pragma unroll
      for (int d = 0; d < L; ++d)
        if (d * M / L == i) send(d, lds0 + slot, on);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (on != 0) sent();
    slot = next;
  };

  for (int t = t_first; t < t_end; t += t_step) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[nb][mb][e] = 0.0f;
    if constexpr (T::WHOLE) {
      for (int kt = 0; kt + 1 < KT; kt += 2) {
        whole_stage(std::integral_constant<int, 0>{});
        whole_stage(std::integral_constant<int, 1>{});
      }
      if (KT & 1) {
        whole_stage(std::integral_constant<int, 0>{});
#pragma unroll
        for (int j = 0; j < KPW; ++j) {
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) gw[0][j][nb] = gw[T::WHOLE ? 1 : 0][j][nb];
#pragma unroll
          for (int mb = 0; mb < MB; ++mb) gx[0][j][mb] = gx[T::WHOLE ? 1 : 0][j][mb];
        }
      }
    } else {
    for (int kt = 0; kt < KT; ++kt) {
      --stages_left;
      const unsigned next = slot + T::STAGE == ST * T::STAGE ? 0 : slot + T::STAGE;
#pragma unroll
      for (int j = 0; j < KPW; ++j) {
        const bool last = j + 1 == KPW;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < N; ++i) {
          if (last && i == BAR) {
            // The next stage has landed for this wave (all but the ST - 2 stages behind it), after the barrier
            // for every wave; and every wave holds the last operands of this stage, so its slot is free.  (After
            // the last stage of all, what is fetched below is never used.)
            if (stages_left >= ST - 1) wait_loads<(ST - 2) * L>();
            else wait_loads<0>();
            __syncthreads();
            send_slot = lds0 + slot;
            on = __builtin_amdgcn_ballot_w64(loads_left > 0);
            __builtin_amdgcn_sched_barrier(0);
          }
          const int mb = i / NB, nb = i % NB;
          acc[nb][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[j & 1][nb], fx[(j & 1) % XSETS][mb], acc[nb][mb], 0, 0, 0);
          asm volatile("" : "+v"(acc[nb][mb]));   // keeps what follows behind this MFMA
#pragma unroll
          for (int r = 0; r < R; ++r)
            if (fetch_at(r, last ? BAR : 0) == i) {
              if (last) fetch(std::integral_constant<int, 0>{}, next, 0, r);
              else if (j & 1) fetch(std::integral_constant<int, 0>{}, slot, j + 1, r);
              else fetch(std::integral_constant<int, 1>{}, slot, j + 1, r);
            }
          // the loads of a stage are spread over one contraction step's worth of MFMAs from the barrier on
#pragma unroll
          for (int d = 0; d < L; ++d) {
            if (last && BAR + d * N / L == i) send(d, send_slot, on);
            if (j == 0 && BAR + d * N / L == N + i) send(d, send_slot, on);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        if (j == 0 && on != 0) {
          sent();
          on = 0;
        }
      }
      slot = next;
    }
    }

    // ---- epilogue ----------------------------------------------------------------------------
    // register e of block (nb, mb): weight row 16 nb + 4 kg + e, token 16 mb + r16 (wave-relative)
    int n0, m0;
    place(t, &n0, &m0);
    if constexpr (T::WK > 1) {
      // the sums of the other k shares, through LDS
      float* red = reinterpret_cast<float*>(lds + ST * T::STAGE) + (wm * T::WN + wn) * (NB * MB * 4 * 64) + lane;
      constexpr int SHARE = T::WN * T::WM * NB * MB * 4 * 64;
      __syncthreads();   // the region may still be read for the tile before
      if (wk > 0) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
          for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int e = 0; e < 4; ++e) red[(wk - 1) * SHARE + ((nb * MB + mb) * 4 + e) * 64] = acc[nb][mb][e];
      }
      __syncthreads();
      if (wk > 0) continue;
#pragma unroll
      for (int s = 0; s < T::WK - 1; ++s)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
          for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[nb][mb][e] += red[s * SHARE + ((nb * MB + mb) * 4 + e) * 64];
    }
    if constexpr (SPLIT) {
      // The pieces of a tile meet as those of the attention kernel do: device-coherent stores, acknowledged before the piece
      // is counted; the piece that completes the count adds all of them in the order of their shares (its own as well, as it was
      // stored) and goes on to the epilogue.  16 bytes per lane, as many in flight as registers allow.
      constexpr int SHARE_BYTES = T::TN * T::TM * 4, COHERENT = 16;   // (the sc1 bit: past the cache of this XCD)
      const __amdgpu_buffer_rsrc_t res = __builtin_amdgcn_make_buffer_rsrc(
          reinterpret_cast<char*>(a.scratch) + static_cast<long long>(t) * a.splits * SHARE_BYTES, 0, a.splits * SHARE_BYTES, 0x00020000);
      auto slot_of = [&](int s, int nb, int mb) __attribute__((always_inline)) -> int {
        return s * SHARE_BYTES + ((nb * MB + mb) * T::THREADS + tid) * 16;
      };
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[nb][mb]), res, slot_of(share, nb, mb), 0, COHERENT);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      int* const flag = reinterpret_cast<int*>(lds);   // (nothing is staged any more)
      if (tid == 0) *flag = atomicAdd(a.counters + t, 1) == a.splits - 1 ? 1 : 0;
      __syncthreads();
      if (*flag == 0) return;
      if (tid == 0) a.counters[t] = 0;                 // ready for the next launch
      constexpr int AT_ONCE = MB == 1 ? 4 : MB == 2 ? 2 : 1, SHARES = MB >= 8 ? 2 : 4;
#pragma unroll
      for (int n1 = 0; n1 < NB; n1 += AT_ONCE) {
#pragma unroll
        for (int nb = n1; nb < n1 + AT_ONCE && nb < NB; ++nb)
#pragma unroll
          for (int mb = 0; mb < MB; ++mb) acc[nb][mb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        for (int s0 = 0; s0 < a.splits; s0 += SHARES) {
          f32x4 v[SHARES][AT_ONCE][MB];
#pragma unroll
          for (int u = 0; u < SHARES; ++u)
#pragma unroll
            for (int q = 0; q < AT_ONCE; ++q)
#pragma unroll
              for (int mb = 0; mb < MB; ++mb)
                v[u][q][mb] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                    res, slot_of(min(s0 + u, a.splits - 1), min(n1 + q, NB - 1), mb), 0, COHERENT));
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int u = 0; u < SHARES; ++u)
            if (s0 + u < a.splits) {
#pragma unroll
              for (int q = 0; q < AT_ONCE; ++q)
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
                  if (n1 + q < NB) acc[n1 + q < NB ? n1 + q : 0][mb] += v[u][q][mb];
            }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    const int nw = n0 + wn * (T::TN / T::WN), mw = m0 + wm * (T::TM / T::WM) + r16;
    const int lane_col = 16 * (kg & 1) + 8 * (kg >> 1);   // see gather_columns
    auto store8 = [&](const float (&v)[8], __bf16* o) {
      bf16x8 b;
#pragma unroll
      for (int e = 0; e < 8; ++e) b[e] = static_cast<__bf16>(v[e]);
      *reinterpret_cast<bf16x8*>(o) = b;
    };
    if constexpr (ROPE) {
      // RB blocks of the lower half of a head, then the RB blocks of its upper half that they are rotated with.  First all
      // blocks are rotated where they are, then all are stored: loads and stores of a wave are counted in one order, and
      // angles asked for behind a store would be waited for as long as that store takes.  Stores cover whole 64-byte segments
      // wherever a wave has them: in pieces of 32 the same tile costs 4.5 us more for 12288 columns of 1024 tokens (whole: 98
      // us in place of 92 for the plain projection and 11 for the append launch that this saves).
      constexpr int RB = T::ROPE_ROWS / 16;
      constexpr int AH = T::PER_SIMD > 2 ? 1 : MB >= 8 ? 2 : MB % 4 == 0 ? 4 : MB % 3 == 0 ? 3 : MB;   // as registers allow
      auto walk_of = [&](int nb) __attribute__((always_inline)) -> int {
        if constexpr (NB == 6) return n0 + 32 * (nb < 4 ? 4 * wn + nb / 2 : 2 + wn);
        return nw + 16 * nb;
      };
#pragma unroll
      for (int nb = 0; nb < NB; nb += 2 * RB) {
        const int walk = walk_of(nb), in_head = walk & (a.rope - 1);
        if (walk - in_head >= a.rotated) continue;
        const float* const angle = a.angles + (in_head >> 1) + 4 * kg;
#pragma unroll
        for (int m1 = 0; m1 < MB; m1 += AH) {
          f32x4 c[AH][RB], sn[AH][RB];   // on their way together
#pragma unroll
          for (int u = 0; u < AH; ++u)
#pragma unroll
            for (int h = 0; h < RB; ++h) {
              const float* const at = angle + static_cast<long long>(min(mw + 16 * (m1 + u), a.m - 1)) * a.rope + 16 * h;
              c[u][h] = *reinterpret_cast<const f32x4*>(at);
              sn[u][h] = *reinterpret_cast<const f32x4*>(at + a.rope / 2);
            }
#pragma unroll
          for (int u = 0; u < AH; ++u)
#pragma unroll
            for (int h = 0; h < RB; ++h)
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const float x0 = acc[nb + h][m1 + u][e], x1 = acc[nb + RB + h][m1 + u][e];
                acc[nb + h][m1 + u][e] = fmaf(x0, c[u][h][e], -(x1 * sn[u][h][e]));
                acc[nb + RB + h][m1 + u][e] = fmaf(x1, c[u][h][e], x0 * sn[u][h][e]);
              }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int nb = 0; nb < NB; nb += 4) {
        const int walk = walk_of(nb), in_head = walk & (a.rope - 1), head = walk - in_head;
        if (walk >= a.n) continue;
        const int s = head < a.seg[0].end ? 0 : head < a.seg[1].end ? 1 : 2;
        const int ld = a.seg[s].ld;
        const bool two = nb + 4 <= NB;   // units; a single one leaves a lane 8 columns of the lower half or 8 of the upper
        __bf16* const obase = a.seg[s].ptr + head - a.seg[s].first + (in_head >> 1) +
                              (two ? lane_col : (kg & 1) * (a.rope / 2) + 8 * (kg >> 1));
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
          const int tok = mw + 16 * mb;
          __bf16* const o = obase + static_cast<long long>(tok) * ld;
          float v[8], u[8];
          if (two) {
            constexpr int L1 = RB == 2 ? 1 : 2;          // where the second half of the lower columns sits
            gather_columns(acc[nb][mb], acc[min(nb + L1, NB - 1)][mb], v);
            gather_columns(acc[min(nb + 3 - L1, NB - 1)][mb], acc[min(nb + 3, NB - 1)][mb], u);
            if (tok < a.m) {
              store8(v, o);
              store8(u, o + a.rope / 2);
            }
          } else {
            gather_columns(acc[nb][mb], acc[nb + 1][mb], v);
            if (tok < a.m) store8(v, o);
          }
        }
      }
    } else if (a.dual) {
      // blocks nb = 4 i, 4 i + 1 / 4 i + 2, 4 i + 3 are the gate / up rows of the same 32 output columns
      if constexpr (NB % 4 == 0) {
#pragma unroll
        for (int i = 0; i < NB / 4; ++i) {
          if (nw + 64 * i >= a.n) continue;
          const int col0 = ((nw + 64 * i) >> 1) + lane_col;
#pragma unroll
          for (int mb = 0; mb < MB; ++mb) {
            f32x4 act[2];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const float g = acc[4 * i + h][mb][e], u = acc[4 * i + 2 + h][mb][e];
                act[h][e] = g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * u;
              }
            float v[8];
            gather_columns(act[0], act[1], v);
            const int tok = mw + 16 * mb;
            if (tok < a.m) store8(v, a.seg[0].ptr + static_cast<long long>(tok) * a.seg[0].ld + col0);
          }
        }
      } else if constexpr (NB == 2) {
        // 16 rows of each weight: a lane has 4 columns of its token
        if (nw < a.n) {
#pragma unroll
          for (int mb = 0; mb < MB; ++mb) {
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float g = acc[0][mb][e], u = acc[1][mb][e];
              o[e] = static_cast<__bf16>(g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * u);
            }
            const int tok = mw + 16 * mb;
            if (tok < a.m)
              *reinterpret_cast<bf16x4*>(a.seg[0].ptr + static_cast<long long>(tok) * a.seg[0].ld + (nw >> 1) + 4 * kg) = o;
          }
        }
      }
    } else {
#pragma unroll
      for (int nb = 0; nb < NB; nb += 2) {
        const int nblk = nw + 16 * nb;   // first output column of this pair of blocks
        if (nblk >= a.n) continue;
        // segment that holds it (segment edges are multiples of 32)
        int s = 0;
        if (a.n_seg > 1 && nblk >= a.seg[0].end) s = 1;
        if (a.n_seg > 2 && nblk >= a.seg[1].end) s = 2;
        __bf16* obase = a.seg[s].ptr;
        const int ld = a.seg[s].ld, col0 = nblk - a.seg[s].first + lane_col;
        // residual rows first, all of them in flight together (rows past the end repeat the last one)
        bf16x8 r8[MB];
        if (a.res != nullptr) {
#pragma unroll
          for (int mb = 0; mb < MB; ++mb)
            r8[mb] = *reinterpret_cast<const bf16x8*>(a.res + static_cast<long long>(min(mw + 16 * mb, a.m - 1)) * ld + col0);
        } else {
#pragma unroll
          for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int e = 0; e < 8; ++e) r8[mb][e] = static_cast<__bf16>(0.0f);
        }
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
          float v[8];
          gather_columns(acc[nb][mb], acc[nb + 1][mb], v);
          const int tok = mw + 16 * mb;
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] += static_cast<float>(r8[mb][e]);
          if (tok < a.m) store8(v, obase + static_cast<long long>(tok) * ld + col0);
        }
      }
    }
  }
}

// Few tokens: a pass over the weights, bound by how fast they come from memory.  A workgroup owns 16 weight rows (SwiGLU: 8
// columns, their gate rows and their up rows; with rotation: 8 rows of the lower half of a head and the 8 of its upper half that
// they are rotated with) and all (up to 16) tokens; its waves share out k in chunks of 64, and both
// operands go from global memory straight into MFMA fragments, since no wave needs what another one loads: no LDS and no
// barrier until the sums of the shares meet at the end.  Measured and not taken (1 token): the last chunks of a
// row in one go instead of one by one (4096 x 11008: no difference); the loads of eight chunks held in flight by hand (22.2 us ->
// 22.9), two sets of four or of two chunks in turn (24.8, 22.1; 12288 x 4096 19.5 -> 26, 23); lanes without a token asking for
// nothing (no difference); rows as whole 1 KiB loads with fp32 multiply-adds on the vector ALU (29.1, and slower with every
// further token).
// Waves: 16 where a row holds at least four chunks for each of them and there are 512 weight rows, else 8 (one token, 8 -> 16 waves:
// 12288 x 4096 19.5 -> 18.2 us, 5.5 TB/s; 11008 x 4096 SwiGLU 34.4 -> 32.1, 5.6; 4096 x 11008 22.2 -> 21.6; 2048 x 5632 10.0 -> 9.5;
// but 1024 x 2816 5.1 -> 5.3, 2816 x 1024 SwiGLU 4.6 -> 4.8).  The second eight cost a launch 0.15 us; what they gain is requests
// under way to memory.  Time with 16 over time with 8, 1 to 16 tokens on 4096 / 4544 / 5632 / 8192 / 11008 columns, weights from
// memory: 256 rows 1.02 / 0.99 / 1.02 / 1.01 / 0.99, 512 1.02 / 0.94 / 0.96 / 1.00 / 0.98, 1024 1.00 / 0.93 / 0.95 / 1.00 / 0.97,
// 2048 0.98 / 0.92 / 0.94 / 0.97 / 0.95, 4096 and more 0.88 to 0.95.  (From the last-level cache they pay from 5632 rows on: 0.90 to 1.00;
// fewer 0.91 to 1.03.  A model's weights are not there when they are used again.)
// NORM: the tokens come before their RMSNorm; the waves add up the squares of the chunks they multiply anyway, and the norm launch
// and the wait behind it go.  Up to 16 tokens x * gain is what is multiplied, and the factor 1 / rms, which belongs to a token, is
// applied to the sums: as many roundings as with a norm of its own (x * gain instead of x * gain / rms).  Few registers, so that
// two workgroups of 16 waves share a CU: with four chunks in one go (128 registers) 1 token of the 4096-wide layer takes 158 us
// instead of 141.  Not taken either: two blocks of rows per workgroup, which halves that work (+12 us), and persistent workgroups
// that keep the tokens in registers (+25): one workgroup per CU in step with itself does not keep the memory busy.
// Beyond 16 tokens (TB = 2) the waves meet for the sums first and multiply what the norm launch would have stored, so that a row
// is rounded where it has always been (the meeting costs 1.2 us of a 25 us layer).
enum RowsKind { kRowsPlain, kRowsDual, kRowsRope };

struct NormedRowsArgs : GemmArgs {
  const __bf16* gain;
  float eps;
  long long position;      // of the first token (rope)
  double inv_freq[64];     // (rope)
};

template <RowsKind KIND, bool NORM, int WAVES, int RB, int TB>
__global__ __launch_bounds__(64 * WAVES, NORM ? (TB > 1 ? 4 : 8) : WAVES / 4) void linear_rows_kernel(std::conditional_t<NORM, NormedRowsArgs, GemmArgs> a) {
  constexpr bool DUAL = KIND == kRowsDual, ROPE = KIND == kRowsRope;
  static_assert(NORM || !ROPE, "the rotation is only wanted behind a norm");
  static_assert(RB * TB <= WAVES && (!ROPE || 2 * RB * TB <= WAVES), "a wave per block at the end, and per half of its angles");
  __shared__ f32x4 part[RB * TB][WAVES][64];
  __shared__ float squares[NORM ? TB : 1][NORM ? WAVES : 1][64];
  __shared__ float cs[ROPE ? 16 * TB : 1][8 * RB], sn[ROPE ? 16 * TB : 1][8 * RB];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, kg = lane >> 4;
  constexpr int COLS = DUAL ? 8 : 16;
  const int first = blockIdx.x * (COLS * RB), m0 = blockIdx.y * (16 * TB);   // n is a multiple of 32 (of each weight)
  const __bf16* const weight = DUAL && r16 >= COLS ? a.w2 : a.w;
  const int head = first & -a.rope, rope_col = (first - head) >> 1;   // (rope only)
  const int row = ROPE ? head + rope_col + r16 % 8 + (r16 >= 8 ? a.rope / 2 : 0) : first + r16 % COLS;
  const char* const w = reinterpret_cast<const char*>(weight) + 2 * (static_cast<long long>(row) * a.k + 8 * kg);
  const long long w_step = 2ll * (ROPE || DUAL ? 8 : 16) * a.k;   // from a block of rows to the next
  const char* x[TB];
#pragma unroll
  for (int t = 0; t < TB; ++t)
    x[t] = reinterpret_cast<const char*>(a.x) + 2 * (static_cast<long long>(min(m0 + 16 * t + r16, a.m - 1)) * a.k + 8 * kg);
  if constexpr (ROPE) {
    // the angles of 8 RB frequencies for 16 TB tokens, by the last waves
    const int i = tid - 64 * (WAVES - 2 * RB * TB), t = i / (8 * RB), f = i % (8 * RB);
    if (i >= 0 && m0 + t < a.m && head < a.rotated)
      rope_angle(static_cast<double>(a.position + m0 + t) * a.inv_freq[rope_col + f], &cs[t][f], &sn[t][f]);
  }
  f32x4 acc[RB][TB];
#pragma unroll
  for (int b = 0; b < RB; ++b)
#pragma unroll
    for (int t = 0; t < TB; ++t) acc[b][t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  const int chunks = a.k / 64;
  auto load_w = [&](bf16x8 (&f)[2][RB], int c) __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int b = 0; b < RB; ++b) f[h][b] = *reinterpret_cast<const bf16x8*>(w + b * w_step + 128ll * c + 64 * h);
  };
  auto load_x = [&](bf16x8 (&f)[2][TB], int c) __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int t = 0; t < TB; ++t) f[h][t] = *reinterpret_cast<const bf16x8*>(x[t] + 128ll * c + 64 * h);
  };
  auto multiply = [&](const bf16x8 (&fw)[2][RB], const bf16x8 (&fx)[2][TB]) __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int t = 0; t < TB; ++t)
#pragma unroll
        for (int b = 0; b < RB; ++b) acc[b][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[h][b], fx[h][t], acc[b][t], 0, 0, 0);
  };
  const char* gain_at = nullptr;
  if constexpr (NORM) gain_at = reinterpret_cast<const char*>(a.gain) + 16 * kg;
  auto load_gain = [&](bf16x8 (&f)[2], int c) __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < 2; ++h) f[h] = *reinterpret_cast<const bf16x8*>(gain_at + 128ll * c + 64 * h);
  };
  float ss[TB];
#pragma unroll
  for (int t = 0; t < TB; ++t) ss[t] = 0.0f;
  auto squared = [&](const bf16x8 (&f)[2][TB]) __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int t = 0; t < TB; ++t)
#pragma unroll
        for (int e = 0; e < 8; ++e) ss[t] = fmaf(static_cast<float>(f[h][t][e]), static_cast<float>(f[h][t][e]), ss[t]);
  };
  auto scaled = [&](bf16x8 (&f)[2][TB], const float (&rinv)[TB], const bf16x8 (&gain)[2]) __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int t = 0; t < TB; ++t)
#pragma unroll
        for (int e = 0; e < 8; ++e)
          f[h][t][e] = static_cast<__bf16>(static_cast<float>(f[h][t][e]) * rinv[t] * static_cast<float>(gain[h][e]));
  };
  if constexpr (NORM && TB == 1) {
    for (int c = wave; c < chunks; c += WAVES) {
      bf16x8 fw[2][RB], fx[2][TB], fg[2];
      load_w(fw, c);
      load_x(fx, c);
      load_gain(fg, c);
      squared(fx);
      scaled(fx, {1.0f}, fg);
      multiply(fw, fx);
    }
    squares[0][wave][lane] = ss[0];
  } else if constexpr (NORM) {
    // first the squares of all chunks, of which the first KEEP stay in registers, then the products
    constexpr int KEEP = 2;
    bf16x8 kw[KEEP][2][RB], kx[KEEP][2][TB], kgain[KEEP][2];
#pragma unroll
    for (int u = 0; u < KEEP; ++u)
      if (wave + u * WAVES < chunks) {
        load_x(kx[u], wave + u * WAVES);
        load_w(kw[u], wave + u * WAVES);
        load_gain(kgain[u], wave + u * WAVES);
      }
#pragma unroll
    for (int u = 0; u < KEEP; ++u)
      if (wave + u * WAVES < chunks) squared(kx[u]);
    for (int c = wave + KEEP * WAVES; c < chunks; c += WAVES) {
      bf16x8 fx[2][TB];
      load_x(fx, c);
      squared(fx);
    }
#pragma unroll
    for (int t = 0; t < TB; ++t) squares[t][wave][lane] = ss[t];
    __syncthreads();
    float rinv[TB];
#pragma unroll
    for (int t = 0; t < TB; ++t) {
      float sum = 0.0f;
#pragma unroll
      for (int u = 0; u < WAVES; ++u) sum += squares[t][u][lane];
      sum += __shfl_xor(sum, 16);
      sum += __shfl_xor(sum, 32);
      rinv[t] = 1.0f / sqrtf(sum / static_cast<float>(a.k) + a.eps);
    }
#pragma unroll
    for (int u = 0; u < KEEP; ++u)
      if (wave + u * WAVES < chunks) {
        scaled(kx[u], rinv, kgain[u]);
        multiply(kw[u], kx[u]);
      }
    for (int c = wave + KEEP * WAVES; c < chunks; c += WAVES) {
      bf16x8 fw[2][RB], fx[2][TB], fg[2];
      load_w(fw, c);
      load_x(fx, c);
      load_gain(fg, c);
      scaled(fx, rinv, fg);
      multiply(fw, fx);
    }
  } else {
    auto steps = [&](int c, auto count_tag) __attribute__((always_inline)) {
      constexpr int COUNT = decltype(count_tag)::value;
      bf16x8 fw[COUNT][2][RB], fx[COUNT][2][TB];
#pragma unroll
      for (int u = 0; u < COUNT; ++u) {
        load_w(fw[u], c + u * WAVES);
        load_x(fx[u], c + u * WAVES);
      }
#pragma unroll
      for (int u = 0; u < COUNT; ++u) multiply(fw[u], fx[u]);
    };
    int c = wave;
    if constexpr (RB * TB == 1) {
      constexpr int AHEAD = 64 / WAVES;   // chunks of a wave in one go: all of a 4096-deep row
      for (; c + (AHEAD - 1) * WAVES < chunks; c += AHEAD * WAVES) steps(c, std::integral_constant<int, AHEAD>{});
    } else {                              // short rows: one chunk per wave, some have two (in a loop alone 1.06 of the time)
      if (c < chunks) steps(c, std::integral_constant<int, 1>{});
      c += WAVES;
    }
    for (; c < chunks; c += WAVES) steps(c, std::integral_constant<int, 1>{});
  }
#pragma unroll
  for (int b = 0; b < RB; ++b)
#pragma unroll
    for (int t = 0; t < TB; ++t) part[b * TB + t][wave][lane] = acc[b][t];
  __syncthreads();
  if (wave >= RB * TB) return;
  // a block per wave, of it rows 4 kg .. 4 kg + 3 of a token per lane
  const int b = wave / TB, t = wave % TB, n0 = first + b * COLS, tok = m0 + 16 * t + r16;
  f32x4 v = part[wave][0][lane];
#pragma unroll
  for (int u = 1; u < WAVES; ++u) v += part[wave][u][lane];
  if constexpr (NORM && TB == 1) {
    float sum = 0.0f;
#pragma unroll
    for (int u = 0; u < WAVES; ++u) sum += squares[0][u][lane];
    sum += __shfl_xor(sum, 16);
    sum += __shfl_xor(sum, 32);
    v *= 1.0f / sqrtf(sum / static_cast<float>(a.k) + a.eps);
  }
  bf16x4 o;
  if constexpr (DUAL) {
    // the up rows of this lane's columns are 32 lanes on
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float g = v[e], u = __shfl_xor(v[e], 32);
      o[e] = static_cast<__bf16>(g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * u);
    }
    if (kg >= 2 || tok >= a.m) return;
    *reinterpret_cast<bf16x4*>(a.seg[0].ptr + static_cast<long long>(tok) * a.seg[0].ld + n0 + 4 * kg) = o;
  } else if constexpr (ROPE) {
    const int s = head < a.seg[0].end ? 0 : head < a.seg[1].end ? 1 : 2;
    const int i = 8 * b + 4 * (kg & 1);      // of the angles of this lane's columns
    f32x4 other;
#pragma unroll
    for (int e = 0; e < 4; ++e) other[e] = __shfl_xor(v[e], 32);   // the other half of the pairs
    if (tok >= a.m) return;
    if (head < a.rotated) {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = fmaf(v[e], cs[16 * t + r16][i + e], (kg >= 2 ? other[e] : -other[e]) * sn[16 * t + r16][i + e]);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = static_cast<__bf16>(v[e]);
    *reinterpret_cast<bf16x4*>(a.seg[s].ptr + static_cast<long long>(tok) * a.seg[s].ld + head - a.seg[s].first + rope_col + i +
                               (kg >= 2 ? a.rope / 2 : 0)) = o;
  } else {
    if (tok >= a.m) return;
    int s = 0;
    if (a.n_seg > 1 && n0 >= a.seg[0].end) s = 1;
    if (a.n_seg > 2 && n0 >= a.seg[1].end) s = 2;
    const long long at = static_cast<long long>(tok) * a.seg[s].ld + n0 - a.seg[s].first + 4 * kg;
    if (a.res != nullptr) {
      const bf16x4 r = *reinterpret_cast<const bf16x4*>(a.res + at);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += static_cast<float>(r[e]);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = static_cast<__bf16>(v[e]);
    *reinterpret_cast<bf16x4*>(a.seg[s].ptr + at) = o;
  }
}

namespace {

// Stages between the starts of neighbouring weight tiles, 0: all start at the first.  A pass of few tokens over deep rows is bound by
// the weights' way from memory, and its workgroups walk the rows in step: they ask for the same columns of all rows at a time.
// Memory is dealt out in pieces of 256 bytes over 128 channels (rows 32 KB apart lie on one), so where that is a few channels only,
// tiles that start three stages apart and wrap around keep the others busy.  Weights from memory, in step -> apart:
//   rows a multiple of 4 KB apart: 12288 x 8192, 20 / 77 tokens 44.5 -> 38.4 / 53.9 -> 49.5 us; 22016 x 4096, 77 tokens 47.7 ->
//   40.9; 16384-deep rows 0.76 to 0.95 of the time; 4096 x 4096 the same;
//   one, two or three rows within 256 bytes (three: 512 above) of a multiple of 32 KB: 4096 x 11008, 20 / 77 tokens 29.9 -> 27.5 /
//   33.7 -> 30.4; 12288 x 5504, 20 tokens 35.9 -> 27.8; 12288 x 16320, 20 tokens 121 -> 74.
// Elsewhere it gains nothing and costs up to a fifth (of all k from 4096 to 18432 in steps of 128: 12288 x 16000, 20 tokens 1.22, 4096 x
// 16896, 77 tokens 1.17, 12288 x 5120 1.02 of the time), and so does k = 12288 in the 64 x 64 tile with 128-deep stages (1.07 to 1.11,
// alone among the multiples of 2048).  With fewer weight rows too few workgroups share the memory: at the distances above 256 / 512
// rows take 0.99 to 1.02 / 0.99 to 1.01 of the time, 1024 0.97 to 1.00.  (Weights that are in the last-level cache gain less and less
// often: 4096 x 11008 0.92 of the time, most others 0.97 to 1.03.  A model's weights are not, from one use to the next.)  64 x 64 tiles
// of 64-deep stages with three and more token tiles gain at the multiples of 8192 (two channels: 8192 x 8192, 182 tokens 67.9 -> 64.6)
// but not at the others (6144 x 6144, 160 tokens 1.00, and up to 1.10 with the weights in the last-level cache).
// From 257 tokens on the tiles that share an operand in the L2 lose more by it (11008 x 4096 SwiGLU, 1000 tokens 166 -> 172).
// Starts eight stages apart are worse.
// One more class gains, whatever its rows' distance: a weight larger than the last-level cache (256 MB) whose last token tile is at
// most five eighths full (the workgroups of that tile read the last token again and again): 12288 x 14080, 144 tokens 135.7 ->
// 105.6; 200 / 250 tokens 0.99 / 1.00 of the time.
template <class T>
int stagger_of(const GemmArgs& a) {
  if (T::TN * T::TM > 128 * 256 || a.m > 256 || a.k < 4096 || a.n < 1024) return 0;   // (few tokens do not get the larger tiles)
  const int tiles_m = (a.m + T::TM - 1) / T::TM, apart = static_cast<int>(2ll * a.k % 32768);
  auto one_channel = [&](int rows, int above) {
    const int distance = rows * apart % 32768;
    return distance <= above || distance >= 32768 - 256;
  };
  if (a.k % 2048 == 0) {
    const bool gains = !(T::TN == 64 && T::TM == 64) || (T::TK == 64 ? tiles_m <= 2 || a.k % 8192 == 0 : a.k != 12288);
    if (gains) return 3;
  } else if (one_channel(1, 256) || one_channel(2, 256) || one_channel(3, 512)) {
    return 3;
  }
  const int in_last = a.m - (tiles_m - 1) * T::TM;
  return tiles_m > 1 && 8 * in_last <= 5 * T::TM && 2ll * a.n * a.k > 256ll << 20 ? 3 : 0;
}

template <class T>
auto tile_kernel(const GemmArgs& a) -> void (*)(GemmArgs) {
  if constexpr (T::TN * T::TM <= 128 * 256) {
    if (stagger_of<T>(a) != 0) return a.rope != 0 ? linear_kernel<T, true, false, true> : linear_kernel<T, false, false, true>;
  }
  return a.rope != 0 ? linear_kernel<T, true, false, false> : linear_kernel<T, false, false, false>;
}

// Whatever the runtime may refuse before a launch: asked for ahead where a call is two launches, so that it enqueues both or none.
template <class T>
bool tile_ready(const GemmArgs& a) {
  return T::LDS <= 64 * 1024 || grant_lds(reinterpret_cast<const void*>(tile_kernel<T>(a)), T::LDS);
}

template <class T>
int launch_tile(GemmArgs& a, hipStream_t stream) {
  a.stagger = stagger_of<T>(a);
  a.tiles_n = (a.n + T::TN - 1) / T::TN;
  a.tiles_m = (a.m + T::TM - 1) / T::TM;
  const int per = (a.tiles_n * a.tiles_m + 7) / 8;
  constexpr int PER_CU = T::PER_SIMD * 4 / T::NW;
  const unsigned grid = 8u * static_cast<unsigned>(std::min(per, 32 * PER_CU));
  return launch_kernel(tile_kernel<T>(a), dim3(grid), dim3(T::THREADS), a, stream, T::LDS);
}

// a.splits workgroups per tile, all of them in one round
template <class T>
int launch_split(GemmArgs& a, hipStream_t stream) {
  a.stagger = stagger_of<T>(a);
  a.tiles_n = (a.n + T::TN - 1) / T::TN;
  a.tiles_m = (a.m + T::TM - 1) / T::TM;
  const unsigned pieces = 8u * static_cast<unsigned>((a.tiles_n * a.tiles_m * a.splits + 7) / 8);
  return launch_kernel(a.stagger != 0 ? linear_kernel<T, false, true, true> : linear_kernel<T, false, true, false>, dim3(pieces),
                       dim3(T::THREADS), a, stream, T::LDS);
}

template <RowsKind KIND, bool NORM, class Args>
int launch_rows(Args& a, hipStream_t stream) {
  const unsigned blocks = static_cast<unsigned>(a.n / 16);   // dual: a.n counts the rows of both weights
  if constexpr (NORM || KIND == kRowsPlain) {
    if (a.m > 16) {
      const dim3 grid(blocks / 2, static_cast<unsigned>((a.m + 31) / 32));
      if (a.k <= (NORM ? 1024 : 512)) return launch_kernel(linear_rows_kernel<KIND, NORM, 8, 2, 2>, grid, dim3(512), a, stream);
      return launch_kernel(linear_rows_kernel<KIND, NORM, 16, 2, 2>, grid, dim3(1024), a, stream);
    }
  }
  if (a.k >= 4096 && a.n >= 512) return launch_kernel(linear_rows_kernel<KIND, NORM, 16, 1, 1>, dim3(blocks), dim3(1024), a, stream);
  return launch_kernel(linear_rows_kernel<KIND, NORM, 8, 1, 1>, dim3(blocks), dim3(512), a, stream);
}

// ---- which kernel a shape gets ----------------------------------------------------------------------
// A tile is good when it is large (LDS and L2 traffic per MFMA: at 256 x 256 the matrix pipes are busy 85 % of a step, at
// 128 x 128 the loads take as long as the MFMAs) and when the tiles of the problem fill whole rounds of the 256 CUs; which
// of the two wins changes with every few hundred tokens.  So the choice is made on a cost: T = fixed + KT * (rounds * step +
// full * step_full) + rounds * per_round, in microseconds, KT = k / 64, rounds over the CUs of the fullest XCD, full = how
// many rounds keep more than half the CUs busy (the clock drops then; the last round counts by how far it is beyond the half).
// The constants are a non-negative least-squares fit to 4000 launches timed on MI355X (1 to 5824 tokens, 13 (n, k) pairs of 256
// to 22016 x 256 to 11008, plain / residual / SwiGLU); choosing by the fit costs 2 % against choosing by hindsight, 10 % and
// more in 12 of 300 shapes.  Tiles that were measured and never needed: 256 x 128, 192 x 128, 128 x 64, 64 x 32.
struct TileChoice {
  int tn, tm, tk, per_cu;
  bool dual;
  float fixed, per_round, step, step_full;
  int (*launch)(GemmArgs&, hipStream_t);
  bool (*ready)(const GemmArgs&);
  int (*split)(GemmArgs&, hipStream_t);   // nullptr: none
};

template <class T, bool SPLIT = false>
constexpr TileChoice choice(int per_cu, bool dual, float fixed, float per_round, float step, float step_full) {
  TileChoice c = {T::TN, T::TM, T::TK, per_cu, dual, fixed, per_round, step, step_full, launch_tile<T>, tile_ready<T>, nullptr};
  if constexpr (SPLIT) c.split = launch_split<T>;
  return c;
}

const TileChoice kTiles[] = {
    choice<GemmTile<256, 256, 64, 2, 4, 2, 1, 2>>(1, true, 6.59f, 0.00f, 1.245f, 0.208f),
    choice<GemmTile<256, 192, 64, 2, 4, 2, 1, 2>>(1, true, 5.44f, 0.00f, 1.084f, 0.137f),
    choice<GemmTile<192, 256, 64, 2, 2, 4, 1, 2>>(1, false, 5.84f, 0.00f, 1.012f, 0.202f),
    choice<GemmTile<192, 192, 64, 3, 3, 4, 1, 3>>(1, true, 3.76f, 1.97f, 0.714f, 0.173f),
    choice<GemmTile<128, 256, 64, 3, 2, 4, 1, 2>, true>(1, true, 4.29f, 1.28f, 0.679f, 0.155f),
    choice<GemmTile<128, 192, 64, 4, 2, 4, 1, 2>>(1, true, 4.04f, 0.83f, 0.536f, 0.155f),
    choice<GemmTile<128, 128, 64, 5, 2, 4, 1, 2, true>, true>(1, true, 4.73f, 0.00f, 0.420f, 0.106f),
    choice<GemmTile<64, 128, 64, 6, 1, 8, 1, 2, true>, true>(1, true, 3.51f, 0.85f, 0.303f, 0.042f),
    choice<GemmTile<64, 64, 64, 5, 1, 4, 1, 2, true>>(2, true, 4.16f, 0.00f, 0.241f, 0.205f),
    choice<GemmTile<64, 64, 128, 4, 2, 2, 2, 2, true>>(1, true, 3.48f, 0.89f, 0.179f, 0.029f),
    choice<GemmTile<32, 64, 128, 5, 1, 4, 2, 2, true>>(1, true, 3.32f, 0.79f, 0.137f, 0.023f),
    choice<GemmTile<32, 32, 128, 8, 1, 2, 4, 2, true>>(1, true, 3.28f, 0.78f, 0.112f, 0.001f),
};

int64_t tiles_per_xcd(const TileChoice& c, const GemmArgs& a) {   // 64 bits: the query takes sizes that no memory holds
  return (static_cast<int64_t>((a.n + c.tn - 1) / c.tn) * ((a.m + c.tm - 1) / c.tm) + 7) / 8;
}

float tile_cost(const TileChoice& c, const GemmArgs& a) {
  const int slots = 32 * c.per_cu;
  const int64_t per_xcd = tiles_per_xcd(c, a), rounds = (per_xcd + slots - 1) / slots;
  const float last = static_cast<float>(per_xcd - (rounds - 1) * slots) / slots;
  const float full = rounds - 1 + std::max(0.0f, 2.0f * last - 1.0f);
  return c.fixed + a.k / 64 * (rounds * c.step + full * c.step_full) + rounds * c.per_round;
}

const TileChoice* choose_tile(const GemmArgs& a) {
  const TileChoice* best = nullptr;
  float best_cost = 0.0f;
  for (const TileChoice& c : kTiles) {
    if ((a.dual && !c.dual) || a.k % c.tk != 0) continue;
    const float cost = tile_cost(c, a);
    if (best == nullptr || cost < best_cost) {
      best = &c;
      best_cost = cost;
    }
  }
  return best;
}

// With k shared out over `splits` workgroups per tile, all in one round: the loop is that much shorter, and the merge costs 3.5 us and
// 0.024 us per KB that the last piece reads back (a tile's sums, once per share).  Pays where k is deep and the tiles are few.  The down
// projection of a 4096-wide layer (4096 x 11008, weights from memory), tokens: time before -> after: 77: 31.8 -> 28.2 us
// (64 x 128, four shares); 250: 51.2 -> 41.5 (128 x 128, four); 500: 71.8 -> 63.6 (128 x 128, two); 1000: 103.1 -> 94.5 (128 x 256,
// two).  4096 x 4096 and 2048 x 5632 would gain nothing to 5 %, so a split has to promise more than that.
float split_cost(const TileChoice& c, const GemmArgs& a, int splits) {
  const int64_t pieces = static_cast<int64_t>((a.n + c.tn - 1) / c.tn) * ((a.m + c.tm - 1) / c.tm) * splits;
  const int stages = a.k / c.tk;
  const float full = std::max(0.0f, static_cast<float>(pieces) / 128.0f - 1.0f);
  return c.fixed + c.per_round + (stages + splits - 1) / splits * (c.step + full * c.step_full) + 3.5f +
         0.024f * splits * static_cast<float>(c.tn * c.tm / 256);
}

// The tile and number of shares to split a launch that would get `whole` into, or nullptr.
const TileChoice* choose_split(const GemmArgs& a, const TileChoice& whole, const SharedScratch& shared, int* splits) {
  const TileChoice* best = nullptr;
  float best_cost = 0.95f * tile_cost(whole, a);
  for (const TileChoice& c : kTiles) {
    if (c.split == nullptr || a.k % c.tk != 0) continue;
    const int64_t tiles = static_cast<int64_t>((a.n + c.tn - 1) / c.tn) * ((a.m + c.tm - 1) / c.tm);
    if (tiles > shared.n_counters) continue;
    for (int s = 2; s <= 8 && tiles * s <= 256 && a.k / c.tk / s >= 16 && tiles * s * c.tn * c.tm * 4 <= shared.bytes; ++s) {
      const float cost = split_cost(c, a, s);
      if (cost < best_cost) {
        best = &c;
        best_cost = cost;
        *splits = s;
      }
    }
  }
  return best;
}

// A long launch whose tiles leave its last round nearly empty goes out as two: one of the large tiles (128 x 256 and more) on as many
// columns as fill whole rounds, and whatever is best on the columns left over.  (The sums of those columns may be taken in another order
// than the whole launch would take them, where the second tile's waves share k.)  22016 x 4096 SwiGLU rows
// are 86 tiles of 256, so 3072 tokens are 4.03 rounds: 432 -> 395 us; 700 tokens 125 -> 115, 1500 236 -> 212, 3712 537 -> 487;
// 11264 x 2048 at 6000 tokens 226 -> 209; 4096 x 11008, 2304 / 4800 tokens: 206 -> 189 / 394 -> 360.  The two
// have to promise 4 % together, and are only looked for where that is more than the search (1 us) and the second launch.  Short rows
// without SwiGLU stay whole: the fit is pessimistic there (4096 x 4096, 4800 tokens: 152 us expected, 137 measured, 143 in two).
struct TwoParts {
  const TileChoice* first;   // nullptr: one launch
  const TileChoice* second;
  int columns;               // weight rows walked by the first
};

TwoParts choose_two(const GemmArgs& a, const TileChoice& whole) {
  TwoParts best = {nullptr, nullptr, 0};
  if (a.k < (a.dual ? 1024 : 8192)) return best;
  float best_cost = 0.96f * tile_cost(whole, a);
  if (best_cost < 60.0f) return best;
  for (const TileChoice& c : kTiles) {
    if (c.tn * c.tm < 128 * 256 || c.per_cu != 1 || (a.dual && !c.dual) || a.k % c.tk != 0) continue;
    const int64_t tiles_m = (a.m + c.tm - 1) / c.tm, tiles = static_cast<int64_t>((a.n + c.tn - 1) / c.tn) * tiles_m;
    const int64_t columns = tiles / 256 * 256 / tiles_m * c.tn;
    if (columns <= 0 || columns >= a.n) continue;
    GemmArgs part = a;
    part.n = static_cast<int>(columns);
    const float first = tile_cost(c, part) + 1.0f;
    if (first >= best_cost) continue;
    part.n = a.n - part.n;
    const TileChoice* const rest = choose_tile(part);
    const float cost = first + tile_cost(*rest, part);
    if (cost < best_cost) {
      best = TwoParts{&c, rest, static_cast<int>(columns)};
      best_cost = cost;
    }
  }
  return best;
}

// Up to 8 tokens (16 where there are fewer than 8192 weight rows) the direct kernel is the fastest: at 1 token 8.4 / 19.1 /
// 22.1 us for n x k = 4096 x 4096 / 12288 x 4096 / 4096 x 11008 (weights at 4.0 / 5.3 / 4.1 TB/s) against 10.4 / 23.3 / 25.6;
// at 16 tokens 10.2 / 24.8 / 26.8 against 11.4 / 23.6 / 28.5.
// SwiGLU reads more rows per column and gives way to the tiles at 4 tokens where there are 16384 rows or more: n x k =
// 11008 x 4096 at 1 / 4 / 8 tokens 34.7 / 38.3 / 43.3 us (5.2 TB/s at 1) against 41.2 / 41.2 / 41.5; 5632 x 2048 at 1 / 8 / 12
// 10.4 / 12.5 / 13.7 against 12.7 / 13.1 / 13.1; 2816 x 1024 at 1 / 16 4.9 / 6.0 against 6.2 / 6.2.
// Beyond that, one round of workgroups of 32 rows x 32 tokens where k has an odd number of 64-column chunks, which only the tiles
// with 64-deep stages can walk, and few of them.  Time in blocks over time in tiles, 32 to 8192 columns, 17 to 4000 tokens: k = 448 0.68 to
// 0.76, 576 0.70 to 0.76, 704 0.74 to 0.78, 832 0.74 to 0.80, 960 0.75 to 0.81 (256 columns of 17 / 400 tokens, k = 704: 6.0 / 6.3 -> 4.4
// / 4.8 us); 64 to 320 0.58 to 1.42.  (Deeper rows would gain as well, 1088 0.70 to 0.83, 1984 0.73 to 0.93, 3008 0.74 to 0.96; the rule
// has not been carried there.)  Rows of an even number of chunks have better tiles: 256 4.6 -> 4.3 us, 1024 the same, 2816 8.2 -> 12.0.
bool one_round_of_blocks(const GemmArgs& a) { return static_cast<int64_t>(a.n / 32) * ((a.m + 31) / 32) <= 256; }
bool takes_rows(const GemmArgs& a) {
  if (a.m > 16) return !a.dual && a.k % 128 != 0 && a.k > 384 && a.k < 1024 && one_round_of_blocks(a);
  return a.m <= (a.n < 8192 ? 16 : a.dual && a.n >= 16384 ? 4 : 8);
}

// With the norm inside, the direct kernel also saves the norm's launch, and pays for it with a load, a conversion and the squares
// for every weight fragment: whole layers behind 512 tokens, norm apart -> inside, 1 / 16 tokens: hidden 256 28.0 -> 21.1 / 28.1 ->
// 22.3 us; 1024 29.5 -> 23.8 / 35.6 -> 29.3; 2048 47.4 -> 42.2 / 56.9 -> 53.3 (the append launch that is saved
// included).  Wide SwiGLU layers are better off with the norm apart: 11008 x 4096 at 1 token 4.8 + 32.5 us against 39.6; and wide
// projections beyond 8 tokens with the tiles (12288 x 4096 at 1 token inside: 23.4 us; apart 4.8 + 18.5, and 4.8 for the append).
// (Both lines are coarse in the depth, us of a projection, apart -> inside: SwiGLU of 12288 rows, 1 / 8 / 16 tokens: 1024 columns -1.5 /
// -1.2 / -2.4, 4096 +0.8 / +1.7 / +3.6, 8192 +2.0 / +4.8 / +11; q/k/v of 4096 rows -2.4 to -5.0 up to 8192 columns, of 6144 +4.7 to +8.8 there.)
// Beyond 16 tokens the direct kernel takes blocks of 32 rows x 32 tokens, and every block reads and squares its tokens itself: it pays
// while rows are short and the blocks fill few rounds of the chip.  A projection alone, norm apart -> inside, us per call, over 17 to
// 256 tokens and 192 to 8192 rows that are one round: 256 columns -2.2 to -2.9, 768 -1.4 to -3.0, 1024 -0.6 to -2.3, 1152 +0.1 to
// -1.8; then q/k/v and SwiGLU of 1024 rows and more: 1280 +0.2 to -1.4 and -0.5 to -1.8, 1408 +0.3 to -1.2 and -0.2 to -1.6, 1536
// +0.8 to -0.8 and 0.0 to -1.5, 1792 +1.2 to -0.7 and +0.3 to -1.0, 2048 +2.1 to -1.0 and +1.4 to -0.8; fewer rows: 1280 +0.5 to
// -0.8, 1536 +1.2 to 0.0, 4096 +8.4 to +4.1.  Rows of an odd number of 64-column chunks would otherwise go to the one tile that can
// walk them: 1344 -1.0 to -3.2, 1984 -0.3 to -3.3, 3264 -0.1 to -3.8, 4032 +1.7 to -3.2.  Two rounds: 512 columns -0.4 to -1.7, 768
// +0.5 to -0.7, 896 +0.4 to +1.9; three: 128 columns -0.1 to -1.1, 256 0.0 to -0.6, 512 +0.6 to +1.5.  Whole layers: hidden 256, 17 /
// 256 tokens 30.4 -> 23.4 / 32.3 -> 26.2 us (the down projection's share of it as above); 1024, 17 / 160 tokens 38.0 -> 35.6 /
// 44.1 -> 42.5.
bool takes_normed_rows(const GemmArgs& a) {
  if (a.m > 16) {
    const int64_t blocks = static_cast<int64_t>(a.n / 32) * ((a.m + 31) / 32);
    if (blocks > 256) return a.k <= (blocks <= 512 ? 832 : blocks <= 768 ? 128 : 0);
    return a.k <= (a.k % 128 != 0 ? 3264 : a.n < 1024 ? 1152 : a.dual ? 1792 : 1408);
  }
  return a.dual ? a.n < 16384 : a.m <= (a.n < 8192 ? 16 : 8);
}

}  // namespace

namespace {

void linear_args(const void* x, const void* w, const void* w2, const void* residual, void* const* out, const int* seg_cols,
                 int n_seg, int64_t m, int64_t n_out, int64_t k, GemmArgs* args) {
  GemmArgs& a = *args;
  a.x = static_cast<const __bf16*>(x);
  a.w = static_cast<const __bf16*>(w);
  a.w2 = static_cast<const __bf16*>(w2);
  a.res = static_cast<const __bf16*>(residual);
  a.n_seg = n_seg;
  int first = 0;
  for (int s = 0; s < 3; ++s) {
    if (s < n_seg) {
      a.seg[s].ptr = static_cast<__bf16*>(out[s]);
      a.seg[s].first = first;
      a.seg[s].end = first + seg_cols[s];
      a.seg[s].ld = seg_cols[s];
      first += seg_cols[s];
    } else {
      a.seg[s] = OutSegment{nullptr, 0, 0, 0};
    }
  }
  a.dual = w2 != nullptr ? 1 : 0;
  a.rope = 0;
  a.rotated = 0;
  a.angles = nullptr;
  a.splits = 1;
  a.scratch = nullptr;
  a.counters = nullptr;
  a.m = static_cast<int>(m);
  a.n = static_cast<int>(a.dual ? 2 * n_out : n_out);
  a.k = static_cast<int>(k);
  a.stagger = 0;   // (for the tile to decide)
}

}  // namespace

int launch_linear(const void* x, const void* w, const void* w2, const void* residual,
                  void* const* out, const int* seg_cols, int n_seg,
                  int64_t m, int64_t n_out, int64_t k, hipStream_t stream, const SharedScratch* shared) {
  GemmArgs a;
  linear_args(x, w, w2, residual, out, seg_cols, n_seg, m, n_out, k, &a);
  if (takes_rows(a)) return a.dual ? launch_rows<kRowsDual, false>(a, stream) : launch_rows<kRowsPlain, false>(a, stream);
  const TileChoice* const whole = choose_tile(a);
  if (n_seg > 1) return whole->launch(a, stream);
  if (shared != nullptr && !a.dual) {
    const TileChoice* const c = choose_split(a, *whole, *shared, &a.splits);
    if (c != nullptr) {
      a.scratch = shared->data;
      a.counters = shared->counters;
      return c->split(a, stream);
    }
  }
  const TwoParts two = choose_two(a, *whole);
  if (two.first == nullptr) return whole->launch(a, stream);
  const int columns = a.dual ? two.columns / 2 : two.columns;   // of the output
  GemmArgs rest = a;
  a.n = two.columns;
  rest.n -= two.columns;
  rest.w += static_cast<int64_t>(columns) * k;
  if (a.dual) rest.w2 += static_cast<int64_t>(columns) * k;
  if (rest.res != nullptr) rest.res += columns;
  rest.seg[0].ptr += columns;
  if (!two.first->ready(a) || !two.second->ready(rest)) return KVRA_ELAUNCH;   // neither goes out
  const int rc = two.first->launch(a, stream);
  return rc != KVRA_OK ? rc : two.second->launch(rest, stream);
}

int launch_norm_qkv_append(const void* x, const void* gain, float eps, void* h, float* angles, const void* wqkv, void* const* out,
                           const int* seg_cols, int64_t position, float rope_base, int head_dim, int64_t m, int64_t k,
                           hipStream_t stream) {
  NormedRowsArgs a;
  linear_args(x, wqkv, nullptr, nullptr, out, seg_cols, 3, m, static_cast<int64_t>(seg_cols[0]) + seg_cols[1] + seg_cols[2], k, &a);
  const bool rotate = rope_base > 0.0f;
  a.rope = head_dim;
  a.rotated = rotate ? seg_cols[0] + seg_cols[1] : 0;
  if (takes_normed_rows(a)) {
    a.gain = static_cast<const __bf16*>(gain);
    a.eps = eps;
    a.position = position;
    const double* const inv = rope_frequencies(rope_base, head_dim);
    for (int i = 0; i < 64; ++i) a.inv_freq[i] = inv[i];
    return launch_rows<kRowsRope, true>(a, stream);
  }
  const int rc = rotate ? launch_rms_norm_angles(x, gain, h, m, static_cast<int>(k), eps, position, head_dim, rope_base, angles, stream)
                        : launch_rms_norm(x, gain, h, m, static_cast<int>(k), eps, stream);
  if (rc != KVRA_OK) return rc;
  a.x = static_cast<const __bf16*>(h);
  a.angles = angles;
  return choose_tile(a)->launch(a, stream);
}

int launch_norm_swiglu(const void* x, const void* gain, float eps, void* h, const void* w_gate, const void* w_up, void* out,
                       int64_t m, int64_t n_out, int64_t k, hipStream_t stream) {
  NormedRowsArgs a;
  const int cols = static_cast<int>(n_out);
  linear_args(x, w_gate, w_up, nullptr, &out, &cols, 1, m, n_out, k, &a);
  if (takes_normed_rows(a)) {
    a.gain = static_cast<const __bf16*>(gain);
    a.eps = eps;
    return launch_rows<kRowsDual, true>(a, stream);
  }
  const int rc = launch_rms_norm(x, gain, h, m, static_cast<int>(k), eps, stream);
  if (rc != KVRA_OK) return rc;
  return launch_linear(h, w_gate, w_up, nullptr, &out, &cols, 1, m, n_out, k, stream);
}

int linear_plan(int64_t m, int64_t n_out, int64_t k, bool dual, LinearPlan* plan) {
  GemmArgs a = {};
  a.dual = dual ? 1 : 0;
  a.m = static_cast<int>(m);
  a.n = static_cast<int>(dual ? 2 * n_out : n_out);
  a.k = static_cast<int>(k);
  if (takes_rows(a)) {
    *plan = a.m > 16 ? LinearPlan{32, 32, 0, 1} : LinearPlan{16, 16, 0, 1};
    return KVRA_OK;
  }
  const TileChoice* c = choose_tile(a);
  const TwoParts two = choose_two(a, *c);
  if (two.first != nullptr) {
    c = two.first;
    a.n = two.columns;
  }
  const int64_t per_xcd = tiles_per_xcd(*c, a);
  const int64_t workgroups = std::min<int64_t>(per_xcd, 32 * c->per_cu);   // of an XCD
  *plan = LinearPlan{c->tn, c->tm, c->tk, static_cast<int>((per_xcd + workgroups - 1) / workgroups)};
  return KVRA_OK;
}

// ---- RMSNorm ------------------------------------------------------------------------------------
// y[t, :] = x[t, :] / sqrt(mean(x[t, :]^2) + eps) * gain, fp32 arithmetic, one workgroup per token.
// HBM-bound: every element is read once and written once with 16-byte accesses.  The gain is on its way with the row (with
// few rows the kernel is a chain of latencies), and there is a variant for one, two and four pieces per thread: with four in all
// of them a narrow row spends its time on branches around pieces that it does not have (and the early gain doubles
// those).  Gain late, four -> gain early, four -> as it is: 5208 x 256 4.9 -> 5.5 -> 4.0 us; 4000 x 1024 5.2 -> 5.5 -> 4.5;
// 1898 x 2048 4.15 -> 4.3 -> 3.9; 5824 x 4096 15.3 -> 14.7 -> 14.7 (6.5 TB/s).
struct NormArgs {
  const __bf16* x;
  const __bf16* gain;
  __bf16* y;
  int rows;
  int hidden;
  float eps;
};
struct NormAngleArgs : NormArgs {
  float* angles;           // [rows][head_dim]: cos of a token's head_dim / 2 angles, then their sin
  int head_dim;
  long long position;      // of the first row
  double inv_freq[64];
};

constexpr int kNormThreads = 256;
constexpr int kNormMaxPieces = 4;   // 16-byte pieces a thread keeps in registers: hidden <= 8192

// The last wave of a row also forms the angles of its token for the projection that follows, while the row is on its way.
__device__ __forceinline__ void norm_angles(const NormArgs&, int) {}
__device__ __forceinline__ void norm_angles(const NormAngleArgs& a, int tid) {
  const int i = tid - (kNormThreads - 64);
  if (i < 0 || i >= a.head_dim / 2) return;
  float* const row = a.angles + static_cast<long long>(blockIdx.x) * a.head_dim;
  rope_angle(static_cast<double>(a.position + blockIdx.x) * a.inv_freq[i], row + i, row + a.head_dim / 2 + i);
}

template <int PIECES, class Args>   // at most so many per thread
__global__ __launch_bounds__(kNormThreads) void rms_norm_kernel(Args a) {
  __shared__ float part[kNormThreads / 64];
  const int tid = threadIdx.x;
  const int pieces = a.hidden / 8;
  const bf16x8* xr = reinterpret_cast<const bf16x8*>(a.x + static_cast<long long>(blockIdx.x) * a.hidden);
  const bf16x8* gr = reinterpret_cast<const bf16x8*>(a.gain);
  bf16x8 v[PIECES], g[PIECES];
  float ss = 0.0f;
#pragma unroll
  for (int i = 0; i < PIECES; ++i) {
    const int p = tid + i * kNormThreads;
    if (p < pieces) {
      v[i] = xr[p];
      g[i] = gr[p];
    }
  }
  norm_angles(a, tid);
#pragma unroll
  for (int i = 0; i < PIECES; ++i) {
    if (tid + i * kNormThreads < pieces) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float f = static_cast<float>(v[i][e]);
        ss = fmaf(f, f, ss);
      }
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) ss += __shfl_xor(ss, off);
  if ((tid & 63) == 0) part[tid >> 6] = ss;
  __syncthreads();
  float tot = 0.0f;
#pragma unroll
  for (int w = 0; w < kNormThreads / 64; ++w) tot += part[w];
  const float rinv = 1.0f / sqrtf(tot / static_cast<float>(a.hidden) + a.eps);
  bf16x8* yr = reinterpret_cast<bf16x8*>(a.y + static_cast<long long>(blockIdx.x) * a.hidden);
#pragma unroll
  for (int i = 0; i < PIECES; ++i) {
    const int p = tid + i * kNormThreads;
    if (p < pieces) {
      bf16x8 o;
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = static_cast<__bf16>(static_cast<float>(v[i][e]) * rinv * static_cast<float>(g[i][e]));
      yr[p] = o;
    }
  }
}

namespace {

template <class Args>
int launch_norm(Args& a, const void* x, const void* gain, void* y, int64_t rows, int hidden, float eps, hipStream_t stream) {
  a.x = static_cast<const __bf16*>(x);
  a.gain = static_cast<const __bf16*>(gain);
  a.y = static_cast<__bf16*>(y);
  a.rows = static_cast<int>(rows);
  a.hidden = hidden;
  a.eps = eps;
  const dim3 grid(static_cast<unsigned>(rows)), block(kNormThreads);
  const int per_thread = (hidden / 8 + kNormThreads - 1) / kNormThreads;
  if (per_thread == 1) return launch_kernel(rms_norm_kernel<1, Args>, grid, block, a, stream);
  if (per_thread == 2) return launch_kernel(rms_norm_kernel<2, Args>, grid, block, a, stream);
  return launch_kernel(rms_norm_kernel<kNormMaxPieces, Args>, grid, block, a, stream);
}

}  // namespace

int launch_rms_norm(const void* x, const void* gain, void* y, int64_t rows, int hidden, float eps, hipStream_t stream) {
  NormArgs a;
  return launch_norm(a, x, gain, y, rows, hidden, eps, stream);
}

int launch_rms_norm_angles(const void* x, const void* gain, void* y, int64_t rows, int hidden, float eps, int64_t position,
                           int head_dim, float rope_base, float* angles, hipStream_t stream) {
  NormAngleArgs a;
  a.angles = angles;
  a.head_dim = head_dim;
  a.position = position;
  const double* const inv = rope_frequencies(rope_base, head_dim);
  for (int i = 0; i < 64; ++i) a.inv_freq[i] = inv[i];
  return launch_norm(a, x, gain, y, rows, hidden, eps, stream);
}

int rms_norm_max_hidden() { return kNormThreads * kNormMaxPieces * 8; }

}  // namespace kvra
