// The attention launch for few rows (short chunks: an extension step, a follow-up turn, a short prompt; few heads): the
// same products, roundings and merge as chunk_attn_kernel (kvra_attn.hip), another split of the work.
//
// What bounds it.  With few rows there is little to do per key and the time goes into latencies, one after the other, and
// into the K/V stream.  chunk_attn_kernel gives 256 rows to a workgroup whose waves walk all keys together, a barrier or two
// per key tile: with one slice of 32 rows seven of its eight waves only help to stage, and a launch of a few such units is a
// chain of tile steps.  Here a workgroup owns ONE slice of 32 virtual rows (token * G + head in group) and its eight waves
// share out the KEY tiles (wave w: tiles w, w + 8, ...), so that the chain is an eighth as long; nothing is shared between
// waves until the end and there is no barrier in the loop.  Each wave has its own K tile in registers and its own V tile in
// LDS (the transposing reads need it there): 32 KB per wave are in flight, 256 KB per CU, which is what the memory needs to
// stay busy.  K goes through a small LDS buffer of the wave, 16 keys at a time, from the order that loads whole rows to the
// operand layout: loaded in operand layout, 16 neighbouring lanes ask for 16 different rows, and the address
// unit, not the memory, sets the pace (32 heads x 128, 77 tokens behind 5824: 37.5 us; as it is 30.5, tiled kernel 36.8).  The price is that every slice reads its K/V through
// the L2 (32 FLOP per byte): the rule that takes a launch here (rows_splits) weighs that.
// The eight partial results meet in LDS; where there are fewer slices than CUs the key tiles are also split over
// workgroups, which meet through the scratch like the pieces of chunk_attn_kernel do.
#include "kvra_attn_device.h"

#include <algorithm>

namespace kvra {

constexpr int kRowsWaves = 8;
constexpr int kRowsThreads = 64 * kRowsWaves;
constexpr int kRowsKeys = 64;          // keys of a tile

struct RowsArgs {
  const __bf16* q;
  const __bf16* k;
  const __bf16* v;
  __bf16* out;
  int prefix;
  int chunk;
  int H;
  int Hkv;
  int G;
  int slices;        // slices of 32 virtual rows per kv head
  int splits;        // workgroups that share the key tiles of a slice
  int by_xcd;        // Hkv * splits is a multiple of 8: the slices of a (head, split) pair share an XCD
  float c_log2;      // scale * log2(e)
  float* scratch;    // splits > 1: rows_slot_floats(D) per workgroup
  int* counters;     // splits > 1: pieces counted so far, one per slice; all zero between launches
};

constexpr int rows_slot_floats(int D) { return (D / 32 * 16 + 2) * 64; }

template <int D>
__global__ __launch_bounds__(kRowsThreads, 2) void attn_rows_kernel(RowsArgs a) {
  constexpr int BN = kRowsKeys;
  constexpr int KB = BN / 16;              // 16-key blocks of a tile
  constexpr int CPR = D / 8;               // 16-byte pieces per K/V row
  constexpr int KS = D / 32;               // contraction steps of S^T = K Q^T
  constexpr int DB = D / 16;               // 16-row blocks of O^T
  constexpr int QB = 2;                    // 16-query blocks of a slice
  constexpr int RPB = 256 / (D * 2);       // rows per 256-byte LDS bank span
  constexpr int TILE_BYTES = BN * D * 2;
  constexpr int LOADS = BN * CPR / 64;     // wave loads per V tile
  constexpr int RPL = 64 / CPR;            // rows one wave load moves
  constexpr int R = DB * QB * 4;           // registers of O per lane
  constexpr int RW = R / kRowsWaves;       // of which a wave merges this many
  static_assert(R * 64 * 4 == TILE_BYTES, "a wave's O takes the place of its V tile");
  constexpr int K_BYTES = 16 * D * 2;      // a wave's buffer for 16 keys of K
  // LDS, all of it: the V tiles of the waves, then their K buffers
  extern __shared__ u32x4 smem[];
  char* const lds = reinterpret_cast<char*>(smem);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform by construction
  const int n = lane & 15, g4 = lane >> 4;

  // workgroup -> (kv head, split, slice); ids go round-robin over the 8 XCDs.  Last slices first: they see the most keys.
  int pair, slice;
  if (a.by_xcd) {
    const int rest = blockIdx.x >> 3;
    slice = a.slices - 1 - rest % a.slices;
    pair = (blockIdx.x & 7) + 8 * (rest / a.slices);
  } else {
    const int pairs = a.Hkv * a.splits;
    slice = a.slices - 1 - blockIdx.x / pairs;
    pair = blockIdx.x % pairs;
  }
  const int g = pair / a.splits, split = pair - g * a.splits;

  const int VR = a.chunk * a.G, total = a.prefix + a.chunk;
  const int v0 = slice * 32, row_hi = min(v0 + 32, VR);
  const int wmin = a.prefix + v0 / a.G;                 // last visible key of the slice's first and last row
  const int wmax = a.prefix + (row_hi - 1) / a.G;
  const int tiles = wmax / BN + 1;
  const int t_lo = static_cast<int>(static_cast<long long>(tiles) * split / a.splits);
  const int t_hi = static_cast<int>(static_cast<long long>(tiles) * (split + 1) / a.splits);

  // lane-constant byte offsets inside a tile.  Piece p = 64 i + lane of a tile = (row p / CPR, slot p % CPR); the lane that
  // owns slot (row, slot) fetches column piece slot ^ f(row), so that the reads below are free of bank conflicts (the same f
  // as in chunk_attn_kernel; it repeats every 16 / RPL loads for K, every second one for V)
  // Only the first of each set of addresses is kept: the others differ from it by an XOR (of the piece) and a multiple of the
  // row step, formed where they are used.
  constexpr int KP = 16 / RPL;             // wave loads per 16 keys
  static_assert(16 % (RPB * CPR) == 0 && 2 * RPL % (RPB * CPR / 2) == 0, "where f(row) repeats");
  const unsigned row_bytes = static_cast<unsigned>(a.Hkv) * D * 2;
  const unsigned load_row = static_cast<unsigned>(lane / CPR) * row_bytes;
  const unsigned k_off = load_row + static_cast<unsigned>(lane % CPR ^ lane / CPR / RPB) * 16;
  const unsigned v_off = load_row + static_cast<unsigned>(lane % CPR ^ 2 * (lane / CPR / RPB % (CPR / 2))) * 16;
  constexpr unsigned V_XOR = D == 128 ? 128 : 0;   // of every second V load
  const unsigned lds0 = static_cast<unsigned>(reinterpret_cast<uintptr_t>((lds_void*)smem)) + wave * TILE_BYTES;
  char* const k_buf = lds + kRowsWaves * TILE_BYTES + wave * K_BYTES;
  const unsigned k_addr = static_cast<unsigned>(n * CPR + (g4 ^ n / RPB % CPR)) * 16;
  const int v_row = 4 * g4 + (n >> 2);
  const unsigned v_addr = lds0 + static_cast<unsigned>(v_row * CPR + ((n & 3) >> 1 ^ 2 * (v_row / RPB % (CPR / 2)))) * 16 + (n & 1) * 8;
  auto uniform = [](unsigned v) __attribute__((always_inline)) -> unsigned {
    return static_cast<unsigned>(__builtin_amdgcn_readfirstlane(static_cast<int>(v)));
  };
  // first byte of tile t of this head in a cache, and the bytes from there to the end of the rows that exist (at most a tile)
  auto tile_at = [&](const __bf16* cache, int t) __attribute__((always_inline)) -> unsigned long long {
    return reinterpret_cast<unsigned long long>(cache + static_cast<long long>(g) * D) +
           static_cast<unsigned long long>(t) * BN * row_bytes;
  };
  auto tile_bytes = [&](int t) __attribute__((always_inline)) -> unsigned { return min(total - t * BN, BN) * row_bytes; };

  u32x4 kf[LOADS];
  auto load_k = [&](int t) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t res = __builtin_amdgcn_make_buffer_rsrc(
        reinterpret_cast<void*>(tile_at(a.k, t)), 0, static_cast<int>(tile_bytes(t)), 0x00020000);
    unsigned off = k_off, step = RPL * row_bytes;
    asm volatile("" : "+v"(off), "+s"(step));   // (opaque, so that nothing is formed ahead and kept through the loop)
#pragma unroll
    for (int i = 0; i < LOADS; ++i)
      kf[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(res, static_cast<int>((off ^ 64u * (i % KP)) + i * step), 0, 0));
  };
  auto load_v = [&](int t) __attribute__((always_inline)) {
    const unsigned long long at = tile_at(a.v, t);
    const u32x4 res = {uniform(static_cast<unsigned>(at)), uniform(static_cast<unsigned>(at >> 32) & 0xFFFFu),
                       uniform(tile_bytes(t)), 0x00020000u};
    unsigned off = v_off, step = RPL * row_bytes;
    asm volatile("" : "+v"(off), "+s"(step));
#pragma unroll
    for (int i = 0; i < LOADS; ++i) lds_dma16(res, (off ^ V_XOR * (i & 1)) + i * step, lds0 + i * 1024);
  };

  int t = t_lo + wave;
  if (t < t_hi) {
    load_k(t);
    load_v(t);
  }

  // Q fragments: B operand of S^T, lane (n, g4) holds Q[row n][32 ks + 8 g4 .. +7], times scale * log2(e) (rounded to bf16
  // again); rows past the end repeat the last one
  bf16x8 qf[KS][QB];
  int qpos[QB];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const int vr = min(v0 + 16 * qb + n, row_hi - 1), r = vr / a.G, h = g * a.G + (vr - r * a.G);
    qpos[qb] = a.prefix + r;
    const __bf16* qrow = a.q + (static_cast<long long>(r) * a.H + h) * D;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8 raw = *reinterpret_cast<const bf16x8*>(qrow + 32 * ks + 8 * g4);
#pragma unroll
      for (int e = 0; e < 8; ++e) qf[ks][qb][e] = static_cast<__bf16>(static_cast<float>(raw[e]) * a.c_log2);
    }
  }

  f32x4 o[DB][QB];
  float m[QB], l[QB];   // l: of this lane's quarter of the keys
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    m[qb] = kNoKeyYet;
    l[qb] = 0.0f;
#pragma unroll
    for (int db = 0; db < DB; ++db) o[db][qb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  }

  for (; t < t_hi; t += kRowsWaves) {
    f32x4 s[KB][QB];
    // 16 keys at a time through the wave's buffer (LDS operations of a wave are carried out in order)
    auto put_k = [&](int kb) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < KP; ++i) *reinterpret_cast<u32x4*>(k_buf + i * 1024 + lane * 16) = kf[kb * KP + i];
    };
    put_k(0);
    unsigned ka = k_addr, va = v_addr;
    asm volatile("" : "+v"(ka), "+v"(va));
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      bf16x8 kq[KS];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) kq[ks] = *reinterpret_cast<const bf16x8*>(k_buf + (ka ^ 64u * ks));
      if (kb + 1 < KB) put_k(kb + 1);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
          s[kb][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kq[ks], qf[ks][qb], ks == 0 ? f32x4{0.0f, 0.0f, 0.0f, 0.0f} : s[kb][qb], 0, 0, 0);
    }
    // the V tile was sent for right behind this K tile: it has landed, or is about to
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    const bool more = t + kRowsWaves < t_hi;
    if (more) load_k(t + kRowsWaves);

    // register e of block (kb, qb) is key  t*BN + 16 kb + 4 g4 + e  of query 16 qb + n
    if (t * BN + BN - 1 > wmin) {
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        const int rel = qpos[qb] - t * BN - 4 * g4;   // largest still-visible key offset (minus 4 g4)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (16 * kb + e > rel) s[kb][qb][e] = -INFINITY;
      }
    }
    u32x4 pf[KB / 2][QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      float tmax = s[0][qb][0];
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int e = 0; e < 4; ++e) tmax = fmaxf(tmax, s[kb][qb][e]);
      tmax = fmaxf(tmax, other_half(tmax));
      tmax = fmaxf(tmax, other_row(tmax));
      const float mn = fmaxf(m[qb], tmax);             // a row that has met no visible key stays at kNoKeyYet: weights 0
      const float alpha = __builtin_amdgcn_exp2f(m[qb] - mn);
      m[qb] = mn;
      float psum = 0.0f;
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int e = 0; e < 4; e += 2) {
          typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
          const float p0 = __builtin_amdgcn_exp2f(s[kb][qb][e] - mn), p1 = __builtin_amdgcn_exp2f(s[kb][qb][e + 1] - mn);
          psum += p0 + p1;
          const bf16x2 pp = {static_cast<__bf16>(p0), static_cast<__bf16>(p1)};
          pf[kb / 2][qb][2 * (kb % 2) + e / 2] = __builtin_bit_cast(unsigned, pp);
        }
      l[qb] = fmaf(l[qb], alpha, psum);
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int e = 0; e < 4; ++e) o[db][qb][e] *= alpha;
    }
    // contraction slot 8 g4 + 4 b + u of step kk is key 32 kk + 16 b + 4 g4 + u on both operands; reads kept PF ahead of the
    // MFMAs and nothing moved across (left to itself the compiler hoists them all, and spills)
    constexpr int NV = KB / 2 * DB, PF = 4;
    auto vread = [&](int i) __attribute__((always_inline)) -> bf16x8 {
      s16x8 vf;
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const s16x4 u = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (lds_s16x4*)static_cast<uintptr_t>((va ^ 32u * (i % DB)) + (32 * (i / DB) + 16 * b) * CPR * 16));
        vf[4 * b + 0] = u[0]; vf[4 * b + 1] = u[1]; vf[4 * b + 2] = u[2]; vf[4 * b + 3] = u[3];
      }
      return __builtin_bit_cast(bf16x8, vf);
    };
    __builtin_amdgcn_sched_barrier(0);
    bf16x8 vq[PF];
#pragma unroll
    for (int i = 0; i < PF; ++i) vq[i] = vread(i);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const bf16x8 cur = vq[i % PF];
      if (i + PF < NV) vq[i % PF] = vread(i + PF);
#pragma unroll
      for (int qb = 0; qb < QB; ++qb)
        o[i % DB][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cur, __builtin_bit_cast(bf16x8, pf[i / DB][qb]), o[i % DB][qb], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    // every read of this V tile is back before the next one is sent to its place
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (more) load_v(t + kRowsWaves);
  }

  // ---- the eight waves' results meet in LDS: wave w merges registers RW w .. of all of them ------------------------
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {        // the whole row's sum, in each of the row's four lanes
    l[qb] += other_half(l[qb]);
    l[qb] += other_row(l[qb]);
    if (g4 == qb) {                        // (to the wave's K buffer, which it has finished with)
      reinterpret_cast<float*>(k_buf)[16 * qb + n] = m[qb];
      reinterpret_cast<float*>(k_buf)[32 + 16 * qb + n] = l[qb];
    }
  }
  auto wave_ml = [&](int w, int i) __attribute__((always_inline)) -> float {
    return reinterpret_cast<const float*>(lds + kRowsWaves * TILE_BYTES + w * K_BYTES)[i];
  };
  float* const lds_o = reinterpret_cast<float*>(smem);   // [wave][register][lane]: a wave's own part is its own V tile
#pragma unroll
  for (int i = 0; i < R; ++i) lds_o[(wave * R + i) * 64 + lane] = o[i / 8][i / 4 % 2][i % 4];
  __syncthreads();
  const int r0 = wave * RW;                              // register (db * QB + qb) * 4 + e
  constexpr int QW = RW >= 8 ? 2 : 1;                    // query blocks this wave's registers belong to
  const int qb0 = QW == 2 ? 0 : r0 / 4 % 2;
  float acc[RW], am[QW], al[QW];
#pragma unroll
  for (int j = 0; j < QW; ++j) {
    const int row = 16 * (qb0 + j) + n;
    float mw[kRowsWaves];
    am[j] = kNoKeyYet;
    al[j] = 0.0f;
#pragma unroll
    for (int w = 0; w < kRowsWaves; ++w) {
      mw[w] = wave_ml(w, row);
      am[j] = fmaxf(am[j], mw[w]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[4 * j + i] = 0.0f;
#pragma unroll
    for (int w = 0; w < kRowsWaves; ++w) {
      const float weight = __builtin_amdgcn_exp2f(mw[w] - am[j]);
      al[j] = fmaf(wave_ml(w, 32 + row), weight, al[j]);
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[4 * j + i] = fmaf(lds_o[(w * R + r0 + 4 * j + i) * 64 + lane], weight, acc[4 * j + i]);
    }
  }
  static_assert(RW == 4 * QW, "");

  if (a.splits > 1) {
    // as between the pieces of chunk_attn_kernel: device-coherent stores, acknowledged before the piece is counted; the
    // piece that completes the count merges all of them in their order
    const int unit = g * a.slices + slice;
    float* const slots = a.scratch + static_cast<long long>(unit) * a.splits * rows_slot_floats(D);
    float* const mine = slots + static_cast<long long>(split) * rows_slot_floats(D);
#pragma unroll
    for (int i = 0; i < RW; ++i) store_coherent(mine + (r0 + i) * 64 + lane, acc[i]);
#pragma unroll
    for (int j = 0; j < QW; ++j)
      if (wave < 2 / QW && g4 == 0) {       // (d = 128: wave 0 has both query blocks; d = 64: waves 0 and 1 one each)
        store_coherent(mine + R * 64 + 16 * (qb0 + j) + n, am[j]);
        store_coherent(mine + R * 64 + 64 + 16 * (qb0 + j) + n, al[j]);
      }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    int* const last_flag = reinterpret_cast<int*>(lds + kRowsWaves * TILE_BYTES) + 64;   // behind m and l of wave 0
    if (tid == 0) *last_flag = atomicAdd(a.counters + unit, 1) == a.splits - 1 ? 1 : 0;
    __syncthreads();
    if (*last_flag == 0) return;
    if (tid == 0) a.counters[unit] = 0;     // ready for the next launch
#pragma unroll
    for (int j = 0; j < QW; ++j) {
      am[j] = kNoKeyYet;
      al[j] = 0.0f;
    }
#pragma unroll
    for (int i = 0; i < RW; ++i) acc[i] = 0.0f;
    constexpr int AHEAD = 8;                // partial results on their way together
    for (int p0 = 0; p0 < a.splits; p0 += AHEAD) {
      float pv[AHEAD][RW], pm[AHEAD][QW], pl[AHEAD][QW];
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) {
        const float* p = slots + static_cast<long long>(min(p0 + u, a.splits - 1)) * rows_slot_floats(D);
#pragma unroll
        for (int i = 0; i < RW; ++i) pv[u][i] = load_coherent(p + (r0 + i) * 64 + lane);
#pragma unroll
        for (int j = 0; j < QW; ++j) {
          pm[u][j] = load_coherent(p + R * 64 + 16 * (qb0 + j) + n);
          pl[u][j] = load_coherent(p + R * 64 + 64 + 16 * (qb0 + j) + n);
        }
      }
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) {
        if (p0 + u >= a.splits) break;
#pragma unroll
        for (int j = 0; j < QW; ++j) {
          const float mn = fmaxf(am[j], pm[u][j]);
          const float wa = __builtin_amdgcn_exp2f(am[j] - mn), wb = __builtin_amdgcn_exp2f(pm[u][j] - mn);
          am[j] = mn;
          al[j] = fmaf(pl[u][j], wb, al[j] * wa);
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[4 * j + i] = fmaf(pv[u][4 * j + i], wb, acc[4 * j + i] * wa);
        }
      }
    }
  }

  // register e of block (db, qb) is column 16 db + 4 g4 + e of row n
#pragma unroll
  for (int j = 0; j < QW; ++j) {
    const int vr = v0 + 16 * (qb0 + j) + n, db = r0 / 8;
    if (vr >= row_hi) continue;
    const int r = vr / a.G, h = g * a.G + (vr - r * a.G);
    const float inv = 1.0f / al[j];
    bf16x4 w;
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = static_cast<__bf16>(acc[4 * j + e] * inv);
    *reinterpret_cast<bf16x4*>(a.out + (static_cast<long long>(r) * a.H + h) * D + 16 * db + 4 * g4) = w;
  }
}

int64_t attn_rows_slot_bytes(int head_dim) { return static_cast<int64_t>(rows_slot_floats(head_dim)) * sizeof(float); }

int launch_attn_rows(const void* q, const void* k_cache, const void* v_cache, int64_t prefix_len, int64_t chunk_len,
                     int n_q_heads, int n_kv_heads, int head_dim, float scale, void* out, int splits, float* scratch,
                     int* counters, hipStream_t stream) {
  RowsArgs a;
  a.q = static_cast<const __bf16*>(q);
  a.k = static_cast<const __bf16*>(k_cache);
  a.v = static_cast<const __bf16*>(v_cache);
  a.out = static_cast<__bf16*>(out);
  a.prefix = static_cast<int>(prefix_len);
  a.chunk = static_cast<int>(chunk_len);
  a.H = n_q_heads;
  a.Hkv = n_kv_heads;
  a.G = n_q_heads / n_kv_heads;
  a.slices = static_cast<int>((chunk_len * a.G + 31) / 32);
  a.splits = splits;
  a.by_xcd = n_kv_heads * splits % 8 == 0 ? 1 : 0;
  a.c_log2 = scale * 1.4426950408889634f;
  a.scratch = scratch;
  a.counters = counters;
  const dim3 grid(static_cast<unsigned>(a.slices) * static_cast<unsigned>(n_kv_heads * splits)), block(kRowsThreads);
  const unsigned smem = kRowsWaves * (kRowsKeys + 16) * static_cast<unsigned>(head_dim) * 2u;   // V tiles, K buffers
  return head_dim == 128 ? launch_kernel(attn_rows_kernel<128>, grid, block, a, stream, smem)
                         : launch_kernel(attn_rows_kernel<64>, grid, block, a, stream, smem);
}

}  // namespace kvra
