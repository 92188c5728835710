// kvra_append_kv: rotary embedding + KV-cache population of one chunk (App. C listing, cache
// concatenation step; Sec. 4.3 contiguity).  HBM-bound streaming kernel: every byte of K, V
// (and Q) is read once and written once with 128-bit accesses.
#include "kvra_rope_device.h"

namespace kvra {

typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));

struct AppendArgs {
  const unsigned short* k_in;
  const unsigned short* v_in;
  unsigned short* q;        // may be null
  unsigned short* k_cache;
  unsigned short* v_cache;
  long long prefix_len;
  int chunk_len;
  int n_q_heads;
  int n_kv_heads;
  int use_rope;
  double inv_freq[64];      // base^(-2i/d), i < d/2, formed on the host in fp64
};

__device__ __forceinline__ float bf16_to_f32(unsigned short b) {
  return __uint_as_float(static_cast<unsigned int>(b) << 16);
}

__device__ __forceinline__ unsigned short f32_to_bf16_rne(float x) {
  // round to nearest, ties to even, on the bit pattern; a NaN stays a (quiet) NaN instead of
  // being carried into an infinity or a zero by the rounding increment
  unsigned int u = __float_as_uint(x);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return static_cast<unsigned short>((u >> 16) | 0x0040u);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return static_cast<unsigned short>(u >> 16);
}

// One workgroup serves TOK consecutive tokens (TOK * D/2 <= 256): TOK * D/2 threads form cos/sin of
// (prefix + row) * inv_freq[i] in fp64 and park them in LDS as fp32; all threads move "pair units" (a 16-byte piece of the
// low half of a head row and its partner in the high half) of K and Q, and plain 16-byte pieces of V.
// A short chunk is a chain of latencies, not of traffic, so everything a thread needs first - its frequency (from the
// kernel arguments), its first pieces of V and its first units of K and Q - is loaded together, ahead of the angles.
// Long chunks use the largest TOK (every thread has an angle); short ones use fewer tokens per workgroup so that the launch
// still puts several workgroups on every CU.  Before (V, then the library's sincos, then K, then Q) -> after, back to back
// launches: 160 tokens, 2 heads x 64: 4.4 -> 3.4 us; 1003 tokens, 71 heads on 1: 7.6 -> 5.3; 1024 tokens, 32 heads x 128: 9.3
// -> 8.2; 5824 tokens: 43.2 -> 43.0 (6.7 TB/s, much of it from the last-level cache).
// Without rotation nothing waits for angles, and V and K are two plain copies: loaded together like the rest, 1183 tokens of 32
// heads took 6.0 us, one after the other 5.3 (two streams of a read and a write each overlap better across waves than one of
// four).  With rotation but without queries V leaves before the angles: 1132 tokens 6.6 -> 6.45 us (6.2 before either).
template <int D, int TOK>
__global__ __launch_bounds__(256) void append_kv_kernel(AppendArgs a) {
  constexpr int HALF = D / 2;
  static_assert(TOK * HALF <= 256, "one thread per (token, frequency)");
  constexpr int PAIRS = D / 16;            // pair units per head row
  constexpr int CHUNKS = D / 8;            // 16-byte pieces per head row
  constexpr int AHEAD = 2;                 // pieces and units of a thread on their way together
  __shared__ float cs[TOK][HALF];
  __shared__ float sn[TOK][HALF];

  const int tid = threadIdx.x;
  const int tok0 = blockIdx.x * TOK;
  const int ntok = min(TOK, a.chunk_len - tok0);
  const int Hkv = a.n_kv_heads, H = a.n_q_heads;

  // V: bit-exact copy; without rotation K as well
  const int v_total = ntok * Hkv * CHUNKS;
  const long long from = static_cast<long long>(tok0) * Hkv * CHUNKS, to = (a.prefix_len + tok0) * Hkv * CHUNKS;
  const u16x8* v_src = reinterpret_cast<const u16x8*>(a.v_in) + from;
  u16x8* v_dst = reinterpret_cast<u16x8*>(a.v_cache) + to;
  if (!a.use_rope) {
#pragma unroll 4
    for (int u = tid; u < v_total; u += 256) v_dst[u] = v_src[u];
    const u16x8* k_src = reinterpret_cast<const u16x8*>(a.k_in) + from;
    u16x8* k_dst = reinterpret_cast<u16x8*>(a.k_cache) + to;
    for (int u = tid; u < v_total; u += 512) {
      const u16x8 k0 = k_src[u], k1 = k_src[min(u + 256, v_total - 1)];
      k_dst[u] = k0;
      if (u + 256 < v_total) k_dst[u + 256] = k1;
    }
    return;
  }

  const int t_mine = tid / HALF;
  const bool has_angle = t_mine < ntok;
  double freq = 0.0;
  if (has_angle) freq = a.inv_freq[tid % HALF];

  u16x8 v[AHEAD];
#pragma unroll
  for (int i = 0; i < AHEAD; ++i)
    if (tid + 256 * i < v_total) v[i] = v_src[tid + 256 * i];

  auto store_v = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < AHEAD; ++i)
      if (tid + 256 * i < v_total) v_dst[tid + 256 * i] = v[i];
  };

  // units of a token: those of its K heads, which go to the cache, then those of its Q heads, in place
  const int heads = Hkv + (a.q != nullptr ? H : 0);
  const int per_tok = heads * PAIRS, total = ntok * per_tok;
  u16x8 lo[AHEAD], hi[AHEAD];
  unsigned short* dst[AHEAD];
  int where[AHEAD];                        // offset of the unit's cos/sin, in floats
  auto load_units = [&](int u0) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) {
      const int u = u0 + 256 * i;
      if (u >= total) break;
      const int t = TOK == 1 ? 0 : u / per_tok;
      const int rem = u - t * per_tok;
      const int head = rem / PAIRS, j = rem % PAIRS;
      const unsigned short* src;
      if (head < Hkv) {
        src = a.k_in + (static_cast<long long>(tok0 + t) * Hkv + head) * D + 8 * j;
        dst[i] = a.k_cache + ((a.prefix_len + tok0 + t) * Hkv + head) * D + 8 * j;
      } else {
        dst[i] = a.q + (static_cast<long long>(tok0 + t) * H + (head - Hkv)) * D + 8 * j;
        src = dst[i];
      }
      where[i] = t * HALF + 8 * j;
      lo[i] = *reinterpret_cast<const u16x8*>(src);
      hi[i] = *reinterpret_cast<const u16x8*>(src + HALF);
    }
  };
  load_units(tid);
  // One wait for all of it: behind the branches above the compiler does not know how many loads are on their way, and would
  // wait for everything, the stores before included, ahead of each store (1132 tokens, 32 heads x 128: 9.3 us, so 9.1).
  __builtin_amdgcn_s_waitcnt(0x0F70);
  // Without queries V is half of what is moved: it leaves before the angles are worked out.
  if (a.q == nullptr) store_v();

  if (has_angle) {
    const double phi = static_cast<double>(a.prefix_len + tok0 + t_mine) * freq;
    rope_angle(phi, &cs[t_mine][tid % HALF], &sn[t_mine][tid % HALF]);
  }
  __syncthreads();

  if (a.q != nullptr) store_v();
  for (int u0 = tid; u0 < total; u0 += 256 * AHEAD) {
    if (u0 != tid) load_units(u0);
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) {
      if (u0 + 256 * i >= total) break;
      const float* c = &cs[0][0] + where[i];
      const float* s = &sn[0][0] + where[i];
      u16x8 olo, ohi;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float x0 = bf16_to_f32(lo[i][e]), x1 = bf16_to_f32(hi[i][e]);
        olo[e] = f32_to_bf16_rne(fmaf(x0, c[e], -(x1 * s[e])));
        ohi[e] = f32_to_bf16_rne(fmaf(x1, c[e], x0 * s[e]));
      }
      *reinterpret_cast<u16x8*>(dst[i]) = olo;
      *reinterpret_cast<u16x8*>(dst[i] + HALF) = ohi;
    }
  }
#pragma unroll 4
  for (int u = tid + 256 * AHEAD; u < v_total; u += 256) v_dst[u] = v_src[u];
}

const double* rope_frequencies(float rope_base, int head_dim) {
  // a program calls with one base and head size: the powers (0.9 us of a 4 us call) are formed when either changes
  struct Frequencies {
    float base = 0.0f;
    int head_dim = 0;
    double inv[64] = {};
  };
  static thread_local Frequencies f;
  if (rope_base > 0.0f && (f.base != rope_base || f.head_dim != head_dim)) {
    for (int i = 0; i < head_dim / 2; ++i) f.inv[i] = std::pow(static_cast<double>(rope_base), -2.0 * i / head_dim);
    f.base = rope_base;
    f.head_dim = head_dim;
  }
  return f.inv;
}

int launch_append_kv(const void* k_in, const void* v_in, void* q_inout, void* k_cache, void* v_cache,
                     int64_t prefix_len, int64_t chunk_len, int n_q_heads, int n_kv_heads, int head_dim,
                     float rope_base, hipStream_t stream) {
  AppendArgs a;
  a.k_in = static_cast<const unsigned short*>(k_in);
  a.v_in = static_cast<const unsigned short*>(v_in);
  a.q = static_cast<unsigned short*>(q_inout);
  a.k_cache = static_cast<unsigned short*>(k_cache);
  a.v_cache = static_cast<unsigned short*>(v_cache);
  a.prefix_len = prefix_len;
  a.chunk_len = static_cast<int>(chunk_len);
  a.n_q_heads = n_q_heads;
  a.n_kv_heads = n_kv_heads;
  a.use_rope = rope_base > 0.0f ? 1 : 0;
  const double* const inv = rope_frequencies(rope_base, head_dim);   // (without rotation nothing reads them)
  for (int i = 0; i < 64; ++i) a.inv_freq[i] = inv[i];
  // tokens per workgroup: the most that phase 1 can serve, halved until the grid holds about
  // eight workgroups per CU (256 CUs) or one token per workgroup is reached
  int tok = 256 / (head_dim / 2);
  while (tok > 1 && (chunk_len + tok - 1) / tok < 2048) tok >>= 1;
  const unsigned grid = static_cast<unsigned>((chunk_len + tok - 1) / tok);
  const dim3 g(grid), b(256);
  if (head_dim == 128) {
    if (tok == 4) return launch_kernel(append_kv_kernel<128, 4>, g, b, a, stream);
    if (tok == 2) return launch_kernel(append_kv_kernel<128, 2>, g, b, a, stream);
    return launch_kernel(append_kv_kernel<128, 1>, g, b, a, stream);
  }
  if (tok == 8) return launch_kernel(append_kv_kernel<64, 8>, g, b, a, stream);
  if (tok == 4) return launch_kernel(append_kv_kernel<64, 4>, g, b, a, stream);
  if (tok == 2) return launch_kernel(append_kv_kernel<64, 2>, g, b, a, stream);
  return launch_kernel(append_kv_kernel<64, 1>, g, b, a, stream);
}

}  // namespace kvra
