// Row-wise kernels of the decoder step: embedding + RMSNorm, residual add +
// RMSNorm, q/k/v bias + RoPE + paged KV append, and Gumbel-max sampling with
// a Philox4x64-10 counter-based generator.  They move little data, so they
// are written for latency: every load of a thread is issued before the first
// use, and small batches are spread over several blocks per row.
#include "device_common.hpp"
#include "kernels.hpp"

namespace rollpack {

LaunchEvents& launch_events() {
  thread_local LaunchEvents ev;
  return ev;
}

namespace {

// Rows are processed by one block of up to 1024 threads, each owning two
// 4-element chunks, so every load of a row is in flight at once.
constexpr int kRowChunks = 2;

template <typename T> struct Vec4;
template <> struct Vec4<float> {
  static __device__ __forceinline__ float4 load(const float* p, size_t i) { return *reinterpret_cast<const float4*>(p + i); }
  static __device__ __forceinline__ void store(float* p, size_t i, float4 v) { *reinterpret_cast<float4*>(p + i) = v; }
};
template <> struct Vec4<bf16_t> {
  static __device__ __forceinline__ float4 load(const bf16_t* p, size_t i) {
    const uint2 u = *reinterpret_cast<const uint2*>(p + i);
    return make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16),
                       __uint_as_float(u.y & 0xffff0000u));
  }
  static __device__ __forceinline__ void store(bf16_t* p, size_t i, float4 v) {
    uint2 u;
    u.x = static_cast<uint32_t>(f32_to_bf16(v.x)) | (static_cast<uint32_t>(f32_to_bf16(v.y)) << 16);
    u.y = static_cast<uint32_t>(f32_to_bf16(v.z)) | (static_cast<uint32_t>(f32_to_bf16(v.w)) << 16);
    *reinterpret_cast<uint2*>(p + i) = u;
  }
};

__device__ __forceinline__ float block_sum(float v, float* red) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  float t = 0.f;
  for (int i = 0; i < nw; ++i) t += red[i];
  return t;
}

// The norm gains of this thread's chunks, loaded with the row so that the reduction does not delay them.
template <typename T>
__device__ __forceinline__ void load_gains(const T* g, int H, float4 (&gv)[kRowChunks]) {
#pragma unroll
  for (int v = 0; v < kRowChunks; ++v) {
    const int c = threadIdx.x + v * blockDim.x;
    if (c < H / 4) gv[v] = Vec4<T>::load(g, 4 * c);
  }
}

// x holds the row (kRowChunks float4 per thread); writes h = x * rsqrt(mean(x^2)+eps) * g.
template <typename T>
__device__ __forceinline__ void norm_store(const float4 (&xv)[kRowChunks], const float4 (&gv)[kRowChunks], int H, float eps,
                                           T* h, float* red) {
  const int nc = H / 4;
  float ss = 0.f;
#pragma unroll
  for (int v = 0; v < kRowChunks; ++v) {
    const int c = threadIdx.x + v * blockDim.x;
    if (c < nc) ss += xv[v].x * xv[v].x + xv[v].y * xv[v].y + xv[v].z * xv[v].z + xv[v].w * xv[v].w;
  }
  ss = block_sum(ss, red);
  const float inv = 1.0f / sqrtf(ss / H + eps);
#pragma unroll
  for (int v = 0; v < kRowChunks; ++v) {
    const int c = threadIdx.x + v * blockDim.x;
    if (c < nc) {
      Vec4<T>::store(h, 4 * static_cast<size_t>(c),
                     make_float4(xv[v].x * inv * gv[v].x, xv[v].y * inv * gv[v].y, xv[v].z * inv * gv[v].z,
                                 xv[v].w * inv * gv[v].w));
    }
  }
}

template <typename T>
__global__ __launch_bounds__(1024) void k_embed_norm(EmbedArgs a) {
  __shared__ float red[16];
  const int i = blockIdx.x;
  float4 gv[kRowChunks];
  load_gains(static_cast<const T*>(a.norm_g), a.H, gv);
  int tok = a.in_tok[i];
  if (tok < 0) tok = a.tokens_cur[a.row_slot[i]];
  const T* e = static_cast<const T*>(a.embed) + static_cast<size_t>(tok) * a.H;
  float* x = a.x + static_cast<size_t>(i) * a.H;
  const int nc = a.H / 4;
  float4 xv[kRowChunks];
#pragma unroll
  for (int v = 0; v < kRowChunks; ++v) {
    const int c = threadIdx.x + v * blockDim.x;
    if (c < nc) {
      xv[v] = Vec4<T>::load(e, 4 * c);
      *reinterpret_cast<float4*>(x + 4 * c) = xv[v];
    }
  }
  norm_store<T>(xv, gv, a.H, a.eps, static_cast<T*>(a.h) + static_cast<size_t>(i) * a.H, red);
}

// THREADS: 1024, whose registers hold the row, its gains and up to 13 partials of it; or 512, for rows of at
// most 4,096 elements, which hold 16.  (With 1,024 threads 14-16 partials and the gains spilled: 7.2 us at
// 65 rows of H = 896 against 4.5.)
template <typename T, int S, int THREADS>
__global__ __launch_bounds__(THREADS) void k_add_rmsnorm(AddNormArgs a) {
  __shared__ float red[16];
  const int i = blockIdx.x;
  float* x = a.x + static_cast<size_t>(i) * a.H;
  const int nc = a.H / 4;
  const size_t plane = static_cast<size_t>(a.M) * a.H;
  float4 xv[kRowChunks];
  constexpr bool kEarlyGains = S <= 13 || THREADS <= 512;
  float4 pv[S > 0 ? S : 1][kRowChunks], gv[kRowChunks];
  if (kEarlyGains) load_gains(static_cast<const T*>(a.norm_g), a.H, gv);
#pragma unroll
  for (int v = 0; v < kRowChunks; ++v) {
    const int c = threadIdx.x + v * blockDim.x;
    if (c < nc) {
      xv[v] = *reinterpret_cast<const float4*>(x + 4 * c);
#pragma unroll
      for (int s = 0; s < S; ++s)
        pv[s][v] = *reinterpret_cast<const float4*>(a.part + s * plane + static_cast<size_t>(i) * a.H + 4 * c);
    }
  }
  if (S > 0) {
#pragma unroll
    for (int v = 0; v < kRowChunks; ++v) {
      const int c = threadIdx.x + v * blockDim.x;
      if (c < nc) {
#pragma unroll
        for (int s = 0; s < S; ++s) {
          xv[v].x += pv[s][v].x; xv[v].y += pv[s][v].y; xv[v].z += pv[s][v].z; xv[v].w += pv[s][v].w;
        }
        *reinterpret_cast<float4*>(x + 4 * c) = xv[v];
      }
    }
  }
  if (!kEarlyGains) load_gains(static_cast<const T*>(a.norm_g), a.H, gv);
  norm_store<T>(xv, gv, a.H, a.eps, static_cast<T*>(a.h) + static_cast<size_t>(i) * a.H, red);
}

// fp32 model: one thread per rotated (q or k) pair or per v element; blockIdx.y strides
// the row's items so small batches still fill the GPU.
__global__ __launch_bounds__(256) void k_rope_append(RopeArgs a) {
  const int i = blockIdx.x;
  const int hd = a.hd, half = hd / 2;
  const int nq_el = a.n_q * hd, nk_el = a.n_kv * hd;
  const int nqkv = nq_el + 2 * nk_el;
  const int n_pairs = (a.n_q + a.n_kv) * half;
  const int t = blockIdx.y * blockDim.x + threadIdx.x;
  if (t >= n_pairs + nk_el) return;
  const float* __restrict__ prow = a.part + static_cast<size_t>(i) * nqkv;
  const int pos = a.pos[i];
  const int slot = a.slot[i];
  const int page = a.page_table[static_cast<size_t>(slot) * a.pt_stride + pos / kPageTokens];
  const int off = pos % kPageTokens;
  if (t < n_pairs) {
    const int head = t / half, d = t % half;
    const int n1 = head * hd + d, n2 = n1 + half;
    const bool isq = head < a.n_q;
    const float* b = static_cast<const float*>(isq ? a.bq : a.bk);
    const int bi = isq ? n1 : n1 - nq_el;
    const float u1 = prow[n1] + b[bi], u2 = prow[n2] + b[bi + half];
    const float c = a.rope_cos[static_cast<size_t>(pos) * half + d];
    const float sn = a.rope_sin[static_cast<size_t>(pos) * half + d];
    float* dst = isq ? static_cast<float*>(a.q_out) + static_cast<size_t>(i) * nq_el + n1
                     : static_cast<float*>(a.k_pool) +
                           ((static_cast<size_t>(page) * a.n_kv + head - a.n_q) * kPageTokens + off) * hd + d;
    dst[0] = u1 * c - u2 * sn;
    dst[half] = u2 * c + u1 * sn;
  } else {
    const int e = t - n_pairs;
    const int kh = e / hd, d = e % hd;
    // V page: two 32-token halves, each [hd][32 tokens]
    const size_t idx = (static_cast<size_t>(page) * a.n_kv + kh) * hd * kPageTokens + (off >> 5) * hd * 32 + d * 32 + (off & 31);
    static_cast<float*>(a.v_pool)[idx] = prow[nq_el + nk_el + e] + static_cast<const float*>(a.bv)[e];
  }
}

// The bf16 prefill's bias, RoPE and append, 16 bytes of partials at a time.  The first blocks take the
// q and k pairs, four consecutive dimension pairs per thread.  The rest take 64 tokens x 64 value
// dimensions each and turn them through LDS: a V page holds a dimension's 32 tokens side by side, so
// lanes store along tokens (64-byte runs) instead of 2 bytes per cache line.  The S partials are all loaded
// before the first is added (one after the other, seven of them took 7.5 us at 65 tokens against 3.8).
// 11,500 tokens of the 7B shape: 66 us (4.6 TB/s) against 140 for one pair or value per thread; 9,216 tokens of
// the 0.5B 14.6 against 24.8 us.
constexpr int kRopeTok = 64, kRopeDim = 64;

template <int S>
__global__ __launch_bounds__(256) void k_rope_prefill(RopeArgs a, int qk_blocks_per_row) {
  __shared__ bf16_t sv[kRopeDim][kRopeTok + 2];
  const int hd = a.hd, half = hd / 2;
  const int nq_el = a.n_q * hd, nk_el = a.n_kv * hd, nqkv = nq_el + 2 * nk_el;
  const size_t plane = static_cast<size_t>(a.M) * nqkv;
  auto sum4 = [&](const float* p) {
    float4 w[S];
#pragma unroll
    for (int s = 0; s < S; ++s) w[s] = *reinterpret_cast<const float4*>(p + s * plane);
#pragma unroll
    for (int s = 1; s < S; ++s) {
      w[0].x += w[s].x; w[0].y += w[s].y; w[0].z += w[s].z; w[0].w += w[s].w;
    }
    return w[0];
  };
  const int n_qk = a.M * qk_blocks_per_row;
  if (static_cast<int>(blockIdx.x) < n_qk) {
    const int i = blockIdx.x / qk_blocks_per_row;
    const int t = (blockIdx.x - i * qk_blocks_per_row) * 256 + threadIdx.x;
    const int per_head = half / 4;
    if (t >= (a.n_q + a.n_kv) * per_head) return;
    const int head = t / per_head, d = (t - head * per_head) * 4, n1 = head * hd + d;
    const bool isq = head < a.n_q;
    const int pos = a.pos[i];
    const float* p = a.part + static_cast<size_t>(i) * nqkv + n1;
    const bf16_t* b = static_cast<const bf16_t*>(isq ? a.bq : a.bk) + (isq ? n1 : n1 - nq_el);
    float4 u1 = sum4(p), u2 = sum4(p + half);
    float b1[4], b2[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      b1[e] = bf16_to_f32(b[e]);
      b2[e] = bf16_to_f32(b[half + e]);
    }
    const float4 c = *reinterpret_cast<const float4*>(a.rope_cos + static_cast<size_t>(pos) * half + d);
    const float4 sn = *reinterpret_cast<const float4*>(a.rope_sin + static_cast<size_t>(pos) * half + d);
    u1.x += b1[0]; u1.y += b1[1]; u1.z += b1[2]; u1.w += b1[3];
    u2.x += b2[0]; u2.y += b2[1]; u2.z += b2[2]; u2.w += b2[3];
    const float4 r1 = make_float4(u1.x * c.x - u2.x * sn.x, u1.y * c.y - u2.y * sn.y, u1.z * c.z - u2.z * sn.z, u1.w * c.w - u2.w * sn.w);
    const float4 r2 = make_float4(u2.x * c.x + u1.x * sn.x, u2.y * c.y + u1.y * sn.y, u2.z * c.z + u1.z * sn.z, u2.w * c.w + u1.w * sn.w);
    if (isq) {
      bf16_t* q = static_cast<bf16_t*>(a.q_out) + static_cast<size_t>(i) * nq_el;
      Vec4<bf16_t>::store(q, n1, r1);
      Vec4<bf16_t>::store(q, n1 + half, r2);
    } else {
      const int page = a.page_table[static_cast<size_t>(a.slot[i]) * a.pt_stride + pos / kPageTokens], off = pos % kPageTokens;
      bf16_t* k = static_cast<bf16_t*>(a.k_pool) + (static_cast<size_t>(page) * a.n_kv + head - a.n_q) * kPageTokens * hd;
      Vec4<bf16_t>::store(k, k_page_offset(off, d, hd), r1);  // four dimensions of an 8-dimension run
      Vec4<bf16_t>::store(k, k_page_offset(off, d + half, hd), r2);
    }
    return;
  }
  const int vb = blockIdx.x - n_qk, d_blocks = nk_el / kRopeDim;
  const int i0 = vb / d_blocks * kRopeTok, d0 = vb % d_blocks * kRopeDim;  // within one KV head: hd is a multiple of 64
  const int dd = (threadIdx.x & 15) * 4;
#pragma unroll
  for (int j = 0; j < kRopeTok / 16; ++j) {
    const int tok = (threadIdx.x >> 4) + 16 * j, i = i0 + tok;
    if (i >= a.M) break;
    const float4 u = sum4(a.part + static_cast<size_t>(i) * nqkv + nq_el + nk_el + d0 + dd);
    const bf16_t* b = static_cast<const bf16_t*>(a.bv) + d0 + dd;
    sv[dd + 0][tok] = f32_to_bf16(u.x + bf16_to_f32(b[0]));
    sv[dd + 1][tok] = f32_to_bf16(u.y + bf16_to_f32(b[1]));
    sv[dd + 2][tok] = f32_to_bf16(u.z + bf16_to_f32(b[2]));
    sv[dd + 3][tok] = f32_to_bf16(u.w + bf16_to_f32(b[3]));
  }
  __syncthreads();
  const int tok = threadIdx.x & 63, i = i0 + tok, w = threadIdx.x >> 6;
  if (i >= a.M) return;
  const int pos = a.pos[i], page = a.page_table[static_cast<size_t>(a.slot[i]) * a.pt_stride + pos / kPageTokens], off = pos % kPageTokens;
  // V page: two 32-token halves, each [hd][32 tokens]
  bf16_t* v = static_cast<bf16_t*>(a.v_pool) + (static_cast<size_t>(page) * a.n_kv + d0 / hd) * hd * kPageTokens + (off >> 5) * hd * 32 + (off & 31);
#pragma unroll
  for (int k = 0; k < kRopeDim / 4; ++k) v[(d0 % hd + w * (kRopeDim / 4) + k) * 32] = sv[w * (kRopeDim / 4) + k][tok];
}

// ---- sampling -------------------------------------------------------------

constexpr uint64_t kPhiloxM0 = 0xD2E7470EE14C6C93ull;
constexpr uint64_t kPhiloxM1 = 0xCA5A826395121157ull;
constexpr uint64_t kPhiloxW0 = 0x9E3779B97F4A7C15ull;
constexpr uint64_t kPhiloxW1 = 0xBB67AE8584CAA73Bull;

// Philox4x64, 10 rounds (Salmon et al., SC'11).
__device__ __forceinline__ void philox4x64_10(uint64_t& x0, uint64_t& x1, uint64_t& x2, uint64_t& x3,
                                              uint64_t k0, uint64_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const unsigned __int128 p0 = static_cast<unsigned __int128>(kPhiloxM0) * x0;  // four 32 x 32 products each
    const unsigned __int128 p1 = static_cast<unsigned __int128>(kPhiloxM1) * x2;
    const uint64_t hi0 = static_cast<uint64_t>(p0 >> 64), lo0 = static_cast<uint64_t>(p0);
    const uint64_t hi1 = static_cast<uint64_t>(p1 >> 64), lo1 = static_cast<uint64_t>(p1);
    const uint64_t n0 = hi1 ^ x1 ^ k0, n2 = hi0 ^ x3 ^ k1;
    x0 = n0; x1 = lo1; x2 = n2; x3 = lo0;
    k0 += kPhiloxW0;
    k1 += kPhiloxW1;
  }
}

// Top 23 bits of a 32-bit word -> (m + 0.5) * 2^-23, exact in fp32, in (0, 1).
__device__ __forceinline__ float word_to_gumbel(uint32_t w) {
  const float u = (static_cast<float>(w >> 9) + 0.5f) * 1.1920928955078125e-07f;
  return -logf(-logf(u));
}

__device__ __forceinline__ void take_best(float& bv, int& bi, float v, int i) {
  const bool take = (v > bv) | ((v == bv) & (i < bi));  // no branch; a NaN is never taken
  bv = take ? v : bv;
  bi = take ? i : bi;
}

// Running log-sum-exp state (max m, sum of exp(x - m)); combining two states
// rescales the smaller-max sum.
__device__ __forceinline__ void lse_merge(float& m, float& s, float m2, float s2) {
  if (m2 == -INFINITY) return;
  if (m2 > m) { s = s * expf(m - m2) + s2; m = m2; } else { s += s2 * expf(m2 - m); }
}

// Pass 1: block (row, chunk) scores kSampleChunk vocabulary entries and
// writes its best (score, index) and the log-sum-exp state of logits / T
// over the chunk.  Pass 2: one wave per row reduces the chunk winners (ties
// -> lowest index), records the token and its log-probability
// logits[token] / T - logsumexp(logits / T) (T = 1 for greedy rows).
constexpr int kSampleChunk = 2048;

__global__ __launch_bounds__(256) void k_sample_partial(SampleArgs a) {
  __shared__ float sv[4], sm[4], ss[4];
  __shared__ int si[4];
  const int row = blockIdx.x;
  const float* l = a.logits + static_cast<size_t>(row) * a.V;
  const int gi = blockIdx.y * (kSampleChunk / 8) + threadIdx.x;  // 8 entries per thread, one Philox block
  const int vb = gi * 8;
  float lv[8];
  const bool whole = vb + 8 <= a.V && a.V % 4 == 0;  // then the entries are two 16-byte loads
  if (whole) {
    const float4 p = *reinterpret_cast<const float4*>(l + vb), q = *reinterpret_cast<const float4*>(l + vb + 4);
    lv[0] = p.x; lv[1] = p.y; lv[2] = p.z; lv[3] = p.w;
    lv[4] = q.x; lv[5] = q.y; lv[6] = q.z; lv[7] = q.w;
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) lv[e] = vb + e < a.V ? l[vb + e] : -INFINITY;
  }
  const int slot = a.row_slot[row];
  const float temp = a.slot_temp[slot];
  float best = -INFINITY;
  int besti = 0x7fffffff;
  float lm = -INFINITY, ls = 0.f;  // log-sum-exp state of logits / T
  if (vb < a.V) {
    if (temp == 0.f) {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        take_best(best, besti, vb + e < a.V ? lv[e] : NAN, vb + e);
    } else {
      const float inv_t = 1.0f / temp;
      uint64_t x0 = static_cast<uint64_t>(a.row_pos[row]), x1 = static_cast<uint64_t>(gi), x2 = 0, x3 = 0;
      philox4x64_10(x0, x1, x2, x3, a.slot_seed[slot], a.slot_id[slot]);
      const uint64_t outs[4] = {x0, x1, x2, x3};
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t w = (e & 1) ? static_cast<uint32_t>(outs[e >> 1] >> 32) : static_cast<uint32_t>(outs[e >> 1]);
        lv[e] *= inv_t;
        take_best(best, besti, vb + e < a.V ? lv[e] + word_to_gumbel(w) : NAN, vb + e);
      }
    }
    // the thread's log-sum-exp around its own maximum (entries past V are -inf and add nothing)
#pragma unroll
    for (int e = 0; e < 8; ++e) lm = fmaxf(lm, lv[e]);
    if (lm > -INFINITY) {
#pragma unroll
      for (int e = 0; e < 8; ++e) ls += expf(lv[e] - lm);
    }
  }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
    const float ov = __shfl_xor(best, m, 64);
    const int oi = __shfl_xor(besti, m, 64);
    take_best(best, besti, ov, oi);
    const float om = __shfl_xor(lm, m, 64);
    const float os = __shfl_xor(ls, m, 64);
    lse_merge(lm, ls, om, os);
  }
  if ((threadIdx.x & 63) == 0) {
    sv[threadIdx.x >> 6] = best; si[threadIdx.x >> 6] = besti;
    sm[threadIdx.x >> 6] = lm; ss[threadIdx.x >> 6] = ls;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) {
      take_best(best, besti, sv[w], si[w]);
      lse_merge(lm, ls, sm[w], ss[w]);
    }
    const size_t c = static_cast<size_t>(row) * gridDim.y + blockIdx.y;
    a.cand_val[c] = best;
    a.cand_idx[c] = besti;
    a.cand_m[c] = lm;
    a.cand_s[c] = ls;
  }
}

__global__ __launch_bounds__(64) void k_sample_final(SampleArgs a, int chunks) {
  const int row = blockIdx.x;
  const int slot = a.row_slot[row], hist = a.row_hist[row];
  const float temp = a.slot_temp[slot];
  float best = -INFINITY;
  int besti = 0x7fffffff;
  float lm = -INFINITY, ls = 0.f;
  for (int c = threadIdx.x; c < chunks; c += 64) {
    const size_t i = static_cast<size_t>(row) * chunks + c;
    take_best(best, besti, a.cand_val[i], a.cand_idx[i]);
    lse_merge(lm, ls, a.cand_m[i], a.cand_s[i]);
  }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
    const float ov = __shfl_xor(best, m, 64);
    const int oi = __shfl_xor(besti, m, 64);
    take_best(best, besti, ov, oi);
    const float om = __shfl_xor(lm, m, 64);
    const float os = __shfl_xor(ls, m, 64);
    lse_merge(lm, ls, om, os);
  }
  if (threadIdx.x == 0) {
    if (besti == 0x7fffffff) besti = 0;  // all-NaN row: deterministic fallback
    const float inv_t = temp == 0.f ? 1.f : 1.0f / temp;
    const float s_tok = a.logits[static_cast<size_t>(row) * a.V + besti] * inv_t;
    const size_t h = static_cast<size_t>(slot) * a.hist_stride + hist;
    a.tokens_cur[slot] = besti;
    a.hist[h] = besti;
    a.logp_hist[h] = s_tok - (lm + logf(ls));
  }
}

__global__ __launch_bounds__(256) void k_gather_rows(const uint8_t* src, const int32_t* rows, int row_bytes,
                                                      uint8_t* out) {
  const int i = blockIdx.x;
  const uint8_t* s = src + static_cast<size_t>(rows[i]) * row_bytes;
  uint8_t* d = out + static_cast<size_t>(i) * row_bytes;
  if ((row_bytes & 15) == 0) {
    for (int b = threadIdx.x * 16; b < row_bytes; b += 256 * 16)
      *reinterpret_cast<uint4*>(d + b) = *reinterpret_cast<const uint4*>(s + b);
  } else {
    for (int b = threadIdx.x; b < row_bytes; b += 256) d[b] = s[b];
  }
}

}  // namespace

namespace {
int row_threads(int H) {
  int t = (H / 4 + kRowChunks - 1) / kRowChunks;
  t = (t + 63) / 64 * 64;
  return t < 64 ? 64 : t;
}

template <typename T, int S>
void launch_add_norm_s(const AddNormArgs& a, int threads, hipStream_t s) {
  if (S > 13 && threads <= 512) launch_kernel((k_add_rmsnorm<T, S, (S > 13 ? 512 : 1024)>), dim3(a.M), dim3(threads), 0, s, a);
  else launch_kernel((k_add_rmsnorm<T, S, 1024>), dim3(a.M), dim3(threads), 0, s, a);
}

template <typename T>
hipError_t launch_add_norm_t(const AddNormArgs& a, hipStream_t s) {
  const int th = row_threads(a.H);
  const int S = a.part ? a.splits : 0;
  switch (S) {
    case 0: launch_add_norm_s<T, 0>(a, th, s); break;
    case 1: launch_add_norm_s<T, 1>(a, th, s); break;
    case 2: launch_add_norm_s<T, 2>(a, th, s); break;
    case 3: launch_add_norm_s<T, 3>(a, th, s); break;
    case 4: launch_add_norm_s<T, 4>(a, th, s); break;
    case 5: launch_add_norm_s<T, 5>(a, th, s); break;
    case 6: launch_add_norm_s<T, 6>(a, th, s); break;
    case 7: launch_add_norm_s<T, 7>(a, th, s); break;
    case 8: launch_add_norm_s<T, 8>(a, th, s); break;
    case 9: launch_add_norm_s<T, 9>(a, th, s); break;
    case 10: launch_add_norm_s<T, 10>(a, th, s); break;
    case 11: launch_add_norm_s<T, 11>(a, th, s); break;
    case 12: launch_add_norm_s<T, 12>(a, th, s); break;
    case 13: launch_add_norm_s<T, 13>(a, th, s); break;
    case 14: launch_add_norm_s<T, 14>(a, th, s); break;
    case 15: launch_add_norm_s<T, 15>(a, th, s); break;
    case 16: launch_add_norm_s<T, 16>(a, th, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// fp32 model: one partial, no K split.
hipError_t launch_rope_f32(const RopeArgs& a, hipStream_t s) {
  if (a.splits != 1) return hipErrorInvalidValue;
  const int items = (a.n_q + a.n_kv) * (a.hd / 2) + a.n_kv * a.hd;
  launch_kernel(k_rope_append, dim3(a.M, (items + 255) / 256), dim3(256), 0, s, a);
  return hipGetLastError();
}

// bf16 prefill.  Partials, tables and pools are 256-byte aligned parts of the engine's workspaces.
hipError_t launch_rope_bf16(const RopeArgs& a, hipStream_t s) {
  if (a.hd % kRopeDim) return hipErrorInvalidValue;
  const int per_row = ((a.n_q + a.n_kv) * (a.hd / 8) + 255) / 256;
  const int v_blocks = (a.M + kRopeTok - 1) / kRopeTok * (a.n_kv * a.hd / kRopeDim);
  const dim3 grid(a.M * per_row + v_blocks);
  switch (a.splits) {
#define RP_ROPE(S) case S: launch_kernel(k_rope_prefill<S>, grid, dim3(256), 0, s, a, per_row); break;
    RP_ROPE(1) RP_ROPE(2) RP_ROPE(3) RP_ROPE(4) RP_ROPE(5) RP_ROPE(6) RP_ROPE(7) RP_ROPE(8)
    RP_ROPE(9) RP_ROPE(10) RP_ROPE(11) RP_ROPE(12) RP_ROPE(13) RP_ROPE(14) RP_ROPE(15) RP_ROPE(16)
#undef RP_ROPE
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
}  // namespace

hipError_t launch_embed_norm(int bf16, const EmbedArgs& a, hipStream_t s) {
  if (a.M <= 0) return hipSuccess;
  if (a.H % 4 || a.H > 4 * kRowChunks * 1024) return hipErrorInvalidValue;
  const int th = row_threads(a.H);
  if (bf16) launch_kernel(k_embed_norm<bf16_t>, dim3(a.M), dim3(th), 0, s, a);
  else launch_kernel(k_embed_norm<float>, dim3(a.M), dim3(th), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_add_rmsnorm(int bf16, const AddNormArgs& a, hipStream_t s) {
  if (a.M <= 0) return hipSuccess;
  if (a.H % 4 || a.H > 4 * kRowChunks * 1024) return hipErrorInvalidValue;
  return bf16 ? launch_add_norm_t<bf16_t>(a, s) : launch_add_norm_t<float>(a, s);
}

hipError_t launch_rope_append(int bf16, const RopeArgs& a, hipStream_t s) {
  if (a.M <= 0) return hipSuccess;
  return bf16 ? launch_rope_bf16(a, s) : launch_rope_f32(a, s);
}

int sample_chunks(int V) { return (V + kSampleChunk - 1) / kSampleChunk; }

hipError_t launch_sample(const SampleArgs& a, hipStream_t s) {
  if (a.B <= 0) return hipSuccess;
  const int chunks = sample_chunks(a.V);
  launch_kernel(k_sample_partial, dim3(a.B, chunks), dim3(256), 0, s, a);
  launch_kernel(k_sample_final, dim3(a.B), dim3(64), 0, s, a, chunks);
  return hipGetLastError();
}

// Streaming read of a buffer: each wave walks its own contiguous share, 8 one-KB loads (16 bytes
// per lane) in flight per step, 8 waves per CU: the practical HBM read ceiling that measurement
// reports next to the nominal peak.  The values feed an empty asm so that every load is issued.
constexpr int kStreamWaves = 2048;

// Non-temporal loads: the stream is read once, and marking it so measured
// 6.9-7.0 TB/s against 6.1 TB/s with plain loads over 2 GiB.
typedef unsigned u32x4_nt __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256) void k_stream_read(const uint4* p, size_t n16) {
  const u32x4_nt* pn = reinterpret_cast<const u32x4_nt*>(p);
  const int lane = threadIdx.x & 63;
  const size_t wave = static_cast<size_t>(blockIdx.x) * (blockDim.x / 64) + (threadIdx.x >> 6);
  const size_t share = (n16 / 64 / kStreamWaves) * 64;  // whole 1 KB runs per wave
  const size_t begin = wave * share, end = begin + share;
  uint32_t acc = 0;
  size_t i = begin + lane;
  for (; i + 7 * 64 < end; i += 8 * 64) {
    u32x4_nt v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = __builtin_nontemporal_load(pn + i + j * 64);
#pragma unroll
    for (int j = 0; j < 8; ++j) acc ^= v[j].x ^ v[j].y ^ v[j].z ^ v[j].w;
  }
  for (; i < end; i += 64) acc ^= p[i].x;
  for (size_t t = kStreamWaves * share + wave * 64 + lane; t < n16; t += static_cast<size_t>(kStreamWaves) * 64)
    acc ^= p[t].x;  // the remainder past the waves' equal shares
  asm volatile("" : : "v"(acc));
}

hipError_t launch_stream_read(const void* buf, size_t bytes, hipStream_t s) {
  if (bytes < 16) return hipErrorInvalidValue;
  launch_kernel(k_stream_read, dim3(kStreamWaves / 4), dim3(256), 0, s, static_cast<const uint4*>(buf), bytes / 16);
  return hipGetLastError();
}

hipError_t launch_gather_rows(const void* src, const int32_t* rows, int n, int H, int esize, void* out,
                              hipStream_t s) {
  if (n <= 0) return hipSuccess;
  launch_kernel(k_gather_rows, dim3(n), dim3(256), 0, s, static_cast<const uint8_t*>(src), rows,
                     H * esize, static_cast<uint8_t*>(out));
  return hipGetLastError();
}

}  // namespace rollpack
