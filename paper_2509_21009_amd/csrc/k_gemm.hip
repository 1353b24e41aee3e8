// Dense projections C[m, n] = sum_k A[m, k] * W[n, k] of the decoder
// (q/k/v, o, gate/up, down, LM head).  W is [out, in] row-major, A is the
// [M, K] activation matrix; both are K-contiguous.
//
// bf16 kernels use gfx950 MFMA (v_mfma_f32_16x16x32_bf16) with fp32
// accumulation and W as the 16-row "A" operand, activations as the
// 16-column "B" operand, so one MFMA yields a [16 n, 16 m] tile of C^T.
//
//  * k_gemm_ring (up to 64 rows): a block's 4 waves take interleaved 64-wide K units of
//    the same weight rows; weights and activations are copied into per-wave LDS
//    rings, and the waves reduce through LDS; blockIdx.y splits K further and
//    writes fp32 partials that the consumer kernel sums.
//  * k_gemm_deep (M <= 16, mid-sized weight matrices and large vocabularies): the same split
//    of the work with weights in a ring of register stages; a stage is a
//    64-wide K unit in which each lane reads 32 contiguous bytes of a
//    row, so one wave's two back-to-back loads cover the row's whole
//    128-byte line.  Activations (L2-resident) are loaded one stage ahead
//    into a single buffer.
//    With the packed copy of the weights (launch_pack_weights)
//    each load instruction of either reads one contiguous 1 KB run instead, non-temporal
//    (the weights are read once per step), the same operands in every lane.
//  * k_gemm_tiled (M > 64: prefill and large decode batches): 128- or
//    256-row x 128- or 256-row block tiles of 32x32x16 MFMAs, half tiles
//    copied from global memory straight into a swizzled LDS ring.
//  * k_gemm_f32: fp32 MFMA for the fp32 model (no reduced precision).
//
// The SiLU epilogue pairs gate row i with up row i in one thread and writes
// silu(gate) * up once, rounded to the storage type.
#include "device_common.hpp"
#include "gemm_plan.hpp"
#include "kernels.hpp"
#include "lds_dma.hpp"

namespace rollpack {

namespace {

template <typename T>
__device__ __forceinline__ const T* seg_row(const WSeg& W, int n, int K) {
  int base = 0;
  for (int s = 0; s < 3; ++s) {
    if (s == W.n_seg - 1 || n < base + W.rows[s])
      return static_cast<const T*>(W.ptr[s]) + static_cast<size_t>(n - base) * K;
    base += W.rows[s];
  }
  return static_cast<const T*>(W.ptr[0]);
}

__device__ __forceinline__ float silu(float z) { return z / (1.0f + expf(-z)); }
// The same for results that are rounded to bf16, in 16 instructions instead of about 35: exp(-z) as
// 2^t (1 + dl) with t the rounded product -z log2(e) and dl = d ln 2 from what it is off by (bounded, so
// that infinities pass), and the quotient z / (1 + 2^t) corrected once by its remainder, which takes dl and what
// the sum 1 + 2^t lost in: at most 1.8e-7 off over [-80, 100], 3.4e-8 in the root mean
// square, and of 16.8M values 134 round to another bf16 than the exact ones (the full sequence 1.8e-7, 4.0e-8, 143).
// v_rcp_f32 flushes results below 2^-126, z below -87.3, whose quotients down to -2.5e-37 are normal bf16
// values: the reciprocal is taken of a quarter of the sum and scaled back, which changes no other value
// (over [-88.72, -87.3] 1.2e-7 off as the full sequence; prefill of 9,216 tokens of the 0.5B model 9.08 ms against
// 9.07 without).  Infinities leave a NaN remainder, which the bound turns into a finite one: an infinite quotient
// or a zero one stays.
__device__ __forceinline__ float silu_fast(float z) {
  constexpr float kL2e = -1.44269504088896341f, kL2eLo = -1.925963033500e-8f, kLn2 = 0.693147180559945309f;
  const float t = z * kL2e;
  const float d = __builtin_amdgcn_fmed3f(__builtin_fmaf(z, kL2eLo, __builtin_fmaf(z, kL2e, -t)), -1e-4f, 1e-4f);
  const float p = __builtin_amdgcn_exp2f(t), r = __builtin_amdgcn_rcpf(__builtin_fmaf(p, 0.25f, 0.25f)) * 0.25f, q = z * r;
  const float rem = __builtin_fmaf(-(q * p), d * kLn2, __builtin_fmaf(-q, p, z - q));
  return __builtin_fmaf(__builtin_amdgcn_fmed3f(rem, -3e38f, 3e38f), r, q);
}
// fp32 -> bf16 storage, round to nearest even (v_cvt_pk_bf16_f32).
__device__ __forceinline__ bf16_t bf16_of(float f) { return __builtin_bit_cast(bf16_t, static_cast<__bf16>(f)); }

// ---- decode-regime weight streaming, deep register pipeline ----------------
// Block: 4 waves on the same 16R weight rows (with the SiLU epilogue: R/2
// gate fragments and the R/2 up fragments of the same output indices).
// A stage is a 64-wide K unit: lane (g, r) loads bytes [32g, 32g + 32) of
// the unit's 128 bytes of row r as two 16-byte loads, and MFMA k-step j of
// the unit takes the j-th of them from both operands, so every product of
// the unit is formed exactly once.  Wave w takes units w, w + 4, ... of the
// block's K range, so the block reads whole 512-byte runs of each row.
// Weight fragments use one buffer resource each: rows past the end of the
// matrix (the ragged last block) read as zeros and are never stored.
// Weight loads of the deep kernel: row-major (plain) or packed (non-temporal:
// aux bit 1 is the nt cache policy).
template <bool PACKED>
__device__ __forceinline__ bf16x8_t load_w16(__amdgpu_buffer_rsrc_t r, int off) {
  return __builtin_bit_cast(bf16x8_t, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, PACKED ? 2 : 0));
}

template <int R, int D, bool SILU, bool PACKED>
__global__ __launch_bounds__(256) void k_gemm_deep(GemmArgs a, int units_per_split) {
  static_assert(!SILU || R % 2 == 0, "SiLU pairs gate and up fragments");
  __shared__ __attribute__((aligned(16))) f32x4_t red[3][R][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, r = lane & 15;
  const int K = a.K, KU = K / 64;
  const int u0 = blockIdx.y * units_per_split;
  const int u1 = min(u0 + units_per_split, KU);
  const int nblk = max(u1 - u0, 0);
  const int nk = nblk > wave ? (nblk - wave + 3) / 4 : 0;
  const uint32_t row_bytes = static_cast<uint32_t>(K) * 2u;

  const WSeg& W = PACKED ? a.Wp : a.W;
  __amdgpu_buffer_rsrc_t rw[R];
#pragma unroll
  for (int t = 0; t < R; ++t) {
    const bf16_t* base;
    int valid;
    if (SILU) {
      const int row0 = (blockIdx.x * (R / 2) + t % (R / 2)) * 16;
      valid = row0 < a.N ? min(16, a.N - row0) : 0;
      base = static_cast<const bf16_t*>(W.ptr[t / (R / 2)]) + static_cast<size_t>(valid ? row0 : 0) * K;
    } else {
      const int row0 = (blockIdx.x * R + t) * 16;
      int b = 0, sg = 0;
      while (sg < W.n_seg - 1 && row0 >= b + W.rows[sg]) b += W.rows[sg++];
      valid = row0 < a.N ? min(16, W.rows[sg] - (row0 - b)) : 0;
      base = static_cast<const bf16_t*>(W.ptr[sg]) + static_cast<size_t>(valid ? row0 - b : 0) * K;
    }
    // a packed tile is whole (16 rows) or absent; a row-major one may be ragged
    rw[t] = buffer_rsrc(base, static_cast<uint32_t>(PACKED ? (valid ? 16 : 0) : valid) * row_bytes);
  }
  // rows m >= M of the activations read as zeros
  const __amdgpu_buffer_rsrc_t ra =
      buffer_rsrc(a.A, static_cast<uint32_t>(a.M) * static_cast<uint32_t>(a.lda) * 2u);
  const int kb = (u0 + wave) * 128 + g * 32;
  // row-major: lane (g, r) reads 32 bytes of row r per unit (two 16-byte pieces), units 128 bytes
  // apart; packed: the unit's 2 KB run, the lane's 16 bytes in each 1 KB half
  const int woff = PACKED ? (u0 + wave) * 2048 + lane * 16 : r * static_cast<int>(row_bytes) + kb;
  constexpr int kWStep = PACKED ? 4 * 2048 : 4 * 128, kWHalf = PACKED ? 1024 : 16;
  const int aoff = r * static_cast<int>(a.lda) * 2 + kb;

  f32x4_t acc[R];
#pragma unroll
  for (int t = 0; t < R; ++t) acc[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  // Weights: a ring of D stages.  Activations: one buffer, loaded one stage
  // ahead, after the weights of the current stage and before those of later
  // stages; vector loads complete in issue order, so waiting for the
  // activations of stage s never waits for weights of later stages.
  bf16x8_t wv[D][R][2], av[2];
  auto load_w = [&](int s, int unit) {
    const int o = unit * kWStep;
#pragma unroll
    for (int t = 0; t < R; ++t) {
      wv[s][t][0] = load_w16<PACKED>(rw[t], woff + o);
      wv[s][t][1] = load_w16<PACKED>(rw[t], woff + o + kWHalf);
    }
  };
  auto load_a = [&](int unit) {
    const int o = unit * 512;
    av[0] = load_bf16x8(ra, aoff + o);
    av[1] = load_bf16x8(ra, aoff + o + 16);
  };
  auto compute = [&](int s) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int t = 0; t < R; ++t) acc[t] = mfma16x16x32(wv[s][t][j], av[j], acc[t]);
  };

  // The prologue loads unconditionally (stages past the wave's range are
  // in bounds and never used) and the scheduling barriers keep the issue
  // order, so every path into the main loop has the same loads in flight and
  // the compiler's wait counts there are exact.
  load_w(0, 0);
  __builtin_amdgcn_sched_barrier(0);
  load_a(0);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int s = 1; s < D; ++s) {
    load_w(s, s);
    __builtin_amdgcn_sched_barrier(0);
  }
  int i = 0;
  for (; i + 2 * D <= nk; i += D) {
#pragma unroll
    for (int s = 0; s < D; ++s) {
      compute(s);
      __builtin_amdgcn_sched_barrier(0);
      load_a(i + s + 1);
      __builtin_amdgcn_sched_barrier(0);
      load_w(s, i + s + D);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int j = 0; j < 2 * D; ++j) {
    if (i + j < nk) {
      compute(j % D);
      __builtin_amdgcn_sched_barrier(0);
      if (i + j + 1 < nk) load_a(i + j + 1);
      __builtin_amdgcn_sched_barrier(0);
      if (i + j + D < nk) load_w(j % D, i + j + D);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  if (wave > 0) {
#pragma unroll
    for (int t = 0; t < R; ++t) red[wave - 1][t][lane] = acc[t];
  }
  __syncthreads();
  if (wave > 0) return;
#pragma unroll
  for (int t = 0; t < R; ++t) acc[t] = acc[t] + red[0][t][lane] + red[1][t][lane] + red[2][t][lane];

  // lane (g, r) holds C^T[row base + t*16 + 4g + e][m = r]
  if (r >= a.M) return;
  if (SILU) {
#pragma unroll
    for (int t = 0; t < R / 2; ++t) {
      const int i0 = (blockIdx.x * (R / 2) + t) * 16 + g * 4;
      if (i0 >= a.N) continue;
      const f32x4_t gv = acc[t], uv = acc[t + R / 2];
      uint2 pk;
      pk.x = static_cast<uint32_t>(f32_to_bf16(silu(gv[0]) * uv[0])) |
             (static_cast<uint32_t>(f32_to_bf16(silu(gv[1]) * uv[1])) << 16);
      pk.y = static_cast<uint32_t>(f32_to_bf16(silu(gv[2]) * uv[2])) |
             (static_cast<uint32_t>(f32_to_bf16(silu(gv[3]) * uv[3])) << 16);
      *reinterpret_cast<uint2*>(static_cast<bf16_t*>(a.act_out) + static_cast<size_t>(r) * a.N + i0) = pk;
    }
  } else {
#pragma unroll
    for (int t = 0; t < R; ++t) {
      const int n = (blockIdx.x * R + t) * 16 + g * 4;
      if (n >= a.N) continue;
      *reinterpret_cast<f32x4_t*>(a.part + (static_cast<size_t>(blockIdx.y) * a.M + r) * a.N + n) = acc[t];
    }
  }
}

// ---- decode-regime weight streaming through private LDS rings ---------------
// k_gemm_deep's work split (4 waves on the same R weight fragments, K units
// interleaved over the waves, no barrier until the end).  From 17 activation
// rows on, a register ring starves: a stage's MFMAs and the wait for the
// next stage's activations run while one stage of weights is in flight (R = 10
// fragments x 4 activation tiles leave no registers for more), and gate/up of
// the 7B took 62 us at 64 rows against 46 at 16.  Here weights and activations are copied
// into LDS (buffer_load ... lds), 40 KB per wave: two units of activations and a
// ring of the next 12-18 weight fragments, each refilled as soon as it is in
// registers, so about 30 KB per wave stay in flight whatever the MFMAs do.  A wave
// waits for its own copies by count (they complete in order) and reads a
// fragment while the MFMAs of the one before run.  Copies past the wave's last
// unit are out of the resource's range: they move nothing and keep the counts.
// Gate/up of the 7B streams its packed weights at 5.7-6.0 TB/s from 1 to 64 rows
// (45.0-47.6 us).  The non-temporal mark on the packed copies is worth 10%
// (54 us without it at 64 rows).
template <int R, int MT, bool SILU, bool PACKED>
__global__ __launch_bounds__(256) void k_gemm_ring(GemmArgs a, int units_per_split) {
  static_assert(R % 2 == 0, "register buffers alternate by fragment; SiLU pairs gate and up fragments");
  constexpr int WAVE_LDS = 40960, A_UNIT = MT * 2048, SLOTS = (WAVE_LDS - 2 * A_UNIT) / 2048;
  static_assert(SLOTS >= R, "the counts below assume an activation unit among the copies of the last SLOTS fragments");
  static_assert(4 * R * MT * 1024 <= 4 * WAVE_LDS, "the final reduction reuses the rings");
  __shared__ __attribute__((aligned(1024))) uint8_t smem[4 * WAVE_LDS];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, r = lane & 15;
  const int K = a.K, KU = K / 64;
  const int u0 = blockIdx.y * units_per_split;
  const int u1 = min(u0 + units_per_split, KU);
  const int nblk = max(u1 - u0, 0);
  const int nk = nblk > wave ? (nblk - wave + 3) / 4 : 0;
  const uint32_t row_bytes = static_cast<uint32_t>(K) * 2u;

  const WSeg& W = PACKED ? a.Wp : a.W;
  u32x4_raw rw[R];
#pragma unroll
  for (int t = 0; t < R; ++t) {
    const bf16_t* base;
    int valid;
    if (SILU) {
      const int row0 = (blockIdx.x * (R / 2) + t % (R / 2)) * 16;
      valid = row0 < a.N ? min(16, a.N - row0) : 0;
      base = static_cast<const bf16_t*>(W.ptr[t / (R / 2)]) + static_cast<size_t>(valid ? row0 : 0) * K;
    } else {
      const int row0 = (blockIdx.x * R + t) * 16;
      int b = 0, sg = 0;
      while (sg < W.n_seg - 1 && row0 >= b + W.rows[sg]) b += W.rows[sg++];
      valid = row0 < a.N ? min(16, W.rows[sg] - (row0 - b)) : 0;
      base = static_cast<const bf16_t*>(W.ptr[sg]) + static_cast<size_t>(valid ? row0 - b : 0) * K;
    }
    // a packed tile is whole (16 rows) or absent; a row-major one may be ragged
    rw[t] = raw_rsrc(base, static_cast<uint32_t>(PACKED ? (valid ? 16 : 0) : valid) * row_bytes);
  }
  // rows m >= M of the activations read as zeros
  const u32x4_raw ra = raw_rsrc(a.A, static_cast<uint32_t>(a.M) * static_cast<uint32_t>(a.lda) * 2u);

  // A row-major copy instruction takes 8 rows of one 128-byte line; LDS chunk lane & 7 of a row holds
  // global chunk (lane & 7) ^ ((row >> 1) & 7), which keeps the fragment reads free of bank conflicts.
  // A packed one takes 1 KB of a tile's 2 KB unit run.
  const int c8 = lane >> 3, ch = lane & 7;
  typedef const __attribute__((address_space(3))) char lds_char;
  const uint32_t lds0 = static_cast<uint32_t>((uintptr_t)(lds_char*)(smem)) + static_cast<uint32_t>(wave * WAVE_LDS);
  constexpr int kOut = 0x40000000;  // past every resource
  int aoff[2], woff[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int row = h * 8 + c8, gc = ch ^ ((row >> 1) & 7);
    aoff[h] = row * static_cast<int>(a.lda) * 2 + (u0 + wave) * 128 + gc * 16;
    woff[h] = PACKED ? (u0 + wave) * 2048 + h * 1024 + lane * 16
                     : row * static_cast<int>(row_bytes) + (u0 + wave) * 128 + gc * 16;
  }
  const int lda16 = 16 * static_cast<int>(a.lda) * 2;
  auto copy_a = [&](int i) {  // unit i of the wave into activation buffer i & 1
    const int o = i < nk ? i * 512 : kOut;
    const uint32_t dst = __builtin_amdgcn_readfirstlane(lds0 + static_cast<uint32_t>((i & 1) * A_UNIT));
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int h = 0; h < 2; ++h) dma16(ra, dst + mt * 2048 + h * 1024, aoff[h] + mt * lda16 + o);
  };
  auto copy_w = [&](int t, int i, int slot) {  // fragment t of the wave's unit i into a ring slot
    const int o = i < nk ? i * (PACKED ? 4 * 2048 : 512) : kOut;
    const uint32_t dst = __builtin_amdgcn_readfirstlane(lds0 + static_cast<uint32_t>(2 * A_UNIT + slot * 2048));
    if (PACKED) {
      dma16_nt(rw[t], dst, woff[0] + o);
      dma16_nt(rw[t], dst + 1024, woff[1] + o);
    } else {
      dma16(rw[t], dst, woff[0] + o);
      dma16(rw[t], dst + 1024, woff[1] + o);
    }
  };
  const int rsw = (r >> 1) & 7;
  const int rd_row[2] = {r * 128 + ((2 * g) ^ rsw) * 16, r * 128 + ((2 * g + 1) ^ rsw) * 16};
  const uint8_t* base = smem + wave * WAVE_LDS;
  bf16x8_t av[MT][2], wv[2][2];
  auto read_a = [&](int i) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        av[mt][j] = *reinterpret_cast<const bf16x8_t*>(base + (i & 1) * A_UNIT + mt * 2048 + rd_row[j]);
  };
  auto read_w = [&](int buf, int slot) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
      wv[buf][j] = *reinterpret_cast<const bf16x8_t*>(base + 2 * A_UNIT + slot * 2048 + (PACKED ? j * 1024 + lane * 16 : rd_row[j]));
  };

  f32x4_t acc[R][MT];
#pragma unroll
  for (int t = 0; t < R; ++t)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[t][mt] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  constexpr int kLgkm0 = 0xc07f;  // s_waitcnt lgkmcnt(0)
  copy_a(0);
  copy_a(1);
#pragma unroll
  for (int f = 0; f < SLOTS; ++f) copy_w(f % R, f / R, f);
  wait_vmcnt<2 * (SLOTS - 1)>();  // fragment 0, and with it both activation units
  read_w(0, 0);
  __builtin_amdgcn_s_waitcnt(kLgkm0);
  copy_w(SLOTS % R, SLOTS / R, 0);
  int slot = 0;
  for (int i = 0; i < nk; ++i) {
    // activations of unit i: after them, those of unit i + 1 and two units of fragments were issued
    wait_vmcnt<4 * R + 2 * MT>();
    read_a(i);
    __builtin_amdgcn_s_waitcnt(kLgkm0);
    copy_a(i + 2);
#pragma unroll
    for (int t = 0; t < R; ++t) {
      // the next fragment: after it, SLOTS - 1 fragments and at least one activation unit were issued
      wait_vmcnt<2 * (SLOTS - 1) + 2 * MT>();
      slot = slot + 1 == SLOTS ? 0 : slot + 1;
      read_w((t + 1) & 1, slot);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[t][mt] = mfma16x16x32(wv[t & 1][j], av[mt][j], acc[t][mt]);
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_waitcnt(kLgkm0);
      copy_w((t + 1 + SLOTS) % R, i + (t + 1 + SLOTS) / R, slot);
    }
  }
  wait_vmcnt<0>();  // no copy may land in LDS from here on
  __syncthreads();
  f32x4_t* red = reinterpret_cast<f32x4_t*>(smem);
#pragma unroll
  for (int t = 0; t < R; ++t)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) red[((t * MT + mt) * 4 + wave) * 64 + lane] = acc[t][mt];
  __syncthreads();
  // lane (g, r) of accumulator (t, mt) holds C^T[row base + t*16 + 4g + e][m = mt*16 + r]
  auto total = [&](int t, int mt) {
    const f32x4_t* p = red + (t * MT + mt) * 4 * 64 + lane;
    return p[0] + p[64] + p[128] + p[192];
  };
  for (int q = wave; q < (SILU ? R / 2 : R) * MT; q += 4) {
    const int t = q / MT, mt = q % MT, m = mt * 16 + r;
    if (m >= a.M) continue;
    if (SILU) {
      const int i0 = (blockIdx.x * (R / 2) + t) * 16 + g * 4;
      if (i0 >= a.N) continue;
      const f32x4_t gv = total(t, mt), uv = total(t + R / 2, mt);
      uint2 pk;
      pk.x = static_cast<uint32_t>(bf16_of(silu_fast(gv[0]) * uv[0])) | (static_cast<uint32_t>(bf16_of(silu_fast(gv[1]) * uv[1])) << 16);
      pk.y = static_cast<uint32_t>(bf16_of(silu_fast(gv[2]) * uv[2])) | (static_cast<uint32_t>(bf16_of(silu_fast(gv[3]) * uv[3])) << 16);
      *reinterpret_cast<uint2*>(static_cast<bf16_t*>(a.act_out) + static_cast<size_t>(m) * a.N + i0) = pk;
    } else {
      const int n = (blockIdx.x * R + t) * 16 + g * 4;
      if (n >= a.N) continue;
      *reinterpret_cast<f32x4_t*>(a.part + (static_cast<size_t>(blockIdx.y) * a.M + m) * a.N + n) = total(t, mt);
    }
  }
}

// ---- prefill / large-batch tiled MFMA GEMM ---------------------------------
// Block tile: BM activation rows (m, 128 or 256) x BN weight rows (n, 128 or
// 256), K step 64, on v_mfma_f32_32x32x16_bf16.  Activations are the MFMA row
// operand and weights the column operand, so the 32 lanes of one accumulator
// register hold 32 consecutive n: coalesced stores.
//
// What bounds it is the CU's load path, not the MFMA pipes: a 256 x 256 tile
// moves 64 KB into LDS per K step for 2048 cycles of MFMA per SIMD.  With
// 64-byte K steps (half a cache line of every row) the loads alone took 86% of
// the kernel's time, and a burst of a stage's copies at the barrier kept the
// waves from issuing MFMAs until it was accepted.  Hence:
//  * K steps of 64 elements: a copy instruction (buffer_load_dwordx4 ... lds, no
//    register staging) takes 8 rows of one whole 128-byte line each;
//  * the tile is two activation halves x two weight halves, and a K step has
//    four phases, one per pair of halves.  A phase computes one pair from
//    registers while it reads the next half's fragments and issues the copies
//    of one half tile of a later stage, two per wave, between its MFMAs.
//    Fragments of halves 0 are read during the step before, those of halves 1
//    in its first two phases, so a half's LDS is free again well before its
//    stage ends: two stages (128 KB at 256 x 256) give every copy at least one
//    whole K step to land, with two barriers per step.
// The copies are inline assembly, so the compiler neither tracks them nor
// waits for all of them before a barrier; the kernel waits with explicit vmcnt
// counts (vector loads complete in order).  Measured at 9,216 rows of the 7B
// shapes: 1,270-1,290 TFLOP/s over the four projections (gate/up 1,280, down
// 1,320-1,360) against 1,126 with 32-element steps, three stages and a burst
// per stage; at 397 rows 270 against 278 us.  Measured and not kept: wave
// priorities around the MFMAs (2% slower), and blocks that walk several tiles
// and copy ahead across the epilogue (within 0.5% at the 7B shapes, 8% slower on
// the 0.5B LM head).
// The 16-byte chunk j of LDS row r holds global chunk j ^ ((r >> 1) & 7): a
// row is 128 bytes, half of the 64 banks, so sixteen consecutive rows of a
// fragment read hit sixteen distinct 16-byte bank groups.  Rows past M or N
// read as zeros through the buffer resources (range-checked loads); a 16-row
// block of a weight tile lies in one weight segment.  Each XCD takes a
// contiguous run of the (split, tile) order, split-major (block ids equal mod
// 8), and the order walks gm m tiles of one weight panel before the next panel,
// so the 32 tiles an XCD runs at once share gm activation tiles and 32 / gm
// weight panels in its L2.  gm is 8 for wide products (>= 64 panels: gate/up,
// the LM head) and 2 for narrow ones.
// The 16-byte chunk j of LDS row r (128 bytes) holds global chunk j ^ gswz(r).
__device__ __forceinline__ int gswz(int r) { return (r >> 1) & 7; }

template <int BM, int BN>
struct TiledCfg {
  static constexpr int WN = BN / 64, WM = BM == 128 && BN == 128 ? 2 : 8 / WN;  // waves along n and m
  static constexpr int WAVES = WM * WN;
  static constexpr int MT = BM / 2 / WM / 32;          // 32-row activation tiles of a wave per half
  static constexpr int NST = BM * BN == 256 * 256 ? 2 : BM * BN == 128 * 128 ? 2 : 3;  // LDS stages
  static constexpr int LA = BM / 16 / WAVES, LB = BN / 16 / WAVES;  // 1 KB copies of a wave per half tile
  static_assert(MT >= 1 && LA >= 1 && LB >= 1 && WN * 32 == BN / 2, "tile shape");
};

template <int BM, int BN, bool SILU>
__global__ __launch_bounds__((64 * TiledCfg<BM, BN>::WAVES)) void k_gemm_tiled(GemmArgs a, int kblocks_per_split, int n_mb, int n_nb, int nb0, int gm) {
  using C = TiledCfg<BM, BN>;
  constexpr int MT = C::MT, NST = C::NST, LA = C::LA, LB = C::LB, WAVES = C::WAVES;
  constexpr int ROWB = kGBK * 2;                                   // bytes of an LDS row
  constexpr int HA = BM / 2 * ROWB, HB = BN / 2 * ROWB, STAGE = 2 * (HA + HB);  // bytes: half tiles, a stage
  constexpr int KS = kGBK / 16;                                    // MFMA k-steps of a stage
  __shared__ __attribute__((aligned(1024))) uint8_t smem[NST * STAGE];
  // Work items are (split, tile) pairs, split-major, and each XCD takes a contiguous run of
  // them (block ids equal mod 8 run on one XCD): the XCDs get equal shares of a split launch
  // (per-tile runs would hand one XCD all splits of its tiles, more blocks than its 32 CUs
  // when the tile count is not a multiple of 8), and an XCD's blocks read few K ranges of
  // the activations, which its L2 then holds.
  const int n_tiles = n_mb * n_nb;
  const int n_items = n_tiles * a.splits;
  const int per_xcd = (n_items + 7) / 8;
  const int q = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (q >= n_items) return;  // block-uniform: padding of the XCD-ordered grid
  const int split = q / n_tiles, t = q - split * n_tiles;
  // Grouped order: consecutive tiles walk gm m tiles of one weight panel, then the next panel.
  const int gsz = gm * n_nb, grp = t / gsz, first = grp * gm, gcur = min(gm, n_mb - first);
  const int mb = first + (t - grp * gsz) % gcur, nb = nb0 + (t - grp * gsz) / gcur;  // panels nb0 .. nb0 + n_nb - 1
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % C::WM, wn = wave / C::WM;
  const int l32 = lane & 31, lh = lane >> 5;
  const int K = a.K;

  // Copies: wave w fills 8-row blocks w, w + WAVES, ... of each half tile; lane -> row lane >> 3 of
  // the block, LDS chunk lane & 7, which holds global chunk (lane & 7) ^ gswz(row).
  const u32x4_raw ars = raw_rsrc(a.A, static_cast<uint32_t>(a.M) * static_cast<uint32_t>(a.lda) * 2u);
  int aoff[2][LA], woff[2][LB];
  u32x4_raw wrs[2][LB];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
#pragma unroll
    for (int i = 0; i < LA; ++i) {
      const int r = (wave + WAVES * i) * 8 + (lane >> 3);
      aoff[h][i] = ((mb * BM + h * (BM / 2) + r) * static_cast<int>(a.lda) + ((lane & 7) ^ gswz(r)) * 8) * 2;
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      const int r0 = (wave + WAVES * i) * 8;
      const int r = r0 + (lane >> 3);
      const bf16_t* wb;
      int rel0, rows_valid;
      if (SILU) {  // half 0: gate, half 1: up, of the same output indices
        wb = static_cast<const bf16_t*>(a.W.ptr[h]);
        rel0 = nb * (BN / 2) + r0;
        rows_valid = a.N;
      } else {
        const int n0 = nb * BN + h * (BN / 2) + r0;
        int b = 0, sg = 0;
        while (sg < a.W.n_seg - 1 && n0 >= b + a.W.rows[sg]) b += a.W.rows[sg++];
        wb = static_cast<const bf16_t*>(a.W.ptr[sg]);
        rel0 = n0 - b;
        rows_valid = n0 < a.N ? a.W.rows[sg] : 0;
      }
      wrs[h][i] = raw_rsrc(wb, static_cast<uint32_t>(rows_valid) * static_cast<uint32_t>(K) * 2u);
      woff[h][i] = ((rel0 + (lane >> 3)) * K + ((lane & 7) ^ gswz(r)) * 8) * 2;
    }
  }
  typedef const __attribute__((address_space(3))) char lds_char;
  const uint32_t lds0 = static_cast<uint32_t>((uintptr_t)(lds_char*)(smem));

  f32x16_t acc[2][2][MT];
#pragma unroll
  for (int ah = 0; ah < 2; ++ah)
#pragma unroll
    for (int bh = 0; bh < 2; ++bh)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[ah][bh][mt][e] = 0.f;

  const int kb0 = split * kblocks_per_split;
  const int kb1 = min(kb0 + kblocks_per_split, K / kGBK);
  auto copy_a = [&](int h, int i, int st, int kb) {
    dma16(ars, __builtin_amdgcn_readfirstlane(lds0 + static_cast<uint32_t>(st * STAGE + h * HA + (wave + WAVES * i) * 1024)),
          aoff[h][i] + kb * ROWB);
  };
  auto copy_b = [&](int h, int i, int st, int kb) {
    dma16(wrs[h][i],
          __builtin_amdgcn_readfirstlane(lds0 + static_cast<uint32_t>(st * STAGE + 2 * HA + h * HB + (wave + WAVES * i) * 1024)),
          woff[h][i] + kb * ROWB);
  };
  // Fragment reads: lane (lh, l32) takes chunk 2 ks + lh of row l32 of a 32-row group; gswz depends on l32 only.
  const int sw = gswz(l32);
  const uint32_t arow = (wm * MT * 32 + l32) * ROWB, brow = 2 * HA + (wn * 32 + l32) * ROWB;
  bf16x8_t af[2][MT][KS], bw[2][KS];
  auto rd_a = [&](int h, int ks, int st) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
      af[h][mt][ks] = *reinterpret_cast<const bf16x8_t*>(smem + st * STAGE + arow + (((2 * ks + lh) ^ sw) * 16) + h * HA + mt * 32 * ROWB);
  };
  auto rd_b = [&](int h, int ks, int st) {
    bw[h][ks] = *reinterpret_cast<const bf16x8_t*>(smem + st * STAGE + brow + (((2 * ks + lh) ^ sw) * 16) + h * HB);
  };
  auto mm = [&](int ah, int bh, int ks) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[ah][bh][mt] = mfma32x32x16(af[ah][mt][ks], bw[bh][ks], acc[ah][bh][mt]);
  };

  // Copies past the last stage still issue (they read later columns, or zeros past the matrix, into
  // stages nobody reads again), so that every wait counts the same copies.
#pragma unroll
  for (int s = 0; s < NST; ++s) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int i = 0; i < LA; ++i) copy_a(h, i, s, kb0 + s);
#pragma unroll
      for (int i = 0; i < LB; ++i) copy_b(h, i, s, kb0 + s);
    }
  }
  constexpr int AHEAD = (LA + LB) * (2 * NST - 2);  // copies issued after the half tiles a barrier waits for
  wait_vmcnt<AHEAD + LA + LB>();
  __syncthreads();
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    rd_a(0, ks, 0);
    rd_b(0, ks, 0);
  }
  int st = 0;
  for (int kb = kb0; kb < kb1; ++kb) {
    const int nx = st + 1 == NST ? 0 : st + 1;
    wait_vmcnt<AHEAD>();  // halves 1 of stage kb have landed
    __syncthreads();      // for all waves, which have halves 0 of stage kb in registers
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if (ks < LA) copy_a(0, ks, st, kb + NST);
      rd_b(1, ks, st);
      mm(0, 0, ks);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if (ks < LB) copy_b(0, ks, st, kb + NST);
      rd_a(1, ks, st);
      mm(0, 1, ks);
      __builtin_amdgcn_sched_barrier(0);
    }
    wait_vmcnt<AHEAD>();  // halves 0 of stage kb + 1 have landed
    __syncthreads();      // for all waves, which have halves 1 of stage kb in registers
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if (ks < LB) copy_b(1, ks, st, kb + NST);
      rd_a(0, ks, nx);
      mm(1, 0, ks);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if (ks < LA) copy_a(1, ks, st, kb + NST);
      rd_b(0, ks, nx);
      mm(1, 1, ks);
      __builtin_amdgcn_sched_barrier(0);
    }
    st = nx;
  }
  wait_vmcnt<0>();  // no copy may land in this block's LDS after it ends

  // acc register e of tile (ah, mt): m = ah BM/2 + (wm MT + mt) 32 + 8 (e/4) + 4 lh + e%4, n = bh BN/2 + wn 32 + l32.
  // Stores go through a resource over the 32 rows of an (ah, mt) tile, which drops rows past M; columns past N
  // start out of range.  (A branch per element doubled the kernel's code: 2-3 us of instruction fetch a launch.)
  // Offsets are 32-bit, so the rows of a resource are few: 32 rows of up to 2^24 columns stay below kOut.
  constexpr int ESZ = SILU ? 2 : 4, kOut = static_cast<int>(0x80000000u);
  char* out = SILU ? static_cast<char*>(a.act_out) : reinterpret_cast<char*>(a.part + static_cast<size_t>(split) * a.M * a.N);
  int voff[2];
#pragma unroll
  for (int bh = 0; bh < (SILU ? 1 : 2); ++bh) {
    const int n = SILU ? nb * (BN / 2) + wn * 32 + l32 : nb * BN + bh * (BN / 2) + wn * 32 + l32;
    voff[bh] = n < a.N ? (4 * lh * a.N + n) * ESZ : kOut;
  }
#pragma unroll
  for (int ah = 0; ah < 2; ++ah)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int m0 = mb * BM + ah * (BM / 2) + (wm * MT + mt) * 32, rows = max(min(32, a.M - m0), 0);
      const uint64_t base = reinterpret_cast<uint64_t>(out) + static_cast<uint64_t>(m0) * static_cast<uint32_t>(a.N * ESZ);
      const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(base)),  // scalar: else a loop per store
                     hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(base >> 32));
      const __amdgpu_buffer_rsrc_t ors =
          buffer_rsrc(reinterpret_cast<void*>(static_cast<uint64_t>(hi) << 32 | lo),
                      __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(rows) * static_cast<uint32_t>(a.N * ESZ)));
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int row = (8 * (e >> 2) + (e & 3)) * a.N * ESZ;
        if (SILU) {
          __builtin_amdgcn_raw_buffer_store_b16(bf16_of(silu_fast(acc[ah][0][mt][e]) * acc[ah][1][mt][e]), ors, voff[0] + row, 0, 0);
        } else {
#pragma unroll
          for (int bh = 0; bh < 2; ++bh)
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[ah][bh][mt][e]), ors, voff[bh] + row, 0, 0);
        }
      }
    }
}

// ---- fp32 model ------------------------------------------------------------
// One block per 16 weight rows (with the SiLU epilogue: 16 gate and the 16 up
// rows of the same outputs) and up to 64 activation rows, on
// v_mfma_f32_16x16x4_f32 (fp32 products and sums).  The small fp32 decoder's
// products are launch- and latency-bound, so the K range is spread over the
// block's 4 waves in interleaved 16-wide chunks, whose loads are all independent:
// lane (g, r) reads elements 4g .. 4g + 3 of a row's chunk, and MFMA j takes the
// j-th of them from both operands, so every product is formed once.  VEC: rows
// are 16-byte aligned (one load per chunk); otherwise element loads.
// 8 rows, K = 256: 3-4 us a launch against 33-64 us for one 64 x 64 tile per
// block walking all of K (4-32 blocks, a barrier per 16 elements).
template <int MT, bool SILU, bool VEC>
__global__ __launch_bounds__(256) void k_gemm_f32(GemmArgs a) {
  constexpr int R = SILU ? 2 : 1, U = 4;  // weight fragments; chunks in flight per wave
  __shared__ __attribute__((aligned(16))) f32x4_t red[3][R * MT][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, r = lane & 15;
  const int K = a.K, m0 = blockIdx.y * (16 * MT);
  const float* wrow[R];
  const float* arow[MT];
  const int n_ld = min(static_cast<int>(blockIdx.x) * 16 + r, a.N - 1);  // rows past the end are not stored
#pragma unroll
  for (int t = 0; t < R; ++t)
    wrow[t] = SILU ? static_cast<const float*>(a.W.ptr[t]) + static_cast<size_t>(n_ld) * K : seg_row<float>(a.W, n_ld, K);
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
    arow[mt] = static_cast<const float*>(a.A) + static_cast<size_t>(min(m0 + mt * 16 + r, a.M - 1)) * a.lda;
  auto load4 = [&](const float* p, int k) {
    f32x4_t v{0.f, 0.f, 0.f, 0.f};
    if (VEC) {
      if (k < K) v = *reinterpret_cast<const f32x4_t*>(p + k);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (k + j < K) v[j] = p[k + j];
    }
    return v;
  };
  f32x4_t acc[R][MT];
#pragma unroll
  for (int t = 0; t < R; ++t)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[t][mt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const int n_chunks = (K + 15) / 16;
  for (int c0 = wave; c0 < n_chunks; c0 += 4 * U) {
    f32x4_t wv[U][R], av[U][MT];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = (c0 + 4 * u) * 16 + 4 * g;  // chunks past the end load zeros
#pragma unroll
      for (int t = 0; t < R; ++t) wv[u][t] = load4(wrow[t], k);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) av[u][mt] = load4(arow[mt], k);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int t = 0; t < R; ++t)
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
            acc[t][mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[u][t][j], av[u][mt][j], acc[t][mt], 0, 0, 0);
  }
  if (wave > 0) {
#pragma unroll
    for (int t = 0; t < R; ++t)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) red[wave - 1][t * MT + mt][lane] = acc[t][mt];
  }
  __syncthreads();
  if (wave > 0) return;
  // lane (g, r) holds C^T[n = 16 block + 4g + e][m = m0 + mt*16 + r]
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int m = m0 + mt * 16 + r;
    if (m >= a.M) continue;
    f32x4_t v[R];
#pragma unroll
    for (int t = 0; t < R; ++t)
      v[t] = acc[t][mt] + red[0][t * MT + mt][lane] + red[1][t * MT + mt][lane] + red[2][t * MT + mt][lane];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int n = blockIdx.x * 16 + 4 * g + e;
      if (n >= a.N) continue;
      if (SILU) static_cast<float*>(a.act_out)[static_cast<size_t>(m) * a.N + n] = silu(v[0][e]) * v[R - 1][e];
      else a.part[static_cast<size_t>(m) * a.N + n] = v[0][e];
    }
  }
}

template <int MT, bool SILU>
void launch_f32_t(const GemmArgs& a, hipStream_t s) {
  dim3 grid((a.N + 15) / 16, (a.M + 16 * MT - 1) / (16 * MT));
  uintptr_t addr = reinterpret_cast<uintptr_t>(a.A);
  for (int sg = 0; sg < a.W.n_seg; ++sg) addr |= reinterpret_cast<uintptr_t>(a.W.ptr[sg]);
  if (addr % 16 == 0 && a.K % 4 == 0 && a.lda % 4 == 0)
    launch_kernel((k_gemm_f32<MT, SILU, true>), grid, dim3(256), 0, s, a);
  else
    launch_kernel((k_gemm_f32<MT, SILU, false>), grid, dim3(256), 0, s, a);
}

template <bool SILU>
void launch_f32(const GemmArgs& a, hipStream_t s) {
  if (a.M <= 16) launch_f32_t<1, SILU>(a, s);
  else if (a.M <= 32) launch_f32_t<2, SILU>(a, s);
  else launch_f32_t<4, SILU>(a, s);
}

template <int R, int D, bool SILU>
void launch_deep_t(const GemmArgs& a, hipStream_t s) {
  const int KU = a.K / 64;
  const int ups = (KU + a.splits - 1) / a.splits;
  const int per = SILU ? R / 2 : R;
  const int nb = (a.N / 16 + per - 1) / per;
  if (a.Wp.n_seg > 0)
    launch_kernel((k_gemm_deep<R, D, SILU, true>), dim3(nb, a.splits), dim3(256), 0, s, a, ups);
  else
    launch_kernel((k_gemm_deep<R, D, SILU, false>), dim3(nb, a.splits), dim3(256), 0, s, a, ups);
}

template <int R, int MT, bool SILU>
void launch_ring_t(const GemmArgs& a, hipStream_t s) {
  const int KU = a.K / 64;
  const int ups = (KU + a.splits - 1) / a.splits;
  const int per = SILU ? R / 2 : R;
  const int nb = (a.N / 16 + per - 1) / per;
  if (a.Wp.n_seg > 0)
    launch_kernel((k_gemm_ring<R, MT, SILU, true>), dim3(nb, a.splits), dim3(256), 0, s, a, ups);
  else
    launch_kernel((k_gemm_ring<R, MT, SILU, false>), dim3(nb, a.splits), dim3(256), 0, s, a, ups);
}

template <bool SILU>
bool launch_ring(const GemmArgs& a, int R, hipStream_t s) {
#define RP_RING(R_)                                           \
  if (R == R_) {                                              \
    switch ((a.M + 15) / 16) {                                \
      case 1: launch_ring_t<R_, 1, SILU>(a, s); return true;  \
      case 2: launch_ring_t<R_, 2, SILU>(a, s); return true;  \
      case 3: launch_ring_t<R_, 3, SILU>(a, s); return true;  \
      case 4: launch_ring_t<R_, 4, SILU>(a, s); return true;  \
      default: return false;                                  \
    }                                                         \
  }
  RP_RING(2) RP_RING(4) RP_RING(6) RP_RING(8) RP_RING(10)
#undef RP_RING
  return false;
}

// One thread per 16-byte piece of the packed matrix (the layout of launch_pack_weights).
__global__ void k_pack_weights(const uint4* __restrict__ w, uint4* __restrict__ p, int rows, int K) {
  const size_t n = static_cast<size_t>(rows) * K / 8;
  const size_t tile_pieces = static_cast<size_t>(2) * K;  // 16 rows x K / 8
  for (size_t q = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x; q < n;
       q += static_cast<size_t>(gridDim.x) * blockDim.x) {
    const size_t t = q / tile_pieces, rem = q % tile_pieces;
    const int u = static_cast<int>(rem >> 7), j = static_cast<int>(rem >> 6) & 1, l = static_cast<int>(rem) & 63;
    p[q] = w[((t * 16 + (l & 15)) * static_cast<size_t>(K) + 64 * u + 16 * (l >> 4) + 8 * j) / 8];
  }
}

template <bool SILU>
bool launch_deep(const GemmArgs& a, int R, int D, hipStream_t s) {
  if (R == 10 && D == 2) { launch_deep_t<10, 2, SILU>(a, s); return true; }
  if (R == 8 && D == 2) { launch_deep_t<8, 2, SILU>(a, s); return true; }
  if (R == 4 && D == 4) { launch_deep_t<4, 4, SILU>(a, s); return true; }
  return false;
}

// Columns [n_lo, n_hi) of the product, n_lo at a panel's start.
void launch_tiled(const GemmArgs& a, int bm, int bn, int n_lo, int n_hi, hipStream_t s) {
  const bool silu = a.epi == kEpiSiluMul;
  const int kbps = (a.K / kGBK + a.splits - 1) / a.splits;
  const int n_nb = panels(n_hi - n_lo, bn, silu), nb0 = n_lo / (silu ? bn / 2 : bn);
  const int n_mb = (a.M + bm - 1) / bm;
  const int per_xcd = (n_mb * n_nb * a.splits + 7) / 8;
  const int gm = n_nb >= 64 ? 8 : 2;
  dim3 grid(8 * per_xcd);
#define RP_TILED(BM_, BN_)                                                                                   \
  if (bm == BM_ && bn == BN_) {                                                                              \
    constexpr int threads = 64 * TiledCfg<BM_, BN_>::WAVES;                                                  \
    if (silu) launch_kernel((k_gemm_tiled<BM_, BN_, true>), grid, dim3(threads), 0, s, a, kbps, n_mb, n_nb, nb0, gm); \
    else launch_kernel((k_gemm_tiled<BM_, BN_, false>), grid, dim3(threads), 0, s, a, kbps, n_mb, n_nb, nb0, gm);     \
  }
  RP_TILED(128, 128) RP_TILED(128, 256) RP_TILED(256, 128) RP_TILED(256, 256)
#undef RP_TILED
}

}  // namespace

int gemm_pick_splits(int bf16, int M, int N, int K, bool silu, int max_splits) {
  return plan_gemm(bf16, M, N, K, silu, 1, max_splits).splits;
}

hipError_t launch_pack_weights(const void* w, void* packed, int rows, int K, hipStream_t s) {
  if (!w || !packed || rows <= 0 || rows % 16 || K <= 0 || K % 64 ||
      (reinterpret_cast<uintptr_t>(w) | reinterpret_cast<uintptr_t>(packed)) % 16)
    return hipErrorInvalidValue;
  launch_kernel(k_pack_weights, dim3(2048), dim3(256), 0, s, static_cast<const uint4*>(w), static_cast<uint4*>(packed),
                rows, K);
  return hipGetLastError();
}

hipError_t launch_gemm(int bf16, const GemmArgs& a, hipStream_t s) {
  if (a.M <= 0) return hipSuccess;
  const bool silu = a.epi == kEpiSiluMul;
  if (a.splits < 1 || (silu && a.splits != 1)) return hipErrorInvalidValue;
  const GemmPlan plan = plan_launch(bf16, a.M, a.N, a.K, silu, a.splits);
  const int kernel = plan.kernel;
  if (!bf16 || kernel == kKF32) {
    if (bf16 || a.splits != 1) return hipErrorInvalidValue;
    if (silu) launch_f32<true>(a, s);
    else launch_f32<false>(a, s);
    return hipGetLastError();
  }
  if (kernel == kKTiled) {
    if (a.K % kGBK != 0 || (silu && a.N % 128 != 0) || (!silu && a.N % 8 != 0)) return hipErrorInvalidValue;
    // 32-bit buffer offsets; every weight segment but the last a whole number of 16-row blocks
    if (static_cast<int64_t>(a.M + 256) * a.lda * 2 >= (int64_t{1} << 31) || a.N >= 1 << 24) return hipErrorInvalidValue;
    for (int sg = 0; sg < a.W.n_seg; ++sg) {
      if (static_cast<int64_t>(a.W.rows[sg]) * a.K * 2 >= (int64_t{1} << 31)) return hipErrorInvalidValue;
      if (!silu && sg < a.W.n_seg - 1 && a.W.rows[sg] % 16 != 0) return hipErrorInvalidValue;
    }
    launch_tiled(a, plan.bm, plan.bn, 0, plan.n_first, s);
    if (plan.n_first < a.N) launch_tiled(a, plan.bm2, plan.bn2, plan.n_first, a.N, s);
    return hipGetLastError();
  }
  if (a.K % 64 != 0 || a.N % 16 != 0) return hipErrorInvalidValue;
  // 32-bit buffer offsets: activations, and one fragment's 16 weight rows
  if (static_cast<int64_t>(a.M) * a.lda * 2 >= (int64_t{1} << 30) || static_cast<int64_t>(a.K) * 32 >= (int64_t{1} << 30))
    return hipErrorInvalidValue;
  bool ok = false;
  if (kernel == kKRing) ok = silu ? launch_ring<true>(a, plan.R, s) : launch_ring<false>(a, plan.R, s);
  else if (kernel == kKDeep) ok = silu ? launch_deep<true>(a, plan.R, plan.D, s) : launch_deep<false>(a, plan.R, plan.D, s);
  if (!ok) return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace rollpack
