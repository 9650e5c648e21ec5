// Bandwidth-trivial kernels of the stage: RMSNorm, rotary embedding fused with the KV-cache
// append, KV import/export, and the one-time weight repack.
//
// The KV cache (paper Sec. 2.1: per-token keys and values kept so that a decode step only
// processes the new token) is paged in fixed-size pages addressed through per-request block
// tables.  Physical layout per layer:
//   K pool  [num_pages][n_kv_heads][row bytes / 64][page_size][64 bytes]   (a key row in 64-byte pieces,
//           piece g of the page's 16 tokens together: what one decode-attention load instruction fetches
//           is then contiguous, see k_pool_byte)
//   V pool  [num_pages][n_kv_heads][head_dim][page_size]   (token index fastest)
// Keys are stored after rotation.  The V layout puts 8 consecutive tokens of one channel in
// 16 bytes, which is exactly the MFMA operand of the P*V product in both attention kernels.
#include "tdp_device.h"
#include "tdp_kernels.h"

namespace tdp {

// ------------------------------------------------------------------ RMSNorm
// y = x * g / sqrt(mean(x^2) + eps); one workgroup per row, fp32 statistics.  x is the residual
// stream: bf16 as handed over by the previous stage, fp32 between the layers of this stage.
template <bool F32_IN>
__device__ __forceinline__ void load8(const void* row, int c, float (&f)[8]) {
  if (F32_IN) {
    const f32x4 a = *reinterpret_cast<const f32x4*>((const float*)row + c * 8);
    const f32x4 b = *reinterpret_cast<const f32x4*>((const float*)row + c * 8 + 4);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f[i] = a[i];
      f[i + 4] = b[i];
    }
  } else {
    const bf16x8 v = ld_bf16x8((const bf16*)row + c * 8);
#pragma unroll
    for (int i = 0; i < 8; ++i) f[i] = (float)v[i];
  }
}

template <bool F32_IN>
__global__ __launch_bounds__(256) void rmsnorm_kernel(const void* __restrict__ x, int64_t ldx,
                                                      const float* __restrict__ gain, float eps, int d,
                                                      bf16* __restrict__ y, OperandLayout y_lay) {
  const int row = blockIdx.x;
  const void* xr = F32_IN ? (const void*)((const float*)x + (int64_t)row * ldx)
                          : (const void*)((const bf16*)x + (int64_t)row * ldx);
  const int chunks = d / 8;
  // the row is read once: a thread keeps its first KEEP chunks (a row of up to 8192 elements whole) in
  // registers between the two passes and re-reads only what lies beyond
  constexpr int KEEP = 4;
  float keep[KEEP][8];
  float ss = 0.f;
#pragma unroll
  for (int k = 0; k < KEEP; ++k) {
    const int c = threadIdx.x + 256 * k;
    if (c < chunks) {
      load8<F32_IN>(xr, c, keep[k]);
#pragma unroll
      for (int i = 0; i < 8; ++i) ss += keep[k][i] * keep[k][i];
    }
  }
  for (int c = threadIdx.x + 256 * KEEP; c < chunks; c += 256) {
    float f[8];
    load8<F32_IN>(xr, c, f);
#pragma unroll
    for (int i = 0; i < 8; ++i) ss += f[i] * f[i];
  }
  __shared__ float red[4];
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  const float tot = red[0] + red[1] + red[2] + red[3];
  const float inv = 1.0f / sqrtf(tot / (float)d + eps);
  auto emit = [&](int c, const float (&f)[8]) {
    const f32x4 g0 = *reinterpret_cast<const f32x4*>(gain + c * 8);
    const f32x4 g1 = *reinterpret_cast<const f32x4*>(gain + c * 8 + 4);
    bf16x8 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      o[i] = (bf16)(f[i] * inv * g0[i]);
      o[i + 4] = (bf16)(f[i + 4] * inv * g1[i]);
    }
    st_bf16x8(y + operand_offset(y_lay, row, c * 8), o);
  };
#pragma unroll
  for (int k = 0; k < KEEP; ++k) {
    const int c = threadIdx.x + 256 * k;
    if (c < chunks) emit(c, keep[k]);
  }
  for (int c = threadIdx.x + 256 * KEEP; c < chunks; c += 256) {
    float f[8];
    load8<F32_IN>(xr, c, f);
    emit(c, f);
  }
}

hipError_t launch_rmsnorm(const void* x, int x_is_f32, int64_t ldx, const float* gain, float eps, int M, int d,
                          void* y, OperandLayout y_layout, hipStream_t s) {
  if (M <= 0) return hipSuccess;
  if (x_is_f32)
    rmsnorm_kernel<true><<<M, 256, 0, s>>>(x, ldx, gain, eps, d, (bf16*)y, y_layout);
  else
    rmsnorm_kernel<false><<<M, 256, 0, s>>>(x, ldx, gain, eps, d, (bf16*)y, y_layout);
  return hipGetLastError();
}

// Sum of split-K partials, eight consecutive columns at a time: acc = p_0 + p_1 + ... in split order
// (partial z of a row lies z * split_stride floats further on).  The partials are fetched UN
// splits at a time so that all of a thread's loads are in flight together: a loop that loads and adds
// one split per turn pays one memory round trip per split, which is what a launch of few rows
// (small decode batches) consists of.  `splits` is uniform, so the guards are scalar branches.
template <int NCOL, int UN>
__device__ __forceinline__ void sum_partials8(const float* const (&first)[NCOL], int64_t split_stride, int splits,
                                              float (&acc)[NCOL][8]) {
#pragma unroll
  for (int c = 0; c < NCOL; ++c)
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[c][i] = 0.f;
  for (int z0 = 0; z0 < splits; z0 += UN) {
    float f[UN][NCOL][8];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      if (z0 + u < splits) {
#pragma unroll
        for (int c = 0; c < NCOL; ++c) load8<true>(first[c] + (int64_t)(z0 + u) * split_stride, 0, f[u][c]);
      } else {
#pragma unroll
        for (int c = 0; c < NCOL; ++c)
#pragma unroll
          for (int i = 0; i < 8; ++i) f[u][c][i] = 0.f;
      }
    }
#pragma unroll
    for (int u = 0; u < UN; ++u)
#pragma unroll
      for (int c = 0; c < NCOL; ++c)
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[c][i] += f[u][c][i];
  }
}

// The row is formed first: h = residual + the split-K partials of the projection in front of the
// norm (summed in split order), stored as the fp32 residual stream, then normalised.  Up to 1024 threads
// per row: at d = 8192 every thread has one 8-element chunk, which it keeps in registers between the
// two passes; beyond that a thread re-reads what it wrote itself.
template <bool F32_RES>
__global__ __launch_bounds__(1024) void rmsnorm_sum_kernel(const void* __restrict__ residual, int64_t ldr,
                                                          const float* __restrict__ ws, int splits, int M,
                                                          int64_t ld_ws, float* __restrict__ h_out, int64_t ldh,
                                                          const float* __restrict__ gain, float eps, int d,
                                                          bf16* __restrict__ y, OperandLayout y_lay) {
  const int row = blockIdx.x;
  const void* rr = F32_RES ? (const void*)((const float*)residual + (int64_t)row * ldr)
                           : (const void*)((const bf16*)residual + (int64_t)row * ldr);
  float* hr = h_out + (int64_t)row * ldh;
  const int chunks = d / 8, threads = blockDim.x;
  const int64_t split_stride = (int64_t)M * ld_ws;
  float ss = 0.f;
  float keep[8];  // this thread's first chunk of h
  for (int c = threadIdx.x; c < chunks; c += threads) {
    float f[8], acc[1][8];
    load8<F32_RES>(rr, c, f);
    const float* const first[1] = {ws + (int64_t)row * ld_ws + c * 8};
    sum_partials8<1, 8>(first, split_stride, splits, acc);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      acc[0][i] += f[i];
      ss += acc[0][i] * acc[0][i];
    }
    *reinterpret_cast<f32x4*>(hr + c * 8) = f32x4{acc[0][0], acc[0][1], acc[0][2], acc[0][3]};
    *reinterpret_cast<f32x4*>(hr + c * 8 + 4) = f32x4{acc[0][4], acc[0][5], acc[0][6], acc[0][7]};
    if (c == (int)threadIdx.x) {
#pragma unroll
      for (int i = 0; i < 8; ++i) keep[i] = acc[0][i];
    }
  }
  __shared__ float red[16];
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  float tot = 0.f;
  for (int w = 0; w < threads / 64; ++w) tot += red[w];
  const float inv = 1.0f / sqrtf(tot / (float)d + eps);
  for (int c = threadIdx.x; c < chunks; c += threads) {
    float f[8];
    if (c == (int)threadIdx.x) {
#pragma unroll
      for (int i = 0; i < 8; ++i) f[i] = keep[i];
    } else {
      load8<true>(hr, c, f);
    }
    const f32x4 g0 = *reinterpret_cast<const f32x4*>(gain + c * 8);
    const f32x4 g1 = *reinterpret_cast<const f32x4*>(gain + c * 8 + 4);
    bf16x8 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      o[i] = (bf16)(f[i] * inv * g0[i]);
      o[i + 4] = (bf16)(f[i + 4] * inv * g1[i]);
    }
    st_bf16x8(y + operand_offset(y_lay, row, c * 8), o);
  }
}

// Threads of a row's workgroup: one per chunk of eight elements in whole waves, 1024 at most (waves without a chunk only
// lengthen the start and the barrier; 307 rows of 4096 9.4 -> 8.4 us, a two-layer step of 350 requests of the toy shape
// 76.4 -> 73.4).  The sum of squares does not depend on it: a thread holds the same chunks, waves without any added zero.
static int norm_threads(int d) {
  const int t = (d / 8 + 63) / 64 * 64;
  return t < 256 ? 256 : t < 1024 ? t : 1024;
}

hipError_t launch_rmsnorm_sum(const void* residual, int residual_is_f32, int64_t ldr, const float* ws, int splits,
                              int64_t ld_ws, float* h_out, int64_t ldh, const float* gain, float eps, int M, int d,
                              void* y, OperandLayout y_layout, hipStream_t s) {
  if (M <= 0) return hipSuccess;
  const int threads = norm_threads(d);
  if (residual_is_f32)
    rmsnorm_sum_kernel<true><<<M, threads, 0, s>>>(residual, ldr, ws, splits, M, ld_ws, h_out, ldh, gain, eps, d, (bf16*)y,
                                               y_layout);
  else
    rmsnorm_sum_kernel<false><<<M, threads, 0, s>>>(residual, ldr, ws, splits, M, ld_ws, h_out, ldh, gain, eps, d,
                                                (bf16*)y, y_layout);
  return hipGetLastError();
}

// ------------------------------------------------------------------ token -> (sequence, position)
__device__ __forceinline__ void locate_token(int t, const int32_t* ctx_lens, const int32_t* cu_seqlens,
                                             int n_seqs, int max_pages_per_seq, int& seq, int& pos) {
  if (ctx_lens) {  // decode: one token per request
    seq = t;
    pos = decode_position(ctx_lens[t], max_pages_per_seq);
  } else {         // prefill: largest s with cu_seqlens[s] <= t
    int lo = 0, hi = n_seqs - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (cu_seqlens[mid] <= t) lo = mid; else hi = mid - 1;
    }
    seq = lo;
    pos = t - cu_seqlens[lo];
  }
}

// ------------------------------------------------------------------ RoPE + KV append
// The projection arrives in fp32 - the GEMM's fp32 output, or its split-K
// partials, summed here in split order (plus the bias) - so the rotation works on unrounded sums and
// every query and key element is rounded exactly once, after the rotation.  q heads are rotated and
// written to the bf16 row the attention kernels read; k heads are rotated and written to the token's
// slot of the K pool; v heads are written (transposed) to the V pool, or, in prefill, rounded into
// the bf16 row for the page-by-page append that follows.  Rotation pairs channel i with channel
// i + head_dim/2 and turns the pair by pos * base^(-2i/head_dim); the table holds (cos, sin) of that
// angle, computed in double precision on the host.
//
// (Small decode batches do this inside the attention kernel, see attn_decode_rotates, an unsplit projection of a prefill in its
// epilogue, see gemm_can_rotate.)
//
// A unit is eight rotated pairs or eight values; a token's units are walked by gridDim.y workgroups of 256 threads.
// Bound: reading the partials for many rows, one round trip per dependent look-up for few.  In decode, and in prefill
// where there are partials to sum, every unit has a thread of its own, which asks for the partials of UN splits at
// once; only a prefill without partials takes one workgroup per token (its look-ups are shared).  As one workgroup of 1024
// threads per token that fetched a split per turn, a launch of 48 (7B shape) / 128 (13B shape) / 512 tokens took
// 11.3 / 17.6 / 20.5 us, now 8.1 / 16 / 21 (what is left of the last two is the value append: 2-byte stores
// 32 bytes apart).
template <int UN>
__global__ __launch_bounds__(256) void rope_kv_kernel(bf16* __restrict__ qkv, int64_t ld, int n_q_heads,
                                                      KvLayout kv, const float2* __restrict__ table,
                                                      const int32_t* __restrict__ ctx_lens,
                                                      const int32_t* __restrict__ cu_seqlens, int n_seqs,
                                                      const int32_t* __restrict__ block_tables,
                                                      int max_pages_per_seq, const float* __restrict__ proj,
                                                      int splits, int n_tokens, const float* __restrict__ bias,
                                                      int v_to_row) {
  const int t = blockIdx.x;
  // NCOL groups of eight consecutive projection outputs of this token, starting at columns col[]
  const int64_t split_stride = (int64_t)n_tokens * ld;
  auto proj8 = [&](auto& f, auto... col) {
    constexpr int NCOL = sizeof...(col);
    const float* const first[NCOL] = {(proj + (int64_t)t * ld + col)...};
    const int cols[NCOL] = {col...};
    sum_partials8<NCOL, UN>(first, split_stride, splits, f);
    if (bias) {
#pragma unroll
      for (int c = 0; c < NCOL; ++c) {
        float g[8];
        load8<true>(bias + cols[c], 0, g);
#pragma unroll
        for (int i = 0; i < 8; ++i) f[c][i] += g[i];
      }
    }
  };
  int seq, pos;
  locate_token(t, ctx_lens, cu_seqlens, n_seqs, max_pages_per_seq, seq, pos);
  const int dh = kv.head_dim, half = dh >> 1;
  const int page = block_tables[(int64_t)seq * max_pages_per_seq + pos / kv.page_size];
  const int slot = pos % kv.page_size;
  bf16* row = qkv + (int64_t)t * ld;
  const float2* cs = table + (int64_t)pos * half;
  const int head_shift = dh == 128 ? 3 : 2;  // units of eight pairs per head
  const int rot_units = (n_q_heads + kv.n_kv_heads) << head_shift;
  const int units = rot_units + kv.n_kv_heads * dh / 8;
  const int v_col = (n_q_heads + kv.n_kv_heads) * dh;
  bf16* vpool = (bf16*)kv.v_pool;
  for (int w = blockIdx.y * 256 + threadIdx.x; w < units; w += gridDim.y * 256) {
    if (w < rot_units) {
      const int head = w >> head_shift;
      const int c0 = (w & ((1 << head_shift) - 1)) * 8;
      bf16* hp = row + (int64_t)head * dh;
      float ab[2][8];
      proj8(ab, head * dh + c0, head * dh + half + c0);
      const float(&a)[8] = ab[0];
      const float(&b)[8] = ab[1];
      float fra[8], frb[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) rotate_pair(a[i], b[i], cs[c0 + i], i, fra[i], frb[i]);
      // byte offsets of this thread's two 8-channel pieces in the K pool (a piece never straddles a 64-byte cut)
      const int esz = kv.fp8 ? 1 : 2;
      const int64_t k_lo = head >= n_q_heads ? k_pool_byte(kv, page, head - n_q_heads, slot, c0 * esz) : 0;
      const int64_t k_hi = head >= n_q_heads ? k_pool_byte(kv, page, head - n_q_heads, slot, (half + c0) * esz) : 0;
      if (head >= n_q_heads && kv.fp8) {
        // 8-bit cache: the rotated key goes from fp32 straight to its code (one rounding)
        uint2 ca = make_uint2(0u, 0u), cb = make_uint2(0u, 0u);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          ca.x |= f32_to_e4m3(fra[i] / kv.k_scale) << (8 * i);
          ca.y |= f32_to_e4m3(fra[4 + i] / kv.k_scale) << (8 * i);
          cb.x |= f32_to_e4m3(frb[i] / kv.k_scale) << (8 * i);
          cb.y |= f32_to_e4m3(frb[4 + i] / kv.k_scale) << (8 * i);
        }
        *reinterpret_cast<uint2*>((uint8_t*)kv.k_pool + k_lo) = ca;
        *reinterpret_cast<uint2*>((uint8_t*)kv.k_pool + k_hi) = cb;
        continue;
      }
      bf16x8 ra, rb;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        ra[i] = (bf16)fra[i];
        rb[i] = (bf16)frb[i];
      }
      if (head < n_q_heads) {
        st_bf16x8(hp + c0, ra);
        st_bf16x8(hp + half + c0, rb);
      } else {
        st_bf16x8(reinterpret_cast<bf16*>((uint8_t*)kv.k_pool + k_lo), ra);
        st_bf16x8(reinterpret_cast<bf16*>((uint8_t*)kv.k_pool + k_hi), rb);
      }
    } else {
      const int c = (w - rot_units) * 8;  // value channel, counted through the heads
      float fv[1][8];
      proj8(fv, v_col + c);
      const float(&f)[8] = fv[0];
      if (v_to_row) {  // prefill: the values are appended page by page (v_append_pages_kernel)
        bf16x8 o;
#pragma unroll
        for (int i = 0; i < 8; ++i) o[i] = (bf16)f[i];
        st_bf16x8(row + v_col + c, o);
        continue;
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        // pools are [page][kv head][channel][16 slots]
        const int64_t vi = ((int64_t)page * kv.n_kv_heads * dh + c + i) * kv.page_size + slot;
        // the value is a bf16 quantity in both forms of the cache (the 8-bit code is taken from it)
        const bf16 vb = (bf16)f[i];
        if (kv.fp8)
          ((uint8_t*)kv.v_pool)[vi] = (uint8_t)f32_to_e4m3((float)vb / kv.v_scale);
        else
          vpool[vi] = vb;
      }
    }
  }
}

// The page that chunk w of a grid over (sequence, page) pairs stands for: the last sequence s with cu_seqlens[s] / 16 + s
// <= w and its page w - (cu_seqlens[s] / 16 + s); the numbering leaves every sequence room for all its pages, a chunk past
// a sequence's last page gives false.  The last sequence ends at total_tokens.
__device__ __forceinline__ bool locate_page(int w, const int32_t* cu_seqlens, int n_seqs, int total_tokens, int& seq,
                                            int& p, int& t_first, int& n) {
  int lo = 0, hi = n_seqs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if ((cu_seqlens[mid] >> 4) + mid <= w) lo = mid; else hi = mid - 1;
  }
  seq = lo;
  t_first = cu_seqlens[lo];
  const int end = lo == n_seqs - 1 ? total_tokens : min(cu_seqlens[lo + 1], total_tokens);
  p = w - ((t_first >> 4) + lo);
  if (p < 0 || p * 16 >= end - t_first) return false;
  n = min(16, end - t_first - p * 16);
  return true;
}

// A page's 16 tokens x up to CH channels, turned round in LDS between token rows and the transposed V page.
constexpr int kPageChannels = 512;
template <int CH>
using PageTile = bf16[16][CH + 8];  // [token][channel]; rows 4 banks apart
// piece i (16 bytes of a token row): eight pieces of a row, then the 16 tokens, then the next 64 channels - a wave's
// instruction covers 8 tokens x 128 bytes
__device__ __forceinline__ int page_piece_token(int i) { return (i >> 3) & 15; }
__device__ __forceinline__ int page_piece_channel(int i) { return ((i & 7) + ((i >> 7) << 3)) * 8; }

// tile -> page [channel][16 tokens], tokens < n only; all 256 threads (8-bit: with few channels, two threads for each)
template <bool KV8, int CH, bool NT>
__device__ __forceinline__ void store_v_page(const PageTile<CH>& tile, uint8_t* v_page, int channels, int n, float v_scale) {
  if constexpr (KV8) {
    constexpr int PARTS = CH < 256 ? 2 : 1, TOK = 16 / PARTS;
    for (int i = threadIdx.x; i < channels * PARTS; i += 256) {
      const int c = i / PARTS, t0 = i % PARTS * TOK;
      if (t0 >= n) continue;
      uint32_t w[TOK / 4];
#pragma unroll
      for (int q = 0; q < TOK / 4; ++q) w[q] = 0u;
#pragma unroll
      for (int t = 0; t < TOK; ++t)
        if (t0 + t < n) w[t >> 2] |= f32_to_e4m3((float)tile[t0 + t][c] / v_scale) << (8 * (t & 3));
      uint8_t* dst = v_page + c * 16 + t0;
      if (t0 + TOK <= n) {
        if constexpr (TOK == 16) *reinterpret_cast<uint4*>(dst) = make_uint4(w[0], w[1], w[2], w[3]);
        else *reinterpret_cast<uint2*>(dst) = make_uint2(w[0], w[1]);
      } else {
#pragma unroll
        for (int t = 0; t < TOK; ++t)
          if (t0 + t < n) dst[t] = (uint8_t)(w[t >> 2] >> (8 * (t & 3)));
      }
    }
  } else {
    // two channels and eight tokens per thread: dword reads of the tile
    for (int i = threadIdx.x; i < channels; i += 256) {
      const int t0 = (i & 1) * 8, c = i & ~1;
      if (t0 >= n) continue;
      bf16x8 a, b;
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const bf16x2 ab = *reinterpret_cast<const bf16x2*>(&tile[t0 + t][c]);
        a[t] = ab[0];
        b[t] = ab[1];
      }
      bf16* dst = reinterpret_cast<bf16*>(v_page) + c * 16 + t0;
      if (t0 + 8 <= n) {
        st_bf16x8_once<NT>(dst, a);
        st_bf16x8_once<NT>(dst + 16, b);
      } else {
#pragma unroll
        for (int t = 0; t < 8; ++t)
          if (t0 + t < n) {
            dst[t] = a[t];
            dst[16 + t] = b[t];
          }
      }
    }
  }
}

// Prefill, values rounded to bf16 in the token rows: the values of one page (up to 16 consecutive tokens of one
// prompt) are appended by one workgroup per 512 channels, so that a channel's row of the transposed V page is written
// as one piece (token by token every 2-byte store dirtied a 32-byte sector of its own: measured ten
// times the bytes).  Turned round in LDS like the import (kv_move_kernel): rows are read in whole lines and a page is
// written 16 bytes per lane; with the 16 x 8 block of a thread in registers and one workgroup for all channels a
// launch took 10.7 us on a prompt of 307 tokens (32 x 128 channels) and 35 us on 19,346 (8 x 128), now 5.3 and 24.7.
template <bool KV8>
__global__ __launch_bounds__(256) void v_append_pages_kernel(const bf16* __restrict__ qkv, int64_t ld, int v_col,
                                                             KvLayout kv, const int32_t* __restrict__ cu_seqlens,
                                                             int n_seqs, int total_tokens,
                                                             const int32_t* __restrict__ block_tables,
                                                             int max_pages_per_seq) {
  constexpr int CH = kPageChannels, PER = 16 * CH / 8 / 256;
  __shared__ __attribute__((aligned(16))) PageTile<CH> tile;
  int seq, p, t_first, n;
  if (!locate_page(blockIdx.x, cu_seqlens, n_seqs, total_tokens, seq, p, t_first, n)) return;
  const int64_t page = block_tables[(int64_t)seq * max_pages_per_seq + p];
  const int dkv = kv.n_kv_heads * kv.head_dim, c0 = blockIdx.y * CH, channels = min(CH, dkv - c0);
  const bf16* src = qkv + (int64_t)(t_first + p * 16) * ld + v_col + c0;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int i = threadIdx.x + 256 * j, tok = page_piece_token(i), ch = page_piece_channel(i);
    if (i < channels * 2 && tok < n) st_bf16x8(&tile[tok][ch], ld_bf16x8(src + (int64_t)tok * ld + ch));
  }
  __syncthreads();
  store_v_page<KV8, CH, false>(tile, (uint8_t*)kv.v_pool + (page * dkv + c0) * (KV8 ? 16 : 32), channels, n, kv.v_scale);
}

__global__ __launch_bounds__(256) void token_pages_kernel(const int32_t* __restrict__ cu_seqlens, int n_seqs, int n_tokens,
                                                          const int32_t* __restrict__ block_tables, int max_pages_per_seq,
                                                          int2* __restrict__ token_pages) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t >= n_tokens) return;
  int seq, pos;
  locate_token(t, nullptr, cu_seqlens, n_seqs, max_pages_per_seq, seq, pos);
  token_pages[t] = make_int2(pos, block_tables[(int64_t)seq * max_pages_per_seq + pos / 16]);
}

hipError_t launch_token_pages(const int32_t* cu_seqlens, int n_seqs, int n_tokens, const int32_t* block_tables, int max_pages_per_seq,
                              int2* token_pages, hipStream_t s) {
  if (n_tokens <= 0) return hipSuccess;
  token_pages_kernel<<<(n_tokens + 255) / 256, 256, 0, s>>>(cu_seqlens, n_seqs, n_tokens, block_tables, max_pages_per_seq, token_pages);
  return hipGetLastError();
}

hipError_t launch_v_append(const void* qkv, int64_t ld, int n_tokens, int n_q_heads, const KvLayout& kv, const int32_t* cu_seqlens,
                           int n_seqs, const int32_t* block_tables, int max_pages_per_seq, hipStream_t s) {
  if (n_tokens <= 0) return hipSuccess;
  const int dkv = kv.n_kv_heads * kv.head_dim, v_col = n_q_heads * kv.head_dim + dkv;
  const dim3 grid((n_tokens >> 4) + n_seqs + 1, (dkv + kPageChannels - 1) / kPageChannels);
  if (kv.fp8)
    v_append_pages_kernel<true><<<grid, 256, 0, s>>>((const bf16*)qkv, ld, v_col, kv, cu_seqlens, n_seqs, n_tokens, block_tables,
                                                     max_pages_per_seq);
  else
    v_append_pages_kernel<false><<<grid, 256, 0, s>>>((const bf16*)qkv, ld, v_col, kv, cu_seqlens, n_seqs, n_tokens, block_tables,
                                                      max_pages_per_seq);
  return hipGetLastError();
}

hipError_t launch_rope_kv(void* qkv, int64_t ld, int n_tokens, int n_q_heads, const KvLayout& kv,
                          const float2* rope_table, int max_pos, const int32_t* ctx_lens,
                          const int32_t* cu_seqlens, int n_seqs, const int32_t* block_tables,
                          int max_pages_per_seq, const float* proj, int splits, const float* bias, hipStream_t s) {
  (void)max_pos;
  if (n_tokens <= 0) return hipSuccess;
  // prefill: the values go page by page; decode (one token per request) has nothing to gather
  const int paged_v = ctx_lens == nullptr;
  const int dh = kv.head_dim;
  const int units = (n_q_heads + kv.n_kv_heads) * (dh / 16) + kv.n_kv_heads * dh / 8;
  const dim3 grid(n_tokens, splits > 1 || !paged_v ? (units + 255) / 256 : 1);
  if (splits > 1)
    rope_kv_kernel<2><<<grid, 256, 0, s>>>((bf16*)qkv, ld, n_q_heads, kv, rope_table, ctx_lens, cu_seqlens, n_seqs,
                                           block_tables, max_pages_per_seq, proj, splits, n_tokens, bias, paged_v);
  else
    rope_kv_kernel<1><<<grid, 256, 0, s>>>((bf16*)qkv, ld, n_q_heads, kv, rope_table, ctx_lens, cu_seqlens, n_seqs,
                                           block_tables, max_pages_per_seq, proj, 1, n_tokens, bias, paged_v);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || !paged_v) return e;
  return launch_v_append(qkv, ld, n_tokens, n_q_heads, kv, cu_seqlens, n_seqs, block_tables, max_pages_per_seq, s);
}

// ------------------------------------------------------------------ KV import / export
// One workgroup moves 16 tokens x up to CH channels of K and of V between the packed arrays and one page.  Bound: HBM
// (every byte read once and written once).  A wave's instruction covers 8 tokens x 128 bytes, i.e. whole
// lines of the packed side and runs of 512 bytes of the key page; values turn round in LDS, so that the
// transposed page is read and written 16 bytes (8 tokens of a channel; 8-bit: all 16) at a time.  Element by element,
// with 2-byte accesses on both sides, 23,000 tokens of 40 x 128 channels took 790 us in and 450 us out (0.96 GB each:
// 1.2 and 2.1 TB/s); like this 195 and 192 us (4.9 TB/s; a plain copy reaches 4.7).
// Non-temporal loads (NTL) and stores (NTS), by the bytes of the packed keys and values, plain below 16 MiB.  What stands behind a move
// counts as much as the move: an imported cache is there for the next step to read.  All us, 13B shape, both ways in turn; "in + out":
// import and export of three caches in turn; "step": import, then the decode step that reads it.
//   Import, 16 bits: stores up to 64 MiB (34 MB in + out 34.9 -> 29.2, step 152.9 and 153.7; 50 MB 48.8 -> 46.8, step 160.5 and 161.6), from
//   there on the packed arrays are loaded so and the pages stored as usual (90 MB in + out 84.3 -> 80.8, step 180.0 -> 176.9; 250 MB 210.7 ->
//   209.3, step 274.0 -> 262.6; arrays just written, import, step 371 -> 358).  Pages stored so cost the step more than the move gains: 250
//   MB, step 289 with non-temporal stores, 285 with both.
//   Import, 8 bits: half the bytes are stored, plain, and from 64 MiB on loaded so (90 MB in + out 88.0 -> 84.5, step 188.6 -> 186.8).
//   Export: stores (decode step, then export: 70 MB 175.6 -> 170.6, 8 bits 171.0 -> 167.0), from 256 MiB on, what the memory-side cache
//   holds, 16-bit loads as well (400 MB 389.9 -> 377.3, stores alone 381.8).  Below that a cache may still hold the pages (24 MB, the
//   same cache again and again, 17.5 and 22.0).
template <bool KV8, bool TO_PAGES, int CH, bool NTL, bool NTS>
__global__ __launch_bounds__(256) void kv_move_kernel(bf16* __restrict__ k_packed, bf16* __restrict__ v_packed,
                                                      KvLayout kv, const int32_t* __restrict__ cu_seqlens, int n_seqs,
                                                      int total_tokens, const int32_t* __restrict__ block_tables,
                                                      int max_pages_per_seq) {
  constexpr int PER = 16 * CH / 8 / 256;  // 16-byte pieces of K (and of V) per thread
  __shared__ __attribute__((aligned(16))) PageTile<CH> tile;
  int seq, p, t_first, n;
  if (!locate_page(blockIdx.x, cu_seqlens, n_seqs, total_tokens, seq, p, t_first, n)) return;
  const int64_t page = block_tables[(int64_t)seq * max_pages_per_seq + p];
  const int dh = kv.head_dim, dkv = kv.n_kv_heads * dh, dh_shift = dh == 128 ? 7 : 6;
  const int c0 = blockIdx.y * CH;
  const int channels = min(CH, dkv - c0);  // a multiple of 64
  const int64_t at = (int64_t)(t_first + p * 16) * dkv + c0;
  bf16* kp = k_packed + at;
  bf16* vp = v_packed + at;
  uint8_t* v_page = (uint8_t*)kv.v_pool + (page * dkv + c0) * (KV8 ? 16 : 32);  // [channel][16 tokens]
  const int pieces = channels * 2;
  auto k_at = [&](int tok, int ch) {
    const int c = c0 + ch;
    return (uint8_t*)kv.k_pool + k_pool_byte(kv, page, c >> dh_shift, tok, (c & (dh - 1)) * (KV8 ? 1 : 2));
  };
  if constexpr (TO_PAGES) {
    bf16x8 k[PER], v[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int i = threadIdx.x + 256 * j, tok = page_piece_token(i), ch = page_piece_channel(i);
      if (i < pieces && tok < n) {
        k[j] = ld_bf16x8_once<NTL>(kp + (int64_t)tok * dkv + ch);
        v[j] = ld_bf16x8_once<NTL>(vp + (int64_t)tok * dkv + ch);
      }
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int i = threadIdx.x + 256 * j, tok = page_piece_token(i), ch = page_piece_channel(i);
      if (i < pieces && tok < n) {
        st_bf16x8(&tile[tok][ch], v[j]);
        if constexpr (KV8) {
          uint2 c = make_uint2(0u, 0u);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            c.x |= f32_to_e4m3((float)k[j][e] / kv.k_scale) << (8 * e);
            c.y |= f32_to_e4m3((float)k[j][4 + e] / kv.k_scale) << (8 * e);
          }
          *reinterpret_cast<uint2*>(k_at(tok, ch)) = c;
        } else {
          st_bf16x8_once<NTS>(reinterpret_cast<bf16*>(k_at(tok, ch)), k[j]);
        }
      }
    }
    __syncthreads();
    store_v_page<KV8, CH, NTS>(tile, v_page, channels, n, kv.v_scale);
  } else {
    bf16x8 k[PER];
    uint2 k8[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int i = threadIdx.x + 256 * j, tok = page_piece_token(i), ch = page_piece_channel(i);
      if (i < pieces && tok < n) {
        if constexpr (KV8) k8[j] = *reinterpret_cast<const uint2*>(k_at(tok, ch));
        else k[j] = ld_bf16x8_once<NTL>(reinterpret_cast<const bf16*>(k_at(tok, ch)));
      }
    }
    if constexpr (KV8) {
      constexpr int PARTS = CH < 256 ? 2 : 1, TOK = 16 / PARTS;
      for (int i = threadIdx.x; i < channels * PARTS; i += 256) {
        const int c = i / PARTS, t0 = i % PARTS * TOK;
        uint32_t w[TOK / 4];
        if constexpr (TOK == 16) {
          const uint4 raw = *reinterpret_cast<const uint4*>(v_page + c * 16);
          w[0] = raw.x, w[1] = raw.y, w[2] = raw.z, w[3] = raw.w;
        } else {
          const uint2 raw = *reinterpret_cast<const uint2*>(v_page + c * 16 + t0);
          w[0] = raw.x, w[1] = raw.y;
        }
#pragma unroll
        for (int t = 0; t < TOK; ++t)
          tile[t0 + t][c] = (bf16)(e4m3_to_f32((w[t >> 2] >> (8 * (t & 3))) & 255u) * kv.v_scale);
      }
    } else {
      for (int i = threadIdx.x; i < channels; i += 256) {
        const int t0 = (i & 1) * 8, c = i & ~1;
        const bf16* src = reinterpret_cast<const bf16*>(v_page) + c * 16 + t0;
        const bf16x8 a = ld_bf16x8_once<NTL>(src), b = ld_bf16x8_once<NTL>(src + 16);
#pragma unroll
        for (int t = 0; t < 8; ++t) *reinterpret_cast<bf16x2*>(&tile[t0 + t][c]) = bf16x2{a[t], b[t]};
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int i = threadIdx.x + 256 * j, tok = page_piece_token(i), ch = page_piece_channel(i);
      if (i < pieces && tok < n) {
        if constexpr (KV8) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            k[j][e] = (bf16)(e4m3_to_f32((k8[j].x >> (8 * e)) & 255u) * kv.k_scale);
            k[j][4 + e] = (bf16)(e4m3_to_f32((k8[j].y >> (8 * e)) & 255u) * kv.k_scale);
          }
        }
        st_bf16x8_once<NTS>(kp + (int64_t)tok * dkv + ch, k[j]);
        st_bf16x8_once<NTS>(vp + (int64_t)tok * dkv + ch, ld_bf16x8(&tile[tok][ch]));
      }
    }
  }
}

// The same element by element, for packed arrays that are not 16-byte aligned and for the smallest 8-bit imports.
__global__ __launch_bounds__(256) void kv_copy_kernel(int to_pages, bf16* __restrict__ k_packed,
                                                      bf16* __restrict__ v_packed, KvLayout kv,
                                                      const int32_t* __restrict__ cu_seqlens, int n_seqs,
                                                      const int32_t* __restrict__ block_tables,
                                                      int max_pages_per_seq) {
  const int t = blockIdx.x;
  int seq, pos;
  locate_token(t, nullptr, cu_seqlens, n_seqs, max_pages_per_seq, seq, pos);
  const int dh = kv.head_dim;
  const int page = block_tables[(int64_t)seq * max_pages_per_seq + pos / kv.page_size];
  const int slot = pos % kv.page_size;
  bf16* kpool = (bf16*)kv.k_pool;
  bf16* vpool = (bf16*)kv.v_pool;
  for (int w = threadIdx.x; w < kv.n_kv_heads * dh; w += 256) {
    const int kvh = w / dh, c = w % dh;
    const int64_t ki = k_pool_byte(kv, page, kvh, slot, c * (kv.fp8 ? 1 : 2)) / (kv.fp8 ? 1 : 2);  // element index
    const int64_t vi = (((int64_t)page * kv.n_kv_heads + kvh) * dh + c) * kv.page_size + slot;
    const int64_t pi = (int64_t)t * kv.n_kv_heads * dh + w;
    if (kv.fp8) {
      // packed side stays bf16: import encodes value / scale, export gives code value * scale
      uint8_t* k8 = (uint8_t*)kv.k_pool;
      uint8_t* v8 = (uint8_t*)kv.v_pool;
      if (to_pages) {
        k8[ki] = (uint8_t)f32_to_e4m3((float)k_packed[pi] / kv.k_scale);
        v8[vi] = (uint8_t)f32_to_e4m3((float)v_packed[pi] / kv.v_scale);
      } else {
        k_packed[pi] = (bf16)(e4m3_to_f32(k8[ki]) * kv.k_scale);
        v_packed[pi] = (bf16)(e4m3_to_f32(v8[vi]) * kv.v_scale);
      }
    } else if (to_pages) {
      kpool[ki] = k_packed[pi];
      vpool[vi] = v_packed[pi];
    } else {
      k_packed[pi] = kpool[ki];
      v_packed[pi] = vpool[vi];
    }
  }
}

// ------------------------------------------------------------------ E4M3 conversion (diagnostic)
__global__ void e4m3_encode_kernel(const float* __restrict__ src, uint8_t* __restrict__ dst, int64_t n, float scale) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = (uint8_t)f32_to_e4m3(src[i] / scale);
}
// decodes four codes per thread with the conversion the attention kernel uses; n is rounded up to
// a multiple of four by the caller's buffers
__global__ void e4m3_decode_kernel(const uint32_t* __restrict__ src, float* __restrict__ dst, int64_t n4) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n4) return;
  uint32_t lo, hi;
  e4m3x4_to_bf16x4(src[i], lo, hi);
  float4 o;
  o.x = __uint_as_float(lo << 16);
  o.y = __uint_as_float(lo & 0xffff0000u);
  o.z = __uint_as_float(hi << 16);
  o.w = __uint_as_float(hi & 0xffff0000u);
  reinterpret_cast<float4*>(dst)[i] = o;
}

hipError_t launch_e4m3_convert(int to_codes, const void* src, void* dst, int64_t n, float scale, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (to_codes)
    e4m3_encode_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>((const float*)src, (uint8_t*)dst, n, scale);
  else
    e4m3_decode_kernel<<<(unsigned)((n / 4 + 255) / 256), 256, 0, s>>>((const uint32_t*)src, (float*)dst, n / 4);
  return hipGetLastError();
}

hipError_t launch_kv_copy(int to_pages, void* k_packed, void* v_packed, const KvLayout& kv,
                          const int32_t* cu_seqlens, int n_seqs, int total_tokens,
                          const int32_t* block_tables, int max_pages_per_seq, hipStream_t s) {
  if (total_tokens <= 0) return hipSuccess;
  const int dkv = kv.n_kv_heads * kv.head_dim, pages = (total_tokens >> 4) + n_seqs + 1;
  const bool aligned = (((uintptr_t)k_packed | (uintptr_t)v_packed) & 15) == 0;
  // 8-bit imports of a few small tokens go element by element: one or two codes per thread instead of 16 in a row (128 channels,
  // 256 / 2048 tokens 4.3 / 4.4 us against 4.6 / 4.9 page by page; 3072 tokens 5.8 against 5.0)
  const bool few = kv.fp8 && to_pages && dkv <= 256 && total_tokens <= 2048;
  if (aligned && !few) {
    // 128 channels per workgroup as long as the chip could hold the workgroups of 512 channels all at once (eight per CU): the
    // time is then a thread's own chain, above all the conversions of an 8-bit import, 16 of them and not 64 (1024 channels, 8 bits:
    // 32 / 1024 tokens 4.5 / 5.9 us against 11.2 / 11.8, 15,138 tokens 29 against 36; bf16 within 0.3 us).  With more
    // of them throughput counts (8 bits, 4096 channels, 21,768 tokens: 142 us with 512 channels, 153 with 128).
    const bool narrow = pages * ((dkv + kPageChannels - 1) / kPageChannels) < 2048;
    const int ch = narrow ? 128 : kPageChannels;
    const int64_t bytes = 4ll * total_tokens * dkv;  // of the packed keys and values
    const dim3 grid(pages, (dkv + ch - 1) / ch);
    const bool some = bytes >= 16ll << 20, many = bytes >= 64ll << 20, most = bytes >= 256ll << 20;  // (see the kernel)
#define TDP_MOVE_(KV8, TO, CH, NTL, NTS)                                                                                           \
  kv_move_kernel<KV8, TO, CH, NTL, NTS><<<grid, 256, 0, s>>>((bf16*)k_packed, (bf16*)v_packed, kv, cu_seqlens, n_seqs, total_tokens, \
                                                             block_tables, max_pages_per_seq)
#define TDP_MOVE(KV8, TO, NTS) \
  do { if (narrow) TDP_MOVE_(KV8, TO, 128, false, NTS); else TDP_MOVE_(KV8, TO, kPageChannels, false, NTS); } while (0)
    // (2047 workgroups of 512 channels are less than 64 MiB)
    if (to_pages) {
      if (kv.fp8 && many) TDP_MOVE_(true, true, kPageChannels, true, false);
      else if (kv.fp8) TDP_MOVE(true, true, false);
      else if (many) TDP_MOVE_(false, true, kPageChannels, true, false);
      else if (some) TDP_MOVE(false, true, true);
      else TDP_MOVE(false, true, false);
    } else {
      if (kv.fp8 && some) TDP_MOVE(true, false, true);
      else if (kv.fp8) TDP_MOVE(true, false, false);
      else if (most) TDP_MOVE_(false, false, kPageChannels, true, true);
      else if (some) TDP_MOVE(false, false, true);
      else TDP_MOVE(false, false, false);
    }
#undef TDP_MOVE
#undef TDP_MOVE_
    return hipGetLastError();
  }
  kv_copy_kernel<<<total_tokens, 256, 0, s>>>(to_pages, (bf16*)k_packed, (bf16*)v_packed, kv, cu_seqlens,
                                              n_seqs, block_tables, max_pages_per_seq);
  return hipGetLastError();
}

// ------------------------------------------------------------------ weight repack (one-time)
// dst(row_of(n), k) = bf16(src[k][n]) through a 32x32 LDS transpose; dst is in the weight layout
// (layout_weights) with dst_ld columns.
__global__ __launch_bounds__(256) void repack_kernel(const void* __restrict__ src, int src_is_f32,
                                                     int64_t K, int64_t N, int64_t ld_src, bf16* __restrict__ dst,
                                                     OperandLayout lay, int64_t row_off, int mode) {
  __shared__ float tile[32][33];
  const int64_t k0 = (int64_t)blockIdx.y * 32, n0 = (int64_t)blockIdx.x * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
  for (int r = ty; r < 32; r += 8) {
    const int64_t k = k0 + r, n = n0 + tx;
    float v = 0.f;
    if (k < K && n < N)
      v = src_is_f32 ? ((const float*)src)[k * ld_src + n] : (float)((const bf16*)src)[k * ld_src + n];
    tile[r][tx] = v;
  }
  __syncthreads();
  for (int r = ty; r < 32; r += 8) {
    const int64_t n = n0 + r, k = k0 + tx;
    if (n < N && k < K) {
      int64_t row;
      if (mode == 0) row = row_off + n;
      else row = (n / 32) * 64 + (n % 32) + (mode == 2 ? 32 : 0);
      dst[operand_offset(lay, (int)row, (int)k)] = (bf16)tile[tx][r];
    }
  }
}

hipError_t launch_repack_ld(const void* src, int src_is_f32, int64_t rows_in, int64_t cols_out, int64_t ld_src,
                            void* dst, int64_t dst_ld, int64_t row_off, int mode, hipStream_t s) {
  dim3 grid((unsigned)((cols_out + 31) / 32), (unsigned)((rows_in + 31) / 32));
  repack_kernel<<<grid, 256, 0, s>>>(src, src_is_f32, rows_in, cols_out, ld_src, (bf16*)dst, layout_weights(dst_ld),
                                     row_off, mode);
  return hipGetLastError();
}

hipError_t launch_repack(const void* src, int src_is_f32, int64_t rows_in, int64_t cols_out, void* dst,
                         int64_t dst_ld, int64_t row_off, int mode, hipStream_t s) {
  return launch_repack_ld(src, src_is_f32, rows_in, cols_out, cols_out, dst, dst_ld, row_off, mode, s);
}

__global__ void convert_vec_kernel(const void* __restrict__ src, int src_is_f32, int64_t n,
                                   float* __restrict__ dst) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = src_is_f32 ? ((const float*)src)[i] : (float)((const bf16*)src)[i];
}

hipError_t launch_convert_vec(const void* src, int src_is_f32, int64_t n, float* dst, hipStream_t s) {
  convert_vec_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(src, src_is_f32, n, dst);
  return hipGetLastError();
}

// ---- optional validation of device-side tables ---------------------------------------------
// The stage calls trust the tables they are given; these kernels are what a caller runs first when
// it does not.  They read a table only at (row < n, entry < max_pages_per_seq), whatever the lengths
// say, so they are safe on any input.  res[0] counts violations, res[1] keeps the smallest
// row * 8 + kind among them.
enum TableFault { kFaultLength = 1, kFaultPage = 2, kFaultShared = 3, kFaultPrefix = 4 };

__device__ __forceinline__ void table_fault(int32_t* res, int row, int kind) {
  atomicAdd(&res[0], 1);
  atomicMin(&res[1], row * 8 + kind);
}

__global__ void table_check_init_kernel(int32_t* __restrict__ owner, int num_pages, int32_t* __restrict__ res) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < num_pages) owner[i] = -1;
  if (i == 0) {
    res[0] = 0;
    res[1] = 0x7fffffff;
  }
}

// tokens of row r after the call (decode: ctx + 1; prefill: the prompt's length), or -1 if the
// length itself is invalid
__device__ __forceinline__ int table_row_tokens(int decode, const int32_t* lens, int r, int max_pos) {
  const int64_t n = decode ? (int64_t)lens[r] + 1 : (int64_t)lens[r + 1] - (int64_t)lens[r];
  const int64_t lo = decode ? 1 : 0;
  return (n < lo || n > max_pos) ? -1 : (int)n;
}

// pass 1: lengths, page ranges, and every page the call will WRITE is claimed by its row
// (decode: the page of position ctx; prefill: every page of the prompt)
__global__ __launch_bounds__(64) void table_check_claim_kernel(int decode, const int32_t* __restrict__ lens,
                                                               const int32_t* __restrict__ tables, int n_rows,
                                                               int max_pages_per_seq, int num_pages, int total_tokens,
                                                               int32_t* __restrict__ owner, int32_t* __restrict__ res) {
  const int r = blockIdx.x;
  if (!decode && r == 0 && threadIdx.x == 0) {
    if (lens[0] != 0) table_fault(res, 0, kFaultPrefix);
    if (lens[n_rows] != total_tokens) table_fault(res, n_rows - 1, kFaultPrefix);
  }
  const int n = table_row_tokens(decode, lens, r, max_pages_per_seq * 16);
  if (n < 0) {
    if (threadIdx.x == 0) table_fault(res, r, kFaultLength);
    return;
  }
  const int n_pages = (n + 15) / 16;
  for (int j = threadIdx.x; j < n_pages; j += 64) {
    const int p = tables[(int64_t)r * max_pages_per_seq + j];
    if (p < 0 || p >= num_pages) {
      table_fault(res, r, kFaultPage);
      continue;
    }
    if (!decode || j == n_pages - 1) {
      if (atomicCAS(&owner[p], -1, r) != -1) table_fault(res, r, kFaultShared);
    }
  }
}

// pass 2 (decode): no page that a row only reads is written by any row of the batch
__global__ __launch_bounds__(64) void table_check_read_kernel(const int32_t* __restrict__ lens,
                                                              const int32_t* __restrict__ tables,
                                                              int max_pages_per_seq, int num_pages,
                                                              const int32_t* __restrict__ owner,
                                                              int32_t* __restrict__ res) {
  const int r = blockIdx.x;
  const int n = table_row_tokens(1, lens, r, max_pages_per_seq * 16);
  if (n < 0) return;
  const int n_pages = (n + 15) / 16;
  for (int j = threadIdx.x; j < n_pages - 1; j += 64) {
    const int p = tables[(int64_t)r * max_pages_per_seq + j];
    if (p >= 0 && p < num_pages && owner[p] != -1) table_fault(res, r, kFaultShared);
  }
}

hipError_t launch_table_check(int decode, const int32_t* lens, const int32_t* tables, int n_rows,
                              int max_pages_per_seq, int num_pages, int total_tokens, int32_t* owner, int32_t* res,
                              hipStream_t s) {
  table_check_init_kernel<<<(num_pages + 255) / 256, 256, 0, s>>>(owner, num_pages, res);
  table_check_claim_kernel<<<n_rows, 64, 0, s>>>(decode, lens, tables, n_rows, max_pages_per_seq, num_pages,
                                                 total_tokens, owner, res);
  if (decode)
    table_check_read_kernel<<<n_rows, 64, 0, s>>>(lens, tables, max_pages_per_seq, num_pages, owner, res);
  return hipGetLastError();
}

// ---- pipeline ends: row gather (token embedding; last-token selection), bf16 conversion, argmax ----

// dst[m][:] = src[idx[m]][:]; one workgroup per row, 16-byte pieces.  An index outside
// [0, n_src_rows) is clamped into range, so a bad id can never read outside the table.
__global__ __launch_bounds__(256) void gather_rows_kernel(const bf16* __restrict__ src, int64_t ld_src,
                                                          int64_t n_src_rows, const int32_t* __restrict__ idx,
                                                          int d, bf16* __restrict__ dst, int64_t ld_dst) {
  const int m = blockIdx.x;
  int64_t r = idx[m];
  r = r < 0 ? 0 : (r >= n_src_rows ? n_src_rows - 1 : r);
  const bf16* sp = src + r * ld_src;
  bf16* dp = dst + (int64_t)m * ld_dst;
  for (int c = threadIdx.x * 8; c < d; c += 256 * 8) st_bf16x8(dp + c, ld_bf16x8(sp + c));
}

hipError_t launch_gather_rows(const void* src, int64_t ld_src, int64_t n_src_rows, const int32_t* idx, int M, int d,
                              void* dst, int64_t ld_dst, hipStream_t s) {
  if (M <= 0) return hipSuccess;
  gather_rows_kernel<<<M, 256, 0, s>>>((const bf16*)src, ld_src, n_src_rows, idx, d, (bf16*)dst, ld_dst);
  return hipGetLastError();
}

__global__ void to_bf16_kernel(const void* __restrict__ src, int src_is_f32, int64_t n, bf16* __restrict__ dst) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = src_is_f32 ? (bf16)((const float*)src)[i] : ((const bf16*)src)[i];
}

hipError_t launch_to_bf16(const void* src, int src_is_f32, int64_t n, void* dst, hipStream_t s) {
  to_bf16_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(src, src_is_f32, n, (bf16*)dst);
  return hipGetLastError();
}

// out[m] = the lowest index among the largest of logits[m][0 .. n).  One workgroup per row.  NaNs
// never win a comparison; a row of NaNs gives 0.  The rule "greater, or equal at a lower index" does not depend on the
// order of comparisons, so a thread may have many loads in flight: up to 8 x 16 bytes per turn, with 1024 threads a row of
// 32000 in one (a row is aligned by its first up to three elements).  Bound: the latency of a row's first bytes for a few rows,
// reading the logits for many.  With 256 threads that load and compare one element per turn a launch took 42 us for 48
// rows of 32000 and 46 us for 512; like this 7 and 14.
template <int THREADS>
__global__ __launch_bounds__(THREADS) void argmax_rows_kernel(const float* __restrict__ logits, int64_t ld, int n,
                                                              int32_t* __restrict__ out) {
  constexpr int UN = 8, WAVES = THREADS / 64;
  constexpr bool SHORT = THREADS < 1024;
  __shared__ Best s_best[WAVES];
  const float* row = logits + (int64_t)blockIdx.x * ld;
  const int tid = threadIdx.x;
  Best best = no_best();
  const int head = min(n, (int)((16 - ((uintptr_t)row & 15)) & 15) / 4);
  const int n4 = (n - head) / 4, tail = head + n4 * 4;
  const f32x4* body = reinterpret_cast<const f32x4*>(row + head);
  if (tid < head) take_best(best, row[tid], tid);
  if (tid < n - tail) take_best(best, row[tail + tid], tail + tid);
  for (int j0 = 0; j0 < n4; j0 += THREADS * UN) {
    f32x4 v[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u)  // (past the end: the last piece again; short rows have fewer than UN pieces per thread)
      if (!SHORT || j0 + u * THREADS < n4) v[u] = body[min(j0 + u * THREADS + tid, n4 - 1)];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      if (SHORT && j0 + u * THREADS >= n4) break;
      const int at = head + 4 * min(j0 + u * THREADS + tid, n4 - 1);
#pragma unroll
      for (int e = 0; e < 4; ++e) take_best(best, v[u][e], at + e);
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) take_best_of_lane(best, o);
  if ((tid & 63) == 0) s_best[tid >> 6] = best;
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < WAVES; ++w) take_best(best, s_best[w].value, s_best[w].index);
    out[blockIdx.x] = best.index == kNoIndex ? 0 : best.index;
  }
}

// The same with the largest element of every piece of `width` columns known (GemmArgs::row_max): a wave per row takes the first of
// the pieces with the largest one, up to eight per lane in flight, and finds it there.
__global__ __launch_bounds__(256) void argmax_pieces_kernel(const float* __restrict__ row_max, int count, int width,
                                                            const float* __restrict__ logits, int64_t ld, int n, int M,
                                                            int32_t* __restrict__ out) {
  constexpr int UN = 8;
  const int m = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (m >= M) return;
  const float* maxima = row_max + (int64_t)m * count;
  const float* row = logits + (int64_t)m * ld;
  Best piece = no_best();
  for (int i0 = 0; i0 < count; i0 += 64 * UN) {
    float v[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u)
      if (i0 + u * 64 < count) v[u] = maxima[min(i0 + u * 64 + lane, count - 1)];
#pragma unroll
    for (int u = 0; u < UN; ++u)
      if (i0 + u * 64 < count) take_best(piece, v[u], min(i0 + u * 64 + lane, count - 1));
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) take_best_of_lane(piece, o);
  // (a largest element of minus infinity can be that of a piece of NaN: all of the row is looked through)
  const bool known = piece.value > -INFINITY;
  const int begin = known ? piece.index * width : 0, end = known ? min(begin + width, n) : n;
  Best best = no_best();
  for (int i = begin + lane; i < end; i += 64) take_best(best, row[i], i);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) take_best_of_lane(best, o);
  if (lane == 0) out[m] = best.index == kNoIndex ? 0 : best.index;
}

hipError_t launch_argmax_pieces(const float* row_max, int count, int width, const float* logits, int64_t ld, int M, int n,
                                int32_t* out, hipStream_t s) {
  if (M <= 0) return hipSuccess;
  argmax_pieces_kernel<<<(M + 3) / 4, 256, 0, s>>>(row_max, count, width, logits, ld, n, M, out);
  return hipGetLastError();
}

hipError_t launch_argmax_rows(const float* logits, int64_t ld, int M, int n, int32_t* out, hipStream_t s) {
  if (M <= 0) return hipSuccess;
  // As many threads as the row keeps busy: more of them only lengthen the workgroup's start and its last step, and on short rows
  // the loads past the end (a row of 1000: 2.7 us with 128 threads, 3.8 with 1024, 5.9 with 1024 that all load eight
  // pieces; 512 rows 3.2 / 5.5 / 9.0; a row of 4000 3.3 with 256 / 3.8 / 5.9; of 16000 4.8 with 512, 5.0 with 1024).  From
  // 20000 on all eight pieces are there and are loaded without asking (32000: 5.9 us against 6.5).
#define TDP_ARGMAX(THREADS) argmax_rows_kernel<THREADS><<<M, THREADS, 0, s>>>(logits, ld, n, out)
  if (n <= 512) TDP_ARGMAX(64);
  else if (n <= 2048) TDP_ARGMAX(128);
  else if (n <= 5000) TDP_ARGMAX(256);
  else if (n < 20000) TDP_ARGMAX(512);
  else TDP_ARGMAX(1024);
#undef TDP_ARGMAX
  return hipGetLastError();
}

}  // namespace tdp
