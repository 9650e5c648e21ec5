// Attention kernels of the stage: paged GQA decode attention (split over the KV range, then
// merged) and var-len causal prefill attention.  Both read K and V through the block tables.
//
// Decode (paper Sec. 2.1): each request contributes one query token that attends to its whole
// cache, so the kernel streams K/V once from HBM and is bandwidth bound.  The query heads that
// share a K/V head (GQA, Sec. 4.1) form the 16-wide "N" side of a 16x16x32 MFMA, so every K/V
// byte is loaded once per group and goes from global memory straight into MFMA operand
// registers: no LDS and no cross-lane transposes.
//
// The trick that avoids transposing the probabilities: scores are formed transposed,
// S^T[token][q] = K[token][:] . Q[q][:], and the rows of each MFMA tile are assigned to tokens in
// the order that makes a lane's accumulator elements the 8 consecutive tokens it must supply as
// the "B" operand of O^T[channel][q] += V^T[channel][token] P^T[token][q].
#include "tdp_device.h"
#include "tdp_kernels.h"

namespace tdp {

// Floats past the caches of an XCD, for workgroups of other XCDs in the same launch.
__device__ __forceinline__ void store_agent(float* p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 load_agent2(const float* p) {  // (8-byte aligned)
  return __builtin_bit_cast(float2, __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_AGENT));
}

constexpr float kNegBig = -1.0e30f;  // finite stand-in for -inf: exp2 gives exactly 0, no inf-inf

// =====================================================================================
// Decode.  Work item = (request, span of span_len tokens of its context); one workgroup
// of four waves per (item, kv head).  The four waves split the span's 32-token blocks evenly and
// merge their partial softmax states through LDS; a request whose context fits one span is
// finished there (no partials in HBM), longer ones leave one partial per span, which the workgroup
// that finishes last combines.  The item list is compact (built once per decode step by attn_plan_kernel), so the grid
// holds no workgroup that finds nothing to do except at its very end.
// Keys and values are requested as non-temporal: a launch reads each of them exactly once, and as
// ordinary loads they evict everything else from L2 on their way through (measured: 5.9 TB/s against
// 5.5 at batch 512, 5.7 against 5.2 at batch 256).
// =====================================================================================

// items[i] = (request, span index, tokens to attend to = ctx + 1, 0) for every span of the batch, and
// (-1, ...) for the rest of the list up to max_items, so a workgroup learns everything about its
// work - or that it has none - from one 16-byte record.  item_pages[i][j] = physical page of the j-th
// 16-token page of item i's span (span_len / 16 entries), entries past the request's last page clamped to
// it: with this list a decode workgroup needs no look-up that depends on another look-up before its
// first K/V load.  Longest work first: all full spans, then the requests' last (partial) spans by sixteenth
// of span_len, longest sixteenth first, so the workgroups that run at the end of the launch are short
// (with quarters the launch ended on workgroups of up to a quarter span in random order); in order of the
// requests within a class.
// Bound: a chain of look-ups and barriers.  Every workgroup counts the whole batch (thread t the t-th part of it) and
// scans the counts a wave per class, then each of its four waves writes the items and pages of one request: one launch
// instead of one workgroup that scanned 256 counts in turn and a second launch that copied the pages of its list
// (16 / 200 / 512 requests: 9.6 / 11.2 / 11.9 us together, now 5.6 / 6.9 / 7.6).
// A length that its block-table row cannot hold is brought into the row's range (decode_position, also in the rotation), so
// that the list never outgrows its buffer and the grid: every span counted here is made, and spans_done ends at zero,
// whatever ctx_lens holds.
__global__ __launch_bounds__(256) void attn_plan_kernel(const int32_t* __restrict__ ctx_lens, int batch, int span_len,
                                                        const int32_t* __restrict__ block_tables,
                                                        int max_pages_per_seq, int4* __restrict__ items, int max_items,
                                                        int32_t* __restrict__ item_pages) {
  constexpr int NP = 16;      // parts of a span
  constexpr int NB = NP + 1;  // class 0: full spans; 1..NP: last span with > (NP-c)/NP of span_len
  __shared__ __attribute__((aligned(16))) int part[NB][256];  // counts of (class, thread); then how many items of the class lie in front
  __shared__ int class_total[NB];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int per = (batch + 255) / 256;
  const int piece = span_len / NP;
  auto last_class = [&](int n_total, int n) {  // tokens in the last span: 1 .. span_len
    const int rem = n_total - (n - 1) * span_len;
    return NP - min((rem - 1) / piece, NP - 1);
  };
#pragma unroll
  for (int c = 0; c < NB; ++c) part[c][tid] = 0;
  for (int b = tid * per; b < min((tid + 1) * per, batch); ++b) {
    const int n_total = decode_position(ctx_lens[b], max_pages_per_seq) + 1;
    const int n = (n_total + span_len - 1) / span_len;
    part[0][tid] += n - 1;
    part[last_class(n_total, n)][tid] += 1;
  }
  __syncthreads();
  for (int c = wave; c < NB; c += 4) {  // exclusive prefix over the threads, four counts per lane
    int4 v = *reinterpret_cast<const int4*>(&part[c][lane * 4]);
    const int own = v.x + v.y + v.z + v.w;
    int incl = own;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int up = __shfl_up(incl, o, 64);
      if (lane >= o) incl += up;
    }
    const int before = incl - own;
    *reinterpret_cast<int4*>(&part[c][lane * 4]) = make_int4(before, before + v.x, before + v.x + v.y, before + v.x + v.y + v.z);
    if (lane == 63) class_total[c] = incl;
  }
  __syncthreads();
  int class_base[NB];
  int total = 0;
#pragma unroll
  for (int c = 0; c < NB; ++c) {
    class_base[c] = total;
    total += class_total[c];
  }
  for (int i = total + blockIdx.x * 256 + tid; i < max_items; i += gridDim.x * 256) items[i] = make_int4(-1, 0, 0, 0);
  const int b = blockIdx.x * 4 + wave;  // this wave's request
  if (b >= batch) return;
  const int own = b / per;              // the thread that counted it
  const int n_total = decode_position(ctx_lens[b], max_pages_per_seq) + 1;
  const int n = (n_total + span_len - 1) / span_len;
  const int cl = last_class(n_total, n);
  int full_at = part[0][own], last_at = part[cl][own];
#pragma unroll
  for (int c = 1; c < NB; ++c) last_at += c == cl ? class_base[c] : 0;
  for (int b2 = own * per; b2 < b; ++b2) {  // requests of the same thread in front of this one
    const int t2 = decode_position(ctx_lens[b2], max_pages_per_seq) + 1, n2 = (t2 + span_len - 1) / span_len;
    full_at += n2 - 1;
    last_at += last_class(t2, n2) == cl ? 1 : 0;
  }
  const int pages_per_span = span_len >> 4, last_page = (n_total - 1) / 16;
  auto at = [&](int k) { return k < n - 1 ? full_at + k : last_at; };
  for (int k = lane; k < n; k += 64) items[at(k)] = make_int4(b, k, n_total, 0);
  constexpr int UN = 4;
  for (int e0 = 0; e0 < n * pages_per_span; e0 += 64 * UN) {  // entry e is page e % pages_per_span of span e / pages_per_span
    int page[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u)
      page[u] = block_tables[(int64_t)b * max_pages_per_seq + min(e0 + u * 64 + lane, last_page)];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int e = e0 + u * 64 + lane;
      if (e < n * pages_per_span)
        item_pages[(int64_t)at(e / pages_per_span) * pages_per_span + e % pages_per_span] = page[u];
    }
  }
}

// ROTATE: the workgroup makes its queries itself, and that of a request's last span appends the new token's key and value, both from
// the fp32 projection (its finished output, or its split-K partials, summed in split order, plus the bias), rounded once, as
// rope_kv_kernel does; see attn_decode_rotates for when.  Three waves rotate the queries into LDS, a thread four pairs of
// channels, while the fourth appends: the one that reads the new token's page, later in its range and behind its own stores.
//
// KV8 = the pools hold E4M3 codes (one byte per element) instead of bf16.  A 16-byte load then carries
// 16 elements, which become two MFMA operands after conversion, so the block grows to 64 tokens
// (four pages) and the assignment of MFMA k-indices to channels (scores) and of score rows to
// tokens changes with it; the arithmetic after the conversion is the bf16 kernel's.  The cache
// scales ride along for free: k_scale in the softmax scale, v_scale in the final division.
template <int DH, bool KV8, bool ROTATE>
__global__ __launch_bounds__(256, 3) void attn_decode_kernel(const DecodeQueries dq, int batch,
                                                          int n_q_heads, KvLayout kv,
                                                          const int4* __restrict__ items,
                                                          const int32_t* __restrict__ item_pages, int item_pitch,
                                                          const int32_t* __restrict__ ctx_lens,
                                                          float* __restrict__ part_o, float* __restrict__ part_ml,
                                                          unsigned* __restrict__ spans_done, int max_spans,
                                                          int span_len, bf16* __restrict__ out,
                                                          OperandLayout out_lay, float scale_log2, float out_scale) {
  constexpr int KS = DH / 32;          // k-steps of the score MFMA
  constexpr int DT = DH / 16;          // 16-channel tiles of the output
  constexpr int BT = KV8 ? 64 : 32;    // tokens per block
  constexpr int NT = BT / 16;          // score tiles per block
  constexpr int NP = BT / 32;          // k-steps of the output MFMA per block
  constexpr int LT = BT / 4;           // consecutive tokens of a block whose scores end up in one lane
  const int Hkv = kv.n_kv_heads;
  const int item = blockIdx.x / Hkv, kvh = blockIdx.x % Hkv;
  // the two look-ups a workgroup starts with are independent of each other: its work record and
  // its span's page list (lane j holds pages j, 64 + j, ...; at most 256 pages per span)
  const int pages_per_span = span_len >> 4;
  const int lane = threadIdx.x & 63;
  const int wave = ROTATE ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : threadIdx.x >> 6;
  int my_pages[4];
#pragma unroll
  for (int j = 0; j < 4; ++j)
    my_pages[j] = item_pages[(int64_t)item * item_pitch + min(lane + 64 * j, item_pitch - 1)];
  // without a work list (see attn_decode_planned) item b is the whole context of request b and its pages are the block table's
  // row, whose entries behind the request's last page are not page ids and are not used
  const int4 it = items ? items[item] : make_int4(item, 0, decode_position(ctx_lens[item], item_pitch) + 1, 0);
  if (it.x < 0) return;
  const int b = it.x, span = it.y;
  const int n_total = it.z;  // ctx + 1: with the new token
  const int last_entry = items ? pages_per_span - 1 : (n_total - 1) >> 4;
  const int s_begin = span * span_len;
  const int s_end = min(s_begin + span_len, n_total);
  const int G = n_q_heads / Hkv;
  const int r16 = lane & 15, kg = lane >> 4;
  const bf16* kpool = (const bf16*)kv.k_pool;
  const bf16* vpool = (const bf16*)kv.v_pool;
  const uint8_t* kpool8 = (const uint8_t*)kv.k_pool;
  const uint8_t* vpool8 = (const uint8_t*)kv.v_pool;
  // this wave's share of the span, in whole blocks
  const int n_blocks = (s_end - s_begin + BT - 1) / BT;
  const int t_begin = s_begin + BT * ((wave * n_blocks) >> 2);
  const int t_end = min(s_begin + BT * (((wave + 1) * n_blocks) >> 2), s_end);

  __shared__ __attribute__((aligned(16))) bf16 s_q[ROTATE ? 16 : 1][DH + 8];
  if constexpr (ROTATE) {
    auto page_of = [&](int i) {  // i is wave-uniform
      const int r = i >> 6;
      return __builtin_amdgcn_readlane(r == 0 ? my_pages[0] : r == 1 ? my_pages[1] : r == 2 ? my_pages[2] : my_pages[3], i & 63);
    };
    constexpr int KU = DH / 8, VU = DH / 4, ZN = 8;  // units of a head: four pairs, four values; splits asked for at once
    static_assert(KU + VU <= 64, "one wave appends");
    const bool owner = s_end == n_total;  // of the new token
    // a unit's columns of the projection: four pairs (col0 + i, col1 + i) of the channels c0 + i, c0 + i + DH / 2 of a head, or four
    // values col0 + i
    struct Unit {
      int c0, col0, col1;
      f32x4 part[ZN][2], bias[2];
      float4 cs[2];
    } unit;
    const float* const row = dq.proj + (int64_t)b * dq.ld;
    const int64_t split_stride = (int64_t)batch * dq.ld;
    const int pos = n_total - 1;
    auto fetch = [&](int head, int index, int distance) {
      unit.c0 = index * 4;
      unit.col0 = head * DH + unit.c0;
      unit.col1 = unit.col0 + distance;
  #pragma unroll
      for (int z = 0; z < ZN; ++z) {
        if (z < dq.splits) {
          unit.part[z][0] = *reinterpret_cast<const f32x4*>(row + z * split_stride + unit.col0);
          unit.part[z][1] = *reinterpret_cast<const f32x4*>(row + z * split_stride + unit.col1);
        } else {
          unit.part[z][0] = unit.part[z][1] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
      }
      const float4* cs = reinterpret_cast<const float4*>(dq.rope_table + (int64_t)pos * (DH / 2) + unit.c0 % (DH / 2));
      unit.cs[0] = cs[0];
      unit.cs[1] = cs[1];
      if (dq.bias) {
        unit.bias[0] = *reinterpret_cast<const f32x4*>(dq.bias + unit.col0);
        unit.bias[1] = *reinterpret_cast<const f32x4*>(dq.bias + unit.col1);
      }
    };
    auto sums = [&](f32x4 (&f)[2]) {
      f[0] = f[1] = f32x4{0.f, 0.f, 0.f, 0.f};
  #pragma unroll
      for (int z = 0; z < ZN; ++z)
  #pragma unroll
        for (int c = 0; c < 2; ++c) f[c] += unit.part[z][c];
      for (int z = ZN; z < dq.splits; ++z) {
        f[0] += *reinterpret_cast<const f32x4*>(row + z * split_stride + unit.col0);
        f[1] += *reinterpret_cast<const f32x4*>(row + z * split_stride + unit.col1);
      }
      if (dq.bias) {
        f[0] += unit.bias[0];
        f[1] += unit.bias[1];
      }
    };
    auto rotated = [&](float (&lo)[4], float (&hi)[4]) {
      f32x4 ab[2];
      sums(ab);
      const float2 t2[4] = {{unit.cs[0].x, unit.cs[0].y}, {unit.cs[0].z, unit.cs[0].w},
                            {unit.cs[1].x, unit.cs[1].y}, {unit.cs[1].z, unit.cs[1].w}};
  #pragma unroll
      for (int i = 0; i < 4; ++i) rotate_pair(ab[0][i], ab[1][i], t2[i], unit.c0 + i, lo[i], hi[i]);
    };
    auto four = [](const float (&f)[4]) {
      bf16x4 r;
  #pragma unroll
      for (int i = 0; i < 4; ++i) r[i] = (bf16)f[i];
      return r;
    };
    auto codes4 = [](const float (&f)[4], float scale) -> uint32_t {
      uint32_t c = 0u;
  #pragma unroll
      for (int i = 0; i < 4; ++i) c |= f32_to_e4m3(f[i] / scale) << (8 * i);
      return c;
    };
    if (wave < 3) {
      if ((int)threadIdx.x < G * KU) fetch(kvh * G + threadIdx.x / KU, threadIdx.x % KU, DH / 2);
    } else if (owner) {
      if (lane < KU) fetch(n_q_heads + kvh, lane, DH / 2);
      else if (lane < KU + VU) fetch(n_q_heads + Hkv + kvh, lane - KU, 0);
    }

    if (wave < 3) {
      for (int i = threadIdx.x; i < G * KU; i += 192) {
        if (i != (int)threadIdx.x) fetch(kvh * G + i / KU, i % KU, DH / 2);  // (more than twelve heads)
        float lo[4], hi[4];
        rotated(lo, hi);
        *reinterpret_cast<bf16x4*>(&s_q[i / KU][unit.c0]) = four(lo);
        *reinterpret_cast<bf16x4*>(&s_q[i / KU][DH / 2 + unit.c0]) = four(hi);
      }
    } else if (owner) {
      const int64_t page = page_of((pos >> 4) - (s_begin >> 4));
      const int slot = pos & 15;
      if (lane < KU) {
        float lo[4], hi[4];
        rotated(lo, hi);
        constexpr int ESZ = KV8 ? 1 : 2;
        uint8_t* k_lo = (uint8_t*)kv.k_pool + k_pool_byte(kv, page, kvh, slot, unit.c0 * ESZ);
        uint8_t* k_hi = (uint8_t*)kv.k_pool + k_pool_byte(kv, page, kvh, slot, (DH / 2 + unit.c0) * ESZ);
        if constexpr (KV8) {  // from fp32 straight to the code: one rounding
          *reinterpret_cast<uint32_t*>(k_lo) = codes4(lo, kv.k_scale);
          *reinterpret_cast<uint32_t*>(k_hi) = codes4(hi, kv.k_scale);
        } else {
          *reinterpret_cast<bf16x4*>(k_lo) = four(lo);
          *reinterpret_cast<bf16x4*>(k_hi) = four(hi);
        }
      } else if (lane < KU + VU) {
        f32x4 f[2];
        sums(f);
        const int64_t at = ((page * Hkv + kvh) * DH + unit.c0) * 16 + slot;  // [page][kv head][channel][16 slots]
  #pragma unroll
        for (int i = 0; i < 4; ++i) {
          // the value is a bf16 quantity in both forms of the cache (the 8-bit code is taken from it)
          const bf16 x = (bf16)f[0][i];
          if constexpr (KV8)
            ((uint8_t*)kv.v_pool)[at + i * 16] = (uint8_t)f32_to_e4m3((float)x / kv.v_scale);
          else
            ((bf16*)kv.v_pool)[at + i * 16] = x;
        }
      }
      // (read back by other lanes of this wave, whose memory operations are carried out in order)
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    __syncthreads();
  }

  // Query fragments.  bf16 pools: k-step kk covers channels kk*32 + kg*8 .. +8.  8-bit pools: a
  // lane's 16-byte key load covers channels ld*64 + kg*16 .. +16, whose halves feed k-steps 2 ld and
  // 2 ld + 1, so the query is gathered in that order.
  bf16x8 qf[KS];
  {
    const bf16* qp = ROTATE ? &s_q[r16][0] : (const bf16*)dq.qkv + (int64_t)b * dq.ld + (int64_t)(kvh * G + (r16 < G ? r16 : 0)) * DH;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      const int ch = KV8 ? (kk >> 1) * 64 + kg * 16 + (kk & 1) * 8 : kk * 32 + kg * 8;
      qf[kk] = r16 < G ? ld_bf16x8(qp + ch) : zero_bf16x8();
    }
  }
  f32x4 o[DT];
#pragma unroll
  for (int d = 0; d < DT; ++d) o[d] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = kNegBig, lsum = 0.f;

  if (t_begin < t_end) {
    // token (within its block) of this lane's row in score tile t: (r16/4)*LT + t*4 + r16%4; the
    // lane's own accumulator elements are then tokens kg*LT + t*4 + i, i.e. LT consecutive tokens
    const int krow0 = (r16 >> 2) * LT + (r16 & 3);
    // The span's page ids sit one per lane; the loop reads them with v_readlane, so no table load
    // sits between two blocks.  Entries past the request's last page were clamped to it by the
    // planner; pages of a span's last block that lie past the span are clamped to its last entry here.
    const int page_base = s_begin >> 4;

    // One block = the K fragments of NT score tiles and the V^T fragments of all channel tiles, 8 KiB
    // each per wave (head_dim 128).  K is fetched one block ahead into one of two register sets; V of
    // a block is fetched into a single set at the start of the block's own turn and is consumed
    // at its end, behind the score MFMAs and the softmax.  Per wave 16 KiB are in flight, and the
    // kernel fits three workgroups per CU (with both halves double-buffered it needed 198
    // registers, two workgroups per CU).  Measured: the same time either way (0.46-0.49 ms per
    // launch at batch 512, the spread coming from where the pools happen to lie in memory).
    struct KBlock {
      bf16x8 kf[2][KS];  // bf16 pools: [score tile][k-step]; 8-bit pools: 16 raw bytes per entry, [t / 2][(t % 2) * KS/2 + ld]
    };
    struct VBlock {
      bf16x8 vf[DT];     // bf16 pools: 8 tokens of a channel; 8-bit pools: 16 raw bytes = 16 tokens of a channel
    };
    auto page_of = [&](int i) -> int64_t {  // i is wave-uniform
      const int r = i >> 6;
      const int v = r == 0 ? my_pages[0] : r == 1 ? my_pages[1] : r == 2 ? my_pages[2] : my_pages[3];
      return __builtin_amdgcn_readlane(v, i & 63);
    };
    auto load_k = [&](int tb, KBlock& blk) {
      const int pi = (tb >> 4) - page_base;
      int64_t page[BT / 16];
#pragma unroll
      for (int j = 0; j < BT / 16; ++j) page[j] = page_of(min(pi + j, last_entry));
      if constexpr (KV8) {
        // score tile t, row r16 -> token (r16/4)*16 + t*4 + r16%4: page r16/4 of the block, slot t*4 + r16%4
        const int64_t kpage = (r16 >> 2) == 0 ? page[0] : (r16 >> 2) == 1 ? page[1] : (r16 >> 2) == 2 ? page[2] : page[3];
        // (K pool: 64-byte pieces of the 16 token rows of a page lie together, piece l at l * 1024)
        const uint8_t* kp = kpool8 + (kpage * Hkv + kvh) * (16 * DH) + (r16 & 3) * 64 + kg * 16;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int l = 0; l < KS / 2; ++l)
            blk.kf[t >> 1][(t & 1) * (KS / 2) + l] = ld_bf16x8_nt(reinterpret_cast<const bf16*>(kp + (t * 4) * 64 + l * 1024));
      } else {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const int tok = krow0 + t * 4;
          // (K pool: the 32 channels of k-step kk are one 64-byte piece; piece kk of the page's 16 tokens is
          // contiguous, so the 16 rows x 64 bytes of one instruction are four runs of 256 bytes)
          const bf16* kp = kpool + (page[tok >> 4 & 1] * Hkv + kvh) * (16 * DH) + (tok & 15) * 32 + kg * 8;
#pragma unroll
          for (int kk = 0; kk < KS; ++kk) blk.kf[t][kk] = ld_bf16x8_nt(kp + kk * (16 * 32));
        }
      }
    };
    auto load_v = [&](int tb, VBlock& blk) {
      const int pi = (tb >> 4) - page_base;
      int64_t page[BT / 16];  // the look-up index must be wave-uniform: all pages first, then the lane's pick
#pragma unroll
      for (int j = 0; j < BT / 16; ++j) page[j] = page_of(min(pi + j, last_entry));
      if constexpr (KV8) {
        // channel r16 of tile d, the 16 tokens of page kg of the block
        const int64_t vpage = kg == 0 ? page[0] : kg == 1 ? page[1] : kg == 2 ? page[2] : page[3];
        const uint8_t* vp = vpool8 + ((vpage * Hkv + kvh) * DH + r16) * 16;
#pragma unroll
        for (int d = 0; d < DT; ++d) blk.vf[d] = ld_bf16x8_nt(reinterpret_cast<const bf16*>(vp + d * 16 * 16));
      } else {
        const int64_t vpage = kg < 2 ? page[0] : page[1];
        const bf16* vp = vpool + ((vpage * Hkv + kvh) * DH + r16) * 16 + (kg & 1) * 8;
#pragma unroll
        for (int d = 0; d < DT; ++d) blk.vf[d] = ld_bf16x8_nt(vp + d * 16 * 16);
      }
    };
    auto compute_block = [&](int tb, KBlock& blk, VBlock& vblk) {
      f32x4 s[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        s[t] = f32x4{0.f, 0.f, 0.f, 0.f};
        if constexpr (KV8) {
#pragma unroll
          for (int l = 0; l < KS / 2; ++l) {
            bf16x8 k0, k1;
            e4m3x16_to_bf16x8x2(__builtin_bit_cast(uint4, blk.kf[t >> 1][(t & 1) * (KS / 2) + l]), k0, k1);
            s[t] = mfma16(k0, qf[2 * l], s[t]);
            s[t] = mfma16(k1, qf[2 * l + 1], s[t]);
          }
        } else {
#pragma unroll
          for (int kk = 0; kk < KS; ++kk) s[t] = mfma16(blk.kf[t][kk], qf[kk], s[t]);
        }
      }
      // lane holds tokens tb + kg*LT + t*4 + i of column q = r16
      const int tok_base = tb + kg * LT;
      float mx = kNegBig;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float v = (tok_base + t * 4 + i < n_total) ? s[t][i] * scale_log2 : kNegBig;
          s[t][i] = v;
          mx = fmaxf(mx, v);
        }
      mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      const float m_new = fmaxf(m, mx);
      const float alpha = exp2f(m - m_new);
      bf16x8 pb[NP];
      float psum = 0.f;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float pv = exp2f(s[t][i] - m_new);
          psum += pv;
          pb[t >> 1][(t & 1) * 4 + i] = (bf16)pv;
        }
      lsum = lsum * alpha + psum;
      m = m_new;
      const bool tail = tb + BT > n_total;  // slots past the context may hold anything, even NaN
#pragma unroll
      for (int d = 0; d < DT; ++d) {
        o[d] *= alpha;
        if constexpr (KV8) {
          uint4 raw = __builtin_bit_cast(uint4, vblk.vf[d]);
          if (tail) {  // keep the first n_total - tok_base bytes (tokens tok_base .. tok_base + 15)
            const int keep = min(max(n_total - tok_base, 0), 16);
            auto mask = [&](int w) -> uint32_t {
              const int k4 = min(max(keep - 4 * w, 0), 4);
              return k4 == 4 ? 0xffffffffu : (1u << (8 * k4)) - 1u;
            };
            raw.x &= mask(0);
            raw.y &= mask(1);
            raw.z &= mask(2);
            raw.w &= mask(3);
          }
          bf16x8 v0, v1;
          e4m3x16_to_bf16x8x2(raw, v0, v1);
          o[d] = mfma16(v0, pb[0], o[d]);
          o[d] = mfma16(v1, pb[NP - 1], o[d]);
        } else {
          if (tail) {
#pragma unroll
            for (int j = 0; j < 8; ++j)
              if (tok_base + j >= n_total) vblk.vf[d][j] = (bf16)0.0f;
          }
          o[d] = mfma16(vblk.vf[d], pb[0], o[d]);
        }
      }
    };

    // Two blocks per trip, K ping-pongs between two register sets.  Every block is loaded exactly
    // once: the steady-state loop only runs while two more blocks follow (its loads are
    // unconditional, so the compiler's wait counts stay exact), the last one or two blocks are
    // peeled off.
    KBlock k0, k1;
    VBlock v;
    int tb = t_begin;
    load_k(tb, k0);
    for (; tb + 2 * BT < t_end; tb += 2 * BT) {
      load_v(tb, v);
      load_k(tb + BT, k1);
      compute_block(tb, k0, v);
      load_v(tb + BT, v);
      load_k(tb + 2 * BT, k0);
      compute_block(tb + BT, k1, v);
    }
    if (tb + BT < t_end) {
      load_v(tb, v);
      load_k(tb + BT, k1);
      compute_block(tb, k0, v);
      load_v(tb + BT, v);
      compute_block(tb + BT, k1, v);
    } else {
      load_v(tb, v);
      compute_block(tb, k0, v);
    }
    lsum += __shfl_xor(lsum, 16, 64);
    lsum += __shfl_xor(lsum, 32, 64);
  }

  // ---- merge the four waves' states through LDS (fixed wave order: results do not depend on
  // which physical pages held the tokens)
  __shared__ float s_o[4][16][DH + 4];
  __shared__ float s_m[4][16], s_l[4][16];
#pragma unroll
  for (int d = 0; d < DT; ++d) *reinterpret_cast<f32x4*>(&s_o[wave][r16][d * 16 + kg * 4]) = o[d];
  if (kg == 0) {
    s_m[wave][r16] = m;
    s_l[wave][r16] = lsum;
  }
  __syncthreads();
  const int n_spans = (n_total + span_len - 1) / span_len;
  for (int e = threadIdx.x; e < G * DH; e += 256) {
    const int q = e / DH, c = e % DH;
    const float m0 = s_m[0][q], m1 = s_m[1][q], m2 = s_m[2][q], m3 = s_m[3][q];
    const float mt = fmaxf(fmaxf(m0, m1), fmaxf(m2, m3));
    const float w0 = exp2f(m0 - mt), w1 = exp2f(m1 - mt), w2 = exp2f(m2 - mt), w3 = exp2f(m3 - mt);
    const float num = w0 * s_o[0][q][c] + w1 * s_o[1][q][c] + w2 * s_o[2][q][c] + w3 * s_o[3][q][c];
    const float den = w0 * s_l[0][q] + w1 * s_l[1][q] + w2 * s_l[2][q] + w3 * s_l[3][q];
    const int h = kvh * G + q;
    if (n_spans == 1) {
      out[operand_offset(out_lay, b, h * DH + c)] = (bf16)(num / den * out_scale);
    } else {
      const int64_t slot = ((int64_t)b * n_q_heads + h) * max_spans + span;
      if (spans_done) {
        store_agent(part_o + slot * DH + c, num);
        if (c == 0) {
          store_agent(part_ml + slot * 2 + 0, mt);
          store_agent(part_ml + slot * 2 + 1, den);
        }
      } else {
        part_o[slot * DH + c] = num;
        if (c == 0) {
          part_ml[slot * 2 + 0] = mt;
          part_ml[slot * 2 + 1] = den;
        }
      }
    }
  }
  if (n_spans == 1 || !spans_done) return;
  // ---- a request of several spans: whoever finishes last combines them, in the order of the spans whoever that is,
  //   out = sum_k o_k 2^(m_k - m) / sum_k l_k 2^(m_k - m).
  // The spans of a request are made on different XCDs, whose L2s do not see each other: partials are stored
  // and read at agent scope (past the L2), each wave waits until its stores have arrived, and only then is the span
  // counted.  The last one puts the counter back to zero for the next launch.  (A second kernel, attn_decode_merge_kernel, costs
  // a launch of 4.5 to 5 us in every layer for small batches, 10 us for 512 requests, nearly all of its workgroups with nothing
  // to do; where it still is the better way, see attn_decode_counts_spans.)
  __shared__ int s_last;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned* done = spans_done + (int64_t)b * Hkv + kvh;
    const unsigned before = __hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_last = before + 1 == (unsigned)n_spans;
    if (s_last) __hip_atomic_store(done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (!s_last) return;
  // Four channels of one query head per thread; eight spans are asked for at once, so up to eight cost one round trip.  With more
  // than two such turns, threads that a small group of heads leaves over share the spans out: `parts` runs of them, each with a
  // maximum of its own, put together through LDS.  (391 spans, a layer in all: 16 K/V heads of 128 channels with one query head each
  // 259 us on 32 threads, 201 in eight runs, 240 with the separate kernel; four requests, 8 K/V heads of 64 channels with four
  // query heads each 324, 266 and 312.)  Up to two turns the order is one run's whatever the heads.
  constexpr int UN = 8;
  const int columns = G * (DH / 4);
  const int parts = n_spans > 2 * UN && columns <= 128 ? 256 / columns : 1;
  float* const s_parts = &s_o[0][0][0];  // [part][column][4 sums, denominator, maximum]
  static_assert(256 * 6 <= 4 * 16 * (DH + 4), "a record per thread");
  for (int e = threadIdx.x; e < columns * parts; e += 256) {
    const int part = e / columns, r = e - part * columns;
    const int q = r / (DH / 4), c = r % (DH / 4) * 4, h = kvh * G + q;
    const int64_t base = ((int64_t)b * n_q_heads + h) * max_spans;
    const int k_begin = part * n_spans / parts, k_end = (part + 1) * n_spans / parts;
    float2 ml[UN], oa[UN], ob[UN];
    auto fetch = [&](int k0) {
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        const int64_t slot = base + min(k0 + u, k_end - 1);
        ml[u] = load_agent2(part_ml + slot * 2);
        oa[u] = load_agent2(part_o + slot * DH + c);
        ob[u] = load_agent2(part_o + slot * DH + c + 2);
      }
    };
    fetch(k_begin);
    float mt = kNegBig;
#pragma unroll
    for (int u = 0; u < UN; ++u) mt = fmaxf(mt, ml[u].x);  // (past the end: the last span again)
    for (int k = k_begin + UN; k < k_end; ++k) mt = fmaxf(mt, load_agent2(part_ml + (base + k) * 2).x);
    float num[4] = {0.f, 0.f, 0.f, 0.f}, den = 0.f;
    for (int k0 = k_begin; k0 < k_end; k0 += UN) {
      if (k0 > k_begin) fetch(k0);
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        if (k0 + u >= k_end) break;
        const float w = exp2f(ml[u].x - mt);
        den += w * ml[u].y;
        num[0] += w * oa[u].x;
        num[1] += w * oa[u].y;
        num[2] += w * ob[u].x;
        num[3] += w * ob[u].y;
      }
    }
    if (parts > 1) {
      float* rec = s_parts + e * 6;
#pragma unroll
      for (int i = 0; i < 4; ++i) rec[i] = num[i];
      rec[4] = den;
      rec[5] = mt;
    } else {
      bf16x4 o4;
#pragma unroll
      for (int i = 0; i < 4; ++i) o4[i] = (bf16)(num[i] / den * out_scale);
      *reinterpret_cast<bf16x4*>(out + operand_offset(out_lay, b, h * DH + c)) = o4;
    }
  }
  if (parts == 1) return;
  __syncthreads();
  if ((int)threadIdx.x < columns) {
    const int r = threadIdx.x, q = r / (DH / 4), c = r % (DH / 4) * 4, h = kvh * G + q;
    float mt = kNegBig;
    for (int part = 0; part < parts; ++part) mt = fmaxf(mt, s_parts[(part * columns + r) * 6 + 5]);
    float num[4] = {0.f, 0.f, 0.f, 0.f}, den = 0.f;
    for (int part = 0; part < parts; ++part) {
      const float* rec = s_parts + (part * columns + r) * 6;
      const float w = exp2f(rec[5] - mt);
      den += w * rec[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) num[i] += w * rec[i];
    }
    bf16x4 o4;
#pragma unroll
    for (int i = 0; i < 4; ++i) o4[i] = (bf16)(num[i] / den * out_scale);
    *reinterpret_cast<bf16x4*>(out + operand_offset(out_lay, b, h * DH + c)) = o4;
  }
}

// The same by a kernel of its own, in the order of the spans.
template <int DH>
__global__ __launch_bounds__(DH) void attn_decode_merge_kernel(const float* __restrict__ part_o,
                                                               const float* __restrict__ part_ml,
                                                               const int32_t* __restrict__ ctx_lens,
                                                               int max_pages_per_seq, int n_q_heads, int max_spans,
                                                               int span_len, bf16* __restrict__ out,
                                                               OperandLayout out_lay, float out_scale) {
  const int h = blockIdx.x, b = blockIdx.y, c = threadIdx.x;
  const int n_spans = (decode_position(ctx_lens[b], max_pages_per_seq) + span_len) / span_len;
  if (n_spans <= 1) return;  // finished by the attention kernel itself
  const int64_t base = ((int64_t)b * n_q_heads + h) * max_spans;
  float m = kNegBig;
  for (int k = 0; k < n_spans; ++k) m = fmaxf(m, part_ml[(base + k) * 2]);
  float num = 0.f, den = 0.f;
  for (int k = 0; k < n_spans; ++k) {
    const float w = exp2f(part_ml[(base + k) * 2] - m);
    den += w * part_ml[(base + k) * 2 + 1];
    num += w * part_o[(base + k) * DH + c];
  }
  out[operand_offset(out_lay, b, h * DH + c)] = (bf16)(num / den * out_scale);
}

// Span length.  A workgroup's fixed costs (start-up, the merge of its four waves, its partial
// result) are paid once per span, so spans should be as long as the batch allows while the launch
// still has several workgroups per CU; a context that fits one span needs no partials at all.
// Measured on the 70B shape (attention ms per layer at spans 256 / 1024 / 2048 / 4096): batch 16:
// .032 / .028 / .035 / .046; batch 128: .158 / .138 / .137 / .138; batch 512: .610 / .521 / .494 / .487.
int attn_decode_span(int batch, int n_kv_heads) {
  const int units = batch * n_kv_heads;
  return units >= 4096 ? 4096 : units >= 1024 ? 2048 : units >= 128 ? 1024 : kDecodeSpanMin;
}

int attn_decode_items(int batch, int max_spans, int span_len) {
  // max_spans counts spans of the minimum length; longer spans need proportionally fewer slots
  return batch * ((max_spans * kDecodeSpanMin + span_len - 1) / span_len);
}

// Whether the attention kernel combines the spans itself.  A workgroup that counts its span waits until its partials have arrived
// and for the count, a few us in which it holds its slot under a saturated memory system; the second kernel is a launch in
// every layer and reads the partials of all query heads again.  With four query heads or more per K/V head the count is ahead (a layer
// with 8 K/V heads of 128 channels, 16 to 200 requests of 500 to 39,000 tokens: 0 to 7 % with eight, 0 to 5 % with five, 4 to -1 % with
// four).  With one or two the second kernel is, from about ten spans on: one, 16 heads, 16 requests of 9000 / 20,000 / 39,000 tokens 239 /
// 488 / 927 us with the count, 231 / 455 / 833 with the second kernel; 40 heads 537 / 1119 / 2165 and 522 / 1089 / 2063; two, 8 K/V heads, 64
// requests 422 / 892 / 1721 and 417 / 868 / 1653 (3000 tokens level, 500 tokens 1.5 to 2.5 us for a kernel that finds nothing to do).
// How long the contexts are is known on the device alone: the line goes by the longest that the block tables allow.  Spans
// below 1024 tokens stay with the count: they are for small batches, where the second kernel walks hundreds of them
// in a row (one request of 100,000 tokens, 16 heads: 240 us, with the count 201).
bool attn_decode_counts_spans(int batch, int n_q_heads, int n_kv_heads, int max_spans, int span_len) {
  return n_q_heads > 2 * n_kv_heads || span_len < 1024 || attn_decode_items(batch, max_spans, span_len) < 10 * batch;
}

// Whether a decode step makes a work list.  Without one a workgroup's look-ups are the request's length and its table row.
// The list is what orders work (longest first) and cuts it into spans: with at most one span per request and no more
// workgroups than run at once (three per CU) it does neither, and its launch was 4 of 67 us of a two-layer step of
// the toy shape with four requests.
bool attn_decode_planned(int batch, int n_kv_heads, int max_spans, int span_len) {
  return attn_decode_items(batch, max_spans, span_len) > batch || batch * n_kv_heads > 3 * 256;
}

// Whether the attention kernel rotates the queries and appends the new keys and values itself.  A kernel in front of it is a launch in
// every layer, 4 to 8 us for small batches.  As long as there are no more (request, K/V head) pairs than three workgroups per CU the
// rotation is ahead inside or level, two layers, us, both ways in turn on one card: 70B, 8 / 16 / 64 requests 586 / 604 / 747 with the kernel in
// front, 579 / 598 / 747 inside; 7B, 2 / 16 requests 229 / 268 and 222 / 262; Qwen, 48 481 and 476; toy widths, 4 / 256 requests 67.0 / 75.1 and
// 66.3 / 72.4.  At 880 pairs the two are level, and beyond that every value stored among the reads costs more than it does in front of
// them: 13B, 5120 pairs, 1202 and 1258.
// A request of several spans has its queries rotated once per span.  Beside spans of 1024 tokens and more that is lost in the reads at any
// length (QKV and attention of one layer, inside / in front, 128 to 768 pairs, contexts of 1000 to 100,000 tokens: 0.93 to 1.01, 70B with 64
// requests of 20,000 972 / 978 us).  Beside the spans of 256 of fewer than 128 pairs it is not, once there are many of them: 0.92 to 0.99 up to
// 4000 workgroups, level around 5000, and from there 1.01 to 1.04, with 8-bit pools to 1.07 (70B, 8 requests of 10,000 / 30,000 / 100,000
// tokens 171 / 315 / 837 us inside, 172 / 309 / 811 in front; 7B, 8 bits, 3 requests of 20,000 / 100,000 1.02 / 1.05).  How long the contexts
// are is known on the device alone; the line goes by the workgroups of the longest that the block tables allow, at a place where contexts
// spread over that length lose as much as they gain.  (16 query heads on one K/V head need a second turn of the rotating waves:
// 120 requests of 2000 tokens, 960 workgroups, 1.03.)
bool attn_decode_rotates(int batch, int n_kv_heads, int max_spans, int span_len) {
  if (batch * n_kv_heads > 3 * 256) return false;
  return span_len >= 1024 || (int64_t)attn_decode_items(batch, max_spans, span_len) * n_kv_heads <= 8192;
}

hipError_t launch_attn_plan(const int32_t* ctx_lens, const int32_t* block_tables, int max_pages_per_seq, int batch,
                            int max_spans, int span_len, int4* items, int32_t* item_pages, hipStream_t s) {
  if (batch <= 0) return hipSuccess;
  const int max_items = attn_decode_items(batch, max_spans, span_len);
  attn_plan_kernel<<<(batch + 3) / 4, 256, 0, s>>>(ctx_lens, batch, span_len, block_tables, max_pages_per_seq, items,
                                                  max_items, item_pages);
  return hipGetLastError();
}

hipError_t launch_attn_decode(const DecodeQueries& dq, int batch, int n_q_heads, const KvLayout& kv,
                              const int4* items, const int32_t* item_pages, int item_pitch, const int32_t* ctx_lens,
                              float* part_o, float* part_ml, unsigned* spans_done, int max_spans, int span_len,
                              void* out, OperandLayout out_layout, hipStream_t s) {
  if (batch <= 0) return hipSuccess;
  // 8-bit pools hold value / scale: the key scale joins the softmax scale, the value scale the final division
  const float scale_log2 = 1.4426950408889634f / sqrtf((float)kv.head_dim) * (kv.fp8 ? kv.k_scale : 1.0f);
  const float out_scale = kv.fp8 ? kv.v_scale : 1.0f;
  const int max_items = attn_decode_items(batch, max_spans, span_len);
  const unsigned grid = (unsigned)max_items * kv.n_kv_heads;
#define TDP_DECODE_(DH, KV8, ROTATE)                                                                                   \
  attn_decode_kernel<DH, KV8, ROTATE><<<grid, 256, 0, s>>>(dq, batch, n_q_heads, kv, items, item_pages, item_pitch, ctx_lens, \
                                                           part_o, part_ml, spans_done, max_spans, span_len, (bf16*)out, \
                                                           out_layout, scale_log2, out_scale)
#define TDP_DECODE(DH, KV8) do { if (dq.qkv) TDP_DECODE_(DH, KV8, false); else TDP_DECODE_(DH, KV8, true); } while (0)
  if (kv.head_dim == 128) {
    if (kv.fp8) TDP_DECODE(128, true); else TDP_DECODE(128, false);
  } else {
    if (kv.fp8) TDP_DECODE(64, true); else TDP_DECODE(64, false);
  }
#undef TDP_DECODE_
#undef TDP_DECODE
  return hipGetLastError();
}

hipError_t launch_attn_decode_merge(int batch, int n_q_heads, const KvLayout& kv, const int32_t* ctx_lens,
                                    int max_pages_per_seq, const float* part_o, const float* part_ml, int max_spans,
                                    int span_len, void* out, OperandLayout out_layout, hipStream_t s) {
  if (batch <= 0) return hipSuccess;
  const float out_scale = kv.fp8 ? kv.v_scale : 1.0f;
  const dim3 grid(n_q_heads, batch);
#define TDP_MERGE(DH)                                                                                                  \
  attn_decode_merge_kernel<DH><<<grid, DH, 0, s>>>(part_o, part_ml, ctx_lens, max_pages_per_seq, n_q_heads, max_spans, \
                                                   span_len, (bf16*)out, out_layout, out_scale)
  if (kv.head_dim == 128) TDP_MERGE(128); else TDP_MERGE(64);
#undef TDP_MERGE
  return hipGetLastError();
}

// =====================================================================================
// Prefill: var-len packed, causal.  One workgroup of NW waves per tile of NW * 32 query columns that share one K/V
// head; a column is a (position, query head) pair, all G heads of the group at one position, then the next
// position, so any group size fills the waves (128 columns: 16 positions of 8 heads, 25 of 5, 128 of 1; a few
// columns are left over where G does not divide them).  (With a head per wave a group of five fell back to one head
// per workgroup: five times the staging and a tile of one head; 267 us on 6713 tokens of 40 / 8 heads, 245 with pairs
// and 207 with the order of the tiles below.)  Each 32-token
// block of K and V^T is staged once per workgroup in LDS (double buffered, XOR-swizzled against
// bank conflicts) and feeds the MFMAs of all columns, so K/V traffic per MFMA is 1/NW of a
// wave-private scheme.  Two waves share a SIMD, so one wave's softmax arithmetic overlaps the
// other's MFMAs; the softmax itself is trimmed to what a wave64 vector unit can keep up with:
// one FMA + one raw exp2 per score, masking only in blocks that cross the diagonal or the end of
// the prompt, and the running maximum is only raised (and the accumulator rescaled) when a
// block's maximum exceeds it by more than 2^8, which keeps every probability below 256.
// Same transposed-score trick as decode: S^T = K Q^T with score rows permuted so that a lane's
// accumulator elements are the 8 consecutive tokens it supplies to O^T += V^T P^T.
// =====================================================================================
constexpr float kRescaleSlack = 8.0f;  // log2 units

// KV8: the pools hold E4M3 codes; a thread's chunk is then 8 bytes, converted to bf16 on its way into
// LDS (the key scale rides in the softmax scale, the value scale in the final normalisation).
template <int DH, int NW, bool KV8>
__global__ __launch_bounds__(NW * 64, 2) void attn_prefill_kernel(
    const bf16* __restrict__ qkv, int64_t ld, int G, KvLayout kv, const int32_t* __restrict__ cu_seqlens,
    int n_seqs, const int32_t* __restrict__ block_tables, int max_pages_per_seq, bf16* __restrict__ out,
    OperandLayout out_lay, float scale_log2, float out_scale, int np, unsigned np_inverse, int g_inverse) {
  // np = NW * 32 / G positions per workgroup; x / np = umulhi(x, np_inverse) for the lengths that occur (below 2^21),
  // x / G = x * g_inverse >> 16 for columns
  constexpr int NT = NW * 64;
  constexpr int KS = DH / 16;    // k-steps of the score MFMA
  constexpr int DT = DH / 32;    // 32-channel tiles of the output
  constexpr int CR = DH / 8;     // 16-byte chunks per K row
  constexpr int RWK = DH == 128 ? 1 : 2;  // K rows per 256-byte bank window
  constexpr int NCH = 64 * CR / NT;  // chunks of K, and of V^T, per thread per 64-token block
  constexpr int QP = KV8 ? 8 : 4;  // 8-element chunks per 64-byte piece of a key row in the pool
  __shared__ __attribute__((aligned(16))) bf16 sK[2][2][32 * DH];  // [buffer][32-token half]
  __shared__ __attribute__((aligned(16))) bf16 sV[2][2][DH * 32];

  // locate the sequence that owns the query tile
  const int Hkv = kv.n_kv_heads;
  // K/V heads are numbered fastest: workgroups go round-robin to the 8 XCDs, so with a multiple of eight heads every tile
  // of a head reads K/V through the same L2.  The last tiles come first: within a prompt they are the longest.
  const int tile = blockIdx.x / Hkv, kvh = blockIdx.x - tile * Hkv;
  int qt = (int)gridDim.x / Hkv - 1 - tile, s = 0, L = 0;
  for (; s < n_seqs; ++s) {
    L = cu_seqlens[s + 1] - cu_seqlens[s];
    const int nt = (int)__umulhi((unsigned)(L + np - 1), np_inverse);
    if (qt < nt) break;
    qt -= nt;
  }
  if (s == n_seqs) return;
  const int tok0 = cu_seqlens[s];
  const int q0 = qt * np;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, kg = lane >> 5;
  const bf16* kpool = (const bf16*)kv.k_pool;
  const bf16* vpool = (const bf16*)kv.v_pool;

  // the lane's query column and the positions its wave spans
  const int col = wave * 32 + l32;
  const int col_pos = col * g_inverse >> 16;
  const int head = kvh * G + col - col_pos * G;
  const bool real = col < np * G;  // (the columns left over follow the last position, are computed and never stored)
  const int qpos = q0 + min(col_pos, np - 1);  // may lie past the end of the prompt: computed, never stored
  const int p_first = q0 + min(wave * 32 * g_inverse >> 16, np - 1);
  const int p_last = min(q0 + min((wave * 32 + 31) * g_inverse >> 16, np - 1), L - 1);
  bf16x8 qf[KS];
  {
    const bf16* qp = qkv + (int64_t)(tok0 + min(qpos, L - 1)) * ld + (int64_t)head * DH + kg * 8;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) qf[kk] = ld_bf16x8(qp + kk * 16);
  }
  f32x16 o[DT];
#pragma unroll
  for (int d = 0; d < DT; ++d)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[d][i] = 0.f;
  float m = kNegBig, lsum = 0.f;

  const int32_t* bt = block_tables + (int64_t)s * max_pages_per_seq;
  const int last_page = (L - 1) / 16;
  const int kv_end = min(q0 + np, L);
  // token of this lane's row r = l32 in the score tile: (r/16)*16 + ((r%8)/4)*8 + ((r/8)%2)*4 + r%4
  const int krow = (l32 >> 4) * 16 + ((l32 >> 2) & 1) * 8 + ((l32 >> 3) & 1) * 4 + (l32 & 3);
  const bf16* k_frag = &sK[0][0][0] + krow * DH;
  const int k_swz = (krow / RWK) % CR;

  // Staging of the next 64-token block (two 32-token halves).  The pages of a block are looked up a block before its keys and values
  // are requested.  16-bit pools go straight into LDS, an instruction 1 KiB of it, each lane from where the swizzle wants its 16
  // bytes to come: wave w takes the keys of the block's page w, and half of the channels of the values of a half; 8-bit pools go
  // through registers for the conversion.  What that leaves of the registers holds all fragments of a half at once.  (Everything
  // through registers, look-ups and loads in one go, values past the prompt masked on the way, fragments read two by two: 16.0 us
  // for one prompt of 307 tokens of 32 heads, now 12.9; 6713 tokens of 40 / 8 heads 210 -> 183; 19346 of 64 / 8 944 -> 834; 8 bits, 12
  // prompts of a 13B shape, where the look-ups and the fragments alone count, 139 -> 115.  Both halves' scores in front of one
  // softmax over 64 tokens: level.)
  int page[4];
  auto look_up = [&](int kb) {  // never dereference a table entry past the last page
#pragma unroll
    for (int i = 0; i < 4; ++i) page[i] = bt[min((kb >> 4) + i, last_page)];
  };
  bf16x8 kreg[KV8 ? NCH : 1], vreg[KV8 ? NCH : 1];
  const int w = __builtin_amdgcn_readfirstlane(wave);
  const unsigned k_lds = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)&sK[0][0][0];
  const unsigned v_lds = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)&sV[0][0][0];
  constexpr int HEAD = 16 * DH;         // elements of a page, one K/V head
  constexpr int TPI = 512 / DH;         // key rows (tokens) of an instruction
  static_assert(KV8 || (NW == 4 && NCH * TPI == 16), "a wave's instructions make one page of keys");
  // this lane's element offsets into its page of K (instruction j), and into its page of V (instruction 0; 16 channels further on in each)
  int k_off[KV8 ? 1 : NCH];
  const int v_row = lane >> 2, v_chunk = (lane & 3) ^ ((v_row >> 2) & 3);
  const int v_off = ((w & 1) * (DH / 2) + v_row) * 16 + (v_chunk & 1) * 8;
  if constexpr (!KV8) {
#pragma unroll
    for (int j = 0; j < NCH; ++j) {
      const int slot = j * TPI + lane / CR, ktok = (w & 1) * 16 + slot, kc = (lane % CR) ^ ((ktok / RWK) % CR);
      k_off[j] = (kc / QP) * 512 + slot * 32 + kc % QP * 8;
    }
  }
  auto request = [&](unsigned lds_addr, const bf16* from) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_addr), "v"(from) : "memory");
  };
  auto load_block = [&](int buf) {
    if constexpr (KV8) {
#pragma unroll
      for (int j = 0; j < NCH; ++j) {
        const int ci = tid + NT * j;
        // K: consecutive threads walk the pool in address order - the QP chunks of a 64-byte piece, the 16
        // tokens of the page, the pieces of the row, the four pages of the block
        const int kq = ci % QP, kt16 = (ci / QP) % 16, kpiece = (ci / (QP * 16)) % (CR / QP), kpg = ci / (16 * CR);
        const int64_t kp = kpg == 0 ? page[0] : kpg == 1 ? page[1] : kpg == 2 ? page[2] : page[3];
        const int vsub = ci / (DH * 4), vr = (ci >> 2) % DH, vc = ci & 3;
        const int64_t vp = vsub ? (vc < 2 ? page[2] : page[3]) : (vc < 2 ? page[0] : page[1]);
        const int64_t k_at = (kp * Hkv + kvh) * HEAD + (kpiece * 16 + kt16) * (QP * 8) + kq * 8;
        const int64_t v_at = ((vp * Hkv + kvh) * DH + vr) * 16 + (vc & 1) * 8;
        union {
          uint32_t u[4];
          bf16x8 x;
        } ck, cv;
        const uint2 rk = *reinterpret_cast<const uint2*>((const uint8_t*)kv.k_pool + k_at);
        const uint2 rv = *reinterpret_cast<const uint2*>((const uint8_t*)kv.v_pool + v_at);
        e4m3x4_to_bf16x4(rk.x, ck.u[0], ck.u[1]);
        e4m3x4_to_bf16x4(rk.y, ck.u[2], ck.u[3]);
        e4m3x4_to_bf16x4(rv.x, cv.u[0], cv.u[1]);
        e4m3x4_to_bf16x4(rv.y, cv.u[2], cv.u[3]);
        kreg[j] = ck.x;
        vreg[j] = cv.x;
      }
    } else {
      const int64_t k_page = w == 0 ? page[0] : w == 1 ? page[1] : w == 2 ? page[2] : page[3];
      const int64_t v_page = w < 2 ? (v_chunk < 2 ? page[0] : page[1]) : (v_chunk < 2 ? page[2] : page[3]);
      const bf16* kp = kpool + (k_page * Hkv + kvh) * HEAD;
      const bf16* vp = vpool + (v_page * Hkv + kvh) * HEAD + v_off;
      const unsigned half = buf * (64 * DH * 2) + w * (NCH * 1024);
#pragma unroll
      for (int j = 0; j < NCH; ++j) request(k_lds + half + j * 1024, kp + k_off[j]);
#pragma unroll
      for (int j = 0; j < NCH; ++j) request(v_lds + half + j * 1024, vp + j * 256);
    }
  };
  // the block kb has arrived in buffer buf for all waves
  auto settle = [&](int kb, int buf) {
    if constexpr (KV8) {
#pragma unroll
      for (int j = 0; j < NCH; ++j) {
        const int ci = tid + NT * j;
        const int kq = ci % QP, kt16 = (ci / QP) % 16, kpiece = (ci / (QP * 16)) % (CR / QP), kpg = ci / (16 * CR);
        const int ksub = kpg >> 1, ktok = (kpg & 1) * 16 + kt16, kc = kpiece * QP + kq;
        st_bf16x8(&sK[buf][ksub][ktok * DH + ((kc ^ ((ktok / RWK) % CR)) << 3)], kreg[j]);
        const int vsub = ci / (DH * 4), vr = (ci >> 2) % DH, vc = ci & 3;
        st_bf16x8(&sV[buf][vsub][vr * 32 + ((vc ^ ((vr >> 2) & 3)) << 3)], vreg[j]);
      }
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (kb + 64 > L) {  // slots past the prompt may hold anything, even NaN
#pragma unroll
      for (int j = 0; j < NCH; ++j) {
        const int ci = tid + NT * j, vsub = ci / (DH * 4), vr = (ci >> 2) % DH, vc = ci & 3;
        const int keep = L - (kb + vsub * 32 + vc * 8);
        if (keep < 8) {
          bf16* at = &sV[buf][vsub][vr * 32 + ((vc ^ ((vr >> 2) & 3)) << 3)];
          bf16x8 v = ld_bf16x8(at);
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (e >= keep) v[e] = (bf16)0.0f;
          st_bf16x8(at, v);
        }
      }
      __syncthreads();
    }
  };

  look_up(0);
  load_block(0);
  look_up(64);
  settle(0, 0);
  // The queries have arrived as well.  Used here, they are waited for here; left to the loop, each of its turns waits for them again, and so for
  // the requests of the next block, which are behind them in the same counter.
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) asm volatile("" : "+v"(qf[kk]));
  for (int kb0 = 0, buf = 0; kb0 < kv_end; kb0 += 64, buf ^= 1) {
    const bool more = kb0 + 64 < kv_end;
    if (more) load_block(buf ^ 1);
    look_up(kb0 + 128);
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {
      const int kb = kb0 + sub * 32;
      // causal: blocks past the wave's last row contribute nothing
      if (kb > p_last || p_first >= L) continue;
      f32x16 sc;
#pragma unroll
      for (int i = 0; i < 16; ++i) sc[i] = 0.f;
      bf16x8 kf[KS];  // all of the block's fragments first: one LDS round trip and not one per pair of MFMAs
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) kf[kk] = ld_bf16x8(k_frag + (buf * 2 + sub) * 32 * DH + (((kk * 2 + kg) ^ k_swz) << 3));
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) sc = mfma32(kf[kk], qf[kk], sc);
      __builtin_amdgcn_sched_barrier(0);
      bf16x8 vf[DT][2];  // on their way during the softmax
#pragma unroll
      for (int d = 0; d < DT; ++d)
#pragma unroll
        for (int st = 0; st < 2; ++st) {
          const int r = d * 32 + l32;
          vf[d][st] = ld_bf16x8(&sV[buf][sub][r * 32 + (((st * 2 + kg) ^ ((r >> 2) & 3)) << 3)]);
        }
      __builtin_amdgcn_sched_barrier(0);
      // element i of this lane is token kb + (i/8)*16 + kg*8 + i%8 of query column qpos
      if (kb + 31 > p_first || kb + 32 > L) {  // the block crosses the diagonal or the prompt's end
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int tok = kb + (i >> 3) * 16 + kg * 8 + (i & 7);
          if (!(tok <= qpos && tok < L)) sc[i] = kNegBig;
        }
      }
      float mx = sc[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) mx = fmaxf(mx, sc[i]);
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64)) * scale_log2;  // scale > 0: max commutes with it
      if (__any(mx > m + kRescaleSlack)) {
        const float m_new = fmaxf(m, mx);
        const float alpha = __builtin_amdgcn_exp2f(m - m_new);
        lsum *= alpha;
        m = m_new;
#pragma unroll
        for (int d = 0; d < DT; ++d)
#pragma unroll
          for (int i = 0; i < 16; ++i) o[d][i] *= alpha;
      }
      bf16x8 pb[2];
      float psum = 0.f;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float pv = __builtin_amdgcn_exp2f(fmaf(sc[i], scale_log2, -m));
        psum += pv;
        pb[i >> 3][i & 7] = (bf16)pv;
      }
      lsum += psum;
#pragma unroll
      for (int d = 0; d < DT; ++d)
#pragma unroll
        for (int st = 0; st < 2; ++st) o[d] = mfma32(vf[d][st], pb[st], o[d]);
    }
    if (more) settle(kb0 + 64, buf ^ 1);
  }
  lsum += __shfl_xor(lsum, 32, 64);
  if (real && qpos < L) {
    const float inv = out_scale / lsum;
#pragma unroll
    for (int d = 0; d < DT; ++d)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        bf16x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (bf16)(o[d][g * 4 + e] * inv);
        *reinterpret_cast<bf16x4*>(out + operand_offset(out_lay, tok0 + qpos, head * DH + d * 32 + g * 8 + kg * 4)) =
            v;
      }
  }
}

template <int DH, int NW>
static hipError_t launch_attn_prefill_t(const void* qkv, int64_t ld, int total_tokens, int n_seqs, int n_q_heads,
                                        const KvLayout& kv, const int32_t* cu_seqlens, const int32_t* block_tables,
                                        int max_pages_per_seq, void* out, OperandLayout out_layout, hipStream_t s) {
  const float scale_log2 = 1.4426950408889634f / sqrtf((float)kv.head_dim) * (kv.fp8 ? kv.k_scale : 1.0f);
  const float out_scale = kv.fp8 ? kv.v_scale : 1.0f;
  const int G = n_q_heads / kv.n_kv_heads, np = NW * 32 / G;
  // (lengths are at most 2^20 and np at most 256: rounding the inverse up is off by less than 2^-32 x 2^21 x 2^8)
  const unsigned np_inverse = (unsigned)(((1ull << 32) + np - 1) / np);
  const int g_inverse = (65536 + G - 1) / G;  // (columns are below 256 and G at most 16: off by less than 2^-16 x 2^8 x 2^4)
  const unsigned grid = (unsigned)((total_tokens + np - 1) / np + n_seqs) * kv.n_kv_heads;
#define TDP_PREFILL(KV8)                                                                                             \
  attn_prefill_kernel<DH, NW, KV8><<<grid, NW * 64, 0, s>>>((const bf16*)qkv, ld, G, kv, cu_seqlens, n_seqs,         \
                                                            block_tables, max_pages_per_seq, (bf16*)out, out_layout,  \
                                                            scale_log2, out_scale, np, np_inverse, g_inverse)
  if (kv.fp8) TDP_PREFILL(true); else TDP_PREFILL(false);
#undef TDP_PREFILL
  return hipGetLastError();
}

hipError_t launch_attn_prefill(const void* qkv, int64_t ld, int total_tokens, int n_seqs, int n_q_heads,
                               const KvLayout& kv, const int32_t* cu_seqlens, const int32_t* block_tables,
                               int max_pages_per_seq, void* out, OperandLayout out_layout, hipStream_t s) {
  if (total_tokens <= 0 || n_seqs <= 0) return hipSuccess;
  // Four waves and not eight (measured, us: 12 prompts of a 13B shape 170 / 143, 24 of a 7B shape 177 / 159, 8 of 40 / 8
  // heads 258 / 253, 16 of 64 / 8 heads level; 64 channels, 32 / 8 heads: one prompt of 4096 156 / 114, of 16384 1603 / 1499, 16 of
  // 1024 173 / 141, 24 ragged ones 126 / 118; 32 / 32 heads 161 / 113, 1716 / 1491, 175 / 143, 114 / 103): tiles half as long
  // compute less beyond the diagonal and two workgroups of a CU wait at barriers of their own.  One prompt of 100 tokens
  // costs 0.5 to 1.5 us more, a thread stages twice the keys (128 channels 11 / 12, 64 channels 9 / 9).
  if (kv.head_dim == 128)
    return launch_attn_prefill_t<128, 4>(qkv, ld, total_tokens, n_seqs, n_q_heads, kv, cu_seqlens, block_tables,
                                         max_pages_per_seq, out, out_layout, s);
  return launch_attn_prefill_t<64, 4>(qkv, ld, total_tokens, n_seqs, n_q_heads, kv, cu_seqlens, block_tables,
                                      max_pages_per_seq, out, out_layout, s);
}

}  // namespace tdp
