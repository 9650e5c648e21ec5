// bf16 MFMA GEMM for the stage's four projections (paper Sec. 3.4: linear layers dominate the
// execution time of a decode step, and only the batch size sets their cost).
//
//   out[M, N] = epilogue( A[M, K] * W^T ),   A bf16 M x K,  W bf16 Npad x Kpad  (both K-contiguous in
//   32-column blocks; W and the stage's own activations are pair-interleaved, see OperandLayout)
//
// Both operands are K-contiguous, so an MFMA fragment is one 16-byte load.  The product is formed
// transposed, D[n][m] = sum_k W[n][k] A[m][k], with the weights as the MFMA "A" operand: a lane
// then holds four consecutive output columns n of one row m, which makes the epilogue's stores
// 8 bytes wide and lets the SwiGLU epilogue find gate and up of one column in the same lane.
//
// Tiles go from global memory straight into LDS (direct-to-LDS loads, a ring of 32-wide k-stages,
// one barrier per stage) with an XOR swizzle of the 16-byte chunks applied on the global side, so
// that the fragment reads are free of bank conflicts.  For small M (decode) the K range is split
// across workgroups; the fp32 partials are summed by the kernel that consumes the projection, or
// by a reduce kernel that applies the epilogue.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>

#include <initializer_list>
#include <mutex>
#include <type_traits>
#include <unordered_map>

#include "tdp_device.h"
#include "tdp_kernels.h"

namespace tdp {

struct GemmParams {
  const bf16* A;
  const bf16* W;
  bf16* out;
  const void* residual;  // bf16, or fp32 when res_f32
  const float* bias;     // fp32 [Npad] or null
  float* ws;
  OperandLayout a_lay, w_lay, u_lay;
  int64_t Kpad, Npad, ldo, ldr;
  int M, N_store, epilogue, out_f32, res_f32;
  int k_tiles_total, k_tiles_per_split, splits;
  int k_tiles_per_chunk;  // 0, or (splits = 1, small tiles) the K range is summed in chunks of this many k-tiles
  int tiles_m, tiles_n;
  // order of the tiles, see gemm_tile_of_block: bands of band_h + 1 (the first n_tall) or band_h rows of tiles; an
  // XCD takes `chunks` runs of `chunk` tiles, and an eighth of the `rest` tiles behind them
  int band_h, n_tall, chunk_shift, chunks, rest;
  unsigned per_split_inv, tall_inv, low_inv, h_tall_inv, h_low_inv;  // see divide
};
// What the two epilogues that only one projection has need on top.  Their kernels are instances of their own (the type of the
// parameters selects the epilogue): as run-time branches of every instance they cost the others registers, 16 -> 24 spilled ones
// of a 256 x 256 tile, 3 to 4 more and 17 scalar ones of the other tiles of 256 weight rows.
struct GemmRotateParams : GemmParams {
  PrefillRotation rot;
};
struct GemmMaxParams : GemmParams {
  float* row_max;  // [M][2 tiles_n]
};

// silu(z) = z / (1 + e^-z), with the hardware reciprocal (1 ulp) in place of an IEEE division: the
// gated epilogue evaluates it 128 times per lane and tile, and its result is rounded to bf16 anyway.
__device__ __forceinline__ float silu_f(float z) { return z * __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }

// Residual add and store of four consecutive output columns (plain / residual epilogues).
__device__ __forceinline__ void store_row4(const GemmParams& p, int m, int n, float (&v)[4]) {
  if (p.bias) {
    const f32x4 b = *reinterpret_cast<const f32x4*>(p.bias + n);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] += b[e];
  }
  if (p.epilogue == EPI_RESIDUAL) {
    if (p.res_f32) {
      const f32x4 r = *reinterpret_cast<const f32x4*>((const float*)p.residual + (int64_t)m * p.ldr + n);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += r[e];
    } else {
      const bf16x4 r = *reinterpret_cast<const bf16x4*>((const bf16*)p.residual + (int64_t)m * p.ldr + n);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += (float)r[e];
    }
  }
  if (p.out_f32) {
    *reinterpret_cast<f32x4*>((float*)p.out + (int64_t)m * p.ldo + n) = f32x4{v[0], v[1], v[2], v[3]};
  } else {
    bf16x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (bf16)v[e];
    *reinterpret_cast<bf16x4*>(p.out + (int64_t)m * p.ldo + n) = o;
  }
}

// Epilogue of the GEMM kernel (16x16 accumulator tiles): a lane holds, for each (wt, at), output columns
// n..n+3 of row m, with m = row0 + at*16 + l16 and n = col0 + wt*16 + kq*4.  Gate and up rows
// alternate in blocks of 32 weight rows, i.e. tiles wt, wt+1 (gate) pair with wt+2, wt+3 (up).
template <int AT, int WT>
__device__ __forceinline__ void gemm_epilogue16(const GemmParams& p, f32x4 (&acc)[WT][AT], int row0, int col0,
                                                int l16, int kq, int split) {
#pragma unroll
  for (int at = 0; at < AT; ++at) {
    const int m = row0 + at * 16 + l16;
    if (m >= p.M) continue;
    if (p.splits > 1) {
      float* dst = p.ws + ((int64_t)split * p.M + m) * p.Npad;
#pragma unroll
      for (int wt = 0; wt < WT; ++wt) *reinterpret_cast<f32x4*>(dst + col0 + wt * 16 + kq * 4) = acc[wt][at];
    } else if (p.epilogue == EPI_SWIGLU) {
#pragma unroll
      for (int wt = 0; wt < WT; wt += 4)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int j = (col0 + wt * 16) / 2 + h * 16 + kq * 4;
          if (j < p.N_store) {
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (bf16)(silu_f(acc[wt + h][at][e]) * acc[wt + h + 2][at][e]);
            *reinterpret_cast<bf16x4*>(p.out + operand_offset(p.u_lay, m, j)) = o;
          }
        }
    } else {
#pragma unroll
      for (int wt = 0; wt < WT; ++wt) {
        const int n = col0 + wt * 16 + kq * 4;
        if (n < p.N_store) {
          float v[4] = {acc[wt][at][0], acc[wt][at][1], acc[wt][at][2], acc[wt][at][3]};
          store_row4(p, m, n, v);
        }
      }
    }
  }
}

// The plain fp32 epilogue with the largest element of every row among the wave's 16 WT columns (unsplit, no bias; minus infinity
// where there is nothing but NaN).  The exchanges between lanes, two round trips through LDS for each row block, come behind all stores
// and are in flight together: made block by block in front of the next one's stores they took most of what the maxima save (see
// tdp_lm_head).  (Accumulators are read block by block; all read ahead they spill.)
template <int AT, int WT>
__device__ __forceinline__ void gemm_epilogue16_max(const GemmMaxParams& p, f32x4 (&acc)[WT][AT], int row0, int col0,
                                                    int l16, int kq) {
  float mx[AT];
#pragma unroll
  for (int at = 0; at < AT; ++at) {
    const int m = row0 + at * 16 + l16;
    float* out = (float*)p.out + (int64_t)m * p.ldo;
    mx[at] = -INFINITY;
#pragma unroll
    for (int wt = 0; wt < WT; ++wt) {
      const int n = col0 + wt * 16 + kq * 4;
      asm volatile("" : "+a"(acc[wt][at]));
      if (m < p.M && n < p.N_store) {
        const f32x4 v = acc[wt][at];
        *reinterpret_cast<f32x4*>(out + n) = v;
        mx[at] = fmaxf(fmaxf(mx[at], fmaxf(v[0], v[1])), fmaxf(v[2], v[3]));
      }
    }
  }
#pragma unroll
  for (int at = 0; at < AT; ++at) mx[at] = fmaxf(mx[at], __shfl_xor(mx[at], 16, 64));
#pragma unroll
  for (int at = 0; at < AT; ++at) mx[at] = fmaxf(mx[at], __shfl_xor(mx[at], 32, 64));
#pragma unroll
  for (int at = 0; at < AT; ++at) {
    const int m = row0 + at * 16 + l16;
    if (kq == 0 && m < p.M) p.row_max[(int64_t)m * (2 * p.tiles_n) + col0 / (16 * WT)] = mx[at];
  }
}

// The epilogue of an unsplit QKV projection in prefill: bias, rotation, one rounding; queries and values go to the bf16 rows, keys to
// their slots.  A wave's columns are whole heads (16 WT = 128: one of 128 channels or two of 64), so a lane holds both channels of
// its pairs: tile t of a head and tile t + H, H = head_dim / 32.  Bound: the stores, and two look-ups in a row (a token's position,
// then its (cos, sin)), asked for two row blocks at a time.  Against
// an fp32 projection that a kernel of its own reads back (19346 tokens of 70B: 2364 + 219 us; 7959 of 7B: 705 + 128; 6713 of Qwen: 467 +
// 52) the projection is no longer: 2325, 711, 441.
template <int AT, int WT, int H>
__device__ __forceinline__ void gemm_epilogue16_rotate(const GemmRotateParams& p, f32x4 (&acc)[WT][AT], int row0, int col0,
                                                       int l16, int kq) {
  const PrefillRotation& r = p.rot;
  constexpr int DH = 32 * H, AB = 2;
  const bool odd = kq & 1;  // channels 4 .. 7 of eight
  int2 where[AT];
#pragma unroll
  for (int at = 0; at < AT; ++at) where[at] = r.token_pages[min(row0 + at * 16 + l16, p.M - 1)];
#pragma unroll
  for (int hd = 0; hd < WT / (2 * H); ++hd) {
    const int col = col0 + hd * DH, head = col / DH, kvh = head - r.n_q_heads;
    if (kvh >= 2 * r.kv.n_kv_heads) continue;  // padding
    f32x4 bias[2 * H];
    if (p.bias) {
#pragma unroll
      for (int t = 0; t < 2 * H; ++t) bias[t] = *reinterpret_cast<const f32x4*>(p.bias + col + t * 16 + kq * 4);
    }
    const bool value = kvh >= r.kv.n_kv_heads;
#pragma unroll
    for (int a0 = 0; a0 < AT; a0 += AB) {
      float4 cs[AB][H][2];
      if (!value) {
#pragma unroll
        for (int ab = 0; ab < AB; ++ab) {
          if (a0 + ab >= AT) break;
          const float4* table = reinterpret_cast<const float4*>(r.rope_table + (int64_t)where[a0 + ab].x * (DH / 2) + kq * 4);
#pragma unroll
          for (int t = 0; t < H; ++t) {
            cs[ab][t][0] = table[t * 8];
            cs[ab][t][1] = table[t * 8 + 1];
          }
        }
      }
#pragma unroll
      for (int ab = 0; ab < AB; ++ab) {
        const int at = a0 + ab;
        if (at >= AT) break;
        const int m = row0 + at * 16 + l16;
        if (m >= p.M) continue;
        bf16* row = (bf16*)r.qkv + (int64_t)m * r.ld + col + kq * 4;
        const int64_t page = where[at].y;
        const int slot = where[at].x & 15;
#pragma unroll
        for (int t = 0; t < H; ++t) {
          asm volatile("" : "+a"(acc[hd * 2 * H + t][at]), "+a"(acc[hd * 2 * H + t + H][at]));  // (not all read ahead: they would spill)
          f32x4 a = acc[hd * 2 * H + t][at], b = acc[hd * 2 * H + t + H][at];
          if (p.bias) {
            a += bias[t];
            b += bias[t + H];
          }
          float lo[4] = {a[0], a[1], a[2], a[3]}, hi[4] = {b[0], b[1], b[2], b[3]};
          if (!value) {
            const float4 c0 = cs[ab][t][0], c1 = cs[ab][t][1];
            rotate_pair(a[0], b[0], make_float2(c0.x, c0.y), 0, lo[0], hi[0]);  // (channel 0 and 4, ... of eight are alike but for 3)
            rotate_pair(a[1], b[1], make_float2(c0.z, c0.w), 1, lo[1], hi[1]);
            rotate_pair(a[2], b[2], make_float2(c1.x, c1.y), 2, lo[2], hi[2]);
            rotate_pair(a[3], b[3], make_float2(c1.z, c1.w), odd ? 7 : 3, lo[3], hi[3]);
          }
          bf16x4 l4, h4;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            l4[e] = (bf16)lo[e];
            h4[e] = (bf16)hi[e];
          }
          if (value || kvh < 0) {
            *reinterpret_cast<bf16x4*>(row + t * 16) = l4;
            *reinterpret_cast<bf16x4*>(row + (t + H) * 16) = h4;
          } else {
            const int c = t * 16 + kq * 4;
            uint8_t* pool = (uint8_t*)r.kv.k_pool;
            *reinterpret_cast<bf16x4*>(pool + k_pool_byte(r.kv, page, kvh, slot, 2 * c)) = l4;
            *reinterpret_cast<bf16x4*>(pool + k_pool_byte(r.kv, page, kvh, slot, 2 * c + DH)) = h4;
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// The residual epilogue of a whole tile (no split-K, no bias): out = acc + residual.  The residual of
// half the wave's tile is requested in one go - addresses clamped into the matrix instead of guarded,
// so that nothing but loads stands between the first request and the last - and only then added and
// stored: fetched row block by row block behind guards, the loads of one row block were all that
// was ever in flight, and the eight round trips took 45 us per 256 x 256 tile against 12 us for the
// epilogue without a residual (measured; the registers that held the operand fragments are free here).
template <int AT, int WT>
__device__ __forceinline__ void gemm_epilogue16_residual(const GemmParams& p, f32x4 (&acc)[WT][AT], int row0,
                                                         int col0, int l16, int kq) {
  constexpr int AB = AT > 4 ? (AT + 1) / 2 : AT;  // row blocks per batch
  const int n_last = p.N_store - 4;
#pragma unroll
  for (int a0 = 0; a0 < AT; a0 += AB) {
    f32x4 r[AB][WT];
#pragma unroll
    for (int ab = 0; ab < AB; ++ab) {
      if (a0 + ab >= AT) break;
      const int m = min(row0 + (a0 + ab) * 16 + l16, p.M - 1);
#pragma unroll
      for (int wt = 0; wt < WT; ++wt) {
        const int n = min(col0 + wt * 16 + kq * 4, n_last);
        if (p.res_f32) {
          r[ab][wt] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>((const float*)p.residual + (int64_t)m * p.ldr + n));
        } else {
          const bf16x4 t = *reinterpret_cast<const bf16x4*>((const bf16*)p.residual + (int64_t)m * p.ldr + n);
          r[ab][wt] = f32x4{(float)t[0], (float)t[1], (float)t[2], (float)t[3]};
        }
      }
    }
#pragma unroll
    for (int ab = 0; ab < AB; ++ab) {
      if (a0 + ab >= AT) break;
      const int m = row0 + (a0 + ab) * 16 + l16;
#pragma unroll
      for (int wt = 0; wt < WT; ++wt) {
        const int n = col0 + wt * 16 + kq * 4;
        if (m < p.M && n < p.N_store) {
          const f32x4 v = acc[wt][a0 + ab] + r[ab][wt];
          if (p.out_f32) {
            *reinterpret_cast<f32x4*>((float*)p.out + (int64_t)m * p.ldo + n) = v;
          } else {
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (bf16)v[e];
            *reinterpret_cast<bf16x4*>(p.out + (int64_t)m * p.ldo + n) = o;
          }
        }
      }
    }
  }
}

// Workgroup -> (tile_m, tile_n, split).  The tiles are put in one order - by split, by band of up to four rows of
// tiles, and inside a band column by column - so that any run of consecutive tiles is a compact block: the
// workgroups that make it share a band's activation panels and as few weight panels as there can be.
// Workgroups are dealt round-robin to the 8 XCDs, each with its own L2: an XCD takes runs of as many
// tiles as it has slots, the eight XCDs' runs side by side, and what is left is divided evenly.  Every
// workgroup but the last few of the grid has a tile.  (An earlier numbering gave an XCD rectangles of tiles whose
// corners could lie outside the matrix: the workgroups that found nothing to do sat at regular ids, and
// as the dispatcher hands out ids to the four shader engines of an XCD in turn, two of them got all the
// work: with three or six rows of tiles a launch took twice its time, 121 us against 61 at M = 384 on 10240 x 8192.)
// (The look-up stands in front of a workgroup's first request, so its divisions are by multiplication: x / d =
// umulhi(x, ceil(2^32 / d)) while x * d < 2^32, 0 standing for d = 1 and for divisors where that does not hold.)
__device__ __forceinline__ int divide(int x, int d, unsigned inv) {
  return inv ? (int)__umulhi((unsigned)x, inv) : d == 1 ? x : x / d;
}
__device__ __forceinline__ bool gemm_tile_of_block(const GemmParams& p, int& tile_m, int& tile_n, int& split) {
  const int xcd = blockIdx.x & 7;
  int local = blockIdx.x >> 3;
  int t;
  const int whole = p.chunks << p.chunk_shift;  // tiles of this XCD that come in whole runs
  if (local < whole) {
    const int run = local >> p.chunk_shift;
    t = ((run * 8 + xcd) << p.chunk_shift) + (local - (run << p.chunk_shift));
  } else {
    local -= whole;
    const int q = p.rest >> 3, r = p.rest & 7;
    if (local >= q + (xcd < r ? 1 : 0)) return false;
    t = whole * 8 + xcd * q + min(xcd, r) + local;
  }
  const int per_split = p.tiles_m * p.tiles_n;
  split = divide(t, per_split, p.per_split_inv);
  t -= split * per_split;
  const int tall = (p.band_h + 1) * p.tiles_n, low = p.band_h * p.tiles_n;  // tiles per band
  if (t < p.n_tall * tall) {
    const int band = divide(t, tall, p.tall_inv);
    t -= band * tall;
    tile_n = divide(t, p.band_h + 1, p.h_tall_inv);
    tile_m = band * (p.band_h + 1) + t - tile_n * (p.band_h + 1);
  } else {
    t -= p.n_tall * tall;
    const int band = divide(t, low, p.low_inv);
    t -= band * low;
    tile_n = divide(t, p.band_h, p.h_low_inv);
    tile_m = p.n_tall * (p.band_h + 1) + band * p.band_h + t - tile_n * p.band_h;
  }
  return true;
}

// The same pipeline on v_mfma_f32_16x16x32_bf16: a stage of 32 k is exactly one MFMA k-step, a wave
// tile of (TM*32) x (TN*32) is (TM*2) x (TN*2) accumulators of four registers.  Operand bytes read
// from LDS per flop are the same as with 32x32x16 tiles, but the accumulator traffic in the
// register file is half, and on a power-limited part that buys clock: with random operands an
// MFMA-only loop sustains 2.16 PFLOP/s with 16x16x32 against 1.89 with 32x32x16 (measured).
// Fragments of stage t+1 are read under the MFMAs of stage t (two register sets, the stage loop
// is unrolled by two); one barrier per stage, at its start.
//
// WNT: the weight tiles are requested as non-temporal.  With a single row of tiles (M up to the tile's
// rows: the decode sizes) every weight byte is read by exactly one workgroup, so keeping it in L2
// only evicts what is shared - the activation panel, the split-K partials.  Measured at M = 32 ... 256
// on the 70B shapes: +6 to +12 % on the down projection, +2 to +8 % on gate/up, +1 to +4 % on QKV and
// O.  With more tile rows the weights are shared through L2 and the hint costs 5-10 % on the large
// shapes; the one exception that pays is two tile rows on a wide projection without split-K (gate/up at
// M = 512: the two readers of a weight tile are neighbours in the order of the tiles and run at the same
// time, so the second read still finds the line): -1.8 %.
//
// Tiles of up to 128 x 128 can sum K in chunks (see sum_order_splits): a second set of accumulators (which costs 128 x 128
// its second workgroup per CU, so there are two forms of that).
template <int AT, int WT, int NS>
constexpr bool kChunked = AT * WT <= 12 || (AT == 4 && WT == 4 && NS == 9);

// A workgroup of four waves (2 x 2) makes a tile of BM = 32 AT rows x BN = 32 WT weight rows; a wave, AT x WT
// accumulators.
template <int AT, int WT, int NS, bool WNT, typename Params>
__global__ __launch_bounds__(256) void gemm_mi16_kernel(const Params p) {
  constexpr int BM = AT * 32, BN = WT * 32, BK = 32;
  constexpr int CPR = BK / 8;         // 16-byte chunks per row
  // Rows that share one swizzle value.  A fragment read of this kernel is 16 rows x 4 chunks (lane =
  // chunk * 16 + row); measured with SQ_LDS_BANK_CONFLICT on that pattern: the chunk position must
  // turn every 2 rows to be conflict free (4 LDS cycles per ds_read_b128); turning every 4 rows -
  // right for the 32 rows x 2 chunks of the 32x32 kernels - costs 8 cycles per read here.
  constexpr int RW = 2;
  constexpr int RPI = 64 / CPR;       // rows per DMA instruction
  // DMA instructions per wave and stage.  Where the 2 AT row blocks of the activations do not divide by four, the
  // last waves request rows of the tile a second time, into ring rows that nothing reads (BMR > BM).
  constexpr int IPA = (BM / RPI + 3) / 4, IPW = BN / RPI / 4;
  constexpr int BMR = IPA * 4 * RPI;
  constexpr int STAGE = (BMR + BN) * BK;
  static_assert(WT % 4 == 0, "gate/up pairing");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  bf16* smem = reinterpret_cast<bf16*>(smem_raw);  // [NS][BMR + BN][BK]

  int tile_m, tile_n, split;
  if (!gemm_tile_of_block(p, tile_m, tile_n, split)) return;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = (wave >> 1) * (AT * 16);
  const int wn0 = (wave & 1) * (WT * 16);
  const int l16 = lane & 15;
  const int kq = lane >> 4;
  const int m0 = tile_m * BM;
  const int n0 = tile_n * BN;
  const int kt_begin = split * p.k_tiles_per_split * 2;
  int kt_end = kt_begin + p.k_tiles_per_split * 2;
  if (kt_end > p.k_tiles_total * 2) kt_end = p.k_tiles_total * 2;
  const int n_stages = kt_end - kt_begin;  // even: two stages per 64-wide k-tile

  // DMA addressing: a wave-uniform 64-bit base per operand, which moves one k-stage per request,
  // plus loop-invariant 32-bit per-lane byte offsets (scalar base + vector offset needs no vector
  // arithmetic per load).
  typedef const __attribute__((address_space(1))) char* gptr;
  const int r_in = lane / CPR;
  // Instruction j of an operand lands 1 KiB further on in LDS than instruction 0; that distance
  // rides in the instruction's immediate offset, which also moves the global address, so it is
  // taken out of the per-lane offsets again.  The per-lane offset is zero-extended by the hardware
  // and must not go negative: a constant bias keeps it positive and is subtracted from the bases.
  constexpr int kImmBias = 3 * 1024;
  const int valid = min(BM, p.M - m0), spread = (1 << (31 - __builtin_clz(valid))) - 1;
  unsigned a_goff[IPA];  // bytes
#pragma unroll
  for (int j = 0; j < IPA; ++j) {
    const int row = (wave * IPA + j) * RPI + r_in;
    const int c_sw = (lane % CPR) ^ ((row / RW) % CPR);
    // rows past M are computed but never stored; they re-read the tile's valid rows in turn (all of
    // them reading the last valid row makes one hot line for every workgroup of the launch)
    const int m = row < valid ? row : row & spread;
    a_goff[j] = 2u * (unsigned)(operand_row_offset(p.a_lay, m) + c_sw * 8) + (unsigned)(kImmBias - j * 1024);
  }
  // weight rows need no clamp; the swizzle term (row / RW) % CPR does not depend on the row block j
  // (RPI is a multiple of RW * CPR)
  static_assert(RPI % (RW * CPR) == 0, "the swizzle repeats per row block");
  unsigned w_goff[IPW];
#pragma unroll
  for (int j = 0; j < IPW; ++j) {
    const int row = (wave * IPW + j) * RPI + r_in;
    const int c_sw = (lane % CPR) ^ ((row / RW) % CPR);
    w_goff[j] = 2u * (unsigned)(operand_row_offset(p.w_lay, row) + c_sw * 8) + (unsigned)(kImmBias - j * 1024);
  }
  const int64_t a_step = 2 * p.a_lay.kb, w_step = 2 * p.w_lay.kb;  // bytes per k-stage
  // the stage being requested: global bases, index and ring slot; past the last stage the bases
  // stay put, so the tail re-fetches the last stage (valid memory, never read)
  gptr a_req = (gptr)(p.A + operand_row_offset(p.a_lay, m0) + (int64_t)kt_begin * p.a_lay.kb) - kImmBias;
  gptr w_req = (gptr)(p.W + operand_row_offset(p.w_lay, n0) + (int64_t)kt_begin * p.w_lay.kb) - kImmBias;
  int req_t = 0, req_slot = 0;
  constexpr int N_DMA = IPA + IPW;
  // One DMA instruction: 64 lanes x 16 bytes from (scalar base + per-lane byte offset) into 1 KiB
  // of LDS at lds_addr.  Written as assembly to get the scalar-base form (no vector address
  // arithmetic per load); M0 carries the LDS address, and every DMA of this kernel goes through
  // here, so nothing else depends on M0.
  auto dma_aim = [](unsigned lds_addr) { asm volatile("s_mov_b32 m0, %0\n\ts_nop 0" ::"s"(lds_addr) : "memory"); };
#define TDP_DMA16(lane_off, base, imm) \
  asm volatile("global_load_lds_dwordx4 %0, %1 offset:%2" ::"v"(lane_off), "s"(base), "n"(imm) : "memory")
#define TDP_DMA16W(lane_off, base, imm)                                                                              \
  do {                                                                                                               \
    if constexpr (WNT)                                                                                               \
      asm volatile("global_load_lds_dwordx4 %0, %1 offset:%2 nt" ::"v"(lane_off), "s"(base), "n"(imm) : "memory");   \
    else                                                                                                             \
      asm volatile("global_load_lds_dwordx4 %0, %1 offset:%2" ::"v"(lane_off), "s"(base), "n"(imm) : "memory");      \
  } while (0)
  const unsigned ring_base = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)smem_raw;
  static_assert(IPA <= 4 && IPW <= 4, "immediate offsets up to 3 KiB");
  // instruction j of the requested stage: activations first, then weights; M0 is aimed at the
  // wave's first KiB of each operand once per stage
  auto dma_one = [&](int j) {
    const unsigned ring = ring_base + req_slot * (STAGE * 2);
    if (j == 0) dma_aim(ring + (wave * IPA * RPI * BK) * 2);
    if (j == IPA) dma_aim(ring + (BMR * BK + wave * IPW * RPI * BK) * 2);
    switch (j < IPA ? j : j - IPA) {
      case 0: if (j < IPA) TDP_DMA16(a_goff[0], a_req, 0); else TDP_DMA16W(w_goff[0], w_req, 0); break;
      case 1: if (j < IPA) TDP_DMA16(a_goff[1 % IPA], a_req, 1024); else TDP_DMA16W(w_goff[1 % IPW], w_req, 1024); break;
      case 2: if (j < IPA) TDP_DMA16(a_goff[2 % IPA], a_req, 2048); else TDP_DMA16W(w_goff[2 % IPW], w_req, 2048); break;
      default: if (j < IPA) TDP_DMA16(a_goff[3 % IPA], a_req, 3072); else TDP_DMA16W(w_goff[3 % IPW], w_req, 3072); break;
    }
  };
#undef TDP_DMA16
#undef TDP_DMA16W
  auto dma_advance = [&]() {
    ++req_t;
    if (req_t < n_stages) {
      a_req += a_step;
      w_req += w_step;
    }
    req_slot = req_slot + 1 == NS ? 0 : req_slot + 1;
  };
  auto dma_stage = [&]() {
#pragma unroll
    for (int j = 0; j < N_DMA; ++j) dma_one(j);
    dma_advance();
  };

  f32x4 acc[WT][AT];
#pragma unroll
  for (int wt = 0; wt < WT; ++wt)
#pragma unroll
    for (int at = 0; at < AT; ++at) acc[wt][at] = f32x4{0.f, 0.f, 0.f, 0.f};

  // fragment reads: lane (l16, kq) supplies row l16 of a 16-row tile, k = kq*8 .. +8 of the stage
  // Tile wt / at lies 16 rows = 16 * BK elements further on and 16 is a multiple of RW * CPR, so
  // the swizzle term is the lane's alone: one base per operand, the rest are immediate offsets.
  static_assert(16 % (RW * CPR) == 0, "swizzle repeats every 16 rows");
  const int swz = (kq ^ ((l16 / RW) % CPR)) << 3;
  const int w_off = (BMR + wn0 + l16) * BK + swz;
  const int a_off = (wm0 + l16) * BK + swz;
  bf16x8 wf[2][WT], af[2][AT];
  constexpr int PENDING = (NS - 2) * N_DMA;
  int rd_slot = 0;  // ring slot of the stage whose fragments are read next
  int w_next = w_off, a_next = a_off;  // this lane's fragments in that slot (element offsets into smem)
  auto read_frags = [&](int set) {
    const bf16* base = smem + rd_slot * STAGE;
#pragma unroll
    for (int wt = 0; wt < WT; ++wt) wf[set][wt] = ld_bf16x8(base + w_off + wt * 16 * BK);
#pragma unroll
    for (int at = 0; at < AT; ++at) af[set][at] = ld_bf16x8(base + a_off + at * 16 * BK);
  };
  // One stage: its fragments are in register set `set`; the next stage was requested NS-2
  // barriers ago.  The MFMAs are inline assembly so that every accumulator stays in place in its
  // AGPRs (left to itself the register allocator shuttles the 64 accumulator tuples through
  // VGPRs); issue order is therefore explicit: everything that is not an MFMA - the WT + AT fragment reads
  // and the N_DMA requests of the stages ahead, then the stage's bookkeeping - goes behind single MFMAs, a
  // few instructions at a time, so that it issues while the matrix pipe is busy instead of in a gap of
  // the MFMA stream, and is pinned there by scheduling barriers.
  constexpr int N_MFMA = AT * WT;
  constexpr bool GROUPED = AT >= 4 && AT <= WT && N_DMA <= WT;  // a weight read, an activation read, a request per MFMA group
  constexpr int N_OPS = WT + AT + N_DMA;
  auto stage = [&](int set) {
    // vmcnt: this wave's loads of the next stage have landed; lgkmcnt: its reads of this stage are
    // complete, so after the barrier this stage's buffer may be refilled and the next one read
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(PENDING) : "memory");
#pragma unroll
    for (int i = 0; i < N_MFMA; ++i) {
      const int wt = i / AT, at = i % AT;
      asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[wt][at]) : "v"(wf[set][wt]), "v"(af[set][at]));
      if constexpr (GROUPED) {
        if (at < 3) __builtin_amdgcn_sched_barrier(0);
        if (at == 0) wf[set ^ 1][wt] = ld_bf16x8(smem + w_next + wt * 16 * BK);
        if (at == 1 && wt < AT) af[set ^ 1][wt] = ld_bf16x8(smem + a_next + wt * 16 * BK);
        if (at == 2 && wt < N_DMA) dma_one(wt);
        if (at < 3) __builtin_amdgcn_sched_barrier(0);
      } else {
        // operations first .. last - 1 of the list (weight reads, activation reads, requests) are this MFMA's
        const int first = (i * N_OPS + N_MFMA - 2) / (N_MFMA - 1), last = ((i + 1) * N_OPS + N_MFMA - 2) / (N_MFMA - 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int op = first; op < last && op < N_OPS; ++op) {
          if (op < WT) wf[set ^ 1][op] = ld_bf16x8(smem + w_next + op * 16 * BK);
          else if (op < WT + AT) af[set ^ 1][op - WT] = ld_bf16x8(smem + a_next + (op - WT) * 16 * BK);
          else dma_one(op - WT - AT);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      // the bookkeeping, behind MFMAs of the last group that carry nothing else: the request side moves on one
      // stage, and so do the fragment offsets.  (The empty statements make the new values exist here
      // rather than wherever their next use is.)
      if (i == (GROUPED ? (WT - 1) * AT + 3 : N_MFMA - 1)) {
        __builtin_amdgcn_sched_barrier(0);
        ++req_t;
        if (req_t < n_stages) {
          a_req += a_step;
          w_req += w_step;
        }
        asm volatile("" : "+s"(a_req), "+s"(w_req), "+s"(req_t));
        __builtin_amdgcn_sched_barrier(0);
      }
      if (i == (GROUPED ? (WT - 1) * AT + (AT > 4 ? 4 : 3) : N_MFMA - 1)) {
        __builtin_amdgcn_sched_barrier(0);
        req_slot = req_slot + 1 == NS ? 0 : req_slot + 1;
        rd_slot = rd_slot + 1 == NS ? 0 : rd_slot + 1;
        asm volatile("" : "+s"(req_slot), "+s"(rd_slot));
        __builtin_amdgcn_sched_barrier(0);
      }
      if (i == (GROUPED ? (WT - 1) * AT + (AT > 5 ? 5 : AT > 4 ? 4 : 3) : N_MFMA - 1)) {
        __builtin_amdgcn_sched_barrier(0);
        w_next = rd_slot * STAGE + w_off;
        a_next = rd_slot * STAGE + a_off;
        asm volatile("" : "+v"(w_next), "+v"(a_next));
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };

  if (n_stages > 0) {
#pragma unroll
    for (int t = 0; t < NS - 1; ++t) dma_stage();
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(PENDING) : "memory");
    read_frags(0);
    rd_slot = 1 % NS;
    w_next = rd_slot * STAGE + w_off;
    a_next = rd_slot * STAGE + a_off;
    dma_stage();
  }
  if constexpr (kChunked<AT, WT, NS>) {
    // In chunks: what split-K workgroups would leave as partials is added up here in the same order (the requests run on
    // across the ends of the chunks).
    const int chunk = p.k_tiles_per_chunk > 0 ? 2 * p.k_tiles_per_chunk : n_stages;
    f32x4 total[WT][AT];
    for (int t = 0; t < n_stages;) {
      const int end = min(t + chunk, n_stages);
      const bool first = t == 0;
      for (; t < end; t += 2) {
        stage(0);
        stage(1);
      }
      if (end == n_stages && first) break;  // one chunk: the accumulators are the sum
      asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");  // MFMA -> accumulator read, which the compiler cannot see
#pragma unroll
      for (int wt = 0; wt < WT; ++wt)
#pragma unroll
        for (int at = 0; at < AT; ++at) {
          // (pinned on both sides: the accumulators live in the inline MFMAs' registers)
          asm volatile("" : "+a"(acc[wt][at]));
          total[wt][at] = first ? acc[wt][at] : total[wt][at] + acc[wt][at];
          acc[wt][at] = end == n_stages ? total[wt][at] : f32x4{0.f, 0.f, 0.f, 0.f};
          asm volatile("" : "+a"(acc[wt][at]));
        }
      asm volatile("s_nop 7" ::: "memory");  // accumulator write -> MFMA
    }
  } else {
    for (int t = 0; t < n_stages; t += 2) {
      stage(0);
      stage(1);
    }
  }
  // loads still in flight target LDS only; they must land before the workgroup's LDS is released.
  // The nops cover the MFMA -> accumulator-read distance, which the compiler cannot see.
  asm volatile("s_waitcnt vmcnt(0)\n\ts_nop 15\n\ts_nop 15" ::: "memory");
  if constexpr (std::is_same_v<Params, GemmRotateParams>) {
    if (p.rot.kv.head_dim == 128) gemm_epilogue16_rotate<AT, WT, 4>(p, acc, m0 + wm0, n0 + wn0, l16, kq);
    else gemm_epilogue16_rotate<AT, WT, 2>(p, acc, m0 + wm0, n0 + wn0, l16, kq);
  } else if constexpr (std::is_same_v<Params, GemmMaxParams>) {
    gemm_epilogue16_max<AT, WT>(p, acc, m0 + wm0, n0 + wn0, l16, kq);
  } else if (p.splits == 1 && p.epilogue == EPI_RESIDUAL && !p.bias && p.N_store >= 4) {
    gemm_epilogue16_residual<AT, WT>(p, acc, m0 + wm0, n0 + wn0, l16, kq);
  } else {
    gemm_epilogue16<AT, WT>(p, acc, m0 + wm0, n0 + wn0, l16, kq, split);
  }
}

// Sum the split-K partials and apply the epilogue.  One thread per 4 output columns.
__global__ __launch_bounds__(256) void gemm_reduce_kernel(const GemmParams p, int out_cols) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int groups = out_cols / 4;
  if (idx >= (int64_t)p.M * groups) return;
  const int m = (int)(idx / groups);
  const int j = (int)(idx % groups) * 4;
  auto sum_at = [&](int n) {
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    for (int z = 0; z < p.splits; ++z)
      s += *reinterpret_cast<const f32x4*>(p.ws + ((int64_t)z * p.M + m) * p.Npad + n);
    return s;
  };
  if (p.epilogue == EPI_SWIGLU) {
    const int ng = (j / 32) * 64 + (j % 32);
    f32x4 g = sum_at(ng), u = sum_at(ng + 32);
    bf16x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (bf16)(silu_f(g[e]) * u[e]);
    *reinterpret_cast<bf16x4*>(p.out + operand_offset(p.u_lay, m, j)) = o;
  } else {
    const f32x4 t = sum_at(j);
    float v[4] = {t[0], t[1], t[2], t[3]};
    store_row4(p, m, j, v);
  }
}

// Kernel variants; 1 .. kGemmTileMax can be selected by callers (GemmArgs::force_tile), the planner chooses among
// all.  A tile has as many rows as the batch needs, in steps of 32: rows past M cost as much as real ones
// (matrix pipe, LDS reads, power), and with tiles of 128 and 256 rows alone a batch of 307 paid for 512 (gate/up 57344 x
// 8192: 366 us, with 2 x 160 rows 278; M = 384: 371 -> 308; M = 200: 202 -> 180).  128 weight rows per
// tile instead of 256 where the weights are what counts (M up to 128: twice the workgroups, half the split-K
// factor where the order of the sums is free; M = 48, 22016 x 4096: 45 -> 39 us) and
// between 160 and 256 rows on narrow projections.  The ring takes what LDS there is; two or three workgroups
// per CU where a tile is small enough (their fill and epilogue then overlap the neighbour's stages).
enum GemmKind { kOrdinary, kRotating, kMaximum, kKinds };
struct TileInfo {
  int at, wt, ns, wg_per_cu;
  bool chunked;           // can sum K in chunks
  double stage_us;        // a 32-wide stage of one tile on a CU, the matrix pipe's part (see plan_cost)
  const void* kernel[kKinds][2];  // ordinary / non-temporal weight requests; null: see gemm_can_rotate
  int bm() const { return at * 32; }
  int bn() const { return wt * 32; }
  int ring_rows() const { return (at * 2 + 3) / 4 * 64 + bn(); }  // rows of a ring stage (see IPA)
  int lds_bytes() const { return ns * ring_rows() * 64; }
};
template <int AT, int WT, int NS, bool WNT, typename Params>
static const void* kernel_of() {
  if constexpr (std::is_same_v<Params, GemmRotateParams> && WT != 8) return nullptr;
  else return reinterpret_cast<const void*>(&gemm_mi16_kernel<AT, WT, NS, WNT, Params>);
}
#define TDP_KERNELS(AT, WT, NS, PARAMS) {kernel_of<AT, WT, NS, false, PARAMS>(), kernel_of<AT, WT, NS, true, PARAMS>()}
#define TDP_TILE(AT, WT, NS, PER_CU, US)                                                                   \
  {AT, WT, NS, PER_CU, kChunked<AT, WT, NS>, US,                                                           \
   {TDP_KERNELS(AT, WT, NS, GemmParams), TDP_KERNELS(AT, WT, NS, GemmRotateParams), TDP_KERNELS(AT, WT, NS, GemmMaxParams)}}
static const TileInfo kTiles[] = {
    {0, 0, 0, 0, false, 0.0, {}},
    TDP_TILE(8, 8, 4, 1, 0.425),  // 1: 256 x 256
    TDP_TILE(4, 8, 6, 1, 0.252),  // 2: 128 x 256
    TDP_TILE(4, 4, 4, 2, 0.129),  // 3: 128 x 128
    // 224, 192, 160 x 256
    TDP_TILE(7, 8, 4, 1, 0.346), TDP_TILE(6, 8, 5, 1, 0.337), TDP_TILE(5, 8, 5, 1, 0.266),
    // 256, 224, 160, 96 x 128
    TDP_TILE(8, 4, 6, 1, 0.244), TDP_TILE(7, 4, 6, 1, 0.202), TDP_TILE(5, 4, 7, 1, 0.168), TDP_TILE(3, 4, 8, 1, 0.097),
    // 128 x 128 with one workgroup per CU (sums in chunks); 64, 32 x 128
    TDP_TILE(4, 4, 9, 1, 0.129),
    TDP_TILE(2, 4, 6, 2, 0.079), TDP_TILE(1, 4, 4, 3, 0.0415),
};
#undef TDP_TILE
#undef TDP_KERNELS
constexpr int kTileCount = sizeof(kTiles) / sizeof(kTiles[0]);
// The 128 x 128 tile that has room for chunked sums is used for those only: otherwise two workgroups per CU (tile 3) are 7 to 15 %
// faster at the same split-K factor (1367 pairs of launches, M from 1 to 16384).
constexpr int kChunksOnlyTile = 11;

static bool g_print_plan = false;  // tuning aid, read from the environment once (gemm_setup)

hipError_t gemm_setup() {
  static std::once_flag once;
  static hipError_t result = hipSuccess;
  std::call_once(once, [] {
    g_print_plan = getenv("TDP_GEMM_PLAN") != nullptr;
    hipError_t e;
    e = hipSuccess;
    for (int i = 1; i < kTileCount; ++i)
      for (const auto& kind : kTiles[i].kernel)
        for (const void* kernel : kind)
          if (kernel && e == hipSuccess)
            e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kTiles[i].lds_bytes());
    result = e;
  });
  return result;
}

// Estimated time in us of a launch with this tile and split-K factor (per = 64-wide k-tiles of a split).  An XCD
// makes its eighth of the tiles in rounds of 32 CUs x wg_per_cu; a 32-wide stage of a round costs the matrix
// pipe, the LDS fill of a CU, the XCD's reads through its fabric port, the chip's reads of the weights and the
// latency the ring has to cover - none of which hides behind another entirely, hence the power sum;
// a round ends with its epilogue; split-K adds the fp32 partials' round trip and, where no later kernel sums them,
// a reduce launch.  The constants are a least-squares fit to 10,000 launches timed on cold weights (19 projection
// shapes, M from 4 to 19346, 1 to 16 splits): the tile and factor that this picks are on average 1.3 % slower
// than the fastest measured, against 32 % for the rule it replaces (M <= 128, narrow, else; rounds of k-tiles).  Up to 128
// rows the choice is narrower, see sum_order_splits.
// `rotated`: the QKV projection of a stage where its sums are free.  It stores fp32 whether it is split or not, so each
// store costs alike (0.6 us per million elements), and each split more costs the rotation 0.5 us and 0.33 per million
// elements (128 to 512 rows, seven shapes).  Charged for the store of a split alone, like the other projections, 13B at 512 rows took
// 256 x 128 tiles unsplit where 256 x 256 in two splits are faster (with the rotation 79.2 + 51.2 us against 70.5 + 51.9); Qwen at
// 512 rows 56.0 + 16.9 against 45.3 + 17.8, 70B at 384 rows 87.1 + 15.8 against 67.5 + 18.4.  Over 264 cases with M from 129 to
// 16384 the choice was 2.5 % slower than the fastest, now 0.2 %.
// (These costs are of the projection with a rotation kernel behind it.  An unsplit tile of 256 weight rows of a 16-bit prefill stores no
// fp32 and has none, see gemm_can_rotate; the plan, which decode and 8-bit caches share, does not count that in, so it can keep a split
// or a tile of 128 weight rows where rotating in the epilogue would be a little ahead.)
static double plan_cost(const TileInfo& ti, int64_t M, int64_t Npad, int per, int splits, int epilogue, bool defer,
                        bool rotated) {
  const double tm = (double)((M + ti.bm() - 1) / ti.bm()), tn = (double)(Npad / ti.bn());
  const double tiles = tm * tn * splits;
  const int64_t per_xcd = ((int64_t)tiles + 7) / 8, slots = 32 * ti.wg_per_cu;
  const int64_t full = (per_xcd - 1) / slots, last = per_xcd - full * slots;  // full rounds, tiles of the last one
  const double band = tm / (double)(((int64_t)tm + 3) / 4);                   // rows of tiles in a band
  const double mfma = ti.at * ti.wt;
  const double a_rows = ti.ring_rows() - ti.bn(), bn = ti.bn();
  auto stage = [&](int64_t n) {  // n tiles of the XCD at once
    const double per_cu = (double)((n + 31) / 32);
    const double cols = ceil((double)n / band);
    const double on_chip = (double)(8 * n) < tiles ? (double)(8 * n) : tiles;
    const double terms[5] = {per_cu * ti.stage_us,
                             per_cu * ti.ring_rows() * (0.064 / 117.6),
                             ((band < n ? band : (double)n) * a_rows + cols * bn) * (512e-6 / 11.1),
                             on_chip / tm * bn * (64e-6 / 18.3),
                             0.21 / (ti.ns - 1)};
    double sum = 0;
    for (double t : terms) sum += t * sqrt(t);  // power 1.5
    return cbrt(sum * sum);
  };
  auto epi = [&](int64_t n) { return 0.94 + 0.12 * mfma * (double)((n + 31) / 32); };
  double us = 1.9 + full * (2 * per * stage(slots) + epi(slots)) + 2 * per * stage(last) + epi(last);
  const double elems = M * (double)Npad;
  if (rotated) {
    us += 0.6e-6 * splits * elems + (splits - 1) * (0.5 + 0.33e-6 * elems);
  } else if (splits > 1) {
    us += 0.81e-6 * splits * elems + 0.15 * splits;
    if (!defer) us += 5.4;
    else if (epilogue == EPI_STORE) us += 0.4e-6 * (splits - 1) * elems;  // read by the rotation
  }
  return us * (1.0 + 0.004 * tm);  // ties: fewer rows of tiles, the weights are read fewer times
}

// The order in which a projection of up to 128 rows sums over K, as a split-K factor.  fp32 sums in another order differ in
// their last bits, which the bf16 roundings behind them carry through every layer: about 0.5 % of a
// hidden state after a few layers, as much as bf16 itself costs, and enough to turn a greedy token between near-equal
// logits (measured once in four runs: 2 of 48 over four layers and a vocabulary of 32000).  The distance to the 64-bit result is the
// same in either order.  What the rule below is for is nothing but this: decode batches of up to 128 rows give the bits that they
// gave when every such launch was made of 128 x 256 tiles, one per CU (in super-blocks dealt to the XCDs, 1.8 us per round
// of k-tiles plus the partials' round trip - the cost that it minimises), whatever tile makes the sum now: as that many split-K
// workgroups or, where the tile has registers for it, chunk by chunk in one.  The factor depends on M, N, K and the
// workspace, so a request's bits may change with the batch around it (4096 x 4096 is 16 splits up to 64 rows, 11 at 128), and above
// 128 rows the plan is free.  Keeping it costs what a freer factor would gain: 13B decode, 128 rows, two layers 1206 against 1172
// us; 7B token step, 48 rows, 796 against 738.
// Short sums (K <= 1024) are free: there another order moves a hidden state by 3e-5 at most, and a freer factor takes a
// two-layer stage of hidden size 256 from 66 to 59 us.
constexpr int kSumOrderRows = 128, kSumOrderKTiles = 16;
static int sum_order_splits(int64_t M, int64_t Npad, int k_tiles, int64_t workspace_elems) {
  const int tn = (int)(Npad / 256);
  int most = k_tiles / 4 < 16 ? (k_tiles / 4 > 0 ? k_tiles / 4 : 1) : 16;
  if (most > k_tiles) most = k_tiles;
  int best = 1;
  double best_cost = 1e300;
  for (int sp = 1; sp <= most; ++sp) {
    if (sp > 1 && sp * M * Npad > workspace_elems) break;
    const int per = (k_tiles + sp - 1) / sp;
    if ((k_tiles + per - 1) / per != sp) continue;
    for (int lg = 5; lg >= 0; --lg) {
      const int size = 1 << lg, n_sb = (tn + size - 1) / size;
      int load[8] = {0, 0, 0, 0, 0, 0, 0, 0}, longest = 0;
      for (int g = 0; g < n_sb * sp; ++g) {
        const int sb = g % n_sb;
        load[g & 7] += (sb + 1) * size <= tn ? size : tn - sb * size;
      }
      for (int x : load) longest = x > longest ? x : longest;
      double cost = (double)((longest + 31) / 32) * (per + 6.0);
      if (sp > 1) cost += 1.1e-6 * sp * M * (double)Npad + 2.0;
      cost *= 1.0 + 0.02 * (5 - lg);
      if (cost < best_cost) {
        best_cost = cost;
        best = sp;
      }
    }
  }
  return best;
}

static GemmPlan search_plan(const GemmPlanKey& a) {
  GemmPlan plan{0, 1, 0};
  const int k_tiles_total = (int)(a.Kpad / 64);
  const bool forced = a.force_tile >= 1 && a.force_tile <= kGemmTileMax;
  double best_cost = 1e300;
  // up to kSumOrderRows rows the order of the sums is given, and only how it is made is chosen
  const int order = a.force_splits <= 0 && !forced && a.M <= kSumOrderRows && k_tiles_total > kSumOrderKTiles
                        ? sum_order_splits(a.M, a.Npad, k_tiles_total, a.workspace_elems) : 0;
  const bool rotated = a.defer && a.epilogue == EPI_STORE && order == 0;
  for (int t = forced ? a.force_tile : 1; t <= (forced ? a.force_tile : kTileCount - 1); ++t) {
    const int64_t tiles1 = (int64_t)((a.M + kTiles[t].bm() - 1) / kTiles[t].bm()) * ((a.Npad + kTiles[t].bn() - 1) / kTiles[t].bn());
    const int k_splits_max = k_tiles_total / 2 < 16 ? (k_tiles_total / 2 > 0 ? k_tiles_total / 2 : 1) : 16;
    int sp = a.force_splits > 0 ? a.force_splits : 1, sp_max = a.force_splits > 0 ? a.force_splits : k_splits_max;
    if (order > 0) sp_max = order;
    if (sp > k_tiles_total) sp = sp_max = k_tiles_total;
    for (; sp <= sp_max; ++sp) {
      const int per = (k_tiles_total + sp - 1) / sp;
      const int real_sp = (k_tiles_total + per - 1) / per;
      const bool chunks = order > 1 && real_sp == 1;
      if (real_sp != sp && a.force_splits <= 0) continue;  // same schedule as a smaller factor
      if (order > 1 && sp != order && (sp > 1 || !kTiles[t].chunked)) continue;
      if (t == kChunksOnlyTile && !chunks && !forced) continue;
      if (real_sp > 1 && (int64_t)real_sp * a.M * a.Npad > a.workspace_elems) break;
      // (four rounds of tiles: nothing is left for a split to gain)
      if (real_sp > 1 && a.force_splits <= 0 && order == 0 && tiles1 * real_sp > 1024 * kTiles[t].wg_per_cu) break;
      double cost = plan_cost(kTiles[t], a.M, a.Npad, per, real_sp, a.epilogue, a.defer, rotated);
      // (chunks: the sums between them stop the matrix pipe, and a workgroup's waves do it together; 128 x 15360 x 5120 in
      // two rows of 64 x 128: 48.6 us where the estimate is 40, against 39.4 as four splits)
      if (chunks) cost *= 1.1;
      if (cost < best_cost) {
        best_cost = cost;
        plan = GemmPlan{t, real_sp, chunks ? (k_tiles_total + order - 1) / order : 0};
      }
    }
  }
  if (plan.tile == 0) plan = GemmPlan{forced ? a.force_tile : 1, 1, 0};  // the workspace holds no such split
  return plan;
}

// The search costs tens of microseconds on the host and its answer depends only on the problem's shape, so it
// is remembered (a serving loop asks for the same few shapes every step).
GemmPlan gemm_plan(const GemmPlanKey& key) {
  struct Hash {
    size_t operator()(const GemmPlanKey& k) const {
      uint64_t h = 0x9e3779b97f4a7c15ull;
      for (uint64_t v : {(uint64_t)k.M, (uint64_t)k.force_tile, (uint64_t)k.force_splits, (uint64_t)(k.epilogue * 2 + k.defer),
                         (uint64_t)k.Npad, (uint64_t)k.Kpad, (uint64_t)k.workspace_elems})
        h = (h ^ v) * 0xff51afd7ed558ccdull + (h >> 29);
      return (size_t)h;
    }
  };
  static std::mutex mutex;
  static std::unordered_map<GemmPlanKey, GemmPlan, Hash> cache;
  {
    std::lock_guard<std::mutex> lock(mutex);
    const auto it = cache.find(key);
    if (it != cache.end()) return it->second;
  }
  const GemmPlan plan = search_plan(key);
  std::lock_guard<std::mutex> lock(mutex);
  if (cache.size() < 65536) cache[key] = plan;
  return plan;
}

bool gemm_form_fits(const GemmPlan& f, int M, int64_t Npad, int64_t Kpad, int64_t workspace_elems) {
  const int k_tiles = (int)(Kpad / 64);
  if (f.tile < 1 || f.tile >= kTileCount || f.splits < 1 || f.splits > k_tiles || f.chunk < 0) return false;
  const int per = (k_tiles + f.splits - 1) / f.splits;
  if ((k_tiles + per - 1) / per != f.splits) return false;  // the last splits would have nothing to sum
  if (f.chunk > 0 && (f.splits > 1 || !kTiles[f.tile].chunked)) return false;
  return f.splits == 1 || f.splits * (int64_t)M * Npad <= workspace_elems;
}

void gemm_tile_size(int tile, int* rows, int* weight_rows) {
  *rows = kTiles[tile].bm();
  *weight_rows = kTiles[tile].bn();
}

static GemmPlan plan_of(const GemmArgs& a) {
  const bool defer = a.splits_used != nullptr && a.epilogue != EPI_SWIGLU;
  return a.form.tile ? a.form : gemm_plan({a.M, a.force_tile, a.force_splits, a.epilogue, defer, a.Npad, a.Kpad, a.workspace_elems});
}

// (A wave of a tile of 256 weight rows has 128 columns, whole heads.  Not for 8-bit pools: with the conversion in it the epilogue is too
// long to be unrolled, and accumulators that are indexed at run time live in memory: 20 times the time.)
bool gemm_can_rotate(const GemmArgs& a) {
  const GemmPlan plan = plan_of(a);
  return a.epilogue == EPI_STORE && plan.splits == 1 && kTiles[plan.tile].kernel[kRotating][0];
}

hipError_t launch_gemm(const GemmArgs& a, hipStream_t s) {
  if (a.M <= 0) return hipSuccess;
  GemmParams p;
  p.A = (const bf16*)a.A;
  p.W = (const bf16*)a.W;
  p.out = (bf16*)a.out;
  p.residual = a.residual;
  p.bias = a.epilogue == EPI_SWIGLU ? nullptr : a.bias;
  p.out_f32 = a.epilogue == EPI_SWIGLU ? 0 : a.out_f32;
  p.res_f32 = a.residual_f32;
  p.ws = a.workspace;
  p.a_lay = a.a_layout;
  p.w_lay = layout_weights(a.Kpad);
  p.u_lay = a.u_layout;
  p.Kpad = a.Kpad;
  p.Npad = a.Npad;
  p.ldo = a.ldo;
  p.ldr = a.ldr;
  p.M = a.M;
  p.N_store = a.N_store;
  p.epilogue = a.epilogue;
  p.k_tiles_total = (int)(a.Kpad / 64);
  const bool defer = a.splits_used != nullptr && a.epilogue != EPI_SWIGLU;
  const GemmPlan plan = plan_of(a);
  const TileInfo& ti = kTiles[plan.tile];
  const int splits = plan.splits;
  p.tiles_m = (a.M + ti.bm() - 1) / ti.bm();
  p.tiles_n = (int)(a.Npad / ti.bn());
  p.k_tiles_per_split = (p.k_tiles_total + splits - 1) / splits;
  p.splits = splits;
  p.k_tiles_per_chunk = plan.chunk;
  const bool maximum = a.row_max && splits == 1 && a.epilogue == EPI_STORE && a.out_f32 && !a.bias;
  if (a.row_max_width) *a.row_max_width = maximum ? ti.bn() / 2 : 0;
  const int bands = (p.tiles_m + 3) / 4;
  p.band_h = p.tiles_m / bands;
  p.n_tall = p.tiles_m % bands;
  const int tiles = p.tiles_m * p.tiles_n * splits;
  p.chunk_shift = 5 + (ti.wg_per_cu > 2 ? 2 : ti.wg_per_cu - 1);  // (an XCD's slots, or the next power of two)
  p.chunks = tiles >> (3 + p.chunk_shift);
  p.rest = tiles - (p.chunks << (3 + p.chunk_shift));
  auto inverse = [&](int64_t d) { return d > 1 && d * tiles < (1ll << 32) ? (unsigned)(((1ll << 32) + d - 1) / d) : 0u; };
  p.per_split_inv = inverse((int64_t)p.tiles_m * p.tiles_n);
  p.tall_inv = inverse((int64_t)(p.band_h + 1) * p.tiles_n);
  p.low_inv = inverse((int64_t)p.band_h * p.tiles_n);
  p.h_tall_inv = inverse(p.band_h + 1);
  p.h_low_inv = inverse(p.band_h);
  if (g_print_plan)
    fprintf(stderr, "gemm plan: M=%d N=%lld K=%lld tile=%d tiles=%dx%d splits=%d (k-tiles %d each)\n",
            a.M, (long long)a.Npad, (long long)a.Kpad, plan.tile, p.tiles_m, p.tiles_n, splits, p.k_tiles_per_split);
  dim3 grid((tiles + 7) / 8 * 8);
  // a single row of tiles reads every weight byte once: request them as non-temporal (also two rows of a
  // wide projection, see the kernel's comment)
  const bool wnt = p.tiles_m == 1 || (p.tiles_m == 2 && a.Npad >= 32768 && splits == 1);
  auto launch = [&](GemmKind kind, auto params) {
    void* args[] = {&params};
    return hipLaunchKernel(ti.kernel[kind][wnt ? 1 : 0], grid, dim3(256), args, ti.lds_bytes(), s);
  };
  hipError_t e = a.rotation ? launch(kRotating, GemmRotateParams{p, *a.rotation})
                 : maximum  ? launch(kMaximum, GemmMaxParams{p, a.row_max})
                            : launch(kOrdinary, p);
  if (e != hipSuccess) return e;
  if (a.splits_used) *a.splits_used = defer ? splits : 1;
  if (splits > 1 && !defer) {
    const int out_cols = a.N_store;  // (gated epilogue: columns of the result, half the weight rows)
    const int64_t n_thr = (int64_t)a.M * (out_cols / 4);
    gemm_reduce_kernel<<<(unsigned)((n_thr + 255) / 256), 256, 0, s>>>(p, out_cols);
    e = hipGetLastError();
  }
  return e;
}

}  // namespace tdp
