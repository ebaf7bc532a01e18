// TQ4 encode-and-append: each 256-element K or V vector is divided by its
// norm, rotated by H_256 S / 16 (unnormalised Hadamard matrix H_256, random
// signs S) and every rotated coordinate replaced by the index of one of 16
// shared centroids (Sec. 3.1, eq. codec).  The indices are packed eight per
// u32 word and stored with the fp16 norm at the vector's page slot
// (Appendix A, Table codec; Background, page table).
//
// A wave transforms four vectors at a time, one per row of 16 lanes (see
// jfkv_fwht.h); two 16-byte loads per lane fetch a row's vector.  The norm
// is a wave-wide sum of squares: IEEE addition commutes, so every lane of the
// butterfly reduction ends with the same sum.
//
// What bounds the kernels: vector issue, then HBM.  Per vector ~80 vector
// instructions and 4 LDS reads (~146 and ~25 with a lane per four elements).
// K and V of 262,143 rows of 4 heads: 460 -> 314 us (2.9 -> 4.3 TB/s);
// reconstruction of 2 heads over 196,608 positions: 169 -> 108 us (3.0 -> 4.7
// TB/s; a large copy reaches 5.1).
//
// Index of a coordinate: the number of midpoint thresholds between adjacent
// centroids that it strictly exceeds (a coordinate on a threshold keeps the
// lower index), over the float32 midpoints (c_j + c_{j+1}) / 2.  It is read
// from a table of 64 buckets of the coordinate range: the bucket map
// floor(y / w + o), clamped, is monotone, so every threshold whose own
// bucket is lower lies below y and every one in a higher bucket above it;
// an entry holds the count of thresholds in lower buckets and the one
// threshold of its bucket (+inf if none), and the index is that count plus
// one comparison.  The table is held 32 times, copy k in the k-th pair of
// banks, so that a wave's reads of random entries do not collide; the map is
// computed in the mantissa of 2^15 + bucket (a fraction of 8 bits below the
// bucket number), whose bits, masked, are the entry's byte address.  If a codebook puts two thresholds in one bucket, the block
// uses a 4-step binary search over the midpoints instead.  Both give the
// same index for every y.  y is the transformed vector times one correctly
// rounded reciprocal of 16 rho.
//
// The destination of a row (request, logical position, page) is looked up
// with scalar loads where the four vectors are heads of one row (always, when
// the head count is a multiple of four), otherwise per vector.
// A vector of norm 0 has every coordinate 0.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "jfkv.h"
#include "jfkv_fwht.h"
#include "jfkv_internal.h"

namespace {

using jfkv::fwht_from1;
using jfkv::partner;
using jfkv::RowLane;

constexpr int kD = 256;          // head dimension of the format
constexpr int kWavesPerBlock = 4;
constexpr int kBatch = 4;        // vectors of a wave at a time
constexpr int kLevels = 16;
constexpr int kBuckets = 64;     // index buckets (at most one threshold each)
constexpr int kCopies = 32;      // of the bucket table: one per pair of LDS banks

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// Rows and operands are 8-byte aligned, by contract; global memory takes a
// 16-byte access at any 4-byte address, and nothing else here relies on the
// alignment of a u32x4 in memory.

// Sums of the fp16 halves (x, y) of a word in float32, one mixed-precision fma
// each (the compiler converts both halves first): x + y, x - y, and q + x * x +
// y * y (the squares exact, two roundings).
__device__ __forceinline__ float add_halves(uint32_t w) {
  float r;
  asm("v_fma_mix_f32 %0, %1, 1.0, %1 op_sel:[0,0,1] op_sel_hi:[1,0,1]" : "=v"(r) : "v"(w));
  return r;
}
__device__ __forceinline__ float sub_halves(uint32_t w) {
  float r;
  asm("v_fma_mix_f32 %0, %1, 1.0, -%1 op_sel:[0,0,1] op_sel_hi:[1,0,1]" : "=v"(r) : "v"(w));
  return r;
}
__device__ __forceinline__ float add_squares(uint32_t w, float q) {
  asm("v_fma_mix_f32 %0, %1, %1, %0 op_sel_hi:[1,1,0]" : "+v"(q) : "v"(w));
  asm("v_fma_mix_f32 %0, %1, %1, %0 op_sel:[1,1,0] op_sel_hi:[1,1,0]" : "+v"(q) : "v"(w));
  return q;
}

// a * b in float32, with +0 for either zero.  (Written out: the compiler makes
// an fma that is then rounded to fp16 a mixed-precision one, which rounds once.)
__device__ __forceinline__ float mul_pz(float a, float b) {
  float r;
  asm("v_fma_f32 %0, %1, %2, 0" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

// Sign bits of a lane's elements' signs, as bits of fp16 pairs.
__device__ __forceinline__ void sign_bits(uint32_t (&sx)[2][4], const float* signs, int chunk) {
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float* sp = signs + 128 * h + 8 * chunk + 2 * i;
      sx[h][i] = (__builtin_bit_cast(uint32_t, sp[0]) >> 31 << 15) |
                 (__builtin_bit_cast(uint32_t, sp[1]) & 0x80000000u);
    }
}

__global__ __launch_bounds__(64 * kWavesPerBlock) void tq4_encode_kernel(
    uint32_t* __restrict__ words, __half* __restrict__ norms, const u32x4* __restrict__ x,
    const float* __restrict__ signs, const float* __restrict__ centroids,
    const int32_t* __restrict__ cu_tok, const int32_t* __restrict__ start_pos,
    const int32_t* __restrict__ block_tables, int B, int max_pages, int Hkv, int P, int NP,
    int n_vec) {
  // thresholds for a 4-step binary search: entry 15 is +inf (never passed)
  __shared__ float thr[kLevels];
  // bucket table: y falls in bucket b = clamp(floor(y * bk_inv + bk_off),
  // 0, kBuckets - 1), a monotone map, so every threshold in a lower bucket is
  // below y and every one in a higher bucket above it; entry b holds their
  // count (below) and the bucket's own threshold (+inf if none)
  __shared__ __attribute__((aligned(256 * kBuckets))) float2 bucket[kBuckets][kCopies];
  __shared__ int s_multi;  // a bucket holds two thresholds: binary search instead
  const int tid = threadIdx.x;
  if (tid < kLevels)
    thr[tid] = tid < kLevels - 1 ? (centroids[tid] + centroids[tid + 1]) * 0.5f : INFINITY;
  if (tid == 0) s_multi = 0;
  __syncthreads();
  // buckets of width (t_14 - t_0) / (kBuckets - 2) from one width below t_0
  const float t_first = thr[0], t_last = thr[kLevels - 2];
  const float bk_inv = (float)(kBuckets - 2) / (t_last - t_first);
  constexpr float kMagic = 32768.0f;  // 8 bits of fraction below the bucket number
  constexpr uint32_t kMask = (kBuckets - 1) << 8;
  const float bk_off = kMagic + 1.0f - t_first * bk_inv;
  auto bucket_bits = [&](float y) {  // the bucket number in bits 8..13
    return __builtin_bit_cast(uint32_t, __builtin_amdgcn_fmed3f(fmaf(y, bk_inv, bk_off), kMagic,
                                                                kMagic + (kBuckets - 1)));
  };
  for (int i = tid; i < kBuckets * 4; i += 64 * kWavesPerBlock) {
    const uint32_t bk = i >> 2;
    int below = 0, inside = 0;
    float t_in = INFINITY;
    for (int k = 0; k < kLevels - 1; ++k) {
      const uint32_t bt = (bucket_bits(thr[k]) & kMask) >> 8;
      below += bt < bk;
      if (bt == bk) {
        ++inside;
        t_in = thr[k];
      }
    }
    for (int k = 0; k < kCopies / 4; ++k)
      bucket[bk][(i & 3) * (kCopies / 4) + k] = make_float2(__builtin_bit_cast(float, below), t_in);
    if (inside > 1 || !(bk_inv > 0.0f) || !isfinite(bk_inv)) s_multi = 1;  // benign race: all write 1
  }
  __syncthreads();
  const bool use_buckets = s_multi == 0;  // block-uniform

  const int lane = tid & 63;
  const RowLane rl(lane & 15);
  const int g = lane >> 4;  // vector of the batch
  // (the table is aligned to its size: an entry's address is base | bits | copy)
  const uint32_t copy = (uint32_t)(uintptr_t)&bucket[0][lane & (kCopies - 1)];
  uint32_t sx[2][4];  // the signs of the lane's elements, as bits of fp16 pairs
  sign_bits(sx, signs, rl.chunk);

  // wave-uniform: the batches wave, wave + W, ... (the host bounds n_vec by
  // INT32_MAX)
  const int W = (int)gridDim.x * kWavesPerBlock;
  int batch = (int)blockIdx.x * kWavesPerBlock + __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_batch = (n_vec - 1) / kBatch + 1;
  if (batch >= n_batch) return;
  u32x4 raw[2];
  const int lane_x = g * (kD / 8) + rl.chunk;       // in a batch of rows
  const int lane_w = g * P * (kD / 8) + rl.chunk;   // in the words of neighbouring KV heads
  auto load = [&](int bt) {
    const u32x4* src = x + (int64_t)bt * (kBatch * (kD / 8));
    // (past the end: the last vector again)
    const int at = n_vec - bt * kBatch >= kBatch
                       ? lane_x
                       : min(g, n_vec - bt * kBatch - 1) * (kD / 8) + rl.chunk;
    raw[0] = __builtin_nontemporal_load(src + at);
    raw[1] = __builtin_nontemporal_load(src + at + kD / 16);
  };
  // slot of KV head 0 of a row, (page * Hkv) * P + slot in the page; -1: none
  auto row_slot = [&](int row) -> int64_t {
    int32_t lo = 0, hi = B;  // request: largest b with cu_tok[b] <= row
    while (hi - lo > 1) {
      const int32_t mid = (lo + hi) >> 1;
      if (cu_tok[mid] <= row) lo = mid; else hi = mid;
    }
    const int64_t pos = (int64_t)start_pos[lo] + (row - cu_tok[lo]);
    if (pos < 0 || pos >= (int64_t)max_pages * P) return -1;
    const int lp = (int)pos / P;
    const int page = block_tables[(int64_t)lo * max_pages + lp];
    if ((unsigned)page >= (unsigned)NP) return -1;
    return (int64_t)page * Hkv * P + ((int)pos - lp * P);
  };

  load(batch);
  for (;;) {
    const int vec0 = batch * kBatch;
    const bool more = n_batch - batch > W;

    // destination: wave-uniform where the batch is heads kv0 .. of one row
    const int row0 = vec0 / Hkv, kv0 = vec0 - row0 * Hkv;
    const bool one_row = kv0 + kBatch <= Hkv;
    int64_t slot_row = -1, slot_vec = -1;
    if (one_row) {
      slot_row = row_slot(row0);
    } else if (vec0 + g < n_vec) {
      const int row = (vec0 + g) / Hkv;
      slot_vec = row_slot(row);
      if (slot_vec >= 0) slot_vec += (int64_t)(vec0 + g - row * Hkv) * P;
    }

    // stage 0 with the signs; squares of fp16 values are exact in float32.
    // The sums of squares: groups of four elements, then element index bits
    // 7, 6, .. 2 in turn
    float e[2][8], ss[2][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t w = raw[h][i] ^ sx[h][i];
        e[h][2 * i] = add_halves(w);
        e[h][2 * i + 1] = sub_halves(w);
        float& q = ss[h][i >> 1];
        q = add_squares(raw[h][i], (i & 1) ? q : 0.0f);
      }
    }
    if (more) load(batch + W);  // the registers are free; it returns during the transform
    float n0 = ss[0][0] + ss[1][0], n1 = ss[0][1] + ss[1][1];
    n0 += partner<3>(n0); n1 += partner<3>(n1);
    n0 += partner<2>(n0); n1 += partner<2>(n1);
    n0 += partner<1>(n0); n1 += partner<1>(n1);
    n0 += partner<0>(n0); n1 += partner<0>(n1);
    const float rho = sqrtf(n0 + n1);

    fwht_from1(e, rl);
    // rotated unit vector y = H S x / (16 rho), by one rounded reciprocal
    const float inv = rl.sign * (rho > 0.0f ? __fdiv_rn(1.0f, rho * 16.0f) : 0.0f);

    uint32_t q[2] = {0, 0};  // eight 4-bit indices each, the first in the low bits
    if (use_buckets) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 7; i >= 0; --i) {
          const float y = e[h][i] * inv;
          const f32x2 en = *reinterpret_cast<const __attribute__((address_space(3))) f32x2*>(
              (bucket_bits(y) & kMask) | copy);
          const float b = en.x, t = en.y;
          const uint32_t below = __builtin_bit_cast(uint32_t, b);
          q[h] = (q[h] << 4) + below + (y > t ? 1u : 0u);
        }
    } else {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 7; i >= 0; --i) {
          // off = 4 x the number of thresholds strictly below y found so far
          // (a byte offset, so each level's read takes its constant part as
          // the instruction's offset)
          const float y = e[h][i] * inv;
          int off = 0;
#pragma unroll
          for (int step = 8; step >= 1; step >>= 1) {
            const float t = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(thr) + off +
                                                            4 * (step - 1));
            off += y > t ? 4 * step : 0;
          }
          q[h] = (q[h] << 4) + (uint32_t)(off >> 2);
        }
    }

    if (one_row) {
      if (slot_row >= 0) {
        const int64_t slot0 = slot_row + (int64_t)kv0 * P;
        uint32_t* dst = words + slot0 * (kD / 8);
        dst[lane_w] = q[0];
        dst[lane_w + kD / 16] = q[1];
        if ((lane & 15) == 0) (norms + slot0)[g * P] = __float2half_rn(rho);
      }
    } else if (slot_vec >= 0) {
      uint32_t* dst = words + slot_vec * (kD / 8) + rl.chunk;
      dst[0] = q[0];
      dst[kD / 16] = q[1];
      if ((lane & 15) == 0) norms[slot_vec] = __float2half_rn(rho);
    }
    if (!more) return;
    batch += W;
  }
}

// Page -> operand reconstruction of TQ4 vectors (Appendix A, Table codec:
// page lookup, index unpacking, centroid lookup, inverse rotation, norm
// restoration in one kernel): x_hat = rho_hat S H_256 c[z] / 16 for KV heads
// kv0 .. kv0 + g - 1 at logical positions 0 .. n - 1 of one request, written
// as contiguous fp16 [g][n][256] K (blockIdx.z = 0) or V operands.  Four
// vectors per wave at a time, as in the encoder (H_256 is symmetric): lane c of
// a row of 16 holds index words c and 16 + c (elements 8c .. and 128 + 8c ..),
// looks their centroids up in LDS (16 words in 16 banks: no collisions), runs
// the eight butterfly stages, then multiplies by rho_hat / 16 (fp32) and its
// signs and stores two 16-byte pieces; a vector's 512 bytes are contiguous.  A
// page ID outside the pool gives zeros.
constexpr int kRecBatches = 4;  // batches per wave, their loads issued together

__global__ __launch_bounds__(64 * kWavesPerBlock) void tq4_reconstruct_kernel(
    const uint32_t* __restrict__ k_words, const __half* __restrict__ k_norms,
    const uint32_t* __restrict__ v_words, const __half* __restrict__ v_norms,
    const float* __restrict__ k_signs, const float* __restrict__ v_signs,
    const float* __restrict__ centroids, const int32_t* __restrict__ table, int n, int kv0,
    int Hkv, int P, int NP, uint2* __restrict__ k_out, uint2* __restrict__ v_out) {
  __shared__ float cent[kLevels];
  if (threadIdx.x < kLevels) cent[threadIdx.x] = centroids[threadIdx.x];
  const bool is_v = blockIdx.z != 0;
  const uint32_t* words = is_v ? v_words : k_words;
  const __half* norms = is_v ? v_norms : k_norms;
  uint2* out = is_v ? v_out : k_out;
  const int j = blockIdx.y;
  const int kv = kv0 + j;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  constexpr int kPerWave = kRecBatches * kBatch;
  const int t0 = ((int)blockIdx.x * kWavesPerBlock + wave) * kPerWave;
  const RowLane rl(lane & 15);
  const int g = lane >> 4;

  // the wave's positions lie in one page when the page size is a multiple of
  // them (one scalar lookup), otherwise each is looked up
  uint32_t wd[kRecBatches][2];
  float rho[kRecBatches];
  bool ok[kRecBatches];
  const bool one_page = P % kPerWave == 0;
  const int page0 = one_page && t0 < n ? table[t0 / P] : -1;
  const int slot0 = one_page ? t0 % P : 0;
#pragma unroll
  for (int v = 0; v < kRecBatches; ++v) {
    const int t = t0 + kBatch * v + g;
    int page = page0, slot = slot0 + kBatch * v + g;
    if (!one_page) {
      page = t < n ? table[t / P] : -1;
      slot = t % P;
    }
    ok[v] = t < n && (unsigned)page < (unsigned)NP;
    wd[v][0] = wd[v][1] = 0u;
    rho[v] = 0.0f;
    if (ok[v]) {
      const int64_t vec = ((int64_t)page * Hkv + kv) * P + slot;
      wd[v][0] = words[vec * (kD / 8) + rl.chunk];
      wd[v][1] = words[vec * (kD / 8) + kD / 16 + rl.chunk];
      rho[v] = __half2float(norms[vec]);
    }
  }
  uint32_t sx[2][4];
  sign_bits(sx, is_v ? v_signs : k_signs, rl.chunk);
  __syncthreads();
#pragma unroll
  for (int v = 0; v < kRecBatches; ++v) {
    const int t = t0 + kBatch * v + g;
    if (t0 + kBatch * v >= n) break;  // the whole wave
    float e[2][8];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < 8; i += 2) {
        const uint32_t w = wd[v][h];
        const float c0 = cent[(w >> (4 * i)) & 15u], c1 = cent[(w >> (4 * i + 4)) & 15u];
        e[h][i] = c0 + c1;
        e[h][i + 1] = c0 - c1;
      }
    fwht_from1(e, rl);
    // the lane holds rl.sign times the transform, but sums that cancel are +0
    // in every lane: mul_pz keeps them so, and the sign of a zero does not depend
    // on the lane.  (A norm of 0 enters as the smallest fp32, whose products
    // round to zeros of their signs.)
    float f = rho[v] * 0.0625f;
    if (f == 0.0f) f = copysignf(__FLT_DENORM_MIN__, f);
    f *= rl.sign;
    u32x4 o[2];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        o[h][i] = ok[v] ? __builtin_bit_cast(uint32_t, __floats2half2_rn(mul_pz(e[h][2 * i], f), mul_pz(e[h][2 * i + 1], f))) ^ sx[h][i]
                        : 0u;
    if (t < n) {
      u32x4* dst = reinterpret_cast<u32x4*>(out + ((int64_t)j * n + t) * (kD / 4)) + rl.chunk;
      dst[0] = o[0];
      dst[kD / 16] = o[1];
    }
  }
}

}  // namespace

namespace jfkv {

hipError_t launch_tq4_reconstruct(const jf_kv_layout& L, const void* k_words, const void* k_norms,
                                  const void* v_words, const void* v_norms, const float* k_signs,
                                  const float* v_signs, const float* centroids,
                                  const int32_t* block_table, int32_t n_pos, int32_t kv0,
                                  int32_t num_heads, void* k_out, void* v_out,
                                  hipStream_t stream) {
  if (n_pos == 0) return hipSuccess;
  constexpr int kPerBlock = kWavesPerBlock * kRecBatches * kBatch;
  dim3 grid((unsigned)((n_pos + (int64_t)kPerBlock - 1) / kPerBlock), (unsigned)num_heads, 2);
  hipLaunchKernelGGL(tq4_reconstruct_kernel, grid, dim3(64 * kWavesPerBlock), 0, stream,
                     static_cast<const uint32_t*>(k_words), static_cast<const __half*>(k_norms),
                     static_cast<const uint32_t*>(v_words), static_cast<const __half*>(v_norms),
                     k_signs, v_signs, centroids, block_table, n_pos, kv0, L.num_kv_heads,
                     L.page_size, L.num_pages, static_cast<uint2*>(k_out),
                     static_cast<uint2*>(v_out));
  return hipGetLastError();
}

hipError_t launch_tq4_encode(const jf_kv_layout& L, void* words, void* norms, const void* x,
                             const float* signs, const float* centroids, const int32_t* cu_tok,
                             const int32_t* start_pos, const int32_t* block_tables, int32_t B,
                             int32_t max_pages, int32_t total_tok, hipStream_t stream) {
  const int64_t n_vec = (int64_t)total_tok * L.num_kv_heads;
  // at most kBlocksPerCu blocks per CU, whose waves take batches in turn (each
  // block builds the bucket table once).  Six of them are on the CU at a time (73
  // registers); the other two start as those end, which evens the end out.  5, 6,
  // 8 and 12 blocks: 327, 321, 314 and 312 us for the append above, 37.1, 36.6,
  // 36.7 and 38.5 us for 20,000 rows.
  constexpr int kPerBlock = kWavesPerBlock * kBatch;
  constexpr int64_t kBlocksPerCu = 8;
  const int64_t need = (n_vec + kPerBlock - 1) / kPerBlock;
  const int64_t blocks = need <= 64 * kBlocksPerCu ? need : std::min(need, kBlocksPerCu * num_cus());
  if (n_vec > 0x7fffffffLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL(tq4_encode_kernel, dim3((unsigned)blocks), dim3(64 * kWavesPerBlock), 0,
                     stream, static_cast<uint32_t*>(words), static_cast<__half*>(norms),
                     static_cast<const u32x4*>(x), signs, centroids, cu_tok, start_pos,
                     block_tables, B, max_pages, L.num_kv_heads, L.page_size, L.num_pages,
                     (int)n_vec);
  return hipGetLastError();
}

}  // namespace jfkv
