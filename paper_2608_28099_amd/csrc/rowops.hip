// Row kernels of the probe forward: RMSNorm, RoPE at positions N_b + j with the
// scatter into the attention layouts, final norm + read-out + linear
// classifier, and the debug validation of device-resident metadata.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace sp {
namespace {

// ---------------------------------------------------------------- RMSNorm
// One workgroup (256 threads) per row; the row is read once, 4 values per
// load, and kept in registers between the sum of squares and the scaling
// (d <= 256 * 4 * kRowChunks = 16384, d % 4 == 0).
constexpr int kRowChunks = 16;

template <typename T>
__device__ __forceinline__ void load4(const T* p, float (&v)[4]) {
  if constexpr (sizeof(T) == 4) {
    const float4 x = *reinterpret_cast<const float4*>(p);
    v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
  } else {
    const uint2 x = *reinterpret_cast<const uint2*>(p);
    const T* h = reinterpret_cast<const T*>(&x);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = to_f32(h[e]);
  }
}
template <typename T>
__device__ __forceinline__ void store4(T* p, const float (&v)[4]) {
  if constexpr (sizeof(T) == 4) {
    *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
  } else {
    T h[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) h[e] = from_f32<T>(v[e]);
    *reinterpret_cast<uint2*>(p) = *reinterpret_cast<const uint2*>(h);
  }
}

// Sets kStatusRange in *status (nullable) when an fp16 output leaves fp16's
// range (it is then stored as inf).
__device__ __forceinline__ void flag_range(bool out_of_range, int* status) {
  if (__any(out_of_range) && (threadIdx.x & 63) == 0 && status) atomicOr(status, kStatusRange);
}

// CH: chunks of 1024 values held per row (registers scale with it, so the
// launcher takes the fewest that cover d).
template <typename TI, typename TG, typename TO, int CH>
__global__ __launch_bounds__(256) void rmsnorm_rows(const TI* x, int64_t ld_x, const TG* gain,
                                                    const TG* gain2, TO* out, int64_t ld_out, int d,
                                                    float eps, int* status) {
  constexpr int kRowChunks = CH;
  __shared__ float red[4];
  const int r = blockIdx.x;
  const TI* xr = x + (int64_t)r * ld_x;
  float v[kRowChunks][4], gv[kRowChunks][4];
  float ss = 0.f;
#pragma unroll
  for (int c = 0; c < kRowChunks; ++c) {
    const int i = 4 * (threadIdx.x + 256 * c);
    if (i < d) load4(xr + i, v[c]);
  }
  // the gains are loaded under the row's loads and reduction (one round trip, not two)
#pragma unroll
  for (int c = 0; c < kRowChunks; ++c) {
    const int i = 4 * (threadIdx.x + 256 * c);
    if (i < d) load4(gain + i, gv[c]);
  }
#pragma unroll
  for (int c = 0; c < kRowChunks; ++c) {
    const int i = 4 * (threadIdx.x + 256 * c);
    if (i < d) {
#pragma unroll
      for (int e = 0; e < 4; ++e) ss += v[c][e] * v[c][e];
    }
  }
  ss = block_sum_256(ss, red);
  float inv = 1.0f / sqrtf(ss / (float)d + eps);
  // optional second norm of the result with gain2 (two RMSNorms in a row)
  for (int pass = 0; pass < (gain2 ? 2 : 1); ++pass) {
    float ss2 = 0.f;
#pragma unroll
    for (int c = 0; c < kRowChunks; ++c) {
      const int i = 4 * (threadIdx.x + 256 * c);
      if (i < d) {
        if (pass) load4(gain2 + i, gv[c]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v[c][e] = v[c][e] * inv * gv[c][e];
          ss2 += v[c][e] * v[c][e];
        }
      }
    }
    if (gain2 && pass == 0) {
      ss2 = block_sum_256(ss2, red);
      inv = 1.0f / sqrtf(ss2 / (float)d + eps);
    }
  }
  TO* orow = out + (int64_t)r * ld_out;
  bool oor = false;
#pragma unroll
  for (int c = 0; c < kRowChunks; ++c) {
    const int i = 4 * (threadIdx.x + 256 * c);
    if (i < d) {
      store4(orow + i, v[c]);
      if constexpr (sizeof(TO) == 2)
#pragma unroll
        for (int e = 0; e < 4; ++e) oor |= !(fabsf(v[c][e]) <= 65504.0f);
    }
  }
  if constexpr (sizeof(TO) == 2) flag_range(oor, status);
}

// ---------------------------------------------------------------- RoPE + scatter
// One workgroup per (block of up to kRopeRows soft rows j, sequence b): the
// rotation of pair (i, i + hd/2) at row j's position N_b + t (t = step +
// j % k_task) by angle (N_b + t) * base^(-2i/hd) is computed once per row, in
// fp64, into LDS, then applied to the row's key heads (soft slot step + j)
// and, for rows that carry queries, its query heads, eight pairs per lane
// (16-byte stores of eight bf16 or four fp32 values).  The value heads are not
// rotated; in the one-pass form (per_seq = 0) they are the same for every
// sequence and written by b = 0, in the recursive form every sequence has its
// own row of projections ([B][k] rows) and its own values.  Rows per
// workgroup: as many as keep two workgroups per compute unit (one row each
// made the 27B-shaped batch 8192 workgroups with a few hundred stores each).
// Bound by its stores (queries as hi + lo: 33 MB at 128 sequences of 64 rows per
// KV head).  With 4-byte stores, pow and the library's fp64 sine and cosine it
// took 24.0 us there (41 MB written), 55.7 us at the 27B shape and 12.7 us at the
// 4B shape; now 15.5, 35.9 and 9.7.
// SPLIT (T = bf16): each value x is stored as hi = bf16(x) and lo = bf16(x - hi).
constexpr int kRopeRows = 8;

template <typename T, bool SPLIT>
__device__ __forceinline__ void put8(void* hi, void* lo, int64_t idx, const float (&x)[8]) {  // idx % 8 == 0
  if constexpr (sizeof(T) == 2) {
    u32x4 h, l;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const T h0 = from_f32<T>(x[2 * q]), h1 = from_f32<T>(x[2 * q + 1]);
      const T l0 = from_f32<T>(x[2 * q] - to_f32(h0)), l1 = from_f32<T>(x[2 * q + 1] - to_f32(h1));
      h[q] = (uint32_t)__builtin_bit_cast(uint16_t, h0) | ((uint32_t)__builtin_bit_cast(uint16_t, h1) << 16);
      l[q] = (uint32_t)__builtin_bit_cast(uint16_t, l0) | ((uint32_t)__builtin_bit_cast(uint16_t, l1) << 16);
    }
    *reinterpret_cast<u32x4*>((T*)hi + idx) = h;
    if (SPLIT) *reinterpret_cast<u32x4*>((T*)lo + idx) = l;
  } else {
    static_assert(!SPLIT, "fp32 values are stored whole");
    *reinterpret_cast<f32x4*>((T*)hi + idx) = f32x4{x[0], x[1], x[2], x[3]};
    *reinterpret_cast<f32x4*>((T*)hi + idx + 4) = f32x4{x[4], x[5], x[6], x[7]};
  }
}

// cos and sin of 2 pi x, x in fp64: the nearest quarter turn is taken off exactly,
// the rest (|r| <= pi/4) goes through the Taylor sums to r^12 / r^13, whose first
// dropped terms are below 4e-13.  What is left is the error of x itself, which grows
// with the position: turns per position are within 2^-48.7 of exact (bases up to 1e9,
// the rounding of log2(base) and of its product with the exponent; measured against
// extended precision), the product with the position adds 2^-53.  An angle of 1e6
// radians is then within 2.3e-9, 0.08 of half an fp32 ulp of 1; half an ulp is passed
// at about 1.3e7 radians.
__device__ __forceinline__ void sincos_turns(double x, float& c, float& s) {
  const double q4 = rint(4.0 * x);
  const double r = (4.0 * x - q4) * 1.5707963267948966, r2 = r * r;
  double cr = 1.0 / 479001600.0, sr = 1.0 / 6227020800.0;
  cr = fma(cr, -r2, 1.0 / 3628800.0);
  cr = fma(cr, -r2, 1.0 / 40320.0);
  cr = fma(cr, -r2, 1.0 / 720.0);
  cr = fma(cr, -r2, 1.0 / 24.0);
  cr = fma(cr, -r2, 0.5);
  cr = fma(cr, -r2, 1.0);
  sr = fma(sr, -r2, 1.0 / 39916800.0);
  sr = fma(sr, -r2, 1.0 / 362880.0);
  sr = fma(sr, -r2, 1.0 / 5040.0);
  sr = fma(sr, -r2, 1.0 / 120.0);
  sr = fma(sr, -r2, 1.0 / 6.0);
  sr = fma(sr, -r2, 1.0);
  sr *= r;
  const int q = (int)(long long)q4 & 3;
  const float cf = (float)cr, sf = (float)sr;
  c = q == 0 ? cf : q == 1 ? -sf : q == 2 ? -cf : sf;
  s = q == 0 ? sf : q == 1 ? cf : q == 2 ? -sf : -cf;
}

// The split attention's work list (see RopeParams::items), by one workgroup of
// 256 threads.  Full splits: an exclusive scan of (splits - 1) per sequence; last
// splits: a counting sort by tokens (kListBins bins at most, in hist, so lengths
// within a 1024th of a split may keep any order).  Both passes are bound by the
// latency of their loads, four sequences per thread and pass where there are
// that many.  Their time is proportional to the sequences: forwards of 1024, 4096
// and 16384 sequences on a small head take 62, 184 and 635 us, and took 161, 1798
// and 26392 when every pair of sequences was compared.  A sequence's full splits are
// rotated by its index: in plain order, where their number shares a factor with the
// XCDs, split j of every sequence lands on the same XCD, which then reads one offset of
// every block at a time, and of contiguous blocks those lines lie on few memory
// channels (44 sequences of 4782 tokens in nine splits, two KV heads: 107 us, 68).
constexpr int kListBins = 1024;

__device__ void write_work_list(const RopeParams& p, int batch, int* hist, int* wsum) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  auto len = [&](int b) { return clamp_len(p.seq_lens, b, p.max_seq_len); };
  auto full_splits = [&](int n) { return n > 0 ? (n - 1) / p.split_len : 0; };  // all but the last
  int shift = 0;
  while ((p.split_len >> shift) >= kListBins) ++shift;
  // bin of a last split of n - nf split_len tokens, the longest first
  auto bin = [&](int n, int nf) { return (p.split_len - (n - nf * p.split_len)) >> shift; };
  // the sum of x over the threads before this one; total: over all
  auto scan = [&](int x, int& total) {
    int sum = x;
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(sum, o);
      if (lane >= o) sum += v;
    }
    __syncthreads();
    if (lane == 63) wsum[wave] = sum;
    __syncthreads();
    int off = sum - x;
    total = 0;
    for (int w = 0; w < 4; ++w) {
      if (w < wave) off += wsum[w];
      total += wsum[w];
    }
    return off;
  };

  for (int t = tid; t < kListBins; t += 256) hist[t] = 0;
  __syncthreads();
  const int per = min(4, (batch + 255) / 256);  // consecutive sequences per thread and pass
  int full = 0;                                 // full splits so far
  for (int b0 = 0; b0 < batch; b0 += 256 * per) {
    int nf[4], sum = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int b = b0 + per * tid + i;
      nf[i] = 0;
      if (i < per && b < batch) {
        const int n = len(b);
        nf[i] = full_splits(n);
        atomicAdd(&hist[bin(n, nf[i])], 1);
      }
      sum += nf[i];
    }
    int total, at = full + scan(sum, total);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int b = b0 + per * tid + i;
      int sp = nf[i] > 0 ? b % nf[i] : 0;  // rotated by the sequence (see above)
      for (int j = 0; j < nf[i]; ++j) {
        p.items[at++] = make_int2(b, sp);
        if (++sp == nf[i]) sp = 0;
      }
    }
    full += total;
  }
  __syncthreads();
  int cnt[4], sum = 0, total;
#pragma unroll
  for (int i = 0; i < 4; ++i) sum += cnt[i] = hist[4 * tid + i];
  int at = full + scan(sum, total);
#pragma unroll
  for (int i = 0; i < 4; ++i) {  // (each thread rewrites the four bins that it alone read)
    hist[4 * tid + i] = at;
    at += cnt[i];
  }
  __syncthreads();
#pragma unroll 4
  for (int b = tid; b < batch; b += 256) {
    const int n = len(b), nf = full_splits(n);
    p.items[atomicAdd(&hist[bin(n, nf)], 1)] = make_int2(b, nf);
  }
  if (tid == 0) *p.n_items = full + batch;
}

template <typename T, bool SPLIT>
__global__ __launch_bounds__(256) void rope_scatter(const RopeParams p, int rows_per_block) {
  __shared__ __align__(16) float trig[2 * kRopeRows * 64];  // cos, then sin; hd / 2 <= 64
  __shared__ int wsum[4];
  static_assert(sizeof(trig) >= kListBins * sizeof(int), "the work list's bins use the same LDS");
  float (*cs)[64] = (float (*)[64])trig, (*sn)[64] = cs + kRopeRows;
  int b = blockIdx.y;
  const int j0 = blockIdx.x * rows_per_block;
  if (p.err && *p.err) return;
  if (p.items) {  // grid row 0 is the work list's: dispatched first, it runs beside the rotations
    if (b == 0) {
      if (blockIdx.x == 0) write_work_list(p, gridDim.y - 1, (int*)trig, wsum);
      return;
    }
    --b;
  }
  const int hd = p.hd, half = hd / 2, hp = half / 8;  // hp: lanes per head (eight pairs each)
  const int nj = min(rows_per_block, p.k - j0);
  int n = p.seq_lens[b];
  // a length outside [0, max_seq_len] is clamped (every kernel does the same)
  // and reported through the status word
  if ((n < 0 || n > p.max_seq_len) && blockIdx.x == 0 && threadIdx.x == 0 && p.status)
    atomicOr(p.status, kStatusSeqLen);
  n = n < 0 ? 0 : (n > p.max_seq_len ? p.max_seq_len : n);
  for (int t = threadIdx.x; t < nj * half; t += blockDim.x) {
    const int jr = t / half, i = t % half;
    const int jj = (j0 + jr) % p.k_task;
    const double pos = (double)(n + p.step + jj), ex = -2.0 * (double)i / (double)hd;
    if (p.rope_base >= 1.0) {
      // base^(-2i/hd) / 2 pi, in (0, 1/2 pi]: turns per position
      sincos_turns(pos * ((i ? exp2(ex * p.log2_base) : 1.0) * 0.15915494309189535), cs[jr][i], sn[jr][i]);
    } else {  // angles grow with i and may exceed what a count of turns in fp64 holds
      const double ang = pos * pow(p.rope_base, ex);
      cs[jr][i] = (float)cos(ang);
      sn[jr][i] = (float)sin(ang);
    }
  }
  __syncthreads();
  if (p.clear_padding && blockIdx.x == 0) {
    const float z[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const int rows = p.k / p.k_task * p.q_per_task * p.group, c8 = hd / 8;
    const int64_t bg = (int64_t)b * p.n_kv;
    for (int e = threadIdx.x; e < p.n_kv * (p.r_alloc - rows) * c8; e += blockDim.x) {
      const int row = e / c8 % (p.r_alloc - rows), g = e / c8 / (p.r_alloc - rows);
      put8<T, SPLIT>(p.q, p.q_lo, ((bg + g) * p.r_alloc + rows + row) * hd + 8 * (e % c8), z);
    }
    const int used = p.step + p.k;
    for (int e = threadIdx.x; e < p.n_kv * (p.ks - used) * c8; e += blockDim.x) {
      const int slot = used + e / c8 % (p.ks - used), g = e / c8 / (p.ks - used), i = 8 * (e % c8);
      put8<T, SPLIT>(p.k_soft, p.k_soft_lo, ((bg + g) * p.ks + slot) * hd + i, z);
      if (p.per_seq || b == 0)
        put8<T, SPLIT>(p.v_soft, p.v_soft_lo, (((p.per_seq ? bg : 0) + g) * p.ks + slot) * hd + i, z);
    }
  }
  const int row_len = (p.n_q + 2 * p.n_kv) * hd;
  const float* rows = p.qkv + ((int64_t)(p.per_seq ? b * p.k : 0) + j0) * row_len;
  // head h of the projections of row j0 + jr, pairs i .. i + 7
  auto rotate = [&](int jr, int h, int i, float (&lo8)[8], float (&hi8)[8]) __attribute__((always_inline)) {
    const float* x = rows + (int64_t)jr * row_len + h * hd + i;
#pragma unroll
    for (int v = 0; v < 8; v += 4) {
      const f32x4 xa = *reinterpret_cast<const f32x4*>(x + v), xb = *reinterpret_cast<const f32x4*>(x + half + v);
      const f32x4 c = *reinterpret_cast<const f32x4*>(&cs[jr][i + v]), s = *reinterpret_cast<const f32x4*>(&sn[jr][i + v]);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        lo8[v + e] = xa[e] * c[e] - xb[e] * s[e];
        hi8[v + e] = xb[e] * c[e] + xa[e] * s[e];
      }
    }
  };
  for (int e = threadIdx.x; e < nj * p.n_q * hp; e += blockDim.x) {
    const int jr = e / (p.n_q * hp), h = e / hp % p.n_q, i = 8 * (e % hp);
    const int j = j0 + jr, jj = j % p.k_task;
    if (jj < p.q_first) continue;
    float r0[8], r1[8];
    rotate(jr, h, i, r0, r1);
#pragma unroll
    for (int v = 0; v < 8; ++v) {
      r0[v] *= p.q_scale;
      r1[v] *= p.q_scale;
    }
    const int g = h / p.group, rr = ((j / p.k_task) * p.q_per_task + jj - p.q_first) * p.group + h % p.group;
    const int64_t base = (((int64_t)b * p.n_kv + g) * p.r_alloc + rr) * hd + i;
    put8<T, SPLIT>(p.q, p.q_lo, base, r0);
    put8<T, SPLIT>(p.q, p.q_lo, base + half, r1);
  }
  for (int e = threadIdx.x; e < nj * p.n_kv * hp; e += blockDim.x) {
    const int jr = e / (p.n_kv * hp), g = e / hp % p.n_kv, i = 8 * (e % hp);
    float r0[8], r1[8];
    rotate(jr, p.n_q + g, i, r0, r1);
    const int64_t base = (((int64_t)b * p.n_kv + g) * p.ks + p.step + j0 + jr) * hd + i;
    put8<T, SPLIT>(p.k_soft, p.k_soft_lo, base, r0);
    put8<T, SPLIT>(p.k_soft, p.k_soft_lo, base + half, r1);
  }
  if (p.per_seq || b == 0) {
    const int64_t vb = p.per_seq ? (int64_t)b * p.n_kv : 0;
    for (int e = threadIdx.x; e < nj * p.n_kv * 2 * hp; e += blockDim.x) {
      const int jr = e / (p.n_kv * 2 * hp), g = e / (2 * hp) % p.n_kv, i = 8 * (e % (2 * hp));
      const float* x = rows + (int64_t)jr * row_len + (p.n_q + p.n_kv + g) * hd + i;
      float v[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) v[t] = x[t];
      put8<T, SPLIT>(p.v_soft, p.v_soft_lo, ((vb + g) * p.ks + p.step + j0 + jr) * hd + i, v);
    }
  }
}

// ---------------------------------------------------------------- read-out
// One workgroup per (sequence b, task t, class c):
//   logits[b][t][c] = sum_j w_j * inv_j * sum_i W_cls[t][c][i] gamma_i y_j[i]  (+ bias[t][c]),
// with inv_j = 1 / sqrt(mean_i y_j[i]^2 + eps) over the read-out rows j of task
// t (its last row, w = 1; or all k, w = 1/k): RMSNorm, pooling and the linear
// classifier folded into one pass and one block reduction per row.
template <typename T>
__global__ __launch_bounds__(256) void final_classifier(const ClsParams p) {
  __shared__ float red[4];
  const int b = blockIdx.x, tc = blockIdx.y, d = p.d;  // tc = task * C + class
  if (p.err && *p.err) return;
  const int task = tc / p.n_classes;
  const int j0 = p.pool_mean ? 0 : p.k - 1;
  const float w = p.pool_mean ? 1.0f / (float)p.k : 1.0f;
  const T* wr = (const T*)p.w_cls + (p.cls_rows ? (int64_t)p.cls_rows[tc] : (int64_t)tc) * d;
  const T* gm = (const T*)p.final_norm;
  float wg[kRowChunks][4];  // W_cls[c][i] * gamma_i, reused for every row
#pragma unroll
  for (int q = 0; q < kRowChunks; ++q) {
    const int i = 4 * (threadIdx.x + 256 * q);
    if (i < d) {
      float a[4], g4[4];
      load4(wr + i, a);
      load4(gm + i, g4);
#pragma unroll
      for (int e = 0; e < 4; ++e) wg[q][e] = a[e] * g4[e];
    }
  }
  float logit = 0.f;
  for (int j = j0; j < p.k; ++j) {
    const float* yr = p.y + (((int64_t)b * p.n_tasks + task) * p.k + j) * d;
    float ss = 0.f, dot = 0.f;
#pragma unroll
    for (int q = 0; q < kRowChunks; ++q) {
      const int i = 4 * (threadIdx.x + 256 * q);
      if (i < d) {
        float y4[4];
        load4(yr + i, y4);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          ss += y4[e] * y4[e];
          dot += y4[e] * wg[q][e];
        }
      }
    }
    ss = block_sum_256(ss, red);
    dot = block_sum_256(dot, red);
    logit += w * dot / sqrtf(ss / (float)d + p.eps);
  }
  if (threadIdx.x == 0)
    p.logits[(int64_t)b * p.n_tasks * p.n_classes + tc] = logit + (p.b_cls ? p.b_cls[tc] : 0.f);
}

// ---------------------------------------------------------------- fp16 staging with row scales
// One workgroup per row: max |x| over the row, then the scaled fp16 copy, eight
// values per load (cols % 8 == 0, rows 16-byte aligned).  Bound by two passes of
// load latency: 2-byte loads and a counted exponent took 14.2 us for 9 rows of
// 7680, this 3.0 us.
__global__ __launch_bounds__(1024) void scale_rows_f16(const bf16* x, int64_t ld_x, f16* out,
                                                       float* inv_scale, int cols) {
  __shared__ float red[16];
  const int r = blockIdx.x, tid = threadIdx.x;
  const bf16* xr = x + (int64_t)r * ld_x;
  float mx = 0.f;
  for (int i = 8 * tid; i < cols; i += 8 * 1024) {
    const bf16x8 v = __builtin_bit_cast(bf16x8, ld16v(xr + i));
#pragma unroll
    for (int e = 0; e < 8; ++e) mx = fmaxf(mx, fabsf((float)v[e]));
  }
  for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
  if ((tid & 63) == 0) red[tid >> 6] = mx;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < 16; ++w) mx = fmaxf(mx, red[w]);
  // smallest e >= 0 with mx 2^-e < 2^15 (126 for an infinite entry)
  const int e = mx >= 32768.0f ? min(__builtin_isinf(mx) ? 126 : ilogbf(mx) - 14, 126) : 0;
  const float sc = ldexpf(1.0f, -e);
  f16* orow = out + (int64_t)r * cols;
  for (int i = 8 * tid; i < cols; i += 8 * 1024) {
    const bf16x8 v = __builtin_bit_cast(bf16x8, ld16v(xr + i));
    f16x8 h;
#pragma unroll
    for (int t = 0; t < 8; ++t) h[t] = (f16)((float)v[t] * sc);
    *reinterpret_cast<f16x8*>(orow + i) = h;
  }
  if (tid == 0) inv_scale[r] = ldexpf(1.0f, e);
}

// ---------------------------------------------------------------- validation
__global__ void validate_meta(const ValidateParams p) {
  const int b = blockIdx.x;
  if (b == 0 && p.cls_rows) {
    for (int i = threadIdx.x; i < p.n_cls_rows; i += blockDim.x) {
      const int r = p.cls_rows[i];
      if (r < 0 || (int64_t)r >= p.cls_vocab) atomicOr(p.err, 8);
    }
  }
  const int n = p.seq_lens[b];
  if (n < 0 || n > p.max_seq_len) {
    if (threadIdx.x == 0) atomicOr(p.err, 1);
    return;
  }
  const int nblk = (n + (1 << p.bs_log2) - 1) >> p.bs_log2;
  if (nblk > p.mbps) {
    if (threadIdx.x == 0) atomicOr(p.err, 2);
    return;
  }
  if (!p.block_table) return;
  for (int j = threadIdx.x; j < nblk; j += blockDim.x) {
    const int id = p.block_table[(int64_t)b * p.mbps + j];
    if (id < 0 || (int64_t)id >= p.num_blocks) atomicOr(p.err, 4);
  }
}

// ---------------------------------------------------------------- workspace guards, weight image
__global__ void fill_words(uint32_t* p, size_t n, uint32_t value) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    p[i] = value;
}

// One workgroup per guard area.
__global__ void check_guards(const char* base, const uint64_t* offs, int words, uint32_t value, int* flag,
                             int bit) {
  const uint32_t* g = reinterpret_cast<const uint32_t*>(base + offs[blockIdx.x]);
  bool bad = false;
  for (int i = threadIdx.x; i < words; i += blockDim.x) bad |= g[i] != value;
  if (__any(bad) && (threadIdx.x & 63) == 0) atomicOr(flag, bit);
}

__global__ void bf16_to_f16(const uint32_t* src, uint32_t* dst, size_t n2) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n2; i += (size_t)gridDim.x * blockDim.x)
    dst[i] = bf16x2_to_f16x2(src[i]);
}

__global__ void check_header(const uint32_t* image, const uint32_t* expect, int n_words, int* flag, int bit) {
  const int i = threadIdx.x;
  const bool bad = i < n_words && image[i] != expect[i];
  if (__any(bad) && i == 0) atomicOr(flag, bit);
}

}  // namespace

hipError_t launch_fill_words(uint32_t* p, size_t n, uint32_t value, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const size_t blocks = std::min<size_t>((n + 255) / 256, 4096);
  hipLaunchKernelGGL(fill_words, dim3((unsigned)blocks), dim3(256), 0, s, p, n, value);
  return hipGetLastError();
}

hipError_t launch_check_guards(const char* base, const uint64_t* offs, int n_guards, int words,
                               uint32_t value, int* flag, int bit, hipStream_t s) {
  if (n_guards <= 0) return hipSuccess;
  hipLaunchKernelGGL(check_guards, dim3(n_guards), dim3(64), 0, s, base, offs, words, value, flag, bit);
  return hipGetLastError();
}

hipError_t launch_bf16_to_f16(const void* src, void* dst, size_t n, hipStream_t s) {
  if (n % 2) return hipErrorInvalidValue;
  if (n == 0) return hipSuccess;
  const size_t blocks = std::min<size_t>((n / 2 + 255) / 256, 8192);
  hipLaunchKernelGGL(bf16_to_f16, dim3((unsigned)blocks), dim3(256), 0, s, (const uint32_t*)src,
                     (uint32_t*)dst, n / 2);
  return hipGetLastError();
}

hipError_t launch_check_header(const uint32_t* image, const uint32_t* expect, int n_words, int* flag,
                               int bit, hipStream_t s) {
  if (n_words > 64) return hipErrorInvalidValue;
  hipLaunchKernelGGL(check_header, dim3(1), dim3(64), 0, s, image, expect, n_words, flag, bit);
  return hipGetLastError();
}

hipError_t launch_rmsnorm_rows(DType in_dt, DType gain_dt, DType out_dt, const void* x,
                               int64_t ld_x, const void* gain, const void* gain2, void* out,
                               int64_t ld_out, int rows, int d, float eps, int* status,
                               hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  if (d % 4 || d > 1024 * kRowChunks || ld_x % 4 || ld_out % 4) return hipErrorInvalidValue;
  const dim3 grid(rows), block(256);
  auto run = [&](auto ch) {
    constexpr int CH = decltype(ch)::value;
    if (in_dt == kBF16 && gain_dt == kBF16 && out_dt == kF16)
      hipLaunchKernelGGL((rmsnorm_rows<bf16, bf16, f16, CH>), grid, block, 0, s, (const bf16*)x, ld_x,
                         (const bf16*)gain, (const bf16*)gain2, (f16*)out, ld_out, d, eps, status);
    else if (in_dt == kF32 && gain_dt == kBF16 && out_dt == kF16)
      hipLaunchKernelGGL((rmsnorm_rows<float, bf16, f16, CH>), grid, block, 0, s, (const float*)x, ld_x,
                         (const bf16*)gain, (const bf16*)gain2, (f16*)out, ld_out, d, eps, status);
    else if (in_dt == kF32 && gain_dt == kF32 && out_dt == kF32)
      hipLaunchKernelGGL((rmsnorm_rows<float, float, float, CH>), grid, block, 0, s, (const float*)x, ld_x,
                         (const float*)gain, (const float*)gain2, (float*)out, ld_out, d, eps, status);
    else
      return hipErrorInvalidValue;
    return hipGetLastError();
  };
  const int ch = (d + 1023) / 1024;
  if (ch <= 1) return run(std::integral_constant<int, 1>{});
  if (ch <= 2) return run(std::integral_constant<int, 2>{});
  if (ch <= 3) return run(std::integral_constant<int, 3>{});
  if (ch <= 4) return run(std::integral_constant<int, 4>{});
  if (ch <= 5) return run(std::integral_constant<int, 5>{});
  if (ch <= 8) return run(std::integral_constant<int, 8>{});
  return run(std::integral_constant<int, kRowChunks>{});
}

hipError_t launch_rope_scatter(DType dt, const RopeParams& p, int batch, hipStream_t s) {
  if (p.hd > 128 || p.hd % 16 || p.k < 1) return hipErrorInvalidValue;
  // rows per workgroup: doubled while the grid keeps two workgroups per compute unit
  const int cus = p.num_cus > 0 ? p.num_cus : 256;
  int rpb = 1;
  while (2 * rpb <= kRopeRows && 2 * rpb <= p.k && (int64_t)((p.k + 2 * rpb - 1) / (2 * rpb)) * batch >= 2 * cus)
    rpb *= 2;
  const dim3 grid((p.k + rpb - 1) / rpb, batch + (p.items ? 1 : 0)), block(256);
  if (dt == kBF16)
    hipLaunchKernelGGL((rope_scatter<bf16, true>), grid, block, 0, s, p, rpb);
  else if (dt == kF32)
    hipLaunchKernelGGL((rope_scatter<float, false>), grid, block, 0, s, p, rpb);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_scale_rows_f16(const void* x, int64_t ld_x, void* out, float* inv_scale, int rows,
                                 int cols, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  if (cols % 8 || ld_x % 8 || ((uintptr_t)x & 15) || ((uintptr_t)out & 15)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(scale_rows_f16, dim3(rows), dim3(1024), 0, s, (const bf16*)x, ld_x, (f16*)out,
                     inv_scale, cols);
  return hipGetLastError();
}

hipError_t launch_final_classifier(DType dt, const ClsParams& p, int batch, hipStream_t s) {
  if (p.d % 4 || p.d > 1024 * kRowChunks) return hipErrorInvalidValue;
  const dim3 grid(batch, p.n_tasks * p.n_classes);
  if (dt == kBF16)
    hipLaunchKernelGGL(final_classifier<bf16>, grid, dim3(256), 0, s, p);
  else
    hipLaunchKernelGGL(final_classifier<float>, grid, dim3(256), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_validate(const ValidateParams& p, int batch, hipStream_t s) {
  hipLaunchKernelGGL(validate_meta, dim3(batch), dim3(64), 0, s, p);
  return hipGetLastError();
}

}  // namespace sp
