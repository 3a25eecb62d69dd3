// Plain softmax attention on the vector ALUs, one wavefront per query row
// (forward, dQ) or per key row (dK, dV).  This is the fp32 debug mode's
// attention and the fallback for shapes the MFMA kernels do not take.
// Scores of one row live in LDS (4 bytes x S per wave), so S <= 4096.
// Head dimensions up to 128 run the attn_*_rows kernels below, wider ones the attn_*_simple kernels.
// Operands come through an AttnView: Sq queries from one tensor, Sk keys and values from
// another (the same packed tensor for self-attention).
// Dropout (da.thr != 0): element (i, j) of head (b, h) is kept when
// drop_bits(i*Sk + j, keys of unit b*nh + h) >= da.thr; kept probabilities are scaled by
// da.scale after the softmax, and the backward masks and scales dP the same way.
#include "common.h"
#include "kernels.h"

namespace dp {

template <typename T>
__device__ __forceinline__ float dot_row(const float *__restrict__ qs, const T *__restrict__ p, int dh) {
  float s = 0.f;
  for (int d = 0; d < dh; d += 8) {
    float v[8];
    load8(p + d, v);
#pragma unroll
    for (int i = 0; i < 8; ++i) s += qs[d + i] * v[i];
  }
  return s;
}

template <typename T>
__global__ __launch_bounds__(256) void attn_fwd_simple_kernel(AttnView av, T *__restrict__ o,
                                                              float *__restrict__ lse, int B, int nh, int dh,
                                                              int causal, float scale, DropArgs da) {
  extern __shared__ float smem[];
  const int Sq = av.Sq, S = av.Sk;   // S: the key count
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float *sc = smem + (size_t)wave * (S + dh);
  float *qs = sc + S;
  long row_id = (long)blockIdx.x * 4 + wave;  // (b, h, i)
  const bool active = row_id < (long)B * nh * Sq;  // inactive waves still reach every barrier
  if (!active) row_id = 0;
  const int i = (int)(row_id % Sq);
  const int h = (int)((row_id / Sq) % nh);
  const int b = (int)(row_id / ((long)Sq * nh));
  const int H = nh * dh;
  const size_t ldq = (size_t)av.ldq, ld = (size_t)av.ldkv;
  const T *qrow = (const T *)av.q + ((size_t)b * Sq + i) * ldq + (size_t)h * dh;
  const T *kbase = (const T *)av.k + (size_t)b * S * ld + (size_t)h * dh;
  const T *vbase = (const T *)av.v + (size_t)b * S * ld + (size_t)h * dh;
  for (int d = lane; d < dh; d += 64) qs[d] = ldf(qrow + d);
  __syncthreads();
  const int jn = !active ? 0 : causal ? i + 1 : S;
  float m = -INFINITY;
  for (int j = lane; j < jn; j += 64) {
    const float s = scale * dot_row(qs, kbase + (size_t)j * ld, dh);
    sc[j] = s;
    m = fmaxf(m, s);
  }
  m = wave_max(m);
  float l = 0.f;
  for (int j = lane; j < jn; j += 64) {
    const float p = expf(sc[j] - m);
    sc[j] = p;
    l += p;
  }
  l = wave_sum(l);
  if (da.thr != 0) {
    const DropKeys keys = drop_keys(da.base, (uint32_t)(b * nh + h));
    for (int j = lane; j < jn; j += 64)
      if (drop_bits((uint32_t)i * (uint32_t)S + (uint32_t)j, keys.k0, keys.k1) < da.thr) sc[j] = 0.f;
  }
  __syncthreads();
  if (!active) return;
  if (lse != nullptr && lane == 0) lse[((size_t)b * nh + h) * Sq + i] = m + logf(l);
  if (o == nullptr) return;
  const float inv = da.scale / l;
  for (int d = lane; d < dh; d += 64) {
    float acc = 0.f;
    const T *v = vbase + d;
    for (int j = 0; j < jn; ++j) acc += sc[j] * ldf(v + (size_t)j * ld);
    stf(o + ((size_t)b * Sq + i) * H + (size_t)h * dh + d, acc * inv);
  }
}

// Per query row i: D_i = <dO_i, O_i>; dS_ij = P_ij (dP_ij - D_i); dQ_i = scale * sum_j dS_ij K_j.
template <typename T>
__global__ __launch_bounds__(256) void attn_bwd_dq_simple_kernel(AttnView av, const T *__restrict__ o,
                                                                 const float *__restrict__ lse,
                                                                 const T *__restrict__ d_o,
                                                                 float *__restrict__ drow, int B, int nh,
                                                                 int dh, int causal, float scale, DropArgs da) {
  extern __shared__ float smem[];
  const int Sq = av.Sq, S = av.Sk;   // S: the key count
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float *sc = smem + (size_t)wave * (S + 2 * dh);
  float *qs = sc + S;
  float *dos = qs + dh;
  long row_id = (long)blockIdx.x * 4 + wave;
  const bool active = row_id < (long)B * nh * Sq;
  if (!active) row_id = 0;
  const int i = (int)(row_id % Sq);
  const int h = (int)((row_id / Sq) % nh);
  const int b = (int)(row_id / ((long)Sq * nh));
  const int H = nh * dh;
  const size_t ldq = (size_t)av.ldq, ld = (size_t)av.ldkv;
  const size_t qoff = ((size_t)b * Sq + i) * ldq + (size_t)h * dh;
  const T *kbase = (const T *)av.k + (size_t)b * S * ld + (size_t)h * dh;
  const T *vbase = (const T *)av.v + (size_t)b * S * ld + (size_t)h * dh;
  const size_t orow = ((size_t)b * Sq + i) * H + (size_t)h * dh;
  float dsum = 0.f;
  for (int d = lane; d < dh; d += 64) {
    qs[d] = ldf((const T *)av.q + qoff + d);
    const float g = ldf(d_o + orow + d);
    dos[d] = g;
    dsum += g * ldf(o + orow + d);
  }
  dsum = wave_sum(dsum);
  __syncthreads();
  const float L = lse[((size_t)b * nh + h) * Sq + i];
  if (active && lane == 0) drow[((size_t)b * nh + h) * Sq + i] = dsum;
  const int jn = !active ? 0 : causal ? i + 1 : S;
  const DropKeys keys = drop_keys(da.base, (uint32_t)(b * nh + h));
  for (int j = lane; j < jn; j += 64) {
    const float p = expf(scale * dot_row(qs, kbase + (size_t)j * ld, dh) - L);
    float dp = dot_row(dos, vbase + (size_t)j * ld, dh);
    if (da.thr != 0)
      dp = drop_bits((uint32_t)i * (uint32_t)S + (uint32_t)j, keys.k0, keys.k1) >= da.thr ? dp * da.scale : 0.f;
    sc[j] = p * (dp - dsum);
  }
  __syncthreads();
  if (!active) return;
  for (int d = lane; d < dh; d += 64) {
    float acc = 0.f;
    const T *k = kbase + d;
    for (int j = 0; j < jn; ++j) acc += sc[j] * ldf(k + (size_t)j * ld);
    stf((T *)av.dq + qoff + d, acc * scale);
  }
}

// Per key row j: dV_j = sum_i P_ij dO_i; dK_j = scale * sum_i dS_ij Q_i.
template <typename T>
__global__ __launch_bounds__(256) void attn_bwd_dkv_simple_kernel(AttnView av,
                                                                  const float *__restrict__ lse,
                                                                  const T *__restrict__ d_o,
                                                                  const float *__restrict__ drow,
                                                                  int B, int nh, int dh,
                                                                  int causal, float scale, DropArgs drop) {
  extern __shared__ float smem[];
  const int S = av.Sq, Sk = av.Sk;   // S: the query count, which bounds the loops over i below
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float *pa = smem + (size_t)wave * (2 * S + 2 * dh);
  float *da = pa + S;
  float *ks = da + S;
  float *vs = ks + dh;
  long row_id = (long)blockIdx.x * 4 + wave;
  const bool active = row_id < (long)B * nh * Sk;
  if (!active) row_id = 0;
  const int j = (int)(row_id % Sk);
  const int h = (int)((row_id / Sk) % nh);
  const int b = (int)(row_id / ((long)Sk * nh));
  const int H = nh * dh;
  const size_t ld = (size_t)av.ldq, ldkv = (size_t)av.ldkv;
  const T *base = (const T *)av.q + (size_t)b * S * ld + (size_t)h * dh;
  const T *dob = d_o + (size_t)b * S * H + (size_t)h * dh;
  const size_t koff = ((size_t)b * Sk + j) * ldkv + (size_t)h * dh;
  for (int d = lane; d < dh; d += 64) {
    ks[d] = ldf((const T *)av.k + koff + d);
    vs[d] = ldf((const T *)av.v + koff + d);
  }
  __syncthreads();
  const int i0 = !active ? S : causal ? j : 0;
  const float *Lr = lse + ((size_t)b * nh + h) * S;
  const float *Dr = drow + ((size_t)b * nh + h) * S;
  const DropKeys keys = drop_keys(drop.base, (uint32_t)(b * nh + h));
  for (int i = i0 + lane; i < S; i += 64) {
    const float p = expf(scale * dot_row(ks, base + (size_t)i * ld, dh) - Lr[i]);
    float dp = dot_row(vs, dob + (size_t)i * H, dh);
    float pv = p;   // what multiplied V in the forward
    if (drop.thr != 0) {
      const bool keep = drop_bits((uint32_t)i * (uint32_t)Sk + (uint32_t)j, keys.k0, keys.k1) >= drop.thr;
      pv = keep ? p * drop.scale : 0.f;
      dp = keep ? dp * drop.scale : 0.f;
    }
    pa[i] = pv;
    da[i] = p * (dp - Dr[i]);
  }
  __syncthreads();
  if (!active) return;
  for (int d = lane; d < dh; d += 64) {
    float acc_v = 0.f, ak = 0.f;
    for (int i = i0; i < S; ++i) {
      acc_v += pa[i] * ldf(dob + (size_t)i * H + d);
      ak += da[i] * ldf(base + (size_t)i * ld + d);
    }
    stf((T *)av.dk + koff + d, ak * scale);
    stf((T *)av.dv + koff + d, acc_v);
  }
}

// ------------------------------------------------------------------ head dimensions up to 128
// What bounds these calls is latency (a stage that checks itself has a few hundred rows), so a wave works on eight of the other side's
// rows at a time: group g of 8 lanes has row 8 u + g of a batch, lane x of the group its elements 32 t + 4 x .. + 3, t < NT.
// A load is 16 bytes a lane (fp32) and 128 contiguous bytes a row, all loads of a batch of 8 U rows go out together, a dot
// product is summed over the group by lane swaps, and the backward's rows are used where they are, for the product that made P and
// for the one that takes it.  (A lane a row, as in the kernels above, touches 64 lines a load and waits for every 32 bytes; sums over
// rows went one row at a time.  us, forward + backward, those kernels / these: fp32 64 rows, 2 heads of 64 7.9 + 21.7 / 5.3 + 11.6; 256 rows, 16 heads
// of 64 42 + 161 / 21 + 53; 4096 rows, 2 heads of 96 3314 + 14722 / 872 + 1958; bf16 64 rows, 2 heads of 40 7.1 + 15.0 / 5.2 + 12.5;
// 1024 rows, 8 heads of 80 298 + 1188 / 181 + 431, causal 213 + 925 / 136 + 286; 4096 rows, 2 heads of 96 1778 + 12419 / 738 + 1808.
// One row a sequence stays behind: bf16, 2 heads of 80, backward 10.7 / 11.3.)
template <typename T> struct Raw4;
template <> struct Raw4<float> { f32x4 v; };
template <> struct Raw4<bf16> { bf16x4 v; };

template <int CTRL> __device__ __forceinline__ float lane_swap(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float group8_sum(float x) {
  x += lane_swap<0xB1>(x);           // lanes 1 0 3 2
  x += lane_swap<0x4E>(x);           // lanes 2 3 0 1
  return x + lane_swap<0x141>(x);    // lane 7 - x of the group
}

// P from a dot product and the row's log-sum-exp.  The scaled product is rounded as the forward rounds it (no fused multiply-subtract),
// so that a row's only key has P = 1 exactly.
__device__ __forceinline__ float row_prob(float dot, float scale, float lse) {
#pragma clang fp contract(off)
  const float s = scale * dot;
  return expf(s - lse);
}

// what a wave and its lanes own, and how they read a row
template <typename T, int NT>
struct Rows {
  int g, x, dh;
  __device__ __forceinline__ Rows(int lane, int dh_) : g(lane >> 3), x(lane & 7), dh(dh_) {}
  __device__ __forceinline__ int col(int t) const { return 32 * t + 4 * x; }
  __device__ __forceinline__ bool has(int t) const { return col(t) < dh; }
  // this lane's elements of a row that only this wave reads (element by element: its alignment is the caller's)
  __device__ __forceinline__ void own(const T *p, float (&v)[NT][4]) const {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[t][e] = has(t) ? ldf(p + col(t) + e) : 0.f;
  }
  // columns past the head's read its last four: dot() leaves them out, and what the others make of them is not stored
  __device__ __forceinline__ void load(const T *p, Raw4<T> (&v)[NT]) const {
#pragma unroll
    for (int t = 0; t < NT; ++t) v[t].v = *reinterpret_cast<const decltype(v[t].v) *>(p + min(col(t), dh - 4));
  }
  __device__ __forceinline__ float dot(const float (&a)[NT][4], const Raw4<T> (&b)[NT]) const {
    float s = 0.f;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) s = has(t) ? s + a[t][e] * (float)b[t].v[e] : s;
    return group8_sum(s);
  }
  static __device__ __forceinline__ void add(float (&acc)[NT][4], float w, const Raw4<T> (&b)[NT]) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[t][e] += w * (float)b[t].v[e];
  }
  // the sum over the groups, stored by the first
  __device__ __forceinline__ void store(float (&acc)[NT][4], float mul, T *p) const {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float v = acc[t][e];
#pragma unroll
        for (int m = 8; m <= 32; m <<= 1) v += __shfl_xor(v, m, 64);
        if (g == 0 && has(t)) stf(p + col(t) + e, v * mul);
      }
  }
};

// The row of this wave among (b, h, i), i < n; false: none (such a wave still reaches every barrier)
__device__ __forceinline__ bool wave_row(int n, int nh, long rows, int &b, int &h, int &i) {
  const long id = (long)blockIdx.x * (blockDim.x >> 6) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const long at = id < rows ? id : 0;
  i = (int)(at % n);
  h = (int)((at / n) % nh);
  b = (int)(at / ((long)n * nh));
  return id < rows;
}

template <typename T, int NT, int U>
__global__ __launch_bounds__(256) void attn_fwd_rows_kernel(AttnView av, T *__restrict__ o, float *__restrict__ lse, int B, int nh,
                                                            int dh, int causal, float scale, DropArgs da) {
  extern __shared__ float smem[];
  const int Sq = av.Sq, S = av.Sk, lane = threadIdx.x & 63;
  float *sc = smem + (size_t)(threadIdx.x >> 6) * S;
  int b, h, i;
  const bool active = wave_row(Sq, nh, (long)B * nh * Sq, b, h, i);
  const Rows<T, NT> r(lane, dh);
  const size_t ld = (size_t)av.ldkv;
  const T *kb = (const T *)av.k + (size_t)b * S * ld + (size_t)h * dh, *vb = (const T *)av.v + (size_t)b * S * ld + (size_t)h * dh;
  const int jn = !active ? 0 : causal ? i + 1 : S;
  float q[NT][4];
  r.own((const T *)av.q + ((size_t)b * Sq + i) * av.ldq + (size_t)h * dh, q);
  float m = -INFINITY;
  for (int j0 = 0; j0 < jn; j0 += 8 * U) {
    Raw4<T> k[U][NT];
#pragma unroll
    for (int u = 0; u < U; ++u) r.load(kb + (size_t)min(j0 + 8 * u + r.g, jn - 1) * ld, k[u]);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = j0 + 8 * u + r.g;
      const float s = scale * r.dot(q, k[u]);
      if (j < jn) {
        if (r.x == 0) sc[j] = s;
        m = fmaxf(m, s);
      }
    }
  }
  m = wave_max(m);
  __syncthreads();
  // P, a key a lane (each of a group's eight lanes working it out for the sum that follows: bf16, 1024 rows, 8 heads of 40, causal
  // 128 us, now 92; fp32, 256 rows, 16 heads of 64 24.0, now 20.9)
  const DropKeys keys = drop_keys(da.base, (uint32_t)(b * nh + h));
  float l = 0.f, acc[NT][4] = {};
  for (int j = lane; j < jn; j += 64) {
    float p = expf(sc[j] - m);
    l += p;
    if (da.thr != 0 && drop_bits((uint32_t)i * (uint32_t)S + (uint32_t)j, keys.k0, keys.k1) < da.thr) p = 0.f;
    sc[j] = p;
  }
  l = wave_sum(l);
  __syncthreads();
  // (whole batches without a guard: behind one the compiler moves the loads to their uses, and a wave waits for each)
  int j0 = 0;
  if (o != nullptr) {
    for (; j0 + 8 * U <= jn; j0 += 8 * U) {
      Raw4<T> v[U][NT];
#pragma unroll
      for (int u = 0; u < U; ++u) r.load(vb + (size_t)(j0 + 8 * u + r.g) * ld, v[u]);
#pragma unroll
      for (int u = 0; u < U; ++u) r.add(acc, sc[j0 + 8 * u + r.g], v[u]);
    }
    for (int j = j0 + r.g; j < jn; j += 8) {
      Raw4<T> v[NT];
      r.load(vb + (size_t)j * ld, v);
      r.add(acc, sc[j], v);
    }
  }
  if (!active) return;
  if (lse != nullptr && lane == 0) lse[((size_t)b * nh + h) * Sq + i] = m + logf(l);
  if (o != nullptr) r.store(acc, da.scale / l, o + ((size_t)b * Sq + i) * (size_t)(nh * dh) + (size_t)h * dh);
}

template <typename T, int NT, int U>
__global__ __launch_bounds__(256) void attn_bwd_dq_rows_kernel(AttnView av, const T *__restrict__ o, const float *__restrict__ lse,
                                                               const T *__restrict__ d_o, float *__restrict__ drow, int B, int nh,
                                                               int dh, int causal, float scale, DropArgs da) {
  const int Sq = av.Sq, S = av.Sk, lane = threadIdx.x & 63;
  int b, h, i;
  if (!wave_row(Sq, nh, (long)B * nh * Sq, b, h, i)) return;
  const Rows<T, NT> r(lane, dh);
  const size_t ld = (size_t)av.ldkv, qoff = ((size_t)b * Sq + i) * av.ldq + (size_t)h * dh;
  const size_t orow = ((size_t)b * Sq + i) * (size_t)(nh * dh) + (size_t)h * dh, lrow = ((size_t)b * nh + h) * Sq + i;
  const T *kb = (const T *)av.k + (size_t)b * S * ld + (size_t)h * dh, *vb = (const T *)av.v + (size_t)b * S * ld + (size_t)h * dh;
  const int jn = causal ? i + 1 : S;
  float q[NT][4], g[NT][4], acc[NT][4] = {};
  r.own((const T *)av.q + qoff, q);
  r.own(d_o + orow, g);
  float dsum = 0.f;
  {
    float ov[NT][4];
    r.own(o + orow, ov);
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) dsum += g[t][e] * ov[t][e];
  }
  dsum = group8_sum(dsum);
  const float L = lse[lrow];
  if (lane == 0) drow[lrow] = dsum;
  const DropKeys keys = drop_keys(da.base, (uint32_t)(b * nh + h));
  for (int j0 = 0; j0 < jn; j0 += 8 * U) {
    Raw4<T> k[U][NT], v[U][NT];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const size_t at = (size_t)min(j0 + 8 * u + r.g, jn - 1) * ld;
      r.load(kb + at, k[u]);
      r.load(vb + at, v[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = j0 + 8 * u + r.g;
      const float p = row_prob(r.dot(q, k[u]), scale, L);
      float dp = r.dot(g, v[u]);
      if (da.thr != 0)
        dp = drop_bits((uint32_t)i * (uint32_t)S + (uint32_t)j, keys.k0, keys.k1) >= da.thr ? dp * da.scale : 0.f;
      if (j < jn) r.add(acc, p * (dp - dsum), k[u]);
    }
  }
  r.store(acc, scale, (T *)av.dq + qoff);
}

template <typename T, int NT, int U>
__global__ __launch_bounds__(256) void attn_bwd_dkv_rows_kernel(AttnView av, const float *__restrict__ lse,
                                                                const T *__restrict__ d_o, const float *__restrict__ drow, int B,
                                                                int nh, int dh, int causal, float scale, DropArgs da) {
  const int S = av.Sq, Sk = av.Sk, lane = threadIdx.x & 63;   // S: the query count
  int b, h, j;
  if (!wave_row(Sk, nh, (long)B * nh * Sk, b, h, j)) return;
  const Rows<T, NT> r(lane, dh);
  const size_t ld = (size_t)av.ldq, H = (size_t)nh * dh, koff = ((size_t)b * Sk + j) * av.ldkv + (size_t)h * dh;
  const T *qb = (const T *)av.q + (size_t)b * S * ld + (size_t)h * dh, *gb = d_o + (size_t)b * S * H + (size_t)h * dh;
  const float *Lr = lse + ((size_t)b * nh + h) * S, *Dr = drow + ((size_t)b * nh + h) * S;
  float k[NT][4], v[NT][4], ak[NT][4] = {}, av_[NT][4] = {};
  r.own((const T *)av.k + koff, k);
  r.own((const T *)av.v + koff, v);
  const DropKeys keys = drop_keys(da.base, (uint32_t)(b * nh + h));
  for (int i0 = causal ? j : 0; i0 < S; i0 += 8 * U) {
    Raw4<T> q[U][NT], g[U][NT];
    float L[U], D[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = min(i0 + 8 * u + r.g, S - 1);
      r.load(qb + (size_t)i * ld, q[u]);
      r.load(gb + (size_t)i * H, g[u]);
      L[u] = Lr[i];
      D[u] = Dr[i];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + 8 * u + r.g;
      const float p = row_prob(r.dot(k, q[u]), scale, L[u]);
      float dp = r.dot(v, g[u]), pv = p;   // pv: what multiplied V in the forward
      if (da.thr != 0) {
        const bool keep = drop_bits((uint32_t)i * (uint32_t)Sk + (uint32_t)j, keys.k0, keys.k1) >= da.thr;
        pv = keep ? p * da.scale : 0.f;
        dp = keep ? dp * da.scale : 0.f;
      }
      if (i < S) {
        r.add(av_, pv, g[u]);
        r.add(ak, p * (dp - D[u]), q[u]);
      }
    }
  }
  r.store(ak, scale, (T *)av.dk + koff);
  r.store(av_, 1.f, (T *)av.dv + koff);
}

// One wave a block while that leaves CUs without work (their rows then come through L1s of their own), four from there on.  Forward +
// backward, one / four: fp32, 64 rows, 4 heads of 128 7.1 + 17.0 / 7.7 + 18.6; 256 rows, 6 heads of 128 18.9 + 43.2 / 19.8 + 45.2, 8
// heads 23.7 + 58.4 / 19.9 + 50.0; bf16, 256 rows, 6 heads of 40 11.4 + 30.4 / 12.6 + 31.6, 8 heads 12.6 + 31.6 / 12.5 + 31.7.
static int waves_a_block(long rows) { return rows >= 2048 ? 4 : 1; }
static unsigned row_grid(long rows, int w) { return (unsigned)((rows + w - 1) / w); }
// The kernel of a head dimension: NT pieces of 32 columns, U (times X) batches of eight rows in flight.  Twice as many pay in the
// forward in bf16 from 64 keys on (64 rows, 2 heads of 112 8.9 / 7.7, but 2 rows 5.4 / 5.8; the backward, which holds two operands,
// 1024 rows, 8 heads of 40 199 / 211).  Three pieces, not four, for 65 to 96 columns: 1024 rows, 8 heads of 96, fp32 273 + 520 / 224 + 423.
#define DP_ATTN_ROWS(KERN, X, rows, lds, ...)                                                                                  \
  do {                                                                                                                         \
    const int w = waves_a_block(rows);                                                                                         \
    const dim3 grid(row_grid(rows, w)), block(64 * w);                                                                         \
    if (dh <= 32) hipLaunchKernelGGL((KERN<T, 1, 4 * X>), grid, block, (size_t)w * (lds), s, __VA_ARGS__);                     \
    else if (dh <= 64) hipLaunchKernelGGL((KERN<T, 2, 4 * X>), grid, block, (size_t)w * (lds), s, __VA_ARGS__);                \
    else if (dh <= 96) hipLaunchKernelGGL((KERN<T, 3, 2 * X>), grid, block, (size_t)w * (lds), s, __VA_ARGS__);                \
    else hipLaunchKernelGGL((KERN<T, 4, 2 * X>), grid, block, (size_t)w * (lds), s, __VA_ARGS__);                              \
  } while (0)

template <typename T>
static hipError_t fwd_t(int B, int nh, int dh, int causal, const AttnView &v, void *o, float *lse, const DropArgs &da,
                        hipStream_t s) {
  const long rows = (long)B * nh * v.Sq;
  if (dh <= 128) {
    constexpr int X = sizeof(T) == 2 ? 2 : 1;
    if (v.Sk >= 64)
      DP_ATTN_ROWS(attn_fwd_rows_kernel, X, rows, (size_t)v.Sk * sizeof(float), v, (T *)o, lse, B, nh, dh, causal,
                   1.0f / sqrtf((float)dh), da);
    else
      DP_ATTN_ROWS(attn_fwd_rows_kernel, 1, rows, (size_t)v.Sk * sizeof(float), v, (T *)o, lse, B, nh, dh, causal,
                   1.0f / sqrtf((float)dh), da);
    return hipGetLastError();
  }
  const size_t smem = 4 * (size_t)(v.Sk + dh) * sizeof(float);
  hipLaunchKernelGGL((attn_fwd_simple_kernel<T>), dim3((unsigned)((rows + 3) / 4)), dim3(256), smem, s, v, (T *)o, lse,
                     B, nh, dh, causal, 1.0f / sqrtf((float)dh), da);
  return hipGetLastError();
}

hipError_t launch_attn_fwd_simple_view(int dtype, int B, int nh, int dh, int causal, const AttnView &v, void *o,
                                       float *lse, hipStream_t s, const DropArgs *drop) {
  if (causal && v.Sq != v.Sk) return hipErrorInvalidValue;
  if ((long)B * v.Sq * nh == 0) return hipSuccess;
  const DropArgs da = drop != nullptr && drop->thr != 0 ? *drop : DropArgs{0u, 0u, 1.f};
  return dtype == kBF16 ? fwd_t<bf16>(B, nh, dh, causal, v, o, lse, da, s)
                        : fwd_t<float>(B, nh, dh, causal, v, o, lse, da, s);
}

template <typename T>
static hipError_t bwd_t(int B, int nh, int dh, int causal, const AttnView &v, const void *o, const float *lse,
                        const void *d_o, float *ws, const DropArgs &da, hipStream_t s) {
  const long qrows = (long)B * nh * v.Sq, krows = (long)B * nh * v.Sk;
  const float scale = 1.0f / sqrtf((float)dh);
  if (dh <= 128) {
    if (qrows > 0 && v.Sk > 0) {
      DP_ATTN_ROWS(attn_bwd_dq_rows_kernel, 1, qrows, 0, v, (const T *)o, lse, (const T *)d_o, ws, B, nh, dh, causal, scale, da);
      hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    if (krows > 0)   // (no queries: dK = dV = 0 is still written)
      DP_ATTN_ROWS(attn_bwd_dkv_rows_kernel, 1, krows, 0, v, lse, (const T *)d_o, ws, B, nh, dh, causal, scale, da);
    return hipGetLastError();
  }
  const dim3 block(256);
  if (qrows > 0 && v.Sk > 0) {
    hipLaunchKernelGGL((attn_bwd_dq_simple_kernel<T>), dim3((unsigned)((qrows + 3) / 4)), block,
                       4 * (size_t)(v.Sk + 2 * dh) * sizeof(float), s, v, (const T *)o, lse, (const T *)d_o, ws, B, nh,
                       dh, causal, scale, da);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (krows > 0)   // (no queries: dK = dV = 0 is still written)
    hipLaunchKernelGGL((attn_bwd_dkv_simple_kernel<T>), dim3((unsigned)((krows + 3) / 4)), block,
                       4 * (size_t)(2 * v.Sq + 2 * dh) * sizeof(float), s, v, lse, (const T *)d_o, ws, B, nh, dh, causal,
                       scale, da);
  return hipGetLastError();
}

hipError_t launch_attn_bwd_simple_view(int dtype, int B, int nh, int dh, int causal, const AttnView &v, const void *o,
                                       const float *lse, const void *d_o, float *ws, hipStream_t s,
                                       const DropArgs *drop) {
  if (causal && v.Sq != v.Sk) return hipErrorInvalidValue;
  if ((long)B * nh == 0) return hipSuccess;
  const DropArgs da = drop != nullptr && drop->thr != 0 ? *drop : DropArgs{0u, 0u, 1.f};
  return dtype == kBF16 ? bwd_t<bf16>(B, nh, dh, causal, v, o, lse, d_o, ws, da, s)
                        : bwd_t<float>(B, nh, dh, causal, v, o, lse, d_o, ws, da, s);
}

hipError_t launch_attn_fwd_simple(int dtype, int B, int S, int nh, int dh, int causal, const void *qkv, void *o,
                                  float *lse, hipStream_t s, const DropArgs *drop) {
  return launch_attn_fwd_simple_view(dtype, B, nh, dh, causal, attn_self_view(qkv, nullptr, S, nh * dh, dtype_size(dtype)),
                                     o, lse, s, drop);
}

hipError_t launch_attn_bwd_simple(int dtype, int B, int S, int nh, int dh, int causal, const void *qkv,
                                  const void *o, const float *lse, const void *d_o, void *dqkv, float *ws,
                                  hipStream_t s, const DropArgs *drop) {
  return launch_attn_bwd_simple_view(dtype, B, nh, dh, causal, attn_self_view(qkv, dqkv, S, nh * dh, dtype_size(dtype)),
                                     o, lse, d_o, ws, s, drop);
}

}  // namespace dp
