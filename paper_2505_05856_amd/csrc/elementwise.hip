// HBM-bound kernels of the stage step: LayerNorm forward/backward, GELU
// forward/backward, column sums (bias gradients), transposes, fills.
//
// LayerNorm works one wavefront per row: a lane owns the same 8-element column
// groups in every row, so the row statistics are wave reductions and the
// dgamma/dbeta column sums accumulate in registers over the rows a block
// visits.  Cross-row reductions are two-pass and ordered (no float atomics), so
// results do not depend on scheduling.
#include "common.h"
#include "kernels.h"

#include <mutex>

#include <type_traits>

namespace dp {

// ------------------------------------------------------------------ LayerNorm
template <typename T, int NC>
__global__ __launch_bounds__(256) void ln_fwd_kernel(const T *__restrict__ x, const T *__restrict__ gamma,
                                                     const T *__restrict__ beta, T *__restrict__ y,
                                                     float *__restrict__ stats, int rows, int cols, float eps,
                                                     int rms) {
  // rms: no mean is subtracted (y = gamma * x / sqrt(mean(x^2) + eps) + beta); the statistics then
  // hold 0 where the mean would be, which is all the backward needs to know about it
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const T *xr = x + (size_t)row * cols;
  // All loads of a row go out before the first use, also those of gamma and beta where the registers hold them: with a guard around
  // each the wave waited for one before it asked for the next.  Lanes past the row read its last columns and use none of them.
  constexpr bool EARLY = NC * sizeof(T) <= 8;
  Raw8<T> xv[NC], gv[EARLY ? NC : 1], bv[EARLY ? NC : 1];
#pragma unroll
  for (int c = 0; c < NC; ++c) xv[c].load(xr + min((c * 64 + lane) * 8, cols - 8));
  if (EARLY && y != nullptr) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int col = min((c * 64 + lane) * 8, cols - 8);
      gv[EARLY ? c : 0].load(gamma + col);
      bv[EARLY ? c : 0].load(beta + col);
    }
  }
  float v[NC][8];
  float sum = 0.f;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int col = (c * 64 + lane) * 8;
    if (col < cols) {
      xv[c].unpack(v[c]);
#pragma unroll
      for (int i = 0; i < 8; ++i) sum += v[c][i];
    }
  }
  const float inv_n = 1.0f / (float)cols;
  const float mean = rms ? 0.f : wave_sum(sum) * inv_n;
  float sq = 0.f;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int col = (c * 64 + lane) * 8;
    if (col < cols) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float d = v[c][i] - mean;
        sq += d * d;
      }
    }
  }
  const float var = wave_sum(sq) * inv_n;
  const float rstd = 1.0f / sqrtf(var + eps);
  if (stats != nullptr && lane == 0) {
    stats[2 * (size_t)row] = mean;
    stats[2 * (size_t)row + 1] = rstd;
  }
  if (y == nullptr) return;
  T *yr = y + (size_t)row * cols;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int col = (c * 64 + lane) * 8;
    if (col < cols) {
      float g[8], b[8], o[8];
      if (EARLY) { gv[EARLY ? c : 0].unpack(g); bv[EARLY ? c : 0].unpack(b); }
      else { load8(gamma + col, g); load8(beta + col, b); }
#pragma unroll
      for (int i = 0; i < 8; ++i) o[i] = g[i] * ((v[c][i] - mean) * rstd) + b[i];
      store8(yr + col, o);
    }
  }
}

// Pass 1 of LayerNorm backward.  Block b handles rows [b*rpb, (b+1)*rpb), one
// wave per row; writes dx and the block's partial row (dgamma | dbeta [| colsum(dx)])
// into part[b][NV*cols], NV = 3 with SUMDX (the column sums of the stored dx are the
// bias gradient of the linear layer that produced LayerNorm's input).
// AHEAD: a wave asks for its next row while it works on the current one (pays when a wave has
// several rows; with two rows a wave the registers it takes cost more than it returns).
// NW waves a block: with 4 a wave has two rows and more; the form of 8 (not AHEAD, blocks of at most eight rows) gives each row of
// a block a wave of its own; the second four leave xhat where the others have dgamma (their dbeta is dy), see the sums' order.
template <typename T, int NC, bool SUMDX, bool AHEAD, int NW>
__global__ __launch_bounds__(64 * NW) void ln_bwd_kernel(const T *dy /* may alias dx */, const T *__restrict__ x,
                                                     const float *__restrict__ stats, const T *__restrict__ gamma,
                                                     const T *__restrict__ dres, T *dx,
                                                     float *__restrict__ part, int rows, int cols, int rpb, int rms) {
  // rms: the forward subtracted no mean (its statistics say mean = 0), so the term that carries the
  // derivative of the mean, mean(g), drops out: dx = rstd (g - xhat mean(g xhat))
  constexpr int NV = SUMDX ? 3 : 2;
  __shared__ float red[NW][NV][512];
  const int lane = threadIdx.x & 63;
  const int wave = NW == 8 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : threadIdx.x >> 6;
  const int row_end = min(rows, (int)(blockIdx.x + 1) * rpb);
  float dg[NC][8], db[NC][8], ds[SUMDX ? NC : 1][8];
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int i = 0; i < 8; ++i) { dg[c][i] = 0.f; db[c][i] = 0.f; if (SUMDX) ds[c][i] = 0.f; }
  const float inv_n = 1.0f / (float)cols;
  // the row stays in registers between the row reductions and the output (wider ones: ln_bwd_wide_kernel)
  static_assert(NC <= 4, "rows of up to 2048 columns");
  if constexpr (AHEAD) {
    // Everything a row needs from memory (x, dy, its statistics, the residual gradient) is asked
    // for while the row before it is being worked on and waits in registers as loaded, so a row
    // costs the wave one trip to memory that overlaps the previous row's work, instead of two in
    // a row (inputs, then the residual gradient).  gamma stays in registers for all rows.
    Raw8<T> xr[NC], dr[NC], rr[NC], gr[NC];
    float mean_n = 0.f, rstd_n = 0.f;
    auto fetch = [&](int row) {
      if (row >= row_end) return;
      const size_t base = (size_t)row * cols;
      mean_n = stats[2 * (size_t)row];
      rstd_n = stats[2 * (size_t)row + 1];
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int col = (c * 64 + lane) * 8;
        if (col < cols) {
          xr[c].load(x + base + col);
          dr[c].load(dy + base + col);
        }
      }
    };
    auto fetch_res = [&](int row) {   // (after the row before it has used its own: one buffer does)
      if (dres == nullptr || row >= row_end) return;
      const size_t base = (size_t)row * cols;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int col = (c * 64 + lane) * 8;
        if (col < cols) rr[c].load(dres + base + col);
      }
    };
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int col = (c * 64 + lane) * 8;
      if (col < cols) gr[c].load(gamma + col);
    }
    fetch(blockIdx.x * rpb + wave);
    fetch_res(blockIdx.x * rpb + wave);
    for (int row = blockIdx.x * rpb + wave; row < row_end; row += NW) {
      const float mean = mean_n, rstd = rstd_n;
      const size_t base = (size_t)row * cols;
      float xh[NC][8], g[NC][8];
      float s1 = 0.f, s2 = 0.f;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int col = (c * 64 + lane) * 8;
        if (col < cols) {
          float d[8], gm[8];
          xr[c].unpack(xh[c]);
          dr[c].unpack(d);
          gr[c].unpack(gm);
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            xh[c][i] = (xh[c][i] - mean) * rstd;
            dg[c][i] += d[i] * xh[c][i];
            db[c][i] += d[i];
            g[c][i] = d[i] * gm[i];
            s1 += g[c][i];
            s2 += g[c][i] * xh[c][i];
          }
        }
      }
      fetch(row + NW);   // the wave's next row (another row of dy: the store below cannot touch it)
      const float m1 = rms ? 0.f : wave_sum(s1) * inv_n, m2 = wave_sum(s2) * inv_n;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int col = (c * 64 + lane) * 8;
        if (col < cols) {
          float o[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) o[i] = rstd * (g[c][i] - m1 - xh[c][i] * m2);
          if (dres != nullptr) {
            float r[8];
            rr[c].unpack(r);
#pragma unroll
            for (int i = 0; i < 8; ++i) o[i] += r[i];
          }
          store8(dx + base + col, o);
          if (SUMDX) {
#pragma unroll
            for (int i = 0; i < 8; ++i) ds[c][i] += (float)(T)o[i];   // the value as stored
          }
        }
      }
      fetch_res(row + NW);
    }
  } else {
    for (int row = blockIdx.x * rpb + wave; row < row_end; row += NW) {
      const float mean = stats[2 * (size_t)row], rstd = stats[2 * (size_t)row + 1];
      const size_t base = (size_t)row * cols;
      float xh[NC][8], g[NC][8];
      float s1 = 0.f, s2 = 0.f;
      Raw8<T> rr[NW > 4 ? NC : 1];   // the residual gradient, asked for with the rest where a wave has one row
      if (NW > 4 && dres != nullptr) {
  #pragma unroll
        for (int c = 0; c < NC; ++c) {
          const int col = (c * 64 + lane) * 8;
          if (col < cols) rr[NW > 4 ? c : 0].load(dres + base + col);
        }
      }
  #pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int col = (c * 64 + lane) * 8;
        if (col < cols) {
          float d[8], gm[8];
          load8(x + base + col, xh[c]);
          load8(dy + base + col, d);
          load8(gamma + col, gm);
  #pragma unroll
          for (int i = 0; i < 8; ++i) {
            xh[c][i] = (xh[c][i] - mean) * rstd;
            if (NW == 8 && wave >= 4) dg[c][i] = xh[c][i]; else dg[c][i] += d[i] * xh[c][i];
            db[c][i] += d[i];
            g[c][i] = d[i] * gm[i];
            s1 += g[c][i];
            s2 += g[c][i] * xh[c][i];
          }
        }
      }
      const float m1 = rms ? 0.f : wave_sum(s1) * inv_n, m2 = wave_sum(s2) * inv_n;
  #pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int col = (c * 64 + lane) * 8;
        if (col < cols) {
          float o[8];
  #pragma unroll
          for (int i = 0; i < 8; ++i) o[i] = rstd * (g[c][i] - m1 - xh[c][i] * m2);
          if (dres != nullptr) {
            float r[8];
            if (NW > 4) rr[NW > 4 ? c : 0].unpack(r); else load8(dres + base + col, r);
  #pragma unroll
            for (int i = 0; i < 8; ++i) o[i] += r[i];
          }
          store8(dx + base + col, o);
          if (SUMDX) {
  #pragma unroll
            for (int i = 0; i < 8; ++i) ds[c][i] += (float)(T)o[i];   // the value as stored
          }
        }
      }
    }
  }
  // ordered block reduction of the waves' column partials, 512 columns at a time
  float *prow = part + (size_t)blockIdx.x * NV * cols;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    if (c * 512 >= cols) break;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      red[wave][0][lane * 8 + i] = dg[c][i];
      red[wave][1][lane * 8 + i] = db[c][i];
      if (SUMDX) red[wave][NV - 1][lane * 8 + i] = ds[c][i];
    }
    __syncthreads();
    if constexpr (NW == 8) {
      // wave w + 4 has the row that comes second in wave w of four: it is added to that wave's sums first (dgamma's product
      // unrounded), so the two forms give the same bits
      const int k = threadIdx.x, col = c * 512 + k;
      if (col < cols) {
        float t[NV];
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          float v[NV];
#pragma unroll
          for (int n = 1; n < NV; ++n) v[n] = red[w][n][k] + red[w + 4][n][k];
          v[0] = __builtin_fmaf(red[w + 4][1][k], red[w + 4][0][k], red[w][0][k]);
#pragma unroll
          for (int n = 0; n < NV; ++n) t[n] = w == 0 ? v[n] : t[n] + v[n];
        }
#pragma unroll
        for (int n = 0; n < NV; ++n) prow[(size_t)n * cols + col] = t[n];
      }
    } else {
      for (int j = threadIdx.x; j < NV * 512; j += 256) {
        const int which = j >> 9, k = j & 511;
        const int col = c * 512 + k;
        if (col < cols) {
          const float t = ((red[0][which][k] + red[1][which][k]) + red[2][which][k]) + red[3][which][k];
          prow[(size_t)which * cols + col] = t;
        }
      }
    }
  }
}

// a + b with both rounded before (no fused multiply-add where one of them is a product)
__device__ __forceinline__ float add_rounded(float a, float b) {
#pragma clang fp contract(off)
  return a + b;
}

// LayerNorm backward for wide rows (more than 2048 columns): a block per row, the columns
// dealt out over its 256 threads (thread t owns the 8-column groups t, t + 256, ...), rows of
// the block's range one after the other.  A thread's column accumulators are then complete sums
// over the block's rows (no reduction across waves at the end), gamma stays in registers, and a
// thread holds 16..32 elements of a row instead of 64..128: several blocks fit a CU where the
// wave-per-row form fits one or two waves a SIMD.  The two row sums cross the waves through LDS
// (one barrier a row; two alternating slots); the next row's loads are issued before that.
// RES says whether there is a residual gradient, and no load has a guard: rows past the block's range are fetched as
// copies of its last row, columns past the row as its last ones, and never used.  (With branches around the loads the
// compiler can no longer count which of the loads in flight a use needs and waits for all of them, which leaves one row
// in flight instead of PF: 8000x2560 bf16 with a residual gradient 67 us, now 45; 16384x4000 147 and 117.)
// FULL: the row is exactly NP * 2048 columns wide and every block has a multiple of four rows, so nothing is guarded at all.  (In fp32
// its additions of the residual gradient and to the sums of dx take dx before it is rounded, the other form's after.)
template <typename T, int NP, bool SUMDX, bool FULL, bool RES>
__global__ __launch_bounds__(256) void ln_bwd_wide_kernel(const T *dy /* may alias dx */, const T *__restrict__ x,
                                                          const float *__restrict__ stats,
                                                          const T *__restrict__ gamma, const T *__restrict__ dres,
                                                          T *dx, float *__restrict__ part, int rows, int cols,
                                                          int rpb, int rms) {
  constexpr int NV = SUMDX ? 3 : 2;
  __shared__ float red[2][2][4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row0 = blockIdx.x * rpb, row_end = min(rows, row0 + rpb);
  float gm[NP][8], dg[NP][8], db[NP][8], ds[SUMDX ? NP : 1][8];
#pragma unroll
  for (int c = 0; c < NP; ++c) {
    const int col = (c * 256 + tid) * 8;
    if (FULL || col < cols) load8(gamma + col, gm[c]);
#pragma unroll
    for (int i = 0; i < 8; ++i) { dg[c][i] = 0.f; db[c][i] = 0.f; if (SUMDX) ds[c][i] = 0.f; }
  }
  const float inv_n = 1.0f / (float)cols;
  // PF rows are in flight per block (a block is one wave per SIMD and only a few blocks share a
  // CU, so the loads of several rows ahead are what keeps the memory system busy).  They wait in
  // registers as loaded (8 bf16 in 4 registers) and are widened when their row is worked on; the
  // row's two statistics travel with them, and the residual gradient of a row is asked for one
  // row ahead, so that no load is issued and awaited inside a row's own work.
  constexpr int PF = 2;
  Raw8<T> xn[PF][NP], dn[PF][NP], rn[2][NP];
  float mean_n[PF], rstd_n[PF];
  auto col_at = [&](int c) { const int col = (c * 256 + tid) * 8; return FULL ? col : min(col, cols - 8); };
  auto fetch = [&](int row, auto buf_tag) {
    constexpr int BUF = decltype(buf_tag)::value;
    row = min(row, row_end - 1);
    const size_t base = (size_t)row * cols;
    mean_n[BUF] = stats[2 * (size_t)row];
    rstd_n[BUF] = stats[2 * (size_t)row + 1];
#pragma unroll
    for (int c = 0; c < NP; ++c) {
      xn[BUF][c].load(x + base + col_at(c));
      dn[BUF][c].load(dy + base + col_at(c));
    }
  };
  auto fetch_res = [&](int row, auto par_tag) {
    constexpr int PAR = decltype(par_tag)::value;
    if (!RES) return;
    const size_t base = (size_t)min(row, row_end - 1) * cols;
#pragma unroll
    for (int c = 0; c < NP; ++c) rn[PAR][c].load(dres + base + col_at(c));
  };
  auto process = [&](int row, auto buf_tag, auto par_tag) {
    constexpr int BUF = decltype(buf_tag)::value;
    constexpr int PAR = decltype(par_tag)::value;
    const float mean = mean_n[BUF], rstd = rstd_n[BUF];
    const size_t base = (size_t)row * cols;
    const bool own = FULL || row < row_end;   // (the last rows of a block come in fours too)
    fetch_res(row + 1, std::integral_constant<int, 1 - PAR>{});
    float xh[NP][8], g[NP][8];
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int c = 0; c < NP; ++c) {
      const int col = (c * 256 + tid) * 8;
      if (FULL || (own && col < cols)) {
        float xv[8], dv[8];
        xn[BUF][c].unpack(xv);
        dn[BUF][c].unpack(dv);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          xh[c][i] = (xv[i] - mean) * rstd;
          dg[c][i] += dv[i] * xh[c][i];
          db[c][i] += dv[i];
          g[c][i] = dv[i] * gm[c][i];
          s1 += g[c][i];
          s2 += g[c][i] * xh[c][i];
        }
      }
    }
    fetch(row + PF, buf_tag);   // this buffer's next row
    s1 = wave_sum(s1); s2 = wave_sum(s2);
    const int slot = (row - row0) & 1;
    if (lane == 0) { red[slot][0][wave] = s1; red[slot][1][wave] = s2; }
    __syncthreads();
    const float m1 = rms ? 0.f : (((red[slot][0][0] + red[slot][0][1]) + red[slot][0][2]) + red[slot][0][3]) * inv_n;
    const float m2 = (((red[slot][1][0] + red[slot][1][1]) + red[slot][1][2]) + red[slot][1][3]) * inv_n;
#pragma unroll
    for (int c = 0; c < NP; ++c) {
      const int col = (c * 256 + tid) * 8;
      if (FULL || (own && col < cols)) {
        float o[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) o[i] = rstd * (g[c][i] - m1 - xh[c][i] * m2);
        if (RES) {
          float r[8];
          rn[PAR][c].unpack(r);
#pragma unroll
          for (int i = 0; i < 8; ++i) o[i] = FULL ? o[i] + r[i] : add_rounded(o[i], r[i]);
        }
        store8(dx + base + col, o);
        if (SUMDX) {
#pragma unroll
          for (int i = 0; i < 8; ++i) {   // the value as stored
            const float v = (float)(T)o[i];
            ds[c][i] = FULL ? ds[c][i] + v : add_rounded(ds[c][i], v);
          }
        }
      }
    }
  };
  using I0 = std::integral_constant<int, 0>; using I1 = std::integral_constant<int, 1>;
  fetch(row0, I0{});
  fetch(row0 + 1, I1{});
  fetch_res(row0, I0{});
  // (the trip count of the loop is the same for every thread of the block: the barriers inside match;
  //  rows alternate between the two buffers)
  for (int row = row0; row < row_end; row += 4) {
    // (fences: the rows' instruction streams stay apart, or their temporaries add up)
    process(row, I0{}, I0{});
    __builtin_amdgcn_sched_barrier(0);
    process(row + 1, I1{}, I1{});
    __builtin_amdgcn_sched_barrier(0);
    process(row + 2, I0{}, I0{});
    __builtin_amdgcn_sched_barrier(0);
    process(row + 3, I1{}, I1{});
    __builtin_amdgcn_sched_barrier(0);
  }
  float *prow = part + (size_t)blockIdx.x * NV * cols;
#pragma unroll
  for (int c = 0; c < NP; ++c) {
    const int col = (c * 256 + tid) * 8;
    if (FULL || col < cols) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        prow[col + i] = dg[c][i];
        prow[(size_t)cols + col + i] = db[c][i];
        if (SUMDX) prow[2 * (size_t)cols + col + i] = ds[c][i];
      }
    }
  }
}

// Pass 2: out[j] = sum_{b<nb} part[b][j], summed in a fixed order; column j of the
// `width`-wide partial rows goes to out[j / seg][j % seg].  Block = 64 columns x 16 row groups.
template <typename T>
__global__ __launch_bounds__(1024) void reduce_partials_kernel(const float *__restrict__ part, int nb, int width,
                                                               T *__restrict__ out0, T *__restrict__ out1,
                                                               T *__restrict__ out2, int seg) {
  __shared__ float red[16][64];
  const int cx = threadIdx.x & 63, g = threadIdx.x >> 6;
  const int col = blockIdx.x * 64 + cx;
  float s = 0.f;
  if (col < width) {
    // batches of 8 independent loads: the kernel is latency-bound, not bandwidth-bound
    int b = g;
    for (; b + 7 * 16 < nb; b += 8 * 16) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = part[(size_t)(b + u * 16) * width + col];
#pragma unroll
      for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; b < nb; b += 16) s += part[(size_t)b * width + col];
  }
  red[g][cx] = s;
  __syncthreads();
  if (g == 0 && col < width) {
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) t += red[i][cx];
    const int which = col / seg, k = col - which * seg;
    stf((which == 0 ? out0 : which == 1 ? out1 : out2) + k, t);
  }
}

// The same pass for up to kMaxReduceJobs reductions in one launch: block b belongs to the job
// whose block range contains it and does exactly what reduce_partials_kernel does for it.
struct ReduceJobTable {
  ReduceJob job[kMaxReduceJobs];
  int first_block[kMaxReduceJobs + 1];
  int n;
};
template <typename T>
__global__ __launch_bounds__(1024) void reduce_jobs_kernel(ReduceJobTable t) {
  __shared__ float red[16][64];
  int j = 0;
  while (j + 1 < t.n && (int)blockIdx.x >= t.first_block[j + 1]) ++j;
  const ReduceJob &job = t.job[j];
  const float *__restrict__ part = job.part;
  const int nb = job.nb, width = job.width;
  const int cx = threadIdx.x & 63, g = threadIdx.x >> 6;
  const int col = ((int)blockIdx.x - t.first_block[j]) * 64 + cx;
  float s = 0.f;
  if (col < width) {
    int b = g;
    for (; b + 7 * 16 < nb; b += 8 * 16) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = part[(size_t)(b + u * 16) * width + col];
#pragma unroll
      for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; b < nb; b += 16) s += part[(size_t)b * width + col];
  }
  red[g][cx] = s;
  __syncthreads();
  if (g == 0 && col < width) {
    float tsum = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) tsum += red[i][cx];
    const int which = col / job.seg, k = col - which * job.seg;
    T *dst = (T *)(which == 0 ? job.out0 : which == 1 ? job.out1 : job.out2) + k;
    stf(dst, job.accumulate ? tsum + ldf(dst) : tsum);
  }
}

// Column sums of x [rows, cols]: block (cx, rb) covers 512 columns and rows
// [rb*rpb, (rb+1)*rpb); partial row rb of part[nrb][cols].
template <typename T>
__global__ __launch_bounds__(256) void colsum_kernel(const T *__restrict__ x, float *__restrict__ part, int rows,
                                                     int cols, int rpb) {
  __shared__ float red[4][512];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int col = (blockIdx.x * 64 + lane) * 8;
  const int row_end = min(rows, (int)(blockIdx.y + 1) * rpb);
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (col < cols) {
    for (int row = blockIdx.y * rpb + wave; row < row_end; row += 4) {
      float v[8];
      load8(x + (size_t)row * cols + col, v);
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] += v[i];
    }
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) red[wave][lane * 8 + i] = acc[i];
  __syncthreads();
  for (int k = threadIdx.x; k < 512; k += 256) {
    const int c = blockIdx.x * 512 + k;
    if (c < cols) part[(size_t)blockIdx.y * cols + c] = ((red[0][k] + red[1][k]) + red[2][k]) + red[3][k];
  }
}

// ------------------------------------------------------------------ dropout of a hidden state
// y = (res ? res : 0) + keep * scale * x over n elements (8 a thread); element i's decision is
// drop_bits(i, keys of unit 0).  Forward: x is a linear layer's output, res the residual
// branch.  Backward: x is the gradient of y, no res.
template <typename T>
__global__ __launch_bounds__(256) void dropout_kernel(const T *x /* may alias y */, const T *res /* may alias y */,
                                                      T *y, size_t n8, DropArgs a) {
  const DropKeys k = drop_keys(a.base, 0u);
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n8; i += (size_t)gridDim.x * 256) {
    float v[8], r[8];
    load8(x + i * 8, v);
    if (res != nullptr) load8(res + i * 8, r);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const bool keep = drop_bits((uint32_t)(i * 8 + q), k.k0, k.k1) >= a.thr;
      const float d = keep ? v[q] * a.scale : 0.f;
      v[q] = res != nullptr ? r[q] + d : d;
    }
    store8(y + i * 8, v);
  }
}

// The sum over a block's waves of column k in the order of four waves: with sixteen, a row each, waves w, w + 4, w + 8 and w + 12
// have the rows that wave w of four adds up.
template <int NW> __device__ __forceinline__ float sum_waves(const float (&red)[NW][512], int k) {
  float t = 0.f;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    float v = red[w][k];
#pragma unroll
    for (int u = w + 4; u < NW; u += 4) v += red[u][k];
    t = w == 0 ? v : t + v;
  }
  return t;
}

// y = keep * scale * x over [rows, cols] and the column sums of the stored y, in partial rows as colsum_kernel's: the gradient of
// a dropped hidden state on its way into the linear layer, whose bias gradient the sums are.  One wave a row up to four blocks a CU
// (the draws are vector work, see gelu_bwd_colsum_kernel).
template <typename T, int NW>
__global__ __launch_bounds__(64 * NW) void dropout_colsum_kernel(const T *__restrict__ x, T *__restrict__ y,
                                                                 float *__restrict__ part, int rows, int cols, int rpb, DropArgs a) {
  __shared__ float red[NW][512];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int col = (blockIdx.x * 64 + lane) * 8;
  const int row_end = min(rows, (int)(blockIdx.y + 1) * rpb);
  const DropKeys k = drop_keys(a.base, 0u);
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (col < cols) {
    for (int row = blockIdx.y * rpb + wave; row < row_end; row += NW) {
      const size_t at = (size_t)row * cols + col;
      float v[8];
      load8(x + at, v);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const bool keep = drop_bits((uint32_t)(at + i), k.k0, k.k1) >= a.thr;
        v[i] = keep ? v[i] * a.scale : 0.f;
        acc[i] += (float)(T)v[i];
      }
      store8(y + at, v);
    }
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) red[wave][lane * 8 + i] = acc[i];
  __syncthreads();
  for (int j = threadIdx.x; j < 512; j += 64 * NW) {
    const int c = blockIdx.x * 512 + j;
    if (c < cols) {
      const float t = sum_waves<NW>(red, j);
      part[(size_t)blockIdx.y * cols + c] = t;
    }
  }
}

// ------------------------------------------------------------------ GELU
template <typename T>
__global__ __launch_bounds__(256) void gelu_fwd_kernel(const T *__restrict__ x, T *__restrict__ y, size_t n8,
                                                       int kind) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n8; i += (size_t)gridDim.x * 256) {
    float v[8];
    load8(x + i * 8, v);
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = gelu_f<T>(v[k], kind);
    store8(y + i * 8, v);
  }
}

// dx = dy * gelu'(x) over [rows, cols] plus the column sums of the stored dx (the bias
// gradient of the linear layer in front of the GELU): block (cx, rb) covers 512 columns
// and rows [rb*rpb, (rb+1)*rpb); its partial sums go to part[rb][cols].
template <typename T, int NW>
__global__ __launch_bounds__(64 * NW) void gelu_bwd_colsum_kernel(const T *dy /* may alias dx */,
                                                              const T *__restrict__ x, T *dx,
                                                              float *__restrict__ part, int rows, int cols, int rpb,
                                                              int kind) {
  __shared__ float red[NW][512];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int col = (blockIdx.x * 64 + lane) * 8;
  const int row_end = min(rows, (int)(blockIdx.y + 1) * rpb);
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (col < cols) {
    for (int row = blockIdx.y * rpb + wave; row < row_end; row += NW) {
      const size_t at = (size_t)row * cols + col;
      float v[8], d[8];
      load8(x + at, v);
      load8(dy + at, d);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        v[i] = d[i] * gelu_df<T>(v[i], kind);
        acc[i] += (float)(T)v[i];
      }
      store8(dx + at, v);
    }
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) red[wave][lane * 8 + i] = acc[i];
  __syncthreads();
  for (int k = threadIdx.x; k < 512; k += 64 * NW) {
    const int c = blockIdx.x * 512 + k;
    if (c < cols) {
      const float t = sum_waves<NW>(red, k);
      part[(size_t)blockIdx.y * cols + c] = t;
    }
  }
}

// ------------------------------------------------------------------ few rows: whole columns in one launch
// With few rows a launch is a chain of latencies, and a second launch for the column sums (reduce_partials_kernel) costs
// as much as the work: here a block of 1024 threads owns SC columns (a slab) over all rows, so the sums are complete in it.
// A thread owns 8 of the columns in every 1024/(SC/8)-th row, and its loads of U such rows (U: as many as the launcher's row limit
// leaves it, four at most) are in flight together.

// The block's sums of one vector: `acc` holds a thread's 8 columns.  Rows of a wave by lane exchange, waves through LDS, in a
// fixed order.
template <typename T, int SC>
__device__ __forceinline__ void slab_sums(float (&acc)[8], float (&red)[16][SC], T *__restrict__ out, int col0, int cols) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int m = SC / 8; m <= 32; m <<= 1) acc[i] += __shfl_xor(acc[i], m, 64);
  if (lane < SC / 8)
#pragma unroll
    for (int i = 0; i < 8; ++i) red[wave][lane * 8 + i] = acc[i];
  __syncthreads();
  const int k = threadIdx.x;
  if (k < SC && col0 + k < cols) {
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < 16; ++w) t += red[w][k];
    stf(out + col0 + k, t);
  }
}

// f(row) for every row of this thread's, U of its `load`s ahead of their `use`s
template <int SC, int U, typename Load, typename Use>
__device__ __forceinline__ void slab_rows(int rows, Load &&load, Use &&use) {
  constexpr int STEP = 1024 / (SC / 8);   // rows the block takes at a time
  for (int r0 = threadIdx.x / (SC / 8); r0 < rows; r0 += U * STEP) {
#pragma unroll
    for (int u = 0; u < U; ++u) load(min(r0 + STEP * u, rows - 1), u);   // (rows past the last: not used)
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (r0 + STEP * u < rows) use(r0 + STEP * u, u);
  }
}
// rows up to which the launchers choose the one-launch forms (figures there), and the U for a kernel of at most `limit` rows
constexpr int kColsumSlabRows = 1800;
template <typename T> constexpr int kGeluSlabRows = 1024 / (int)sizeof(T);
template <typename T> constexpr int kLnSlabRows = sizeof(T) == 2 ? 1000 : 512;
constexpr int slab_depth(int limit, int sc) { const int n = (limit * (sc / 8) + 1023) / 1024; return n > 4 ? 4 : n; }

template <typename T, int SC>
__global__ __launch_bounds__(1024) void colsum_slab_kernel(const T *__restrict__ x, T *__restrict__ out, int rows, int cols) {
  __shared__ float red[16][SC];
  const int col0 = blockIdx.x * SC, col = col0 + (threadIdx.x % (SC / 8)) * 8;
  constexpr int U = slab_depth(kColsumSlabRows, SC);
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (col < cols) {
    Raw8<T> v[U];
    slab_rows<SC, U>(rows, [&](int row, int u) { v[u].load(x + (size_t)row * cols + col); },
              [&](int, int u) {
                float a[8];
                v[u].unpack(a);
#pragma unroll
                for (int i = 0; i < 8; ++i) acc[i] += a[i];
              });
  }
  slab_sums(acc, red, out, col0, cols);
}

template <typename T, int SC>
__global__ __launch_bounds__(1024) void gelu_bwd_slab_kernel(const T *dy /* may alias dx */, const T *__restrict__ x, T *dx,
                                                             T *__restrict__ dbias, int rows, int cols, int kind) {
  __shared__ float red[16][SC];
  const int col0 = blockIdx.x * SC, col = col0 + (threadIdx.x % (SC / 8)) * 8;
  constexpr int U = slab_depth(kGeluSlabRows<T>, SC);
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (col < cols) {
    Raw8<T> v[U], g[U];
    slab_rows<SC, U>(rows,
              [&](int row, int u) {
                const size_t at = (size_t)row * cols + col;
                v[u].load(x + at);
                g[u].load(dy + at);
              },
              [&](int row, int u) {
                float a[8], d[8];
                v[u].unpack(a);
                g[u].unpack(d);
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                  a[i] = d[i] * gelu_df<T>(a[i], kind);
                  acc[i] += (float)(T)a[i];   // the value as stored
                }
                store8(dx + (size_t)row * cols + col, a);
              });
  }
  slab_sums(acc, red, dbias, col0, cols);
}

// LayerNorm backward: dgamma and dbeta need no row reductions (the statistics are given), so they come from blocks of their own
// beside those of dx: blocks 0 .. row_blocks-1 take 16 rows each, a wave a row, the others a slab each.  x and dy are read twice,
// the second time out of the caches.  No output may overlap an input (dx may be dres).
constexpr int kLnSlabCols = 32;
template <typename T, int NC>
__global__ __launch_bounds__(1024) void ln_bwd_few_kernel(const T *__restrict__ dy, const T *__restrict__ x,
                                                          const float *__restrict__ stats, const T *__restrict__ gamma,
                                                          const T *__restrict__ dres, T *__restrict__ dx, T *__restrict__ dgamma,
                                                          T *__restrict__ dbeta, int rows, int cols, int n_row_blocks, int rms) {
  constexpr int SC = kLnSlabCols, U = slab_depth(kLnSlabRows<T>, SC);
  __shared__ float red[2][16][SC];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if ((int)blockIdx.x >= n_row_blocks) {
    const int col0 = ((int)blockIdx.x - n_row_blocks) * SC, col = col0 + (threadIdx.x % (SC / 8)) * 8;
    float dg[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, db[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (col < cols) {
      Raw8<T> v[U], g[U];
      float mean[U], rstd[U];
      slab_rows<SC, U>(rows,
                [&](int row, int u) {
                  const size_t at = (size_t)row * cols + col;
                  v[u].load(x + at);
                  g[u].load(dy + at);
                  mean[u] = stats[2 * (size_t)row];
                  rstd[u] = stats[2 * (size_t)row + 1];
                },
                [&](int, int u) {
                  float a[8], d[8];
                  v[u].unpack(a);
                  g[u].unpack(d);
#pragma unroll
                  for (int i = 0; i < 8; ++i) {
                    dg[i] += d[i] * ((a[i] - mean[u]) * rstd[u]);
                    db[i] += d[i];
                  }
                });
    }
    slab_sums(dg, red[0], dgamma, col0, cols);
    slab_sums(db, red[1], dbeta, col0, cols);
    return;
  }
  const int row = blockIdx.x * 16 + wave;
  if (row >= rows) return;
  const size_t base = (size_t)row * cols;
  const float mean = stats[2 * (size_t)row], rstd = stats[2 * (size_t)row + 1], inv_n = 1.0f / (float)cols;
  float xh[NC][8], g[NC][8], r[NC][8];
  float s1 = 0.f, s2 = 0.f;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int col = (c * 64 + lane) * 8;
    if (col < cols) {
      float d[8], gm[8];
      load8(x + base + col, xh[c]);
      load8(dy + base + col, d);
      load8(gamma + col, gm);
      if (dres != nullptr) load8(dres + base + col, r[c]);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        xh[c][i] = (xh[c][i] - mean) * rstd;
        g[c][i] = d[i] * gm[i];
        s1 += g[c][i];
        s2 += g[c][i] * xh[c][i];
      }
    }
  }
  const float m1 = rms ? 0.f : wave_sum(s1) * inv_n, m2 = wave_sum(s2) * inv_n;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int col = (c * 64 + lane) * 8;
    if (col < cols) {
      float o[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) o[i] = rstd * (g[c][i] - m1 - xh[c][i] * m2);
      if (dres != nullptr)
#pragma unroll
        for (int i = 0; i < 8; ++i) o[i] += r[c][i];
      store8(dx + base + col, o);
    }
  }
}

// ------------------------------------------------------------------ misc
template <typename T>
__global__ __launch_bounds__(256) void transpose_kernel(const T *__restrict__ src, T *__restrict__ dst, int rows,
                                                        int cols) {
  __shared__ T tile[32][33];
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
  const int c0 = blockIdx.x * 32, r0 = blockIdx.y * 32;
  for (int i = ty; i < 32; i += 8)
    if (r0 + i < rows && c0 + tx < cols) tile[i][tx] = src[(size_t)(r0 + i) * cols + c0 + tx];
  __syncthreads();
  for (int i = ty; i < 32; i += 8)
    if (c0 + i < cols && r0 + tx < rows) dst[(size_t)(c0 + i) * rows + r0 + tx] = tile[tx][i];
}

__global__ __launch_bounds__(256) void fill_u32_kernel(uint32_t *p, size_t n, uint32_t pattern) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) p[i] = pattern;
}

// ------------------------------------------------------------------ launchers
bool ln_supported(int dtype, int cols) {
  (void)dtype;
  return cols > 0 && cols % 8 == 0 && cols <= 8192;
}

static int ln_chunks(int cols) {
  const int c = (cols + 511) / 512;
  return c <= 1 ? 1 : c <= 2 ? 2 : c <= 4 ? 4 : c <= 8 ? 8 : 16;
}

template <typename T>
static hipError_t ln_fwd_t(int rows, int cols, float eps, const void *x, const void *gamma, const void *beta,
                           void *y, float *stats, hipStream_t s, int rms) {
  const dim3 grid((rows + 3) / 4), block(256);
#define DP_LN_FWD(NC)                                                                                       \
  hipLaunchKernelGGL((ln_fwd_kernel<T, NC>), grid, block, 0, s, (const T *)x, (const T *)gamma,             \
                     (const T *)beta, (T *)y, stats, rows, cols, eps, rms)
  switch (ln_chunks(cols)) {
    case 1: DP_LN_FWD(1); break;
    case 2: DP_LN_FWD(2); break;
    case 4: DP_LN_FWD(4); break;
    case 8: DP_LN_FWD(8); break;
    default: DP_LN_FWD(16); break;
  }
#undef DP_LN_FWD
  return hipGetLastError();
}

hipError_t launch_ln_fwd(int dtype, int rows, int cols, float eps, const void *x, const void *gamma,
                         const void *beta, void *y, float *stats, hipStream_t s, bool rms) {
  if (rows <= 0) return hipSuccess;
  return dtype == kBF16 ? ln_fwd_t<bf16>(rows, cols, eps, x, gamma, beta, y, stats, s, rms ? 1 : 0)
                        : ln_fwd_t<float>(rows, cols, eps, x, gamma, beta, y, stats, s, rms ? 1 : 0);
}

// Where the one-launch forms end (two launches / one, us, in calls one after the other; in a captured graph, where the host's part
// is gone.  Operands from memory, where a slab's short pieces of many rows cost more; in the caches the lines would lie further out):
//   column sums: bf16 1800x1024 9.4 / 6.2; 7.1 / 6.3, 1800x3064 9.6 / 8.3; 9.5 / 8.5, but 2048x1024 in a graph 5.6 / 6.7; fp32
//     1800x1024 9.4 / 6.2; 8.1 / 7.7, but 1800x1528 9.4 / 9.8; 9.2 / 10.3: up to 1800 rows and 8 MiB
//   GELU backward (16 columns a slab up to 1024, 32 from there on): bf16 512x1024 9.8 / 5.4; 9.3 / 5.6, 512x6400 11.6 / 8.9;
//     12.1 / 9.2, but 512x11008 13.2 / 16.4; 13.6 / 15.6; fp32 256x6400 10.9 / 7.7; 11.4 / 8.2, but 256x11008 12.4 / 13.9;
//     12.8 / 13.9, and 500x1024 7.4 / 7.5, 1000x1024 7.9 / 13.2 (on a faster host): 512 and 256 rows, and 8 MiB
//   LayerNorm backward: bf16 1000x768 9.1 / 7.5, 850x1024 in a graph 9.9 / 8.0, but 1024x512 in a graph 7.0 / 8.3 and 1500x1024 9.8 / 11.5;
//     fp32 512x1024 in a graph 9.1 / 7.1, but 1024x1024 9.3 / 11.3: 1000 and 512 rows
constexpr size_t kSlabBytes = (size_t)8 << 20;
// The sums are written while other blocks still read: calls whose outputs lie in what those read keep the two launches.
static bool overlap(const void *a, size_t na, const void *b, size_t nb) {
  const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
  return a != nullptr && b != nullptr && x < y + nb && y < x + na;
}

template <typename T>
static hipError_t ln_bwd_few_t(int rows, int cols, const void *dy, const void *x, const float *stats, const void *gamma,
                               const void *dres, void *dx, void *dgamma, void *dbeta, hipStream_t s, int rms) {
  const int nrb = (rows + 15) / 16;
  const dim3 grid(nrb + (cols + kLnSlabCols - 1) / kLnSlabCols);
#define DP_LN_BWD_FEW(NC)                                                                                              \
  hipLaunchKernelGGL((ln_bwd_few_kernel<T, NC>), grid, dim3(1024), 0, s, (const T *)dy, (const T *)x, stats,             \
                     (const T *)gamma, (const T *)dres, (T *)dx, (T *)dgamma, (T *)dbeta, rows, cols, nrb, rms)
  switch (ln_chunks(cols)) {
    case 1: DP_LN_BWD_FEW(1); break;
    case 2: DP_LN_BWD_FEW(2); break;
    default: DP_LN_BWD_FEW(4); break;
  }
#undef DP_LN_BWD_FEW
  return hipGetLastError();
}

// second pass now, or left to the caller as a job
template <typename T>
static hipError_t reduce_or_defer(const float *part, int nb, int width, int seg, void *o0, void *o1, void *o2,
                                  hipStream_t s, ReduceJob *job) {
  if (job != nullptr) { *job = ReduceJob{part, nb, width, seg, o0, o1, o2, 0}; return hipSuccess; }
  hipLaunchKernelGGL((reduce_partials_kernel<T>), dim3((width + 63) / 64), dim3(1024), 0, s, part, nb, width, (T *)o0,
                     (T *)o1, (T *)o2, seg);
  return hipGetLastError();
}

template <typename T, bool SUMDX>
static hipError_t ln_bwd_t(int rows, int cols, const void *dy, const void *x, const float *stats,
                           const void *gamma, const void *dres, void *dx, void *dgamma, void *dbeta, void *dxsum,
                           void *ws, hipStream_t s, ReduceJob *job, int rms) {
  // A row a wave (us, both passes, 4 waves a block / 8, operands in the caches; from memory): up to 256 blocks, one a CU, at any
  // width (with the sums of dx bf16 2048x2048 16.2 / 13.4; 17.8 / 14.4, but 2049x2048 16.2 / 17.6; 17.9 / 21.1), and for rows of up
  // to 2 KB up to 512 blocks (bf16 4096x1024 14.2 / 13.0; 13.8 / 13.6, fp32 4096x512 11.5 / 9.9; 11.8 / 11.6, but 3072x768 12.5 / 13.1;
  // 13.5 / 15.1), with a residual gradient too up to 384 (bf16 3072x1024 13.0 / 11.5; 13.6 / 13.2, 3600x1024 14.8 / 13.6; 15.5 / 15.6).
  const bool row_a_wave = rows <= 2048 || (cols * sizeof(T) <= 2048 && rows <= (dres == nullptr ? 4096 : 3072));
  int rpb;
  const int nb = row_blocks(rows, 8, &rpb);
  const int nv = SUMDX ? 3 : 2;
  float *part = (float *)ws;
#define DP_LN_BWD_AS(NC, AHEAD, NW)                                                                                    \
  hipLaunchKernelGGL((ln_bwd_kernel<T, NC, SUMDX, AHEAD, NW>), dim3(nb), dim3(64 * NW), 0, s, (const T *)dy, (const T *)x, \
                     stats, (const T *)gamma, (const T *)dres, (T *)dx, part, rows, cols, rpb, rms)
#define DP_LN_BWD(NC)                                                               \
  do {                                                                              \
    if (row_a_wave) DP_LN_BWD_AS(NC, false, 8);                                     \
    else if (NC <= 2 || rpb >= 16) DP_LN_BWD_AS(NC, true, 4);                       \
    else DP_LN_BWD_AS(4, false, 4);   /* (NC = 4) */                                \
  } while (0)
#define DP_LN_BWD_WIDE_AS(NP, FULL, RES)                                                                      \
  hipLaunchKernelGGL((ln_bwd_wide_kernel<T, NP, SUMDX, FULL, RES>), dim3(nb), dim3(256), 0, s, (const T *)dy, \
                     (const T *)x, stats, (const T *)gamma, (const T *)dres, (T *)dx, part, rows, cols, rpb, rms)
#define DP_LN_BWD_WIDE(NP)                                                    \
  do {                                                                        \
    const bool full = cols == NP * 2048 && rows % 4 == 0 && rpb % 4 == 0;     \
    if (dres != nullptr) {                                                    \
      if (full) DP_LN_BWD_WIDE_AS(NP, true, true); else DP_LN_BWD_WIDE_AS(NP, false, true);    \
    } else {                                                                  \
      if (full) DP_LN_BWD_WIDE_AS(NP, true, false); else DP_LN_BWD_WIDE_AS(NP, false, false);  \
    }                                                                         \
  } while (0)
  switch (ln_chunks(cols)) {
    case 1: DP_LN_BWD(1); break;
    case 2: DP_LN_BWD(2); break;
    case 4: DP_LN_BWD(4); break;
    case 8: DP_LN_BWD_WIDE(2); break;     // 2049..4096 columns
    default: DP_LN_BWD_WIDE(4); break;    // up to 8192
  }
#undef DP_LN_BWD_WIDE
#undef DP_LN_BWD_WIDE_AS
#undef DP_LN_BWD
#undef DP_LN_BWD_AS
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return reduce_or_defer<T>(part, nb, nv * cols, cols, dgamma, dbeta, dxsum, s, job);
}

// A sum over no rows is zero: the vectors an empty input leaves behind.
static hipError_t zero_vec(int dtype, void *p, int n, hipStream_t s) {
  if (p == nullptr || n <= 0) return hipSuccess;
  return launch_fill_u32(p, (size_t)n * dtype_size(dtype) / 4, 0u, s);
}

hipError_t launch_ln_bwd(int dtype, int rows, int cols, const void *dy, const void *x, const float *stats,
                         const void *gamma, const void *dres, void *dx, void *dgamma, void *dbeta, void *dxsum,
                         void *ws, hipStream_t s, ReduceJob *job, bool rms) {
  const int r = rms ? 1 : 0;
  if (job != nullptr) job->nb = 0;
  if (rows <= 0) {
    hipError_t e = zero_vec(dtype, dgamma, cols, s);
    if (e == hipSuccess) e = zero_vec(dtype, dbeta, cols, s);
    if (e == hipSuccess) e = zero_vec(dtype, dxsum, cols, s);
    return e;
  }
  const size_t vec = (size_t)cols * dtype_size(dtype), mat = (size_t)rows * vec;
  const auto in_inputs = [&](const void *p, size_t n) {
    return overlap(p, n, dy, mat) || overlap(p, n, x, mat) || overlap(p, n, gamma, vec) || overlap(p, n, stats, 8 * (size_t)rows);
  };
  if (job == nullptr && dxsum == nullptr && rows <= (dtype == kBF16 ? kLnSlabRows<bf16> : kLnSlabRows<float>) && cols <= 2048 && !in_inputs(dx, mat) &&
      !in_inputs(dgamma, vec) && !in_inputs(dbeta, vec) && !overlap(dgamma, vec, dres, mat) && !overlap(dbeta, vec, dres, mat))
    return dtype == kBF16 ? ln_bwd_few_t<bf16>(rows, cols, dy, x, stats, gamma, dres, dx, dgamma, dbeta, s, r)
                          : ln_bwd_few_t<float>(rows, cols, dy, x, stats, gamma, dres, dx, dgamma, dbeta, s, r);
  if (dxsum != nullptr)
    return dtype == kBF16
               ? ln_bwd_t<bf16, true>(rows, cols, dy, x, stats, gamma, dres, dx, dgamma, dbeta, dxsum, ws, s, job, r)
               : ln_bwd_t<float, true>(rows, cols, dy, x, stats, gamma, dres, dx, dgamma, dbeta, dxsum, ws, s, job, r);
  return dtype == kBF16
             ? ln_bwd_t<bf16, false>(rows, cols, dy, x, stats, gamma, dres, dx, dgamma, dbeta, nullptr, ws, s, job, r)
             : ln_bwd_t<float, false>(rows, cols, dy, x, stats, gamma, dres, dx, dgamma, dbeta, nullptr, ws, s, job, r);
}

// The derivative is vector work: up to four blocks a CU their 16 rows go to 16 waves, one each, not to four with four rows each
// one after the other (four waves / 16, us with the second pass, bf16: 700x3072 9.6 / 7.9, 1000x1600 10.9 / 7.2, 4096x1024 10.8 /
// 9.2; the rest is memory: 4096x4096 20.3 / 20.9).
// Blocks of more than 16 rows (8193 rows and more) keep four waves: sixteen would add the rows in another order.
static bool wave_a_row(const dim3 &grid, int rpb) { return (int)(grid.x * grid.y) <= 1024 && rpb <= 16; }
template <typename T>
static hipError_t gelu_bwd_colsum_t(int kind, int rows, int cols, const void *dy, const void *x, void *dx,
                                    void *dbias, void *ws, hipStream_t s, ReduceJob *job) {
  const size_t mat = (size_t)rows * cols * sizeof(T), vec = (size_t)cols * sizeof(T);
  if (job == nullptr && rows <= kGeluSlabRows<T> && mat <= kSlabBytes && !overlap(dbias, vec, dy, mat) && !overlap(dbias, vec, x, mat)) {
    if (cols <= 1024)
      hipLaunchKernelGGL((gelu_bwd_slab_kernel<T, 16>), dim3((cols + 15) / 16), dim3(1024), 0, s, (const T *)dy, (const T *)x,
                         (T *)dx, (T *)dbias, rows, cols, kind);
    else
      hipLaunchKernelGGL((gelu_bwd_slab_kernel<T, 32>), dim3((cols + 31) / 32), dim3(1024), 0, s, (const T *)dy, (const T *)x,
                         (T *)dx, (T *)dbias, rows, cols, kind);
    return hipGetLastError();
  }
  int rpb;
  const int nb = row_blocks(rows, 16, &rpb);
  float *part = (float *)ws;
  const dim3 grid((cols + 511) / 512, nb);
  if (wave_a_row(grid, rpb))
    hipLaunchKernelGGL((gelu_bwd_colsum_kernel<T, 16>), grid, dim3(1024), 0, s, (const T *)dy, (const T *)x, (T *)dx, part, rows,
                       cols, rpb, kind);
  else
    hipLaunchKernelGGL((gelu_bwd_colsum_kernel<T, 4>), grid, dim3(256), 0, s, (const T *)dy, (const T *)x, (T *)dx, part, rows,
                       cols, rpb, kind);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return reduce_or_defer<T>(part, nb, cols, cols, dbias, dbias, dbias, s, job);
}

hipError_t launch_gelu_bwd_colsum(int dtype, int kind, int rows, int cols, const void *dy, const void *x, void *dx,
                                  void *dbias, void *ws, hipStream_t s, ReduceJob *job) {
  if (job != nullptr) job->nb = 0;
  if (rows <= 0) return zero_vec(dtype, dbias, cols, s);
  return dtype == kBF16 ? gelu_bwd_colsum_t<bf16>(kind, rows, cols, dy, x, dx, dbias, ws, s, job)
                        : gelu_bwd_colsum_t<float>(kind, rows, cols, dy, x, dx, dbias, ws, s, job);
}

static int ew_grid(size_t n8) {
  size_t g = (n8 + 255) / 256;
  if (g > 256 * 16) g = 256 * 16;
  return g < 1 ? 1 : (int)g;
}

hipError_t launch_gelu_fwd(int dtype, int kind, size_t n, const void *x, void *y, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const size_t n8 = n / 8;
  if (dtype == kBF16)
    hipLaunchKernelGGL((gelu_fwd_kernel<bf16>), dim3(ew_grid(n8)), dim3(256), 0, s, (const bf16 *)x, (bf16 *)y, n8,
                       kind);
  else
    hipLaunchKernelGGL((gelu_fwd_kernel<float>), dim3(ew_grid(n8)), dim3(256), 0, s, (const float *)x, (float *)y,
                       n8, kind);
  return hipGetLastError();
}

hipError_t launch_dropout(int dtype, size_t n, const void *x, const void *res, void *y, const DropArgs &a,
                          hipStream_t s) {
  if (n == 0) return hipSuccess;
  const size_t n8 = n / 8;
  if (dtype == kBF16)
    hipLaunchKernelGGL((dropout_kernel<bf16>), dim3(ew_grid(n8)), dim3(256), 0, s, (const bf16 *)x, (const bf16 *)res,
                       (bf16 *)y, n8, a);
  else
    hipLaunchKernelGGL((dropout_kernel<float>), dim3(ew_grid(n8)), dim3(256), 0, s, (const float *)x,
                       (const float *)res, (float *)y, n8, a);
  return hipGetLastError();
}

template <typename T>
static hipError_t dropout_colsum_t(int rows, int cols, const void *x, void *y, void *sums, void *ws, const DropArgs &a,
                                   hipStream_t s, ReduceJob *job) {
  int rpb;
  const int nb = row_blocks(rows, 16, &rpb);
  float *part = (float *)ws;
  const dim3 grid((cols + 511) / 512, nb);
  if (wave_a_row(grid, rpb))
    hipLaunchKernelGGL((dropout_colsum_kernel<T, 16>), grid, dim3(1024), 0, s, (const T *)x, (T *)y, part, rows, cols, rpb, a);
  else
    hipLaunchKernelGGL((dropout_colsum_kernel<T, 4>), grid, dim3(256), 0, s, (const T *)x, (T *)y, part, rows, cols, rpb, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return reduce_or_defer<T>(part, nb, cols, cols, sums, sums, sums, s, job);
}

hipError_t launch_dropout_colsum(int dtype, int rows, int cols, const void *x, void *y, void *sums, void *ws, const DropArgs &a,
                                 hipStream_t s, ReduceJob *job) {
  job->nb = 0;
  if (rows <= 0) return zero_vec(dtype, sums, cols, s);
  return dtype == kBF16 ? dropout_colsum_t<bf16>(rows, cols, x, y, sums, ws, a, s, job)
                        : dropout_colsum_t<float>(rows, cols, x, y, sums, ws, a, s, job);
}

template <typename T>
static hipError_t colsum_t(int rows, int cols, const void *x, void *out, void *ws, hipStream_t s, ReduceJob *job) {
  const size_t mat = (size_t)rows * cols * sizeof(T);
  if (job == nullptr && rows <= kColsumSlabRows && mat <= kSlabBytes && !overlap(out, (size_t)cols * sizeof(T), x, mat)) {
    hipLaunchKernelGGL((colsum_slab_kernel<T, 32>), dim3((cols + 31) / 32), dim3(1024), 0, s, (const T *)x, (T *)out, rows, cols);
    return hipGetLastError();
  }
  int rpb;
  const int nb = row_blocks(rows, 16, &rpb);
  float *part = (float *)ws;
  hipLaunchKernelGGL((colsum_kernel<T>), dim3((cols + 511) / 512, nb), dim3(256), 0, s, (const T *)x, part, rows,
                     cols, rpb);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return reduce_or_defer<T>(part, nb, cols, cols, out, out, out, s, job);
}

hipError_t launch_colsum(int dtype, int rows, int cols, const void *x, void *out, void *ws, hipStream_t s,
                         ReduceJob *job) {
  if (job != nullptr) job->nb = 0;
  if (rows <= 0) return zero_vec(dtype, out, cols, s);
  return dtype == kBF16 ? colsum_t<bf16>(rows, cols, x, out, ws, s, job) : colsum_t<float>(rows, cols, x, out, ws, s, job);
}

// ---- column sums without a workspace argument and without any allocation -----------------
// The partial sums of the two-pass reduction go to a file-scope device array instead of a
// caller's workspace.  Every GPU the library runs on holds its own copy of the array at its
// own address until the process ends; the host looks that address up once per device.  All
// calls on a GPU share the array: calls that overlap on one GPU race.
constexpr size_t kStaticScratchBytes = 8u << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

size_t colsum_static_max_bytes() { return kStaticScratchBytes; }

size_t colsum_static_needed_bytes(int rows, int cols) {
  if (rows <= 0) return 0;   // (no rows: no partial sums)
  int rpb;
  return (size_t)row_blocks(rows, 16, &rpb) * (size_t)cols * sizeof(float);
}

// The array's device address on the current device (host code must never use the array's name
// where its memory is meant: the name is a host-side stand-in, not a device address).
static hipError_t scratch_address(void **out) {
  constexpr int kMaxDevices = 64;
  static void *ptr[kMaxDevices] = {};
  static std::mutex lock;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> guard(lock);
  if (ptr[dev] == nullptr) {
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    ptr[dev] = p;
  }
  *out = ptr[dev];
  return hipSuccess;
}

// launch_colsum with the partial sums in the library's own array.  The caller has checked that
// colsum_static_needed_bytes(rows, cols) fits.  Nothing has to start at zero: the first pass
// writes every partial the second pass reads.
hipError_t launch_colsum_static(int dtype, int rows, int cols, const void *x, void *out, hipStream_t s) {
  if (rows <= 0) return zero_vec(dtype, out, cols, s);
  void *ws = nullptr;
  const hipError_t e = scratch_address(&ws);
  if (e != hipSuccess) return e;
  return dtype == kBF16 ? colsum_t<bf16>(rows, cols, x, out, ws, s, nullptr) : colsum_t<float>(rows, cols, x, out, ws, s, nullptr);
}

hipError_t launch_reduce_jobs(int dtype, const ReduceJob *jobs, int n, hipStream_t s) {
  ReduceJobTable t;
  t.n = 0;
  int blocks = 0;
  for (int i = 0; i < n && t.n < kMaxReduceJobs; ++i) {
    if (jobs[i].nb <= 0 || jobs[i].width <= 0) continue;
    t.job[t.n] = jobs[i];
    t.first_block[t.n] = blocks;
    blocks += (jobs[i].width + 63) / 64;
    ++t.n;
  }
  t.first_block[t.n] = blocks;
  if (t.n == 0) return hipSuccess;
  if (dtype == kBF16) hipLaunchKernelGGL((reduce_jobs_kernel<bf16>), dim3(blocks), dim3(1024), 0, s, t);
  else hipLaunchKernelGGL((reduce_jobs_kernel<float>), dim3(blocks), dim3(1024), 0, s, t);
  return hipGetLastError();
}

hipError_t launch_transpose(int dtype, int rows, int cols, const void *src, void *dst, hipStream_t s) {
  const dim3 grid((cols + 31) / 32, (rows + 31) / 32), block(256);
  if (dtype == kBF16)
    hipLaunchKernelGGL((transpose_kernel<bf16>), grid, block, 0, s, (const bf16 *)src, (bf16 *)dst, rows, cols);
  else
    hipLaunchKernelGGL((transpose_kernel<float>), grid, block, 0, s, (const float *)src, (float *)dst, rows, cols);
  return hipGetLastError();
}

hipError_t launch_fill_u32(void *p, size_t n_words, uint32_t pattern, hipStream_t s) {
  if (n_words == 0) return hipSuccess;
  size_t g = (n_words + 255) / 256;
  if (g > 4096) g = 4096;
  hipLaunchKernelGGL(fill_u32_kernel, dim3((int)g), dim3(256), 0, s, (uint32_t *)p, n_words, pattern);
  return hipGetLastError();
}

}  // namespace dp
