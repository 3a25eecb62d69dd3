// fp32 GEMM on the matrix cores (v_mfma_f32_16x16x4_f32: fp32 operands, products and sums).
//
//   NT: C[M,N] = A[M,K] * B[N,K]^T (+ bias, + residual)      TN: C[M,N] = A[K,M]^T * B[K,N] (...)
//
// What bounds it: the fp32 stages are small (a program checks itself with them), so a launch is a chain of
// memory latencies.  The operands therefore go from memory straight into the matrix instructions' registers,
// several 16-deep chunks ahead, without LDS and without a barrier in the loop, and where the output has few
// tiles the four waves of a workgroup share a tile and divide the contraction (their partial sums meet in LDS
// in a fixed order).  A post-LN stage of one 128-wide layer over 128 tokens: 586 -> 157 us a step
// (92 with the tiles of 16 below and the attention of today).
//
// A wave owns (16 F) x (16 F) of C.  Operand fragments are 16 rows x 4 contraction elements, one float a lane:
// lane l is row l%16, element l/16.  Which matrix row a fragment row stands for, and which contraction element,
// is free as long as both operands agree, so both are chosen for wide loads and stores:
//   rows: fragment f, row r is matrix row F*r + f of the wave's part (columns likewise), so a lane's F column
//         results of one row are neighbours in C;
//   NT:   a lane loads 4 consecutive contraction elements of its row (16 bytes); MFMA t of a chunk takes
//         element t of every lane, i.e. the contraction elements {t, 4 + t, 8 + t, 12 + t};
//   TN:   a lane loads the F consecutive rows F*r .. F*r + F-1 of contraction element 4 t + l/16.
// Rows past the matrix repeat its last ones (their results are not stored), chunks past the contraction count
// as zero.
#include "common.h"
#include "kernels.h"

namespace dp {

namespace {

template <int F> struct Vec { typedef float t __attribute__((ext_vector_type(F))); };

// One tile of the product, number `tile`, by the whole workgroup; `part`: LDS of the divided form, [4][16 F][16 F + 4].
template <int F, int D, bool TN, bool SPLIT>
__device__ __forceinline__ void gemm_f32_body(const float *__restrict__ A, const float *__restrict__ B,
                                              const float *__restrict__ bias, const float *res, float *C, int M, int N, int K,
                                              int tiles_n, int tile, float *lds_part) {
  typedef typename Vec<F>::t vecF;
  constexpr int WT = 16 * F, LD = WT + 4;
  auto part = reinterpret_cast<float (*)[WT][LD]>(lds_part);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 15, g = lane >> 4;
  const int tm = tile / tiles_n, tn = tile % tiles_n;
  const int m0 = SPLIT ? tm * WT : tm * 2 * WT + (wave >> 1) * WT;
  const int n0 = SPLIT ? tn * WT : tn * 2 * WT + (wave & 1) * WT;
  const int nch = (K + 15) / 16;                           // chunks of the contraction
  const int first = SPLIT ? wave : 0, stride = SPLIT ? 4 : 1;   // this wave's: first, first + stride, ...

  // NT: where the lane's rows start; TN: the lane's first row within a contraction row
  const float *pa[TN ? 1 : F], *pb[TN ? 1 : F];
  if (TN) {
    pa[0] = A + min(m0 + F * r, M - F);
    pb[0] = B + min(n0 + F * r, N - F);
  } else {
#pragma unroll
    for (int f = 0; f < F; ++f) {
      pa[f] = A + (size_t)min(m0 + F * r + f, M - 1) * K;
      pb[f] = B + (size_t)min(n0 + F * r + f, N - 1) * K;
    }
  }
  // D chunks in flight.  NT: [f] holds 4 contraction elements of row f; TN: [t] holds the F rows of contraction element 4t + g
  constexpr int NV = TN ? 4 : F, VW = TN ? F : 4;
  typedef typename Vec<VW>::t vec;
  vec a[D][NV], b[D][NV];
  // (NT, small tiles: of a chunk past the last, all lanes read one place.  With every lane at its own row those loads touch 16 lines
  //  each and took the memory pipe as long as useful ones: [128 x 128] x 128 in 32x32 tiles 5.3 us, now 4.1; no gain in the other forms)
  auto load = [&](int c, vec (&va)[NV], vec (&vb)[NV]) {
    const bool in = TN || F == 4 || c < nch;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      if (TN) {
        const size_t k = (size_t)min(16 * c + 4 * i + g, K - 1);
        va[i] = *reinterpret_cast<const vec *>(in ? pa[0] + k * M : A);
        vb[i] = *reinterpret_cast<const vec *>(in ? pb[0] + k * N : B);
      } else {
        const int k = min(16 * c + 4 * g, K - 4);
        va[i] = *reinterpret_cast<const vec *>(in ? pa[i] + k : A);
        vb[i] = *reinterpret_cast<const vec *>(in ? pb[i] + k : B);
      }
    }
  };
  // NT without the division (at most four chunks): a sum for each chunk, added in their order, which is what the divided
  // form's waves do with a chunk each: the same bits, and half the error of one chain over all of K.
  constexpr bool BY_CHUNK = !TN && !SPLIT;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  f32x4 acc[F][F], sum[BY_CHUNK ? F : 1][F];
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j) { acc[i][j] = zero; sum[BY_CHUNK ? i : 0][j] = zero; }
#pragma unroll
  for (int s = 0; s < D; ++s) load(first + s * stride, a[s], b[s]);
  for (int c0 = first; c0 < nch; c0 += D * stride) {
#pragma unroll
    for (int s = 0; s < D; ++s) {
      const int c = c0 + s * stride;
      if (16 * c + 16 > K) {   // the last chunk's elements past the contraction, and whole chunks past it
#pragma unroll
        for (int i = 0; i < NV; ++i) {
          const bool out = 16 * c + (TN ? 4 * i + g : 4 * g) >= K;
#pragma unroll
          for (int q = 0; q < VW; ++q) { a[s][i][q] = out ? 0.f : a[s][i][q]; b[s][i][q] = out ? 0.f : b[s][i][q]; }
        }
      }
      if (c < nch) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
          for (int i = 0; i < F; ++i)
#pragma unroll
            for (int j = 0; j < F; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(TN ? a[s][t][i] : a[s][i][t], TN ? b[s][t][j] : b[s][j][t],
                                                               BY_CHUNK && t == 0 ? zero : acc[i][j], 0, 0, 0);
        if (BY_CHUNK) {
#pragma unroll
          for (int i = 0; i < F; ++i)
#pragma unroll
            for (int j = 0; j < F; ++j) sum[BY_CHUNK ? i : 0][j] += acc[i][j];
        }
      }
      load(c + D * stride, a[s], b[s]);
    }
  }
  // element e of acc[i][j] is row F*(4g + e) + i, column F*r + j of the wave's part
  auto put = [&](int row, int col, vecF v) {
    if (row >= M || col >= N) return;
    if (bias != nullptr) v += *reinterpret_cast<const vecF *>(bias + col);
    const size_t at = (size_t)row * N + col;
    if (res != nullptr) v += *reinterpret_cast<const vecF *>(res + at);
    *reinterpret_cast<vecF *>(C + at) = v;
  };
  if (!SPLIT) {
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        vecF v;
#pragma unroll
        for (int j = 0; j < F; ++j) v[j] = BY_CHUNK ? sum[BY_CHUNK ? i : 0][j][e] : acc[i][j][e];
        put(m0 + F * (4 * g + e) + i, n0 + F * r, v);
      }
  } else {
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        vecF v;
#pragma unroll
        for (int j = 0; j < F; ++j) v[j] = acc[i][j][e];
        *reinterpret_cast<vecF *>(&part[wave][F * (4 * g + e) + i][F * r]) = v;
      }
    __syncthreads();
    for (int q = threadIdx.x; q < WT * 16; q += 256) {
      const int row = q / 16, col = F * (q % 16);
      vecF v = *reinterpret_cast<const vecF *>(&part[0][row][col]);
#pragma unroll
      for (int w = 1; w < 4; ++w) v += *reinterpret_cast<const vecF *>(&part[w][row][col]);
      put(m0 + row, n0 + col, v);
    }
  }
}

constexpr int part_floats(int F, bool split) { return split ? 4 * 16 * F * (16 * F + 4) : 4; }

template <int F, int D, bool TN, bool SPLIT>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float *__restrict__ A, const float *__restrict__ B,
                                                       const float *__restrict__ bias, const float *res, float *C, int M,
                                                       int N, int K, int tiles_n) {
  __shared__ __attribute__((aligned(16))) float part[part_floats(F, SPLIT)];
  gemm_f32_body<F, D, TN, SPLIT>(A, B, bias, res, C, M, N, K, tiles_n, blockIdx.x, part);
}

template <int F, int D, bool TN, bool SPLIT>
hipError_t launch_f32(const GemmArgs &a, hipStream_t s) {
  constexpr int T = SPLIT ? 16 * F : 32 * F;
  const int tiles_m = (a.M + T - 1) / T, tiles_n = (a.N + T - 1) / T;
  hipLaunchKernelGGL((gemm_f32_kernel<F, D, TN, SPLIT>), dim3((unsigned)(tiles_m * tiles_n)), dim3(256), 0, s,
                     (const float *)a.A, (const float *)a.B, (const float *)a.bias, (const float *)a.res, (float *)a.C, a.M,
                     a.N, a.K, tiles_n);
  return hipGetLastError();
}

// The two products of a linear layer's backward (NT: dX = dY W^T, TN: dW = X^T dY) in one launch, in the tiles each has alone:
// the first n_nt workgroups are dX's.
struct F32Side {
  const float *A, *B, *res;
  float *C;
  int M, N, K, tiles_n;
};
template <int FN, int FT>
__global__ __launch_bounds__(256) void gemm_f32_pair_kernel(F32Side nt, F32Side tn, int n_nt) {
  __shared__ __attribute__((aligned(16))) float part[part_floats(FN > FT ? FN : FT, true)];
  const int b = blockIdx.x;
  if (b < n_nt) gemm_f32_body<FN, 4, false, true>(nt.A, nt.B, nullptr, nt.res, nt.C, nt.M, nt.N, nt.K, nt.tiles_n, b, part);
  else gemm_f32_body<FT, 4, true, true>(tn.A, tn.B, nullptr, tn.res, tn.C, tn.M, tn.N, tn.K, tn.tiles_n, b - n_nt, part);
}

template <int FN, int FT> hipError_t launch_f32_pair(const GemmArgs &nt, const GemmArgs &tn, hipStream_t s) {
  auto side = [](const GemmArgs &a, int t) {
    return F32Side{(const float *)a.A, (const float *)a.B, (const float *)a.res, (float *)a.C, a.M, a.N, a.K, (a.N + t - 1) / t};
  };
  const F32Side sn = side(nt, 16 * FN), st = side(tn, 16 * FT);
  const int n_nt = (nt.M + 16 * FN - 1) / (16 * FN) * sn.tiles_n, n_tn = (tn.M + 16 * FT - 1) / (16 * FT) * st.tiles_n;
  hipLaunchKernelGGL((gemm_f32_pair_kernel<FN, FT>), dim3((unsigned)(n_nt + n_tn)), dim3(256), 0, s, sn, st, n_nt);
  return hipGetLastError();
}

}  // namespace

// 16-byte loads and stores: four elements of every row, and rows that start on 16 bytes.
bool gemm_f32_supported(const GemmArgs &a) {
  if (a.M < 4 || a.N < 4 || a.K < 4 || a.N % 4 != 0 || a.C2 != nullptr) return false;
  if ((((uintptr_t)a.A | (uintptr_t)a.B | (uintptr_t)a.C | (uintptr_t)a.bias | (uintptr_t)a.res) & 15) != 0) return false;
  return a.mode == kGemmNT ? a.K % 4 == 0 : a.M % 4 == 0;
}

// 64x64 tiles whose waves divide the contraction from half a chip of them on (128), below that 32x32 tiles:
//   [256 x 1024] x 333 TN: 64 tiles of 64x64 10.2 us, 256 of 32x32 7.6; [333 x 256] x 1024 NT 21.2 and 10.3;
//   [1024 x 1024] x 1024 NT: 256 tiles of 64x64 23.6 us (91 TFLOP/s of the 147 the instruction reaches alone),
//   1024 of 32x32 37.0.
// 16x16 tiles while each has a CU to itself (256): a load touches 16 lines whatever the tile, and that many CUs share them.  32x32 / 16x16:
//   [128 x 128] x 128, 512 NT: 4.1 / 3.0 us, 6.7 / 4.2; [128 x 512] x 128 TN 4.1 / 3.2; [256 x 256] x 1024 NT 10.1 / 5.9; past that line
//   [256 x 768] x 256 NT 5.2 / 5.4, [512 x 512] x 300 TN 5.7 / 7.7.
// TN with enough tiles of 128x128 for half the chip: a wave each 64x64, no division ([1024 x 4096] x 4096: 257 us
// against 311).  In NT form, whose loads take 16 rows at a time, the division stays ahead ([4096 x 4096] x 1024 352
// against 505) but for contractions of at most four chunks, which leave its waves one each at most to share the turn
// of the output through LDS over: [7588 x 3192] x 8, 24, 40, 64: 39.2, 42.1, 51.2, 54.5 us without it and 60.2, 71.6,
// 78.8, 85.0 with it, [3076 x 1488] 10.6, 12.2, 15.1, 16.4 and 14.3, 17.1, 18.7, 19.6.
// The vector-ALU kernel takes 52, 139, 168, 769 and 545 us for the products named so far with K > 64, 52.4 to 87.9 and
// 13.9 to 21.9 us for the two of K <= 64, and 20 to 70 us where these kernels take under 7 ([128 x 128..512] x
// 128..512, the products of a stage 128 wide).
namespace {
enum F32Form { k16, k32, k64, kWhole };   // tiles of 16, 32 or 64 whose waves divide the contraction; a wave each 64x64
F32Form f32_form(const GemmArgs &a) {
  auto tiles = [&](int t) { return (long)((a.M + t - 1) / t) * ((a.N + t - 1) / t); };
  if (tiles(128) >= 128 && (a.mode == kGemmTN || a.K <= 64)) return kWhole;
  if (tiles(16) <= 256) return k16;
  return tiles(64) >= 128 ? k64 : k32;
}
}  // namespace

hipError_t launch_gemm_f32(const GemmArgs &a, hipStream_t s) {
  const bool tn = a.mode == kGemmTN;
  switch (f32_form(a)) {
    case kWhole: return tn ? launch_f32<4, 2, true, false>(a, s) : launch_f32<4, 2, false, false>(a, s);
    case k16: return tn ? launch_f32<1, 4, true, true>(a, s) : launch_f32<1, 4, false, true>(a, s);
    case k64: return tn ? launch_f32<4, 2, true, true>(a, s) : launch_f32<4, 2, false, true>(a, s);
    default: return tn ? launch_f32<2, 4, true, true>(a, s) : launch_f32<2, 4, false, true>(a, s);
  }
}

// Where both products run in small tiles, a launch is most of their time.
bool gemm_f32_pair_supported(const GemmArgs &nt, const GemmArgs &tn) {
  return nt.mode == kGemmNT && tn.mode == kGemmTN && nt.bias == nullptr && tn.bias == nullptr && gemm_f32_supported(nt) &&
         gemm_f32_supported(tn) && f32_form(nt) <= k32 && f32_form(tn) <= k32;
}

hipError_t launch_gemm_f32_pair(const GemmArgs &nt, const GemmArgs &tn, hipStream_t s) {
  if (f32_form(nt) == k16) return f32_form(tn) == k16 ? launch_f32_pair<1, 1>(nt, tn, s) : launch_f32_pair<1, 2>(nt, tn, s);
  return f32_form(tn) == k16 ? launch_f32_pair<2, 1>(nt, tn, s) : launch_f32_pair<2, 2>(nt, tn, s);
}

}  // namespace dp
