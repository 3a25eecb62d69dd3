// bf16 GEMMs of one product a launch: the tiles of gemm_dma_tile.h as kernels of their own, and the choice among them.
#include "gemm_dma_tile.h"

#include <cstdio>
#include <cstdlib>

namespace dp {

namespace {

template <int BM, int BN, int WGM, int WGN, int STAGES, bool ACT, bool TN, bool SPLIT>
__global__ __attribute__((amdgpu_waves_per_eu(WGM * WGN / 4, WGM * WGN / 4), amdgpu_flat_work_group_size(64 * WGM * WGN, 64 * WGM * WGN))) void gemm_dma_kernel(
    const bf16 *__restrict__ A, const bf16 *__restrict__ B, const bf16 *__restrict__ bias,
    const bf16 *__restrict__ res, bf16 *__restrict__ C, bf16 *__restrict__ C2, int gelu_kind, int M, int N, int K,
    int tiles_m, int tiles_n) {
  dma_tile_body<BM, BN, WGM, WGN, STAGES, ACT, TN, SPLIT>(A, B, bias, res, C, C2, gelu_kind, M, N, K, tiles_m, tiles_n,
                                                          blockIdx.x, kGroupM);
}

template <int BM, int BN, int WGM, int WGN, int STAGES, bool ACT, bool TN, bool SPLIT>
hipError_t launch_dma_act(const GemmArgs &a, hipStream_t s) {
  constexpr size_t smem = SPLIT ? (size_t)(3 * BM + 2 * BN) * 128 : (size_t)STAGES * (BM + BN) * 128;
  static_assert(smem <= 160 * 1024, "LDS of one CU");
  static bool attr_set = false;
  auto kern = gemm_dma_kernel<BM, BN, WGM, WGN, STAGES, ACT, TN, SPLIT>;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  const int tiles_m = (a.M + BM - 1) / BM, tiles_n = (a.N + BN - 1) / BN;
  hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n), dim3(64 * WGM * WGN), smem, s, (const bf16 *)a.A,
                     (const bf16 *)a.B, (const bf16 *)a.bias, (const bf16 *)a.res, (bf16 *)a.C, (bf16 *)a.C2,
                     a.gelu_kind, a.M, a.N, a.K, tiles_m, tiles_n);
  return hipGetLastError();
}

template <int BM, int BN, int WGM, int WGN, int STAGES, bool TN, bool SPLIT = false>
hipError_t launch_dma_cfg(const GemmArgs &a, hipStream_t s) {
  if (TN) return launch_dma_act<BM, BN, WGM, WGN, STAGES, false, TN, SPLIT>(a, s);   // no epilogue extras in this form
  return a.C2 != nullptr ? launch_dma_act<BM, BN, WGM, WGN, STAGES, true, false, SPLIT>(a, s)
                         : launch_dma_act<BM, BN, WGM, WGN, STAGES, false, false, SPLIT>(a, s);
}

// DPSTAGE_GEMM_TILE=256x192 and the like names the tile of every product that can run in it (tuning aid)
int asked_tile(const GemmArgs &a, int nk) {
  static const char *force = getenv("DPSTAGE_GEMM_TILE");
  int bm = 0, bn = 0;
  if (force == nullptr || sscanf(force, "%dx%d", &bm, &bn) != 2) return -1;
  for (int i = 0; i < kTiles; ++i)
    if (kTileTimes[i].bm == bm && kTileTimes[i].bn == bn && a.M >= bm && a.N >= bn && nk >= fewest_steps(i)) return i;
  return -1;
}

int choose_tile(const GemmArgs &a) {
  const int nk = (a.K + 63) / 64, asked = asked_tile(a, nk);
  if (asked >= 0) return asked;
  int best = -1;
  float best_us = 0.f;
  long best_tiles = 0;
  for (int i = 0; i < kTiles; ++i) {
    const TileTime &t = kTileTimes[i];
    if (a.M < t.bm || a.N < t.bn) continue;
    if (nk < t.min_steps) continue;
    const long tiles = (long)((a.M + t.bm - 1) / t.bm) * ((a.N + t.bn - 1) / t.bn);
    const long rounds = (tiles + kCus - 1) / kCus;
    if ((t.bm == 192 || t.bn == 192) && rounds > kRounds192) continue;
    const float us = (float)rounds * (t.start_us + t.step_us * (float)nk);
    if (best < 0 || us < best_us || (us == best_us && tiles < best_tiles)) { best = i; best_us = us; best_tiles = tiles; }
  }
  return best;
}

template <bool TN>
hipError_t launch_dma_mode(const GemmArgs &a, hipStream_t s) {
  switch (choose_tile(a)) {
    case k256x256: return launch_dma_cfg<256, 256, 2, 2, 2, TN, true>(a, s);
    case k256x192: return launch_dma_cfg<256, 192, 2, 2, 2, TN, true>(a, s);
    case k192x256: return launch_dma_cfg<192, 256, 2, 2, 2, TN, true>(a, s);
    case k192x192: return launch_dma_cfg<192, 192, 2, 2, 3, TN>(a, s);
    case k192x128: return launch_dma_cfg<192, 128, 2, 2, 3, TN>(a, s);
    case k128x192: return launch_dma_cfg<128, 192, 2, 2, 3, TN>(a, s);
    case k256x128: return launch_dma_cfg<256, 128, 2, 2, 3, TN>(a, s);
    case k128x256: return launch_dma_cfg<128, 256, 2, 2, 3, TN>(a, s);
    // (eight waves: with four, [4096 x 1024] x 4096 NT takes 31.2 us instead of 31.7 with operands in the caches,
    //  but 41.4 instead of 38.9 from memory)
    case k128x128: return launch_dma_cfg<128, 128, 4, 2, 4, TN>(a, s);
    case k128x64: return launch_dma_cfg<128, 64, 2, 2, 3, TN>(a, s);
    case k64x128: return launch_dma_cfg<64, 128, 2, 2, 3, TN>(a, s);
    // (four stages, which are asked for before the first MFMA; with eight [4096 x 1600] x 1600 NT takes 43.6 us, not 40.8,
    //  [1000 x 768] x 768 4.9, not 4.5)
    default: return launch_dma_cfg<64, 64, 2, 2, 4, TN>(a, s);
  }
}

}  // namespace

bool gemm_dma_supported(const GemmArgs &a) {
  if (a.M < 128 || a.N < 128 || a.K < kMinK) return false;
  if ((((uintptr_t)a.A | (uintptr_t)a.B) & 15) != 0) return false;
  // the epilogue moves runs of four columns (8 bytes)
  if (a.N % 4 != 0 || (((uintptr_t)a.C | (uintptr_t)a.C2 | (uintptr_t)a.res | (uintptr_t)a.bias) & 7) != 0) return false;
  // lane offsets are 32-bit
  if (a.mode == kGemmNT) return a.K % 8 == 0 && (uint64_t)a.K * 2 * 9 + 4096 <= 0xffffffffull;
  if (a.M % 8 != 0 || a.N % 8 != 0) return false;   // 16-byte rows and tile origins
  const uint64_t ld = (uint64_t)(a.M > a.N ? a.M : a.N) * 2;
  return ((uint64_t)a.K + 4) * ld + 4096 <= 0xffffffffull;
}

void gemm_dma_tile(const GemmArgs &a, int *bm, int *bn) {
  const TileTime &t = kTileTimes[choose_tile(a)];
  *bm = t.bm;
  *bn = t.bn;
}

hipError_t launch_gemm_dma(const GemmArgs &a, hipStream_t s) {
  return a.mode == kGemmNT ? launch_dma_mode<false>(a, s) : launch_dma_mode<true>(a, s);
}

}  // namespace dp
