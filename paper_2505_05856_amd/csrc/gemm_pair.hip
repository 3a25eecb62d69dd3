// The two products of a linear layer's backward in one launch: the input gradient dX = dY W^T (NT form) and the weight
// gradient dW = X^T dY (TN form), which read the same dY and wait for nothing of each other.  The tiles are those of
// gemm_dma_tile.h, so every output has the bits it has from a launch of its own.
//
// Why together.  Alone, either product has to be cut into enough tiles for 256 CUs, and what does not fill a round of
// them is lost: a [1024 x 1024] weight gradient over 4096 tokens ran in 64x64 tiles at 0.5 PFLOP/s, for larger ones
// would have left most CUs idle.  Together they are twice the tiles, so each may be cut into larger ones, which fetch
// fewer bytes a flop, and the tiles of the shorter product fill the round the longer one leaves open.  Two launches /
// one, operands from memory (T tokens, a layer of I inputs and O outputs):
//   T 4096, 4096 -> 1024: 82.9 / 60.9 us    1024 -> 4096: 84.0 / 59.4    1024 -> 3072: 73.1 / 53.9    1024 -> 1024: 32.2 / 31.7
//   T 4096, 6400 -> 1600:  176 /  158 us    1600 -> 6400:  179 /  147    1600 -> 4800:  137 /  110    1600 -> 1600: 67.0 / 54.6
//   T 1000, 3072 ->  768: 22.0 / 16.9 us     768 -> 3072: 22.8 / 17.9     768 ->  768: 11.2 /  7.2
//   T 16384, 11008 -> 4096: 2128 / 2072 us  4096 -> 4096:  844 /  818
// What bounds it: as one product a launch, the clock of the matrix cores at the power they draw where tiles are large,
// and what an XCD can fetch where they are small.
#include "gemm_dma_tile.h"

#include <cmath>
#include <cstdlib>

namespace dp {

namespace {

struct PairSide {
  const bf16 *A, *B, *res;
  bf16 *C;
  int M, N, K, tiles_m, tiles_n, tile;
};

// Groups of four tile rows (eight for one product alone): an XCD has half as many tiles of each product, and four keep the
// panels they share as few.  In eight, T 4096, 1024 -> 4096: 68.5 us for 59.4, T 16384, 4096 -> 12288: 2244 for 2187.
constexpr int kPairGroupM = 4;

template <int BM, int BN, int STAGES, bool TN, bool SPLIT = false>
__device__ __forceinline__ void side_tile(const PairSide &p, int pid) {
  dma_tile_body<BM, BN, 2, 2, STAGES, false, TN, SPLIT>(p.A, p.B, nullptr, p.res, p.C, nullptr, 0, p.M, p.N, p.K, p.tiles_m,
                                                        p.tiles_n, pid, kPairGroupM);
}
// (four waves for every tile, also 128x128, since one launch has one size of workgroup)
template <bool TN> __device__ __forceinline__ void side(const PairSide &p, int pid) {
  switch (p.tile) {
    case k256x256: side_tile<256, 256, 2, TN, true>(p, pid); break;
    case k256x192: side_tile<256, 192, 2, TN, true>(p, pid); break;
    case k192x256: side_tile<192, 256, 2, TN, true>(p, pid); break;
    case k256x128: side_tile<256, 128, 3, TN>(p, pid); break;
    case k128x256: side_tile<128, 256, 3, TN>(p, pid); break;
    case k128x128: side_tile<128, 128, 4, TN>(p, pid); break;
    case k128x64: side_tile<128, 64, 3, TN>(p, pid); break;
    case k64x128: side_tile<64, 128, 3, TN>(p, pid); break;
    default: side_tile<64, 64, 4, TN>(p, pid); break;
  }
}

// The first `n_first` workgroups are the product whose tiles take longer, the rest the other's.
__global__ __attribute__((amdgpu_waves_per_eu(1, 1), amdgpu_flat_work_group_size(256, 256))) void gemm_pair_kernel(
    PairSide nt, PairSide tn, int n_first, int tn_first) {
  const int b = blockIdx.x;
  const bool first = b < n_first;
  const int pid = first ? b : b - n_first;
  if (first == (tn_first != 0)) side<true>(tn, pid);
  else side<false>(nt, pid);
}

// Tile choice: of the 81 pairs of tiles the one with the smallest estimated time.  A tile takes a start plus a time per 64-deep
// k-step; 256 CUs take the tiles in order, the longer ones first; the estimate is 5/8 of when the last CU ends and 3/8 of the
// mean over the CUs (tiles of one size do not take one time).  Starts and steps are fitted to 3800 launches: 32 layers of
// 700 to 16384 tokens, every pair of tiles in both orders, operands from memory; over the 32 the choice takes 2.5 % longer than
// the best pair, 11 % at most.  (256x128 and the like by the kernel of one product: 4.5 + 0.83 a step; what is shared here
// is what an XCD can fetch.)
struct PairTime { int tile; float nt_start, nt_step, tn_start, tn_step; };
constexpr PairTime kPairTimes[] = {
    {k256x256, 11.4f, 1.352f, 16.0f, 1.308f}, {k256x192, 6.8f, 1.095f, 11.0f, 1.025f}, {k192x256, 7.7f, 1.086f, 10.0f, 1.051f},
    {k256x128, 5.3f, 0.823f, 7.9f, 0.787f},   {k128x256, 5.5f, 0.833f, 7.7f, 0.769f},  {k128x128, 2.9f, 0.508f, 4.8f, 0.500f},
    {k128x64, 1.4f, 0.361f, 2.3f, 0.369f},    {k64x128, 1.2f, 0.362f, 2.2f, 0.369f},   {k64x64, 0.9f, 0.219f, 1.6f, 0.211f}};
constexpr int kPairTiles = sizeof(kPairTimes) / sizeof(kPairTimes[0]);

struct Share { int tile, n; float us; };   // a product cut into n tiles of `us` each

// When the last CU ends: the tiles of `a` go first, those of `b` to whichever CU is free first.
float makespan(const Share &a, const Share &b) {
  const int full = a.n / kCus, busy = a.n % kCus, free = kCus - busy;   // `busy` CUs have one tile more of a
  const float t0 = (float)full * a.us, t1 = busy ? t0 + a.us : t0;
  // the smallest T by which all of b fits: T = t0 + k b.us or t1 + k b.us
  auto fits = [&](float T) {
    const long k0 = (long)((T - t0) / b.us + 1e-3f), k1 = T > t1 ? (long)((T - t1) / b.us + 1e-3f) : 0;
    return free * k0 + busy * k1 >= b.n;
  };
  // (all CUs together have taken b no sooner than the mean says)
  const float mean = ((float)a.n * a.us + (float)b.n * b.us) / (float)kCus;
  int k = (int)((mean - t0) / b.us);
  if (k < 1) k = 1;
  while (!fits(t0 + (float)k * b.us)) ++k;
  float end = t0 + (float)k * b.us;
  if (busy) {
    int j = (int)((mean - t1) / b.us);
    if (j < 0) j = 0;
    for (; t1 + (float)j * b.us < end; ++j)
      if (fits(t1 + (float)j * b.us)) { end = t1 + (float)j * b.us; break; }
  }
  return end > t1 ? end : t1;
}

int shares(const GemmArgs &a, bool tn, Share (&out)[kPairTiles]) {
  const int nk = (a.K + 63) / 64;
  int n = 0;
  for (const PairTime &t : kPairTimes) {
    const TileTime &d = kTileTimes[t.tile];
    if (a.M < d.bm || a.N < d.bn || nk < fewest_steps(t.tile)) continue;
    const int tiles = ((a.M + d.bm - 1) / d.bm) * ((a.N + d.bn - 1) / d.bn);
    out[n++] = Share{t.tile, tiles, (tn ? t.tn_start : t.nt_start) + (tn ? t.tn_step : t.nt_step) * (float)nk};
  }
  return n;
}

PairSide pair_side(const GemmArgs &a, const Share &s) {
  const TileTime &d = kTileTimes[s.tile];
  return PairSide{(const bf16 *)a.A, (const bf16 *)a.B, (const bf16 *)a.res, (bf16 *)a.C, a.M, a.N, a.K,
                  (a.M + d.bm - 1) / d.bm, (a.N + d.bn - 1) / d.bn, s.tile};
}

void choose_pair(const GemmArgs &nt, const GemmArgs &tn, Share *best_nt, Share *best_tn) {
  Share sn[kPairTiles], st[kPairTiles];
  const int nn = shares(nt, false, sn), ntn = shares(tn, true, st);
  float best = INFINITY;
  for (int i = 0; i < nn; ++i)
    for (int j = 0; j < ntn; ++j) {
      const float mean = ((float)sn[i].n * sn[i].us + (float)st[j].n * st[j].us) / (float)kCus;
      if (mean >= best) continue;   // (the last CU ends no sooner than the mean)
      const float end = st[j].us > sn[i].us ? makespan(st[j], sn[i]) : makespan(sn[i], st[j]);
      const float us = 0.625f * end + 0.375f * mean;
      if (us < best) { best = us; *best_nt = sn[i]; *best_tn = st[j]; }
    }
}

}  // namespace

// (the tuning aids that name the tile or the kernel of a product are about products one by one)
bool gemm_pair_supported(const GemmArgs &nt, const GemmArgs &tn) {
  static const bool tuned =
      getenv("DPSTAGE_GEMM_TILE") != nullptr || getenv("DPSTAGE_GEMM_NT") != nullptr || getenv("DPSTAGE_GEMM_TN") != nullptr;
  return !tuned && nt.mode == kGemmNT && tn.mode == kGemmTN && nt.bias == nullptr && tn.bias == nullptr && nt.C2 == nullptr &&
         tn.C2 == nullptr && gemm_mfma_supported(nt) && gemm_mfma_supported(tn) && gemm_dma_supported(nt) && gemm_dma_supported(tn);
}

void gemm_pair_tiles(const GemmArgs &nt, const GemmArgs &tn, int tiles[4]) {
  Share a{}, b{};
  choose_pair(nt, tn, &a, &b);
  tiles[0] = kTileTimes[a.tile].bm; tiles[1] = kTileTimes[a.tile].bn;
  tiles[2] = kTileTimes[b.tile].bm; tiles[3] = kTileTimes[b.tile].bn;
}

hipError_t launch_gemm_pair(const GemmArgs &nt, const GemmArgs &tn, hipStream_t s) {
  constexpr size_t smem = 160 * 1024;   // the largest tile's
  static bool attr_set = false;
  if (!attr_set) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(gemm_pair_kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  Share a{}, b{};
  choose_pair(nt, tn, &a, &b);
  const bool tn_first = b.us > a.us;
  hipLaunchKernelGGL(gemm_pair_kernel, dim3((unsigned)(a.n + b.n)), dim3(256), smem, s, pair_side(nt, a), pair_side(tn, b),
                     tn_first ? b.n : a.n, tn_first ? 1 : 0);
  return hipGetLastError();
}

}  // namespace dp
