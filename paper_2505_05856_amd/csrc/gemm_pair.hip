// The two products of a linear layer's backward in one launch: the input gradient dX = dY W^T (NT form) and the weight
// gradient dW = X^T dY (TN form), which read the same dY and wait for nothing of each other.  The tiles are those of
// gemm_dma_tile.h, so every output has the bits it has from a launch of its own.
//
// Why together.  Alone, either product has to be cut into enough tiles for 256 CUs, and what does not fill a round of
// them is lost: a [1024 x 1024] weight gradient over 4096 tokens ran in 64x64 tiles at 0.5 PFLOP/s, for larger ones
// would have left most CUs idle.  Together they are twice the tiles, so each may be cut into larger ones, which fetch
// fewer bytes a flop, and the tiles of the shorter product fill the round the longer one leaves open.  Two launches /
// one, operands from memory (T tokens, a layer of I inputs and O outputs):
//   T 4096, 4096 -> 1024: 78.0 / 64.0 us    1024 -> 4096: 79.8 / 60.6    1024 -> 3072: 70.8 / 54.7    1024 -> 1024: 37.2 / 34.2
//   T 4096, 6400 -> 1600:  162 /  143 us    1600 -> 6400:  165 /  148    1600 -> 4800:  130 /  109    1600 -> 1600: 66.5 / 55.6
//   T 8192, 6400 -> 1600:  312 /  282 us    1600 -> 6400:  283 /  282    1600 -> 4800:  218 /  220    1600 -> 1600:  113 /  101
//   T 1000, 3072 ->  768: 25.2 / 17.7 us     768 -> 3072: 29.2 / 23.8     768 ->  768: 11.1 /  7.3
//   T 16384, 11008 -> 4096: 2116 / 2071 us  4096 -> 11008: 2093 / 2091   4096 -> 4096:  781 /  773
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
// panels they share as few.  In eight, T 4096, 1024 -> 4096: 68.5 us for 59.4, T 16384, 4096 -> 12288: 2244 for 2187.  In two,
// tiles within 8 % of a layer's best take 1.0 % longer over 32 layers, 9 % less to 12 % more.
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

// Tile choice: of the 81 pairs of tiles the one whose last CU ends first by estimate.  A tile takes a start plus a time per
// 64-deep k-step, the longer tiles go first, and workgroups are dealt in turn to 32 groups of 8 CUs (four shader engines of each
// XCD), inside which the CU that is free first takes the next.  That the groups do not share out their tiles decides many
// launches: 132 tiles of 256x256 and then 231 of half the time ([2874 x 2688] x 5376) would end with the long ones if any CU took
// any tile, but a group that has five of the former and seven of the latter starts one of these last (135 us for two launches, 158).
// Starts and steps are fitted to 1082 launches: 591 layers of 128 to 16384 tokens and widths of 128 to 16384 with operands from
// memory (buffers rotated through 700 MB), the 491 smallest of them also from the Infinity Cache, which is where a stage of one
// small layer has them; fitted to one half they do nearly as well on the other.  The choice takes 1.5 % longer than the best pair
// there; 256 CUs as one group took 3.4 % longer.
// Two launches are taken where the same table says that they end sooner (each product's tiles by groups, one product after
// the other, and a launch): 10 of the 1082, mostly products of 170 us and more whose best pair mixes tile sizes.  With that 9 of
// them are longer than two launches by more than 1 %, 5 % at most; with one group and no such rule 67 were, up to 33 %.  Over 200
// layers not in the fit, from memory: 0.807 of two launches' time and four longer by more than 2 % (261 tokens, 2816 -> 11264: 100 us
// for 92), 0.826 and eleven before; 44 drawn stages take 0.926 of their time with two launches, none of them longer.
struct PairTime { int tile; float nt_start, nt_step, tn_start, tn_step; };
constexpr PairTime kPairTimes[] = {
    {k256x256, 10.0f, 1.110f, 14.5f, 1.088f}, {k256x192, 6.8f, 0.925f, 12.9f, 0.918f}, {k192x256, 7.0f, 0.991f, 6.4f, 0.960f},
    {k256x128, 5.3f, 0.681f, 5.3f, 0.978f}, {k128x256, 5.2f, 0.826f, 7.0f, 0.683f}, {k128x128, 3.1f, 0.481f, 3.8f, 0.446f},
    {k128x64, 2.1f, 0.346f, 2.8f, 0.483f}, {k64x128, 1.3f, 0.381f, 2.5f, 0.353f}, {k64x64, 1.1f, 0.222f, 1.8f, 0.211f}};
constexpr int kPairTiles = sizeof(kPairTimes) / sizeof(kPairTimes[0]);
// tiles that only a launch of one product has
constexpr PairTime kSingleTimes[] = {
    {k192x192, 4.0f, 0.783f, 6.0f, 0.712f}, {k192x128, 3.5f, 0.641f, 5.0f, 0.605f}, {k128x192, 3.5f, 0.641f, 5.0f, 0.587f}};
constexpr float kLaunchUs = 6.4f;

struct Share { int tile, n; float us; };   // a product cut into n tiles of `us` each

constexpr int kGroups = 32, kGroupCus = kCus / kGroups;

// When the last CU of a group ends: `na` tiles of `ta` us go first, then `nb` of `tb` to whichever CU is free first.
float group_end(int na, float ta, int nb, float tb) {
  const int full = na / kGroupCus, busy = na % kGroupCus, free = kGroupCus - busy;   // `busy` CUs have one tile more of a
  const float t0 = (float)full * ta, t1 = busy ? t0 + ta : t0;
  if (nb == 0) return t1;
  // the smallest T by which all of b fits: T = t0 + k tb or t1 + k tb
  auto fits = [&](float T) {
    const long k0 = (long)((T - t0) / tb + 1e-3f), k1 = T > t1 ? (long)((T - t1) / tb + 1e-3f) : 0;
    return free * k0 + busy * k1 >= nb;
  };
  // (all CUs together have taken b no sooner than the mean says)
  const float mean = ((float)na * ta + (float)nb * tb) / (float)kGroupCus;
  int k = (int)((mean - t0) / tb);
  if (k < 1) k = 1;
  while (!fits(t0 + (float)k * tb)) ++k;
  float end = t0 + (float)k * tb;
  if (busy) {
    int j = (int)((mean - t1) / tb);
    if (j < 0) j = 0;
    for (; t1 + (float)j * tb < end; ++j)
      if (fits(t1 + (float)j * tb)) { end = t1 + (float)j * tb; break; }
  }
  return end > t1 ? end : t1;
}

// The last group's end, if that is before `limit`.  Group r has the workgroups r, r + 32, ..: how many of a and of both changes
// where a ends and where b does.
float makespan(const Share &a, const Share &b, float limit) {
  auto of = [](int n, int r) { return n > r ? (n - r - 1) / kGroups + 1 : 0; };
  float end = 0.f;
  int last_na = -1, last_nb = -1;
  for (int r : {0, a.n % kGroups, (a.n + b.n) % kGroups}) {
    const int na = of(a.n, r), nb = of(a.n + b.n, r) - na;
    if (end >= limit || (na == last_na && nb == last_nb)) continue;
    last_na = na;
    last_nb = nb;
    const float t = group_end(na, a.us, nb, b.us);
    if (t > end) end = t;
  }
  return end;
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

PairSide pair_side(const GemmArgs &a, int tile) {
  const TileTime &d = kTileTimes[tile];
  return PairSide{(const bf16 *)a.A, (const bf16 *)a.B, (const bf16 *)a.res, (bf16 *)a.C, a.M, a.N, a.K,
                  (a.M + d.bm - 1) / d.bm, (a.N + d.bn - 1) / d.bn, tile};
}

// What a launch of one product takes, in the tile gemm_dma.hip has for it
float single_us(const GemmArgs &a, bool tn) {
  int bm = 0, bn = 0;
  gemm_dma_tile(a, &bm, &bn);
  auto is = [&](const PairTime &t) { return kTileTimes[t.tile].bm == bm && kTileTimes[t.tile].bn == bn; };
  const PairTime *t = kPairTimes;
  for (const PairTime &p : kPairTimes) if (is(p)) t = &p;
  for (const PairTime &p : kSingleTimes) if (is(p)) t = &p;
  const int tiles = ((a.M + bm - 1) / bm) * ((a.N + bn - 1) / bn), nk = (a.K + 63) / 64;
  const int rounds = ((tiles + kGroups - 1) / kGroups + kGroupCus - 1) / kGroupCus;
  return (float)rounds * (tn ? t->tn_start + t->tn_step * (float)nk : t->nt_start + t->nt_step * (float)nk);
}

// (the tuning aids that name the tile or the kernel of a product are about products one by one)
bool pair_runs(const GemmArgs &nt, const GemmArgs &tn) {
  static const bool tuned =
      getenv("DPSTAGE_GEMM_TILE") != nullptr || getenv("DPSTAGE_GEMM_NT") != nullptr || getenv("DPSTAGE_GEMM_TN") != nullptr;
  return !tuned && nt.mode == kGemmNT && tn.mode == kGemmTN && nt.bias == nullptr && tn.bias == nullptr && nt.C2 == nullptr &&
         tn.C2 == nullptr && gemm_mfma_supported(nt) && gemm_mfma_supported(tn) && gemm_dma_supported(nt) && gemm_dma_supported(tn);
}

}  // namespace

bool gemm_pair_plan(const GemmArgs &nt, const GemmArgs &tn, PairPlan *plan) {
  if (!pair_runs(nt, tn)) return false;
  Share sn[kPairTiles], st[kPairTiles];
  const int nn = shares(nt, false, sn), ntn = shares(tn, true, st);
  const Share *best_nt = nullptr, *best_tn = nullptr;
  float best = single_us(nt, false) + single_us(tn, true) + kLaunchUs;
  for (int i = 0; i < nn; ++i)
    for (int j = 0; j < ntn; ++j) {
      const float mean = ((float)sn[i].n * sn[i].us + (float)st[j].n * st[j].us) / (float)kCus;
      if (mean >= best) continue;   // (the last CU ends no sooner than the mean)
      const float us = st[j].us > sn[i].us ? makespan(st[j], sn[i], best) : makespan(sn[i], st[j], best);
      if (us < best) { best = us; best_nt = &sn[i]; best_tn = &st[j]; }
    }
  if (best_nt == nullptr) return false;
  *plan = PairPlan{best_nt->tile, best_nt->n, best_tn->tile, best_tn->n, best_tn->us > best_nt->us};
  return true;
}

void gemm_pair_tiles(const PairPlan &plan, int tiles[4]) {
  tiles[0] = kTileTimes[plan.nt_tile].bm; tiles[1] = kTileTimes[plan.nt_tile].bn;
  tiles[2] = kTileTimes[plan.tn_tile].bm; tiles[3] = kTileTimes[plan.tn_tile].bn;
}

hipError_t launch_gemm_pair(const GemmArgs &nt, const GemmArgs &tn, const PairPlan &plan, hipStream_t s) {
  constexpr size_t smem = 160 * 1024;   // the largest tile's
  static bool attr_set = false;
  if (!attr_set) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(gemm_pair_kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  hipLaunchKernelGGL(gemm_pair_kernel, dim3((unsigned)(plan.nt_tiles + plan.tn_tiles)), dim3(256), smem, s, pair_side(nt, plan.nt_tile),
                     pair_side(tn, plan.tn_tile), plan.tn_first ? plan.tn_tiles : plan.nt_tiles, plan.tn_first ? 1 : 0);
  return hipGetLastError();
}

}  // namespace dp
