// bf16 GEMM on the gfx950 matrix cores with operand tiles brought into LDS by the
// load unit itself (global_load_lds_dwordx4): no staging registers, no LDS store
// instructions, and the requests can be spread between the MFMAs of a k-step.
//
//   NT: C[M,N] = A[M,K] * B[N,K]^T (+ bias, + residual, optional second output gelu(C))
//   TN: C[M,N] = A[K,M]^T * B[K,N]
// fp32 accumulation, bf16 out.
//
// Preconditions (checked by gemm_dma_supported): K >= 64, M >= BM, N >= BN for the tile chosen,
// 16-byte aligned operands and rows.  Ragged edge tiles are shifted back inside the matrix and
// a ragged last k-step inside the operands, so no load is ever guarded.  No split-K: the
// summation order is fixed.
//
// What bounds it.  On real operands the chip lowers its clock to stay inside its power budget: the
// matrix instructions alone, fed from registers, sustain 1.46-1.70 PFLOP/s as v_mfma_f32_32x32x16 and
// 1.92-1.98 as v_mfma_f32_16x16x32 (one probe, same data), which is why the 16x16 form is used; a wave
// owns as large a part of the tile as its registers hold (128x128 of 256x256, four waves) because every
// byte read from LDS, and every instruction beside an MFMA, costs clock: [16384 x 4096] x 4096 NT 422 us
// with 32x32 MFMAs and eight waves of 64x128, 374 us (1.47 PFLOP/s) now; [4096 x 12288] x 16384 TN
// 1261 -> 1128 us.  The same kernel without its operand requests runs at 1.76 GHz instead of 1.56,
// without its LDS reads at 1.75, without both at 1.86.
//
// LDS layout.  The load unit writes the 64 lanes of a request to 1 KB of consecutive LDS,
// so rows cannot be padded; bank conflicts are avoided by swizzling 16-byte chunks
// instead, which costs nothing on the way in: a lane simply fetches the global chunk
// that belongs at its fixed LDS position.
//   NT: a stage holds the A tile [BM rows][64 k] and the B tile [BN rows][64 k] as
//       128-byte rows; chunk c of row r sits at chunk position c ^ ((r >> 1) & 7), which
//       spreads any 16 consecutive rows of one logical chunk (one 16-byte fragment read)
//       over all 16 chunk positions of the 256-byte bank period.
//   TN: a stage holds the tiles as loaded, [64 k rows][BM] and [64 k rows][BN]; fragments
//       come through the transpose read (ds_read_b64_tr_b16); see tn_swizzle.
//       A tile of 192 columns is two panels of 96, [64 k rows][96] each: its 384-byte rows would not divide a request.
#pragma once
#include "common.h"
#include "kernels.h"

#include <type_traits>
#include <utility>

namespace dp {

namespace {

// The kernel's lambdas hold its accumulators and fragments by reference: one that is not inlined would put them in memory.
#define DP_INLINE __attribute__((always_inline))

// f(integral_constant<int, 0>) .. f(integral_constant<int, N-1>): a loop whose index is a constant in every pass,
// whatever its length (the compiler's own unrolling gives up on bodies as long as a slice of 64 MFMAs, and the
// accumulators then go to memory)
template <typename F, int... I> __device__ __forceinline__ void static_for(F &&f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F> __device__ __forceinline__ void static_for(F &&f) {
  static_for(f, std::make_integer_sequence<int, N>{});
}
template <int N> using Count = std::integral_constant<int, N>;

// Where requests and fragment reads of a slice of `mfmas` MFMAs go: request r of n behind MFMA (2 r + 1) mfmas / (2 n),
// read q of n behind MFMA 3/4 q mfmas / n.  Asked the other way round, by plain loops (the request behind MFMA g, or -1;
// the first read behind MFMA g or later): a pack expansion over requests and reads inside the one over MFMAs made this
// file take 2.5 minutes to compile.
constexpr int request_at(int g, int mfmas, int n) {
  for (int r = 0; r < n; ++r)
    if ((2 * r + 1) * mfmas / (2 * n) == g) return r;
  return -1;
}
constexpr int first_read(int g, int mfmas, int n) {
  int q = 0;
  while (q < n && q * mfmas * 3 / 4 / n < g) ++q;
  return q;
}

constexpr int kMinK = 64;        // one whole k-step
constexpr int kGroupM = 8;       // tile rows of a group of the tile order

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// One request: lane l fetches 16 bytes from uniform_base + byte_off and the unit stores
// them at LDS byte M0 + 16*l.  Invisible to the compiler's wait-count pass; the kernel counts
// them itself (vmcnt retires in order).  M0 is reserved by the compiler (never allocated), and
// nothing else in this file makes it emit an M0 user, so it is simply overwritten; one instruction
// has to stand between its write and the request (a no-op, or an MFMA of the main loop).
// The immediate OFF counts on both sides: it is added to the LDS address and to the global one.
template <int ADD> __device__ __forceinline__ void dma_m0(unsigned lds_base) {
  asm volatile("s_add_u32 m0, %0, %1" :: "s"(lds_base), "n"(ADD) : "m0", "scc", "memory");
}
template <int OFF> __device__ __forceinline__ void dma_load(unsigned byte_off, const void *uniform_base) {
  asm volatile("global_load_lds_dwordx4 %0, %1 offset:%2" :: "v"(byte_off), "s"(uniform_base), "n"(OFF) : "memory");
}
__device__ __forceinline__ void dma_gap() { asm volatile("s_nop 0" ::: "memory"); }
template <int N> __device__ __forceinline__ void wait_vmcnt_mem() {
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}
__device__ __forceinline__ const char *uniform_ptr(const char *p) {
  const uint64_t v = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (const char *)(((uint64_t)hi << 32) | lo);
}

// TN: chunk-position swizzle of k row r of a tile whose rows are ROWB bytes.  A half wave's
// transpose read touches k rows {0..3, 8..11} (or those 16 further) x 32 bytes: bits 0 and 1 of the
// row choose the 64-byte quarter of the bank period, bit 3 the 32-byte half of it.  With 128-byte
// rows (two rows a period) bit 0 of the row is part of the address already, with 192-byte rows (a panel of
// 96 columns) both bits are: four rows on end start in four quarters.
template <int ROWB> __device__ __forceinline__ constexpr int tn_swizzle(int r) {
  return (ROWB == 192 ? 0 : ROWB == 128 ? ((r >> 1) & 1) << 2 : (r & 3) << 2) | ((r >> 3) & 1) << 1;
}

// One tile of the product, by the whole workgroup: tile number `pid` of the order below.
template <int BM, int BN, int WGM, int WGN, int STAGES, bool ACT, bool TN, bool SPLIT>
__device__ __forceinline__ void dma_tile_body(
    const bf16 *__restrict__ A, const bf16 *__restrict__ B, const bf16 *__restrict__ bias,
    const bf16 *__restrict__ res, bf16 *__restrict__ C, bf16 *__restrict__ C2, int gelu_kind, int M, int N, int K,
    int tiles_m, int tiles_n, int pid, int group_m) {
  constexpr int BK = 64;
  constexpr int NW = WGM * WGN;
  constexpr int WM = BM / WGM, WN = BN / WGN, FM = WM / 16, FN = WN / 16;
  constexpr int kRowBytes = BK * 2;                  // NT: one LDS row
  constexpr int CPR = BK / 8;                        // NT: chunks per row
  constexpr int A_BYTES = BM * kRowBytes, B_BYTES = BN * kRowBytes, STAGE_BYTES = A_BYTES + B_BYTES;
  // TN: a tile of 192 columns is two panels of 96, each [64 k rows][192 bytes], every wave's part inside one of them
  constexpr bool PANEL_A = TN && BM == 192, PANEL_B = TN && BN == 192;
  constexpr int ROWB_A = PANEL_A ? 192 : BM * 2, ROWB_B = PANEL_B ? 192 : BN * 2;   // TN: bytes of one k row of a tile (panel)
  static_assert((!PANEL_A || (WM == 96 && NW == 4)) && (!PANEL_B || (WN == 96 && NW == 4)), "a wave's part is in one panel");
  constexpr int NIA = A_BYTES / 1024 / NW, NIB = B_BYTES / 1024 / NW;   // requests per wave per stage
  constexpr int NI = NIA + NIB;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  // No load the compiler knows of is in flight here, and it is told so: in a kernel with several of these bodies it otherwise
  // takes the epilogue's loads of one for pending in the main loop of another and waits for all requests there.
  __builtin_amdgcn_s_waitcnt(0x0f70);

  // tile order: each XCD gets a contiguous run of tiles, walked in groups of `group_m` tile rows
  const int nt = tiles_m * tiles_n;
  {
    const int xcd = pid & 7, idx = pid >> 3, base = nt >> 3, rem = nt & 7;
    pid = xcd * base + (xcd < rem ? xcd : rem) + idx;
  }
  const int group = pid / (group_m * tiles_n);
  const int first_m = group * group_m;
  const int gsz = min(tiles_m - first_m, group_m);
  const int tm = first_m + (pid % (group_m * tiles_n)) % gsz;
  const int tn = (pid % (group_m * tiles_n)) / gsz;
  const int m0 = min(tm * BM, M - BM), n0 = min(tn * BN, N - BN);   // (ragged edge tiles are shifted back inside the matrix)

  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = (wave / WGN) * WM, wn = (wave % WGN) * WN;

  // ---- request addressing -------------------------------------------------------------
  // A tile is A_BYTES / 1024 requests of 1 KB of consecutive LDS; which NIA of them a wave issues
  // is chosen so that their lane offsets take two values, one for its even and one for its odd
  // requests (the swizzle of a row depends on its low four bits).
  //   NT: a request is 8 operand rows x 128 bytes; lane l is row l/8, chunk position l%8
  //       and fetches logical chunk (l%8) ^ ((row >> 1) & 7).  Request j of a wave is number
  //       wave*NIA + j of the tile.
  //   TN: a request is RPR = 1024/ROWB k rows of ROWB bytes; lane l is k row l/(64/RPR),
  //       chunk position l%(64/RPR) and fetches logical chunk position ^ tn_swizzle(krow).  A wave
  //       takes whole groups of 8 k rows, every NW-th (their numbers are then all even or all odd).
  //       Panels of 96 columns: three requests are 16 k rows; 16-byte chunk 64 v + l of them (v = 0, 1, 2) is k row
  //       (64 v + l) / 12, position (64 v + l) % 12.  A wave takes its 16 of the 64 k rows in both panels.
  const unsigned lda = (unsigned)(TN ? M : K) * 2u, ldb = (unsigned)(TN ? N : K) * 2u;   // operand row bytes
  constexpr int RPA = TN ? 1024 / ROWB_A : 8, RPB = TN ? 1024 / ROWB_B : 8;              // rows per request (panels: see start)
  constexpr int GA = PANEL_A ? 3 : TN ? 8 / RPA : 1, GB = PANEL_B ? 3 : TN ? 8 / RPB : 1;   // requests per group
  constexpr int VA = PANEL_A ? 3 : 2, VB = PANEL_B ? 3 : 2;                              // values of the lane offsets
  static_assert((PANEL_A || (RPA >= 2 && RPA <= 8)) && (PANEL_B || (RPB >= 2 && RPB <= 8)), "tile width 64, 128, 192 or 256");
  static_assert(NIA % GA == 0 && NIB % GB == 0 && NW % 2 == 0 && NIA % 2 == 0 && NIB % 2 == 0, "requests of a wave");
  // request j of a wave is number (the wave's first) + rel(j) of the tile
  const int first_a = wave * (TN ? GA : NIA), first_b = wave * (TN ? GB : NIB);
  auto rel = [](int j, int g) constexpr { return TN ? NW * (j / g) * g + j % g : j; };
  // requests with consecutive numbers share an M0 (that of their first, the lead); the request's immediate says
  // how far on it is, and its base pointer makes up for that
  auto lead = [](int j, int g) constexpr { return TN ? j / g * g : j / 4 * 4; };
  unsigned voa[VA], vob[VB];
  auto lane_offset = [&](int v, auto panel_tag, auto rowb_tag, int g, unsigned ld) DP_INLINE -> unsigned {
    constexpr int ROWB = decltype(rowb_tag)::value, RPR = TN ? 1024 / ROWB : 8;
    if constexpr (!TN) {
      const int r = lane / CPR, pc = lane % CPR;
      return (unsigned)r * ld + (unsigned)((pc ^ (((8 * v + r) >> 1) % CPR)) << 4);
    } else if constexpr (decltype(panel_tag)::value) {
      const int k = (64 * v + lane) / 12, p = (64 * v + lane) % 12;
      return (unsigned)k * ld + (unsigned)((p ^ tn_swizzle<ROWB>(k)) << 4);
    } else {
      const int k = lane / (64 / RPR), p = lane % (64 / RPR);
      return (unsigned)k * ld + (unsigned)((p ^ tn_swizzle<ROWB>(8 * (wave & 1) + RPR * (v % g) + k)) << 4);
    }
  };
#pragma unroll
  for (int v = 0; v < VA; ++v) voa[v] = lane_offset(v, std::integral_constant<bool, PANEL_A>{}, Count<ROWB_A>{}, GA, lda);
#pragma unroll
  for (int v = 0; v < VB; ++v) vob[v] = lane_offset(v, std::integral_constant<bool, PANEL_B>{}, Count<ROWB_B>{}, GB, ldb);
  // first byte of request j (number q of the tile) of an operand whose tile starts at row or column `at`
  auto start = [&](const bf16 *X, int j, int q, int rows, bool panel, size_t ld, int at) DP_INLINE {
    if (!TN) return (const char *)X + (size_t)(at + rows * q) * ld;
    return panel ? (const char *)X + (size_t)(16 * wave) * ld + (size_t)(at + 96 * (j / 3)) * 2
                 : (const char *)X + (size_t)(rows * q) * ld + (size_t)at * 2;
  };
  const char *pa[NIA], *pb[NIB];
#pragma unroll
  for (int j = 0; j < NIA; ++j)
    pa[j] = uniform_ptr(start(A, j, first_a + rel(j, GA), RPA, PANEL_A, lda, m0) - 1024 * (j - lead(j, GA)));
#pragma unroll
  for (int j = 0; j < NIB; ++j)
    pb[j] = uniform_ptr(start(B, j, first_b + rel(j, GB), RPB, PANEL_B, ldb, n0) - 1024 * (j - lead(j, GB)));

  const int nk = (K + BK - 1) / BK;
  // A K that is no multiple of 64: the k-steps from the second on are shifted back by `dup` elements
  // like ragged edge tiles, and the elements the first step has in common with the second count as zero
  // in the first.
  const int dup = nk * BK - K;
  const unsigned step_a = TN ? BK * lda : BK * 2u, step_b = TN ? BK * ldb : BK * 2u;
  const unsigned back_a = (unsigned)dup * (TN ? lda : 2u), back_b = (unsigned)dup * (TN ? ldb : 2u);
  // request j for the A (B) tile at LDS byte `at`, in the two parts an MFMA goes between
  const unsigned la0 = (unsigned)first_a * 1024u, lb0 = (unsigned)first_b * 1024u;
  auto m0_a = [&](auto j, unsigned at) DP_INLINE { dma_m0<1024 * rel(lead(j, GA), GA)>(at + la0); };
  auto m0_b = [&](auto j, unsigned at) DP_INLINE { dma_m0<1024 * rel(lead(j, GB), GB)>(at + lb0); };
  auto ld_a = [&](auto j) DP_INLINE { dma_load<1024 * (j - lead(j, GA))>(voa[j % VA], pa[j]); };
  auto ld_b = [&](auto j) DP_INLINE { dma_load<1024 * (j - lead(j, GB))>(vob[j % VB], pb[j]); };
  auto req_a = [&](auto j, unsigned at) DP_INLINE { m0_a(j, at); dma_gap(); ld_a(j); };
  auto req_b = [&](auto j, unsigned at) DP_INLINE { m0_b(j, at); dma_gap(); ld_b(j); };
  // lane offsets of the next k-step (from the first to the second: less by what they have in common)
  auto adv_a = [&](bool first) DP_INLINE {
    const unsigned d = first ? step_a - back_a : step_a;
    static_for<VA>([&](auto v) DP_INLINE { voa[v] += d; });
  };
  auto adv_b = [&](bool first) DP_INLINE {
    const unsigned d = first ? step_b - back_b : step_b;
    static_for<VB>([&](auto v) DP_INLINE { vob[v] += d; });
  };

  // ---- fragment addressing --------------------------------------------------------------
  // A fragment is 16 rows (or columns) x 32 contraction elements: lane l holds row l%16, elements
  // 8*(l/16) .. +7; a k-step has two slices of 32.
  // NT: logical chunk 4*ks + l/16 of that row; with the swizzle that is byte (row*128 + x0) ^ (ks << 6).
  // TN: a 16-lane group fetches 4 k rows x 16 columns per transpose read; lane i of the group
  //     supplies the address of k row i/4, columns 4*(i%4).. and receives column i of all
  //     four rows.  Group g starts at k row 8*g; a second read 4 rows on completes the 8
  //     contraction elements of the operand.
  const unsigned x0 = (unsigned)(((lane >> 4) ^ ((lane & 15) >> 1)) << 4);
  const unsigned fa = (unsigned)(wm + (lane & 15)) * kRowBytes + x0;
  const unsigned fb = (unsigned)(wn + (lane & 15)) * kRowBytes + x0;
  const int ti = lane & 15, trow = 8 * (lane >> 4) + (ti >> 2);              // TN: k row within the slice
  const unsigned tlow = (unsigned)(((ti & 3) >> 1) * 16 + (ti & 1) * 8);
  // fragment `blk` of slice ks of the A (B) tile at LDS byte `base`
  auto frag = [&](unsigned base, int blk, int ks, bool is_b) DP_INLINE -> bf16x8 {
    if (!TN) {
      // the block offset has no bits below 128, so it can stay outside the xor (an immediate of the read)
      return *reinterpret_cast<const bf16x8 *>(lds + (((base + (is_b ? fb : fa)) ^ (unsigned)(ks << 6)) + (unsigned)blk * 16u * kRowBytes));
    }
    const unsigned rowb = is_b ? ROWB_B : ROWB_A;
    const bool panel = is_b ? PANEL_B : PANEL_A;
    const unsigned cw = (unsigned)((panel ? 0 : (is_b ? wn : wm) / 8) + blk * 2);   // first chunk of the 16-column block
    const unsigned sw = is_b ? (unsigned)tn_swizzle<ROWB_B>(trow) : (unsigned)tn_swizzle<ROWB_A>(trow);
    if (panel) base += (unsigned)((is_b ? wn : wm) / 96) * (unsigned)(BK * 192);
    const unsigned off = base + (unsigned)trow * rowb + ((cw ^ sw) << 4) + tlow + (unsigned)ks * 32u * rowb;
    union { s16x4 h[2]; bf16x8 v; } u;
    u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(lds + off));
    u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(lds + off + 4u * rowb));
    return u.v;
  };

  f32x4 acc[FM][FN];
  static_for<FM * FN>([&](auto g) DP_INLINE { acc[g / FN][g % FN] = f32x4{0.f, 0.f, 0.f, 0.f}; });

  // The main loop is software-pipelined by hand over the slices: while the MFMAs of a slice issue,
  // the fragments of the next one are read into the other half of a register double buffer and the
  // operand requests of the pass go out, both spread evenly between the MFMAs (a burst of either
  // would hold the wave, and its MFMAs behind them, at the issue of each).  Scheduling barriers pin
  // that order.
  constexpr int MF = FM * FN, NR = FM + FN;   // MFMAs and fragment reads of a slice
  bf16x8 a[2][FM], b[2][FN];
  using Buf0 = std::integral_constant<int, 0>;
  using Buf1 = std::integral_constant<int, 1>;
  using Yes = std::true_type;
  using No = std::false_type;
  // MFMAs of the slice held in buffer USE (if MUL), beside the reads of slice ks of the tiles at
  // base_a, base_b into the other buffer (if READ) and the requests R0 .. R1-1 of the pass: first the B
  // tile's (to LDS byte to_b), then the A tile's (to to_a).  Request r of NREQ goes out behind MFMA
  // (2 r + 1) MF / (2 NREQ), its M0 is written before that MFMA.
  auto slice = [&](auto use_tag, auto mul_tag, auto read_tag, unsigned base_a, unsigned base_b, int ks, auto r0_tag,
                   auto r1_tag, auto nb_tag, unsigned to_b, unsigned to_a) DP_INLINE {
    constexpr int USE = decltype(use_tag)::value, R0 = decltype(r0_tag)::value, R1 = decltype(r1_tag)::value;
    constexpr int NB = decltype(nb_tag)::value, NREQ = R1 - R0;   // NB: requests of the pass that are B's
    constexpr bool MUL = decltype(mul_tag)::value, READ = decltype(read_tag)::value;
    static_assert(NREQ <= MF, "one request a gap: its M0 is the only one written before its MFMA");
    auto read = [&](auto q_tag) DP_INLINE {   // in the order the next slice needs them: the first row block, all columns, the other rows
      constexpr int q = decltype(q_tag)::value;
      if constexpr (q == 0) a[USE ^ 1][0] = frag(base_a, 0, ks, false);
      else if constexpr (q <= FN) b[USE ^ 1][q - 1] = frag(base_b, q - 1, ks, true);
      else a[USE ^ 1][q - FN] = frag(base_a, q - FN, ks, false);
    };
    auto m0 = [&](auto r_tag) DP_INLINE {
      constexpr int r = decltype(r_tag)::value + R0;
      if constexpr (r < NB) {
        if constexpr (lead(r, GB) == r) m0_b(Count<r>{}, to_b);
      } else {
        if constexpr (lead(r - NB, GA) == r - NB) m0_a(Count<r - NB>{}, to_a);
      }
    };
    auto ld = [&](auto r_tag) DP_INLINE {
      constexpr int r = decltype(r_tag)::value + R0;
      if constexpr (r < NB) ld_b(Count<r>{}); else ld_a(Count<r - NB>{});
    };
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (!MUL) {
      if constexpr (READ) static_for<NR>(read);
      static_for<NREQ>([&](auto r_tag) DP_INLINE {
        constexpr int r = decltype(r_tag)::value + R0;
        if constexpr (r < NB) req_b(Count<r>{}, to_b); else req_a(Count<r - NB>{}, to_a);
      });
    } else {
      static_for<MF>([&](auto g_tag) DP_INLINE {
        constexpr int g = decltype(g_tag)::value, r = request_at(g, MF, NREQ);
        constexpr int q0 = READ ? first_read(g, MF, NR) : 0, q1 = READ ? first_read(g + 1, MF, NR) : 0;
        if constexpr (r >= 0) m0(Count<r>{});
        __builtin_amdgcn_sched_barrier(0);
        acc[g / FN][g % FN] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[USE][g % FN], a[USE][g / FN], acc[g / FN][g % FN], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (r >= 0) ld(Count<r>{});
        static_for<q1 - q0>([&](auto q_tag) DP_INLINE { read(Count<q0 + decltype(q_tag)::value>{}); });
        __builtin_amdgcn_sched_barrier(0);
      });
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // the first k-step of a ragged K: its last dup elements belong to the second
  auto mask = [&](auto buf_tag, int ks) DP_INLINE {
    constexpr int BUF = decltype(buf_tag)::value;
    if (dup > 0) {
      const int keep = BK - dup - (32 * ks + 8 * (lane >> 4));   // how many of this lane's elements count
      auto cut = [&](bf16x8 &f) DP_INLINE {
        union { bf16x8 v; unsigned u[4]; } x;
        x.v = f;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          x.u[e] &= keep >= 2 * e + 2 ? 0xffffffffu : keep == 2 * e + 1 ? 0xffffu : 0u;
        f = x.v;
      };
#pragma unroll
      for (int i = 0; i < FM; ++i) cut(a[BUF][i]);
#pragma unroll
      for (int j = 0; j < FN; ++j) cut(b[BUF][j]);
    }
  };
  // One pass of the loop, for k-step kt, entered right behind the barrier that certified
  // stage kt (so no LDS read is in flight on entry, nor at the loop's back edge: the
  // compiler's wait-count pass only places exact partial waits inside straight-line code):
  //   the MFMAs of the second slice of step kt-1 (not FIRST), beside the reads of the first slice of kt;
  //   the MFMAs of the first slice of kt, beside the reads of its second;
  //   every LDS read of stage kt has now been issued: wait for stage kt+1 and pass the
  //     barrier that certifies it and frees stage kt (NEXT); the MFMAs of the second slice
  //     follow in the next pass (or behind the loop).
  // The pass's NB + NA requests (B's first) go out over its two slices, `EARLY` of them in the first.
  auto pass = [&](auto first_tag, auto next_tag, unsigned base_a, unsigned base_b, auto &&wait_next, auto nb_tag,
                  auto na_tag, auto early_tag, unsigned to_b, unsigned to_a) DP_INLINE {
    constexpr bool FIRST = decltype(first_tag)::value, NEXT = decltype(next_tag)::value;
    constexpr int NB = decltype(nb_tag)::value, NA = decltype(na_tag)::value;
    constexpr int EARLY = decltype(early_tag)::value < NB + NA ? decltype(early_tag)::value : NB + NA;
    slice(Buf1{}, std::integral_constant<bool, !FIRST>{}, Yes{}, base_a, base_b, 0, Count<0>{}, Count<EARLY>{}, nb_tag, to_b, to_a);
    if (FIRST) mask(Buf0{}, 0);
    if (MF >= 32) __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): the reads are in by now; one wait instead of one before each use
    slice(Buf0{}, Yes{}, Yes{}, base_a, base_b, 1, Count<EARLY>{}, Count<NB + NA>{}, nb_tag, to_b, to_a);
    if (FIRST) mask(Buf1{}, 1);
    if (NEXT) {
      wait_next();
      __syncthreads();
    }
  };
  auto last_slice = [&]() DP_INLINE {   // the MFMAs of the last slice of the last k-step
    slice(Buf1{}, Yes{}, No{}, 0u, 0u, 0, Count<0>{}, Count<0>{}, Count<0>{}, 0u, 0u);
  };

  if constexpr (SPLIT) {
    // ---- rings of three A tiles and two B tiles ---------------------------------------------
    // A 256x256 k-step fills 64 KB of LDS, so only two whole stages fit, but a third A tile does beside them.
    // Request order A0 B0 A1 B1 A2 | B2 A3 | B3 A4 ...: pass k asks for B(k+1) and A(k+2) behind the barrier that
    // freed the slots of B(k-1) and A(k-1); a B tile so has one step to land and an A tile one to two.  (The
    // launcher sends K < 3 * BK elsewhere.)
    constexpr int EARLY_REQ = (NIA + NIB) * 3 / 4;   // requests of a pass that go out beside its first slice's MFMAs
    static_for<2>([&](auto t) DP_INLINE {
      static_for<NIA>([&](auto i) DP_INLINE { req_a(i, (unsigned)t * A_BYTES); });
      adv_a(t == 0);
      static_for<NIB>([&](auto i) DP_INLINE { req_b(i, 3u * A_BYTES + (unsigned)t * B_BYTES); });
      adv_b(t == 0);
    });
    wait_vmcnt_mem<NIA + NIB>();
    __syncthreads();
    // the rings, in LDS bytes: A(kt), A(kt+1), A(kt+2); B(kt), B(kt+1)
    unsigned a0 = 0, a1 = A_BYTES, a2 = 2 * A_BYTES, b0 = 3 * A_BYTES, b1 = 3 * A_BYTES + B_BYTES;
    // MORE: k-step kt+2 exists (its A tile is requested in this pass)
    auto step = [&](auto first_tag, auto next_tag, auto more_tag) DP_INLINE {
      constexpr bool FIRST = decltype(first_tag)::value, NEXT = decltype(next_tag)::value,
                     MORE = decltype(more_tag)::value;
      pass(first_tag, next_tag, a0, b0,
           [&]() DP_INLINE { if (MORE) wait_vmcnt_mem<NIA>(); else wait_vmcnt_mem<0>(); },
           Count<(!FIRST && NEXT ? NIB : 0)>{}, Count<(MORE ? NIA : 0)>{}, Count<EARLY_REQ>{}, b1, a2);
      if (!FIRST && NEXT) adv_b(false);
      if (MORE) adv_a(false);
      const unsigned ta = a0, tb = b0;
      a0 = a1; a1 = a2; a2 = ta;
      b0 = b1; b1 = tb;
    };
    step(Yes{}, Yes{}, Yes{});
    for (int left = nk - 3; left > 0; --left) step(No{}, Yes{}, Yes{});
    step(No{}, Yes{}, No{});
    step(No{}, No{}, No{});
  } else {
    // ---- ring of STAGES whole stages ------------------------------------------------------
    // Stage k sits in slot k % STAGES.  Stages 0 .. STAGES-2 are requested up front; pass kt
    // asks for stage kt+STAGES-1, spread over its two slices, into the slot the barrier
    // before it freed, so a stage has STAGES-2 steps and more to land.
    static_assert(STAGES >= 3, "the barrier of a step certifies the next stage");
#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s) {
      if (s < nk) {
        static_for<NIA>([&](auto i) DP_INLINE { req_a(i, (unsigned)s * STAGE_BYTES); });
        adv_a(s == 0);
        static_for<NIB>([&](auto i) DP_INLINE { req_b(i, (unsigned)s * STAGE_BYTES + A_BYTES); });
        adv_b(s == 0);
      }
    }
    if (nk >= STAGES - 1) wait_vmcnt_mem<(STAGES - 2) * NI>(); else wait_vmcnt_mem<0>();
    __syncthreads();
    unsigned cur = 0;                                          // LDS byte of k-step kt's stage
    unsigned nxt = (unsigned)(STAGES - 1) * STAGE_BYTES;       // where the requests of this pass go
    // MORE: k-step kt+STAGES-1 exists (requested in this pass; the stages before it then all
    // exist, so the wait for stage kt+1 may leave STAGES-2 stages pending)
    auto step = [&](auto first_tag, auto next_tag, auto more_tag) DP_INLINE {
      constexpr bool MORE = decltype(more_tag)::value;
      pass(first_tag, next_tag, cur, cur + A_BYTES,
           [&]() DP_INLINE { if (MORE) wait_vmcnt_mem<(STAGES - 2) * NI>(); else wait_vmcnt_mem<0>(); },
           Count<(MORE ? NIB : 0)>{}, Count<(MORE ? NIA : 0)>{}, Count<NI / 2>{}, nxt + A_BYTES, nxt);
      if (MORE) { adv_a(false); adv_b(false); }
      cur = cur + STAGE_BYTES == STAGES * STAGE_BYTES ? 0u : cur + STAGE_BYTES;
      nxt = nxt + STAGE_BYTES == STAGES * STAGE_BYTES ? 0u : nxt + STAGE_BYTES;
    };
    if (nk >= STAGES) step(Yes{}, Yes{}, Yes{});
    else if (nk > 1) step(Yes{}, Yes{}, No{});
    else step(Yes{}, No{}, No{});
    int kt = 1;
    for (; kt + STAGES - 1 < nk; ++kt) step(No{}, Yes{}, Yes{});
    for (; kt + 1 < nk; ++kt) step(No{}, Yes{}, No{});
    if (kt < nk) step(No{}, No{}, No{});
  }
  last_slice();

  // ---- epilogue ---------------------------------------------------------------------------
  // The B fragment is the MFMA's first operand, so element e of lane l of acc[i][j] is
  // C[16*i + l%16][16*j + 4*(l/16) + e] of the wave's part: four consecutive columns of one row.  Lane
  // group g = l/16 gives its half of block j or j+1 to group g ^ 1 (v_permlane16_swap) and then holds
  // eight consecutive columns, 16 * (g & 1) + 8 * (g / 2) onward of the two blocks: 16 bytes a lane and
  // 64 contiguous bytes a row for every global access, straight from the registers.
  const bool wide16 = ((((uintptr_t)C | (uintptr_t)C2 | (uintptr_t)res) & 15) | (uintptr_t)(N & 7)) == 0;
  auto swap2 = [](unsigned (&x)[2], unsigned (&y)[2]) DP_INLINE {   // its own inverse
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const auto r = __builtin_amdgcn_permlane16_swap(x[q], y[q], false, false);
      x[q] = r[0]; y[q] = r[1];
    }
  };
  union Half { bf16x4 v; unsigned u[2]; };
  auto epilogue = [&](auto wide_tag) DP_INLINE {
    constexpr bool wide = decltype(wide_tag)::value;
    const int erow = lane & 15, ecol = 16 * ((lane >> 4) & 1) + 8 * (lane >> 5), ebcol = 4 * (lane >> 4);
    const unsigned elane = ((unsigned)erow * (unsigned)N + (unsigned)ecol) * 2u;
    // A tile that was shifted back stores only the part its unshifted position covers: the rest
    // is its neighbour's (written once, so that C may also be the residual operand).
    const int skip_rows = tm * BM - m0, skip_cols = tn * BN - n0;
    Half bv[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      bv[j].u[0] = bv[j].u[1] = 0u;
      if (bias != nullptr) bv[j].v = *reinterpret_cast<const bf16x4 *>(bias + n0 + wn + 16 * j + ebcol);
    }
    static_for<FM>([&](auto i_tag) DP_INLINE {
      constexpr int i = decltype(i_tag)::value;
      const size_t row_off = ((size_t)(m0 + wm + 16 * i) * (size_t)N + (size_t)(n0 + wn)) * 2;
      // the residual of the 16 rows, asked for before its first use (every tile lies inside the matrix, so
      // rows and columns the tile does not own are read too)
      Half r0[FN / 2], r1[FN / 2];
      if (res != nullptr) {
#pragma unroll
        for (int p = 0; p < FN / 2; ++p) {
          const char *at = (const char *)res + row_off + 64 * p + elane;
          if (wide) {
            const uint4 q = *reinterpret_cast<const uint4 *>(at);
            r0[p].u[0] = q.x; r0[p].u[1] = q.y; r1[p].u[0] = q.z; r1[p].u[1] = q.w;
          } else {
            r0[p].v = reinterpret_cast<const bf16x4 *>(at)[0];
            r1[p].v = reinterpret_cast<const bf16x4 *>(at)[1];
          }
        }
      }
      static_for<FN / 2>([&](auto p_tag) DP_INLINE {
        constexpr int p = decltype(p_tag)::value;
        float v[2][4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          v[0][q] = acc[i][2 * p][q] + (float)bv[2 * p].v[q];
          v[1][q] = acc[i][2 * p + 1][q] + (float)bv[2 * p + 1].v[q];
        }
        if (res != nullptr) {
          swap2(r0[p].u, r1[p].u);
#pragma unroll
          for (int q = 0; q < 4; ++q) { v[0][q] += (float)r0[p].v[q]; v[1][q] += (float)r1[p].v[q]; }
        }
        Half o0, o1, g0, g1;
#pragma unroll
        for (int q = 0; q < 4; ++q) { o0.v[q] = (bf16)v[0][q]; o1.v[q] = (bf16)v[1][q]; }
        if (ACT) {
          // fused activation: computed from the value as stored, so that a later standalone
          // GELU of C gives the same bits
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            g0.v[q] = (bf16)gelu_f<bf16>((float)o0.v[q], gelu_kind);
            g1.v[q] = (bf16)gelu_f<bf16>((float)o1.v[q], gelu_kind);
          }
          swap2(g0.u, g1.u);
        }
        swap2(o0.u, o1.u);
        const int row = wm + 16 * i + erow, col = wn + 32 * p + ecol;
        auto put = [&](bf16 *out, const Half &lo, const Half &hi) DP_INLINE {
          char *at = (char *)out + row_off + 64 * p + elane;
          if (wide) *reinterpret_cast<uint4 *>(at) = make_uint4(lo.u[0], lo.u[1], hi.u[0], hi.u[1]);
          else {
            if (col >= skip_cols) reinterpret_cast<bf16x4 *>(at)[0] = lo.v;
            if (col + 4 >= skip_cols) reinterpret_cast<bf16x4 *>(at)[1] = hi.v;
          }
        };
        if (row >= skip_rows && col + (wide ? 0 : 4) >= skip_cols) {
          put(C, o0, o1);
          if (ACT) put(C2, g0, g1);
        }
      });
      __builtin_amdgcn_sched_barrier(0);   // (the row blocks one after the other, or their temporaries add up)
    });
  };
  if (wide16) epilogue(Yes{}); else epilogue(No{});
}

// Tile choice: the tile with the smallest estimated time.  A launch runs in rounds of one tile a CU (the kernels' bound of
// one wave of theirs a SIMD, two of 128x128's, allows no second, also where registers and LDS would); a
// round takes a start (pipeline fill, output) plus a time per 64-deep k-step (us, below: between what full
// rounds take with operands in the caches and with operands from memory, where small tiles, which fetch more
// bytes per flop, lose more).  A larger tile is faster per flop but covers the output in coarser rounds.
// Measured, operands in the caches / from memory:
//   [4096 x 1600] x 6400 NT: 208 tiles of 256x128 71 / 91 us; 416 of 128x128 (the second round half empty) 87 / 116
//   [4096 x 1600] x 1600 NT: 23 / 29 us against 28 / 35; [1600 x 4800] x 4096 TN: 247 of 128x256 55 / 58, 66 / 80
//   [4096 x 4800] x 1600 NT: 304 of 256x256 72 / 73 us, 1216 of 128x128 68 / 89, 608 of 128x256 67 / 82
//   [4096 x 1024] x 1024 NT: 256 of 128x128 10.5 / 13.8 us, 128 of 256x128 15.5 / 19.3, 64 of 256x256 24.5 / 26.9
//   [2048 x 768] x 3072 NT: 192 of 128x64 17.3 / 24.9 us, 96 of 128x128 20.9 / 31.0, 384 of 64x64 21.4 / 30.3
//   [1024 x 1024] x 4096 TN: 256 of 64x64 16.0 / 22.8 us, 64 of 128x128 27.8 / 37.0, 128 of 128x64 22.3 / 31.5
// The tiles of 192 rows or columns are there for outputs that leave a round of the others half empty (operands from memory):
//   [4096 x 4800] x 1600 NT: 400 of 256x192 67 us (304 of 256x256 75, 608 of 128x256 82); [4096 x 3072] x 1024 26.9 (30.0, 37.8)
//   [1600 x 6400] x 4096 TN: 238 of 256x192 78 us (175 of 256x256 84, 350 of 256x128 108); [6144 x 6144] x 2048 128 (148, 154)
//   [3441 x 1280] x 1280 NT: 189 of 128x192 17.0 us (135 of 128x256 20.3); [1664 x 4992] x 1896 TN 234 of 192x192 33 (520 of 128x128 37)
// Over 30 products of drawn stages they take 4 % off the mean, up to 20 %.  Below nine k-steps, where start and output are most of
// a launch, they gain nothing ([2304 x 3328] x 512 NT: 192x192 14.3 us, 128x256 14.0; TN 14.9 and 14.2): min_steps.  Nor
// are they taken for more than four rounds of theirs (kRounds192): CUs do not start a round together, so the more rounds, the less
// is lost in the last one than the estimate says.  52 products of 2 to 3.2 rounds of 256x256 took 0.90 of its time in three or four
// rounds, one of them longer by more than 1 %; 21 of 4 to 4.6 rounds 1.00, eight of them longer, up to [5828 x 12576] x 840 NT
// 145 / 157 us; 17 of 5 and 6 rounds 0.97, five longer, up to [6016 x 14232] x 1608 TN 262 / 285.
struct TileTime { int bm, bn; float start_us, step_us; int min_steps; };   // min_steps: the fewest k-steps it is chosen for
enum { k256x256, k256x192, k192x256, k192x192, k256x128, k128x256, k192x128, k128x192, k128x128, k128x64, k64x128, k64x64, kTiles };
constexpr TileTime kTileTimes[kTiles] = {
    {256, 256, 6.0f, 1.27f, 3}, {256, 192, 5.2f, 1.03f, 9}, {192, 256, 5.2f, 1.03f, 9}, {192, 192, 4.0f, 0.88f, 9},
    {256, 128, 4.5f, 0.83f, 1}, {128, 256, 4.5f, 0.83f, 1}, {192, 128, 3.5f, 0.70f, 9}, {128, 192, 3.5f, 0.70f, 9},
    {128, 128, 2.0f, 0.55f, 1}, {128, 64, 1.5f, 0.40f, 1},  {64, 128, 1.5f, 0.40f, 1},  {64, 64, 1.5f, 0.26f, 1}};
constexpr int kCus = 256, kRounds192 = 4;
// The fewest k-steps a tile can run: the rings of the three largest are filled before the loop (SPLIT)
constexpr int fewest_steps(int tile) { return tile <= k192x256 ? 3 : 1; }

}  // namespace
}  // namespace dp
