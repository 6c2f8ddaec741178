// The expert FFN's grouped GEMM for any K and N that are multiples of 8: row-major weights with fp32 (rounded to bf16 between
// LDS and the MFMA) or bf16 activations, and packed weights where the tiles here are faster than the 256 x 256 tiles of
// ffn.hip (few rows per segment, few experts, narrow outputs: pick_packed there).
//
// A work-group makes tiles of up to BM rows x BN columns in k-steps of 64 (fp32: 32) with four waves (2 along m x 2 along
// n, 16-row subtiles interleaved between the waves of an axis).  Both operands reach LDS by direct-to-LDS copies into a
// ring of stages that fills half of a compute unit's LDS: two work-groups per compute unit (one's epilogue and barriers
// run beside the other's MFMAs).  Slot functions: 64-byte weight rows (packed, or beside fp32) chunk ^ (row/2 mod 4),
// 128-byte rows chunk ^ (row/2 mod 8); a packed block's 16-column groups are that image already and are copied as they are.
// An fp32 row's even chunks come ahead of its odd ones: a lane's 8 values are two chunks side by side, and in plain order
// conflicts took 0.40 of the LDS-active cycles (now 0; d = 1024, h = 4096, E = 16, 3 330 rows, first GEMM 66.7 -> 65.9 us, with
// Z stored 69.2 -> 68.1: the copies, not the reads, are what the steps wait for).
// Copies past K are clamped into the row and overwritten with zeros on both sides by the lanes that fetched them (an
// infinity times zero would be a NaN).
//
// Every output element is one chain of MFMAs over K in ascending order, as in the 256 x 256 kernels: an element has the same
// bits whichever kernel and tile shape makes it, so a token's result does not depend on the batch's size or capacity.
//
// What bounds it: with few rows the weight stream (5.0 to 5.5 TB/s of 820 MB at 32 to 64 rows per expert, d = 1600,
// h = 6400, E = 40), with more rows all copies to LDS together, 8 to 13 TB/s, of which the activations are the larger part
// the more rows and the fewer columns a tile has.  Hence
//   - the widest tile that still fills the chip in whole turns (any_tiles below picks it);
//   - in runs the tiles of one segment are on one XCD, whose L2 then fetches the segment's activations once, where tiles dealt
//     to the XCDs make each L2 fetch all of them (any_tiles says where that pays);
//   - packed weights here too: E = 16, d = 1024, h = 4096, both GEMMs: 64 rows 37 + 41 -> 29 + 28 us (one wave per 64
//     columns with the weights straight in registers, as ffn_gemm_few has it up to 32 rows), 128 rows 45 + 68
//     (256 x 256 tiles) -> 32 + 36; E = 4, d = 2048, h = 8192, 100 rows, second GEMM 117 -> 46.
#include <math.h>

#include <algorithm>
#include <atomic>
#include <type_traits>

#include "common.h"
#include "ffn_any.h"
#include "ffn_epilogue.h"

namespace locmoe {
namespace {

constexpr int kAnyThreads = 256;
constexpr int kAnyLds = 80 * 1024;   // half of a compute unit's
constexpr int kFine = 128;           // rows of an m-tile of a short list
constexpr int kPackBlock = 16384;    // packed weights: 256 columns x 32 k-values

template <bool A_F32>
struct AnyK {
  static constexpr int kBK = A_F32 ? 32 : 64;
  static constexpr int kARow = 128;   // bytes of an activation row in LDS: one line
  static constexpr int kWRow = kBK * 2;
};
// at most BM rows and BN columns per tile
template <int BM_, int BN_>
struct AnyTile {
  static constexpr int BM = BM_, BN = BN_;
};
template <bool A_F32, class TL, int NJ>
struct AnyShape : AnyK<A_F32> {
  static constexpr int kABytes = 32 * NJ * AnyK<A_F32>::kARow;
  static constexpr int kStage = kABytes + TL::BN * AnyK<A_F32>::kWRow;
  static constexpr int kStages = kAnyLds / kStage > 6 ? 6 : kAnyLds / kStage;
  static_assert(kStages >= 2, "one stage is filled while another is read");
};
// Byte offset, inside a row of RB bytes (a k-step), of the 16-byte chunk that this lane of a 1 KiB copy fetches; the
// copy's block of 1024 / RB rows is number wave + 4 i of the operand.  PAIRS (fp32 rows, whose fragments are two chunks
// side by side): the even chunks of a row come first, so that a read meets the banks as a read of a bf16 row does.
template <int RB, bool PAIRS>
__device__ __forceinline__ uint32_t any_chunk(int wave, int lane) {
  constexpr int L = RB / 16;
  const int row = (RB == 128 ? (wave & 1) * 8 : 0) + lane / L;  // modulo 16
  const int c = (lane & (L - 1)) ^ ((row >> 1) & (L - 1));
  return (uint32_t)((PAIRS ? (c & (L / 2 - 1)) * 2 + c / (L / 2) : c) << 4);
}

// vmcnt(n C) for a run-time n <= MAX
template <int C, int MAX>
__device__ __forceinline__ void wait_younger(int n) {
  static_assert(MAX * C <= 63, "the counter's range");
  if constexpr (MAX == 0) {
    wait_vmcnt<0>();
  } else {
    if (n >= MAX) wait_vmcnt<MAX * C>();
    else wait_younger<C, MAX - 1>(n);
  }
}

// One tile of at most 32 NJ rows.  rows_left: live rows from the tile's first (>= 1).  W: the tile's first weight row, or
// (packed) the first block of the 256 columns that the tile's first lies in.  FAR: a tile's rows reach further than 32-bit
// offsets do.
template <bool A_F32, bool PACKED, int EPI, bool OUT_F32, class TL, int NJ, bool FAR>
__device__ __forceinline__ void any_tile(const char* __restrict__ A, const char* __restrict__ W, void* __restrict__ Cout,
                                         uint16_t* aux, size_t crow0, int rows_left, int n0, int Kdim, int Ndim,
                                         uint32_t lds0, char* smem) {
  using S = AnyShape<A_F32, TL, NJ>;
  constexpr int BN = TL::BN;
  constexpr int NI = BN / 32;                                  // 16-column subtiles of a wave
  constexpr int kSub = S::kBK / 32;                            // MFMA depths per k-step
  constexpr int kARows = 1024 / S::kARow, kWRows = 1024 / S::kWRow;  // rows of a 1 KiB copy
  constexpr int CA = 32 * NJ / kARows / 4, CW = BN / kWRows / 4;     // copies per wave and step
  constexpr int C = CA + CW;
  static_assert(!PACKED || !A_F32, "packed weights go with bf16 activations");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1, kq = lane >> 4, l16 = lane & 15;

  // copies: block wave + 4 i of an operand's stage; rows past the segment's end and columns past the last repeat the
  // last ones (not stored)
  using off_t = std::conditional_t<FAR, uint64_t, uint32_t>;
  const off_t ldA = (off_t)Kdim * (A_F32 ? 4 : 2), ldW = (off_t)Kdim * 2;
  off_t rowA[CA], rowW[CW];
#pragma unroll
  for (int i = 0; i < CA; ++i)
    rowA[i] = (off_t)min((wave + 4 * i) * kARows + lane / (64 / kARows), rows_left - 1) * ldA;
#pragma unroll
  for (int i = 0; i < CW; ++i) {
    if (PACKED) {  // one 16-column group of one of the step's two packed blocks
      const int c = wave + 4 * i, half = c / (BN / 16), n = min((c % (BN / 16)) * 16 + n0, Ndim - 16);
      rowW[i] = (off_t)((n >> 8) - (n0 >> 8)) * ((off_t)Kdim * 512) + (off_t)half * kPackBlock + (n & 255) * 64 + lane * 16;
    } else {
      rowW[i] = (off_t)min((wave + 4 * i) * kWRows + lane / (64 / kWRows), Ndim - n0 - 1) * ldW;
    }
  }
  const uint32_t chA = any_chunk<S::kARow, A_F32>(wave, lane), chW = any_chunk<S::kWRow, false>(wave, lane);
  const int KT = (Kdim - 1) / S::kBK + 1;
  auto copy = [](const char* base, off_t off, uint32_t lds) {
    if constexpr (FAR) dma_1k_far(base + off, lds);
    else dma_1k(base, off, lds);
  };
  auto issue = [&](int s, int stage) {
    const uint32_t base = lds0 + (uint32_t)stage * S::kStage + (uint32_t)wave * 1024;
    const off_t ka = min((off_t)s * S::kARow + chA, ldA - 16), kw = min((off_t)s * S::kWRow + chW, ldW - 16);
#pragma unroll
    for (int i = 0; i < CW; ++i) {
      if (PACKED) copy(W + (size_t)s * (2 * kPackBlock), rowW[i], base + S::kABytes + i * 4096);
      else copy(W, rowW[i] + kw, base + S::kABytes + i * 4096);
    }
#pragma unroll
    for (int i = 0; i < CA; ++i) copy(A, rowA[i] + ka, base + i * 4096);
  };

  // fragment addresses inside a stage: lane l reads the 8 values k = 8 (l/16) .. +7 of row l%16 (two chunks if fp32)
  int off_a[2], off_w[kSub];
  constexpr int kWStep = PACKED ? 64 : S::kWRow;  // bytes between weight rows in LDS
  {
    const int ra = wm * 16 + l16, rw = wn * 16 + l16;  // (subtiles are 32 rows apart: the same swizzle)
#pragma unroll
    for (int i = 0; i < 2; ++i)
      off_a[i] = ra * S::kARow + (((4 * i + kq) ^ ((ra >> 1) & 7)) << 4);
#pragma unroll
    for (int i = 0; i < kSub; ++i) {
      if (PACKED) off_w[i] = S::kABytes + i * BN * 64 + rw * 64 + ((kq ^ ((rw >> 1) & 3)) << 4);
      else off_w[i] = S::kABytes + rw * S::kWRow + (((4 * i + kq) ^ ((rw >> 1) & (S::kWRow / 16 - 1))) << 4);
    }
  }
  f32x4 acc[NI][NJ];
#pragma unroll
  for (int a = 0; a < NI; ++a)
#pragma unroll
    for (int b = 0; b < NJ; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};

#pragma unroll
  for (int s = 0; s < S::kStages - 1; ++s)
    if (s < KT) issue(s, s);
  int stage = 0, fill = S::kStages - 1;
  for (int s = 0; s < KT; ++s) {
    // this step's copies have landed when at most the younger steps' are outstanding (copies complete in issue order
    // and the loop has no other vector memory access)
    wait_younger<C, S::kStages - 2>(KT - 1 - s);
    if (!PACKED && s == KT - 1 && (Kdim & (S::kBK - 1))) {
      char* st = smem + stage * S::kStage + wave * 1024 + lane * 16;
      const uint4 zero = make_uint4(0, 0, 0, 0);
      if ((off_t)s * S::kARow + chA >= ldA) {
#pragma unroll
        for (int i = 0; i < CA; ++i) *(uint4*)(st + i * 4096) = zero;
      }
      if ((off_t)s * S::kWRow + chW >= ldW) {
#pragma unroll
        for (int i = 0; i < CW; ++i) *(uint4*)(st + S::kABytes + i * 4096) = zero;
      }
    }
    __syncthreads();
    if (s + S::kStages - 1 < KT) issue(s + S::kStages - 1, fill);  // into the stage that was read one step ago
    const char* st = smem + stage * S::kStage;
#pragma unroll
    for (int ks = 0; ks < kSub; ++ks) {
      bf16x8 fw[NI], fa[NJ];
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) fw[ni] = *(const bf16x8*)(st + off_w[ks] + ni * 32 * kWStep);
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const char* p = st + j * 32 * S::kARow;
        if (A_F32) {
          const f32x4 a = *(const f32x4*)(p + off_a[0]), b = *(const f32x4*)(p + off_a[1]);
          const u32x4 v = {pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3]), pack_bf16x2(b[0], b[1]), pack_bf16x2(b[2], b[3])};
          fa[j] = __builtin_bit_cast(bf16x8, v);
        } else {
          fa[j] = *(const bf16x8*)(p + off_a[ks]);
        }
      }
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
          acc[ni][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[ni], fa[j], acc[ni][j], 0, 0, 0);
    }
    fill = stage;
    stage = stage + 1 == S::kStages ? 0 : stage + 1;
  }
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int m = (2 * j + wm) * 16 + l16;
    if (m < rows_left) {
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) {
        const int n = n0 + (2 * ni + wn) * 16 + kq * 4;  // a lane holds D[n .. n+3][m]
        if (n < Ndim)  // Ndim % 8 == 0 and n % 4 == 0: the quad is entirely inside or outside
          store_quad<EPI, OUT_F32>(Cout, aux, crow0 + m, Ndim, n, acc[ni][j][0], acc[ni][j][1], acc[ni][j][2],
                                   acc[ni][j][3]);
      }
    }
  }
}

// Inclusive sum over the wave's lanes
__device__ __forceinline__ int wave_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);   // row_shr:1, 2, 4, 8: within 16 lanes
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast:15 into rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // row_bcast:31 into rows 2 and 3
  return v;
}

// The live m-tiles (those of one weight tile in a row, the weight tiles of a segment in a row) form a list, which every
// wave counts out for itself from seg_off; XCD x (work-groups with equal id mod 8) takes the x-th eighth of it.  (Eighths of
// equal bytes instead of equal numbers of tiles are slower where segments are uneven, up to 1.7 times: a tile's time hardly
// depends on its rows.)  (A
// work-group per possible m-tile, most of them without rows, fills the compute units unevenly: work-groups go to the shader
// engines in turn, and where every second one leaves at once, half of the engines stay empty.  Rows even in 0 .. 224,
// d = 2048, h = 8192, E = 32: 340 + 363 us so, 261 + 267 from a list.)
// DEALT: weight tile nt of segment r is XCD (r NT + nt) mod 8's instead, and every XCD has a list of its own: with fp32
// activations (E = 16, d = 1024, h = 4096, 255 rows: 68 against 72 us) and most lists of row-major weights (any_tiles).
// A list that fills the XCD's `slots` (two per compute unit) once or twice is cut into m-tiles of kFine rows where
// that does not take another turn: rows even in 0 .. 256, d = 4096, h = 16384, E = 8, second GEMM: 389 us with up to 192
// rows, 308 with up to 128.
template <bool A_F32, bool PACKED, int EPI, bool OUT_F32, class TL, bool DEALT, bool FAR>
__global__ __launch_bounds__(kAnyThreads, 2) void ffn_gemm_any(const char* __restrict__ A, const char* __restrict__ W,
                                                               void* __restrict__ Cout, uint16_t* aux,
                                                               const int32_t* __restrict__ seg_off,
                                                               const int32_t* __restrict__ buf_expert, int Kdim,
                                                               int Ndim, int NT, int E, int slots) {
  constexpr int BN = TL::BN, kBM = TL::BM;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
  const int xcd = blockIdx.x & 7, lane = threadIdx.x & 63;
  // segments r0 .. r0 + 63, one per lane: first row, rows, expert, m-tiles, inclusive sum of their tiles (`all`: the last
  // of these); `before` tiles precede them
  int r0 = 0, before = 0, seg_l = 0, rows_l = 0, e_l = 0, mtc_l = 0, cum = 0, all = 0;
  int nt_l = 0, cols_l = NT;  // the first of a segment's weight tiles that the list has, and how many it has
  auto look = [&]() {
    const int rl = r0 + lane;
    seg_l = seg_off[min(rl, E)];
    rows_l = seg_off[min(rl + 1, E)] - seg_l;
    e_l = buf_expert[min(rl, E - 1)];
    mtc_l = (rows_l + kBM - 1) / kBM;
    if (DEALT) {
      nt_l = (xcd - rl * NT) & 7;
      cols_l = nt_l < NT ? (NT - 1 - nt_l) / 8 + 1 : 0;
    }
    cum = wave_scan(cols_l * mtc_l);
    all = __builtin_amdgcn_readlane(cum, 63);
  };
  look();
  const int lists = (DEALT ? 1 : 8) * slots;  // work-group slots that a list fills
  long long total = all;
  if (E > 64) {
    for (r0 = 64; r0 < E; r0 += 64) { look(); total += all; }
    r0 = 0;
    look();
  } else if (kFine < kBM && total <= 2 * lists) {
    const int mtc_f = (rows_l + kFine - 1) / kFine;
    const int cum_f = wave_scan(cols_l * mtc_f), all_f = __builtin_amdgcn_readlane(cum_f, 63);
    if (all_f <= (total <= lists ? 1 : 2) * lists) {
      mtc_l = mtc_f;
      cum = cum_f;
      total = all = all_f;
    }
  }
  const int lo = DEALT ? 0 : (int)(total * xcd / 8), hi = DEALT ? (int)total : (int)(total * (xcd + 1) / 8);
  const unsigned stride = gridDim.x >> 3;
  for (unsigned q = blockIdx.x >> 3; q < (unsigned)(hi - lo); q += stride) {
    const int t = lo + (int)q;
    while (t >= before + all) {
      before += all;
      r0 += 64;
      look();
    }
    const int k = __builtin_popcountll(__ballot(before + cum <= t));
    const int in = t - before - (k ? __builtin_amdgcn_readlane(cum, k - 1) : 0);
    const int seg0 = __builtin_amdgcn_readlane(seg_l, k), rows = __builtin_amdgcn_readlane(rows_l, k);
    const int e = __builtin_amdgcn_readlane(e_l, k);
    const int mtc = __builtin_amdgcn_readlane(mtc_l, k);
    int nt = in, mt = 0, span = (rows + 15) & ~15;
    if (mtc > 1) {  // rows evenly over the m-tiles, in whole subtiles: at most kBM (a multiple of 16), the last has some
      nt = in / mtc;
      mt = in - nt * mtc;
      span = ((rows + mtc - 1) / mtc + 15) & ~15;
    }
    if (DEALT) nt = __builtin_amdgcn_readlane(nt_l, k) + 8 * nt;
    const int m0 = mt * span, n0 = nt * BN;
    const int left = __builtin_amdgcn_readfirstlane(min(rows - m0, span));
    const char* At = A + ((size_t)seg0 + m0) * Kdim * (A_F32 ? 4 : 2);
    const char* Wt = W + ((size_t)e * Ndim + (PACKED ? n0 & ~255 : n0)) * Kdim * 2;
    // (the copies of a tile overwrite what the last step of the one before read)
    if (q >= stride) __syncthreads();
#define LOCMOE_ANY_TILE(NJ) \
  any_tile<A_F32, PACKED, EPI, OUT_F32, TL, NJ, FAR>(At, Wt, Cout, aux, (size_t)seg0 + m0, left, n0, Kdim, Ndim, lds0, smem)
    const int nj = (left + 31) >> 5;
    if (nj == 1) LOCMOE_ANY_TILE(1);
    else if (nj == 2) LOCMOE_ANY_TILE(2);
    else if (nj == 3) LOCMOE_ANY_TILE(3);
    else if (kBM == 128 || nj == 4) LOCMOE_ANY_TILE(4);
    else if constexpr (kBM > 128) {
      if (kBM == 160 || nj == 5) LOCMOE_ANY_TILE(5);
      else if constexpr (kBM > 160) LOCMOE_ANY_TILE(6);
    }
#undef LOCMOE_ANY_TILE
  }
}

template <bool A_F32, bool PACKED, int EPI, bool OUT_F32, class TL, bool DEALT, bool FAR>
int launch_any(const void* A, const void* W, void* C, void* aux, const int32_t* seg_off, const int32_t* buf_expert, int E,
               int rows_max, int T, int Kdim, int Ndim, hipStream_t st) {
  const int NT = ceil_div(Ndim, TL::BN);
  // m-tiles: at most those of full segments, and at most a partial one per segment beside those that T rows fill
  const int bm = std::min(TL::BM, kFine);
  const long long mtiles = std::min((long long)E * ceil_div(rows_max, bm), (long long)E + T / bm);
  const long long tiles = DEALT ? 8 * ceil_div(NT, 8) * mtiles : (NT * mtiles + 7) / 8 * 8;
  if (tiles > 0x7FFFFFFFLL) return LOCMOE_ERR_SHAPE;
  // (a launch takes fewer than 2^32 threads along x: a longer list is walked in turns)
  const long long grid = std::min<long long>(tiles, 1 << 23);
  auto kern = ffn_gemm_any<A_F32, PACKED, EPI, OUT_F32, TL, DEALT, FAR>;
  static std::atomic<uint64_t> lds_allowed;
  if (!allow_lds((const void*)kern, kAnyLds, lds_allowed)) return LOCMOE_ERR_HIP;
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(kAnyThreads), kAnyLds, st, (const char*)A, (const char*)W, C,
                     (uint16_t*)aux, seg_off, buf_expert, Kdim, Ndim, NT, E, cu_count() / 4);
  return launch_status();
}

// Expected time in us of a GEMM with `rows` rows in each of E segments in tiles of BM x BN: turns of tiles (one or two
// work-groups per compute unit), each an epilogue and K/64 steps, a step bounded by the latency of a stage's copies, by what
// all compute units together copy (17 TB/s) or by LDS and MFMA cycles; all of it no faster than the weights (5 TB/s).
// The constants are a fit to 212 launches; over 750 other GEMMs of 24 layers (E = 4 .. 256, d = 256 .. 4096, h = 512 .. 16384, 1 to
// 4 096 rows per expert, packed and row-major: profiles/ffn_kernels_by_shape_and_spread.txt) it is 12 % off in the mean, and
// of the four shapes of any_fastest it picks one that is on average 1.3 % (at most 23 %) slower than the best of them.  Always
// 192 x 128: 8 %; 160 x 160: 12 %; 128 x 64: 22 %; 128 x 32: 63 %.
double any_time(int BM, int BN, int E, int rows, int Kdim, int Ndim) {
  const int cus = cu_count(), NT = ceil_div(Ndim, BN);
  int mt = ceil_div(rows, BM);
  const long long W = (long long)E * NT * mt, Wf = (long long)E * NT * ceil_div(rows, kFine);
  if (BM > kFine && E <= 64 && W <= 4 * cus && Wf <= (W <= 2 * cus ? 2 : 4) * cus) mt = ceil_div(rows, kFine);
  const long long tiles = (long long)E * NT * mt;
  const int NJ = ceil_div(ceil_div(rows, mt), 32), NI = BN / 32, bytes = 4096 * NJ + 128 * BN;
  const int stages = std::min(6, kAnyLds / bytes);
  const double work = 0.64 / 2400.0 * std::max(64 * (NI + NJ) + bytes / 128, 32 * NI * NJ);
  auto turn = [&](int per_cu) {
    const double step = soft_max(0.47 / (stages - 1) + work, per_cu * cus * (bytes / 17e6), per_cu * work);
    return 0.22 * NI * NJ + ceil_div(Kdim, 64) * step;
  };
  const long long full = tiles / (2 * cus), rest = tiles % (2 * cus);
  double t = 2.5 + full * turn(2) + (rest > cus ? turn(2) : rest ? turn(1) : 0.0);
  if (mt > 1 && tiles <= cus) t *= 1.1;  // (a segment's last tile has few rows, and its compute unit nothing else)
  return soft_max(t, 2.5 + (double)E * Ndim * Kdim * 2 / 5e6);
}

// the tile shape of a GEMM with the shortest expected time, and that time
AnyTiles any_fastest(int E, int rows, int Kdim, int Ndim, double* us) {
  static constexpr int shape[4][2] = {{192, 128}, {160, 160}, {128, 64}, {128, 32}};
  int best = 0;
  for (int i = 0; i < 4; ++i) {
    const double t = any_time(shape[i][0], shape[i][1], E, rows, Kdim, Ndim);
    if (i == 0 || t < *us) { *us = t; best = i; }
  }
  return {shape[best][0], shape[best][1], false, false};
}

}  // namespace

double any_gemm_time(int E, int rows, int Kdim, int Ndim) {
  double us = 0.0;
  any_fastest(E, rows, Kdim, Ndim, &us);
  return us;
}

AnyTiles any_tiles(bool a_f32, bool packed, int E, int rows_max, int T, int Kdim, int Ndim) {
  const int rows = std::min(rows_max, ceil_div(T, E));  // with evenly spread tokens
  if (a_f32) {
    if ((long long)Kdim * 4 * 128 > 0xFFFFFFFFLL) return {128, 128, true, true};
    // 128 columns per tile, or 64 where that leaves some of the chip's work-group slots (two per compute unit) empty
    const bool wide = (long long)E * ceil_div(Ndim, 128) * ceil_div(rows, 128) >= 2 * cu_count();
    return {128, wide ? 128 : 64, true, false};
  }
  // (packed weights have shorter rows; the weight rows' offsets are no larger)
  if (!packed && (long long)Kdim * 2 * 192 > 0xFFFFFFFFLL) return {192, 128, false, true};
  if (packed) {
    double us;
    return any_fastest(E, rows, Kdim, Ndim, &us);
  }
  // Row-major weights.  192 x 128 goes in runs where the XCDs together would fetch more bytes of activations than there are
  // weights, unless a segment's activations are far beyond an XCD's 4 MiB of L2, and with the inner size the shorter one only
  // from twice as many on.  us, dealt / runs, second GEMM: E = 16, d = 1024, h = 4096, 750 rows 131 / 97, 2 048 rows (17 MB)
  // 324 / 276;  E = 64, d = 1024, h = 2736, 188 rows 166 / 124;  E = 6, d = 768, h = 3072, 5 462 rows (34 MB) 227 / 192;
  // E = 8, d = 2048, h = 8192, 4 096 rows (67 MB) 1 243 / 1 351.  First: E = 16, 750 rows 118 / 122;  E = 48, d = 384, h = 1536,
  // 683 rows 81 / 73.
  const bool runs = 8LL * rows >= Ndim && (Kdim > Ndim || 4LL * rows >= Ndim) && (long long)rows * Kdim <= 30000000;
  // 192 x 128, or 192 x 64 dealt where that leaves slots empty, unless another shape is expected 1.05 times as fast (160 x 160
  // of 64 experts or more: 1.03).  The expected times know nothing of uneven tokens, which cost the least in dealt tiles and the
  // most in 160 x 160 of few experts and short lists: 1.25 there (E = 12, d = 1536, h = 4096, 417 rows, first GEMM, these /
  // 192 x 128 dealt: even 80 / 93, 60 % on one expert 71 / 50).  Nothing is asked for where no segment is longer than a subtile or
  // two and few are empty, or the capacity cuts at two thirds of the even share or less: every tile is much the same there.  192 x 64 makes each XCD fetch all activations once more, which the
  // times do not know either: where 192 x 128 goes in runs, it is taken unless it is expected 5 % slower (E = 4, d = 512,
  // h = 2048, 3 000 rows, second GEMM 58 / 32).
  // Over 588 GEMMs of 14 layers, each with four spreads of the tokens (even; a power law; 60 % on one expert; 80 % on four),
  // against 192 x 128 and 192 x 64 dealt alone: 1.05 times as fast (even: 1.07), 39 GEMMs more than 7 % slower for one of the
  // spreads, 14 more than 15 % (the last rule's tiles as 192 x 64 dealt).  With 1.15 and 1.25 asked for and runs for K > N and up to 16 MB only: 1.03 (1.04), 12 and 3; the shape
  // expected fastest, whatever the distance: 1.05 (1.08), 105 and 42 of 518.
  const bool wide = (long long)E * ceil_div(Ndim, 128) * ceil_div(rows, 192) >= 2 * cu_count();
  const double wide_us = any_time(192, 128, E, rows, Kdim, Ndim), narrow_us = any_time(192, 64, E, rows, Kdim, Ndim);
  const bool alike = (rows_max <= 32 && T > 4LL * E) || 2LL * T >= 3LL * E * rows_max;
  AnyTiles t = {192, wide || (runs && wide_us < 1.05 * narrow_us) ? 128 : 64, !runs, false};
  if (t.bn == 64) t.dealt = true;
  double us = t.bn == 128 ? wide_us : narrow_us;
  auto consider = [&](AnyTiles other, double times) {
    const double u = (alike ? 1.0 : times) * any_time(other.bm, other.bn, E, rows, Kdim, Ndim);
    if (u < us) { us = u; t = other; }
  };
  if (wide) consider({192, 64, true, false}, 1.05);
  else if (!runs) consider({192, 128, true, false}, 1.05);
  consider({160, 160, false, false}, E >= 64 ? 1.03 : E >= 16 || rows >= 700 ? 1.05 : 1.25);
  consider({128, 32, false, false}, 1.05);
  // 128 x 64 in runs for 192 x 64 dealt where segments are cut at, or little above, the even share: second GEMM of E = 16, d = 1024,
  // h = 4096, 256 rows, C = 320, 60.4 us (192 x 128 in runs 64.6); E = 40, d = 1600, h = 3200, 8 rows 68.1 / 71.5 dealt.
  // Not where 128 rows make more tiles of a segment (E = 8, d = 4096, h = 10 928, 138 rows, a training step: 2 184 / 2 229 us).
  if (t.bm == 192 && t.bn == 64 && 3LL * rows_max <= 4LL * rows && any_time(128, 64, E, rows, Kdim, Ndim) <= 1.02 * narrow_us)
    t = {128, 64, false, false};
  return t;
}

template <bool A_F32, bool PACKED, int EPI, bool OUT_F32>
int any_gemm(const void* A, const void* W, void* C, void* aux, const int32_t* seg_off, const int32_t* buf_expert, int E,
             int rows_max, int T, int Kdim, int Ndim, hipStream_t st) {
  // (a limit of the interface, see the header; the grid has none that buffers of a card reach)
  if (!PACKED && (A_F32 || Kdim % 64 || Ndim % 256) && (long long)E * ceil_div(rows_max, 64) > 65535)
    return LOCMOE_ERR_SHAPE;
  const AnyTiles t = any_tiles(A_F32, PACKED, E, rows_max, T, Kdim, Ndim);
#define LOCMOE_ANY(BM, BN, DEALT, FAR)                                                                                    \
  return launch_any<A_F32, PACKED, EPI, OUT_F32, AnyTile<BM, BN>, DEALT, FAR>(A, W, C, aux, seg_off, buf_expert, E,        \
                                                                              rows_max, T, Kdim, Ndim, st)
  if constexpr (A_F32) {
    if (t.far) LOCMOE_ANY(128, 128, true, true);
    if (t.bn == 128) LOCMOE_ANY(128, 128, true, false);
    LOCMOE_ANY(128, 64, true, false);
  } else {
    if constexpr (!PACKED) {
      if (t.far) LOCMOE_ANY(192, 128, false, true);
      if (t.dealt && t.bn == 128) LOCMOE_ANY(192, 128, true, false);
      if (t.dealt) LOCMOE_ANY(192, 64, true, false);
    }
    switch (t.bn) {
      case 160: LOCMOE_ANY(160, 160, false, false);
      case 64: LOCMOE_ANY(128, 64, false, false);
      case 32: LOCMOE_ANY(128, 32, false, false);
      default: LOCMOE_ANY(192, 128, false, false);
    }
  }
#undef LOCMOE_ANY
}

#define LOCMOE_ANY_GEMM(...)                                                                                      \
  template int any_gemm<__VA_ARGS__>(const void*, const void*, void*, void*, const int32_t*, const int32_t*, int, \
                                     int, int, int, int, hipStream_t);
LOCMOE_ANY_GEMM(false, true, kEpiNone, false)
LOCMOE_ANY_GEMM(false, true, kEpiGelu, false)
LOCMOE_ANY_GEMM(false, false, kEpiNone, false)
LOCMOE_ANY_GEMM(false, false, kEpiGelu, false)
LOCMOE_ANY_GEMM(false, true, kEpiGeluSave, false)
LOCMOE_ANY_GEMM(false, true, kEpiGeluGrad, false)
LOCMOE_ANY_GEMM(false, false, kEpiGeluSave, false)
LOCMOE_ANY_GEMM(false, false, kEpiGeluGrad, false)
LOCMOE_ANY_GEMM(false, false, kEpiNone, true)
LOCMOE_ANY_GEMM(true, false, kEpiGelu, false)
LOCMOE_ANY_GEMM(true, false, kEpiGeluSave, false)
LOCMOE_ANY_GEMM(true, false, kEpiGeluGrad, false)
}  // namespace locmoe
