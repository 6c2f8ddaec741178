// Weight gradients of Eq. 1's two linear maps, per expert segment of the send buffer:
//   dW_out[e] = dout_e^T . H_e   ([d,h]),   dW_in[e] = dZ_e^T . send_e   ([h,d])
// i.e. G[e][m][n] = sum over the segment's rows r of P[r][m] * Q[r][n].  Both operands are stored with the
// contracted axis (the rows) outermost, the opposite of what an MFMA lane wants (8 consecutive k for one
// m or n).  gfx950's transposing LDS read (ds_read_b64_tr_b16) delivers exactly that from a k-major tile:
// within 16 lanes, lane i receives element i%4 of the 8-byte groups addressed by lanes i/4, i/4+4, i/4+8,
// i/4+12, so when lane s addresses row k0 + s/4, columns c0 + 4 (s%4).., lane i ends up with column c0 + i
// of rows k0..k0+3.
// The contraction is short (a segment has at most C rows) and the output is large (E d h values per weight):
// at the paper's headline shape writing G takes a quarter of the kernel's time (measured by leaving the stores
// out), the rest is the MFMA loop at the rate of the forward GEMMs.
#include <algorithm>

#include "common.h"

namespace locmoe {
namespace {

constexpr int kWgTile = 256;              // output tile: 256 (m) x 256 (n)
constexpr int kWgK = 32;                  // rows of the segment per step
constexpr int kWgThreads = 512;           // eight waves, each 64 x 128 of the tile

typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;

// MFMA kernel for shapes whose d and h are multiples of 256 (the paper's).  One work-group per compute unit
// walks through its tiles; the operand tiles of the next three k-steps (of this tile or the next) are always in flight as direct global->LDS copies
// into a ring of four stages, so the short contraction (at most C rows: 16 steps at C = 501) never starts
// cold.  Copies complete in issue order among themselves, so a counted wait (as many as were issued after the
// step's own) tells when a step's data has landed, also with the previous tile's stores still in flight.
// Eight waves, two per SIMD: one's fragment reads, address arithmetic and epilogue run beside the other's MFMAs, which is
// worth more than the 24 transposing reads per 32 MFMAs (four waves of 128 x 128: 32 per 64) cost.  Both GEMMs, us, four
// waves / eight: E = 64, d = 4096, h = 16384: 400 rows 7 876 / 7 607, uneven up to 501 6 523 / 6 056, 128 rows 3 995 / 3 708;
// E = 32, d = 2048, h = 8192, uneven up to 1 024 rows 1 549 / 1 423 (986 TFLOP/s);  E = 16, d = 1024, h = 4096, up to 640
// 162 / 145.  A higher wave priority around the MFMAs: up to 6 % slower.
// LDS rows are 512 B with the 16-byte chunk index XORed by 2 s(row), s = row mod 4 plus
// 4 (bit 3 of the row): the eight rows that 32 lanes of the transposing read touch (rows r..r+3 and r+8..r+11,
// 32 B each) then fall into all 64 banks once; with row mod 4 alone half of the LDS cycles were bank conflicts.
// Rows past the segment's end are read clamped (finite duplicates of the last row) and the P side's copies of
// them are overwritten with zeros by the wave that fetched them, so their products vanish.
// Tiles: XCD x (work-groups x mod 8) owns whole segments, so an expert's operands live in one L2; inside a
// segment, 32 consecutive tiles (the XCD's work-groups at one time) form a block of 4 m-tiles x 8 n-tiles
// (12 operand tiles for 32 outputs).  Segments without rows have no tiles; their gradients are zero-filled at the end (a
// launch of its own for that took 5 us).
constexpr int kWgQBytes = kWgK * kWgTile * 2;   // the Q tile of a step: 32 rows x 256 columns, 16 KiB

struct WgShape {
  static constexpr int kMJ = 4;                    // 16-row m-subtiles per wave: a wave owns 64 x 128 of the tile
  static constexpr int kTM = 4 * kMJ * 16;         // tile rows (m): 256
  static constexpr int kPRow = kTM * 2;            // bytes of a P row in LDS
  static constexpr int kPBytes = kWgK * kPRow;
  static constexpr int kStage = kPBytes + kWgQBytes;
  static constexpr int kStages = 4;
  static constexpr int kSmem = kStages * kStage;   // 128 KiB: one work-group per compute unit
  static constexpr int kPLanes = kPRow / 16;       // lanes per P row in a copy
  static constexpr int kPRowsPerCopy = 64 / kPLanes;
  static constexpr int kPCopies = 4 / kPRowsPerCopy;      // per wave and step (a wave copies 4 of the 32 rows)
  static constexpr int kCopies = kPCopies + 2;            // ... plus two for the Q tile
};

struct WgTile {          // wave-uniform
  const char* P;         // the segment's first row at the tile's first m column
  const char* Q;         // ... n column
  uint16_t* G;           // the output tile's origin
  int rows;              // rows of the segment (> 0)
};

__device__ __forceinline__ const char* uniform_ptr(const char* p) {
  const uint64_t v = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (const char*)(((uint64_t)hi << 32) | lo);
}

// rows k0..k0+3 and k0+4..k0+7 of one column: two transposing reads, four LDS rows apart
template <int ROW_BYTES>
__device__ __forceinline__ bf16x8 read_tr8_sw(lds_cptr p) {
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)p);
  const s16x4 hi =
      __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p + 4 * ROW_BYTES));
  const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, v);
}

__global__ __launch_bounds__(kWgThreads) void wgrad_dma_kernel(
    const uint16_t* __restrict__ P, const uint16_t* __restrict__ Q, uint16_t* __restrict__ G,
    const int32_t* __restrict__ seg_off, const int32_t* __restrict__ buf_expert, int Mdim, int Ndim, int E) {
  using S = WgShape;
  constexpr int MJ = S::kMJ;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int MT = Mdim / S::kTM, NT = Ndim / kWgTile;
  const int tpe = MT * NT;
  const int total = E * tpe;
  const int nwg = gridDim.x;
  // work-groups that run side by side on an XCD take a block of MB x 8 tiles of one segment
  constexpr int MB = 4;
  const bool blocked = (MT % MB == 0) && (NT % 8 == 0);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
  lds_cptr lds = (lds_cptr)(uintptr_t)lds0;

  // Which segments an XCD owns.  With E a multiple of 8 the segments are ranked by descending row count and
  // dealt to the XCDs in boustrophedon order (ranks 0..7 to XCDs 0..7, ranks 8..15 to XCDs 7..0, ...): every
  // XCD gets E/8 segments with nearly the same number of rows, largest first (the headline input: 16 % more
  // steps on the busiest XCD with contiguous eighths of the buffer order, 1 % this way).  Otherwise tile t
  // simply is tile t of the segment-major list.
  __shared__ int32_t s_tab[128];  // segment of this XCD's local rank k
  const bool ranked = (E & 7) == 0;
  if (ranked) {
    int32_t* s_seg = (int32_t*)smem;  // [E+1], before the ring is in use
    for (int t = tid; t <= E; t += kWgThreads) s_seg[t] = seg_off[t];
    __syncthreads();
    const int xcd = blockIdx.x & 7;
    for (int t = tid; t < E; t += kWgThreads) {
      const int mine = s_seg[t + 1] - s_seg[t];
      int rank = 0;
      for (int q = 0; q < E; ++q) {
        const int other = s_seg[q + 1] - s_seg[q];
        rank += (other > mine || (other == mine && q < t)) ? 1 : 0;
      }
      const int deal = rank >> 3, pos = rank & 7;
      if (((deal & 1) ? 7 - pos : pos) == xcd) s_tab[deal] = t;
    }
    __syncthreads();  // the table is complete and nobody reads the staging area any more
  }

  // tile number t of the launch (t mod 8 = XCD) -> segment and position inside it
  auto tile_of = [&](int t, int& rows_out) -> WgTile {
    int r, within;
    if (ranked) {
      const int j = t >> 3, k = j / tpe;  // the XCD's j-th tile lies in its k-th segment
      r = __builtin_amdgcn_readfirstlane(s_tab[k]);
      within = j - k * tpe;
    } else {
      r = t / tpe;
      within = t - r * tpe;
    }
    int mt, nt;
    if (blocked) {
      const int b = within / (MB * 8), i = within % (MB * 8), mb = MT / MB;
      mt = (b % mb) * MB + (i % MB);
      nt = (b / mb) * 8 + (i / MB);
    } else {
      mt = within % MT;
      nt = within / MT;
    }
    const int seg0 = seg_off[r];
    rows_out = seg_off[r + 1] - seg0;
    WgTile w;
    w.rows = rows_out;
    w.P = uniform_ptr((const char*)(P + (size_t)seg0 * Mdim + (size_t)mt * S::kTM));
    w.Q = uniform_ptr((const char*)(Q + (size_t)seg0 * Ndim + (size_t)nt * kWgTile));
    w.G = G + ((size_t)buf_expert[r] * Mdim + (size_t)mt * S::kTM) * Ndim + (size_t)nt * kWgTile;
    return w;
  };
  // the first tile at or after t (in this work-group's sequence) whose segment has rows
  auto next_live = [&](int t, WgTile& w) -> int {
    while (t < total) {
      int rows;
      w = tile_of(t, rows);
      if (rows > 0) break;
      t += nwg;
    }
    return __builtin_amdgcn_readfirstlane(t);
  };

  // G[e] = 0 for experts whose segment has no rows: a share of every such matrix per work-group, at its end
  auto zero_empty = [&]() {
    const size_t chunks = (size_t)Mdim * Ndim / 8;
    for (int r0 = 0; r0 < E; r0 += kWave) {
      const int a = seg_off[min(r0 + lane, E)], b = seg_off[min(r0 + lane + 1, E)];
      unsigned long long empty = __ballot(r0 + lane < E && a == b);
      for (; empty; empty &= empty - 1) {
        uint4* g = (uint4*)G + (size_t)buf_expert[r0 + __builtin_ctzll(empty)] * chunks;
        for (size_t i = (size_t)blockIdx.x * kWgThreads + tid; i < chunks; i += (size_t)nwg * kWgThreads)
          nt_store16(make_uint4(0, 0, 0, 0), g + i);
      }
    }
  };

  WgTile cur;
  int t_cur = next_live(blockIdx.x, cur);
  if (t_cur >= total) return zero_empty();

  // ---- the copy side: a cursor kStages - 1 steps ahead of the compute side
  WgTile pf = cur;
  int t_pf = t_cur, k_pf = 0, stage_pf = 0;
  bool pf_live = true;
  const int prow = lane / S::kPLanes, pch = lane % S::kPLanes;  // P copies: row inside the copy, chunk
  const int qrow = lane >> 5, qch = lane & 31;                  // Q copies
  const uint32_t ldP = (uint32_t)Mdim * 2, ldQ = (uint32_t)Ndim * 2;
  const int swz_hi = ((wave >> 1) & 1) << 2;  // bit 3 of the rows this wave copies (rows 4 wave .. 4 wave + 3)
  // What a copy's source offset is made of, per lane and copy, computed once: the row's byte offset inside a step
  // and the (swizzled) chunk.  A step then costs an add, a min (rows past the segment's end re-read its last row)
  // and an add per copy instead of a multiplication and the swizzle arithmetic (1.1 ms of the 8.3 ms of both GEMMs at E = 64,
  // d = 4096, h = 16384, C = 501, with four waves).  The two copies of an operand land in consecutive KiB of LDS: one M0
  // write serves them, each copy carries its KiB as immediate offset, which the hardware also adds to the source address; it is taken
  // off the chunk term again (from a base 4 KiB below the operand, so that the offset stays non-negative).
  static_assert(S::kPCopies == 2 && S::kPRowsPerCopy == 2, "the copy tables assume 512-byte P rows");
  uint32_t rowP[2], chP[2], rowQ[2], chQ[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int r4p = 2 * q + prow, r4q = 2 * q + qrow;  // row inside the wave's four
    rowP[q] = (uint32_t)(4 * wave + r4p) * ldP;
    chP[q] = (uint32_t)(pch ^ (((r4p & 3) | swz_hi) << 1)) * 16 + 4096 - q * 1024;
    rowQ[q] = (uint32_t)(4 * wave + r4q) * ldQ;
    chQ[q] = (uint32_t)(qch ^ (((r4q & 3) | swz_hi) << 1)) * 16 + 4096 - q * 1024;
  }
  auto issue = [&]() -> bool {
    if (!pf_live) return false;
    const uint32_t sbase = lds0 + (uint32_t)stage_pf * S::kStage;
    const uint32_t kP = (uint32_t)k_pf * ldP, kQ = (uint32_t)k_pf * ldQ;                     // this step's first row
    const uint32_t endP = (uint32_t)(pf.rows - 1) * ldP, endQ = (uint32_t)(pf.rows - 1) * ldQ;  // the segment's last row
    dma_base(sbase + (uint32_t)wave * 4 * S::kPRow);
#pragma unroll
    for (int q = 0; q < 2; ++q) dma_1k_sub(pf.P - 4096, min(rowP[q] + kP, endP) + chP[q], q);
    dma_base(sbase + S::kPBytes + (uint32_t)wave * 2048);
#pragma unroll
    for (int q = 0; q < 2; ++q) dma_1k_sub(pf.Q - 4096, min(rowQ[q] + kQ, endQ) + chQ[q], q);
    stage_pf = stage_pf + 1 == S::kStages ? 0 : stage_pf + 1;
    k_pf += kWgK;
    if (k_pf >= pf.rows) {
      t_pf = next_live(t_pf + nwg, pf);
      pf_live = t_pf < total;
      k_pf = 0;
    }
    return true;
  };
  int ahead = 0;  // steps issued and not yet computed
#pragma unroll
  for (int i = 0; i < S::kStages - 1; ++i) ahead += issue() ? 1 : 0;

  // ---- the compute side
  const int wm = wave >> 1, wn = wave & 1;
  const int kq = lane >> 4, l16 = lane & 15;
  const int sw = (l16 >> 2) | ((kq & 1) << 2);  // the swizzle of the rows this lane addresses
  int off_m[MJ], off_n[8];  // this lane's byte offsets inside a stage for its subtiles
  {
    const int row = 8 * kq + (l16 >> 2), b1 = (l16 & 3) >> 1, inner = (l16 & 1) * 8;
#pragma unroll
    for (int j = 0; j < MJ; ++j) off_m[j] = row * S::kPRow + (((2 * MJ * wm + 2 * j + b1) ^ (sw << 1)) << 4) + inner;
#pragma unroll
    for (int j = 0; j < 8; ++j) off_n[j] = S::kPBytes + row * 512 + (((16 * wn + 2 * j + b1) ^ (sw << 1)) << 4) + inner;
  }
  int stage = 0, stage_last = 0;
  for (;;) {
    f32x4 acc[8][MJ];  // [n subtile][m subtile]: D[n][m], a lane holds n = 4 kq .. +3 for m = l16
#pragma unroll
    for (int a = 0; a < 8; ++a)
#pragma unroll
      for (int b = 0; b < MJ; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int steps = (cur.rows + kWgK - 1) / kWgK;
    for (int s = 0; s < steps; ++s) {
      // this step's copies have landed when at most the younger ones (kCopies per step and wave) are outstanding
      if (ahead >= S::kStages - 1) wait_vmcnt<(S::kStages - 2) * S::kCopies>();
      else if (ahead == 2) wait_vmcnt<S::kCopies>();
      else wait_vmcnt<0>();
      const int rem = cur.rows - s * kWgK;  // live rows of this step
      if (rem < kWgK) {
        char* pt = smem + stage * S::kStage + wave * 4 * S::kPRow;
#pragma unroll
        for (int q = 0; q < S::kPCopies; ++q) {
          const int r4 = S::kPRowsPerCopy * q + prow;
          if (4 * wave + r4 >= rem) *(uint4*)(pt + r4 * S::kPRow + pch * 16) = make_uint4(0, 0, 0, 0);
        }
      }
      __syncthreads();
      ahead += issue() ? 1 : 0;  // into the stage that was read one step ago
      lds_cptr pt = lds + stage * S::kStage;
      bf16x8 fm[MJ], fn[8];
#pragma unroll
      for (int j = 0; j < MJ; ++j) fm[j] = read_tr8_sw<S::kPRow>(pt + off_m[j]);
#pragma unroll
      for (int j = 0; j < 8; ++j) fn[j] = read_tr8_sw<512>(pt + off_n[j]);
#pragma unroll
      for (int ni = 0; ni < 8; ++ni)
#pragma unroll
        for (int mj = 0; mj < MJ; ++mj)
          acc[ni][mj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fn[ni], fm[mj], acc[ni][mj], 0, 0, 0);
      --ahead;
      stage_last = stage;
      stage = stage + 1 == S::kStages ? 0 : stage + 1;
    }
    // Epilogue through LDS: a lane holds 4 consecutive n of one row m, which stored directly are 8-byte
    // pieces in 32-byte runs (measured: 1.5 TB/s, twice the time of the MFMAs).  Each wave turns one 16-row
    // subtile at a time into rows of 256 contiguous bytes in its eighth of the stage that the last step
    // read (free until the next step's copies; a wave's LDS accesses stay in order) and stores 16 bytes per lane, four
    // whole rows per instruction.  The 16-byte chunk index is XORed with the row, which spreads both the 8-byte writes of 32 lanes (16 rows x 2 column
    // groups) and the 16-byte reads of 16 lanes (one row) over all 64 banks.
    __syncthreads();  // every wave has finished reading that stage
    {
      char* mine = smem + stage_last * S::kStage + wave * (S::kStage / 8);
      uint16_t* Gw = cur.G + (size_t)(wm * (MJ * 16)) * Ndim + wn * 128;
      const int rrow = lane >> 4, rcol = lane & 15;
      auto put = [&](int mj) {
        char* buf = mine + l16 * 256 + (kq & 1) * 8;
#pragma unroll
        for (int ni = 0; ni < 8; ++ni) {
          const f32x4 v = acc[ni][mj];
          *(uint2*)(buf + (((2 * ni + (kq >> 1)) ^ l16) << 4)) =
              make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
        }
      };
#pragma unroll
      for (int mj = 0; mj < MJ; ++mj) {
        put(mj);
        const char* buf = mine;
#pragma unroll
        for (int p4 = 0; p4 < 4; ++p4) {
          const int row = 4 * p4 + rrow;
          const uint4 v = *(const uint4*)(buf + row * 256 + ((rcol ^ row) << 4));
          nt_store16(v, (uint4*)(Gw + (size_t)(mj * 16 + row) * Ndim + rcol * 8));  // written once, read by nobody here
        }
      }
    }
    // No drain of the stores: the waits above stay sufficient with stores in flight.  Copies complete in issue
    // order among themselves, so while a step's copy is outstanding so are all younger copies, and the counter
    // exceeds their number whatever the stores do; stores only make a wait last longer.
    t_cur = next_live(t_cur + nwg, cur);
    if (t_cur >= total) break;
  }
  zero_empty();
}

// Any shape and either storage type of the operands that have one (the other operand is bf16): a tile of G per work-group,
// four waves of 64 x 64, or of 128 x 64 with 128 columns of the bf16 operand (launch_wgrad says which), 32 rows of the
// segment per step.  Both operands are staged through registers (the next step's loads are in flight during the current
// one's MFMAs) into double-buffered k-major LDS tiles and fetched with the transposing LDS read; the chunk swizzle is the
// one of the kernel above.
// fp32 values keep all their 24 bits: x = a + b + c with a, b, c the bf16 numbers that hold bits 0..7, 8..15 and
// 16..23 of the significand (cut, not rounded: each remainder is exact), so that three MFMAs sum the same exact
// products as fp32 multiplications would, in fp32: at 60, 500 and 3 000 rows 131, 368 and 1 766 of 2 to 4 million elements
// are not the rounded float64 sum (one thread per element with scalar products, which this replaces: 242, 655, 2 874).
// Bits below bf16's least subnormal, 2^-133, are lost: values under 2^-109 keep fewer than 24 bits (a single product is
// still the rounded one down to 2^-118).  Infinities: see behind the loop.
// The contraction is short and the output large: at T = 4096, d = 1024, h = 4096, 16 experts, fp32 storage (3 662
// kept rows) both launches write 268 MB, 54 us at the rate of a large copy, and multiply 3 x 61 GFLOP, 142 us at the
// rate of a large matrix product; they take 202 us.  Splitting a value was 12 vector operations beside two per MFMA's share
// of a 128 x 128 tile, more than the MFMAs' own cycles; with the remainders unguarded and the upper halves taken by one
// byte permutation per pair it is 5.5: 296 -> 268 us; the wide tile does it, and the LDS reads of the fp32 planes, for twice
// as many products: 202.  At most 80 KiB of LDS leave room for two work-groups per compute unit, so that one's stores run
// beside the other's MFMAs.
constexpr int kAnyThreads = 256;    // four waves, 2 along m x 2 along n

__device__ __forceinline__ int any_swz(int row) { return ((row & 3) | (((row >> 3) & 1) << 2)) << 1; }

// 8 fp32 values -> the three bf16 planes described above, 16 bytes each.  (An infinity leaves a NaN for its remainder: see
// behind the loop.)
__device__ __forceinline__ void split3(const u32x4& lo4, const u32x4& hi4, u32x4 (&out)[3]) {
  uint32_t x[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) x[i] = i < 4 ? lo4[i] : hi4[i - 4];
#pragma unroll
  for (int q = 0; q < 3; ++q) {
#pragma unroll
    for (int i = 0; i < 4; ++i) out[q][i] = __builtin_amdgcn_perm(x[2 * i + 1], x[2 * i], 0x07060302u);  // the upper halves
    if (q < 2) {
#pragma unroll
      for (int i = 0; i < 8; ++i)
        x[i] = __float_as_uint(__uint_as_float(x[i]) - __uint_as_float(x[i] & 0xFFFF0000u));
    }
  }
}

template <int NI, int MJ>
__device__ __forceinline__ bool acc_has_nan(const f32x4 (&acc)[NI][MJ]) {
  bool nan = false;
#pragma unroll
  for (int a = 0; a < NI; ++a)
#pragma unroll
    for (int b = 0; b < MJ; ++b)
#pragma unroll
      for (int v = 0; v < 4; v += 2) nan |= __builtin_isunordered(acc[a][b][v], acc[a][b][v + 1]);
  return nan;
}

// One operand's share of a step for this thread: SUB / 2 pieces of 8 consecutive columns of one row each; the operand's tile
// is 32 rows x 32 SUB columns (SUB 16-column subtiles per wave)
template <bool F32, int SUB>
struct AnyStage {
  static constexpr int kPlanes = F32 ? 3 : 1;
  static constexpr int kRow = 64 * SUB;              // bytes of an LDS row
  static constexpr int kPlane = kWgK * kRow;         // one bf16 plane
  static constexpr int kBytes = kPlanes * kPlane;
  static constexpr int kPieces = SUB / 2, kPerRow = 4 * SUB;
  u32x4 v[F32 ? 2 * kPieces : kPieces];

  // rows at or past `rows` re-read the last row here and become zeros in store()
  __device__ __forceinline__ void load(const char* base, size_t ld, int col0, int cols, int k0, int rows, int tid) {
#pragma unroll
    for (int i = 0; i < kPieces; ++i) {
      const int c = tid + i * kAnyThreads, row = min(k0 + c / kPerRow, rows - 1);
      const int col = min(col0 + (c % kPerRow) * 8, cols - 8);  // columns past the end repeat the last ones (not stored)
      const u32x4* p = (const u32x4*)(base + (size_t)row * ld + (size_t)col * (F32 ? 4 : 2));
      if (F32) { v[2 * i] = p[0]; v[2 * i + 1] = p[1]; }
      else v[i] = p[0];
    }
  }
  __device__ __forceinline__ void store(char* lds, int k0, int rows, int tid) {
    if (k0 + kWgK > rows) {
      const u32x4 z = {0, 0, 0, 0};
#pragma unroll
      for (int i = 0; i < kPieces; ++i)
        if (k0 + (tid + i * kAnyThreads) / kPerRow >= rows) {
          if (F32) v[2 * i] = v[2 * i + 1] = z;
          else v[i] = z;
        }
    }
#pragma unroll
    for (int i = 0; i < kPieces; ++i) {
      const int c = tid + i * kAnyThreads, row = c / kPerRow;
      char* dst = lds + row * kRow + (((c % kPerRow) ^ any_swz(row)) << 4);
      if (F32) {
        u32x4 part[3];
        split3(v[2 * i], v[2 * i + 1], part);
#pragma unroll
        for (int q = 0; q < 3; ++q) *(u32x4*)(dst + q * kPlane) = part[q];
      } else {
        *(u32x4*)dst = v[i];
      }
    }
  }
};

// MJ, NI: 16-wide subtiles of a wave along m and n (the tile is 32 MJ x 32 NI)
template <bool P_F32, bool Q_F32, int MJ, int NI>
__global__ __launch_bounds__(kAnyThreads, 2) void wgrad_any_kernel(const char* __restrict__ P, const char* __restrict__ Q,
                                                                  uint16_t* __restrict__ G,
                                                                  const int32_t* __restrict__ seg_off,
                                                                  const int32_t* __restrict__ buf_expert, int Mdim,
                                                                  int Ndim, int MT, int NT, int total) {
  using SP = AnyStage<P_F32, MJ>;
  using SQ = AnyStage<Q_F32, NI>;
  constexpr int kStageBytes = SP::kBytes + SQ::kBytes;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  // consecutive tiles of a segment share operand tiles: an XCD (work-groups with equal id mod 8) walks a contiguous run
  const int id = blockIdx.x, per = total >> 3, rest = total & 7, x = id & 7;
  const int lin = x * per + min(x, rest) + (id >> 3);
  const int mt = lin % MT, nt = (lin / MT) % NT, r = lin / (MT * NT);
  const int seg0 = seg_off[r], rows = seg_off[r + 1] - seg0;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int m0 = mt * 32 * MJ, n0 = nt * 32 * NI;
  const size_t ldP = (size_t)Mdim * (P_F32 ? 4 : 2), ldQ = (size_t)Ndim * (Q_F32 ? 4 : 2);
  const char* Ps = P + (size_t)seg0 * ldP;
  const char* Qs = Q + (size_t)seg0 * ldQ;

  const int wm = wave >> 1, wn = wave & 1;
  const int kq = lane >> 4, l16 = lane & 15;
  int off_m[MJ], off_n[NI];
  {
    const int row = 8 * kq + (l16 >> 2), b1 = (l16 & 3) >> 1, inner = (l16 & 1) * 8, sw = any_swz(row);
#pragma unroll
    for (int j = 0; j < MJ; ++j) off_m[j] = row * SP::kRow + (((2 * MJ * wm + 2 * j + b1) ^ sw) << 4) + inner;
#pragma unroll
    for (int j = 0; j < NI; ++j) off_n[j] = SP::kBytes + row * SQ::kRow + (((2 * NI * wn + 2 * j + b1) ^ sw) << 4) + inner;
  }
  f32x4 acc[NI][MJ];  // [n subtile][m subtile]
#pragma unroll
  for (int a = 0; a < NI; ++a)
#pragma unroll
    for (int b = 0; b < MJ; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};

  if (rows > 0) {
    SP sp;
    SQ sq;
    sp.load(Ps, ldP, m0, Mdim, 0, rows, tid);
    sq.load(Qs, ldQ, n0, Ndim, 0, rows, tid);
    int buf = 0;
    for (int k0 = 0; k0 < rows; k0 += kWgK) {
      char* st = smem + buf * kStageBytes;
      sp.store(st, k0, rows, tid);
      sq.store(st + SP::kBytes, k0, rows, tid);
      __syncthreads();  // (the other buffer's readers are past the previous step's barrier: one barrier per step)
      sp.load(Ps, ldP, m0, Mdim, k0 + kWgK, rows, tid);
      sq.load(Qs, ldQ, n0, Ndim, k0 + kWgK, rows, tid);
      lds_cptr pt = (lds_cptr)(uintptr_t)(uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)st;
      // (the operand with one plane stays in registers, the other's planes come one after the other)
      if constexpr (SP::kPlanes == 1) {
        bf16x8 fm[MJ];
#pragma unroll
        for (int j = 0; j < MJ; ++j) fm[j] = read_tr8_sw<SP::kRow>(pt + off_m[j]);
#pragma unroll
        for (int q = 0; q < SQ::kPlanes; ++q) {
          bf16x8 fn[NI];
#pragma unroll
          for (int j = 0; j < NI; ++j) fn[j] = read_tr8_sw<SQ::kRow>(pt + q * SQ::kPlane + off_n[j]);
#pragma unroll
          for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int mj = 0; mj < MJ; ++mj)
              acc[ni][mj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fn[ni], fm[mj], acc[ni][mj], 0, 0, 0);
        }
      } else {
        bf16x8 fn[NI];
#pragma unroll
        for (int j = 0; j < NI; ++j) fn[j] = read_tr8_sw<SQ::kRow>(pt + off_n[j]);
#pragma unroll
        for (int q = 0; q < SP::kPlanes; ++q) {
          bf16x8 fm[MJ];
#pragma unroll
          for (int j = 0; j < MJ; ++j) fm[j] = read_tr8_sw<SP::kRow>(pt + q * SP::kPlane + off_m[j]);
#pragma unroll
          for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int mj = 0; mj < MJ; ++mj)
              acc[ni][mj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fn[ni], fm[mj], acc[ni][mj], 0, 0, 0);
        }
      }
      buf ^= 1;
    }
  }
  // An infinity in the fp32 operand has NaNs for its lower planes, and one in the bf16 operand times an fp32 value of at
  // most 16 significant bits (1.0) meets a plane of zeros, where 0 * inf is a NaN and the product an infinity.  A wave whose
  // part of the tile holds a NaN therefore sums it again with the products themselves, row by row in fp32.  (The look at
  // the sums costs 2 % where a segment has 160 rows.)
  if ((P_F32 || Q_F32) && __builtin_expect(__any(acc_has_nan(acc)), 0)) {
    int lm = wm * 16 * MJ + l16, ln = wn * 16 * NI + kq * 4;
    asm volatile("" : "+v"(lm), "+v"(ln));  // (none of this belongs ahead of the loop)
    const int m = m0 + lm, n = n0 + ln;
    auto value = [](const char* row, bool f32, int c) {
      return f32 ? ((const float*)row)[c] : bf16_bits_to_f32(((const uint16_t*)row)[c]);
    };
#pragma unroll
    for (int a = 0; a < NI; ++a)
#pragma unroll
      for (int b = 0; b < MJ; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma nounroll
    for (int k = 0; k < rows; ++k) {
      float p[MJ];
#pragma unroll
      for (int mj = 0; mj < MJ; ++mj) p[mj] = value(Ps + k * ldP, P_F32, min(m + mj * 16, Mdim - 1));
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float q = value(Qs + k * ldQ, Q_F32, min(n + ni * 16 + v, Ndim - 1));
#pragma unroll
          for (int mj = 0; mj < MJ; ++mj) acc[ni][mj][v] = fmaf(p[mj], q, acc[ni][mj][v]);
        }
    }
  }
  // Through LDS, so that a row of the tile leaves as 256 or 512 contiguous bytes (chunk index XORed with the row)
  constexpr int kGRow = 64 * NI;
  __syncthreads();
#pragma unroll
  for (int mj = 0; mj < MJ; ++mj) {
    char* row = smem + (wm * 16 * MJ + mj * 16 + l16) * kGRow + (kq & 1) * 8;
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
      const f32x4 v = acc[ni][mj];
      *(uint2*)(row + (((2 * NI * wn + 2 * ni + (kq >> 1)) ^ l16) << 4)) =
          make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
    }
  }
  __syncthreads();
  uint16_t* Gt = G + ((size_t)buf_expert[r] * Mdim + m0) * Ndim + n0;
  constexpr int kRowLanes = 4 * NI, kRows = kAnyThreads / kRowLanes;  // lanes per row, rows at a time
  const int rrow = tid / kRowLanes, rcol = tid % kRowLanes;
  if (n0 + rcol * 8 < Ndim) {
#pragma unroll
    for (int i = 0; i < 32 * MJ / kRows; ++i) {
      const int row = rrow + kRows * i;
      const uint4 v = *(const uint4*)(smem + row * kGRow + ((rcol ^ (row & 15)) << 4));
      if (m0 + row < Mdim) nt_store16(v, (uint4*)(Gt + (size_t)row * Ndim + rcol * 8));
    }
  }
}

template <bool P_F32, bool Q_F32, int MJ, int NI>
int launch_wgrad_any(const void* P, const void* Q, void* G, const int32_t* seg_off, const int32_t* buf_expert, int E,
                     int Mdim, int Ndim, hipStream_t st) {
  const int MT = ceil_div(Mdim, 32 * MJ), NT = ceil_div(Ndim, 32 * NI);
  const long long tiles = (long long)E * MT * NT;
  if (tiles > 0x7FFFFFFFLL) return LOCMOE_ERR_SHAPE;
  auto any = wgrad_any_kernel<P_F32, Q_F32, MJ, NI>;
  constexpr int stages = 2 * (AnyStage<P_F32, MJ>::kBytes + AnyStage<Q_F32, NI>::kBytes);
  constexpr int smem = std::max(stages, 32 * MJ * 64 * NI);  // 32 to 80 KiB (the tile of G goes through it too)
  static std::atomic<uint64_t> any_lds;
  if (!allow_lds((const void*)any, smem, any_lds)) return LOCMOE_ERR_HIP;
  hipLaunchKernelGGL(any, dim3((unsigned)tiles), dim3(kAnyThreads), smem, st, (const char*)P, (const char*)Q,
                     (uint16_t*)G, seg_off, buf_expert, Mdim, Ndim, MT, NT, (int)tiles);
  return launch_status();
}

template <bool P_F32, bool Q_F32>
int launch_wgrad(const void* P, const void* Q, void* G, const int32_t* seg_off, const int32_t* buf_expert, int E,
                 int rows_max, int Mdim, int Ndim, hipStream_t st) {
  if (!P_F32 && !Q_F32 && Mdim % kWgTile == 0 && Ndim % kWgTile == 0) {
    const long long total = (long long)E * (Mdim / kWgTile) * (Ndim / kWgTile);
    const long long span = (long long)rows_max * (Mdim > Ndim ? Mdim : Ndim) * 2;  // byte offsets inside a segment
    if (total <= 0x3FFFFFFFLL && span < 0x7FFFFFFFLL) {
      using S = WgShape;
      auto kern = wgrad_dma_kernel;
      static std::atomic<uint64_t> lds_allowed;
      if (!allow_lds((const void*)kern, S::kSmem, lds_allowed)) return LOCMOE_ERR_HIP;
      const long long tiles = (long long)E * (Mdim / S::kTM) * (Ndim / kWgTile);
      const long long groups = std::min<long long>((cu_count() / 8) * 8, (tiles + 7) / 8 * 8);
      hipLaunchKernelGGL(kern, dim3((unsigned)groups), dim3(kWgThreads), S::kSmem, st, (const uint16_t*)P,
                         (const uint16_t*)Q, (uint16_t*)G, seg_off, buf_expert, Mdim, Ndim, E);
      return launch_status();
    }
  }
  // With fp32 storage 256 columns of the bf16 operand per tile where that leaves three tiles per compute unit: the fp32
  // operand is split and read from LDS half as often.  Both GEMMs, us, 128 x 128 tiles / 256 wide: E = 16, d = 1024, h = 4096,
  // 229 rows 268 / 202;  E = 4, d = 2048, h = 4096, 714 rows (4 tiles per unit) 295 / 230;  E = 20, d = 640, h = 1712, 60 rows
  // (2.7) 38.1 / 39.2;  E = 6, d = 768, h = 1536, 298 rows (0.8) 39 / 45.  With fewer than 32 tiles per expert also where a segment
  // can be long: E = 48, d = 384, h = 1536 (18), up to 30 rows, 15 in the mean 34.3 / 35.2, with four tokens of five on four experts
  // 33.6 / 34.7;  up to 342 rows 97 / 81 and 70 / 74.  Two bf16 operands: E = 24, d = 768, h = 3072, 455
  // rows 150 / 152;  E = 48, d = 384, h = 1536, 65 rows 30 / 35.
  constexpr int MJ = Q_F32 ? 8 : 4, NI = P_F32 ? 8 : 4;
  if constexpr (MJ != NI) {
    const long long per_expert = (long long)ceil_div(Mdim, 32 * MJ) * ceil_div(Ndim, 32 * NI);
    if (E * per_expert >= 3 * cu_count() && (per_expert >= 32 || rows_max >= 128))
      return launch_wgrad_any<P_F32, Q_F32, MJ, NI>(P, Q, G, seg_off, buf_expert, E, Mdim, Ndim, st);
  }
  return launch_wgrad_any<P_F32, Q_F32, 4, 4>(P, Q, G, seg_off, buf_expert, E, Mdim, Ndim, st);
}

}  // namespace
}  // namespace locmoe

extern "C" int locmoe_expert_ffn_wgrad(const locmoe_desc* desc, const void* send, const void* H, const void* dout,
                                       const void* dZ, const int32_t* seg_off, const int32_t* buf_expert,
                                       void* dW_in, void* dW_out, void* stream) {
  using namespace locmoe;
  if (!desc || !send || !H || !dout || !dZ || !seg_off || !buf_expert || !dW_in || !dW_out) return LOCMOE_ERR_NULL;
  int st = check_desc(desc);
  if (st != LOCMOE_OK) return st;
  hipStream_t s = as_stream(stream);
  const int E = desc->E, d = desc->d, h = desc->h;
  const int rows_max = desc->C < desc->T ? desc->C : desc->T;
  if (desc->x_dtype == LOCMOE_F32) {
    st = launch_wgrad<false, true>(dZ, send, dW_in, seg_off, buf_expert, E, rows_max, h, d, s);   // dW_in[e] = dZ^T . send
    if (st != LOCMOE_OK) return st;
    return launch_wgrad<true, false>(dout, H, dW_out, seg_off, buf_expert, E, rows_max, d, h, s);  // dW_out[e] = dout^T . H
  }
  st = launch_wgrad<false, false>(dZ, send, dW_in, seg_off, buf_expert, E, rows_max, h, d, s);
  if (st != LOCMOE_OK) return st;
  return launch_wgrad<false, false>(dout, H, dW_out, seg_off, buf_expert, E, rows_max, d, h, s);
}
