// The routers the paper compares LocMoE with (Section 2, Section 4), as far as they differ from the LocMoE path:
//   - the gate as a dense layer with a learned weight (Section 3.2.1; the switch router's gate, which GrAP
//     replaces): g[m,i] = omega_i . x_m, a [T,d] x [d,E] contraction.  Top-1 selection, the score and the
//     auxiliary loss of Eq. 5 are locmoe_route's, unchanged.
//   - hash routing: the expert is a fixed, parameter-free function of the token's key; no token feature is read.
// Dispatch, expert FFN and combine are the same kernels for all three routers.
#include <type_traits>

#include "common.h"

namespace locmoe {
namespace {

// ---------------------------------------------------------------------------------------------
// Dense gate, bf16 storage, d a multiple of 64: 64 or 128 tokens x up to 128 experts per work-group, waves of
// 32 tokens each, v_mfma_f32_32x32x16_bf16 with fp32 accumulation.  E is small, so the kernel is bound by the
// one pass over x (T d 2 bytes): 2 T d E flops are 64 flops per byte at E = 64, far below the machine's ridge.
// The weight [E,d] is re-read by every work-group from L2.  Operands go global -> registers -> LDS (16-byte
// chunks, chunk index XORed with row/2 so that a fragment read of 32 rows touches every bank equally); the next
// two k-steps' loads are in flight while the current one is multiplied.
// ---------------------------------------------------------------------------------------------
constexpr int kDgThreads = 256;
constexpr int kDgTokens = 128;                       // tokens per work-group
constexpr int kDgBK = 64;                            // k-step
constexpr int kDgRowBytes = kDgBK * 2;               // 128 B per LDS row
constexpr int kDgTile = 128 * kDgRowBytes;           // 16 KiB: 128 rows of one operand
constexpr int kDgSmem = 4 * kDgTile;                 // x and W, double buffered

__device__ __forceinline__ int dg_swz(int row, int chunk) { return (chunk ^ ((row >> 1) & 7)) << 4; }

// NT: 32-expert tiles per pass, experts [e0, e0 + 32 NT).  TOK: tokens per work-group, 32 per wave; 64 with up to 64 experts
// where the launch says so.
template <int NT, int TOK>
__global__ __launch_bounds__(2 * TOK) void gate_dense_mfma_kernel(const uint16_t* __restrict__ x,
                                                                     const uint16_t* __restrict__ Wg,
                                                                     float* __restrict__ g, int T, int d, int E) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  constexpr int kThreads = 2 * TOK, NW = 8 * 32 * NT / kThreads, kXTile = TOK * kDgRowBytes, kWTile = NT * 32 * kDgRowBytes;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int m0 = blockIdx.x * TOK;
  const int e0 = blockIdx.y * 128;
  // global -> LDS assignment: four x chunks and NW W chunks of 16 bytes per thread and k-step
  const uint16_t* gx[4];
  const uint16_t* gw[NW];
  int lds_x[4], lds_w[NW];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int c = tid + i * kThreads, row = c >> 3, kc = c & 7;
    gx[i] = x + (size_t)min(m0 + row, T - 1) * d + kc * 8;  // rows past T re-read the last token (never stored)
    lds_x[i] = row * kDgRowBytes + dg_swz(row, kc);
  }
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    const int c = tid + i * kThreads, row = c >> 3, kc = c & 7;
    gw[i] = Wg + (size_t)min(e0 + row, E - 1) * d + kc * 8;  // rows past E re-read the last expert (never stored)
    lds_w[i] = row * kDgRowBytes + dg_swz(row, kc);
  }
  const int frow = lane & 31, khalf = lane >> 5;
  const int xrow = wave * 32 + frow;

  f32x16 acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = (f32x16){0};

  // Two register sets hold the two k-steps after the one in LDS: with a work-group per compute unit (T = 32 768) the
  // loads in flight are what bounds this stream of tokens.
  // T = 32 768, d = 2048, E = 32 (134 MB, 1 GB of tokens in turn): 33 us, 36 with one set; the same tokens again and again
  // (they stay in the last-level cache) 20.7 and 22.5.  With more than 96 experts the loads past the last k-step are left
  // out: T = 4 096, d = 2048, E = 128, the same tokens: 24.2 us, 28.7 with them, 25.7 with one set of registers.  Below
  // that the branch costs more than they do: T = 65 536, d = 4096, E = 64: 132 us, 122 without it.
  u32x4 rx[2][4], rw[2][NW];
  const int KT = d / kDgBK;
  auto load = [&](int set, int kt) {
    const int ko = min(kt, KT - 1) * kDgBK;  // (steps after the last re-read the last: never consumed)
#pragma unroll
    for (int i = 0; i < 4; ++i) rx[set][i] = *(const u32x4*)(gx[i] + ko);
#pragma unroll
    for (int i = 0; i < NW; ++i) rw[set][i] = *(const u32x4*)(gw[i] + ko);
  };
  auto store = [&](int set) {
#pragma unroll
    for (int i = 0; i < 4; ++i) *(u32x4*)(smem + set * kXTile + lds_x[i]) = rx[set][i];
#pragma unroll
    for (int i = 0; i < NW; ++i) *(u32x4*)(smem + 2 * kXTile + set * kWTile + lds_w[i]) = rw[set][i];
  };
  auto step = [&](auto par_, int kt) {  // k-step kt, which is in LDS buffer PAR
    constexpr int PAR = decltype(par_)::value;
    const char* sx = smem + PAR * kXTile;
    const char* sw = smem + 2 * kXTile + PAR * kWTile;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const int kc = ks * 2 + khalf;
      const bf16x8 fx = *(const bf16x8*)(sx + xrow * kDgRowBytes + dg_swz(xrow, kc));
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int wrow = t * 32 + frow;
        const bf16x8 fw = *(const bf16x8*)(sw + wrow * kDgRowBytes + dg_swz(wrow, kc));
        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw, fx, acc[t], 0, 0, 0);  // D[expert][token]
      }
    }
    store(1 - PAR);
    if (NT < 4 || kt + 3 < KT) load(1 - PAR, kt + 3);
    __syncthreads();
  };
  load(0, 0);
  load(1, 1);
  store(0);
  load(0, 2);
  __syncthreads();
  int kt = 0;
  for (; kt + 1 < KT; kt += 2) {
    step(std::integral_constant<int, 0>{}, kt);
    step(std::integral_constant<int, 1>{}, kt + 1);
  }
  if (kt < KT) step(std::integral_constant<int, 0>{}, kt);
  // a lane holds experts e0 + 32 t + 8 vq + 4 khalf .. +3 of token m0 + 32 wave + frow
  const int m = m0 + xrow;
  if (m < T) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int vq = 0; vq < 4; ++vq) {
        const int i0 = e0 + t * 32 + vq * 8 + khalf * 4;
        float* dst = g + (size_t)m * E + i0;
        if (i0 + 3 < E && (E & 3) == 0) {
          *(float4*)dst = make_float4(acc[t][vq * 4 + 0], acc[t][vq * 4 + 1], acc[t][vq * 4 + 2], acc[t][vq * 4 + 3]);
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (i0 + q < E) dst[q] = acc[t][vq * 4 + q];
        }
      }
  }
}

// Dense gate, fp32 storage, d a multiple of 32: the same tile and staging with 32 features (128 bytes) per step and
// v_mfma_f32_32x32x2_f32.  Bound by the pass over x up to some 32 experts, above by the fp32 matrix rate (157 TFLOP/s).
// The sums are kept short: two MFMAs from zero, eight such sums per step in fp32, the steps in double, so that the error
// against float64 is no larger than with one wave per token (relative 2-norm 6.8e-8 at any d, which is the last rounding; one wave per token 8e-8 at
// d = 384, 1.2e-7 at 2 048, 1.7e-7 at 5 120).  us, one wave per token / this: T = 32 768, d = 2048, E = 32 1 428 / 90;
// T = 60 000, d = 1280, E = 40 2 096 / 158;  T = 16 000, d = 5120, E = 128 6 922 / 706;  T = 4 193, d = 384, E = 64 57 / 33.
template <int NT>
__global__ __launch_bounds__(kDgThreads) void gate_dense_f32_kernel(const float* __restrict__ x, const float* __restrict__ Wg,
                                                                    float* __restrict__ g, int T, int d, int E) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  constexpr int kBK = kDgRowBytes / 4;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int m0 = blockIdx.x * kDgTokens;
  const int e0 = blockIdx.y * 128;
  const float* gx[4];
  const float* gw[NT];
  int lds_x[4], lds_w[NT];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int c = tid + i * kDgThreads, row = c >> 3, kc = c & 7;
    gx[i] = x + (size_t)min(m0 + row, T - 1) * d + kc * 4;  // rows past T re-read the last token (never stored)
    lds_x[i] = row * kDgRowBytes + dg_swz(row, kc);
  }
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    const int c = tid + i * kDgThreads, row = c >> 3, kc = c & 7;
    gw[i] = Wg + (size_t)min(e0 + row, E - 1) * d + kc * 4;  // rows past E re-read the last expert (never stored)
    lds_w[i] = row * kDgRowBytes + dg_swz(row, kc);
  }
  const int frow = lane & 31, khalf = lane >> 5;
  const int xrow = wave * 32 + frow;
  double sum[NT][16];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int i = 0; i < 16; ++i) sum[t][i] = 0.0;

  u32x4 rx[4], rw[NT];  // the k-step after the one in LDS
  const int KT = d / kBK;
  auto load = [&](int kt) {
    const int ko = min(kt, KT - 1) * kBK;  // (a step after the last re-reads the last: never consumed)
#pragma unroll
    for (int i = 0; i < 4; ++i) rx[i] = *(const u32x4*)(gx[i] + ko);
#pragma unroll
    for (int i = 0; i < NT; ++i) rw[i] = *(const u32x4*)(gw[i] + ko);
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int i = 0; i < 4; ++i) *(u32x4*)(smem + buf * kDgTile + lds_x[i]) = rx[i];
#pragma unroll
    for (int i = 0; i < NT; ++i) *(u32x4*)(smem + (2 + buf) * kDgTile + lds_w[i]) = rw[i];
  };
  load(0);
  store(0);
  load(1);
  __syncthreads();
  for (int kt = 0; kt < KT; ++kt) {
    const char* sx = smem + (kt & 1) * kDgTile;
    const char* sw = smem + (2 + (kt & 1)) * kDgTile;
    f32x16 part[NT];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {  // (a lane's four features go one by one: any order does that both operands have)
      const int kc = ks * 2 + khalf;
      const f32x4 fx = *(const f32x4*)(sx + xrow * kDgRowBytes + dg_swz(xrow, kc));
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int wrow = t * 32 + frow;
        const f32x4 fw = *(const f32x4*)(sw + wrow * kDgRowBytes + dg_swz(wrow, kc));
        f32x16 a = __builtin_amdgcn_mfma_f32_32x32x2f32(fw[0], fx[0], (f32x16){0}, 0, 0, 0);  // D[expert][token]
        f32x16 b = __builtin_amdgcn_mfma_f32_32x32x2f32(fw[2], fx[2], (f32x16){0}, 0, 0, 0);
        a = __builtin_amdgcn_mfma_f32_32x32x2f32(fw[1], fx[1], a, 0, 0, 0);
        b = __builtin_amdgcn_mfma_f32_32x32x2f32(fw[3], fx[3], b, 0, 0, 0);
        part[t] = ks ? part[t] + (a + b) : a + b;
      }
    }
    store((kt + 1) & 1);
    load(kt + 2);
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) sum[t][i] += (double)part[t][i];
    __syncthreads();
  }
  const int m = m0 + xrow;
  if (m < T) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int vq = 0; vq < 4; ++vq) {
        const int i0 = e0 + t * 32 + vq * 8 + khalf * 4;
        float* dst = g + (size_t)m * E + i0;
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (i0 + q < E) dst[q] = (float)sum[t][vq * 4 + q];
      }
  }
}

// Any shape and either storage type: one wave per token, lanes stride over the features, the wave's sum by a
// fixed butterfly.  Correct for every descriptor; used for bf16 rows that are no multiple of 64, fp32 rows that are no multiple
// of 32, and few experts and tokens in fp32 storage.
template <bool BF16>
__global__ __launch_bounds__(256) void gate_dense_generic_kernel(const void* __restrict__ x,
                                                                 const void* __restrict__ Wg,
                                                                 float* __restrict__ g, int T, int d, int E) {
  const int m = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (m >= T) return;
  for (int i = 0; i < E; ++i) {
    float s = 0.f;
    for (int j = lane; j < d; j += kWave) {
      float a, b;
      if (BF16) {
        a = bf16_bits_to_f32(((const uint16_t*)x)[(size_t)m * d + j]);
        b = bf16_bits_to_f32(((const uint16_t*)Wg)[(size_t)i * d + j]);
      } else {
        a = ((const float*)x)[(size_t)m * d + j];
        b = ((const float*)Wg)[(size_t)i * d + j];
      }
      s = fmaf(a, b, s);
    }
    s = group_sum<kWave>(s);
    if (lane == 0) g[(size_t)m * E + i] = s;
  }
}

// ---------------------------------------------------------------------------------------------
// Hash routing.  The 32-bit finalizer of MurmurHash3 (a published bijective mixer of 32-bit integers):
// xor-shift 16, times 0x85EBCA6B, xor-shift 13, times 0xC2B2AE35, xor-shift 16.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t mix32(uint32_t v) {
  v ^= v >> 16;
  v *= 0x85EBCA6Bu;
  v ^= v >> 13;
  v *= 0xC2B2AE35u;
  v ^= v >> 16;
  return v;
}

__global__ void zero_i32_kernel(int32_t* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

constexpr int kHashThreads = 256, kHashPerThread = 8, kHashOneTokens = 2048;

// eid, w and the per-expert counts.  Counts: LDS histogram per block, one integer atomic per non-empty cell
// into cnt (integer sums: the result does not depend on the order).  ONE: a single block of more threads takes all tokens
// and writes its counts, which need not be cleared before (one launch: up to 2 048 tokens).
template <bool ONE>
__global__ __launch_bounds__(ONE ? 1024 : kHashThreads) void route_hash_kernel(const int32_t* __restrict__ key, uint32_t offset,
                                                                  int32_t* __restrict__ eid, float* __restrict__ w,
                                                                  int32_t* __restrict__ cnt, int T, int E) {
  extern __shared__ int32_t hist[];
  constexpr int kThreads = ONE ? 1024 : kHashThreads, kPer = ONE ? kHashOneTokens / 1024 : kHashPerThread;
  for (int i = threadIdx.x; i < E; i += kThreads) hist[i] = 0;
  __syncthreads();
  const int base = blockIdx.x * kThreads * kPer;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int m = base + k * kThreads + threadIdx.x;
    if (m < T) {
      const uint32_t kv = key ? (uint32_t)key[m] : (uint32_t)m;
      const int e = (int)(mix32(kv + offset) % (uint32_t)E);
      eid[m] = e;
      w[m] = 1.0f;
      atomicAdd(&hist[e], 1);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < E; i += kThreads)
    if (ONE) cnt[i] = hist[i];
    else if (hist[i]) atomicAdd(&cnt[i], hist[i]);
}

}  // namespace
}  // namespace locmoe

extern "C" int locmoe_gate_dense(const locmoe_desc* desc, const void* x, const void* Wg, float* g, void* stream) {
  using namespace locmoe;
  if (!desc || !x || !Wg || !g) return LOCMOE_ERR_NULL;
  const int st = check_desc(desc);
  if (st != LOCMOE_OK) return st;
  hipStream_t s = as_stream(stream);
  const int T = desc->T, d = desc->d, E = desc->E;
  if (desc->x_dtype == LOCMOE_BF16 && d % kDgBK == 0) {
    const int passes = ceil_div(E, 128);
    const int nt = passes > 1 ? 4 : ceil_div(E, 32);  // 32-expert tiles per pass
#define LOCMOE_DG(N, TOK)                                                                                        \
  {                                                                                                              \
    constexpr int lds = 2 * (TOK + 32 * N) * kDgRowBytes;                                                        \
    static std::atomic<uint64_t> lds_allowed;                                                                    \
    auto kern = gate_dense_mfma_kernel<N, TOK>;                                                                  \
    if (!allow_lds((const void*)kern, lds, lds_allowed)) return LOCMOE_ERR_HIP;                                  \
    hipLaunchKernelGGL(kern, dim3(ceil_div(T, TOK), passes), dim3(2 * TOK), lds, s, (const uint16_t*)x,          \
                       (const uint16_t*)Wg, g, T, d, E);                                                         \
  }
    // 64 tokens per work-group, which read the weight twice as often, where they take half a turn less of the compute units
    // (up to two turns of 128), and with up to 32 experts where rows are multiples of 4 KiB, which meet in the same channels.
    // In the mean over d = 384 .. 5 120, 128 tokens' time over 64 tokens' (8 to 32 experts; 48 and 64): 16 384 tokens (half a
    // turn of 128) 1.11; 1.21, 24 000 (0.7) 0.99; 0.94, 32 768 (1) 1.02; 0.96, 40 000 (1.2) 1.12; 1.10, 57 000 (1.7) 0.98;
    // 0.91, 65 536 (2) 1.00; 0.93, 80 000 (2.4) 1.04; 0.95.  d = 4 096 with up to 32 experts 1.10 at 32 768 and 65 536 tokens,
    // d = 5 120 0.98 and 0.98.
    const int cus = cu_count(), groups = ceil_div(T, 128);
    const bool few = (groups <= 2 * cus && ceil_div(2 * groups, cus) % 2 == 1) || (nt == 1 && d % 2048 == 0);
    if (nt == 1 && few) LOCMOE_DG(1, 64)
    else if (nt == 1) LOCMOE_DG(1, 128)
    else if (nt == 2 && few) LOCMOE_DG(2, 64)
    else if (nt == 2) LOCMOE_DG(2, 128)
    else if (nt == 3) LOCMOE_DG(3, 128)
    else LOCMOE_DG(4, 128)
#undef LOCMOE_DG
    return launch_status();
  }
  // A tile's step takes about 1.3 us per 32 experts however few its tokens are, one wave per token as much for some 22
  // experts' 32 features, up to 8 192 tokens at a time.  us, one wave per token / tiles: T = 300, d = 2048, E = 8 29 / 80;
  // T = 574, d = 768, E = 12 18 / 32;  T = 9 000, d = 128, E = 4 5.7 / 7.5;  T = 60 000, E = 4 21 / 12;  T = 200, d = 5120,
  // E = 128 1 242 / 696.
  if (desc->x_dtype == LOCMOE_F32 && d % (kDgRowBytes / 4) == 0 && (E >= 24 || (long long)T * E >= 192000)) {
    const int passes = ceil_div(E, 128);
    const int nt = passes > 1 ? 4 : ceil_div(E, 32);
    const dim3 grid(ceil_div(T, kDgTokens), passes);
#define LOCMOE_DG(N)                                                                                                   \
  {                                                                                                                    \
    static std::atomic<uint64_t> lds_allowed;                                                                          \
    auto kern = gate_dense_f32_kernel<N>;                                                                              \
    if (!allow_lds((const void*)kern, kDgSmem, lds_allowed)) return LOCMOE_ERR_HIP;                                    \
    hipLaunchKernelGGL(kern, grid, dim3(kDgThreads), kDgSmem, s, (const float*)x, (const float*)Wg, g, T, d, E);       \
  }
    if (nt == 1) LOCMOE_DG(1) else if (nt == 2) LOCMOE_DG(2) else if (nt == 3) LOCMOE_DG(3) else LOCMOE_DG(4)
#undef LOCMOE_DG
    return launch_status();
  }
  const dim3 grid(ceil_div(T, 4));
  if (desc->x_dtype == LOCMOE_BF16)
    hipLaunchKernelGGL(gate_dense_generic_kernel<true>, grid, dim3(256), 0, s, x, Wg, g, T, d, E);
  else
    hipLaunchKernelGGL(gate_dense_generic_kernel<false>, grid, dim3(256), 0, s, x, Wg, g, T, d, E);
  return launch_status();
}

extern "C" int locmoe_route_hash(const locmoe_desc* desc, const int32_t* key, uint32_t seed, int32_t* eid, float* w,
                                 int32_t* cnt, void* stream) {
  using namespace locmoe;
  if (!desc || !eid || !w || !cnt) return LOCMOE_ERR_NULL;
  const int st = check_desc(desc);
  if (st != LOCMOE_OK) return st;
  hipStream_t s = as_stream(stream);
  const int T = desc->T, E = desc->E;
  if (T <= kHashOneTokens) {
    hipLaunchKernelGGL(route_hash_kernel<true>, dim3(1), dim3(1024), (size_t)E * 4, s, key, seed * 0x9E3779B9u, eid, w, cnt,
                       T, E);
    return launch_status();
  }
  hipLaunchKernelGGL(zero_i32_kernel, dim3(ceil_div(E, 256)), dim3(256), 0, s, cnt, E);
  int rc = launch_status();
  if (rc != LOCMOE_OK) return rc;
  hipLaunchKernelGGL(route_hash_kernel<false>, dim3(ceil_div(T, kHashThreads * kHashPerThread)), dim3(kHashThreads),
                     (size_t)E * 4, s, key, seed * 0x9E3779B9u, eid, w, cnt, T, E);
  return launch_status();
}
