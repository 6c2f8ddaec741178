// Top-1 routing (Eq. 2, Eq. 3) and the forward values of the auxiliary loss (Eq. 5) and the
// locality loss (Eq. 6).  One group of S lanes owns a token; reductions over the expert axis
// run on DPP / cross-lane permutes.  Every sum over tokens is formed from per-block partials in
// a fixed order (integer LDS atomics only, no floating-point atomics), so results are
// deterministic.
#include <math.h>

#include "common.h"

namespace locmoe {
namespace {

constexpr int kRouteThreads = 512;
constexpr int kTokPerGroup = 4;  // tokens a group loads before it starts reducing

// all-reduce (max value, lowest index) over aligned groups of S lanes
template <int S>
__device__ __forceinline__ void group_argmax(float& v, int& i) {
#define LOCMOE_STEP(OV, OI)                                \
  {                                                        \
    const float ov = (OV);                                 \
    const int oi = (OI);                                   \
    const bool take = ov > v || (ov == v && oi < i);       \
    v = take ? ov : v;                                     \
    i = take ? oi : i;                                     \
  }
  if (S >= 2) LOCMOE_STEP(dpp_f32<kDppXor1>(v), dpp_i32<kDppXor1>(i))
  if (S >= 4) LOCMOE_STEP(dpp_f32<kDppXor2>(v), dpp_i32<kDppXor2>(i))
  if (S >= 8) LOCMOE_STEP(dpp_f32<kDppHalfMirror>(v), dpp_i32<kDppHalfMirror>(i))
  if (S >= 16) LOCMOE_STEP(dpp_f32<kDppMirror>(v), dpp_i32<kDppMirror>(i))
  if (S >= 32) LOCMOE_STEP(__shfl_xor(v, 16), __shfl_xor(i, 16))
  if (S >= 64) LOCMOE_STEP(__shfl_xor(v, 32), __shfl_xor(i, 32))
#undef LOCMOE_STEP
}

struct RouteWs {
  int2* cell;      // [blocks][E]: count, bits of the probability sum
  int32_t* home;   // [blocks][N]
  int32_t* local;  // [blocks]
};

__host__ __device__ inline RouteWs route_ws(void* ws, int E, int N) {
  RouteWs r;
  char* p = (char*)ws;
  r.cell = (int2*)p;     p += (size_t)kRouteMaxBlocks * E * 8;
  r.home = (int32_t*)p;  p += (size_t)kRouteMaxBlocks * N * 4;
  r.local = (int32_t*)p;
  return r;
}

// Tokens tok0 .. tok1 - 1 by a work-group of THREADS: eid and w to memory; counts per expert (hist), per home node (hhist) and
// of tokens that stay on their node (local), and each group's probability sums (pacc [THREADS / S][E]) to LDS.  The LDS
// words are complete behind the caller's next barrier.
template <int S, int EPL, int THREADS>
__device__ __forceinline__ void route_tokens(const float* __restrict__ g, const float* __restrict__ eps,
                                             const int32_t* __restrict__ home, const int32_t* __restrict__ e2n,
                                             int32_t* __restrict__ eid, float* __restrict__ w, int32_t* hist,
                                             int32_t* hhist, int32_t* local, float* pacc, int tok0, int tok1, int E,
                                             int N, int relu) {
  constexpr int G = THREADS / S;  // groups (tokens in flight) per block
  const int grp = threadIdx.x / S, j = threadIdx.x % S;
  const int per_node = E / N;  // used only when e2n is NULL (then E % N == 0)
  float epsv[EPL];
#pragma unroll
  for (int k = 0; k < EPL; ++k) {
    const int i = j + k * S;
    epsv[k] = (eps && i < E) ? eps[i] : 0.f;
  }
  float acc[EPL];
#pragma unroll
  for (int k = 0; k < EPL; ++k) acc[k] = 0.f;

  // the loads of the next batch of tokens are issued before the current batch is reduced
  // (the tokens' home nodes come with the batch: fetched where they are used, behind the arg-max, each was a
  // memory round trip of its own on the critical path)
  float v[kTokPerGroup][EPL], nxt[kTokPerGroup][EPL];
  int hv[kTokPerGroup], hnxt[kTokPerGroup];
  auto load_batch = [&](float (&dst)[kTokPerGroup][EPL], int (&hdst)[kTokPerGroup], int base) {
#pragma unroll
    for (int t = 0; t < kTokPerGroup; ++t) {
      const int m = base + t * G + grp;
#pragma unroll
      for (int k = 0; k < EPL; ++k) {
        const int i = j + k * S;
        dst[t][k] = (m < tok1 && i < E) ? g[(size_t)m * E + i] : -INFINITY;
      }
      hdst[t] = (home && j == 0 && m < tok1) ? home[m] : 0;
    }
  };
  load_batch(nxt, hnxt, tok0);
  for (int base = tok0; base < tok1; base += G * kTokPerGroup) {
#pragma unroll
    for (int t = 0; t < kTokPerGroup; ++t) {
#pragma unroll
      for (int k = 0; k < EPL; ++k) v[t][k] = nxt[t][k];
      hv[t] = hnxt[t];
    }
    load_batch(nxt, hnxt, base + G * kTokPerGroup);
#pragma unroll
    for (int t = 0; t < kTokPerGroup; ++t) {
      const int m = base + t * G + grp;
      float best = -INFINITY;
      int bi = 0x7FFFFFFF;
#pragma unroll
      for (int k = 0; k < EPL; ++k) {
        const int i = j + k * S;
        float x = v[t][k] + epsv[k];           // G = g + eps, float32
        if (relu) x = fmaxf(x, 0.f);           // ReLU as printed below Eq. 3
        x = i < E ? x : -INFINITY;
        v[t][k] = x;
        if (x > best) { best = x; bi = i; }    // strict: lowest index wins ties
      }
      group_argmax<S>(best, bi);
      float z[EPL], zs = 0.f;
#pragma unroll
      for (int k = 0; k < EPL; ++k) {
        z[k] = (j + k * S) < E ? expf(v[t][k] - best) : 0.f;
        zs += z[k];
      }
      zs = group_sum<S>(zs);
      const float inv = 1.0f / zs;
      if (m < tok1) {
#pragma unroll
        for (int k = 0; k < EPL; ++k) acc[k] += z[k] * inv;
        if (j == 0) {
          eid[m] = bi;
          w[m] = inv;  // exp(0) / sum
          atomicAdd(&hist[bi], 1);
          if (home) {
            const int hn = hv[t];
            atomicAdd(&hhist[hn], 1);
            const int node = e2n ? e2n[bi] : bi / per_node;
            if (node == hn) atomicAdd(local, 1);
          }
        }
      }
    }
  }
#pragma unroll
  for (int k = 0; k < EPL; ++k) {
    const int i = j + k * S;
    if (i < E) pacc[grp * E + i] = acc[k];
  }
}

template <int S, int EPL>
__global__ __launch_bounds__(kRouteThreads) void route_kernel(
    const float* __restrict__ g, const float* __restrict__ eps, const int32_t* __restrict__ home,
    const int32_t* __restrict__ e2n, int32_t* __restrict__ eid, float* __restrict__ w, void* ws, int T,
    int E, int N, int relu, int tokens_per_block) {
  constexpr int G = kRouteThreads / S;
  extern __shared__ char smem[];
  int32_t* hist = (int32_t*)smem;            // [E]
  int32_t* hhist = hist + E;                 // [N]
  int32_t* local = hhist + N;                // [1]
  float* pacc = (float*)(local + 1);         // [G][E]
  for (int i = threadIdx.x; i < E + N + 1; i += kRouteThreads) hist[i] = 0;
  __syncthreads();
  const int tok0 = blockIdx.x * tokens_per_block;
  route_tokens<S, EPL, kRouteThreads>(g, eps, home, e2n, eid, w, hist, hhist, local, pacc, tok0,
                                      min(T, tok0 + tokens_per_block), E, N, relu);
  __syncthreads();
  RouteWs r = route_ws(ws, E, N);
  for (int i = threadIdx.x; i < E; i += kRouteThreads) {
    float s = 0.f;
    for (int q = 0; q < G; ++q) s += pacc[q * E + i];
    r.cell[(size_t)blockIdx.x * E + i] = make_int2(hist[i], __float_as_int(s));
  }
  for (int i = threadIdx.x; i < N; i += kRouteThreads) r.home[(size_t)blockIdx.x * N + i] = hhist[i];
  if (threadIdx.x == 0) r.local[blockIdx.x] = *local;
}

constexpr int kFinThreads = 1024;
constexpr int kFinWaves = kFinThreads / kWave;

// Sums (and one maximum) over the block of NQ doubles per thread, in a fixed order: a butterfly inside each wave
// (lane i adds lane i ^ o for o = 32 .. 1), the sixteen wave results through LDS, added in wave order by every
// thread.  Two barriers for all NQ quantities together.  ONE: only the first wave holds anything and is asked (with a branch at run
// time instead the finalize kernel took 0.8 us longer either way).
template <int NQ, bool ONE>
__device__ __forceinline__ void block_sums(double (&v)[NQ], double& vmax, double (*part)[kFinWaves]) {
  const int wave = threadIdx.x / kWave;
  if (ONE && wave) return;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) v[q] += __shfl_xor(v[q], o);
    vmax = fmax(vmax, __shfl_xor(vmax, o));
  }
  if (ONE) return;
  if (threadIdx.x % kWave == 0) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) part[q][wave] = v[q];
    part[NQ][wave] = vmax;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kFinWaves; ++w) t += part[q][w];
    v[q] = t;
  }
  double m = part[NQ][0];
#pragma unroll
  for (int w = 1; w < kFinWaves; ++w) m = fmax(m, part[NQ][w]);
  vmax = m;
}

// Adds up columns that thread (q, e), q = tid / E < R, holds a part of.  Result in thread e < E.  More than 16 parts: first
// those of up to eight q in a row, then these sums in order, so that no thread adds more than some R / 8 + 8 words one after
// the other (all R of them in one thread took 3 us of a small layer's route).  Up to 16 parts that costs more in barriers
// than it saves.
__device__ __forceinline__ void column_sums(int32_t& ci, double& ps, int32_t* ipart, double* dpart, int E, int R) {
  const int tid = threadIdx.x;
  ipart[tid] = ci;
  dpart[tid] = ps;
  __syncthreads();
  int parts = R;
  if (R > 16) {
    const int q = tid / E, e = tid - q * E;
    const int len = (R + 7) / 8;  // run j: q = j len .. + len
    parts = 8;
    if (q < parts) {
      const int q1 = min(R, (q + 1) * len);
      ci = 0;
      ps = 0.0;
#pragma unroll 8
      for (int i = q * len; i < q1; ++i) { ci += ipart[i * E + e]; ps += dpart[i * E + e]; }
    }
    __syncthreads();
    if (q < parts) { ipart[tid] = ci; dpart[tid] = ps; }
    __syncthreads();
  }
  if (tid < E) {
    ci = 0;
    ps = 0.0;
#pragma unroll 4
    for (int q = 0; q < parts; ++q) { ci += ipart[q * E + tid]; ps += dpart[q * E + tid]; }
  }
}

struct FinShared {
  double part[6][kFinWaves];
  double dpart[kFinThreads];
  int32_t ipart[kFinThreads];
  int32_t home[1024], pernode[1024];
};

// cnt, Psum and the scalars of Eq. 5 / Eq. 6 from the totals: thread e < E holds expert e's, home[] the tokens per home node
// and pernode[] the experts per node (both behind a barrier), and the threads together the tokens that stay on their node.
// ONE: these and the experts are all in the first wave.
template <bool ONE>
__device__ __forceinline__ void route_scalars(FinShared& sh, int32_t c, double p, int local, const int32_t* e2n, int has_home, int32_t* cnt, float* Psum, float* stats,
                                              int T, int E, int N, float alpha, float mu) {
  const int tid = threadIdx.x;
  // Eq. 5: L_aux = alpha * n * sum_i f_i P_i
  double q[5] = {0.0, 0.0, 0.0, (double)local, 0.0};  // f P, KL(f || D_l), KL(P || D_l) terms, local tokens, empty experts
  double mx = 0.0;
  if (tid < E) {
    cnt[tid] = c;
    Psum[tid] = (float)p;
    const double f = (double)c / T, P = p / T;
    q[0] = f * P;
    mx = (double)c;
    q[4] = c == 0 ? 1.0 : 0.0;
    if (has_home) {
      // Eq. 6 over experts: D_l[i] = T_node(i) / (T * experts on node(i))
      const int nu = e2n ? e2n[tid] : tid / (E / N);
      const double Dl = (double)sh.home[nu] / ((double)T * (double)sh.pernode[nu]);
      if (f > 0.0) q[1] = Dl > 0.0 ? f * log(f / Dl) : INFINITY;
      if (P > 0.0) q[2] = Dl > 0.0 ? P * log(P / Dl) : INFINITY;
    }
  }
  block_sums<5, ONE>(q, mx, sh.part);
  if (tid == 0) {
    stats[0] = (float)((double)alpha * E * q[0]);
    stats[1] = (float)q[1];
    stats[2] = (float)q[2];
    stats[3] = (float)((double)mu * q[1]);
    stats[4] = (float)(q[3] / T);
    stats[5] = (float)mx;
    stats[6] = (float)q[4];
    stats[7] = 0.f;
  }
}

// One block: column sums of the per-block partials, then the scalars of Eq. 5 / Eq. 6.  Bound by latencies (the launch,
// one round trip to partials that other XCDs wrote, LDS, a few double-precision logarithms).  U: rows that a thread adds in
// a round; the loads are unconditional (rows past the end re-read the thread's first row and are not added) and all of a
// round's are issued before the first is used, so U is no larger than the partials need: with 32 rows always, 64 partials
// took 64 loads in each of 1024 threads (T = 8 192, E = 16: 11.4 us).  With more than 16 rows a thread (E = 64 from 32 769
// tokens on) two rounds of 16 were two round trips to memory.  Both launches at T = 65 536, us: E = 64 20.1, E = 128 27.5,
// E = 300 68.5, of which a choice at run time between one wave and all in block_sums took 0.8, the second step of
// column_sums 0.3, and loads that waited for earlier ones 0.2; T = 8 192, E = 16: 10.2.
template <int U, bool ONE>
__global__ __launch_bounds__(kFinThreads) void route_finalize_kernel(
    void* ws, const int32_t* __restrict__ e2n, int has_home, int32_t* __restrict__ cnt,
    float* __restrict__ Psum, float* __restrict__ stats, int nb, int T, int E, int N, float alpha, float mu) {
  __shared__ FinShared sh;
  RouteWs r = route_ws(ws, E, N);
  const int tid = threadIdx.x;
  if (tid < N) { sh.home[tid] = 0; sh.pernode[tid] = 0; }
  const int R = kFinThreads / E;  // thread (rb, e) adds rows rb, rb+R, ... in order
  const int rb = tid / E, e = tid - rb * E;
  constexpr int UH = 8;
  const int Rn = kFinThreads / N;
  const int rn = tid / N, nu = tid - rn * N;
  const bool cols = rb < R && rb < nb, hcols = has_home && rn < Rn && rn < nb;
  int32_t ci = 0, hi = 0;
  double ps = 0.0;
  int local = 0;
  int32_t hvv[UH];
  if (hcols) {  // the home counts go with the first round (looped below if they are many)
    hvv[0] = r.home[(size_t)rn * N + nu];
    if (Rn < nb) {
#pragma unroll
      for (int u = 1; u < UH; ++u) {
        const int b = rn + u * Rn;
        hvv[u] = r.home[(size_t)(b < nb ? b : rn) * N + nu];
      }
    }
  }
  if (has_home && tid < nb) local = r.local[tid];  // (nb <= 512)
  // (24-bit products: a 64-bit multiply-add took a register of a load under way for its unused upper half, and waited for it)
  auto at = [&](int b) { return __umul24(b < nb ? b : rb, E) + e; };
  int b0 = 0;
  if constexpr (U == 32) {  // the first half of the rows is there for certain: one offset per thread, scalar distances
    for (; b0 + U / 2 * R < nb; b0 += U * R) {
      int2 v[U];
      if (cols) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int b = b0 + rb + u * R;
          if (u < U / 2) v[u] = (r.cell + (size_t)(b0 + u * R) * E)[(unsigned)(rb * E + e)];
          else v[u] = r.cell[at(b)];
        }
        __builtin_amdgcn_sched_barrier(0);  // (or the first are waited for before the last are issued)
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const bool live = u < U / 2 || b0 + rb + u * R < nb;
          ci += live ? v[u].x : 0;
          ps += live ? (double)__int_as_float(v[u].y) : 0.0;
        }
      }
    }
  }
  constexpr int UT = U == 32 ? 16 : U;
  for (; b0 < nb; b0 += UT * R) {
    int2 v[UT];
    if (cols) {
#pragma unroll
      for (int u = 0; u < UT; ++u) {
        const int b = b0 + rb + u * R;
        v[u] = r.cell[at(b)];
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < UT; ++u) {
        const bool live = b0 + rb + u * R < nb;
        ci += live ? v[u].x : 0;
        ps += live ? (double)__int_as_float(v[u].y) : 0.0;
      }
    }
  }
  if (hcols) {
    hi = hvv[0];
    if (Rn < nb) {
#pragma unroll
      for (int u = 1; u < UH; ++u) hi += (rn + u * Rn < nb) ? hvv[u] : 0;
      for (int b = rn + UH * Rn; b < nb; b += Rn) hi += r.home[(size_t)b * N + nu];  // (few nodes per thread group: rare)
    }
  }
  asm volatile("" : "+v"(local));  // (its conversion to double stays behind the cells' loads: ahead of them it waited for itself)
  column_sums(ci, ps, sh.ipart, sh.dpart, E, R);  // (its barriers stand behind the zeros above)
  if (has_home) {  // integer adds: any order gives the same counts
    if (hi) atomicAdd(&sh.home[nu], hi);
    if (tid < E) atomicAdd(&sh.pernode[e2n ? e2n[tid] : tid / (E / N)], 1);
  }
  __syncthreads();
  route_scalars<ONE>(sh, ci, ps, local, e2n, has_home, cnt, Psum, stats, T, E, N, alpha, mu);
}

// lanes per token: the whole expert axis up to 16 experts; beyond that, up to 128 experts, 16 lanes with
// several experts each (four tokens per wave side by side: the cross-lane reductions, which dominate the
// instruction count, shrink from six steps to four and are shared by four tokens); one wave per token above
inline int route_lanes(int E) {
  int S = 4;
  while (S < E && S < 16) S *= 2;
  return E > 128 ? 64 : S;
}

// One work-group where its groups take the tokens in one batch.  us in one / two launches: E = 4, 1 024 tokens 8.5 / 11.0,
// 2 048 11.2 / 11.0;  E = 8, 512 tokens 8.5 / 10.2, 1 024 11.4 / 10.3;  E = 16, 192 tokens 8.2 / 9.7, 512 11.9 / 10.0;
// E = 64, 192 tokens 10.4 / 11.1;  E = 128, 192 tokens 16.7 / 16.9.
inline bool route_in_one(int T, int E) { return E <= 64 && T <= kFinThreads / route_lanes(E) * kTokPerGroup; }

// Few tokens: one work-group does all of it, which saves the second launch and the way of the partials through memory.
template <int S, int EPL>
__global__ __launch_bounds__(kFinThreads) void route_one_kernel(
    const float* __restrict__ g, const float* __restrict__ eps, const int32_t* __restrict__ home,
    const int32_t* __restrict__ e2n, int32_t* __restrict__ eid, float* __restrict__ w, int32_t* __restrict__ cnt,
    float* __restrict__ Psum, float* __restrict__ stats, int T, int E, int N, int relu, float alpha, float mu) {
  constexpr int G = kFinThreads / S;
  __shared__ FinShared sh;
  __shared__ int32_t s_local;
  extern __shared__ char smem[];
  int32_t* hist = (int32_t*)smem;    // [E]
  float* pacc = (float*)(hist + E);  // [G][E]
  const int tid = threadIdx.x;
  if (tid < E) hist[tid] = 0;
  if (tid < N) { sh.home[tid] = 0; sh.pernode[tid] = 0; }
  if (tid == 0) s_local = 0;
  __syncthreads();
  route_tokens<S, EPL, kFinThreads>(g, eps, home, e2n, eid, w, hist, sh.home, &s_local, pacc, 0, T, E, N, relu);
  if (home && tid < E) atomicAdd(&sh.pernode[e2n ? e2n[tid] : tid / (E / N)], 1);
  __syncthreads();
  const int R = kFinThreads / E, rb = tid / E, e = tid - rb * E;
  int32_t ci = 0;
  double ps = 0.0;
  if (rb < R) {
#pragma unroll 4
    for (int q = rb; q < G; q += R) ps += (double)pacc[q * E + e];
  }
  column_sums(ci, ps, sh.ipart, sh.dpart, E, R);
  route_scalars<true>(sh, tid < E ? hist[tid] : 0, ps, tid == 0 ? s_local : 0, e2n, home ? 1 : 0, cnt, Psum, stats, T, E, N,
                      alpha, mu);  // (E <= 64)
}

template <int S, int EPL>
void launch_route(const locmoe_desc* p, const float* g, const float* eps, const int32_t* home,
                  const int32_t* e2n, int32_t* eid, float* w, int32_t* cnt, float* Psum, float* stats, void* ws, int nb,
                  int tpb, hipStream_t st) {
  if constexpr (S <= 16) {
    if (route_in_one(p->T, p->E)) {
      const size_t smem = (size_t)p->E * 4 + (size_t)(kFinThreads / S) * p->E * 4;
      hipLaunchKernelGGL((route_one_kernel<S, EPL>), dim3(1), dim3(kFinThreads), smem, st, g, eps, home, e2n, eid, w, cnt,
                         Psum, stats, p->T, p->E, p->N, p->relu, p->alpha, p->mu);
      return;
    }
  }
  constexpr int G = kRouteThreads / S;
  const size_t smem = (size_t)(p->E + p->N + 1) * 4 + (size_t)G * p->E * 4;
  hipLaunchKernelGGL((route_kernel<S, EPL>), dim3(nb), dim3(kRouteThreads), smem, st, g, eps, home, e2n, eid,
                     w, ws, p->T, p->E, p->N, p->relu, tpb);
}

}  // namespace
}  // namespace locmoe

extern "C" int locmoe_route(const locmoe_desc* desc, const float* g, const float* eps, const int32_t* home,
                            const int32_t* e2n, int32_t* eid, float* w, int32_t* cnt, float* Psum,
                            float* stats, void* ws, size_t ws_bytes, void* stream) {
  using namespace locmoe;
  if (!desc || !g || !eid || !w || !cnt || !Psum || !stats) return LOCMOE_ERR_NULL;
  int st = check_desc(desc);
  if (st != LOCMOE_OK) return st;
  if (!e2n && desc->E % desc->N != 0) return LOCMOE_ERR_SHAPE;
  if (!ws || ws_bytes < locmoe_workspace_bytes(desc)) return LOCMOE_ERR_WORKSPACE;
  hipStream_t s = as_stream(stream);
  const int E = desc->E;
  const int S = route_lanes(E);
  const int G = kRouteThreads / S;
  const int step = G * kTokPerGroup;
  int tpb = ceil_div(desc->T, kRouteMaxBlocks);
  tpb = ceil_div(tpb, step) * step;
  const int nb = ceil_div(desc->T, tpb);
  const int epl = ceil_div(E, S);
#define LOCMOE_ROUTE(SS, EE) launch_route<SS, EE>(desc, g, eps, home, e2n, eid, w, cnt, Psum, stats, ws, nb, tpb, s)
  if (S == 4) LOCMOE_ROUTE(4, 1);
  else if (S == 8) LOCMOE_ROUTE(8, 1);
  else if (S == 16 && epl == 1) LOCMOE_ROUTE(16, 1);
  else if (S == 16 && epl == 2) LOCMOE_ROUTE(16, 2);
  else if (S == 16 && epl <= 4) LOCMOE_ROUTE(16, 4);
  else if (S == 16) LOCMOE_ROUTE(16, 8);
  else if (epl <= 4) LOCMOE_ROUTE(64, 4);
  else if (epl <= 8) LOCMOE_ROUTE(64, 8);
  else LOCMOE_ROUTE(64, 16);
#undef LOCMOE_ROUTE
  st = launch_status();
  if (st != LOCMOE_OK) return st;
  if (route_in_one(desc->T, E)) return LOCMOE_OK;
  const int rounds = ceil_div(nb, kFinThreads / E);  // rows of partials per thread
  const bool one = E <= kWave && nb <= kWave;  // (then at most four rows)
  auto fin = rounds <= 1 ? (one ? route_finalize_kernel<1, true> : route_finalize_kernel<1, false>)
           : rounds <= 2 ? (one ? route_finalize_kernel<2, true> : route_finalize_kernel<2, false>)
           : rounds <= 4 ? (one ? route_finalize_kernel<4, true> : route_finalize_kernel<4, false>)
           : rounds <= 8 ? route_finalize_kernel<8, false>
           : rounds <= 16 ? route_finalize_kernel<16, false> : route_finalize_kernel<32, false>;
  hipLaunchKernelGGL(fin, dim3(1), dim3(kFinThreads), 0, s, ws, e2n, home ? 1 : 0, cnt, Psum, stats, nb, desc->T, E,
                     desc->N, desc->alpha, desc->mu);
  return launch_status();
}
