// Capacity-bounded stable dispatch (capacity: Section 3.2.3).
// Up to kDispOneTokens tokens dispatch_one_kernel does it all in one launch; else
//   1. dispatch_hist_kernel   per block of 1024 tokens: count of tokens per expert (few blocks: counted by step 2)
//   2. dispatch_slots_kernel  every block re-derives, from the [blocks,E] count matrix, the
//      tokens before it per expert and the totals, hence kept[], the buffer order and the
//      segment offsets; then ranks its own tokens (wave ballots + ordered wave prefixes)
//   3. dispatch_copy_kernel   send[r,:] = x[row_token[r],:] for r < K, 16-byte vectors
// Integer-only; LDS integer atomics appear only where the result does not depend on their
// order, so slots are bit-identical from run to run.
#include <algorithm>
#include <atomic>

#include "common.h"

namespace locmoe {
namespace {

// Scratch of locmoe_dispatch_static: the [blocks, E] count matrix lives in this array instead of a caller
// workspace.  Host code never uses the array's name as an address: static_scratch() asks the runtime for the
// device address once per device and hands that pointer to the kernels.
constexpr size_t kStaticScratchBytes = size_t(1) << 20;  // 262 144 counts: blocks of 1024 tokens x experts
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

// Device address of `scratch` on the current device (each device holds its own copy), nullptr if the runtime
// refuses.  Asked once per device; later calls read the cached pointer.
void* static_scratch() {
  static std::atomic<void*> cached[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
  void* ptr = cached[dev].load(std::memory_order_acquire);
  if (!ptr) {
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return nullptr;
    cached[dev].store(ptr, std::memory_order_release);
  }
  return ptr;
}

constexpr int kDispThreads = 256;
constexpr int kDispWaves = kDispThreads / kWave;
constexpr int kTokPerWave = kDispatchTokensPerBlock / kDispWaves;  // contiguous tokens per wave
constexpr int kIter = kTokPerWave / kWave;
// Orders this wave's LDS accesses before the call against those after it, for all lanes.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Buffer order (experts sorted by (node, id)): rank[e]; by_rank[r], the node, and seg[r], the first row of the expert at rank r
// (seg[E] = K), from the kept rows tot[e] and nodes node[e].  Called by a work-group of kDispThreads; ends with a barrier.
__device__ __forceinline__ void buffer_order(const int32_t* e2n, const int32_t* tot, const int32_t* node, int32_t* rank,
                                             int32_t* by_rank, int32_t* seg, int E) {
  const int tid = threadIdx.x, lane = tid % kWave;
  for (int e = tid; e < E; e += kDispThreads) {
    int r = e;
    if (e2n) {
      r = 0;
      const int ne = node[e];
#pragma unroll 8
      for (int q = 0; q < E; ++q) r += (node[q] < ne || (node[q] == ne && q < e)) ? 1 : 0;
    }
    rank[e] = r;
    by_rank[r] = node[e];
    seg[r + 1] = tot[e];  // staged: kept of the expert at rank r, scanned below
  }
  __syncthreads();
  if (tid / kWave == 0) {  // inclusive scan of seg[1..E] by one wave: lane owns a contiguous run
    const int per = ceil_div(E, kWave);
    const int lo = lane * per, hi = min(E, lo + per);
    int s = 0;
    for (int i = lo; i < hi; ++i) s += seg[i + 1];
    int incl = s;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
      const int o = __shfl_up(incl, d);
      if (lane >= d) incl += o;
    }
    int run = incl - s;
    if (lane == 0) seg[0] = 0;
    for (int i = lo; i < hi; ++i) {
      run += seg[i + 1];
      seg[i + 1] = run;
    }
  }
  __syncthreads();
}

// The outputs per expert and node, by one work-group
__device__ __forceinline__ void write_segments(const int32_t* tot, const int32_t* rank, const int32_t* by_rank,
                                               const int32_t* seg, int32_t* kept, int32_t* seg_off,
                                               int32_t* node_off, int32_t* buf_expert, int E, int N) {
  const int tid = threadIdx.x;
  for (int e = tid; e < E; e += kDispThreads) {
    kept[e] = tot[e];
    buf_expert[rank[e]] = e;
  }
  for (int i = tid; i <= E; i += kDispThreads) seg_off[i] = seg[i];
  // node nu starts where its first expert (or the next node's that has one) starts; the nodes ascend with the rank
  for (int r = tid; r <= E; r += kDispThreads) {
    const int last = r < E ? min(by_rank[r], N) : N;
    for (int nu = r ? max(by_rank[r - 1], -1) + 1 : 0; nu <= last; ++nu) node_off[nu] = seg[r];
  }
}

// The lanes of a wave that hold the same expert as this one (none of those that are not valid)
__device__ __forceinline__ unsigned long long same_expert(int e, bool valid, int nbits) {
  unsigned long long peers = __ballot(valid);
  for (int bit = 0; bit < nbits; ++bit) {
    const bool set = (e >> bit) & 1;
    const unsigned long long bm = __ballot(valid && set);
    peers &= set ? bm : ~bm;
  }
  return peers;
}

// Tokens per expert, counted by one work-group of kDispThreads into LDS that is zero: before[e] of the tokens ahead of
// `base`, rest[e] of the others.  ALIGNED: base is a multiple of the wave.  Every thread comes by behind(i0) between a round's
// loads and their use.
template <int U, bool ALIGNED, class F>
__device__ __forceinline__ void count_tokens(const int32_t* __restrict__ eid, int32_t* before, int32_t* rest, int base, int T,
                                             F behind) {
  const int tid = threadIdx.x, lane = tid % kWave;
  for (int i0 = 0; i0 < T; i0 += U * kDispThreads) {
    int c[U];
#pragma unroll
    for (int u = 0; u < U; ++u) c[u] = eid[min(i0 + tid + u * kDispThreads, T - 1)];
    behind(i0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int m = i0 + tid + u * kDispThreads;
      if (m < T) {
        // the tokens of the first lane's expert are added at once: additions to one word wait for each other
        const int first = __builtin_amdgcn_readfirstlane(c[u]);
        const bool mine = c[u] == first && (ALIGNED || (m < base) == (__builtin_amdgcn_readfirstlane(m) < base));
        const unsigned long long same = __ballot(mine);
        if (!mine || lane == __builtin_ctzll(same))
          atomicAdd((m < base ? before : rest) + c[u], mine ? __builtin_popcountll(same) : 1);
      }
    }
  }
}

// Few tokens: every work-group counts all tokens' experts for itself (those before its own `per` tokens and the rest),
// hence kept[], the buffer order and its tokens' slots, and copies their rows, whose first kOneLoads 16-byte pieces per
// thread are fetched ahead of the counting.  Bound by latencies: the launch, one round trip to eid, some ten barriers.
// us, this / two launches (slots by blocks of 1024 tokens that count for themselves, then a copy over the kept rows):
//     192 tokens: d = 1024, E = 16 4.7 / 8.1;  d = 1600, E = 40 4.8 / 10.0;  d = 5120, E = 128 5.1 / 14.4
//   4 096 tokens: 8.1 / 11.0;  9.7 / 15.0;  21.5 / 29.8;  4 of 5 tokens on one expert 7.7 / 10.2;  9.1 / 12.9;  16.0 / 20.8
// The line lies where no distribution of the tokens loses (the rows of dropped tokens are fetched in vain); this / three
// launches: 5 120 tokens, 4 of 5 on one expert, d = 1024, E = 16 8.3 / 10.7;  d = 5120, E = 128 19.4 / 17.4.
// From there to kDispSelfBlocks blocks, and with rows beyond kOneMaxChunks pieces, the two launches stay: the slots kernel
// counts for itself.  us, two / three launches: 4 500 tokens, 4 of 5 on one expert, d = 768 fp32, E = 6 10.7 / 11.5;  d = 16 640,
// E = 8: 65 tokens 7.9 / 9.5, 1 024 11.3 / 13.1.  Beyond, some spread loses: 6 000 tokens on two of 16 experts 10.3 / 10.2;
// 8 192 tokens evenly spread 11.3 / 10.9.
constexpr int kDispSelfBlocks = 5;
constexpr int kDispOneTokens = 4096, kOneMaxTok = kWave, kOneLoads = 8, kOneMaxChunks = 2048;
__global__ __launch_bounds__(kDispThreads) void dispatch_one_kernel(
    const uint4* __restrict__ x, const int32_t* __restrict__ eid, const int32_t* __restrict__ e2n,
    int32_t* __restrict__ pos, int32_t* __restrict__ slot, int32_t* __restrict__ kept, int32_t* __restrict__ seg_off,
    int32_t* __restrict__ node_off, int32_t* __restrict__ buf_expert, int32_t* __restrict__ row_token,
    uint4* __restrict__ send, int T, int E, int N, int C, int per, int chunks, int nbits) {
  extern __shared__ int32_t sm[];
  __shared__ int32_t s_slot[kOneMaxTok];
  int32_t* off = sm;        // [E] tokens before this work-group's
  int32_t* tot = off + E;   // [E] the others, then kept rows
  int32_t* node = tot + E;
  int32_t* rank = node + E;
  int32_t* seg = rank + E;  // [E+1], indexed by buffer rank
  int32_t* by_rank = seg + E + 1;
  const int tid = threadIdx.x, lane = tid % kWave;
  const int base = blockIdx.x * per, n = min(per, T - base);
  const unsigned pieces = (unsigned)n * chunks;  // the tokens' rows, one run of 16-byte pieces
  const uint4* src = x + (size_t)base * chunks;
  uint4 v[kOneLoads];
  const int my_e = tid < n ? eid[base + tid] : 0;
  for (int i = tid; i < 2 * E; i += kDispThreads) sm[i] = 0;
  __syncthreads();
  count_tokens<10, false>(eid, off, tot, base, T, [&](int i0) {  // (the rows are fetched behind the first loads)
    if (i0 == 0) {
#pragma unroll
      for (int u = 0; u < kOneLoads; ++u) v[u] = nt_load16(src + min((unsigned)(tid + u * kDispThreads), pieces - 1));
    }
  });
  __syncthreads();
  for (int e = tid; e < E; e += kDispThreads) {
    const int all = off[e] + tot[e];
    tot[e] = all < C ? all : C;  // kept[e] = min(cnt[e], C)
    node[e] = e2n ? e2n[e] : e / (E / N);
  }
  __syncthreads();
  buffer_order(e2n, tot, node, rank, by_rank, seg, E);
  if (blockIdx.x == 0) write_segments(tot, rank, by_rank, seg, kept, seg_off, node_off, buf_expert, E, N);
  if (tid < kWave) {  // the work-group's tokens, one per lane
    const bool valid = tid < n;
    const unsigned long long peers = same_expert(my_e, valid, nbits);
    if (valid) {
      const int p = off[my_e] + __popcll(peers & ((1ull << lane) - 1ull));
      const int s = p < C ? seg[rank[my_e]] + p : -1;
      pos[base + tid] = p;
      slot[base + tid] = s;
      if (s >= 0) row_token[s] = base + tid;
      s_slot[tid] = s;
    }
  }
  __syncthreads();
  for (unsigned c0 = tid; c0 < pieces; c0 += kOneLoads * kDispThreads) {
    int s[kOneLoads];
    unsigned in[kOneLoads];
#pragma unroll
    for (int u = 0; u < kOneLoads; ++u) {
      const unsigned c = min(c0 + u * kDispThreads, pieces - 1), t = c / (unsigned)chunks;
      s[u] = c0 + u * kDispThreads < pieces ? s_slot[t] : -1;
      in[u] = c - t * chunks;
      if (c0 >= kOneLoads * kDispThreads && s[u] >= 0) v[u] = nt_load16(src + c);  // (now only of kept tokens)
    }
#pragma unroll
    for (int u = 0; u < kOneLoads; ++u)
      if (s[u] >= 0) send[(size_t)s[u] * chunks + in[u]] = v[u];  // (plain: the FFN re-reads send right away)
  }
}

__global__ __launch_bounds__(kDispThreads) void dispatch_hist_kernel(const int32_t* __restrict__ eid,
                                                                     int32_t* __restrict__ blockcnt, int T,
                                                                     int E) {
  extern __shared__ int32_t hist[];
  for (int i = threadIdx.x; i < E; i += kDispThreads) hist[i] = 0;
  __syncthreads();
  const int base = blockIdx.x * kDispatchTokensPerBlock;
#pragma unroll
  for (int k = 0; k < kDispatchTokensPerBlock / kDispThreads; ++k) {
    const int m = base + k * kDispThreads + threadIdx.x;
    if (m < T) atomicAdd(&hist[eid[m]], 1);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < E; i += kDispThreads) blockcnt[(size_t)blockIdx.x * E + i] = hist[i];
}

// LDS layout of the slots kernel (ints): off[E] tot[E] node[E] rank[E] by_rank[E] seg[E+1] wcnt[waves][E]
__global__ __launch_bounds__(kDispThreads) void dispatch_slots_kernel(
    const int32_t* __restrict__ eid, const int32_t* __restrict__ e2n, const int32_t* __restrict__ blockcnt,
    int32_t* __restrict__ pos, int32_t* __restrict__ slot, int32_t* __restrict__ kept,
    int32_t* __restrict__ seg_off, int32_t* __restrict__ node_off, int32_t* __restrict__ buf_expert,
    int32_t* __restrict__ row_token, int T, int E, int N, int C, int nblocks, int nbits) {
  extern __shared__ int32_t sm[];
  int32_t* off = sm;
  int32_t* tot = off + E;
  int32_t* node = tot + E;
  int32_t* rank = node + E;
  int32_t* by_rank = rank + E;
  int32_t* seg = by_rank + E;  // [E+1], indexed by buffer rank
  int32_t* wcnt = seg + E + 1;
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const int b = blockIdx.x;
  // this lane's tokens (wave-contiguous), fetched first so that the loads overlap the prefix work below
  const int wbase = b * kDispatchTokensPerBlock + wave * kTokPerWave;
  int my_e[kIter], my_p[kIter];
#pragma unroll
  for (int k = 0; k < kIter; ++k) {
    const int m = wbase + k * kWave + lane;
    my_e[k] = m < T ? eid[m] : -1;
  }

  // tokens per expert in earlier blocks, and in all blocks: thread (rg, e) adds the rows q = rg, rg+R, ...
  // of the [blocks, E] count matrix (independent loads), then the R partials are added in order
  if (!blockcnt) {  // few blocks: counted here, by every block for itself
    int32_t* earlier = wcnt;     // [E] tokens before this block's
    int32_t* later = wcnt + E;   // [E] this block's and after
    for (int i = tid; i < 2 * E; i += kDispThreads) wcnt[i] = 0;
    __syncthreads();
    count_tokens<8, true>(eid, earlier, later, b * kDispatchTokensPerBlock, T, [](int) {});
    __syncthreads();
    for (int e = tid; e < E; e += kDispThreads) {
      const int all = earlier[e] + later[e];
      off[e] = earlier[e];
      tot[e] = all < C ? all : C;  // kept[e] = min(cnt[e], C)
      node[e] = e2n ? e2n[e] : e / (E / N);
    }
  } else {
    const int R = E < kDispThreads ? kDispThreads / E : 1;  // row groups working on one chunk of experts
    int32_t* part_before = wcnt;                             // [R][E] scratch (wcnt is zeroed afterwards)
    int32_t* part_all = wcnt + kDispThreads;                 // R*E <= kDispThreads when R > 1
    for (int e0 = 0; e0 < E; e0 += kDispThreads) {
      const int e = e0 + (R > 1 ? tid % E : tid), rg = R > 1 ? tid / E : 0;
      int before = 0, all = 0;
      if (e < E && rg < R && rg < nblocks) {
        // (unconditional loads - rows past the end re-read row rg and are not added - so that a batch of eight is
        // in flight at once; with the bound inside the loop every load waited for the one before it)
        for (int q0 = rg; q0 < nblocks; q0 += 8 * R) {
          int c[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            const int q = q0 + u * R;
            c[u] = blockcnt[(size_t)(q < nblocks ? q : rg) * E + e];
          }
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            const int q = q0 + u * R;
            before += q < b ? c[u] : 0;   // (b < nblocks: rows past the end are never before this block)
            all += q < nblocks ? c[u] : 0;
          }
        }
      }
      if (R > 1) {
        if (rg < R) { part_before[rg * E + e] = before; part_all[rg * E + e] = all; }
        __syncthreads();
        if (tid < E) {
          before = 0; all = 0;
          for (int q = 0; q < R; ++q) { before += part_before[q * E + tid]; all += part_all[q * E + tid]; }
        }
        __syncthreads();
      }
      const int eo = R > 1 ? tid : e;
      if (eo < E && (R == 1 || tid < E)) {
        off[eo] = before;
        tot[eo] = all < C ? all : C;  // kept[e] = min(cnt[e], C)
        node[eo] = e2n ? e2n[eo] : eo / (E / N);
      }
    }
  }
  __syncthreads();
  for (int i = tid; i < kDispWaves * E; i += kDispThreads) wcnt[i] = 0;
  __syncthreads();
  buffer_order(e2n, tot, node, rank, by_rank, seg, E);
  if (b == 0) write_segments(tot, rank, by_rank, seg, kept, seg_off, node_off, buf_expert, E, N);

  // rank of each token among the block's earlier tokens of the same expert
  int32_t* wc = wcnt + wave * E;
#pragma unroll
  for (int k = 0; k < kIter; ++k) {
    const bool valid = my_e[k] >= 0;
    const int e = valid ? my_e[k] : 0;
    const unsigned long long peers = same_expert(e, valid, nbits);
    const unsigned long long lt = (1ull << lane) - 1ull;
    const int before = __popcll(peers & lt);
    int p = 0;
    if (valid) p = wc[e] + before;       // all lanes read the wave's running count ...
    wave_sync();
    if (valid && before == 0) wc[e] = p + __popcll(peers);  // ... then each group's first lane advances it
    wave_sync();
    my_p[k] = p;
  }
  __syncthreads();
  // ordered prefix over the block's waves (in place: wcnt[w][e] := tokens of e in waves < w)
  for (int e = tid; e < E; e += kDispThreads) {
    int run = off[e];
#pragma unroll
    for (int q = 0; q < kDispWaves; ++q) {
      const int c = wcnt[q * E + e];
      wcnt[q * E + e] = run;
      run += c;
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kIter; ++k) {
    const int m = wbase + k * kWave + lane;
    const int e = my_e[k];
    if (e >= 0) {
      const int p = wc[e] + my_p[k];
      pos[m] = p;
      int s = -1;
      if (p < C) {
        s = seg[rank[e]] + p;
        row_token[s] = m;
      }
      slot[m] = s;
    }
  }
}

// send[r,:] = x[row_token[r],:].  A row is `chunks` 16-byte vectors; LPR lanes share a row.  Blocks walk the
// K kept rows with a grid stride; the token index of the next row is fetched before the current row is
// copied, so the index -> row dependency is off the critical path.
constexpr int kCopyBlocksPerCu = 8;

template <int LPR>
__global__ __launch_bounds__(kDispThreads) void dispatch_copy_kernel(const uint4* __restrict__ x,
                                                                     const int32_t* __restrict__ row_token,
                                                                     const int32_t* __restrict__ seg_off,
                                                                     uint4* __restrict__ send, int E, int chunks) {
  constexpr int RPB = kDispThreads / LPR;
  constexpr int U = 4;
  const int K = seg_off[E];
  const int l = threadIdx.x % LPR;
  const int stride = gridDim.x * RPB;
  int r = blockIdx.x * RPB + threadIdx.x / LPR;
  int tok = r < K ? row_token[r] : 0;
  while (r < K) {
    const int rn = r + stride;
    const int tokn = rn < K ? row_token[rn] : 0;
    const uint4* src = x + (size_t)tok * chunks;
    uint4* dst = send + (size_t)r * chunks;
    int c = l;
    for (; c + (U - 1) * LPR < chunks; c += U * LPR) {
      uint4 v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = nt_load16(src + c + u * LPR);
#pragma unroll
      for (int u = 0; u < U; ++u) dst[c + u * LPR] = v[u];  // plain stores: the FFN re-reads send right away
    }
    for (; c < chunks; c += LPR) dst[c] = nt_load16(src + c);
    r = rn;
    tok = tokn;
  }
}

template <int LPR>
void launch_copy(const void* x, const int32_t* row_token, const int32_t* seg_off, void* send, int E, int rows,
                 int chunks, hipStream_t st) {
  constexpr int RPB = kDispThreads / LPR;
  const int blocks = min(ceil_div(rows, RPB), cu_count() * kCopyBlocksPerCu);
  hipLaunchKernelGGL((dispatch_copy_kernel<LPR>), dim3(blocks), dim3(kDispThreads), 0, st, (const uint4*)x,
                     row_token, seg_off, (uint4*)send, E, chunks);
}


// The launches of the dispatch: one for few tokens, else histogram, slots, copy, up to kDispSelfBlocks blocks of tokens without
// the histogram.  `blockcnt` holds ceil(T/1024) x E counts (every one is written by the first kernel before the second reads
// it: nothing has to be cleared); without a histogram it is not touched.
int dispatch_launch(const locmoe_desc* desc, const void* x, const int32_t* eid, const int32_t* e2n, int32_t* pos,
                    int32_t* slot, int32_t* kept, int32_t* seg_off, int32_t* node_off, int32_t* buf_expert,
                    int32_t* row_token, void* send, int32_t* blockcnt, hipStream_t s) {
  const int T = desc->T, E = desc->E;
  const int nblocks = ceil_div(T, kDispatchTokensPerBlock);
  int nbits = 0;
  while ((1 << nbits) < E) ++nbits;
  const int chunks = desc->d * (desc->x_dtype == LOCMOE_BF16 ? 2 : 4) / 16;
  if (T <= kDispOneTokens && chunks <= kOneMaxChunks) {
    // tokens per work-group: as many as the loads ahead hold, or 8 where they hold fewer (each work-group counts all tokens),
    // and at most ceil(T / 128): 128 work-groups, fewer where T / 128 is rounded up, more where the rows are long
    const int per = std::min(std::min(kOneMaxTok, std::max(8, kOneLoads * kDispThreads / chunks)), ceil_div(T, 128));
    hipLaunchKernelGGL(dispatch_one_kernel, dim3(ceil_div(T, per)), dim3(kDispThreads), ((size_t)E * 6 + 1) * 4, s,
                       (const uint4*)x, eid, e2n, pos, slot, kept, seg_off, node_off, buf_expert, row_token, (uint4*)send,
                       T, E, desc->N, desc->C, per, chunks, nbits);
    return launch_status();
  }
  int st = LOCMOE_OK;
  if (nblocks <= kDispSelfBlocks) {
    blockcnt = nullptr;
  } else {
    hipLaunchKernelGGL(dispatch_hist_kernel, dim3(nblocks), dim3(kDispThreads), (size_t)E * 4, s, eid, blockcnt, T, E);
    st = launch_status();
    if (st != LOCMOE_OK) return st;
  }
  const size_t wcnt_ints = (size_t)kDispWaves * E > 2 * (size_t)kDispThreads ? (size_t)kDispWaves * E : 2 * (size_t)kDispThreads;
  const size_t smem = ((size_t)E * 6 + 1 + wcnt_ints) * 4;
  hipLaunchKernelGGL(dispatch_slots_kernel, dim3(nblocks), dim3(kDispThreads), smem, s, eid, e2n, blockcnt, pos,
                     slot, kept, seg_off, node_off, buf_expert, row_token, T, E, desc->N, desc->C, nblocks, nbits);
  st = launch_status();
  if (st != LOCMOE_OK) return st;
  // at most min(T, E*C) rows can be kept; the kernel reads the real K from seg_off[E]
  const long long cap = (long long)E * desc->C;
  const int rows = (int)(cap < T ? cap : T);
  // lanes per row: every lane should own at least 4 chunks so that 4 loads are in flight before the stores
  if (chunks >= 1024) launch_copy<256>(x, row_token, seg_off, send, E, rows, chunks, s);
  else if (chunks >= 512) launch_copy<128>(x, row_token, seg_off, send, E, rows, chunks, s);
  else if (chunks >= 256) launch_copy<64>(x, row_token, seg_off, send, E, rows, chunks, s);
  else if (chunks >= 128) launch_copy<32>(x, row_token, seg_off, send, E, rows, chunks, s);
  else if (chunks >= 64) launch_copy<16>(x, row_token, seg_off, send, E, rows, chunks, s);
  else launch_copy<8>(x, row_token, seg_off, send, E, rows, chunks, s);
  return launch_status();
}

int dispatch_check(const locmoe_desc* desc, const void* x, const int32_t* eid, const int32_t* e2n, int32_t* pos,
                   int32_t* slot, int32_t* kept, int32_t* seg_off, int32_t* node_off, int32_t* buf_expert,
                   int32_t* row_token, void* send) {
  if (!desc || !x || !eid || !pos || !slot || !kept || !seg_off || !node_off || !buf_expert || !row_token ||
      !send)
    return LOCMOE_ERR_NULL;
  const int st = check_desc(desc);
  if (st != LOCMOE_OK) return st;
  if (!e2n && desc->E % desc->N != 0) return LOCMOE_ERR_SHAPE;
  return LOCMOE_OK;
}

}  // namespace
}  // namespace locmoe

extern "C" int locmoe_dispatch(const locmoe_desc* desc, const void* x, const int32_t* eid, const int32_t* e2n,
                               int32_t* pos, int32_t* slot, int32_t* kept, int32_t* seg_off, int32_t* node_off,
                               int32_t* buf_expert, int32_t* row_token, void* send, void* ws, size_t ws_bytes,
                               void* stream) {
  using namespace locmoe;
  const int st = dispatch_check(desc, x, eid, e2n, pos, slot, kept, seg_off, node_off, buf_expert, row_token, send);
  if (st != LOCMOE_OK) return st;
  if (!ws || ws_bytes < locmoe_workspace_bytes(desc)) return LOCMOE_ERR_WORKSPACE;
  return dispatch_launch(desc, x, eid, e2n, pos, slot, kept, seg_off, node_off, buf_expert, row_token, send,
                         (int32_t*)ws, as_stream(stream));
}

// For callers that cannot allocate: locmoe_dispatch with the count matrix in the library's static scratch.
extern "C" int locmoe_dispatch_static(const locmoe_desc* desc, const void* x, const int32_t* eid, const int32_t* e2n,
                                      int32_t* pos, int32_t* slot, int32_t* kept, int32_t* seg_off,
                                      int32_t* node_off, int32_t* buf_expert, int32_t* row_token, void* send,
                                      void* stream) {
  using namespace locmoe;
  const int st = dispatch_check(desc, x, eid, e2n, pos, slot, kept, seg_off, node_off, buf_expert, row_token, send);
  if (st != LOCMOE_OK) return st;
  const size_t counts = (size_t)ceil_div(desc->T, kDispatchTokensPerBlock) * (size_t)desc->E;
  if (counts * sizeof(int32_t) > kStaticScratchBytes) return LOCMOE_ERR_WORKSPACE;  // beyond the stated maximum
  void* ptr = static_scratch();
  if (!ptr) return LOCMOE_ERR_HIP;
  return dispatch_launch(desc, x, eid, e2n, pos, slot, kept, seg_off, node_off, buf_expert, row_token, send,
                         (int32_t*)ptr, as_stream(stream));
}
