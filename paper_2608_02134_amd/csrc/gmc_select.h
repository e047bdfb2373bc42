// Device code of the batched responsibility selection (included by
// k_select.hip alone: its kernels are static): deterministic top-k, the batch
// pick, the butterfly transpose-reduction and the persistent selection kernels.
#pragma once

#include <type_traits>

#include "gmc_device.h"
#include "gmc_internal.h"

namespace gmc {

// Deterministic top-k over n keys (256-thread block): the `count` largest
// keys, equal keys resolved to the lower index.  Indices are written in
// ascending order to out[0..count).  count must not exceed the number of
// non-zero keys.  Radix selection of the threshold key with 8-bit digits
// (digits shared by every key are skipped; two histogram buffers, so each
// pass needs two block barriers), then one packed scan for the ordered
// compaction (each thread owns a contiguous index segment).
// hist: 512 ints of LDS, scan: >= 16 ints, bc: 2 ints.
__device__ inline void block_topk256(const uint32_t* keys, int n, int count, int* out, int* hist, int* scan,
                              int* bc) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  hist[tid] = 0;
  hist[256 + tid] = 0;
  uint32_t kand = 0xFFFFFFFFu, kor = 0u;
  for (int i = tid; i < n; i += 256) {
    const uint32_t k = keys[i];
    kand &= k;
    kor |= k;
  }
  kand = wave_and_u(kand);
  kor = wave_or_u(kor);
  if (lane == 0) { scan[wave] = static_cast<int>(kand); scan[4 + wave] = static_cast<int>(kor); }
  __syncthreads();
  kand = static_cast<uint32_t>(scan[0]) & static_cast<uint32_t>(scan[1]) & static_cast<uint32_t>(scan[2]) &
         static_cast<uint32_t>(scan[3]);
  kor = static_cast<uint32_t>(scan[4]) | static_cast<uint32_t>(scan[5]) | static_cast<uint32_t>(scan[6]) |
        static_cast<uint32_t>(scan[7]);
  const uint32_t diff = kand ^ kor;                 // bits that vary between keys
  uint32_t mask = 0;
  int top = 24;
  while (top > 0 && ((diff >> top) & 0xFFu) == 0u) {
    mask |= 0xFFu << top;
    top -= 8;
  }
  uint32_t prefix = kand & mask;
  int remaining = count, buf = 0;
  for (int shift = top; shift >= 0; shift -= 8, buf ^= 1) {
    int* h = hist + buf * 256;
    for (int i = tid; i < n; i += 256) {
      const uint32_t k = keys[i];
      if ((k & mask) == prefix) atomicAdd(&h[(k >> shift) & 255u], 1);
    }
    hist[(buf ^ 1) * 256 + tid] = 0;   // read in the previous pass; used by the next one
    __syncthreads();
    if (wave == 0) {
      // wave 0 scans the 256 bins from the top digit down, 4 per lane
      int v[4], loc = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) { v[q] = h[255 - (lane * 4 + q)]; loc += v[q]; }
      int excl = wave_scan_add(loc) - loc;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (excl < remaining && remaining <= excl + v[q]) {
          bc[0] = 255 - (lane * 4 + q);
          bc[1] = remaining - excl;
        }
        excl += v[q];
      }
    }
    __syncthreads();
    prefix |= static_cast<uint32_t>(bc[0]) << shift;
    mask |= 0xFFu << shift;
    remaining = bc[1];
  }
  const uint32_t kth = prefix;
  const int seg = (n + 255) / 256;
  const int i0 = min(n, tid * seg), i1 = min(n, i0 + seg);
  int gt = 0, eq = 0;
  for (int i = i0; i < i1; ++i) {
    const uint32_t k = keys[i];
    gt += k > kth;
    eq += k == kth;
  }
  int tot;
  const int pre = block_exclusive_scan(gt | (eq << 16), scan, &tot);
  int gt_b = static_cast<int>(static_cast<unsigned>(pre) & 0xFFFFu);
  int eq_b = static_cast<int>(static_cast<unsigned>(pre) >> 16);
  for (int i = i0; i < i1; ++i) {
    const uint32_t k = keys[i];
    if (k > kth) {
      out[gt_b + min(eq_b, remaining)] = i;
      ++gt_b;
    } else if (k == kth) {
      if (eq_b < remaining) out[gt_b + eq_b] = i;
      ++eq_b;
    }
  }
  __syncthreads();
}

// Register-resident variant of the same selection for small n: thread t
// holds the keys of its contiguous index segment [t*seg, t*seg + seg) in
// k[0..KPT) (0 past the segment; zero keys are excluded).  The radix windows
// start at the highest bit in which the non-zero keys differ, so the first
// histogram spreads the keys over up to 256 bins.  Passes continue until the
// bin holding the threshold is taken whole (the selection is then every
// non-zero key >= the resolved prefix) or every bit is resolved (the
// threshold is one key value, its first `remaining` copies by index taken).
// Every wave scans the histograms itself, so a radix pass needs one block
// barrier (three histogram buffers rotate).  The block has NW >= 4 waves.
// The selected indices are written to out[0, count) in ascending index order
// and out[count, fill) is filled with index 0.
// hist: 768 ints of LDS, scan: >= 3 NW ints.  least (if given, holding the
// largest word) gets the smallest selected key.
template <int KPT, int NW = 4>
__device__ inline void block_topk_regs(const uint32_t (&k)[KPT], int seg, int count, int* out, int* hist, int* scan,
                                int fill = 64, uint32_t* least = nullptr) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid < 256) {
    hist[tid] = 0;
    hist[256 + tid] = 0;
    hist[512 + tid] = 0;
  }
  uint32_t kand = 0xFFFFFFFFu, kor = 0u;
#pragma unroll
  for (int q = 0; q < KPT; ++q) {
    kand &= k[q] ? k[q] : 0xFFFFFFFFu;
    kor |= k[q];
  }
  kand = wave_and_u(kand);
  kor = wave_or_u(kor);
  if (lane == 0) { scan[wave] = static_cast<int>(kand); scan[NW + wave] = static_cast<int>(kor); }
  __syncthreads();
  kand = static_cast<uint32_t>(scan[0]);
  kor = static_cast<uint32_t>(scan[NW]);
#pragma unroll
  for (int w = 1; w < NW; ++w) {
    kand &= static_cast<uint32_t>(scan[w]);
    kor |= static_cast<uint32_t>(scan[NW + w]);
  }
  const uint32_t diff = kand ^ kor;
  // bits [hi, 32) are shared by every non-zero key; with no differing bit
  // every non-zero key equals kand
  int hi = diff ? 32 - __clz(diff) : 0;
  uint32_t mask = hi >= 32 ? 0u : ~((1u << hi) - 1u);
  uint32_t prefix = kand & mask;
  int remaining = count, buf = 0;
  while (hi > 0) {
    const int lo = max(hi - 8, 0);
    const uint32_t wmask = ((1u << (hi - lo)) - 1u) << lo;
    int* h = hist + buf * 256;
#pragma unroll
    for (int q = 0; q < KPT; ++q)
      if (k[q] != 0u && (k[q] & mask) == prefix) atomicAdd(&h[(k[q] & wmask) >> lo], 1);
    const int nxt = buf == 2 ? 0 : buf + 1;
    if (tid < 256) hist[nxt * 256 + tid] = 0;   // last read two passes ago
    __syncthreads();
    int v[4], loc = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) { v[q] = h[255 - (lane * 4 + q)]; loc += v[q]; }
    const int incl = wave_scan_add(loc);
    int excl = incl - loc;
    const bool hit = excl < remaining && remaining <= incl;
    int dig = 0, rem = 0, inbin = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (excl < remaining && remaining <= excl + v[q]) {
        dig = 255 - (lane * 4 + q);
        rem = remaining - excl;
        inbin = v[q];
      }
      excl += v[q];
    }
    const int src = __ffsll(static_cast<unsigned long long>(__ballot(hit))) - 1;
    dig = __builtin_amdgcn_readlane(dig, src);
    rem = __builtin_amdgcn_readlane(rem, src);
    inbin = __builtin_amdgcn_readlane(inbin, src);
    prefix |= static_cast<uint32_t>(dig) << lo;
    mask |= wmask;
    remaining = rem;
    hi = lo;
    if (inbin == remaining) {
      // every key of the threshold bin is taken: the selection is exactly
      // the non-zero keys >= prefix (its unresolved bits zero)
      remaining = count;
      hi = 0;
    }
    buf = nxt;
  }
  const uint32_t kth = prefix;
  int gt = 0, eq = 0;
#pragma unroll
  for (int q = 0; q < KPT; ++q) {
    gt += k[q] != 0u && k[q] > kth;
    eq += k[q] != 0u && k[q] == kth;
  }
  // exclusive prefix of (gt, eq) over threads: wave scans, then the wave
  // totals (scan[2 NW, 3 NW), untouched earlier in the call) after one barrier
  const int v = gt | (eq << 16);
  const int incl = wave_scan_add(v);
  if (lane == 63) scan[2 * NW + wave] = incl;
  __syncthreads();
  int pre = incl - v;
  for (int w = 0; w < wave; ++w) pre += scan[2 * NW + w];
  int gt_b = static_cast<int>(static_cast<unsigned>(pre) & 0xFFFFu);
  int eq_b = static_cast<int>(static_cast<unsigned>(pre) >> 16);
  const int i0 = tid * seg;
  uint32_t low = 0xFFFFFFFFu;
#pragma unroll
  for (int q = 0; q < KPT; ++q) {
    if (k[q] == 0u) continue;
    if (k[q] > kth) {
      out[gt_b + min(eq_b, remaining)] = i0 + q;
      low = min(low, k[q]);
      ++gt_b;
    } else if (k[q] == kth) {
      if (eq_b < remaining) {
        out[gt_b + eq_b] = i0 + q;
        low = min(low, k[q]);
      }
      ++eq_b;
    }
  }
  if (least && low != 0xFFFFFFFFu) atomicMin(least, low);
  if (tid >= count && tid < fill) out[tid] = 0;
  __syncthreads();
}

// Mark the batch (indices into the pool, ascending) and record it.
__device__ inline void commit_batch(const Shape& sh, const Ws& ws, int p, int round, int bsize, int sel_base,
                             const int* pool_s, const int* chosen, int32_t* trace_batch) {
  int* sel = ws.sel + p * ws.s_sel;
  int* order = ws.order + p * ws.s_ord;
  int* batch = ws.batch + p * ws.s_bat;
  for (int k = threadIdx.x; k < bsize; k += blockDim.x) {
    const int i = pool_s[chosen[k]];
    sel[i] = round;
    order[sel_base + k] = i;
    batch[k] = i;
  }
  if (trace_batch) {
    int32_t* tb = trace_batch + (static_cast<long long>(p) * sh.rounds + round) * sh.b;
    for (int k = threadIdx.x; k < sh.b; k += blockDim.x) tb[k] = (k < bsize) ? pool_s[chosen[k]] : -1;
  }
}

// Ballot-based selection inside one wave.  Keys are held in lanes (KPT per
// lane); the count of keys >= c is a sum of ballot popcounts, so the
// count-th largest key value is found by a 32-step bitwise search with no
// LDS traffic: the largest v with at least `count` keys >= v.
template <int KPT>
__device__ __forceinline__ int wave_count_ge(const uint32_t (&k)[KPT], uint32_t c) {
  int n = 0;
#pragma unroll
  for (int q = 0; q < KPT; ++q) n += __popcll(__ballot(k[q] >= c));
  return n;
}
template <int KPT>
__device__ __forceinline__ uint32_t wave_kth(const uint32_t (&k)[KPT], int count) {
  uint32_t prefix = 0;
  for (int bit = 31; bit >= 0; --bit) {
    const uint32_t cand = prefix | (1u << bit);
    if (wave_count_ge<KPT>(k, cand) >= count) prefix = cand;
  }
  return prefix;
}

// Wave-level top-b of at most 64 keys (lane = pool position, ascending
// source index): rank by (key desc, position asc); chosen positions in
// ascending order.  Called by one whole wave.
__device__ inline void wave_topb(const uint32_t* keys, int psize, int bsize, int* chosen) {
  const int lane = threadIdx.x & 63;
  const unsigned long long below = (1ull << lane) - 1ull;
  const uint32_t k[1] = {(lane < psize) ? keys[lane] : 0u};
  const uint32_t kth = wave_kth<1>(k, bsize);
  const int quota = bsize - __popcll(__ballot(k[0] > kth));
  const unsigned long long eqm = __ballot(lane < psize && k[0] == kth);
  const bool take = lane < psize && (k[0] > kth || (k[0] == kth && __popcll(eqm & below) < quota));
  const unsigned long long tm = __ballot(take);
  if (take) chosen[__popcll(tm & below)] = lane;
}

// Butterfly transpose-reduction: lane l holds v[0..63] (one value per pool
// position); afterwards v[0] in lane l is the sum over all 64 lanes of the
// values for position l.  63 exchanges, fixed order.
template <int O>
__device__ __forceinline__ void transpose_reduce_step(float* v, int lane) {
  const bool hi = (lane & O) != 0;
#pragma unroll
  for (int k = 0; k < O; ++k) {
    const float send = hi ? v[k] : v[k + O];
    const float keep = hi ? v[k + O] : v[k];
    if constexpr (O < 16) v[k] = keep + xor_lane<O>(send);
    else v[k] = keep + __shfl_xor(send, O, kWave);
  }
}
__device__ __forceinline__ float transpose_reduce64(float* v, int lane) {
  transpose_reduce_step<32>(v, lane);
  transpose_reduce_step<16>(v, lane);
  transpose_reduce_step<8>(v, lane);
  transpose_reduce_step<4>(v, lane);
  transpose_reduce_step<2>(v, lane);
  transpose_reduce_step<1>(v, lane);
  return v[0];
}

// ---------------------------------------------------------------------------
// Persistent selection: every round of a small-pool call in one launch.  The
// grid is nblk blocks per problem, sized to be co-resident (one block per CU,
// two for the streamed kernel when it fits twice); block k owns the tokens
// [k tpb, (k + 1) tpb) and keeps its own copy of the coverage b_m in LDS.  A
// round:
//   gains  - u_i of the block's tokens that may enter the pool, from client
//            rows held in registers for the whole call or streamed from the
//            caches; the block's gains are published together (0 for the
//            other tokens), tagged with the pass over them (a round has a
//            second one if the first left out too many)
//   pool   - every block that owns a row chunk (and the last block) waits
//            for the tagged gains and picks the same pool (identical inputs,
//            deterministic top-k)
//   resp   - one block per 64-row chunk, its waves splitting the pool:
//            responsibility softmax over the pool, per-chunk sums per pool
//            token, published tagged
//   batch  - those blocks wait for the tagged chunk sums, add them in chunk
//            order and pick the same batch; the last block records it and
//            block 0 publishes its tokens, which are all the other blocks
//            wait for (with one chunk per block)
//   cov    - one wave per 64-row chunk: b_m <- max(b_m, max_{j in batch}
//            Cbar_mj), published tagged; every block waits for the tags and
//            copies b into LDS
// In the last round only the last block continues after the batch: it
// refreshes its own coverage copy, writes the coverage, F(S) and F(V), and
// the support list (ascending, with each token's slot).
//
// Hand-off buffers are double-buffered by round parity, so a buffer is
// rewritten two rounds after the round that read it, and the hand-offs
// themselves keep that safe: every block owns a token and publishes gains in
// every round, and its gains of round r + 1 go out only when it has finished
// every read of round r.  A block publishes something of round r + 2 only
// after the complete coverage of round r + 1, which the row owners publish
// after they have seen every block's gains of round r + 1.  So nothing of
// round r is overwritten while a block may still read it, with no barrier,
// no heartbeat and no same-address atomics.  Every wait is
// bounded: after kSpinLimit polls, or once this block has recorded a timeout,
// the block records the timeout (device status word) and stops waiting, so
// every wave always exits.  A round's second pass over the gains counts as a
// round in this: it is published after every read of the first one's gains,
// by the blocks without the pool after block 0's request, which they answer
// before block 0 can publish the batch.
constexpr int kSpinLimit = 1 << 18;   // bounded waits (a fraction of a second)
constexpr int kSumsQ = 16;            // chunk sums in flight per lane
constexpr int kCovQ = 16;             // coverage rows in flight per thread

// Marks the call failed (sticky device status bit) after a bounded wait.
__device__ __forceinline__ void mark_timeout(int* cnt, int* failed) {
  raise_status(cnt, kStatusSelect);
  *failed = 1;
}

// Hand-off words of the gains and the chunk sums: a non-negative float with
// the round's tag in its sign bit.  A word's slot is rewritten every second
// round and holds either that round's value or the one of two rounds before
// (zero before the first), so one alternating bit tells them apart, and half
// the bytes of a value with a tag beside it are polled.  (The coverage keeps
// 8-byte words: with packed ones its hand-off measured 2.4 us a round against
// 1.7 at M = 3344, with or without lines shared between two blocks.)
__device__ __forceinline__ unsigned round_tag(int r) { return ((((r >> 1) & 1) ^ 1) & 1u) << 31; }
__device__ __forceinline__ void st_tagged(uint32_t* p, unsigned tb, float v) {
  __hip_atomic_store(p, (__float_as_uint(v) & 0x7FFFFFFFu) | tb, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t ld_tagged(const uint32_t* p) {
  return __hip_atomic_load(const_cast<uint32_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long ld_tagged2(const uint32_t* p) {
  return ld_dev64(reinterpret_cast<const unsigned long long*>(p));
}
__device__ __forceinline__ bool is_stale(uint32_t w, unsigned tb) { return static_cast<int>(w ^ tb) < 0; }
__device__ __forceinline__ uint32_t low_word(unsigned long long w) { return static_cast<uint32_t>(w); }
__device__ __forceinline__ uint32_t high_word(unsigned long long w) { return static_cast<uint32_t>(w >> 32); }
__device__ __forceinline__ float untagged(uint32_t w) { return __uint_as_float(w & 0x7FFFFFFFu); }

// Sum over the block's four waves of a wave-uniform count (scan: 4 ints, free
// again after the next barrier of the caller).
__device__ __forceinline__ int block_total(int n, int* scan) {
  if ((threadIdx.x & 63) == 0) scan[threadIdx.x >> 6] = n;
  __syncthreads();
  const int t = scan[0] + scan[1] + scan[2] + scan[3];
  __syncthreads();
  return t;
}

// Pool of the persistent selection with the keys in registers: thread t
// takes the gains of its contiguous segment (an even number of tokens, so
// that pairs load together; taken tokens key 0), waiting until each carries
// this round's tag.  LAZY: keys below `floor_key` are left out; false if
// fewer than psize are left.
template <int KPT, bool LAZY>
__device__ __forceinline__ bool pool_regs(const Shape& sh, const uint32_t* tu, unsigned tb,
                                          const unsigned char* taken, int psize, int* pool_s, int* hist, int* scan,
                                          int* cnt, int* failed, uint32_t floor_key, uint32_t* least) {
  static_assert(KPT % 2 == 0, "token pairs");
  const int seg = ((sh.N + 255) / 256 + 1) & ~1;
  const int i0 = threadIdx.x * seg;
  const int last = (sh.N - 1) & ~1;
  unsigned long long w[KPT / 2];
  // pairs past the segment or past N re-read the last pair
  auto at = [&](int q) { return min(2 * q < seg ? i0 + 2 * q : last, last); };
  auto stale = [&](int q) {
    return is_stale(low_word(w[q]), tb) || (at(q) + 1 < sh.N && is_stale(high_word(w[q]), tb));
  };
#pragma unroll
  for (int q = 0; q < KPT / 2; ++q) w[q] = ld_tagged2(&tu[at(q)]);
  bool need[KPT];
#pragma unroll
  for (int q = 0; q < KPT; ++q) need[q] = q < seg && i0 + q < sh.N && !taken[min(i0 + q, sh.N - 1)];
  for (int spin = 0;; ++spin) {
    bool pend = false;
#pragma unroll
    for (int q = 0; q < KPT / 2; ++q) pend |= stale(q);
    if (!pend || *failed) break;
    if (spin == kSpinLimit) { mark_timeout(cnt, failed); break; }
    __builtin_amdgcn_s_sleep(1);
#pragma unroll
    for (int q = 0; q < KPT / 2; ++q)
      if (stale(q)) w[q] = ld_tagged2(&tu[at(q)]);
  }
  uint32_t k[KPT];
#pragma unroll
  for (int q = 0; q < KPT / 2; ++q) {
    k[2 * q] = need[2 * q] ? score_key(untagged(low_word(w[q]))) : 0u;
    k[2 * q + 1] = need[2 * q + 1] ? score_key(untagged(high_word(w[q]))) : 0u;
  }
  if constexpr (LAZY) {
    if (threadIdx.x == 0) *least = 0xFFFFFFFFu;
    if (floor_key) {
      int n = 0;
#pragma unroll
      for (int q = 0; q < KPT; ++q) {
        if (k[q] < floor_key) k[q] = 0u;
        n += __popcll(__ballot(k[q] != 0u));
      }
      if (block_total(n, scan) < psize) return false;
    }
    block_topk_regs<KPT>(k, seg, psize, pool_s, hist, scan, 64, least);
  } else {
    block_topk_regs<KPT>(k, seg, psize, pool_s, hist, scan);
  }
  return true;
}

// A wave-uniform value the compiler cannot see through (so it is not
// hoisted out of a loop): through a VGPR and back.
__device__ __forceinline__ int opaque_uniform(int v) {
  asm volatile("" : "+v"(v));
  return __builtin_amdgcn_readfirstlane(v);
}

// One group of 256 client rows (four consecutive rows per lane) of T tokens:
// acc += max(alpha E - b, 0), row by row, so every token's lane sum has one
// order however its rows are held.
template <int T>
__device__ __forceinline__ void gain_group(const float4 a, const float4 b, const float4 (&v)[T], float (&acc)[T]) {
  float x[T][4];
#pragma unroll
  for (int s = 0; s < T; ++s) {
    x[s][0] = __builtin_fmaf(a.x, v[s].x, -b.x);
    x[s][1] = __builtin_fmaf(a.y, v[s].y, -b.y);
    x[s][2] = __builtin_fmaf(a.z, v[s].z, -b.z);
    x[s][3] = __builtin_fmaf(a.w, v[s].w, -b.w);
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int s = 0; s < T; ++s)
#pragma unroll
    for (int e = 0; e < 4; ++e) x[s][e] = fmaxf(x[s][e], 0.f);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int s = 0; s < T; ++s) acc[s] += x[s][e];
}

// Lane sums of T streamed tokens over ng groups, P groups of rows in flight:
// left to itself the compiler waits for each group's rows before it asks for
// the next, which made a round of the document page 16 us of gains.
// bl: coverage in LDS, zero past M up to 256 ng; AL: the row weights al too,
// else al are the M weights in memory, fetched with the rows.
template <int T, int P, bool AL>
__device__ __forceinline__ void stream_gains(const float* const (&row)[T], const float* al, const float* bl, int ng,
                                             int m_rows, int last, int lane, float (&acc)[T]) {
  float4 buf[P][T], abuf[AL ? 1 : P];
  auto load = [&](int g, int q) {
    const int m = min(g, ng - 1) * 256 + lane * 4, mc = min(m, last);
#pragma unroll
    for (int s = 0; s < T; ++s) buf[q][s] = *reinterpret_cast<const float4*>(row[s] + mc);
    if constexpr (!AL) {
      const float4 a = *reinterpret_cast<const float4*>(al + mc);
      const bool in = m < m_rows;   // (the padding rows after M have weight 0)
      abuf[q] = make_float4(in ? a.x : 0.f, in ? a.y : 0.f, in ? a.z : 0.f, in ? a.w : 0.f);
    }
  };
  auto add = [&](int g, int q) {
    const int m = g * 256 + lane * 4;
    gain_group<T>(AL ? *reinterpret_cast<const float4*>(al + m) : abuf[AL ? 0 : q],
                  *reinterpret_cast<const float4*>(bl + m), buf[q], acc);
  };
#pragma unroll
  for (int q = 0; q < P; ++q) load(q, q);
  // whole rounds of P groups with no exit inside, so the loads in flight at
  // the loop head are the same on every path; the tail's groups are loaded
  const int ng_main = ng - ng % P;
  for (int g = 0; g < ng_main; g += P) {
#pragma unroll
    for (int q = 0; q < P; ++q) {
      add(g + q, q);
      __builtin_amdgcn_sched_barrier(0);
      load(g + q + P, q);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int q = 0; q < P - 1; ++q)
    if (ng_main + q < ng) add(ng_main + q, q);
}

// Gains left out.  b_m only grows, so a token's gain never does (term by term
// and in every rounded partial sum), and the gain it had when it was last
// formed bounds it.  A round forms only the gains whose bound reaches a
// threshold theta that every block knows; the others go out as zero.  If at
// least a pool's worth of gains reach theta the pool is the one that all
// gains would give; else the round's gains are formed once more, all of them.
// The first round, and a call that traces its gains, form all; so do the
// kernels whose blocks hold all their tokens, as a wave forms the held ones
// together: with some left out nothing is saved and the rounds that go again
// are lost (M = 6928: 458 us a call with all gains, 482 so; M = 4692,
// N = 2580: 769 and 810).
// theta lies below the smallest gain of the last pool by twice the part that
// this fell by in the last round: of the document page's 52 rounds 4 go again
// and 12 % of the gains are formed, with a fixed 0.8 12 rounds and 18 %.  Per
// call, all gains against these: the document page 1641 and 1469 us, 16
// problems of 1296 tokens 1228 and 1148.
constexpr int kLazyList = 768;    // listed tokens at a time (the words of hist)
constexpr int kLazyAgain = 62, kLazyTheta = 63;   // words of tp beside the batch
__device__ __forceinline__ float next_threshold(float cut, float last_cut, int r) {
  const float fall = r > 0 && last_cut > 0.f ? cut / last_cut : 0.8f;
  const float t = cut * fminf(fmaxf(2.f * fall - 1.f, 0.f), 0.95f);
  return t > 0.f && t < 3e38f ? t : 0.f;   // (no threshold from infinite gains)
}

// RES: eight tokens per block (N <= 8 blocks, M <= 256 kResJ) whose weighted
// client rows alpha_m E[i][m] (Cbar, the product rounded once) stay in
// registers for the whole call, wave w holding the rows
// m = 64 (w + 4 j) + lane, j < kResJ, of all eight tokens; a round's gains
// then read only the coverage.
// R > 0: the rows of each wave's first R tokens stay in registers, up to 256 J
// rows each; a round's gains read weights and coverage from LDS (measured at
// M = 6928, two tokens a wave: 2.2 us of gains a round, 12 us streamed).
// Tokens beyond them, or all with R = 0, are streamed from the caches (S; not
// S: the block has at most 4 R tokens).
constexpr int kResJ = 14;
template <bool RES, int J, int R, int PF, bool AL = true, bool S = true>
__device__ __forceinline__ void select_rounds(const Shape& sh, const Params& pr, const Ws& ws, int nblk,
                                              const SelOut& so, const SelTurn& turn) {
  extern __shared__ __attribute__((aligned(16))) float dyn[];
  // LDS: b_m [mp] | alpha_m [mp] (AL, not with RES) | selected flags [N, padded to
  // 16 bytes] | the block's gains [tpb] | pool keys [N] (only when N exceeds
  // the register top-k)
  // the block owns the tokens [t0, t0 + tpb); its wave w those at 4 s + w
  const int tpb = RES ? 8 : (sh.N + nblk - 1) / nblk, t0 = static_cast<int>(blockIdx.x) * tpb;
  const int ng = (sh.m + 255) / 256, mp = RES ? sh.ldM : 256 * (R > 0 ? J : ng);
  float* bl = dyn;
  float* al = dyn + mp;   // with AL and not with RES
  unsigned char* taken = reinterpret_cast<unsigned char*>(dyn + (RES || !AL ? 1 : 2) * mp);
  float* gsum = reinterpret_cast<float*>(taken + ((sh.N + 15) & ~15));   // the block's gains [tpb], not with RES
  uint32_t* keys = reinterpret_cast<uint32_t*>(gsum + tpb);
  __shared__ int hist[768], scan[16], bc[2], failed, rank_s[4][64];
  __shared__ int pool_s[64], chosen[64], bidx[64];
  __shared__ float rmu[4][64], rden_s[4][64], red[16];
  // gains left out of a round (not with RES): see next_threshold
  constexpr bool LAZY = !RES && S;
  __shared__ float theta_s;
  __shared__ uint32_t cut_s;
  __shared__ int again_s, nlist_s;
  // Cbar of the chunk's rows at the pool's tokens (pool position, row lane),
  // kept from the responsibilities for the coverage refresh
  __shared__ float cpool[64][64];
  const int p = blockIdx.y, blk = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nchunk = (sh.m + 63) / 64;
  // the pool and the chunk sums are needed by the blocks that own a row
  // chunk (responsibilities, coverage) and by the last block (it records the
  // batch); with one chunk per block the others skip both and wait only for
  // the batch's tokens, which block 0 publishes after its pick
  const bool pool_here = nchunk > nblk || blk < nchunk || blk == nblk - 1;
  const bool pool_pub = nchunk + 1 < nblk;
  const float* E = ws.E + p * ws.s_E;
  uint32_t* tu = ws.tu + p * ws.s_tu;
  uint32_t* ts = ws.ts + p * ws.s_ts;
  unsigned long long* tc = ws.tc + p * ws.s_tc;
  const float* alpha_g = ws.alpha + p * ws.s_m;
  int* cnt = ws.cnt + p * ws.s_cnt;
  {
    const float* cov0 = ws.cov + p * ws.s_cov;
    for (int m = tid; m < mp; m += 256) {
      // coverage at the first round: zero, or the image seeds' b_m(S_0);
      // rows past M are zero in both arrays
      bl[m] = sh.nseed > 0 && m < sh.m ? cov0[m] : 0.f;
      if constexpr (!RES && AL) al[m] = m < sh.m ? alpha_g[m] : 0.f;
    }
  }
  {
    const int* sel0 = ws.sel + p * ws.s_sel;
    for (int i = tid; i < sh.N; i += 256) taken[i] = (sh.nseed > 0 && sel0[i] >= 0) ? 1 : 0;
  }
  if (tid == 0) failed = 0;
  float er[RES ? 8 : 1][RES ? kResJ : 1];
  if constexpr (RES) {
    // rows past M and tokens past N hold zeros (clamped loads, then select)
#pragma unroll
    for (int j = 0; j < kResJ; ++j) {
      const int m = 64 * (wave + 4 * j) + lane;
      const int mc = min(m, sh.m - 1);
      const float a = alpha_g[mc];
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const int t = blk * 8 + s;
        const float v = E[static_cast<long long>(min(t, sh.N - 1)) * sh.ldM + mc];
        er[s][j] = (m < sh.m && t < sh.N) ? a * v : 0.f;
      }
    }
  }
  float4 hold[R > 0 ? R : 1][R > 0 ? J : 1];
  if constexpr (R > 0) {
    // the wave's first R tokens, lane-strided like the streamed rows; groups
    // past M (clamped loads) meet zero weights
#pragma unroll
    for (int s = 0; s < R; ++s) {
      const int t = t0 + min(4 * s + wave, tpb - 1);
      const float* row = E + static_cast<long long>(min(t, sh.N - 1)) * sh.ldM;
#pragma unroll
      for (int j = 0; j < J; ++j) {
        const int m = 256 * j + lane * 4;
        hold[s][j] = *reinterpret_cast<const float4*>(row + min(m, sh.ldM - 4));
      }
    }
  }
  __syncthreads();
  int selected = sh.nseed;
  const Shape sh_call = sh;
  const int tid_call = tid;
  // a trace asks for every gain; a batch above 62 leaves tp no words for the
  // threshold and the request to go again
  const bool lazy = LAZY && so.gains == nullptr && sh.b <= kLazyAgain;
  float theta = 0.f, cut = 0.f;
  for (int r = 0, it = 0; r < sh_call.rounds; ++it) {
    // Opaque per-round copies of the shape and the thread index: index math
    // derived from them is redone every round instead of being hoisted out
    // of the loop and kept live (in spill registers) across all rounds.
    Shape sh = sh_call;
    int tid = tid_call;
    sh.N = opaque_uniform(sh.N);
    sh.m = opaque_uniform(sh.m);
    sh.ldM = opaque_uniform(sh.ldM);
    sh.K = opaque_uniform(sh.K);
    sh.b = opaque_uniform(sh.b);
    sh.pool_cap = opaque_uniform(sh.pool_cap);
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = tid >> 6;
    const int psize = min(sh.pool_cap, sh.N - selected);
    const int bsize = min(sh.b, sh.K - selected);
    const unsigned tag = static_cast<unsigned>(r + 1);
    unsigned long long picked = 0;   // pool positions of the batch
    const unsigned tb = round_tag(r), tbu = round_tag(it);
    uint32_t* tur = tu + (it & 1) * handoff_stride(sh.N);
    // whether the block's token l (at t0 + l) needs its gain now
    auto needs = [&](int l) {
      return l < tpb && t0 + l < sh.N && !taken[t0 + l] && (theta <= 0.f || gsum[l] >= theta);
    };
    uint32_t* tsr = ts + (r & 1) * 64LL * nchunk;

    // ---- singleton gains of unselected tokens, two tokens per wave pass with
    //      all their row loads in flight (or the block's rows held in registers),
    //      published with this round's tag
    if constexpr (RES) {
      // per lane: the partial gains of the eight tokens over its rows
      // (b_m >= 0, so rows past M add zero); then summed over the lanes and
      // the four waves, in that order
      float acc[8];
#pragma unroll
      for (int s = 0; s < 8; ++s) acc[s] = 0.f;
#pragma unroll
      for (int j = 0; j < kResJ; ++j) {
        const float b = bl[min(64 * (wave + 4 * j) + lane, sh.ldM - 1)];
#pragma unroll
        for (int s = 0; s < 8; ++s) acc[s] += fmaxf(er[s][j] - b, 0.f);
      }
      transpose_reduce_step<4>(acc, lane);
      transpose_reduce_step<2>(acc, lane);
      transpose_reduce_step<1>(acc, lane);
      float g = acc[0];             // token lane & 7, summed over 8 lanes
      g += xor_lane<8>(g);
      g = add_xor16(g);
      g = add_xor32(g);
      if (lane < 8) rmu[wave][lane] = g;
      __syncthreads();
      if (tid < 8) {
        const int t = blk * 8 + tid;
        const float g = ((rmu[0][tid] + rmu[1][tid]) + rmu[2][tid]) + rmu[3][tid];
        const float u = t < sh.N && !taken[t] ? g : 0.f;
        if (t < sh.N) st_tagged(&tur[t], tbu, u);
        if (so.gains && t < sh.N) so.gains[(static_cast<long long>(p) * sh.rounds + r) * sh.N + t] = u;
      }
    }
    if constexpr (R > 0) {
      // the held tokens: each sum is formed exactly as for a streamed token
      bool any = false;
#pragma unroll
      for (int s = 0; s < R; ++s) any |= needs(4 * s + wave);
      if (!LAZY || __any(any)) {
      float acc[R];
#pragma unroll
      for (int s = 0; s < R; ++s) acc[s] = 0.f;
      // the weights and coverage of the next groups are read ahead
      constexpr int D = 4;
      float4 a[D], b[D];
#pragma unroll
      for (int j = 0; j < D && j < J; ++j) {
        a[j] = *reinterpret_cast<const float4*>(al + j * 256 + lane * 4);
        b[j] = *reinterpret_cast<const float4*>(bl + j * 256 + lane * 4);
      }
#pragma unroll
      for (int j = 0; j < J; ++j) {
        float4 v[R];
#pragma unroll
        for (int s = 0; s < R; ++s) v[s] = hold[s][j];
        gain_group<R>(a[j % D], b[j % D], v, acc);
        if (j + D < J) {
          a[j % D] = *reinterpret_cast<const float4*>(al + (j + D) * 256 + lane * 4);
          b[j % D] = *reinterpret_cast<const float4*>(bl + (j + D) * 256 + lane * 4);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int s = 0; s < R; ++s) acc[s] = wave_sum(acc[s]);
      if (lane == 0)
#pragma unroll
        for (int s = 0; s < R; ++s)
          if (4 * s + wave < tpb) gsum[4 * s + wave] = acc[s];
      }
    }
    if constexpr (!RES) {
      // the block's other tokens that need a gain, listed by its first wave
      // and dealt to the waves, T at a time
      int* list = hist;   // free between the pools
      for (int w0 = 4 * R; S && w0 < tpb; w0 += kLazyList) {
        const int w1 = min(tpb, w0 + kLazyList);
        if (wave == 0) {
          int n = 0;
          for (int l0 = w0; l0 < w1; l0 += 64) {
            const int l = l0 + lane;
            const bool nd = l < w1 && needs(l);
            const unsigned long long mask = __ballot(nd);
            if (nd) list[n + __popcll(mask & ((1ull << lane) - 1ull))] = l;
            n += __popcll(mask);
          }
          if (lane == 0) nlist_s = n;
        }
        __syncthreads();
        const int n = __builtin_amdgcn_readfirstlane(nlist_s);
        auto pass = [&](auto tt, int s0) {
          constexpr int T = decltype(tt)::value;
          int l[T];
          const float* row[T];
          float acc[T];
#pragma unroll
          for (int k = 0; k < T; ++k) {
            // past the list's end its last token again (cache hits)
            l[k] = __builtin_amdgcn_readfirstlane(list[min(4 * (s0 + k) + wave, n - 1)]);
            row[k] = E + static_cast<long long>(t0 + l[k]) * sh.ldM;
            acc[k] = 0.f;
          }
          stream_gains<T, T == 4 ? PF : T == 2 ? 2 * PF : 4 * PF, AL>(row, AL ? al : alpha_g, bl, ng, sh.m, sh.ldM - 4,
                                                                     lane, acc);
#pragma unroll
          for (int k = 0; k < T; ++k) acc[k] = wave_sum(acc[k]);
          if (lane == 0)
#pragma unroll
            for (int k = 0; k < T; ++k)
              if (4 * (s0 + k) + wave < n) gsum[l[k]] = acc[k];
        };
        const int ns = (n - wave + 3) / 4;   // the wave's tokens
        int s0 = 0;
        if constexpr (R == 0)
          for (; s0 + 2 < ns; s0 += 4) pass(std::integral_constant<int, 4>{}, s0);
        for (; s0 + 1 < ns; s0 += 2) pass(std::integral_constant<int, 2>{}, s0);
        if (s0 < ns) pass(std::integral_constant<int, 1>{}, s0);
        if (w1 < tpb) __syncthreads();   // the list is rewritten
      }
      // the block's gains leave together: its words share cache lines with
      // few other blocks, and stores to one line from several XCDs serialise
      __syncthreads();
      for (int l = tid; l < tpb; l += 256) {
        const int t = t0 + l;
        if (t >= sh.N) break;
        const float u = !taken[t] && (!LAZY || gsum[l] >= theta) ? gsum[l] : 0.f;
        st_tagged(&tur[t], tbu, u);
        if (so.gains) so.gains[(static_cast<long long>(p) * sh.rounds + r) * sh.N + t] = u;
      }
    }

    // ---- the pool, identical in every block that needs it (waits for this
    //      round's gains)
    // the batch's tokens, published by block 0 for the blocks without the pool
    unsigned long long* tpr = ws.tp + p * ws.s_tp + (r & 1) * 64;
    const uint32_t floor_key = LAZY && theta > 0.f ? score_key(theta) : 0u;
    float theta_next = 0.f;
    if (pool_here) {
    bool whole = true;   // the pool is certain
    if constexpr (RES) {
      if (sh.N <= 256 * 6)
        pool_regs<6, LAZY>(sh, tur, tbu, taken, psize, pool_s, hist, scan, cnt, &failed, 0u, nullptr);
      else
        pool_regs<8, LAZY>(sh, tur, tbu, taken, psize, pool_s, hist, scan, cnt, &failed, 0u, nullptr);
    } else if (sh.N <= 256 * 8)
      whole = pool_regs<8, LAZY>(sh, tur, tbu, taken, psize, pool_s, hist, scan, cnt, &failed, floor_key, &cut_s);
    else if (sh.N <= 256 * 16)
      whole = pool_regs<16, LAZY>(sh, tur, tbu, taken, psize, pool_s, hist, scan, cnt, &failed, floor_key, &cut_s);
    else {
      int n = 0;
      if (tid == 0) cut_s = 0xFFFFFFFFu;
      for (int base = 0; base < sh.N; base += 256 * 16) {
        unsigned long long w[8];
        auto at = [&](int q) { return min(base + 2 * (q * 256 + tid), (sh.N - 1) & ~1); };
        auto stale = [&](int q) {
          return is_stale(low_word(w[q]), tbu) || (at(q) + 1 < sh.N && is_stale(high_word(w[q]), tbu));
        };
#pragma unroll
        for (int q = 0; q < 8; ++q) w[q] = ld_tagged2(&tur[at(q)]);
        for (int spin = 0;; ++spin) {
          bool pend = false;
#pragma unroll
          for (int q = 0; q < 8; ++q) pend |= stale(q);
          if (!pend || failed) break;
          if (spin == kSpinLimit) { mark_timeout(cnt, &failed); break; }
          __builtin_amdgcn_s_sleep(1);
#pragma unroll
          for (int q = 0; q < 8; ++q)
            if (stale(q)) w[q] = ld_tagged2(&tur[at(q)]);
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const int i = base + 2 * (q * 256 + tid);
          uint32_t k0 = i < sh.N && !taken[i] ? score_key(untagged(low_word(w[q]))) : 0u;
          uint32_t k1 = i + 1 < sh.N && !taken[i + 1] ? score_key(untagged(high_word(w[q]))) : 0u;
          k0 = k0 < floor_key ? 0u : k0;
          k1 = k1 < floor_key ? 0u : k1;
          n += __popcll(__ballot(k0 != 0u)) + __popcll(__ballot(k1 != 0u));
          if (i < sh.N) keys[i] = k0;
          if (i + 1 < sh.N) keys[i + 1] = k1;
        }
      }
      whole = block_total(n, scan) >= psize || floor_key == 0u;   // (the keys are in LDS)
      if (whole) {
        block_topk256(keys, sh.N, psize, pool_s, hist, scan, bc);
        if (tid < psize) atomicMin(&cut_s, keys[pool_s[tid]]);
      }
    }
    if constexpr (LAZY) {
      if (!whole && !failed) {
        // too few gains reached the threshold: once more with all of them
        if (pool_pub && blk == 0 && tid == 0) st_dev64(&tpr[kLazyAgain], tag_value(tag, 0.f));
        theta = 0.f;
        continue;
      }
    }
    if constexpr (!RES) {
      // clamp to valid rows (defensive) and pad past psize with a valid row,
      // masked below (the register top-k pads with row 0 itself)
      int pv = 0;
      if (tid < 64) pv = min(max(pool_s[tid < psize ? tid : 0], 0), sh.N - 1);
      __syncthreads();
      if (tid < 64) pool_s[tid] = pv;
      __syncthreads();
    }
    if constexpr (LAZY) {
      const float last_cut = cut;
      cut = __uint_as_float(cut_s - 1u);
      theta_next = lazy ? next_threshold(cut, last_cut, r) : 0.f;
    }
    }
    if (blk == nblk - 1 && so.pool) {
      int32_t* tp = so.pool + (static_cast<long long>(p) * sh.rounds + r) * sh.pool_cap;
      for (int j = tid; j < sh.pool_cap; j += 256) tp[j] = (j < psize) ? pool_s[j] : -1;
    }

    // ---- responsibilities: one block per 64-row chunk (lane = client row),
    //      its four waves split the pool positions 16 apiece; the per-chunk
    //      sums are published with this round's tag
    for (int c = blk; c < nchunk; c += nblk) {
      const int m = c * 64 + lane;
      const bool row_ok = m < sh.m;
      const int mc = row_ok ? m : 0;
      const float a = row_ok ? alpha_g[mc] : 0.f;
      const float b = bl[mc];
      const int j0 = wave * 16;
      float v[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) v[j] = E[static_cast<long long>(pool_s[j0 + j]) * sh.ldM + mc];
      float mu = 0.f;
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const float cb = a * v[j];
        cpool[j0 + j][lane] = cb;
        const float rr = (j0 + j < psize) ? fmaxf(cb - b, 0.f) : 0.f;
        v[j] = rr;
        mu = fmaxf(mu, rr);
      }
      rmu[wave][lane] = mu;
      __syncthreads();
      mu = fmaxf(fmaxf(rmu[0][lane], rmu[1][lane]), fmaxf(rmu[2][lane], rmu[3][lane]));
      const float inv = mu > 0.f ? 1.f / (pr.tau_r * mu + pr.resp_eps) : 0.f;
      const float zmax = mu * inv;
      float den = 0.f;
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const float ex = (j0 + j < psize) ? __expf(v[j] * inv - zmax) : 0.f;
        den += ex;
        v[j] *= ex;    // rho numerator times R; scaled by 1/den below
      }
      rden_s[wave][lane] = den;
      __syncthreads();
      den = ((rden_s[0][lane] + rden_s[1][lane]) + rden_s[2][lane]) + rden_s[3][lane];
      const float rden = mu > 0.f ? 1.f / den : 0.f;
#pragma unroll
      for (int j = 0; j < 16; ++j) v[j] *= rden;
      // sum over the 64 rows per pool position: butterfly inside 16-lane
      // groups, then across the four groups
      transpose_reduce_step<8>(v, lane);
      transpose_reduce_step<4>(v, lane);
      transpose_reduce_step<2>(v, lane);
      transpose_reduce_step<1>(v, lane);
      float tot = v[0];
      tot = add_xor16(tot);
      tot = add_xor32(tot);
      if (lane < 16) st_tagged(&tsr[static_cast<long long>(c) * 64 + j0 + lane], tb, tot);
      __syncthreads();   // rmu / rden_s are reused by the next chunk
    }

    // ---- the batch, identical in every block with the pool: each wave waits
    //      for the tagged sums of a quarter of the chunks (16 loads in
    //      flight) and adds them in chunk order; the quarters are added in
    //      wave order.  The other blocks wait for the batch's tokens alone.
    if (!pool_here) {
      // nothing left for these blocks in the last round, unless its gains may
      // be asked for once more
      if (r + 1 == sh.rounds && (!LAZY || theta <= 0.f)) break;
      if (wave == 0) {
        const bool mine = lane < bsize || (lazy && lane == kLazyTheta);
        const bool poll = mine || (theta > 0.f && lane == kLazyAgain);
        unsigned long long bw = poll ? ld_dev64(&tpr[lane]) : 0ull;
        bool again = false;
        for (int spin = 0;; ++spin) {
          again = LAZY && __any(theta > 0.f && lane == kLazyAgain && tag_of(bw) == tag);
          if (again || !__any(mine && tag_of(bw) != tag) || failed) break;
          if (spin == kSpinLimit) { mark_timeout(cnt, &failed); break; }
          __builtin_amdgcn_s_sleep(1);
          if (poll && tag_of(bw) != tag) bw = ld_dev64(&tpr[lane]);
        }
        if constexpr (LAZY) {
          if (lane == 0) again_s = again ? 1 : 0;
          if (lane == kLazyTheta) theta_s = lazy ? value_of(bw) : 0.f;
        }
        if (lane < bsize && !again) {
          const int i = min(max(__float_as_int(value_of(bw)), 0), sh.N - 1);
          bidx[lane] = i;
          taken[i] = 1;
        }
      }
      __syncthreads();
      if constexpr (LAZY) {
        if (again_s) {
          theta = 0.f;
          continue;
        }
        theta_next = theta_s;
      }
    } else {
    {
      const int per = (nchunk + 3) / 4;
      const int c_end = min(nchunk, (wave + 1) * per);
      float s = 0.f;
      for (int c0 = wave * per; c0 < c_end; c0 += kSumsQ) {
        uint32_t w[kSumsQ];
#pragma unroll
        for (int q = 0; q < kSumsQ; ++q) w[q] = ld_tagged(&tsr[static_cast<long long>(min(c0 + q, c_end - 1)) * 64 + lane]);
        for (int spin = 0;; ++spin) {
          bool pend = false;
#pragma unroll
          for (int q = 0; q < kSumsQ; ++q) pend |= is_stale(w[q], tb);
          if (!pend || failed) break;
          if (spin == kSpinLimit) { mark_timeout(cnt, &failed); break; }
          __builtin_amdgcn_s_sleep(1);
#pragma unroll
          for (int q = 0; q < kSumsQ; ++q)
            if (is_stale(w[q], tb)) w[q] = ld_tagged(&tsr[static_cast<long long>(min(c0 + q, c_end - 1)) * 64 + lane]);
        }
#pragma unroll
        for (int q = 0; q < kSumsQ; ++q)
          if (c0 + q < c_end) s += untagged(w[q]);
      }
      rmu[wave][lane] = s;   // free: the responsibility loop ended with a barrier
    }
    __syncthreads();
    {
      // top-b of the pool by (score, lower position): a position's rank is
      // the number of positions that go before it; each wave counts against
      // its 16 positions, the counts meet in LDS
      const float s = ((rmu[0][lane] + rmu[1][lane]) + rmu[2][lane]) + rmu[3][lane];
      if (blk == nblk - 1 && so.scores && wave == 0 && lane < sh.pool_cap)
        so.scores[(static_cast<long long>(p) * sh.rounds + r) * sh.pool_cap + lane] = lane < psize ? s : 0.f;
      const uint32_t key = lane < psize ? score_key(s) : 0u;
      int rank = 0;
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const int j = wave * 16 + q;
        const uint32_t kj = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(key), j));
        rank += (kj > key || (kj == key && j < lane)) ? 1 : 0;
      }
      rank_s[wave][lane] = rank;
      __syncthreads();
      rank = (rank_s[0][lane] + rank_s[1][lane]) + (rank_s[2][lane] + rank_s[3][lane]);
      const bool take = lane < psize && rank < bsize;
      picked = __ballot(take);
      if (wave == 0 && take) {
        const int k = __popcll(picked & ((1ull << lane) - 1ull));
        const int i = pool_s[lane];
        chosen[k] = lane;
        bidx[k] = i;
        taken[i] = 1;
        if (pool_pub && blk == 0) st_dev64(&tpr[k], tag_value(tag, __int_as_float(i)));
      }
      if (lazy && pool_pub && blk == 0 && tid == kLazyTheta) st_dev64(&tpr[kLazyTheta], tag_value(tag, theta_next));
    }
    }
    const bool last = r + 1 == sh.rounds;
    // the last block records the batch (and alone finishes the last round)
    if (blk == nblk - 1) {
      __syncthreads();   // chosen and bidx are in LDS
      commit_batch(sh, ws, p, r, bsize, selected, pool_s, chosen, so.batch);
    } else if (last) {
      break;
    }
    if (!last) {
      // ---- coverage refresh with the batch, published with this round's
      //      tag: with one chunk per block, by the chunk's responsibility
      //      block (its pool columns, the batch among them, were just read
      //      here), wave w taking the picked ones of its 16 pool positions;
      //      otherwise one wave per 64-row chunk
      unsigned long long* tcr = tc + (r & 1) * handoff_stride(sh.m);
      if (nchunk <= nblk) {
        if (blk < nchunk) {
          const int m = blk * 64 + lane;
          // the batch's Cbar values were kept in LDS by this block's
          // responsibility pass over the same rows
          float cm = bl[min(m, sh.m - 1)];
          unsigned mine = static_cast<unsigned>(picked >> (16 * wave)) & 0xFFFFu;
          while (mine) {
            const int j = __builtin_ctz(mine);
            mine &= mine - 1;
            cm = fmaxf(cm, cpool[16 * wave + j][lane]);
          }
          rmu[wave][lane] = cm;   // free: last read before the barrier after the ranks
          __syncthreads();
          if (wave == 0 && m < sh.m)
            st_dev64(&tcr[m], tag_value(tag, fmaxf(fmaxf(rmu[0][lane], rmu[1][lane]), fmaxf(rmu[2][lane], rmu[3][lane]))));
        }
      } else {
        __syncthreads();   // bidx is in LDS
        for (int c = blk * 4 + wave; c < nchunk; c += 4 * nblk) {
          const int m = c * 64 + lane;
          const int mc = min(m, sh.m - 1);
          const float a = alpha_g[mc];
          float cm = bl[mc];
          for (int k0 = 0; k0 < bsize; k0 += 16) {
            float v[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) v[q] = E[static_cast<long long>(bidx[min(k0 + q, bsize - 1)]) * sh.ldM + mc];
#pragma unroll
            for (int q = 0; q < 16; ++q) cm = fmaxf(cm, a * v[q]);
          }
          if (m < sh.m) st_dev64(&tcr[m], tag_value(tag, cm));
        }
      }
      // ---- every block copies the refreshed coverage into LDS, waiting for
      //      the tags
      for (int m0 = 0; m0 < sh.m; m0 += 256 * kCovQ) {
        unsigned long long w[kCovQ];
#pragma unroll
        for (int q = 0; q < kCovQ; ++q) w[q] = ld_dev64(&tcr[min(m0 + q * 256 + tid, sh.m - 1)]);
        for (int spin = 0;; ++spin) {
          bool pend = false;
#pragma unroll
          for (int q = 0; q < kCovQ; ++q) pend |= tag_of(w[q]) != tag;
          if (!pend || failed) break;
          if (spin == kSpinLimit) { mark_timeout(cnt, &failed); break; }
          __builtin_amdgcn_s_sleep(1);
#pragma unroll
          for (int q = 0; q < kCovQ; ++q)
            if (tag_of(w[q]) != tag) w[q] = ld_dev64(&tcr[min(m0 + q * 256 + tid, sh.m - 1)]);
        }
#pragma unroll
        for (int q = 0; q < kCovQ; ++q)
          if (m0 + q * 256 + tid < sh.m) bl[m0 + q * 256 + tid] = value_of(w[q]);
      }
      __syncthreads();
      selected += bsize;
      theta = theta_next;
      ++r;
      continue;
    }

    // ---- the last round (last block only): coverage refresh of the LDS copy
    //      with two row groups per trip, 16 batch rows each, all loads in flight
    for (int m0 = tid * 4; m0 < sh.m; m0 += 2048) {
      float4 c[2];
      c[0] = c[1] = make_float4(0.f, 0.f, 0.f, 0.f);
      for (int k0 = 0; k0 < bsize; k0 += 16) {
        // indices past the batch repeat its last row: a maximum is unchanged
        float4 v[2][16];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int q = 0; q < 16; ++q)
            v[h][q] = *reinterpret_cast<const float4*>(E + static_cast<long long>(bidx[min(k0 + q, bsize - 1)]) * sh.ldM +
                                                       min(m0 + h * 1024, sh.ldM - 4));
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int q = 0; q < 16; ++q) {
            c[h].x = fmaxf(c[h].x, v[h][q].x); c[h].y = fmaxf(c[h].y, v[h][q].y);
            c[h].z = fmaxf(c[h].z, v[h][q].z); c[h].w = fmaxf(c[h].w, v[h][q].w);
          }
      }
      // alpha_m >= 0, so alpha_m max_j Et[j][m] = max_j Cbar_mj exactly
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int m = m0 + h * 1024;
        if (m < sh.m) {
          const float4 a = *reinterpret_cast<const float4*>(alpha_g + m);
          float4 b = *reinterpret_cast<const float4*>(bl + m);
          b.x = fmaxf(b.x, a.x * c[h].x); b.y = fmaxf(b.y, a.y * c[h].y);
          b.z = fmaxf(b.z, a.z * c[h].z); b.w = fmaxf(b.w, a.w * c[h].w);
          *reinterpret_cast<float4*>(bl + m) = b;
        }
      }
    }
    selected += bsize;
    __syncthreads();
    if (last) {
      // the last block: the coverage, F(S) = sum_m b_m and F(V) = sum_m
      // max_i Cbar_mi, then the support list in ascending source order with
      // each token's slot
      float* cov = ws.cov + p * ws.s_cov;
      const float* peak = ws.peak + p * ws.s_m;
      float fs = 0.f, fv = 0.f;
      for (int m = tid; m < sh.m; m += 256) {
        cov[m] = bl[m];
        fs += bl[m];
        fv += peak[m];
      }
      fs = block_sum(fs, red);
      fv = block_sum(fv, red);
      int* sup = ws.sup + p * ws.s_sup;
      int* slot = ws.slot + p * ws.s_slot;
      int base = 0;
      for (int b0 = 0; b0 < sh.N; b0 += 256) {
        const int i = b0 + tid;
        const int f = (i < sh.N && taken[i]) ? 1 : 0;
        int tot;
        const int pos = base + block_exclusive_scan(f, scan, &tot);
        if (i < sh.N) {
          slot[i] = f ? pos : -1;
          if (f) sup[pos] = i;
        }
        base += tot;
      }
      if (tid == 0) {
        float* st = ws.stats + p * ws.s_st;
        st[2] = fs;
        st[3] = fv;
        st[4] = static_cast<float>(sh.K);
        st[5] = static_cast<float>(sh.rounds);
        st[6] = static_cast<float>(sh.m);
        st[7] = static_cast<float>(sh.N - sh.K);
        problem_done(turn);
      }
      break;
    }
  }
}

// Streamed rows only.
static __global__ void __launch_bounds__(256)
select_stream_kernel(Shape sh, Params pr, Ws ws, int nblk, SelOut so, SelTurn turn) {
  select_rounds<false, 0, 0, 4>(sh, pr, ws, nblk, so, turn);
}
// The same with the row weights read from memory, for more rows than both
// arrays fit in LDS.
static __global__ void __launch_bounds__(256)
select_wide_kernel(Shape sh, Params pr, Ws ws, int nblk, SelOut so, SelTurn turn) {
  select_rounds<false, 0, 0, 2, false>(sh, pr, ws, nblk, so, turn);
}
// Eight tokens per block, rows split over its waves.
static __global__ void __launch_bounds__(256)
select_split_kernel(Shape sh, Params pr, Ws ws, int nblk, SelOut so, SelTurn turn) {
  select_rounds<true, 0, 0, 4>(sh, pr, ws, nblk, so, turn);
}
// What a selection block may share a CU with (512 registers a SIMD lane, 160
// KB of LDS): the gate block of the context's next call (its four waves, one
// per SIMD, at most kGateRegs) and either a selection of the other entry point
// (both then at most kHalfRegs, with LDS for both) or a wave of that entry point
// that waits for its turn: the static call's first kernel (kWaitRegs, beside at
// most kWholeRegs) or the context's last message kernel (beside a static
// selection, at most kHalfRegs and kHalfLdsStatic).  The resource tests hold
// the built kernels to these.
constexpr int kGateRegs = 24, kWaitRegs = 16, kHalfRegs = 240, kWholeRegs = 472;
constexpr int kSelStaticLds = 23552, kHalfLds = 44 * 1024, kHalfLdsStatic = 112 * 1024;
constexpr bool hold_half(int J, int R, bool S) { return !S && J * R <= 20; }

// R tokens of up to 256 J client rows held per wave.  One wave per SIMD, so
// up to 512 registers, but J R is kept near 75 (see kWholeRegs).
template <int J, int R, bool S>
static __global__ void __attribute__((amdgpu_flat_work_group_size(256, 256), amdgpu_waves_per_eu(1, 1)))
select_hold_kernel(Shape sh, Params pr, Ws ws, int nblk, SelOut so, SelTurn turn) {
  select_rounds<false, J, R, 2, true, S>(sh, pr, ws, nblk, so, turn);
}

}  // namespace gmc
