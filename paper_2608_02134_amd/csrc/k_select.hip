// Batched responsibility selection (Sec. 3.3 Eq. coverage, Eq.
// responsibility; App. H Eq. cond-responsibility and the totality rule).
//
// The client energies are stored token-major, Et[i][m] (row stride ldM), and
// Cbar_mi = alpha_m Et[i][m] is formed on the fly.  Token-major makes every
// token's singleton gain u_i = sum_m [Cbar_mi - b_m]_+ one contiguous
// reduction owned by a single wave, so no cross-block partial sums exist.
// One round:
//   cov   - b_m <- max(b_m, max_{j in previous batch} Cbar_mj), rows in parallel,
//           batch columns split over blocks; in-place atomicMax on the bit
//           pattern (non-negative floats order like their bits), so the
//           result is independent of arrival order
//   gains - u_i per token; the last block picks the pool, the min(4b, N-|S|)
//           largest gains of unselected tokens (ties to the lower index)
//   resp  - pool of at most 64: one lane per client row computes the
//           responsibility softmax of R over the pool and its contributions
//           rho R; a butterfly transpose-reduction sums them per pool token;
//           the last block adds the block sums in order and picks the batch.
//           Larger pools (bounded path): per-row max and softmax denominator
//           first (rowstat), then one wave per pool token sums its column
//           (colsum), the last block picks the batch.
// Every reduction has a fixed order, so results are bitwise repeatable.
// Zero-gain tokens key just above excluded ones, so once gains vanish the
// lowest source indices fill the budget.
#include <mutex>

#include "gmc_device.h"
#include "gmc_internal.h"
#include "gmc_kernels.h"
#include "gmc_occupancy.h"
#include "gmc_select.h"

namespace gmc {

constexpr int kCpw = 4;                 // gains kernel: tokens per wave
constexpr int kGainCols = 4 * kCpw;     // tokens per block
constexpr int kCpwF = 4;                // fused gains kernel: tokens per wave
constexpr int kGainColsF = 4 * kCpwF;
constexpr int kLdsKeys = 12288;         // pool top-k keys live in LDS up to this N


// ---------------------------------------------------------------------------
// coverage refresh with a batch
// ---------------------------------------------------------------------------
constexpr int kCovCols = 32;   // batch columns per block

__global__ void __launch_bounds__(256) cov_kernel(Shape sh, Ws ws, int nb) {
  const int p = blockIdx.z, m = blockIdx.x * 256 + threadIdx.x;
  if (m >= sh.m) return;
  const int j0 = blockIdx.y * kCovCols, j1 = min(nb, j0 + kCovCols);
  const float a = ws.alpha[p * ws.s_m + m];
  const int* bat = ws.batch + p * ws.s_bat;
  const float* E = ws.E + p * ws.s_E + m;
  float c = 0.f;
  for (int j = j0; j < j1; ++j) c = fmaxf(c, a * E[static_cast<long long>(bat[j]) * sh.ldM]);
  atomicMax(reinterpret_cast<unsigned*>(&ws.cov[p * ws.s_cov + m]), __float_as_uint(c));
}

// ---------------------------------------------------------------------------
// singleton gains and the pool
// ---------------------------------------------------------------------------
// Singleton gains u_i = sum_m alpha_m max(E_mi - b_m, 0) of every token, four
// per wave; the client rows are streamed with non-temporal loads (the matrix
// is read once per round and is larger than the caches).  With kTail the last block to finish picks the pool itself (keys
// in LDS, or in global memory for large N); without it pool_topk_kernel
// follows.
template <bool kGlobalKeys, bool kTail = true>
__global__ void __launch_bounds__(256)
gains_kernel(Shape sh, Ws ws, int round, int psize, SelOut so) {
  extern __shared__ uint32_t keys_lds[];
  __shared__ int hist[512], scan[16], bc[2], flag;
  const int p = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int col0 = blockIdx.x * kGainCols + wave * kCpw;
  const float* alpha = ws.alpha + p * ws.s_m;
  const float* cov = ws.cov + p * ws.s_cov;
  const float* E = ws.E + p * ws.s_E;
  float* u = ws.u + p * ws.s_u;
  float acc[kCpw];
  const float* col[kCpw];
#pragma unroll
  for (int c = 0; c < kCpw; ++c) {
    acc[c] = 0.f;
    col[c] = E + static_cast<long long>(min(col0 + c, sh.N - 1)) * sh.ldM;
  }
#pragma unroll 4
  for (int m = lane * 4; m < sh.m; m += 256) {
    const float4 a = *reinterpret_cast<const float4*>(alpha + m);
    const float4 b = *reinterpret_cast<const float4*>(cov + m);
#pragma unroll
    for (int c = 0; c < kCpw; ++c) {
      const float4 v = ld_stream4(col[c] + m);
      acc[c] += fmaxf(a.x * v.x - b.x, 0.f);
      acc[c] += fmaxf(a.y * v.y - b.y, 0.f);
      acc[c] += fmaxf(a.z * v.z - b.z, 0.f);
      acc[c] += fmaxf(a.w * v.w - b.w, 0.f);
    }
  }
#pragma unroll
  for (int c = 0; c < kCpw; ++c) {
    const float s = wave_sum(acc[c]);
    if (lane == 0 && col0 + c < sh.N) st_dev(&u[col0 + c], s);
  }
  if constexpr (!kTail) return;

  // tail: the pool, the psize largest gains among unselected tokens
  int* cnt = ws.cnt + p * ws.s_cnt;
  if (!last_arrival(&cnt[0], gridDim.x, &flag)) return;
  if (tid == 0) st_dev(&cnt[0], 0);
  uint32_t* keys = kGlobalKeys ? ws.keys + p * ws.s_keys : keys_lds;
  const int* sel = ws.sel + p * ws.s_sel;
  // loads go to registers in batches first (keys may alias global memory, so
  // interleaved stores would serialise them)
  for (int base = 0; base < sh.N; base += 256 * 16) {
    float g[16];
    int sl[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int i = min(base + q * 256 + tid, sh.N - 1);
      g[q] = ld_dev(&u[i]);
      sl[q] = sel[i];
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int i = base + q * 256 + tid;
      if (i < sh.N) {
        keys[i] = (sl[q] >= 0) ? 0u : score_key(g[q]);
        if (so.gains) so.gains[(static_cast<long long>(p) * sh.rounds + round) * sh.N + i] = (sl[q] >= 0) ? 0.f : g[q];
      }
    }
  }
  __syncthreads();
  int* pool = ws.pool + p * ws.s_pool;
  block_topk256(keys, sh.N, psize, pool, hist, scan, bc);
  if (so.pool) {
    int32_t* tp = so.pool + (static_cast<long long>(p) * sh.rounds + round) * sh.pool_cap;
    for (int j = tid; j < sh.pool_cap; j += 256) tp[j] = (j < psize) ? pool[j] : -1;
  }
}

// The pool of a per-round call: the psize largest gains among unselected
// tokens, ascending by index, equal gains resolved to the lower index (the
// same selection as the gains kernel's tail).  One 1024-thread block per
// problem: the keys are made from coalesced loads into LDS (dynamic, N
// words), then thread t takes tokens [t seg, t seg + seg) into registers
// (seg <= KPT), so every radix pass works on registers and LDS histograms.
constexpr int kPoolW = 16;   // waves of the pool top-k block
template <int KPT>
__global__ void __launch_bounds__(64 * kPoolW) pool_topk_kernel(Shape sh, Ws ws, int round, int psize,
                                                                 SelOut so) {
  extern __shared__ uint32_t keys_lds[];
  __shared__ int hist[768], scan[3 * kPoolW];
  const int p = blockIdx.x, tid = threadIdx.x;
  const float* u = ws.u + p * ws.s_u;
  const int* sel = ws.sel + p * ws.s_sel;
  constexpr int kT = 64 * kPoolW;
  float g[KPT];
  int sl[KPT];
#pragma unroll
  for (int q = 0; q < KPT; ++q) {
    const int i = min(q * kT + tid, sh.N - 1);
    g[q] = u[i];
    sl[q] = sel[i];
  }
#pragma unroll
  for (int q = 0; q < KPT; ++q) {
    const int i = q * kT + tid;
    if (i < sh.N) {
      keys_lds[i] = sl[q] < 0 ? score_key(g[q]) : 0u;
      if (so.gains) so.gains[(static_cast<long long>(p) * sh.rounds + round) * sh.N + i] = (sl[q] >= 0) ? 0.f : g[q];
    }
  }
  __syncthreads();
  const int seg = (sh.N + kT - 1) / kT;
  const int i0 = tid * seg;
  uint32_t k[KPT];
#pragma unroll
  for (int q = 0; q < KPT; ++q) k[q] = (q < seg && i0 + q < sh.N) ? keys_lds[i0 + q] : 0u;
  int* pool = ws.pool + p * ws.s_pool;
  block_topk_regs<KPT, kPoolW>(k, seg, psize, pool, hist, scan, 0);
  if (so.pool) {
    int32_t* tp = so.pool + (static_cast<long long>(p) * sh.rounds + round) * sh.pool_cap;
    for (int j = tid; j < sh.pool_cap; j += 64 * kPoolW) tp[j] = (j < psize) ? pool[j] : -1;
  }
}


// Batch of a small pool from the responsibility block sums (one whole wave):
// scores summed in block order, top-b by (score desc, index asc).  Leaves
// the pool in pool_s and the chosen source indices, ascending, in bidx.
__device__ void small_batch(const Shape& sh, const Ws& ws, int p, int psize, int bsize, int nblk,
                            int* pool_s, uint32_t* keys, int* chosen, int* bidx, float* scores) {
  const int lane = threadIdx.x & 63;
  pool_s[lane] = (lane < psize) ? ws.pool[p * ws.s_pool + lane] : 0;
  const float* sp = ws.spart + p * ws.s_spart;
  float s = 0.f;
  int b = 0;
  for (; b + 8 <= nblk; b += 8) {
    float t[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) t[q] = sp[static_cast<long long>(b + q) * 64 + lane];
#pragma unroll
    for (int q = 0; q < 8; ++q) s += t[q];
  }
  for (; b < nblk; ++b) s += sp[static_cast<long long>(b) * 64 + lane];
  if (scores && lane < sh.pool_cap) scores[lane] = lane < psize ? s : 0.f;
  keys[lane] = score_key(s);
  __builtin_amdgcn_wave_barrier();
  wave_topb(keys, psize, bsize, chosen);
  __builtin_amdgcn_wave_barrier();
  if (lane < bsize) bidx[lane] = pool_s[chosen[lane]];
}

// Small pools, fused round: (1) the previous round's batch from the
// responsibility sums, recorded by block 0; (2) the coverage refresh
// b_m <- max(b_m, max_{j in batch} Cbar_mj) for every row, into LDS (block 0
// also stores it; a block that reads an already refreshed b_m recomputes the
// same value, since max(b_new, Cbar_mB) = b_new); (3) singleton gains of the
// block's tokens; (4) last block: the pool of this round, excluding the
// selected set and the batch just chosen.
template <bool kGlobalKeys>
__global__ void __launch_bounds__(256)
gains_fused_kernel(Shape sh, Ws ws, int round, int psize, int prev_psize, int prev_bsize, int prev_base,
                   SelOut so) {
  extern __shared__ __attribute__((aligned(16))) float dyn[];      // refreshed coverage [ldM], then LDS keys [N]
  __shared__ int hist[512], scan[16], bc[2], flag;
  __shared__ int pool_s[64], chosen[64], bidx[64];
  __shared__ __attribute__((aligned(16))) uint32_t bkeys[64];
  const int p = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  float* bnew = dyn;
  const float* alpha = ws.alpha + p * ws.s_m;
  float* cov = ws.cov + p * ws.s_cov;
  const float* E = ws.E + p * ws.s_E;
  const int nb = round > 0 ? prev_bsize : 0;
  if (round > 0) {
    float* sc = (so.scores && blockIdx.x == 0)
                    ? so.scores + (static_cast<long long>(p) * sh.rounds + round - 1) * sh.pool_cap : nullptr;
    if (wave == 0)
      small_batch(sh, ws, p, prev_psize, prev_bsize, (sh.m + 255) / 256, pool_s, bkeys, chosen, bidx, sc);
    __syncthreads();
    if (blockIdx.x == 0) commit_batch(sh, ws, p, round - 1, prev_bsize, prev_base, pool_s, chosen, so.batch);
    // two row chunks per trip, all their batch-column loads in flight together
    for (int m0 = tid * 4; m0 < sh.m; m0 += 2048) {
      float4 c[2], a[2], b[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int m = min(m0 + h * 1024, sh.ldM - 4);
        a[h] = *reinterpret_cast<const float4*>(alpha + m);
        b[h] = *reinterpret_cast<const float4*>(cov + m);
        c[h] = make_float4(0.f, 0.f, 0.f, 0.f);
      }
      for (int k0 = 0; k0 < nb; k0 += 16) {
        // indices past the batch repeat its last column: a maximum is unchanged
        float4 v[2][16];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int q = 0; q < 16; ++q)
            v[h][q] = *reinterpret_cast<const float4*>(
                E + static_cast<long long>(bidx[min(k0 + q, nb - 1)]) * sh.ldM + min(m0 + h * 1024, sh.ldM - 4));
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int q = 0; q < 16; ++q) {
            c[h].x = fmaxf(c[h].x, a[h].x * v[h][q].x); c[h].y = fmaxf(c[h].y, a[h].y * v[h][q].y);
            c[h].z = fmaxf(c[h].z, a[h].z * v[h][q].z); c[h].w = fmaxf(c[h].w, a[h].w * v[h][q].w);
          }
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int m = m0 + h * 1024;
        if (m < sh.m) {
          const float4 r = make_float4(fmaxf(b[h].x, c[h].x), fmaxf(b[h].y, c[h].y), fmaxf(b[h].z, c[h].z),
                                       fmaxf(b[h].w, c[h].w));
          *reinterpret_cast<float4*>(bnew + m) = r;
          if (blockIdx.x == 0) *reinterpret_cast<float4*>(cov + m) = r;
        }
      }
    }
  } else {
    // the coverage before the first round: zero, or the image seeds' b_m(S_0)
    for (int m = tid * 4; m < sh.m; m += 1024)
      *reinterpret_cast<float4*>(bnew + m) =
          sh.nseed > 0 ? *reinterpret_cast<const float4*>(cov + m) : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  __syncthreads();
  const int col0 = blockIdx.x * kGainColsF + wave * kCpwF;
  float* u = ws.u + p * ws.s_u;
  float acc[kCpwF];
  const float* col[kCpwF];
#pragma unroll
  for (int c = 0; c < kCpwF; ++c) {
    acc[c] = 0.f;
    col[c] = E + static_cast<long long>(min(col0 + c, sh.N - 1)) * sh.ldM;
  }
#pragma unroll 4
  for (int m = lane * 4; m < sh.m; m += 256) {
    const float4 a = *reinterpret_cast<const float4*>(alpha + m);
    const float4 b = *reinterpret_cast<const float4*>(bnew + m);
#pragma unroll
    for (int c = 0; c < kCpwF; ++c) {
      const float4 v = *reinterpret_cast<const float4*>(col[c] + m);
      acc[c] += fmaxf(a.x * v.x - b.x, 0.f);
      acc[c] += fmaxf(a.y * v.y - b.y, 0.f);
      acc[c] += fmaxf(a.z * v.z - b.z, 0.f);
      acc[c] += fmaxf(a.w * v.w - b.w, 0.f);
    }
  }
#pragma unroll
  for (int c = 0; c < kCpwF; ++c) {
    const float s = wave_sum(acc[c]);
    if (lane == 0 && col0 + c < sh.N) st_dev(&u[col0 + c], s);
  }

  int* cnt = ws.cnt + p * ws.s_cnt;
  if (!last_arrival(&cnt[0], gridDim.x, &flag)) return;
  if (tid == 0) st_dev(&cnt[0], 0);
  uint32_t* keys = kGlobalKeys ? ws.keys + p * ws.s_keys : reinterpret_cast<uint32_t*>(dyn + sh.ldM);
  const int* sel = ws.sel + p * ws.s_sel;
  for (int base = 0; base < sh.N; base += 256 * 16) {
    float g[16];
    int sl[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int i = min(base + q * 256 + tid, sh.N - 1);
      g[q] = ld_dev(&u[i]);
      sl[q] = sel[i];
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int i = base + q * 256 + tid;
      if (i < sh.N) {
        bool taken = sl[q] >= 0;
        for (int k = 0; k < nb; ++k) taken |= bidx[k] == i;
        keys[i] = taken ? 0u : score_key(g[q]);
        if (so.gains) so.gains[(static_cast<long long>(p) * sh.rounds + round) * sh.N + i] = taken ? 0.f : g[q];
      }
    }
  }
  __syncthreads();
  int* pool = ws.pool + p * ws.s_pool;
  block_topk256(keys, sh.N, psize, pool, hist, scan, bc);
  if (so.pool) {
    int32_t* tp = so.pool + (static_cast<long long>(p) * sh.rounds + round) * sh.pool_cap;
    for (int j = tid; j < sh.pool_cap; j += 256) tp[j] = (j < psize) ? pool[j] : -1;
  }
}

// Small pools, after the last round: its batch from the responsibility sums.
__global__ void __launch_bounds__(64) final_batch_kernel(Shape sh, Ws ws, int round, int psize, int bsize,
                                                         int sel_base, SelOut so) {
  __shared__ int pool_s[64], chosen[64], bidx[64];
  __shared__ __attribute__((aligned(16))) uint32_t keys[64];
  const int p = blockIdx.x;
  small_batch(sh, ws, p, psize, bsize, (sh.m + 255) / 256, pool_s, keys, chosen, bidx,
              so.scores ? so.scores + (static_cast<long long>(p) * sh.rounds + round) * sh.pool_cap : nullptr);
  __syncthreads();
  commit_batch(sh, ws, p, round, bsize, sel_base, pool_s, chosen, so.batch);
}

// Pool of at most 64: per-block responsibility sums; the batch is picked by
// the next kernel (the next round's gains, or the final batch kernel).
__global__ void __launch_bounds__(256) resp_small_kernel(Shape sh, Params pr, Ws ws, int psize) {
  __shared__ int pool_s[64];
  __shared__ float wsum[4][64];
  const int p = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid < 64) pool_s[tid] = (tid < psize) ? ws.pool[p * ws.s_pool + tid] : 0;
  __syncthreads();
  const int m = blockIdx.x * 256 + tid;
  const bool row_ok = m < sh.m;
  const int mc = row_ok ? m : 0;   // clamped: every load below is unconditional
  const float* E = ws.E + p * ws.s_E + mc;
  float v[64];
  float mu = 0.f;
  const float a = row_ok ? ws.alpha[p * ws.s_m + mc] : 0.f;
  const float c = ws.cov[p * ws.s_cov + mc];
#pragma unroll
  for (int j = 0; j < 64; ++j) v[j] = E[static_cast<long long>(pool_s[j]) * sh.ldM];
#pragma unroll
  for (int j = 0; j < 64; ++j) {
    const float r = (j < psize) ? fmaxf(a * v[j] - c, 0.f) : 0.f;
    v[j] = r;
    mu = fmaxf(mu, r);
  }
  if (mu > 0.f) {
    const float inv = 1.f / (pr.tau_r * mu + pr.resp_eps);
    const float zmax = mu * inv;
    float den = 0.f;
    float ex[64];
#pragma unroll
    for (int j = 0; j < 64; ++j) {
      ex[j] = (j < psize) ? __expf(v[j] * inv - zmax) : 0.f;
      den += ex[j];
    }
    const float rden = 1.f / den;
#pragma unroll
    for (int j = 0; j < 64; ++j) v[j] = ex[j] * rden * v[j];
  } else {
#pragma unroll
    for (int j = 0; j < 64; ++j) v[j] = 0.f;
  }
  wsum[wave][lane] = transpose_reduce64(v, lane);
  __syncthreads();
  float* sp = ws.spart + p * ws.s_spart;
  if (tid < psize)
    sp[static_cast<long long>(blockIdx.x) * 64 + tid] = ((wsum[0][tid] + wsum[1][tid]) + wsum[2][tid]) + wsum[3][tid];
}

// Large pools: per-row max mu_m and softmax denominator over the pool.
// Block = 64 rows (lane = row) x 16 waves splitting the pool positions (the
// grid is only m / 64 blocks, so the waves supply the loads in flight).
constexpr int kRsW = 16;
__global__ void __launch_bounds__(64 * kRsW) rowstat_kernel(Shape sh, Params pr, Ws ws, int psize) {
  __shared__ float part[kRsW][64];
  __shared__ float mu_s[64];
  const int p = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int m = blockIdx.x * 64 + lane;
  const bool row_ok = m < sh.m;
  const float a = row_ok ? ws.alpha[p * ws.s_m + m] : 0.f;
  const float c = row_ok ? ws.cov[p * ws.s_cov + m] : 0.f;
  const float* E = ws.E + p * ws.s_E + (row_ok ? m : 0);
  const int* pool = ws.pool + p * ws.s_pool;
  const int q = (psize + kRsW - 1) / kRsW, j0 = wave * q, j1 = min(psize, j0 + q);
  float mx = 0.f;
#pragma unroll 32
  for (int j = j0; j < j1; ++j) mx = fmaxf(mx, fmaxf(a * E[static_cast<long long>(pool[j]) * sh.ldM] - c, 0.f));
  part[wave][lane] = mx;
  __syncthreads();
  if (wave == 0) {
    float mm = part[0][lane];
#pragma unroll
    for (int w = 1; w < kRsW; ++w) mm = fmaxf(mm, part[w][lane]);
    mu_s[lane] = mm;
  }
  __syncthreads();
  const float mu = mu_s[lane];
  const float inv = mu > 0.f ? 1.f / (pr.tau_r * mu + pr.resp_eps) : 0.f;
  const float zmax = mu * inv;
  float den = 0.f;
  if (mu > 0.f)
#pragma unroll 32
    for (int j = j0; j < j1; ++j)
      den += __expf(fmaxf(a * E[static_cast<long long>(pool[j]) * sh.ldM] - c, 0.f) * inv - zmax);
  __syncthreads();
  part[wave][lane] = den;
  __syncthreads();
  if (wave == 0 && row_ok) {
    float d = part[0][lane];
#pragma unroll
    for (int w = 1; w < kRsW; ++w) d += part[w][lane];
    float* rs = ws.rstat + p * ws.s_rstat;
    rs[m] = inv;
    rs[sh.ldM + m] = zmax;
    rs[2 * sh.ldM + m] = mu > 0.f ? 1.f / d : 0.f;
  }
}

// Large pools: one wave per pool position sums rho R over all client rows;
// the last block picks the batch, with the keys in registers (at most 2048
// positions; from keys in LDS the kernel took 35.6 us at M = 11520 and 26.5 at
// M = 5752, now 32.2 and 22.7: the pick is most of what is left).
__global__ void __launch_bounds__(256)
colsum_kernel(Shape sh, Ws ws, int round, int psize, int bsize, int sel_base, SelOut so) {
  __shared__ int hist[768], scan[16], flag;
  __shared__ int chosen[1024];
  const int p = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int jj = blockIdx.x * 4 + wave;
  const int* pool = ws.pool + p * ws.s_pool;
  const float* rs = ws.rstat + p * ws.s_rstat;
  const float* alpha = ws.alpha + p * ws.s_m;
  const float* cov = ws.cov + p * ws.s_cov;
  float* sv = ws.u + p * ws.s_u;        // scores reuse the gains buffer
  if (jj < psize) {
    const float* col = ws.E + p * ws.s_E + static_cast<long long>(pool[jj]) * sh.ldM;
    float acc = 0.f;
    for (int m = lane * 4; m < sh.m; m += 256) {
      const float4 v = *reinterpret_cast<const float4*>(col + m);
      const float4 a = *reinterpret_cast<const float4*>(alpha + m);
      const float4 c = *reinterpret_cast<const float4*>(cov + m);
      const float4 inv = *reinterpret_cast<const float4*>(rs + m);
      const float4 zm = *reinterpret_cast<const float4*>(rs + sh.ldM + m);
      const float4 rd = *reinterpret_cast<const float4*>(rs + 2 * sh.ldM + m);
      float r;
      r = fmaxf(a.x * v.x - c.x, 0.f); acc += __expf(r * inv.x - zm.x) * rd.x * r;
      r = fmaxf(a.y * v.y - c.y, 0.f); acc += __expf(r * inv.y - zm.y) * rd.y * r;
      r = fmaxf(a.z * v.z - c.z, 0.f); acc += __expf(r * inv.z - zm.z) * rd.z * r;
      r = fmaxf(a.w * v.w - c.w, 0.f); acc += __expf(r * inv.w - zm.w) * rd.w * r;
    }
    const float s = wave_sum(acc);
    if (lane == 0) st_dev(&sv[jj], s);
  }
  int* cnt = ws.cnt + p * ws.s_cnt;
  if (!last_arrival(&cnt[4], gridDim.x, &flag)) return;
  if (tid == 0) st_dev(&cnt[4], 0);
  // thread t owns the positions [t seg, t seg + seg)
  const int seg = (psize + 255) / 256;
  float g[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) g[q] = ld_dev(&sv[min(tid * seg + min(q, seg - 1), psize - 1)]);
  uint32_t key[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) key[q] = q < seg && tid * seg + q < psize ? score_key(g[q]) : 0u;
  if (so.scores) {
    float* sc = so.scores + (static_cast<long long>(p) * sh.rounds + round) * sh.pool_cap;
#pragma unroll
    for (int q = 0; q < 8; ++q)
      if (key[q]) sc[tid * seg + q] = g[q];
    for (int j = psize + tid; j < sh.pool_cap; j += 256) sc[j] = 0.f;
  }
  block_topk_regs<8>(key, seg, bsize, chosen, hist, scan, 0);
  commit_batch(sh, ws, p, round, bsize, sel_base, pool, chosen, so.batch);
}


// F(S) = sum_m b_m(S) and F(V) = sum_m max_i Cbar_mi via per-block partials
// reduced in order by the last block.
__global__ void __launch_bounds__(256) objective_kernel(Shape sh, Ws ws) {
  __shared__ float red[16];
  __shared__ int flag;
  const int p = blockIdx.y, m = blockIdx.x * 256 + threadIdx.x;
  float c = 0.f, pk = 0.f;
  if (m < sh.m) {
    c = ws.cov[p * ws.s_cov + m];
    pk = ws.peak[p * ws.s_m + m];
  }
  const float fs = block_sum(c, red);
  const float fv = block_sum(pk, red);
  float* sp = ws.spart + p * ws.s_spart;
  if (threadIdx.x == 0) {
    st_dev(&sp[2 * blockIdx.x], fs);
    st_dev(&sp[2 * blockIdx.x + 1], fv);
  }
  int* cnt = ws.cnt + p * ws.s_cnt;
  if (!last_arrival(&cnt[2], gridDim.x, &flag)) return;
  if (threadIdx.x == 0) {
    st_dev(&cnt[2], 0);
    float a = 0.f, b = 0.f;
#pragma unroll 8
    for (unsigned k = 0; k < gridDim.x; ++k) { a += ld_dev(&sp[2 * k]); b += ld_dev(&sp[2 * k + 1]); }
    float* st = ws.stats + p * ws.s_st;
    st[2] = a;
    st[3] = b;
    st[4] = static_cast<float>(sh.K);
    st[5] = static_cast<float>(sh.rounds);
    st[6] = static_cast<float>(sh.m);
    st[7] = static_cast<float>(sh.N - sh.K);
  }
}


static void launch_cov(const Shape& sh, const Ws& ws, int nb, hipStream_t st) {
  hipLaunchKernelGGL(cov_kernel, dim3((sh.m + 255) / 256, (nb + kCovCols - 1) / kCovCols, sh.B), dim3(256), 0,
                     st, sh, ws, nb);
}

// Variants of the persistent selection.  The grid never exceeds what the
// device holds at once (checked against the kernel's occupancy), so on a
// device not shared with other work every block is resident from the start.
// The launch is an ordinary one: a cooperative launch costs a cross-queue
// synchronisation on each side of the kernel, and the bounded waits already
// turn a block that never becomes resident (a device saturated by foreign
// work) into a reported timeout rather than a hang.
struct SelVariant {
  const void* fn;
  int J, R;            // rows / 256 and tokens per wave held in registers (0: none)
  bool streams;        // takes more tokens than the held ones
  bool half;           // at most kHalfRegs registers
  KernelRoom room;
};
enum { kSelStream, kSelWide, kSelSplit, kSelHold };   // g_sel: hold variants, each kind by J, then R
static SelVariant g_sel[] = {
    {reinterpret_cast<const void*>(select_stream_kernel), 0, 0, true, true},
    {reinterpret_cast<const void*>(select_wide_kernel), 0, 0, true, true},
    {reinterpret_cast<const void*>(select_split_kernel), 0, 0, false, true},
#define GMC_HOLD(J, R, S) {reinterpret_cast<const void*>(select_hold_kernel<J, R, S>), J, R, S, hold_half(J, R, S), {}},
    GMC_HOLD(4, 5, false) GMC_HOLD(8, 5, false) GMC_HOLD(14, 3, false) GMC_HOLD(14, 5, false) GMC_HOLD(20, 2, false)
    GMC_HOLD(20, 3, false) GMC_HOLD(24, 3, false) GMC_HOLD(28, 2, false) GMC_HOLD(32, 2, false) GMC_HOLD(36, 2, false)
    GMC_HOLD(48, 1, false)
    GMC_HOLD(4, 5, true) GMC_HOLD(8, 5, true) GMC_HOLD(14, 5, true) GMC_HOLD(20, 3, true) GMC_HOLD(24, 3, true)
    GMC_HOLD(28, 2, true) GMC_HOLD(32, 2, true) GMC_HOLD(36, 2, true) GMC_HOLD(48, 1, true)
#undef GMC_HOLD
};
static std::mutex g_sel_mu;
static int g_n_cu = -1, g_lds_max = 0;

// The device's CUs and LDS per block, 0 CUs if unknown (g_sel_mu held).
static int device_cus() {
  if (g_n_cu < 0) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&g_n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipDeviceGetAttribute(&g_lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
      g_n_cu = 0;
  }
  return g_n_cu;
}

// Blocks of a variant that one CU holds at once, 0 if none (g_sel_mu held).
static int variant_per_cu(SelVariant& v, size_t lds) {
  if (device_cus() <= 0 || lds > static_cast<size_t>(g_lds_max)) return 0;
  // failures: too much LDS beside the static arrays, another variant is taken
  auto ok = [](hipError_t e) {
    if (e != hipSuccess) (void)hipGetLastError();
    return e == hipSuccess;
  };
  return v.room.blocks(
      lds,
      [&](size_t n) {
        return ok(hipFuncSetAttribute(v.fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(n)));
      },
      [&](size_t n, int* blocks) { return ok(hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, v.fn, 256, n)); });
}

// The turn words of every device.
static __device__ int sel_turn_words[4];

hipError_t selection_turn(int** words) {
  static std::mutex mu;
  static int* known[64] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess || dev < 0 || dev >= 64) return e != hipSuccess ? e : hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(mu);
  if (!known[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(sel_turn_words));
    if (e != hipSuccess) return e;
    known[dev] = static_cast<int*>(p);
  }
  *words = known[dev];
  return hipSuccess;
}

__global__ void __launch_bounds__(64) take_turn_kernel(SelTurn turn, int problems) {
  if (threadIdx.x == 0) take_turn(turn, problems);
}
hipError_t launch_take_turn(const SelTurn& turn, int problems, hipStream_t st) {
  hipLaunchKernelGGL(take_turn_kernel, dim3(1), dim3(64), 0, st, turn, problems);
  return hipGetLastError();
}
__global__ void __launch_bounds__(64) leave_turn_kernel(SelTurn turn) {
  if (threadIdx.x == 0) leave_turn(turn);
}
hipError_t launch_leave_turn(const SelTurn& turn, hipStream_t st) {
  hipLaunchKernelGGL(leave_turn_kernel, dim3(1), dim3(64), 0, st, turn);
  return hipGetLastError();
}

struct SelPlan {
  const SelVariant* v = nullptr;   // null: the call does not qualify
  int nblk = 0;                    // blocks per problem
  size_t lds = 0;
  bool turn = false;               // needs the device without another selection
};

// The persistent variant of a call: not with large pools or keys beyond LDS.
// Per token the row-split kernel forms the sums in its own order; held and
// streamed rows share another, so a shape keeps one result whichever of them
// it takes.
// Beside a selection of the other entry point (see SelTurn): half variants
// with one block per CU, up to kHalfLds (context) and kHalfLdsStatic of LDS,
// fit a CU side by side, with the gate of the context's next call.  The static
// entry takes only these (what is larger runs round by round, with no waits
// between blocks), so the common one-image calls of a context need no turn;
// its other calls take one.
static SelPlan select_plan(const Shape& sh, int party) {
  SelPlan pl;
  if (sh.pool_cap > 64 || sh.N > kLdsKeys) return pl;
  std::lock_guard<std::mutex> lk(g_sel_mu);
  // LDS besides the static arrays (see select_rounds)
  auto lds_of = [&](const SelVariant& v, int blocks) {
    const size_t groups = v.R ? v.J : (sh.m + 255) / 256;
    const size_t rows = &v == &g_sel[kSelSplit] ? sh.ldM : &v == &g_sel[kSelWide] ? 256 * groups : 512 * groups;
    return 4 * (rows + static_cast<size_t>(sh.N + 15) / 16 * 4 + static_cast<size_t>((sh.N + blocks - 1) / blocks) +
                (sh.N > 256 * 16 ? sh.N : 0));
  };
  // blocks with at least one token each
  auto full = [&](int blocks) { const int t = (sh.N + blocks - 1) / blocks; return (sh.N + t - 1) / t; };
  auto take = [&](SelVariant& v, int blocks, int per_cu) {
    const size_t lds = lds_of(v, blocks);
    const bool half = v.half && blocks * sh.B <= g_n_cu &&
                      lds + kSelStaticLds <= static_cast<size_t>(party == kPartyStatic ? kHalfLdsStatic : kHalfLds);
    if (party == kPartyStatic && !half) return false;
    if (min(variant_per_cu(v, lds), per_cu) * g_n_cu < blocks * sh.B) return false;
    pl.turn = !half;
    pl.v = &v;
    pl.nblk = blocks;
    pl.lds = lds;
    return true;
  };
  if (device_cus() < 1) return pl;
  // about two gain tokens per wave
  const int want = max((sh.N + 7) / 8, ((sh.m + 63) / 64 + 3) / 4);
  const int one = min(min(g_n_cu / sh.B, want), kMaxPersist);   // one block per CU
  if (one >= 1 && sh.N <= 8 * one && sh.m <= 256 * kResJ && take(g_sel[kSelSplit], (sh.N + 7) / 8, 1)) return pl;
  if (one >= 1) {
    // rows in registers: the narrowest variant the rows fit, of those the
    // fewest tokens per wave that cover the block's, else the most.
    const int nblk = full(one), tokens = ((sh.N + nblk - 1) / nblk + 3) / 4;
    SelVariant* best = nullptr;
    for (int i = kSelHold; i < static_cast<int>(sizeof(g_sel) / sizeof(g_sel[0])); ++i) {
      SelVariant& v = g_sel[i];
      if (256 * v.J < sh.m || v.streams != (tokens > v.R) || (best && (v.J > best->J || best->R >= tokens))) continue;
      best = &v;
    }
    // With every token held they win wherever they were measured (us a call,
    // held / streamed at two blocks per CU; 8 heads, d = 512 unless said):
    // J = 4 137 / 159, 8 198 / 217, 14 191 / 208, 20 264 / 298, 24 292 / 326,
    // 28 390 / 433, 32 330 / 383, 36 473 / 534, 48 372 / 390.  With some of
    // them streamed, which one block per CU does with half the waves, they win
    // up to 16 problems: J = 4 and 8 by 1 to 5 %, 14 (d = 3584, N = 1296) with 2
    // problems 357 / 420, 4 507 / 561, 8 723 / 743; 20 466 / 488, 24 540 / 566,
    // 28 726 / 750, 32 742 / 782 (the page 1489 / 1531), 36 914 / 951, 48 546 /
    // 551 and 852 / 875 (but 407 / 403 with two tokens a wave).  They lose with
    // more problems (32: J = 14 2256 / 2182, 20 1346 / 1304) and, where two
    // streamed blocks fit a CU with ease (J <= 14), with less than two fifths
    // of the tokens held (16 problems: J = 14 with 24 % 1148 / 1138, 8 with
    // 33 % 524 / 511).
    if (best && best->streams && (sh.B > 16 || (best->J <= 14 && 5 * best->R < 2 * tokens))) best = nullptr;
    if (best && take(*best, nblk, 1)) return pl;
  }
  // streamed: two blocks per CU where they fit, twice the waves in flight.
  // Beyond LDS for weights and coverage the weights come from memory: against
  // the kernel that read them so for every M, M = 19152 1103 -> 1027 us a call
  // (4 problems 1930 -> 1796), M = 23552, N = 4096 2458 -> 2018; the rounds as
  // launches of their own take 1105, 1586 and 1883.
  for (const int i : {kSelStream, kSelWide})
    for (int per = 2; per >= 1; --per) {
      const int blocks = min(min(per * g_n_cu / sh.B, want), kMaxPersist);
      if (blocks >= 1 && take(g_sel[i], full(blocks), per)) return pl;
    }
  return pl;
}

bool selection_needs_turn(const Shape& sh) {
  return sh.rounds > 0 && select_plan(sh, kPartyContext).turn;
}

hipError_t launch_selection(const Shape& sh, const Params& pr, const Ws& ws, const SelOut& so, const SelTurn& turn,
                            hipStream_t st, bool* support_ready) {
  *support_ready = false;
  if (sh.rounds == 0) {
    // the image seeds already fill the budget (K = I): only the objective;
    // the assignment builds the support list from the selection marks
    timer_mark(kStObjective, true, st);
    hipLaunchKernelGGL(objective_kernel, dim3((sh.m + 255) / 256, sh.B), dim3(256), 0, st, sh, ws);
    timer_mark(kStObjective, false, st);
    return hipGetLastError();
  }
  if (const SelPlan pl = select_plan(sh, turn.party); pl.v) {
    timer_mark(kStSelect, true, st);
    Shape a0 = sh;
    Params a1 = pr;
    Ws a2 = ws;
    int a3 = pl.nblk;
    SelOut a4 = so;
    SelTurn a5 = turn;
    void* args[] = {&a0, &a1, &a2, &a3, &a4, &a5};
    const hipError_t e = hipLaunchKernel(pl.v->fn, dim3(pl.nblk, sh.B), dim3(256), args, pl.lds, st);
    if (e != hipSuccess && turn.words) (void)launch_leave_turn(turn, st);
    timer_mark(kStSelect, false, st);
    *support_ready = true;
    return e != hipSuccess ? e : hipGetLastError();
  }
  // round by round: no waits between blocks
  if (turn.words) {
    const hipError_t e = launch_leave_turn(turn, st);
    if (e != hipSuccess) return e;
  }
  const bool global_keys = sh.N > kLdsKeys;
  const size_t key_lds = global_keys ? 0 : static_cast<size_t>(sh.N) * sizeof(uint32_t);
  // unfused rounds pick the pool in a 1024-thread register top-k kernel
  // (keys per thread: 4, 8 or 16); beyond 16 * 1024 tokens the gains
  // kernel's last block does it over keys in global memory
  const int pool_seg = (sh.N + 64 * kPoolW - 1) / (64 * kPoolW);
  const int pool_kpt = pool_seg <= 4 ? 4 : pool_seg <= 8 ? 8 : pool_seg <= 16 ? 16 : 0;
  static int pool_lds_granted = 48 * 1024;
  const size_t fused_lds = static_cast<size_t>(sh.ldM) * sizeof(float) + key_lds;
  // small pools fuse the batch pick and the coverage refresh into the gains
  // kernel while the refreshed coverage fits in LDS next to the keys
  // fused only while the call is latency-bound: every fused block re-reads
  // the batch columns, which costs more than a launch once the client
  // matrix is large
  const long long cbar_bytes = 4LL * sh.B * sh.N * sh.m;
  const bool fused = sh.pool_cap <= 64 && fused_lds <= 56 * 1024 && cbar_bytes <= (48LL << 20);
  const dim3 gg((sh.N + kGainCols - 1) / kGainCols, sh.B);
  const dim3 ggf((sh.N + kGainColsF - 1) / kGainColsF, sh.B);
  int selected = sh.nseed, prev_psize = 0, prev_bsize = 0, prev_base = 0;
  for (int r = 0; r < sh.rounds; ++r) {
    const int psize = min(sh.pool_cap, sh.N - selected);
    const int bsize = min(sh.b, sh.K - selected);
    if (fused) {
      timer_mark(kStGains, true, st);
      if (global_keys)
        hipLaunchKernelGGL(gains_fused_kernel<true>, ggf, dim3(256), fused_lds, st, sh, ws, r, psize,
                           prev_psize, prev_bsize, prev_base, so);
      else
        hipLaunchKernelGGL(gains_fused_kernel<false>, ggf, dim3(256), fused_lds, st, sh, ws, r, psize,
                           prev_psize, prev_bsize, prev_base, so);
      timer_mark(kStGains, false, st);
      timer_mark(kStResp, true, st);
      hipLaunchKernelGGL(resp_small_kernel, dim3((sh.m + 255) / 256, sh.B), dim3(256), 0, st, sh, pr, ws,
                         psize);
      timer_mark(kStResp, false, st);
    } else {
      if (r > 0) {
        timer_mark(kStCov, true, st);
        launch_cov(sh, ws, sh.b, st);
        timer_mark(kStCov, false, st);
      }
      timer_mark(kStGains, true, st);
      if (pool_kpt > 0) {
        hipLaunchKernelGGL((gains_kernel<true, false>), gg, dim3(256), 0, st, sh, ws, r, psize, so);
        // the pool's own kernel is timed with the responsibilities
        timer_mark(kStGains, false, st);
        timer_mark(kStResp, true, st);
        const dim3 gp(sh.B), bp(64 * kPoolW);
        const size_t pl = static_cast<size_t>(sh.N) * sizeof(uint32_t);
        if (pool_kpt == 16 && static_cast<int>(pl) > pool_lds_granted) {
          // 64 KB of keys next to the static histograms: grant the dynamic LDS once
          const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(pool_topk_kernel<16>),
                                                   hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(pl));
          if (e != hipSuccess) return e;
          pool_lds_granted = static_cast<int>(pl);
        }
        if (pool_kpt == 4)
          hipLaunchKernelGGL(pool_topk_kernel<4>, gp, bp, pl, st, sh, ws, r, psize, so);
        else if (pool_kpt == 8)
          hipLaunchKernelGGL(pool_topk_kernel<8>, gp, bp, pl, st, sh, ws, r, psize, so);
        else
          hipLaunchKernelGGL(pool_topk_kernel<16>, gp, bp, pl, st, sh, ws, r, psize, so);
      } else {
        if (global_keys)
          hipLaunchKernelGGL(gains_kernel<true>, gg, dim3(256), 0, st, sh, ws, r, psize, so);
        else
          hipLaunchKernelGGL(gains_kernel<false>, gg, dim3(256), key_lds, st, sh, ws, r, psize, so);
        timer_mark(kStGains, false, st);
        timer_mark(kStResp, true, st);
      }
      if (sh.pool_cap <= 64)
        hipLaunchKernelGGL(resp_small_kernel, dim3((sh.m + 255) / 256, sh.B), dim3(256), 0, st, sh, pr, ws,
                           psize);
      else {
        hipLaunchKernelGGL(rowstat_kernel, dim3((sh.m + 63) / 64, sh.B), dim3(64 * kRsW), 0, st, sh, pr, ws, psize);
        hipLaunchKernelGGL(colsum_kernel, dim3((psize + 3) / 4, sh.B), dim3(256), 0, st, sh, ws, r, psize, bsize,
                           selected, so);
      }
      if (sh.pool_cap <= 64)
        hipLaunchKernelGGL(final_batch_kernel, dim3(sh.B), dim3(64), 0, st, sh, ws, r, psize, bsize, selected,
                           so);
      timer_mark(kStResp, false, st);
    }
    prev_psize = psize;
    prev_bsize = bsize;
    prev_base = selected;
    selected += bsize;
  }
  timer_mark(kStObjective, true, st);
  if (fused)
    hipLaunchKernelGGL(final_batch_kernel, dim3(sh.B), dim3(64), 0, st, sh, ws, sh.rounds - 1, prev_psize,
                       prev_bsize, prev_base, so);
  launch_cov(sh, ws, prev_bsize, st);
  hipLaunchKernelGGL(objective_kernel, dim3((sh.m + 255) / 256, sh.B), dim3(256), 0, st, sh, ws);
  timer_mark(kStObjective, false, st);
  return hipGetLastError();
}

}  // namespace gmc
