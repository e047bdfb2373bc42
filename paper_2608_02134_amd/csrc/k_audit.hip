// Signed-message realisation audit (App. G Eq. cond-message-error; App. I
// Eq. cond-message-decomposition, Eq. cond-softmax-bound, Eq.
// cond-message-polar; Prop. 2 Eq. message-bound).
//
// For every query/head client g = (h, t) the native attention of the next
// block is re-run twice, over the Full visual keys and values and over the
// compact ones at the K carriers, with the same nonvisual denominator:
//   y_g  = sum_i a_gi v_i,     y~_g = sum_j abar_gj v~_j,
//   M_gj = sum_(i in C_j) a_gi (the Full attention grouped by carrier),
//   term1_g = y_g - sum_j M_gj v~_j,  term2_g = sum_j (M_gj - abar_gj) v~_j,
//   l1_g = ||M_g - abar_g||_1,  bound_g = max_j |log M_gj + LSE_F - s~_gj|.
// Kernels: the Full pass (log-sum-exp, then attention written to scratch and
// the message), the grouped mass per carrier, the compact pass with every
// per-client statistic, and the weighted per-problem reduction (e_M,
// amplitude ratio, cosine).
//
// Both passes: one block of eight waves per 16 clients of one kv head, the
// 16-key tiles dealt to the waves.  Logits are formed transposed, S^T = K Q^T
// on MFMA straight from memory, so that lane l holds client l % 16 against the
// keys 4 (l / 16) + e; these attention values are then the B operand of the
// fp32 MFMAs that add V^T a^T as they stand (step e takes key 4 k + e as its
// k slot k), with dims ordered so that a lane's share of a value row is
// contiguous.  Attention and sums stay fp32.  What bounds them is the chain
// of short dependent steps per tile on 112 blocks (Qwen2.5-VL-7B boundary,
// 1296 tokens, 256 carriers, 64 queries: Full pass 1295 -> 39 us, mass with
// its member lists 984 -> 7, compact pass 287 -> 21 against scalar fp32 dots
// from LDS).
#include <type_traits>

#include "gmc_device.h"
#include "gmc_internal.h"
#include "gmc_kernels.h"

namespace gmc {

constexpr int kAudRows = 16;   // clients per block
constexpr int kAudW = 8;       // waves per block

// Client rows of block tile: r < 16 -> (h, t) of kv head g, or invalid.
struct AudTile {
  int p, g, rb, rows_g;
  __device__ AudTile(const Shape& sh) {
    p = blockIdx.z;
    g = blockIdx.y;
    rb = blockIdx.x * kAudRows;
    rows_g = sh.hg * sh.T;
  }
  __device__ bool valid(int r) const { return rb + r < rows_g; }
  __device__ int head(const Shape& sh, int r) const { return g * sh.hg + (rb + r) / sh.T; }
  __device__ int query(const Shape& sh, int r) const { return (rb + r) % sh.T; }
  // client row index m = h T + t of the problem
  __device__ int mrow(const Shape& sh, int r) const { return head(sh, r) * sh.T + query(sh, r); }
};

// C consecutive elements (element-aligned addresses: the tensors may be views
// at any element) as fp32 or as an MFMA fragment.
template <typename T>
using GlobalPtr = const __attribute__((address_space(1))) T*;
template <typename T, int C>
__device__ __forceinline__ void aud_load(GlobalPtr<T> src, float (&v)[C]) {
  struct __attribute__((packed, aligned(sizeof(T)))) Pack { T x[C]; };
  Pack pk;
  __builtin_memcpy(&pk, (const T*)src, sizeof(pk));
#pragma unroll
  for (int c = 0; c < C; ++c) v[c] = to_f32(pk.x[c]);
}
__device__ __forceinline__ Frag<bf16_t> aud_frag(const bf16_t* src) {
  struct __attribute__((packed, aligned(2))) Pack { uint32_t x[4]; };
  const Pack pk = *reinterpret_cast<const Pack*>(src);
  Frag<bf16_t> f;
  f.v = __builtin_bit_cast(bf16x8, make_uint4(pk.x[0], pk.x[1], pk.x[2], pk.x[3]));
  return f;
}
__device__ __forceinline__ Frag<float> aud_frag(const float* src) {
  Frag<float> f;
#pragma unroll
  for (int c = 0; c < 8; ++c) f.v[c] = src[c];
  return f;
}

// A value row of zeros.
static __device__ const float aud_zeros[256] = {};

// One block's queries and its way over the rows of a [rows][Hkv][dh] tensor.
template <typename T, int DH>
struct AudBlock {
  static constexpr int KS = DH / 32, DT = DH / 16;   // DT: dims per lane, and dim tiles
  AudTile tl;
  int lane, wave, r, kg;      // client r = lane % 16, key group kg = lane / 16
  bool rv;
  int m;                      // the lane's client row
  float scale;
  long long stride;
  Frag<T> qf[KS];

  __device__ AudBlock(const Shape& sh, const T* text_q) : tl(sh) {
    lane = threadIdx.x & 63;
    wave = wave_id();
    r = lane & 15;
    kg = lane >> 4;
    rv = tl.valid(r);
    m = rv ? tl.mrow(sh, r) : 0;
    scale = rsqrtf(static_cast<float>(DH));
    stride = static_cast<long long>(sh.hkv) * DH;
    const T* q = text_q + ((static_cast<long long>(tl.p) * sh.T + (rv ? tl.query(sh, r) : 0)) * sh.hq +
                           (rv ? tl.head(sh, r) : 0)) * DH;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if (rv) qf[ks] = aud_frag(q + ks * 32 + kg * 8);
      else qf[ks] = frag_zero<T>();
    }
  }
  __device__ const T* base(const Shape& sh, const T* x, int rows) const {
    return x + static_cast<long long>(tl.p) * rows * stride + tl.g * DH;
  }
  // key fragments of tile ct (rows past the end repeat the last)
  __device__ void keys(const T* kb, int ct, int rows, Frag<T> (&kf)[KS]) const {
    const T* kr = kb + min(ct * 16 + r, rows - 1) * stride + kg * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) kf[ks] = aud_frag(kr + ks * 32);
  }
  // scaled logits of client r against the tile's keys 4 kg + e
  __device__ floatx4 logits(const Frag<T> (&kf)[KS]) const {
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) acc = mma(kf[ks], qf[ks], acc);
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] *= scale;
    return acc;
  }
  // the same from memory, two fragments at a time: for wide fp32 heads, whose
  // queries and message sums leave no registers for a tile's keys
  __device__ floatx4 logits_lean(const T* kb, int ct, int rows) const {
    const T* kr = kb + min(ct * 16 + r, rows - 1) * stride + kg * 8;
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      acc = mma(aud_frag(kr + ks * 32), qf[ks], acc);
      if (ks & 1) __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] *= scale;
    return acc;
  }
  // the lane's dims (DT of them, from DT (lane % 16)) of value row `row`; past
  // the end zeros (the attention there is zero, but another row loaded in its
  // place may hold infinities)
  __device__ void values(const T* vb, int row, int rows, float (&v)[DT]) const {
    GlobalPtr<T> src = row < rows ? (GlobalPtr<T>)(vb + row * stride) : (GlobalPtr<T>)aud_zeros;
    aud_load<T, DT>(src + r * DT, v);
  }

  // log-sum-exp of the block's clients over the rows, with the nonvisual part;
  // every lane gets its client's
  __device__ float lse(const Shape& sh, const T* kb, int rows, const float* nonvis, float (*red_m)[kAudRows],
                       float (*red_s)[kAudRows], float* lse_s) const {
    float mx = -INFINITY, sm = 0.f;
    const int nt = (rows + 15) / 16;
    // kAhead tiles of keys in flight
    constexpr int kAhead = KS * static_cast<int>(sizeof(Frag<T>) / 4) <= 16 ? 4 : 1;
    for (int c0 = wave; c0 < nt; c0 += kAhead * kAudW) {
    Frag<T> kf[kAhead][KS];
#pragma unroll
    for (int x = 0; x < kAhead; ++x) keys(kb, min(c0 + x * kAudW, nt - 1), rows, kf[x]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int x = 0; x < kAhead; ++x) {
      const int ct = c0 + x * kAudW;
      if (ct >= nt) break;
      const floatx4 s = logits(kf[x]);
      float nm = mx;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (ct * 16 + 4 * kg + e < rows) nm = fmaxf(nm, s[e]);
      // (all -inf or NaN so far: the former add nothing, a NaN stays)
      const float ref = nm == -INFINITY ? 0.f : nm;
      float t = sm * __expf(mx - ref);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (ct * 16 + 4 * kg + e < rows) t += __expf(s[e] - ref);
      sm = t;
      mx = nm;
    }
    }
    // the four key groups of a client, then the waves in order (without a
    // finite logit a sum is zero or NaN)
    float gm = fmaxf(mx, xor_lane<16>(mx));
    gm = fmaxf(gm, xor_lane<32>(gm));
    const float gs = add_xor32(add_xor16(mx == -INFINITY ? sm : sm * __expf(mx - gm)));
    if (lane < 16) { red_m[wave][lane] = gm; red_s[wave][lane] = gs; }
    __syncthreads();
    const int q = threadIdx.x;
    if (q < kAudRows) {
      float mm = -INFINITY;
      for (int w = 0; w < kAudW; ++w) mm = fmaxf(mm, red_m[w][q]);
      float s = 0.f;
      for (int w = 0; w < kAudW; ++w) s += red_m[w][q] == -INFINITY ? red_s[w][q] : red_s[w][q] * __expf(red_m[w][q] - mm);
      float D = mm + logf(s);
      if (nonvis && tl.valid(q)) {
        const float nv = nonvis[(static_cast<long long>(tl.p) * sh.hq + tl.head(sh, q)) * sh.T + tl.query(sh, q)];
        const float hi = fmaxf(D, nv), lo = fminf(D, nv);
        D = hi + log1pf(expf(lo - hi));
      }
      lse_s[q] = D;
    }
    __syncthreads();
    return lse_s[r];
  }
};

// Adds the waves' message tiles in wave order into ys[16][DH + 1] (LDS).
// Element e of tile t in lane l: client l % 16, dim DT (4 (l / 16) + e) + t.
template <int DH>
__device__ __forceinline__ void aud_add_waves(const floatx4 (&acc)[DH / 16], float* ys, int lane, int wave) {
  constexpr int DT = DH / 16;
  float* row = ys + (lane & 15) * (DH + 1) + DT * 4 * (lane >> 4);
  for (int w = 0; w < kAudW; ++w) {
    if (wave == w) {
      // every read before the first write: they would otherwise alternate
      // in dependent LDS round trips
      floatx4 sum[DT];
#pragma unroll
      for (int t = 0; t < DT; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[t][e] = w == 0 ? 0.f : row[DT * e + t];
#pragma unroll
      for (int t = 0; t < DT; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) row[DT * e + t] = sum[t][e] + acc[t][e];
    }
    __syncthreads();
  }
}

template <typename T, int DH>
__global__ void __launch_bounds__(64 * kAudW) audit_full_kernel(Shape sh, AudWs aw, const T* text_q, const T* vis_k,
                                                                const T* vis_v, const float* nonvis_lse) {
  constexpr int DT = DH / 16;
  __shared__ float red_m[kAudW][kAudRows], red_s[kAudW][kAudRows], lse_s[kAudRows], ys[kAudRows * (DH + 1)];
  const AudBlock<T, DH> ab(sh, text_q);
  const T* kb = ab.base(sh, vis_k, sh.N);
  const T* vb = ab.base(sh, vis_v, sh.N);
  const float D = ab.lse(sh, kb, sh.N, nonvis_lse, red_m, red_s, lse_s);
  const int mg1 = sh.mg1;
  if (threadIdx.x < kAudRows && ab.rv) aw.lse[static_cast<long long>(ab.tl.p) * mg1 + ab.m] = D;
  // attention to scratch, message y_g = sum_i a_gi v_i
  float* A = aw.A + static_cast<long long>(ab.tl.p) * sh.N * mg1 + ab.m;
  floatx4 y[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t) y[t] = floatx4{0.f, 0.f, 0.f, 0.f};
  // the next tile's keys and values load while this one is computed
  const int nt = (sh.N + 15) / 16;
  Frag<T> kf[2][DH / 32];
  float v2[2][4][DT];
  auto load = [&](int ct, int b) {
    ab.keys(kb, min(ct, nt - 1), sh.N, kf[b]);
#pragma unroll
    for (int e = 0; e < 4; ++e) ab.values(vb, min(ct, nt - 1) * 16 + 4 * ab.kg + e, sh.N, v2[b][e]);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto add = [&](int c0, int e, float s, const float (&v)[DT]) {
    const bool ok = c0 + e < sh.N;
    const float a = ok ? __expf(s - D) : 0.f;
    if (ok && ab.rv) A[static_cast<long long>(c0 + e) * mg1] = a;
#pragma unroll
    for (int t = 0; t < DT; ++t) y[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[t], a, y[t], 0, 0, 0);
  };
  auto step = [&](int ct, int b) {
    const floatx4 s = ab.logits(kf[b]);
#pragma unroll
    for (int e = 0; e < 4; ++e) add(ct * 16 + 4 * ab.kg, e, s[e], v2[b][e]);
  };
  if constexpr (sizeof(T) == 4 && DH > 224) {
    // a tile's keys and values spill beside the queries and the message
    for (int ct = ab.wave; ct < nt; ct += kAudW) {
      const int c0 = ct * 16 + 4 * ab.kg;
      const floatx4 s = ab.logits_lean(kb, ct, sh.N);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float v[DT];
        ab.values(vb, c0 + e, sh.N, v);
        add(c0, e, s[e], v);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  } else if constexpr (sizeof(T) == 4 && DH > 128) {
    // one tile's fragments fill the registers
    for (int ct = ab.wave; ct < nt; ct += kAudW) {
      load(ct, 0);
      step(ct, 0);
    }
  } else {
  load(ab.wave, 0);
  for (int ct = ab.wave; ct < nt; ct += 2 * kAudW) {
    load(ct + kAudW, 1);
    step(ct, 0);
    if (ct + kAudW >= nt) break;
    load(ct + 2 * kAudW, 0);
    step(ct + kAudW, 1);
  }
  }
  aud_add_waves<DH>(y, ys, ab.lane, ab.wave);
  for (int x = threadIdx.x; x < kAudRows * DH; x += 64 * kAudW) {
    const int q = x / DH, d = x % DH;
    if (ab.tl.valid(q)) aw.Y[(static_cast<long long>(ab.tl.p) * mg1 + ab.tl.mrow(sh, q)) * DH + d] = ys[q * (DH + 1) + d];
  }
}

// Grouped Full mass M_gj = sum_(i in C_j) a_gi: one block per carrier and 1024
// client rows.  The carrier's members (slots clamped to [0, K)) are listed
// in ascending order by a ballot scan of the carrier map, 2048 tokens a
// pass; each thread adds the members of four client rows, coalesced over
// rows.
constexpr int kMassQ = 4;    // client rows per thread
constexpr int kMassP = 8;    // carrier entries per thread and pass
__global__ void __launch_bounds__(256) audit_mass_kernel(Shape sh, AudWs aw, const int32_t* carrier) {
  __shared__ unsigned long long masks[kMassP][4];
  __shared__ int members[kMassP * 256];
  const int j = blockIdx.x, p = blockIdx.z, tid = threadIdx.x, lane = tid & 63, wave = wave_id();
  const int mg1 = sh.mg1, m0 = blockIdx.y * 256 * kMassQ + tid;
  const int32_t* cr = carrier + static_cast<long long>(p) * sh.N;
  const float* A = aw.A + static_cast<long long>(p) * sh.N * mg1;
  float s[kMassQ] = {};
  for (int base = 0; base < sh.N; base += kMassP * 256) {
    int c[kMassP];
#pragma unroll
    for (int q = 0; q < kMassP; ++q) {
      const int i = base + q * 256 + tid;
      c[q] = i < sh.N ? min(max(cr[i], 0), sh.K - 1) : -1;
    }
    unsigned long long bal[kMassP];
#pragma unroll
    for (int q = 0; q < kMassP; ++q) bal[q] = __ballot(c[q] == j);
    __syncthreads();   // the previous pass is done with masks and members
    if (lane == 0)
#pragma unroll
      for (int q = 0; q < kMassP; ++q) masks[q][wave] = bal[q];
    __syncthreads();
    const int cnt = lane < 4 * kMassP ? __popcll(masks[lane >> 2][lane & 3]) : 0;
    const int incl = wave_scan_add(cnt);
    const int total = __builtin_amdgcn_readlane(incl, 4 * kMassP - 1);
#pragma unroll
    for (int q = 0; q < kMassP; ++q) {
      const int off = __builtin_amdgcn_readlane(incl - cnt, q * 4 + wave);
      if ((bal[q] >> lane) & 1ull)
        members[off + __popcll(bal[q] & ((1ull << lane) - 1ull))] = base + q * 256 + tid;
    }
    __syncthreads();
#pragma unroll 4
    for (int x = 0; x < total; ++x) {
      const float* row = A + static_cast<long long>(members[x]) * mg1;
#pragma unroll
      for (int q = 0; q < kMassQ; ++q) s[q] += row[min(m0 + q * 256, mg1 - 1)];
    }
  }
  float* Mt = aw.Mt + (static_cast<long long>(p) * sh.K + j) * mg1;
#pragma unroll
  for (int q = 0; q < kMassQ; ++q)
    if (m0 + q * 256 < mg1) Mt[m0 + q * 256] = s[q];
}

// Compact pass: abar over the carriers' keys (+ the same nonvisual part),
// y~, sum_j M_gj v~_j, the two decomposition terms, l1 and its bound, and
// every per-client statistic.
template <typename T, int DH>
__global__ void __launch_bounds__(64 * kAudW)
audit_compact_kernel(Shape sh, AudWs aw, const T* text_q, const T* comp_k, const T* comp_v, const float* nonvis_lse,
                     float* rows_out, float* vec_out) {
  constexpr int DT = DH / 16;
  __shared__ float red_m[kAudW][kAudRows], red_s[kAudW][kAudRows], lse_s[kAudRows];
  __shared__ float ys[kAudRows * (DH + 1)], ms[kAudRows * (DH + 1)];
  const AudBlock<T, DH> ab(sh, text_q);
  const T* kb = ab.base(sh, comp_k, sh.K);
  const T* vb = ab.base(sh, comp_v, sh.K);
  const float D = ab.lse(sh, kb, sh.K, nonvis_lse, red_m, red_s, lse_s);
  const int mg1 = sh.mg1;
  const float lse_f = ab.rv ? aw.lse[static_cast<long long>(ab.tl.p) * mg1 + ab.m] : 0.f;
  const float* Mt = aw.Mt + static_cast<long long>(ab.tl.p) * sh.K * mg1 + ab.m;
  floatx4 yc[DT], my[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t) yc[t] = my[t] = floatx4{0.f, 0.f, 0.f, 0.f};
  float l1 = 0.f, bound = 0.f;
  const int nt = (sh.K + 15) / 16;
  for (int ct = ab.wave; ct < nt; ct += kAudW) {
    const int c0 = ct * 16 + 4 * ab.kg;
    // wide fp32 heads: a tile's keys and values spill beside the queries and the
    // two messages, so a value row is loaded when its turn comes, and above 192
    // dims the keys too (8 heads, 1296 tokens, 256 carriers, 64 queries: 256 dims
    // 223 -> 199 us an audit, 224 dims 173 -> 167)
    constexpr bool kLean = sizeof(T) == 4 && DH > 160, kLeanKeys = kLean && DH > 192;
    float v[4][DT], mm[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if constexpr (!kLean) ab.values(vb, c0 + e, sh.K, v[e]);
      mm[e] = Mt[static_cast<long long>(min(c0 + e, sh.K - 1)) * mg1];
    }
    floatx4 s;
    if constexpr (kLeanKeys) {
      s = ab.logits_lean(kb, ct, sh.K);
    } else {
      Frag<T> kf[DH / 32];
      ab.keys(kb, ct, sh.K, kf);
      __builtin_amdgcn_sched_barrier(0);
      s = ab.logits(kf);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if constexpr (kLean) {
        __builtin_amdgcn_sched_barrier(0);
        ab.values(vb, c0 + e, sh.K, v[e]);
      }
      const bool ok = c0 + e < sh.K && ab.rv;
      const float a = ok ? __expf(s[e] - D) : 0.f;
      mm[e] = ok ? mm[e] : 0.f;
      if (ok) {
        l1 += fabsf(mm[e] - a);
        bound = fmaxf(bound, fabsf(logf(mm[e]) + lse_f - s[e]));
      }
#pragma unroll
      for (int t = 0; t < DT; ++t) {
        yc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[e][t], a, yc[t], 0, 0, 0);
        my[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[e][t], mm[e], my[t], 0, 0, 0);
      }
    }
  }
  aud_add_waves<DH>(yc, ys, ab.lane, ab.wave);
  aud_add_waves<DH>(my, ms, ab.lane, ab.wave);
  // l1 and bound of a client: its four key groups, then the waves in order
  l1 = add_xor32(add_xor16(l1));
  bound = fmaxf(bound, xor_lane<16>(bound));
  bound = fmaxf(bound, xor_lane<32>(bound));
  if (ab.lane < 16) { red_s[ab.wave][ab.lane] = l1; red_m[ab.wave][ab.lane] = bound; }
  __syncthreads();
  // per-client statistics: 32 lanes per client (waves 2 k and 2 k + 1 take
  // four clients), dims strided over them
  const int q = threadIdx.x >> 5, l = threadIdx.x & 31;
  const bool qv = ab.tl.valid(q);
  const int mq = qv ? ab.tl.mrow(sh, q) : 0;
  const float* yf = aw.Y + (static_cast<long long>(ab.tl.p) * mg1 + mq) * DH;
  float acc[6] = {};
  for (int d = l; d < DH; d += 32) {
    const float y = yf[d], c = ys[q * (DH + 1) + d], mid = ms[q * (DH + 1) + d];
    const float t1 = y - mid, t2 = mid - c, df = y - c;
    acc[0] += y * y;
    acc[1] += c * c;
    acc[2] += y * c;
    acc[3] += df * df;
    acc[4] += t1 * t1;
    acc[5] += t2 * t2;
    if (vec_out && qv) {
      float* vo = vec_out + ((static_cast<long long>(ab.tl.p) * mg1 + mq) * 4) * DH;
      vo[d] = y;
      vo[DH + d] = c;
      vo[2 * DH + d] = t1;
      vo[3 * DH + d] = t2;
    }
  }
#pragma unroll
  for (int k = 0; k < 6; ++k) acc[k] = add_xor16(group16_sum(acc[k]));
  if (l == 0 && qv) {
    float l1s = 0.f, bm = 0.f;
    for (int w = 0; w < kAudW; ++w) { l1s += red_s[w][q]; bm = fmaxf(bm, red_m[w][q]); }
    const long long o = (static_cast<long long>(ab.tl.p) * mg1 + mq) * kAuditRow;
    const float st[kAuditRow] = {acc[0], acc[1], acc[2], acc[3], acc[4], acc[5], l1s, bm};
#pragma unroll
    for (int k = 0; k < kAuditRow; ++k) {
      aw.rowst[o + k] = st[k];
      if (rows_out) rows_out[o + k] = st[k];
    }
  }
}

// Weighted stack over the clients of a problem (sqrt(w_g) y_g): e_M, alpha,
// kappa and the norms; weights NULL = uniform 1 / (Hq T).
__global__ void __launch_bounds__(1024) audit_reduce_kernel(Shape sh, AudWs aw, const float* weights, float* out) {
  __shared__ float red[16];
  const int p = blockIdx.x;
  float s[4] = {0.f, 0.f, 0.f, 0.f};
  float gap = -INFINITY;
  for (int m = threadIdx.x; m < sh.mg1; m += blockDim.x) {
    const int h = m / sh.T, t = m % sh.T;
    const float w = weights ? weights[(static_cast<long long>(p) * sh.hq + h) * sh.T + t] : 1.f / sh.mg1;
    const float* rs = aw.rowst + (static_cast<long long>(p) * sh.mg1 + m) * kAuditRow;
    s[0] += w * rs[0];
    s[1] += w * rs[1];
    s[2] += w * rs[2];
    s[3] += w * rs[3];
    gap = fmaxf(gap, rs[6] - rs[7]);
  }
  const float yy = block_sum(s[0], red), cc = block_sum(s[1], red);
  const float yc = block_sum(s[2], red), dd = block_sum(s[3], red);
  const float gmax = block_max(gap, red);
  if (threadIdx.x == 0) {
    float* o = out + static_cast<long long>(p) * kAuditOut;
    const float ny = sqrtf(yy), nc = sqrtf(cc), nd = sqrtf(dd);
    o[0] = nd / (ny + 1e-8f);
    o[1] = ny > 0.f ? nc / ny : 0.f;
    o[2] = (ny > 0.f && nc > 0.f) ? yc / (ny * nc) : 0.f;
    o[3] = ny;
    o[4] = nc;
    o[5] = nd;
    o[6] = gmax;
    o[7] = 0.f;
  }
}

template <typename T, int DH>
static void audit_passes(const Shape& sh, const AudWs& aw, const void* text_q, const void* vis_k, const void* vis_v,
                         const void* comp_k, const void* comp_v, const int32_t* carrier, const float* nonvis_lse,
                         float* rows_out, float* vec_out, hipStream_t st) {
  const dim3 grid((sh.hg * sh.T + kAudRows - 1) / kAudRows, sh.hkv, sh.B), block(64 * kAudW);
  const T* q = static_cast<const T*>(text_q);
  hipLaunchKernelGGL((audit_full_kernel<T, DH>), grid, block, 0, st, sh, aw, q, static_cast<const T*>(vis_k),
                     static_cast<const T*>(vis_v), nonvis_lse);
  hipLaunchKernelGGL(audit_mass_kernel, dim3(sh.K, (sh.mg1 + 256 * kMassQ - 1) / (256 * kMassQ), sh.B), dim3(256), 0, st,
                     sh, aw, carrier);
  hipLaunchKernelGGL((audit_compact_kernel<T, DH>), grid, block, 0, st, sh, aw, q, static_cast<const T*>(comp_k),
                     static_cast<const T*>(comp_v), nonvis_lse, rows_out, vec_out);
}

hipError_t launch_audit(const Shape& sh, const AudWs& aw, const void* text_q, const void* vis_k,
                        const void* vis_v, const void* comp_k, const void* comp_v, const int32_t* carrier,
                        const float* weights, const float* nonvis_lse, float* rows_out, float* vec_out, float* out,
                        hipStream_t st) {
  switch (sh.dh) {
#define GMC_AUDIT(DH)                                                                                                 \
    case DH:                                                                                                          \
      if (sh.dtype == 0)                                                                                              \
        audit_passes<float, DH>(sh, aw, text_q, vis_k, vis_v, comp_k, comp_v, carrier, nonvis_lse, rows_out, vec_out, st); \
      else                                                                                                            \
        audit_passes<bf16_t, DH>(sh, aw, text_q, vis_k, vis_v, comp_k, comp_v, carrier, nonvis_lse, rows_out, vec_out, st); \
      break;
    GMC_AUDIT(32) GMC_AUDIT(64) GMC_AUDIT(96) GMC_AUDIT(128)
    GMC_AUDIT(160) GMC_AUDIT(192) GMC_AUDIT(224) GMC_AUDIT(256)
#undef GMC_AUDIT
    default: return hipErrorInvalidValue;
  }
  hipLaunchKernelGGL(audit_reduce_kernel, dim3(sh.B), dim3(1024), 0, st, sh, aw, weights, out);
  return hipGetLastError();
}

}  // namespace gmc
