// gumbel_kernel.h — Gumbel-max verification (paper App. G.2, Alg. rs_gumbel)
// and the Gumbel-max draft sampler on gfx950.
//
// Verification keeps the accept loop of the multinomial path (row_stats and
// decide, plus pair_pass when overlaps are requested) and replaces the CDF
// inversion: the token at the emitting position n is
//   argmax_v [log r_v + G_v] = argmax_v r_v / E_v,   E_v = -ln U_v ~ Exp(1),
// with r = max(0, p_n - q_n) after a rejection and r = p_K for the bonus.
// gumbel_pass reads the emitting row (pair) part by part and keeps each
// part's best key and its first index, for the residual and, where the part
// has no residual mass, for p_n (the fallback when no part has any); it also
// sums the overlap of the emitting step.  gumbel_finish combines the parts.
//
// The draft sampler scores z_v s - log2 E_v (log2 units of z/T + G) in one
// read per row, part by part, then combines the parts; T = 0 scores the raw
// logits (the greedy token).
#pragma once

#include "sv_device.h"
#include "verify_kernel.h"

namespace sv {

constexpr uint64_t kTagGumbelVerify = 2;
constexpr uint64_t kTagGumbelSample = 3;
constexpr int kNoIndex = 0x7fffffff;

// E = -ln U for element k (0..7) of a Philox block: word (k >> 1), its top 24
// bits (even k) or bits 8..31 (odd k), U = (bits + 1/2) 2^-24.  The largest
// keys r / E come from U close to 1, where E must keep its relative
// precision: there y = 1 - U is exact in float32 and E = -ln(1 - y) is its
// Taylor series y + y^2/2 + ... + y^6/6 (truncation below 1e-8 relative for
// y < 1/16); elsewhere E = -ln2 log2(U) with the hardware log2 (U exact below
// 1/2, one rounding of at most 2^-25 above, i.e. below 5e-7 relative in E).
__device__ __forceinline__ float exp_variate(const Philox4x64& g, int k) {
  const uint64_t w = g.w[(k >> 1) & 3];
  const uint32_t bits = (k & 1) ? static_cast<uint32_t>((w >> 8) & 0xFFFFFFull) : static_cast<uint32_t>(w >> 40);
  constexpr float kInv24 = 5.9604644775390625e-8f;  // 2^-24
  constexpr float kHalf24 = 2.98023223876953125e-8f;  // 2^-25
  // one conversion (exact: bits < 2^24); u = (bits + 1/2) 2^-24 rounded once
  // by an FMA, y = 1 - bits 2^-24 (exact) - 2^-25, exact wherever it is used
  // (y < 1/16, where it has at most 21 significant bits)
  const float f = static_cast<float>(bits);
  const float y = fmaf(-f, kInv24, 1.0f) - kHalf24;
  const float u = fmaf(f, kInv24, kHalf24);
  // both forms, then a select: no divergent branch per element; the series
  // in Horner form with fused multiply-adds (5 FMAs and a multiply)
  const float series =
      y * fmaf(y, fmaf(y, fmaf(y, fmaf(y, fmaf(y, 0.166666672f, 0.2f), 0.25f), 0.333333343f), 0.5f), 1.f);
  const float viaLog = -0.693147182f * __builtin_amdgcn_logf(u);
  return y < 0.0625f ? series : viaLog;
}

struct GumbelBest {  // one part of the emitting row
  float kr;          // largest r / E over the part (-1 or 0: no residual mass)
  int ir;            // its first index
  float kp;          // largest p / E (fallback to p_n)
  int ip;
};

// ---------------------------------------------------------------------------
// The scan of a row part for its best key, bound by the VALU: one Philox
// block (about 280 instructions) gives the variates of eight elements, and
// the variates' logarithms, quotients and comparisons cost as much again
// where every element goes through them.  Almost no element needs them:
//  - E = -ln U >= y for any lower bound y of 1 - U, and y comes from 23 of
//    the 24 bits with two instructions (var_bound), so an upper bound of the
//    key needs one logarithm (sampler) or none (verification).  Only a wave
//    one of whose elements reaches the best key so far forms exact keys;
//  - y >= 2^-25, so a block of eight elements whose largest weight times
//    2^25 stays below the best key needs no variates at all.  The blocks
//    that do are packed through a queue in LDS, so that every lane of a wave
//    that draws variates has a block to draw them for.
// The best key so far is that of the workgroup (kept in LDS); a bound equal
// to it still counts, so the result is the one of comparing every element,
// the first index among equal keys included.  Each lane takes eight
// consecutive elements (one 16-byte vector of bfloat16, two of float32).
// A block costs about 700 cycles for its Philox rounds and 1010 with the
// bounds, 1430 to 1570 with the exact keys (of a wave, at 5 to 8 waves per
// SIMD).  R = 768 rows of V = 151936, spreads 1 to 8: the sampler 152.7 ->
// 107 us a call in bfloat16, 231 -> 127 in float32; rows with one token 22
// above the rest 153 -> 87; Gumbel-max verification at B = 256, K = 3 258 ->
// 207 with overlaps, 183 -> 145 without.
constexpr int kScanQueue = 128;          // queue entries per wave: a step adds up to 64 to fewer than 64
constexpr int kScanTile = kThreads * 8;  // elements per workgroup and step, a block per lane
constexpr float kVarMax = 25.01f;                     // -log2 E < 25 + 1e-7

// t with 2 t <= 1 - U (0 where the bound says nothing): f = 1/2 + the top 23
// bits times 2^-24, t = (1 - 2^-24) - f (exact).
__device__ __forceinline__ float var_bound(const Philox4x64& g, int k) {
  const uint64_t w = g.w[k >> 1];
  const uint32_t x = (k & 1) ? static_cast<uint32_t>(w) : static_cast<uint32_t>(w >> 32);
  const float f = __uint_as_float(0x3f000000u | (x >> 9));
  return 0.999999940395355224609375f - f;
}

// Floats ordered as signed integers, for the workgroup's best key in LDS.
__device__ __forceinline__ int key_order(float v) {
  const int i = __float_as_int(v);
  return i ^ ((i >> 31) & 0x7fffffff);
}
__device__ __forceinline__ float key_unorder(int i) { return __int_as_float(i ^ ((i >> 31) & 0x7fffffff)); }

struct ScanShared {
  float q[kWaves][8][kScanQueue];
  int qv[kWaves][kScanQueue];
  int best;  // key_order of the workgroup's best key
};

// The keys of the draft sampler: weight a = z s, key a - log2 E.  A weight that
// is NaN or +inf may come from a finite logit whose product overflows, so the
// data-error test then looks at the logits (kLogits).
struct KeyScore {
  static constexpr bool kLogits = true;
  float lo;  // the best key so far, less the rounding of a key near it
  static constexpr float kNone = -INFINITY;
  __device__ __forceinline__ void set(float thr) { lo = thr - (1e-3f + 1e-6f * fabsf(thr)); }
  // whether a block whose largest weight is mx can hold such a key (NaN and +inf can)
  __device__ __forceinline__ bool block(float mx) const { return !(mx + kVarMax < lo); }
  __device__ __forceinline__ float bound(float a, float t) const { return a - __builtin_amdgcn_logf(t); }
  __device__ __forceinline__ bool reaches(float mx) const { return !(mx - 1.f < lo); }
  static __device__ __forceinline__ float key(float a, float e) { return a - __builtin_amdgcn_logf(e); }
  static __device__ __forceinline__ bool counts(float a) { return a > -INFINITY; }
};

// The keys of verification: weight r >= 0 (a probability or a residual), key r / E.
struct KeyRatio {
  static constexpr bool kLogits = false;
  float c25, c2;  // the best key so far, less its rounding, times 2^-25 and times 2
  static constexpr float kNone = 0.f;
  __device__ __forceinline__ void set(float thr) {
    c2 = thr * 1.9999f;
    c25 = thr * 2.9799e-8f;
  }
  __device__ __forceinline__ bool block(float mx) const { return mx > 0.f && mx >= c25; }
  __device__ __forceinline__ float bound(float r, float t) const { return fmaf(-c2, t, r); }
  __device__ __forceinline__ bool reaches(float mx) const { return mx >= 0.f; }
  static __device__ __forceinline__ float key(float r, float e) { return __fdividef(r, e); }
  static __device__ __forceinline__ bool counts(float r) { return r > 0.f; }
};

// Eight consecutive logits from element v0 (-inf at and beyond V).
template <class E>
struct Block8 {
  static constexpr int NV = 8 / E::EPV;
  typename E::vec w[NV];
  __device__ __forceinline__ void load(const typename E::raw* row, int v0, int V) {
    const int off = v0 + 8 <= V ? v0 : 0;
#pragma unroll
    for (int h = 0; h < NV; ++h)
      w[h] = load_vec<E>(row + off + h * E::EPV);
  }
  __device__ __forceinline__ void widen(float (&x)[8]) const {
#pragma unroll
    for (int h = 0; h < NV; ++h) {
      float y[E::EPV];
      E::widen(w[h], y);
#pragma unroll
      for (int k = 0; k < E::EPV; ++k) x[h * E::EPV + k] = y[k];
    }
  }
};
template <class E>
__device__ __forceinline__ void block_elements(const typename E::raw* row, int v0, int V, float (&x)[8]) {
#pragma unroll
  for (int k = 0; k < 8; ++k) x[k] = v0 + k < V ? E::one(row + v0 + k) : -INFINITY;
}

// The best key and its first index over the elements [e0, e1) of one row
// (e0 a multiple of kScanTile), whole workgroup.  weight(v0, x, y, r) turns a
// block's logits (x of row rx, y of row ry where BOTH) into its weights.
// row_best (may be null): the best key that any part of the row has found so
// far, as key_order; it starts at kNone, and a bound below it at any time is
// below the row's best key, so the results don't depend on when it is read.
// Every thread receives the results: Key::kNone and kNoIndex where no element
// counts.  *bad (sampler): whether a logit is NaN or +inf.
template <class E, class Key, bool BOTH, class Weight>
__device__ __forceinline__ void gumbel_scan(const typename E::raw* rx, const typename E::raw* ry, int e0,
                                            int e1, int V, uint64_t c0, uint64_t c2, uint64_t tag,
                                            uint64_t seed, Weight weight, int* row_best, ScanShared& sh,
                                            RedLds<4>& red, RedLds<1>& red1, float* best, int* index, bool* bad) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  Key key;
  float bk = Key::kNone;
  int bi = kNoIndex;
  bool isbad = false;
  int qn = 0;  // entries of this wave's queue
  const bool vec = V >= 8;
  Block8<E> nx, ny;
  auto load = [&](int es) {
    const int v0 = es + static_cast<int>(threadIdx.x) * 8;
    nx.load(rx, v0 < e1 ? v0 : V, V);
    if (BOTH) ny.load(ry, v0 < e1 ? v0 : V, V);
  };
  if (vec && e0 < e1) load(e0);
  if (threadIdx.x == 0)
    sh.best = row_best ? __hip_atomic_load(row_best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : key_order(Key::kNone);
  __syncthreads();
  for (int es = e0; es < e1; es += kScanTile) {
    const bool last = es + kScanTile >= e1;
    float thr = key_unorder(__hip_atomic_load(&sh.best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
    key.set(thr);
    Block8<E> wx, wy;
    if (vec) {  // this step's blocks, and the loads of the next step's behind them
      wx = nx;
      if (BOTH) wy = ny;
      if (!last) load(es + kScanTile);
    }
    const int v0 = es + static_cast<int>(threadIdx.x) * 8;
    float x[8], y[8], r[8];
    if (vec && v0 + 8 <= V) {
      wx.widen(x);
      if (BOTH) wy.widen(y);
    } else {
      block_elements<E>(rx, v0, V, x);
      if (BOTH) block_elements<E>(ry, v0, V, y);
    }
    weight(x, y, r);
    float mx = r[0];
#pragma unroll
    for (int k = 1; k < 8; ++k) mx = max_nan(mx, r[k]);
    if (Key::kLogits && !(mx < INFINITY)) {
#pragma unroll
      for (int k = 0; k < 8; ++k) isbad |= !(x[k] < INFINITY);
    }
    const bool need = v0 < e1 && v0 < V && key.block(mx);
    const uint64_t m = __ballot(need);
    if (need) {
      const int at = qn + static_cast<int>(__builtin_amdgcn_mbcnt_hi(
                              static_cast<uint32_t>(m >> 32),
                              __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0u)));
#pragma unroll
      for (int k = 0; k < 8; ++k) sh.q[wave][k][at] = r[k];
      sh.qv[wave][at] = v0;
    }
    qn += __popcll(m);
    while (qn >= 64 || (last && qn > 0)) {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      const int first = qn >= 64 ? qn - 64 : 0;
      const bool on = first + lane < qn;
      const int at = on ? first + lane : first;
      const int vq = sh.qv[wave][at];
      float rq[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) rq[k] = sh.q[wave][k][at];
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      qn = first;
      const Philox4x64 g = philox4x64_10(c0, static_cast<uint64_t>(static_cast<uint32_t>(vq) >> 3), c2, tag, seed, 0ull);
      float mq = key.bound(rq[0], var_bound(g, 0));
#pragma unroll
      for (int k = 1; k < 8; ++k) mq = max_nan(mq, key.bound(rq[k], var_bound(g, k)));
      const bool cand = on && key.reaches(mq);
      if (__ballot(cand) != 0) {
        if (cand) {
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            const float kk = Key::key(rq[k], exp_variate(g, k));
            const bool better = Key::counts(rq[k]) & ((kk > bk) | ((kk == bk) & (vq + k < bi)));
            bk = better ? kk : bk;
            bi = better ? vq + k : bi;
          }
        }
        const float wb = wave_max(bk);
        if (wb > thr) {
          if (lane == 0) atomicMax(&sh.best, key_order(wb));
          thr = wb;
          key.set(thr);
        }
      }
    }
  }
  // the workgroup's best key, its first index, and the data-error flag
  float v[4] = {bk, isbad ? 1.f : 0.f, -INFINITY, -INFINITY};
  wg_max<4>(v, red);
  *index = wg_min_int(bk == v[0] ? bi : kNoIndex, red1);
  *best = v[0];
  *bad = v[1] > 0.f;
  if (row_best && threadIdx.x == 0 && *index != kNoIndex)
    __hip_atomic_fetch_max(row_best, key_order(v[0]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One workgroup per (batch row, part): parts of `tiles` tiles (kScanTile
// elements each) spread evenly over P workgroups.
__device__ __forceinline__ void scan_part(int V, int P, int part, int* e0, int* e1) {
  const int tiles = (V + kScanTile - 1) / kScanTile;
  *e0 = static_cast<int>(static_cast<int64_t>(part) * tiles / P) * kScanTile;
  const int64_t end = static_cast<int64_t>(part + 1) * tiles / P * kScanTile;
  *e1 = end < V ? static_cast<int>(end) : V;
}

template <class E>
__global__ __launch_bounds__(kThreads) void gumbel_pass_kernel(VerifyArgs a, GumbelBest* __restrict__ best, int P) {
  __shared__ ScanShared scan;
  __shared__ RedLds<4> red;
  __shared__ RedLds<1> red1;
  const RowsDesc& d = a.rows;
  const int K = a.K;
  const int b = static_cast<int>(blockIdx.x) / P, part = static_cast<int>(blockIdx.x) - b * P;
  const int n = a.decision[b];
  if (n < 0) return;  // data error: decide has written the row
  const bool residual = n < K;
  int bb, e0, e1;
  bool bad;
  const typename E::raw* rt = row_of<E>(d, target_row(a, b, n), &bb);
  const typename E::raw* rd = row_of<E>(d, draft_row(a, b, residual ? n : 0), &bb);
  const float s = scale_of(temperature_of(d, b));
  const RowNorm nt = a.norms[target_row(a, b, n)];
  const RowNorm nd = a.norms[draft_row(a, b, residual ? n : 0)];
  scan_part(d.V, P, part, &e0, &e1);
  GumbelBest o;
  o.kr = -1.f;
  o.ir = kNoIndex;
  o.kp = -1.f;
  o.ip = kNoIndex;
  if (residual) {
    // float32 over eight blocks (64 elements) of a thread, float64 beyond, like the
    // other steps' overlaps (float64 from each block on: the sum keeps the
    // exponentials' common error, +6e-8, of which the rounding of the float32
    // sums hides a third)
    double al = 0.0;
    float sum = 0.f;
    int blocks = 0;
    gumbel_scan<E, KeyRatio, true>(
        rt, rd, e0, e1, d.V, static_cast<uint64_t>(b), a.offset, kTagGumbelVerify, a.seed,
        [&](const float (&x)[8], const float (&y)[8], float (&r)[8]) {
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            const float p = prob(x[k], s, nt.M, nt.invD);
            const float mn = fminf(p, prob(y[k], s, nd.M, nd.invD));
            r[k] = p - mn;
            sum += mn;
          }
          if ((++blocks & 7) == 0) {
            al += static_cast<double>(sum);
            sum = 0.f;
          }
        },
        nullptr, scan, red, red1, &o.kr, &o.ir, &bad);
    if (a.overlap) {  // the step's overlap over this part (pair_pass_kernel leaves the step out)
      double v[4] = {al + static_cast<double>(sum), 0.0, 0.0, 0.0};
      wg_sum<4>(v, red);
      if (threadIdx.x == 0) a.pairs[(static_cast<int64_t>(b) * K + n) * d.C + part].alpha = v[0];
    }
  }
  // p_n itself: the bonus row, or the fallback of a row without residual
  // mass, of which every part is without
  if (!(o.kr > 0.f)) {
    gumbel_scan<E, KeyRatio, false>(
        rt, rt, e0, e1, d.V, static_cast<uint64_t>(b), a.offset, kTagGumbelVerify, a.seed,
        [&](const float (&x)[8], const float (&)[8], float (&r)[8]) {
#pragma unroll
          for (int k = 0; k < 8; ++k) r[k] = prob(x[k], s, nt.M, nt.invD);
        },
        nullptr, scan, red, red1, &o.kp, &o.ip, &bad);
  }
  if (threadIdx.x == 0) best[static_cast<int64_t>(b) * P + part] = o;
}

// Wave-wide argmax over C chunk entries (key, first index), every lane gets it.
__device__ __forceinline__ void wave_argmax(float& key, int& idx) {
  float m = key;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
  idx = wave_min_int(key == m ? idx : kNoIndex);
  key = m;
}

// One wave per batch row: overlaps and the Gumbel-max token.
__global__ __launch_bounds__(kThreads) void gumbel_finish_kernel(VerifyArgs a, const GumbelBest* __restrict__ best,
                                                                   int P) {
  const int b = blockIdx.x * kWaves + (threadIdx.x >> 6);
  if (b >= a.B) return;
  const int lane = threadIdx.x & 63;
  const int K = a.K, C = a.rows.C;
  const int n = a.decision[b];
  if (n < 0) return;
  const GumbelBest* gb = best + static_cast<int64_t>(b) * P;
  float kr = -1.f, kp = -1.f;
  int ir = kNoIndex, ip = kNoIndex;
  for (int cc = lane; cc < P; cc += 64) {  // parts in order: strict ">" keeps the first
    const GumbelBest e = gb[cc];
    if (e.kr > kr) { kr = e.kr; ir = e.ir; }
    if (e.kp > kp) { kp = e.kp; ip = e.ip; }
  }
  wave_argmax(kr, ir);
  wave_argmax(kp, ip);
  for (int i = 0; i < K && a.overlap != nullptr; ++i) {
    double x = 0.0;
    const PairStat* ps = a.pairs + static_cast<int64_t>(b * K + i) * C;
    // per chunk, or per part where the Gumbel pass summed it
    for (int cc = lane; cc < (i == n ? P : C); cc += 64) x += ps[cc].alpha;
    x = wave_sum(x);
    if (lane == 0) a.overlap[static_cast<int64_t>(b) * K + i] = static_cast<float>(x);
  }
  // the residual's argmax, or p_n's when the residual has no mass
  if (lane == 0) a.emitted[static_cast<int64_t>(b) * (K + 1) + n] = (kr > 0.f) ? ir : (kp > 0.f ? ip : -1);
}

// ---------------------------------------------------------------------------
// Gumbel-max draft sampler

struct SampleBest {  // one part of a row
  float k;           // best key (-inf: none)
  int i;             // its first index (kNoIndex: none), or -1 for a data error in the part
};

struct GumbelSampleArgs {
  RowsDesc rows;  // tper = 1, nb = R rows
  int R;
  uint64_t seed, offset;
  int32_t* token;
  SampleBest* best;  // [R][P]
  int P;             // parts per row
  int* row_best;     // [R]: the row's best key so far, as key_order (null: not shared)
};
__global__ __launch_bounds__(kThreads) void gumbel_sample_init_kernel(GumbelSampleArgs a) {
  const int r = blockIdx.x * kThreads + threadIdx.x;
  if (r < a.R) a.row_best[r] = key_order(KeyScore::kNone);
}

// One workgroup per (row, part).  A greedy row (T = 0) compares its logits.
template <class E>
__global__ __launch_bounds__(kThreads) void gumbel_sample_pass_kernel(GumbelSampleArgs a) {
  __shared__ ScanShared scan;
  __shared__ RedLds<4> red;
  __shared__ RedLds<1> red1;
  const RowsDesc& d = a.rows;
  const int V = d.V, P = a.P;
  // every row's first part, then every row's second part, ...: a part starts
  // with the best key of the parts before it
  const int part = static_cast<int>(blockIdx.x) / a.R, r = static_cast<int>(blockIdx.x) - part * a.R;
  int bb, e0, e1;
  const typename E::raw* row = row_of<E>(d, r, &bb);
  const float T = temperature_of(d, r);
  const float s = temperature_ok(T) ? scale_of(T) : 1.0f;
  scan_part(V, P, part, &e0, &e1);
  float ks = -INFINITY;
  int is = kNoIndex;
  bool bad = false;
  if (T == 0.f) {
    for (int es = e0; es < e1; es += kScanTile) {
      const int v0 = es + static_cast<int>(threadIdx.x) * 8;
      float x[8];
      if (v0 + 8 <= V) {
        Block8<E> w;
        w.load(row, v0, V);
        w.widen(x);
      } else {
        block_elements<E>(row, v0, V, x);
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        if (x[k] != x[k] || x[k] == INFINITY) bad = true;
        if (x[k] > ks) { ks = x[k]; is = v0 + k; }
      }
    }
    float m[4] = {ks, bad ? 1.f : 0.f, -INFINITY, -INFINITY};
    wg_max<4>(m, red);
    is = wg_min_int(ks == m[0] ? is : kNoIndex, red1);
    ks = m[0];
    bad = m[1] > 0.f;
  } else {
    gumbel_scan<E, KeyScore, false>(
        row, row, e0, e1, V, static_cast<uint64_t>(r), a.offset, kTagGumbelSample, a.seed,
        [&](const float (&x)[8], const float (&)[8], float (&w)[8]) {
#pragma unroll
          for (int k = 0; k < 8; ++k) w[k] = x[k] * s;
        },
        a.row_best ? a.row_best + r : nullptr, scan, red, red1, &ks, &is, &bad);
  }
  if (threadIdx.x == 0) {
    SampleBest o;
    o.k = ks;
    o.i = bad ? -1 : is;
    a.best[static_cast<int64_t>(r) * P + part] = o;
  }
}

// One wave per row: the best chunk's token, or -1 for a data error.
__global__ __launch_bounds__(kThreads) void gumbel_sample_finish_kernel(GumbelSampleArgs a) {
  const int r = blockIdx.x * kWaves + (threadIdx.x >> 6);
  if (r >= a.R) return;
  const int lane = threadIdx.x & 63;
  const SampleBest* gb = a.best + static_cast<int64_t>(r) * a.P;
  float k = -INFINITY;
  int i = kNoIndex, bad = 0;
  for (int cc = lane; cc < a.P; cc += 64) {
    const SampleBest e = gb[cc];
    if (e.k > k) { k = e.k; i = e.i; }
    bad |= e.i < 0 ? 1 : 0;
  }
  wave_argmax(k, i);
  bad = -wave_min_int(-bad);
  if (lane == 0) {
    const float T = temperature_of(a.rows, r);
    const bool t_ok = T == 0.f || temperature_ok(T);
    a.token[r] = (t_ok && !bad && k > -INFINITY && i != kNoIndex) ? i : -1;
  }
}

}  // namespace sv
