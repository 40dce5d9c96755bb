// resident_kernel.h — the TV loss with every logit read once: each
// (target, draft) pair stays in registers from its first read until its
// gradient is written.
//
// A pair is spread over a group of G workgroups, one per slice of the
// vocabulary (up to NV tiles of one vector per thread), and a position's K
// pairs over K such groups, since the gradient of a step needs the overlaps
// of all of them.  The K * G workgroups of a position exchange their partial
// sums twice through records in the workspace:
//   1 load the slice of both rows; per-slice statistics (m, D) of each row;
//     exchange -> the two row normalisers;
//   2 alpha, S and 1 - S over the slice; the element's draft exponential and
//     its indicator 1[q <= p] replace the two logits in their registers;
//     exchange -> every step's alpha, S -> the chain factors;
//   3 write the gradient from the registers, and issue the next position's
//     loads of a tile as soon as the tile's registers are free.
// Against the passes that read the pair again for each stage this moves 8
// instead of 14 bytes per bfloat16 pair element.
//
// Workgroups take tickets in the order they start, and a group is K * G
// consecutive tickets, so that every group but the last one started is
// complete: a complete group finishes without waiting for a workgroup that
// has not started, whatever else runs on the device.  Every wait is bounded
// all the same; a wait that gives up raises a flag that turns the loss into
// NaN.  The records start as all ones (kRecordEmpty) and each is one 64-bit
// word, complete once it is not; all exchanges are relaxed agent-scope
// atomics of whole words, so no fence is needed.  The partial sums are added
// in slice order, so the results do not depend on timing.
#pragma once

#include "fused_kernel.h"
#include "tv_kernel.h"

namespace sv {

constexpr int kResThreads = 512;
constexpr int kResWaves = kResThreads / 64;
constexpr int kResMaxGroup = 40;   // workgroups of one position (K * G)
constexpr int kResMaxSlices = 16;  // G
constexpr int kResWords = 6;       // exchange words per slice: (m, D, D) and (alpha, S, 1 - S)
constexpr int kResHeadWords = 8;   // ticket and failure flag, before the records

// Tiles per row and slice held in registers: bfloat16 takes 4 registers per
// tile and pair, float32 8, 152 of the 256 that one workgroup per CU leaves
// each thread.  A pair of V = 151936 bfloat16 logits then spans two CUs.
// Smaller slices with more workgroups per CU wait longer for each other's
// records than they gain by overlapping: N = 4096, K = 3 takes 3.57 ms with
// this shape, 3.94 ms with two workgroups of 128 registers per CU, 4.24 with
// four of 256 threads, 3.75 with 1024 threads at 128 registers.
template <class E> struct ResCap;
template <> struct ResCap<BF16H> { static constexpr int NV = 38; };
template <> struct ResCap<F32> { static constexpr int NV = 19; };

// What the registers of a tile hold once its logits are consumed: the four
// signed draft exponentials.
__device__ __forceinline__ void res_put(u32x2& t, u32x2& d, const float (&o)[4]) {
  t.x = __float_as_uint(o[0]); t.y = __float_as_uint(o[1]);
  d.x = __float_as_uint(o[2]); d.y = __float_as_uint(o[3]);
}
__device__ __forceinline__ void res_get(const u32x2& t, const u32x2& d, float (&o)[4]) {
  o[0] = __uint_as_float(t.x); o[1] = __uint_as_float(t.y);
  o[2] = __uint_as_float(d.x); o[3] = __uint_as_float(d.y);
}
__device__ __forceinline__ void res_put(u32x4& t, u32x4&, const float (&o)[4]) {
  t.x = __float_as_uint(o[0]); t.y = __float_as_uint(o[1]);
  t.z = __float_as_uint(o[2]); t.w = __float_as_uint(o[3]);
}
__device__ __forceinline__ void res_get(const u32x4& t, const u32x4&, float (&o)[4]) {
  o[0] = __uint_as_float(t.x); o[1] = __uint_as_float(t.y);
  o[2] = __uint_as_float(t.z); o[3] = __uint_as_float(t.w);
}
__device__ __forceinline__ u32x2 res_neg_inf(const BF16H*) { return u32x2{0xFF80FF80u, 0xFF80FF80u}; }
__device__ __forceinline__ u32x4 res_neg_inf(const F32*) {
  return u32x4{0xFF800000u, 0xFF800000u, 0xFF800000u, 0xFF800000u};
}

// The vector's elements moved down by n (0 to 4), -inf from the top.
__device__ __forceinline__ void res_shift(u32x2& w, int n) {
  const uint64_t ninf = 0xFF80FF80FF80FF80ull;
  uint64_t v = (static_cast<uint64_t>(w.y) << 32) | w.x;
  v = n == 0 ? v : (n >= 4 ? ninf : (v >> (16 * n)) | (ninf << (64 - 16 * n)));
  w.x = static_cast<uint32_t>(v);
  w.y = static_cast<uint32_t>(v >> 32);
}
__device__ __forceinline__ void res_shift(u32x4& w, int n) {
  const uint32_t ninf = 0xFF800000u;
  const uint32_t a = w.x, b = w.y, c = w.z, d = w.w;
  w.x = n == 0 ? a : (n == 1 ? b : (n == 2 ? c : (n == 3 ? d : ninf)));
  w.y = n == 0 ? b : (n == 1 ? c : (n == 2 ? d : ninf));
  w.z = n == 0 ? c : (n == 1 ? d : ninf);
  w.w = n == 0 ? d : ninf;
}

// Opaque to the compiler: values derived from a held register (widened
// logits, tile conditions) are formed again after this point instead of being
// kept in registers of their own.
__device__ __forceinline__ void res_opaque(u32x2& w) { asm volatile("" : "+v"(w.x), "+v"(w.y)); }
__device__ __forceinline__ void res_opaque(u32x4& w) {
  asm volatile("" : "+v"(w.x), "+v"(w.y), "+v"(w.z), "+v"(w.w));
}
__device__ __forceinline__ int res_opaque_s(int v) {
  asm volatile("" : "+s"(v));
  return v;
}

struct ResArgs {
  int G;           // slices per row
  int tiles;       // tiles per row
  int groups;      // position groups of the launch
  uint32_t* head;  // [0] ticket counter (starts all ones), [2] failure flag (0: a wait gave up)
  uint64_t* rec;   // [N][K][G][kResWords]
  unsigned spin_limit;
};

struct ResLds {
  double red[kResWaves][4];
  double x[kResMaxGroup * 3];
  float c[8];   // rt, rd, tau, -, A1, A0
  double cc[2]; // cT, cD
  uint32_t ticket;
  int fail;
};

__device__ __forceinline__ uint64_t res_word(double v) {
  const uint64_t w = static_cast<uint64_t>(__double_as_longlong(v));
  return w == kRecordEmpty ? w - 1 : w;
}
__device__ __forceinline__ uint64_t res_word(float a, float b) {
  const uint64_t w = (static_cast<uint64_t>(__float_as_uint(b)) << 32) | __float_as_uint(a);
  return w == kRecordEmpty ? w - 1 : w;
}

// One wave: `W` consecutive words of the lanes with `on`, once they are
// complete, or kRecordEmpty in the place of a word where the wait gave up
// (*ok false).
template <int W>
__device__ __forceinline__ void res_wait(const uint64_t* p, bool on, unsigned limit, uint64_t (&v)[W], bool* ok) {
#pragma unroll
  for (int i = 0; i < W; ++i) v[i] = on ? kRecordEmpty : 0;
  for (unsigned s = 0; s < limit; ++s) {
    bool wait = false;
#pragma unroll
    for (int i = 0; i < W; ++i)
      if (on) v[i] = ld_agent(p + i);
#pragma unroll
    for (int i = 0; i < W; ++i) wait = wait || v[i] == kRecordEmpty;
    if (__ballot(wait) == 0) return;
    __builtin_amdgcn_s_sleep(1);
  }
  *ok = false;
}

// One wave: the statistics (m, D) of up to 64 parts, one per lane (-inf, 0
// in the lanes without one), combined; every lane gets the result.
__device__ __forceinline__ void res_combine(float& m, double& D) {
  const float mw = wave_max(m);
  if (D == D) D = m == -INFINITY ? 0.0 : D * static_cast<double>(__builtin_amdgcn_exp2f(m - mw));
  D = wave_sum(D);
  m = mw;
}

__device__ __forceinline__ float res_uniform(float v) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

// (m, D) of one row's slice held in w[]: per thread a running reference over
// CH tiles at a time, then over the workgroup's 64-lane waves.
template <class E, int NV>
__device__ __forceinline__ void res_stats(const typename E::vec (&w)[NV], float s, float* m, double* D) {
  constexpr int CH = 5;
  float ref = -INFINITY;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j0 = 0; j0 < NV; j0 += CH) {
    float mx = -INFINITY;
#pragma unroll
    for (int j = j0; j < j0 + CH && j < NV; ++j) {
      float x[4];
      E::widen(w[j], x);
#pragma unroll
      for (int k = 0; k < 4; ++k) mx = max_nan(mx, x[k]);
    }
    const float nr = max_nan(ref, mx * s);
    if (nr != -INFINITY) {
      const float f = ref == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ref - nr);
#pragma unroll
      for (int k = 0; k < 4; ++k) acc[k] *= f;
#pragma unroll
      for (int j = j0; j < j0 + CH && j < NV; ++j) {
        float x[4];
        E::widen(w[j], x);
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[k] += __builtin_amdgcn_exp2f(fmaf(x[k], s, -nr));
      }
      ref = nr;
    }
  }
  const float wm = wave_max(ref);
  double d = (static_cast<double>(acc[0]) + static_cast<double>(acc[1])) +
             (static_cast<double>(acc[2]) + static_cast<double>(acc[3]));
  if (d == d) d = ref == -INFINITY ? 0.0 : d * static_cast<double>(__builtin_amdgcn_exp2f(ref - wm));
  *m = wm;
  *D = wave_sum(d);
}

// Moves 8 bytes per bfloat16 pair element (both logits read, the gradient
// written) against the 14 of the passes in tv_kernel.h.  Bound by the parts
// of a position that do not overlap on a CU: of 35 us per position (V =
// 151936, G = 2), 15 write the gradient and issue the next loads, 8 wait for
// those and sum the statistics, 7 are the second sums' arithmetic and 6 the
// two exchanges (time stamps per phase).  N = 4096, K = 3, V = 151936: 4.82
// -> 3.49 ms a call in bfloat16; N = 1024 in float32 1.92 -> 1.30 ms.
template <class E, int NV>
__global__ __launch_bounds__(kResThreads, 2) void tv_resident_kernel(TvArgs a, ResArgs r) {
  using vec = typename E::vec;
  constexpr int EPV = E::EPV;
  static_assert(EPV == 4, "four elements per vector");
  constexpr int TILE = kResThreads * EPV;
  __shared__ ResLds sh;
  const RowsDesc& d = a.rows;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int K = a.K, V = d.V, G = r.G, PG = K * G;
  if (tid == 0) {
    sh.ticket = atomicAdd(r.head, 1u) + 1u;
    sh.fail = 0;
  }
  __syncthreads();
  const int tk = __builtin_amdgcn_readfirstlane(static_cast<int>(sh.ticket));
  const int grp = tk / PG, mem = tk - grp * PG;
  const int k = mem / G, w = mem - k * G;
  const int t0 = static_cast<int>(static_cast<int64_t>(w) * r.tiles / G);
  const int nt = static_cast<int>(static_cast<int64_t>(w + 1) * r.tiles / G) - t0;
  // slot j holds tile tb + j, for the slots from NV - nt: the slice's last
  // tile, the only one that can reach past the row, is in the last slot
  const int j0 = NV - nt, tb = t0 - j0;
  const float s = scale_of(d.temp_scalar);
  vec xt[NV], xd[NV];
#pragma unroll
  for (int j = 0; j < NV; ++j) xt[j] = xd[j] = res_neg_inf(static_cast<const E*>(nullptr));

  // byte offset of this thread's vector inside a tile; in the last slot the
  // last `over` elements of a vector lie past the row: the row's last whole
  // vector is read in its place, shifted down and filled with -inf
  const uint32_t voff = static_cast<uint32_t>(tid) * sizeof(vec);
  const int vlast = (tb + NV - 1) * TILE + tid * EPV;
  const int over = min(max(vlast + EPV - V, 0), EPV);
  auto tile_load = [&](const typename E::raw* row, int j) -> vec {
    if (j == NV - 1) return load_vec<E>(row + (over > 0 ? V - EPV : vlast));
    const char* base = reinterpret_cast<const char*>(row + static_cast<int64_t>(tb + j) * TILE);
    return load_any(reinterpret_cast<const typename E::any*>(base + voff));
  };
  auto row_t = [&](int n) {
    return static_cast<const typename E::raw*>(d.tgt) + static_cast<int64_t>(n) * d.tsb + static_cast<int64_t>(k) * d.tsk;
  };
  auto row_d = [&](int n) {
    return static_cast<const typename E::raw*>(d.drf) + static_cast<int64_t>(n) * d.dsb + static_cast<int64_t>(k) * d.dsk;
  };
  if (grp < a.N) {
    const typename E::raw *rt = row_t(grp), *rd = row_d(grp);
#pragma unroll
    for (int j = 0; j < NV; ++j)
      if (j >= j0) {
        xt[j] = tile_load(rt, j);
        xd[j] = tile_load(rd, j);
      }
  }
  for (int n = grp; n < a.N; n += r.groups) {
    res_shift(xt[NV - 1], over);
    res_shift(xd[NV - 1], over);
    float mt, md;
    double Dt, Dd;
    res_stats<E, NV>(xt, s, &mt, &Dt);
    res_stats<E, NV>(xd, s, &md, &Dd);
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      res_opaque(xt[j]);
      res_opaque(xd[j]);
    }
    if (lane == 0) {
      sh.red[wave][0] = static_cast<double>(mt);
      sh.red[wave][1] = Dt;
      sh.red[wave][2] = static_cast<double>(md);
      sh.red[wave][3] = Dd;
    }
    __syncthreads();
    uint64_t* rec = r.rec + (static_cast<int64_t>(n) * K + k) * G * kResWords;
    if (wave == 0) {
      // the workgroup's waves, then the group's slices, one per lane
      float m2[2] = {-INFINITY, -INFINITY};
      double D2[2] = {0.0, 0.0};
      if (lane < kResWaves) {
        m2[0] = static_cast<float>(sh.red[lane][0]);
        D2[0] = sh.red[lane][1];
        m2[1] = static_cast<float>(sh.red[lane][2]);
        D2[1] = sh.red[lane][3];
      }
      res_combine(m2[0], D2[0]);
      res_combine(m2[1], D2[1]);
      bool ok = true;
      if (G > 1) {
        if (lane < 3)
          st_agent(rec + w * kResWords + lane,
                   lane == 0 ? res_word(m2[0], m2[1]) : (lane == 1 ? res_word(D2[0]) : res_word(D2[1])));
        uint64_t v[3];
        res_wait<3>(rec + lane * kResWords, lane < G, r.spin_limit, v, &ok);
        const bool on = lane < G;
        m2[0] = on ? __uint_as_float(static_cast<uint32_t>(v[0])) : -INFINITY;
        m2[1] = on ? __uint_as_float(static_cast<uint32_t>(v[0] >> 32)) : -INFINITY;
        D2[0] = on ? __longlong_as_double(static_cast<long long>(v[1])) : 0.0;
        D2[1] = on ? __longlong_as_double(static_cast<long long>(v[2])) : 0.0;
        res_combine(m2[0], D2[0]);
        res_combine(m2[1], D2[1]);
      }
      // p = 2^(z_t s - rt) cT and q = 2^(z_d s - rd) cD, r the row's
      // M + log2 D rounded to float32 and c = 2^(r - (M + log2 D)) its
      // rounding; q <= p exactly where z_d - z_t <= tau.  Lane 0 forms the
      // target's, lane 1 the draft's.
      const double lz = static_cast<double>(lane == 0 ? m2[0] : m2[1]) + log2(lane == 0 ? D2[0] : D2[1]);
      const float rz = static_cast<float>(lz);
      if (lane < 2) {
        sh.c[lane] = rz;
        sh.cc[lane] = exp2(static_cast<double>(rz) - lz);
      }
      const double td = (dpp::lane(lz, 1) - dpp::lane(lz, 0)) / static_cast<double>(s);
      float tau = static_cast<float>(td);
      if (static_cast<double>(tau) > td) tau = nextafterf(tau, -INFINITY);
      if (lane == 0) {
        sh.c[2] = tau;
        if (!ok) sh.fail = 1;
      }
    }
    __syncthreads();
    float ap = 0.f, aq = 0.f, sc = 0.f;
    {
      const float rt = res_uniform(sh.c[0]), rd = res_uniform(sh.c[1]), tau = res_uniform(sh.c[2]);
      const int jp = res_opaque_s(j0);
#pragma unroll
      for (int j = 0; j < NV; ++j)
        if (j >= jp) {
          float zt[4], zd[4], o[4];
          E::widen(xt[j], zt);
          E::widen(xd[j], zd);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float ep = __builtin_amdgcn_exp2f(fmaf(zt[i], s, -rt));
            const float eq = __builtin_amdgcn_exp2f(fmaf(zd[i], s, -rd));
            const bool le = zd[i] - zt[i] <= tau;
            ap += le ? 0.f : ep;
            aq += le ? eq : 0.f;
            sc += le ? 0.f : eq;
            o[i] = le ? eq : -eq;
          }
          res_put(xt[j], xd[j], o);
        }
    }
    const double sp = wave_sum(static_cast<double>(ap)), sq = wave_sum(static_cast<double>(aq)),
                 sx = wave_sum(static_cast<double>(sc));
    if (lane == 0) {
      sh.red[wave][0] = sp;
      sh.red[wave][1] = sq;
      sh.red[wave][2] = sx;
    }
    __syncthreads();
    if (wave == 0) {
      const bool on = lane < kResWaves;
      const double p = wave_sum(on ? sh.red[lane][0] : 0.0), q = wave_sum(on ? sh.red[lane][1] : 0.0),
                   x = wave_sum(on ? sh.red[lane][2] : 0.0);
      const double cT = sh.cc[0], cD = sh.cc[1];
      // (a target normaliser that is NaN makes S and 1 - S NaN as well)
      const double part[3] = {cT * p + cD * q, cD * q + (cT - cT), cD * x + (cT - cT)};
      if (lane < 3) st_agent(rec + w * kResWords + 3 + lane, res_word(lane == 0 ? part[0] : (lane == 1 ? part[1] : part[2])));
      bool ok = true;
      const uint64_t* all = r.rec + static_cast<int64_t>(n) * PG * kResWords;
      uint64_t v[3];
      res_wait<3>(all + lane * kResWords + 3, lane < PG, r.spin_limit, v, &ok);
      if (lane < PG)
#pragma unroll
        for (int i = 0; i < 3; ++i) sh.x[lane * 3 + i] = __longlong_as_double(static_cast<long long>(v[i]));
      if (lane == 0 && !ok) sh.fail = 1;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      // lane i < K: step i's alpha, S and 1 - S, slices in order
      double al = 0.0, S = 0.0, Sc = 0.0;
      if (lane < K)
        for (int i = 0; i < G; ++i) {
          al += sh.x[(lane * G + i) * 3];
          S += sh.x[(lane * G + i) * 3 + 1];
          Sc += sh.x[(lane * G + i) * 3 + 2];
        }
      double gk, L;
      chain_factor_of(K, a.mode, k, [&](int i) -> double { return dpp::lane(al, i); }, &gk, &L);
      gk = a.scale * gk * static_cast<double>(a.inv_t);
      const double A1 = gk * dpp::lane(Sc, k) * sh.cc[1], A0 = -gk * dpp::lane(S, k) * sh.cc[1];
      if (lane == 0) {
        sh.c[4] = static_cast<float>(A1);
        sh.c[5] = static_cast<float>(A0);
        if (mem == 0) a.loss_pos[n] = a.scale * L;
        if (sh.fail) st_agent(reinterpret_cast<uint64_t*>(r.head + 2), 0ull);
      }
      if (mem == 0 && a.overlap && lane < K) a.overlap[static_cast<int64_t>(n) * K + lane] = static_cast<float>(al);
    }
    __syncthreads();
    if (sh.fail) return;  // (uniform) a wait gave up: the loss becomes NaN
    // the gradient, and the next position's loads of each tile behind it
    const int nn = n + r.groups;
    const bool more = nn < a.N;
    const typename E::raw *rt = row_t(more ? nn : n), *rd = row_d(more ? nn : n);
    const float A1 = res_uniform(sh.c[4]), nA0 = -res_uniform(sh.c[5]);
    float* gr = a.grad + (static_cast<int64_t>(n) * K + k) * V;
    const int jw = res_opaque_s(j0);
#pragma unroll
    for (int j = 0; j < NV; ++j)
      if (j >= jw) {
        float o[4];
        res_get(xt[j], xd[j], o);
        f32x4 g;
        g.x = o[0] * (o[0] < 0.f ? nA0 : A1);
        g.y = o[1] * (o[1] < 0.f ? nA0 : A1);
        g.z = o[2] * (o[2] < 0.f ? nA0 : A1);
        g.w = o[3] * (o[3] < 0.f ? nA0 : A1);
        char* base = reinterpret_cast<char*>(gr + static_cast<int64_t>(tb + j) * TILE);
        if (j < NV - 1 || over == 0) {
          __builtin_nontemporal_store(g, reinterpret_cast<f32x4_any*>(base + static_cast<uint32_t>(tid) * 16u));
        } else {
          if (over < 4) gr[vlast] = g.x;
          if (over < 3) gr[vlast + 1] = g.y;
          if (over < 2) gr[vlast + 2] = g.z;
        }
        if (more) {
          xt[j] = tile_load(rt, j);
          xd[j] = tile_load(rd, j);
        }
      }
  }
}

// The total loss (tv_loss_kernel), NaN where a wait of the resident pass gave up.
__global__ __launch_bounds__(kThreads) void tv_resident_loss_kernel(TvArgs a, const uint32_t* __restrict__ head) {
  __shared__ RedLds<1> red;
  double acc = 0.0;
  for (int p = threadIdx.x; p < a.N; p += kThreads) acc += a.loss_pos[p];
  double v[1] = {acc};
  wg_sum<1>(v, red);
  if (threadIdx.x == 0) *a.loss = head[2] == 0u ? NAN : static_cast<float>(v[0]);
}

}  // namespace sv
