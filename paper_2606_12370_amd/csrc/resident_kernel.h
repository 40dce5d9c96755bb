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
// consecutive tickets and takes positions n = group, group + groups, ...  A
// group whose workgroups have all started finishes whatever else runs on the
// device.  That they all start is not certain: other work may hold the
// device, or a stream's CU mask may be narrower than a group.  So a workgroup
// whose first records stay away waits for its group to become complete, and in
// the end marks an incomplete one as given up; no gradient is written before
// the group is complete.  The workgroups of a marked group leave, those that
// start later too, and tv_resident_finish_kernel computes its positions alone,
// one workgroup a position, slice after slice with the same sums and without
// waiting: the same bits as those of a complete group.  (A launch of its own:
// in the main kernel that code takes registers which cost every call 2 %.)
// The records start as all ones (kRecordEmpty) and each is one 64-bit
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
constexpr int kResSumTiles = 16;   // tiles (of four elements a thread) that a float32 sum spans
constexpr int kResHeadWords = 8;   // 64-bit words of counters before the records
constexpr uint32_t kResGaveUp = 0x10000u;  // added to a group's arrivals (at most kResMaxGroup)

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
  // [0] tickets, [1] finished workgroups of the finish launch, each less one;
  // 0 once a group gave up [2], once a complete group lost a record [3]
  uint32_t* head;
  uint64_t* rec;   // [N][K][G][kResWords]
  uint32_t* state; // [groups]: arrived workgroups less one, plus kResGaveUp
  // polls (about a microsecond each) of a workgroup: for its first position's
  // records before it looks at its group; for the group to become complete, and
  // the same once some group has given up; for a record of a complete group
  unsigned first_polls, group_polls, next_group_polls, record_polls;
  uint32_t hold;  // groups with a bit of it never count as complete (0 except in tests)
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

// One thread of a workgroup of group grp: true once all `need` workgroups of the
// group have started, false once the group has given up, which this one
// marks after its polls.  (A round per arrival may follow: the mark is set
// only on an incomplete group.)
__device__ __forceinline__ bool res_formed(const ResArgs& r, int grp, uint32_t need) {
  uint32_t* st = r.state + grp;
  for (unsigned s = 0;; ++s) {
    const uint32_t v = __hip_atomic_load(st, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t flag = __hip_atomic_load(r.head + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (v + 1u == need) return true;
    if (v + 1u >= kResGaveUp) return false;
    if (s >= (flag == 0u ? r.next_group_polls : r.group_polls)) {
      uint32_t seen = v;
      if (__hip_atomic_compare_exchange_strong(st, &seen, v + kResGaveUp, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT)) {
        __hip_atomic_store(r.head + 2, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return false;
      }
      continue;
    }
    __builtin_amdgcn_s_sleep(1);
  }
}

// Wave 0: three consecutive words of the lanes with `on`, once they are
// complete and (FIRST) the counter *st, less one, is at `need`; false after
// `polls` looks.
template <bool FIRST>
__device__ __forceinline__ bool res_poll(const uint64_t* p, bool on, unsigned polls, const uint32_t* st,
                                         uint32_t need, uint64_t (&v)[3]) {
  for (unsigned s = 0; s < polls; ++s) {
    bool wait = FIRST && threadIdx.x == 0 &&
                __hip_atomic_load(st, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u != need;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      v[i] = on ? ld_agent(p + i) : 0;
      wait = wait || v[i] == kRecordEmpty;
    }
    if (__ballot(wait) == 0) return true;
    __builtin_amdgcn_s_sleep(1);
  }
  return false;
}

// The wait of an exchange; false: the group has given up, or the records of a
// complete group stay away (its workgroups all run, so that takes a device
// that stops one of them for a second; head[3] then makes the loss NaN).  At
// the group's first position (`first`) the group itself must be complete too: a
// complete group is never marked as given up, so no group that is marked has
// written any of its gradient.
template <bool ALONE>
__device__ __forceinline__ bool res_wait(const ResArgs& r, int grp, int PG, bool first, const uint64_t* p, bool on,
                                         uint64_t (&v)[3]) {
  if (!ALONE && first) {
    const uint32_t need = static_cast<uint32_t>(PG) + (static_cast<uint32_t>(grp) & r.hold);
    if (res_poll<true>(p, on, r.first_polls, r.state + grp, need, v)) return true;
    int formed = 0;
    if (threadIdx.x == 0) formed = res_formed(r, grp, need) ? 1 : 0;
    if (__builtin_amdgcn_readfirstlane(formed) == 0) return false;
  }
  const bool ok = res_poll<false>(p, on, ALONE ? 1u << 20 : r.record_polls, nullptr, 0u, v);
  if (!ALONE && !ok && threadIdx.x == 0)
    __hip_atomic_store(r.head + 3, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return ok;
}

// What a workgroup holds of a pair: slice w of step k.  Slot j holds tile
// tb + j, for the slots from j0: the slice's last tile, the only one that can
// reach past the row, is in the last slot.  There the last `over` elements of
// a vector lie past the row: the row's last whole vector is read in its place,
// shifted down and filled with -inf.
struct ResSlice {
  int k, w, mem, j0, tb, vlast, over;
};
template <class E, int NV>
__device__ __forceinline__ ResSlice res_slice_of(const ResArgs& r, int mem, int V) {
  constexpr int TILE = kResThreads * E::EPV;
  ResSlice c;
  c.mem = mem;
  c.k = mem / r.G;
  c.w = mem - c.k * r.G;
  const int t0 = static_cast<int>(static_cast<int64_t>(c.w) * r.tiles / r.G);
  const int nt = static_cast<int>(static_cast<int64_t>(c.w + 1) * r.tiles / r.G) - t0;
  c.j0 = NV - nt;
  c.tb = t0 - c.j0;
  c.vlast = (c.tb + NV - 1) * TILE + static_cast<int>(threadIdx.x) * E::EPV;
  c.over = min(max(c.vlast + E::EPV - V, 0), E::EPV);
  return c;
}
template <class E, int NV>
__device__ __forceinline__ typename E::vec res_tile_load(const ResSlice& c, const typename E::raw* row, int j, int V) {
  constexpr int TILE = kResThreads * E::EPV;
  if (j == NV - 1) return load_vec<E>(row + (c.over > 0 ? V - E::EPV : c.vlast));
  const char* base = reinterpret_cast<const char*>(row + static_cast<int64_t>(c.tb + j) * TILE);
  return load_any(reinterpret_cast<const typename E::any*>(base + threadIdx.x * static_cast<uint32_t>(sizeof(typename E::vec))));
}
template <class E>
__device__ __forceinline__ const typename E::raw* res_row_t(const RowsDesc& d, int n, int k) {
  return static_cast<const typename E::raw*>(d.tgt) + static_cast<int64_t>(n) * d.tsb + static_cast<int64_t>(k) * d.tsk;
}
template <class E>
__device__ __forceinline__ const typename E::raw* res_row_d(const RowsDesc& d, int n, int k) {
  return static_cast<const typename E::raw*>(d.drf) + static_cast<int64_t>(n) * d.dsb + static_cast<int64_t>(k) * d.dsk;
}

// A workgroup's part of position n, its slice loaded in xt / xd; behind the
// gradient the loads of position nn (if below N).  With ALONE one workgroup
// takes all slices of the position in turn, and the call ends after stage
// `stages`: 1 the statistics published, 2 the sums published, 3 the gradient.
// False: the group has given up (or lost a record).
template <class E, int NV, bool ALONE>
__device__ __forceinline__ bool res_position(const TvArgs& a, const ResArgs& r, const ResSlice& c, int n, int nn,
                                             int grp, int stages,
                                             typename E::vec (&xt)[NV], typename E::vec (&xd)[NV], ResLds& sh) {
  constexpr int EPV = E::EPV;
  static_assert(EPV == 4, "four elements per vector");
  constexpr int TILE = kResThreads * EPV;
  const RowsDesc& d = a.rows;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int K = a.K, V = d.V, G = r.G, PG = K * G;
  const float s = scale_of(d.temp_scalar);
  const bool first = !ALONE && n == grp;  // the group may not be complete yet
  res_shift(xt[NV - 1], c.over);
  res_shift(xd[NV - 1], c.over);
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
  uint64_t* rec = r.rec + (static_cast<int64_t>(n) * K + c.k) * G * kResWords;
  bool ok = true;  // (wave 0) the group has not given up
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
    if (ALONE && stages == 1 && G == 1) return true;
    if (G > 1) {
      if (lane < 3)
        st_agent(rec + c.w * kResWords + lane,
                 lane == 0 ? res_word(m2[0], m2[1]) : (lane == 1 ? res_word(D2[0]) : res_word(D2[1])));
      if (ALONE && stages == 1) return true;
    }
    if (G > 1) {
      uint64_t v[3];
      ok = res_wait<ALONE>(r, grp, PG, first, rec + lane * kResWords, lane < G, v);
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
      if (!ALONE && !ok) sh.fail = 1;
    }
  } else if (ALONE && stages == 1) {
    return true;
  }
  __syncthreads();
  if (first && sh.fail) return false;  // (uniform; at a later position below)
  // float32 over kResSumTiles tiles (64 elements) of a thread, float64 beyond
  double sp = 0.0, sq = 0.0, sx = 0.0;
  {
    float ap = 0.f, aq = 0.f, sc = 0.f;
    const float rt = res_uniform(sh.c[0]), rd = res_uniform(sh.c[1]), tau = res_uniform(sh.c[2]);
    const int jp = res_opaque_s(c.j0);
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
        if ((NV - 1 - j) % kResSumTiles == 0) {
          sp += static_cast<double>(ap);
          sq += static_cast<double>(aq);
          sx += static_cast<double>(sc);
          ap = aq = sc = 0.f;
        }
      }
  }
  sp = wave_sum(sp);
  sq = wave_sum(sq);
  sx = wave_sum(sx);
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
    if (lane < 3 && ok)
      st_agent(rec + c.w * kResWords + 3 + lane, res_word(lane == 0 ? part[0] : (lane == 1 ? part[1] : part[2])));
    if (ALONE && stages == 2) return true;
    const uint64_t* all = r.rec + static_cast<int64_t>(n) * PG * kResWords;
    uint64_t v[3];
    if (ok) ok = res_wait<ALONE>(r, grp, PG, first, all + lane * kResWords + 3, lane < PG, v);
    if (lane < PG)
#pragma unroll
      for (int i = 0; i < 3; ++i) sh.x[lane * 3 + i] = __longlong_as_double(static_cast<long long>(v[i]));
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // lane i < K: step i's alpha, S and 1 - S, slices in order
    double al = 0.0, S = 0.0, Sc = 0.0;
    if (lane < K)
      for (int i = 0; i < G; ++i) {
        al += sh.x[(lane * G + i) * 3];
        S += sh.x[(lane * G + i) * 3 + 1];
        Sc += sh.x[(lane * G + i) * 3 + 2];
      }
    // the draft's probabilities normalised by their own sum, S + (1 - S): the
    // errors of the exponentials they share fall out
    const double qn = 1.0 / (S + Sc);
    al = (al - S) + S * qn;
    S *= qn;
    Sc *= qn;
    double gk, L;
    chain_factor_of(K, a.mode, c.k, [&](int i) -> double { return dpp::lane(al, i); }, &gk, &L);
    gk = a.scale * gk * static_cast<double>(a.inv_t) * dpp::lane(qn, c.k) * sh.cc[1];
    const double A1 = gk * dpp::lane(Sc, c.k), A0 = -gk * dpp::lane(S, c.k);
    if (lane == 0) {
      sh.c[4] = static_cast<float>(A1);
      sh.c[5] = static_cast<float>(A0);
      if (!ALONE && !ok) sh.fail = 1;
      if (c.mem == 0 && ok) a.loss_pos[n] = a.scale * L;
    }
    if (c.mem == 0 && ok && a.overlap && lane < K) a.overlap[static_cast<int64_t>(n) * K + lane] = static_cast<float>(al);
  } else if (ALONE && stages == 2) {
    return true;
  }
  __syncthreads();
  if (!ALONE && sh.fail) return false;  // (uniform)
  // the gradient, and the next position's loads of each tile behind it
  const bool more = !ALONE && nn < a.N;
  const typename E::raw *rt = res_row_t<E>(d, more ? nn : n, c.k), *rd = res_row_d<E>(d, more ? nn : n, c.k);
  const float A1 = res_uniform(sh.c[4]), nA0 = -res_uniform(sh.c[5]);
  float* gr = a.grad + (static_cast<int64_t>(n) * K + c.k) * V;
  const int jw = res_opaque_s(c.j0);
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
      char* base = reinterpret_cast<char*>(gr + static_cast<int64_t>(c.tb + j) * TILE);
      if (j < NV - 1 || c.over == 0) {
        __builtin_nontemporal_store(g, reinterpret_cast<f32x4_any*>(base + static_cast<uint32_t>(tid) * 16u));
      } else {
        if (c.over < 4) gr[c.vlast] = g.x;
        if (c.over < 3) gr[c.vlast + 1] = g.y;
        if (c.over < 2) gr[c.vlast + 2] = g.z;
      }
      if (more) {
        xt[j] = res_tile_load<E, NV>(c, rt, j, V);
        xd[j] = res_tile_load<E, NV>(c, rd, j, V);
      }
    }
  return true;
}

// Moves 8 bytes per bfloat16 pair element (both logits read, the gradient
// written) against the 14 of the passes in tv_kernel.h.  Bound by the parts
// of a position that do not overlap on a CU: of 35 us per position (V =
// 151936, G = 2), 15 write the gradient and issue the next loads, 8 wait for
// those and sum the statistics, 7 are the second sums' arithmetic and 6 the
// two exchanges (time stamps per phase).  N = 4096, K = 3, V = 151936: 4.82
// -> 3.50 ms a call in bfloat16; N = 1024 in float32 1.92 -> 1.25 ms.
template <class E, int NV>
__global__ __launch_bounds__(kResThreads, 2) void tv_resident_kernel(TvArgs a, ResArgs r) {
  __shared__ ResLds sh;
  const RowsDesc& d = a.rows;
  const int PG = a.K * r.G;
  if (threadIdx.x == 0) {
    sh.ticket = atomicAdd(r.head, 1u) + 1u;
    sh.fail = 0;
  }
  __syncthreads();
  const int tk = __builtin_amdgcn_readfirstlane(static_cast<int>(sh.ticket));
  const int grp = tk / PG;
  const ResSlice c = res_slice_of<E, NV>(r, tk - grp * PG, d.V);
  // (the old value is not asked for: to read it would wait for all of the loads
  // below, whose number varies; a group that has given up never passes its
  // first wait)
  if (threadIdx.x == 0) atomicAdd(r.state + grp, 1u);
  typename E::vec xt[NV], xd[NV];
#pragma unroll
  for (int j = 0; j < NV; ++j) xt[j] = xd[j] = res_neg_inf(static_cast<const E*>(nullptr));
  if (grp < a.N) {
    const typename E::raw *rt = res_row_t<E>(d, grp, c.k), *rd = res_row_d<E>(d, grp, c.k);
#pragma unroll
    for (int j = 0; j < NV; ++j)
      if (j >= c.j0) {
        xt[j] = res_tile_load<E, NV>(c, rt, j, d.V);
        xd[j] = res_tile_load<E, NV>(c, rd, j, d.V);
      }
  }
  for (int n = grp; n < a.N; n += r.groups)
    if (!res_position<E, NV, false>(a, r, c, n, n + r.groups, grp, 3, xt, xd, sh)) return;
}

// The positions of groups that gave up (none as a rule: one load tells), then
// the total loss, the position losses added in tv_loss_kernel's order, NaN
// where a complete group lost a record.
template <class E, int NV>
__global__ __launch_bounds__(kResThreads, 2) void tv_resident_finish_kernel(TvArgs a, ResArgs r) {
  __shared__ ResLds sh;
  const RowsDesc& d = a.rows;
  const int tid = threadIdx.x, PG = a.K * r.G;
  auto losses = [&]() -> double {
    double acc = 0.0;
    if (tid < kThreads)
      for (int p = tid; p < a.N; p += kThreads) acc += a.loss_pos[p];
    return acc;
  };
  const uint32_t flag = r.head[2], lost = r.head[3];
  double acc = 0.0;
  if (blockIdx.x == 0) acc = losses();  // (with the flags still on their way)
  if (__builtin_expect(flag != 0u, 1)) {
    if (blockIdx.x != 0) return;
  } else {
    for (int n = blockIdx.x; n < a.N; n += static_cast<int>(gridDim.x)) {
      if (r.state[n % r.groups] + 1u < kResGaveUp) continue;
      for (int stages = 1; stages <= 3; ++stages)
        for (int mem = 0; mem < PG; ++mem) {
          const ResSlice c = res_slice_of<E, NV>(r, mem, d.V);
          const typename E::raw *rt = res_row_t<E>(d, n, c.k), *rd = res_row_d<E>(d, n, c.k);
          typename E::vec xt[NV], xd[NV];
#pragma unroll
          for (int j = 0; j < NV; ++j) {
            xt[j] = xd[j] = res_neg_inf(static_cast<const E*>(nullptr));
            if (j >= c.j0) {
              xt[j] = res_tile_load<E, NV>(c, rt, j, d.V);
              xd[j] = res_tile_load<E, NV>(c, rd, j, d.V);
            }
          }
          res_position<E, NV, true>(a, r, c, n, a.N, 0, stages, xt, xd, sh);
          __syncthreads();
        }
    }
    // the last workgroup to finish adds the losses
    __threadfence();
    __syncthreads();
    if (tid == 0) sh.ticket = atomicAdd(r.head + 1, 1u) + 1u;
    __syncthreads();
    if (sh.ticket != gridDim.x - 1u) return;
    __threadfence();
    acc = losses();
  }
  acc = wave_sum(acc);
  if ((tid & 63) == 0) sh.red[tid >> 6][0] = acc;
  __syncthreads();
  if (tid == 0) {
    double v = sh.red[0][0];
    for (int w = 1; w < kWaves; ++w) v += sh.red[w][0];
    *a.loss = lost == 0u ? NAN : static_cast<float>(v);
  }
}

}  // namespace sv
