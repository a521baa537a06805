// Kernels of the rank-one lamination path (gfx950), as templates; the
// r1_kernels_<dtype>_<dim>d.hip units instantiate them.
//
//   k_depth1    one wavefront per point: W^1 (and its laminate stress) -- the
//               min over directions of the line hulls at the centre;
//               k_depth1_split: several wavefronts per point, for small batches.
//   k_outer     depth 2, one workgroup per (point, outer direction): the outer
//               line's samples are inner envelopes W^1(F + t_i R), computed by
//               the block's waves into LDS; wave 0 then takes the outer hull.
//   k_finalize  depth 2, one wavefront per point: min over outer directions,
//               then the stress through the two-level lamination tree.
//
// Lamination is eq. 3.3 of arXiv 2211.14318 on the lines of Section 4.1; the
// stress is eq. 5.2 (first case) evaluated as Algorithm 3 on a binary tree.
#pragma once
#include "r1_device.hpp"
#include "r1_launch.hpp"

namespace r1k {
using namespace r1d;

template <typename T>
struct OuterRes {       // hull of one outer line at the centre
  T h;
  int mp, mq, capped;
};
static_assert(sizeof(OuterRes<float>) == 16 && sizeof(OuterRes<double>) == 24,
              "r1_outer_res_bytes() must match OuterRes");

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

template <typename T, int D>
__device__ __forceinline__ bool load_point(const KArgs& a, int64_t p, double* G, double& bn) {
  const T* F = static_cast<const T*>(a.F);
  bool fin = true;
#pragma unroll
  for (int k = 0; k < D * D; ++k) {
    G[k] = double(F[int64_t(k) * a.n + p]);
    fin = fin && isfinite(G[k]);
  }
  bn = double(static_cast<const T*>(a.beta_n)[p]);
  return fin && isfinite(bn);
}

template <int D>
__device__ __forceinline__ void line_point(const double* G, const Level& lv, int dir, double t, double* out) {
#pragma unroll
  for (int i = 0; i < D; ++i)
#pragma unroll
    for (int j = 0; j < D; ++j) out[i * D + j] = G[i * D + j] + t * lv.a[dir * D + i] * lv.b[dir * D + j];
}

__device__ __forceinline__ double t_of(const Level& lv, int m) {   // t at offset m from the centre
  if (lv.lay && m > 0) return static_cast<const double*>(lv.lay)[m - 1];   // the same value, tabled
  return lv.tau * double(2 * m) / double(lv.n_t - 1);
}

// Inner envelope at G and its laminate stress (P^1 = xi P0(G+) + (1-xi) P0(G-)).
template <typename T, int D, int S, int K, int M>
__device__ Env<T> envelope_with_stress(const KArgs& a, const Level& lv, const Layout<T, S, K>& lay,
                                       double bn, const double* G, double* P) {
  Point<T> q = make_point<T, M>(a.mat, bn);
  double cof[D * D];
  cofactor<D>(G, cof);
  T wc = w_point<T, D, M>(q, G, cof);
  Env<T> e = {wc, 0, 0, 0, inf_v<T>(), inf_v<T>()};
  if (wc < inf_v<T>()) e = envelope_at<T, D, S, K, M>(q, G, wc, lv, lay);
  double Gm[D * D], Gp[D * D], Pm[D * D], Pp[D * D];
  line_point<D>(G, lv, e.dir, -t_of(lv, e.mp), Gm);
  line_point<D>(G, lv, e.dir, t_of(lv, e.mq), Gp);
  stress_at<T, D, M>(q, a.mat, bn, Gm, Pm);
  stress_at<T, D, M>(q, a.mat, bn, Gp, Pp);
  double xi = (e.mp + e.mq) ? double(e.mp) / double(e.mp + e.mq) : 1.0;
#pragma unroll
  for (int k = 0; k < D * D; ++k) P[k] = xi * Pp[k] + (1.0 - xi) * Pm[k];
  return e;
}

template <typename T, int D>
__device__ __forceinline__ void write_bad_point(const KArgs& a, int64_t p, bool nonfinite, bool want_p) {
  T val = nonfinite ? T(__builtin_nan("")) : inf_v<T>();
  static_cast<T*>(a.W)[p] = val;
  if (want_p && a.P)
#pragma unroll
    for (int k = 0; k < D * D; ++k) static_cast<T*>(a.P)[int64_t(k) * a.n + p] = T(__builtin_nan(""));
  if (a.flags) a.flags[p] = nonfinite ? R1_PT_NONFINITE : R1_PT_DETLE0;
  if (a.tree)
    for (int k = 0; k < R1_TREE_NODES; ++k)
      a.tree[p * R1_TREE_NODES + k] = r1_laminate{0, 0, 0, 1.0f};
}

// The one-level laminate's stress at point p (eq. 5.2 on the one-level tree of
// Algorithm 3): P = xi P0(F+) + (1 - xi) P0(F-), F-/+ = G -/+ t a(x)b at offsets
// mp, mq of direction dir, xi = mp / (mp + mq), written to row k of P.  One
// thread's work; the one-level kernels and the batched point work share it, so
// that both give the same bits.
template <typename T, int D, int M>
__device__ __forceinline__ void laminate_stress1(const KArgs& a, int64_t p, const Level& lv, const Point<T>& q,
                                                 const double* G, double bn, int dir, int mp, int mq) {
  double Gm[D * D], Gp[D * D], Pm[D * D], Pp[D * D];
  line_point<D>(G, lv, dir, -t_of(lv, mp), Gm);
  line_point<D>(G, lv, dir, t_of(lv, mq), Gp);
  stress_at<T, D, M>(q, a.mat, bn, Gm, Pm);
  stress_at<T, D, M>(q, a.mat, bn, Gp, Pp);
  const double xi = (mp + mq) ? double(mp) / double(mp + mq) : 1.0;
#pragma unroll
  for (int k = 0; k < D * D; ++k)
    static_cast<T*>(a.P)[int64_t(k) * a.n + p] = T(fma(xi, Pp[k], (1.0 - xi) * Pm[k]));
}

// Per-point constants of a one-level envelope: the geometry (which holds G),
// the constants of W, W at the point, and the point's state (0: finite and
// admissible; 1: non-finite input; 2: W(F) = +inf, det F <= 0).
template <typename T, int D, int M>
struct PointSetup {
  typename GeomOf<D, M>::type g;
  Point<T> q;
  double bn;
  T wc;
  Centre<T> c;             // (J0, c0 alone for the double-well energy)
  int state;
};

template <typename T, int D, int M>
__device__ __forceinline__ PointSetup<T, D, M> point_setup(const KArgs& a, int64_t p) {
  PointSetup<T, D, M> s;
  double G[D * D];
  const bool fin = load_point<T, D>(a, p, G, s.bn);
  s.q = make_point<T, M>(a.mat, s.bn);
  double cof[D * D];
  cofactor<D>(G, cof);
  const double zero[D] = {};
  const Line<T> L = line_setup<T, D, M>(s.q, G, cof, zero, zero);       // W(F) as w_point takes it
  if (M == kFamSTVK || s.q.model == 0) {
    s.c = make_centre<T, M>(s.q, L.J0, L.c0);
    s.wc = fma(s.c.ws, s.q.sc, s.q.B);
  } else {
    s.c = Centre<T>{L.J0, L.c0, T(0), T(0), T(0)};
    s.wc = w_sample_doublewell<T>(T(0), L);
  }
  s.g = make_geom_m<D, M>(G);
  s.state = !fin ? 1 : (s.wc < inf_v<T>() ? 0 : 2);
  return s;
}

// Writes point p's one-level result e (one thread): W, tree and flags as requested
// by a, and with kDefer its laminate (direction, m_-, m_+) as integers in the first
// T slot of rows 0, 1, 2 of P, where k_stress1 finds it; else its stress.
template <typename T, int D, int M, bool kDefer>
__device__ __forceinline__ void write_depth1(const KArgs& a, int64_t p, const Level& lv, const Point<T>& q,
                                             const double* G, double bn, const Env<T>& e) {
  static_cast<T*>(a.W)[p] = e.h;
  if (a.want_stress && a.P) {
    if constexpr (kDefer) {
      T* P = static_cast<T*>(a.P);
      *reinterpret_cast<int32_t*>(P + p) = e.dir;
      *reinterpret_cast<int32_t*>(P + a.n + p) = e.mp;
      *reinterpret_cast<int32_t*>(P + 2 * a.n + p) = e.mq;
    } else {
      laminate_stress1<T, D, M>(a, p, lv, q, G, bn, e.dir, e.mp, e.mq);
    }
  }
  const int c = (lv.n_t - 1) / 2;
  if (a.tree) {
    float xi = (e.mp + e.mq) ? float(double(e.mp) / double(e.mp + e.mq)) : 1.0f;
    a.tree[p * R1_TREE_NODES] = r1_laminate{e.dir, c - e.mp, c + e.mq, xi};
    for (int k = 1; k < R1_TREE_NODES; ++k) a.tree[p * R1_TREE_NODES + k] = r1_laminate{0, 0, 0, 1.0f};
  }
  if (a.flags) a.flags[p] = (capped(e) ? R1_PT_ITERCAP : 0) | (near_tie(e) ? R1_PT_TIE : 0);
}

// One-level envelope of point p on level lv with stress, tree and flags as
// requested by a (wave-level: every lane of the wave calls it).
template <typename T, int D, int S, int K, int M>
__device__ __forceinline__ void point_depth1(const KArgs& a, int64_t p, const Level& lv) {
  const Layout<T, S, K> lay = make_layout<T, S, K>(lv);
  const PointSetup<T, D, M> s = point_setup<T, D, M>(a, p);
  if (s.state != 0) {
    if (lane_id() == 0) write_bad_point<T, D>(a, p, s.state == 1, a.want_stress);
    return;
  }
  const Env<T> e = envelope_geom<T, D, S, K, M>(s.q, s.g, s.wc, lv, lay);
  if (lane_id() == 0) write_depth1<T, D, M, false>(a, p, lv, s.q, s.g.G, s.bn, e);
}

// The coefficients of the line through a point along direction dir of lv.
template <typename T, int D, int M>
__device__ __forceinline__ Line<T> level_line(const PointSetup<T, D, M>& s, const Level& lv, int dir) {
  double a[D], b[D];
#pragma unroll
  for (int i = 0; i < D; ++i) { a[i] = lv.a[dir * D + i]; b[i] = lv.b[dir * D + i]; }
  return line_of<T, D, M>(s.q, s.g, a, b);
}

// One-level launch: a block of 4 waves takes a.pts_per_wave (<= kPointsPerWave)
// points per wave.  Their constants are formed by one thread per point into LDS
// first (a point's FP64 set-up then costs a lane, not a wavefront), then the
// coefficients of their lines by one lane per (point, direction) into the wave's
// table, then each wave laminates its points one after the other.
constexpr int kPointsPerWave = 8;
constexpr int kPointsPerBlock = 4 * kPointsPerWave;

// Points per wave for n points: kPointsPerWave, or fewer where that would leave
// the launch under 2048 blocks (small batches keep the device filled).
inline int one_level_points_per_wave(int64_t n) {
  const int64_t q = (n + 4 * 2048 - 1) / (4 * 2048);
  return int(q < 1 ? 1 : (q > kPointsPerWave ? kPointsPerWave : q));
}

// Registers: FP32 as measured per variant; FP64 lines of up to 8 samples per lane at
// three waves per SIMD (168 registers, 8 bytes spilled; 183 and two waves left free,
// where the logarithm's dependent chains leave issue slots empty: 500,000 points
// 16 x 201 7.05 -> 6.10 ms, 95,464 points 128 x 221 10.34 -> 9.28 ms, 3D 68,910 points
// 256 x 113 7.04 -> 6.46 ms).
template <typename T, int K, int D, int M>
constexpr int depth1_waves() {
  if (sizeof(T) == 8) return K <= 8 ? 3 : 1;
  return (D == 2 && M == kFamNH && K <= 14) ? 4 : K <= 16 ? 3 : 1;
}

// Whether k_depth1 leaves lines out (line_proof).  FP64: whenever there is more than one
// wave step.  FP32, 60,000 points, without / with: 3D 128 x 257 1501 / 911 us, 2D 32 x 257
// (eight steps) 422 / 349; two steps, 2D 16 x 129, 152 / 153; four steps, 16 x 257, 241 /
// 220 and 1,000,000 points 16 x 201 1950 / 1480.  The bound would thus pay at four steps
// too.  It is taken from five on, for a reason outside this kernel: the network's inference
// laminates the points with the fewest provable lines (262,144 points 16 x 201: plain 530
// us without and 457 with the bound, inference 498 with it) and would no longer be the
// faster of the two at its workload.
template <typename T, int S>
constexpr bool depth1_proves_lines(int n_dir) { return n_dir > (sizeof(T) == 4 ? 4 : 1) * (kWave / S); }

template <typename T, int D, int S, int K, int M>
__global__ __launch_bounds__(256, (depth1_waves<T, K, D, M>())) void k_depth1(KArgs a) {
  __shared__ PointSetup<T, D, M> ps[kPointsPerBlock];
  __shared__ LineTable<T, M> tabs[4];
  __shared__ int orders[4][M == kFamSTVK ? 1 : kTabLines];
  __shared__ ProofPoint<T> proofs[M == kFamSTVK ? 1 : kPointsPerBlock];
  const int per_block = 4 * a.pts_per_wave;
  const int64_t p0 = int64_t(blockIdx.x) * per_block;
  const int n_dir = a.lv0.n_dir, n_off = (a.lv0.n_t - 1) / 2;
  // lines shown to have a vertex at the centre are not sampled (depth1_proves_lines)
  const bool prove = M == kFamNH && a.mat.model == 0 && a.lv0.ab2 == a.lv0.ab2 && depth1_proves_lines<T, S>(n_dir);
  if (int(threadIdx.x) < per_block && p0 + threadIdx.x < a.n) {
    const PointSetup<T, D, M> s = point_setup<T, D, M>(a, p0 + threadIdx.x);
    ps[threadIdx.x] = s;
    if constexpr (M == kFamNH)
      if (prove)
        proofs[threadIdx.x] = proof_point<T>(s.q, s.c, T(s.q.kq * a.lv0.ab2), n_off, float(a.lv0.tau));
  }
  __syncthreads();
  const Layout<T, S, K> lay = make_layout<T, S, K>(a.lv0);
  const int wave = threadIdx.x / kWave;
  LineTable<T, M>& tab = tabs[wave];
  // few directions: the lines of all of the wave's points at once; else a point's,
  // kTabLines at a time
  const bool whole = n_dir * a.pts_per_wave <= kTabLines;
  if (whole) {
    for (int e = lane_id(); e < n_dir * a.pts_per_wave; e += kWave) {
      const int i = e / n_dir, slot = i * 4 + wave;
      if (p0 + slot < a.n) tab.put(e, level_line<T, D, M>(ps[slot], a.lv0, e - i * n_dir));
    }
    wave_lds_fence();
  }
  for (int i = 0; i < a.pts_per_wave; ++i) {
    const int slot = i * 4 + wave;
    const int64_t p = p0 + slot;
    if (p >= a.n) break;                      // wave-uniform
    const PointSetup<T, D, M>& s = ps[slot];
    if (s.state != 0) {
      if (lane_id() == 0) write_bad_point<T, D>(a, p, s.state == 1, a.want_stress);
      continue;
    }
    const T c2u = T(s.q.kq * a.lv0.ab2);
    LineProof<T> pf{};
    if (prove) pf = line_proof<T>(proofs[slot], n_off, float(a.lv0.tau));
    Env<T> e = env_none<T>();
    for (int m0 = 0; m0 < n_dir; m0 += kTabLines) {
      const int n = min(n_dir - m0, kTabLines);
      if (!whole) {
        wave_lds_fence();                      // reads of the entries before are done
        for (int m = lane_id(); m < n; m += kWave) tab.put(m, level_line<T, D, M>(s, a.lv0, m0 + m));
        wave_lds_fence();
      }
      const int off = whole ? i * n_dir : -m0;
      const auto lines = [&](int dir) { return tab.get(dir + off, s.c); };
      // the directions to visit: all, or those not proven
      int* order = nullptr;
      int first = m0, end = m0 + n;
      if (M != kFamSTVK && prove) {
        order = orders[wave];
        first = end = 0;
        wave_lds_fence();
        for (int d0 = m0; d0 < m0 + n; d0 += kWave) {
          const int dir = d0 + lane_id();
          const bool valid = dir < m0 + n;
          const bool proven = valid && pf(lines(valid ? dir : m0));
          const unsigned long long mp = __ballot(proven), mo = __ballot(valid && !proven);
          if (mp) env_merge(e, proven_env(s.c.ws, d0, mp));
          if (valid && !proven) order[end + __popcll(mo & ((1ull << lane_id()) - 1ull))] = dir;
          end += __popcll(mo);
        }
        wave_lds_fence();
      }
      e = envelope_scan<T, S, K, M>(s.q, s.wc, end, lay, lines, nullptr, 0, c2u, order, &s.c, first, kWave / S, e);
    }
    e = envelope_finish<T, M>(s.q, s.wc, e);
    if (lane_id() == 0) write_depth1<T, D, M, true>(a, p, a.lv0, s.q, s.g.G, s.bn, e);
  }
}

// Few points: a block of up to kSplitWaves waves takes one point, each wave a share
// of its directions, so that a batch that would leave most of the chip idle behind
// one wave's serial loop of lines per point (64 points x 16 directions: 35 us on 64
// waves) spreads over it.  Each wave forms the point's constants by itself (the
// latency of one lane's set-up, no barrier); the waves' minima meet in LDS in the
// order of the one-wave scan (value, then direction), so the result is the same;
// one thread then takes the stress (laminate_stress1, as k_stress1 does).
constexpr int kSplitWaves = 8;

template <typename T, int D, int S, int K, int M>
__global__ __launch_bounds__(kWave * kSplitWaves) void k_depth1_split(KArgs a) {
  __shared__ Env<T> part[kSplitWaves];
  const int64_t p = blockIdx.x;
  const int wave = threadIdx.x / kWave, waves = blockDim.x / kWave;
  const Level& lv = a.lv0;
  const PointSetup<T, D, M> s = point_setup<T, D, M>(a, p);
  if (s.state != 0) {                            // the same in every wave
    if (threadIdx.x == 0) write_bad_point<T, D>(a, p, s.state == 1, a.want_stress);
    return;
  }
  constexpr int NSEG = kWave / S;
  const Layout<T, S, K> lay = make_layout<T, S, K>(lv);
  Env<T> e = envelope_scan<T, S, K, M>(s.q, s.wc, lv.n_dir, lay, [&](int dd) { return level_line<T, D, M>(s, lv, dd); },
                                       nullptr, 0, T(s.q.kq * lv.ab2), nullptr, &s.c, wave * NSEG, waves * NSEG);
  if (lane_id() == 0) part[wave] = e;
  __syncthreads();
  if (wave != 0) return;
  e = part[0];
  for (int w = 1; w < waves; ++w) env_merge(e, part[w]);
  e = envelope_finish<T, M>(s.q, s.wc, e);
  if (threadIdx.x == 0) write_depth1<T, D, M, false>(a, p, lv, s.q, s.g.G, s.bn, e);
}

// Waves per point of a one-level launch of n points: 1 (k_depth1) or 2 .. kSplitWaves
// (k_depth1_split).  More waves per point shorten a point's serial loop of line steps
// until the chip is full; what a split point repeats (its set-up on every wave, the lines'
// coefficients on every lane of a step) then costs more than it gains, the sooner the
// fewer steps it has to share.  Hence bounds on the launch's waves by the number of steps:
// for 4 waves a point 3 to 16 per SIMD (1024 SIMDs), for 8 less, since a SIMD holds two of
// such a block where a lane takes more than 128 registers, and for 2, which leave most of
// the loop, little beyond one.  3D neo-Hooke lines are mostly proven not to need sampling
// by k_depth1, which the split does not do: it is left earlier there.
// Measured over 1,300 launches (n 64 .. 8192, 16 .. 400 directions, 65 .. 1025 samples): the
// choice takes 0.8% more than the best of 1, 2, 4 and 8 in the mean (a model of rounds of
// waves the chip holds at once 5%).  us for w = 1, 2, 4, 8, * the choice: FP64 2D 16 x 129,
// 512 points 23 16 13* 17; FP64 3D 64 x 257, 4096: 204* 253 260 366; FP32 3D 256 x 513,
// 8192: 565* 735 717 1051, 256 x 1025, 300: 348 231 134 117*; FP32 2D 256 x 1025, 4096:
// 830 734 654* 684; FP64 2D St. Venant-Kirchhoff 64 x 257, 2500: 130 113* 110 156, 256 x 257,
// 6000: 814 771* 741 1112.
template <typename T, int D, int S, int K, int M>
inline int one_level_waves(int64_t n, int n_dir) {
  const int steps = (n_dir + kWave / S - 1) / (kWave / S);
  constexpr bool light = sizeof(T) == 4 && M == kFamNH && (K <= 8 || D == 2);   // registers: 4 waves a SIMD
  const int64_t four = steps <= 8    ? (light ? 4096 : 3072)
                       : steps <= 32 ? (light ? 8192 : 6144)
                                     : (D == 3 && M == kFamNH ? 6400 : 16384);
  const int64_t eight = light ? 4096 : steps <= 32 ? 2048 : 2560;
  constexpr bool stvk2 = D == 2 && M == kFamSTVK;
  const int64_t two = stvk2 && sizeof(T) == 8 && steps > 32 ? 16384 : light || stvk2 ? 5000 : 3072;
  int w = 8 * n <= eight ? kSplitWaves : 4 * n <= four ? 4 : 2 * n <= two ? 2 : 1;
  while (w > steps) w /= 2;
  return w;
}

// Laminate stress of the one-level points (eq. 5.2 on the one-level tree of
// Algorithm 3: P = xi P0(F+) + (1 - xi) P0(F-)), one thread per point, after
// k_depth1: it reads the laminate k_depth1 left in P (see write_depth1) and
// overwrites it with the stress.  Points k_depth1 found bad (W NaN or +inf)
// already hold NaN stresses.
template <typename T, int D, int M>
__global__ __launch_bounds__(256) void k_stress1(KArgs a) {
  const int64_t p = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (p >= a.n) return;
  const T w = static_cast<const T*>(a.W)[p];
  if (!(w < inf_v<T>())) return;
  T* P = static_cast<T*>(a.P);
  const int dir = *reinterpret_cast<const int32_t*>(P + p);
  const int mp = *reinterpret_cast<const int32_t*>(P + a.n + p);
  const int mq = *reinterpret_cast<const int32_t*>(P + 2 * a.n + p);
  double G[D * D], bn;
  load_point<T, D>(a, p, G, bn);
  laminate_stress1<T, D, M>(a, p, a.lv0, make_point<T, M>(a.mat, bn), G, bn, dir, mp, mq);
}

// Outer hull of an LDS-resident line (wave-wide, S = 64): wl[m-1] / wr[m-1] are
// the samples at offsets -m / +m, m = 1..c (NaN or +inf = absent).  Same search
// as hull_centre: a values-only vertex test, then alternating tangent queries.
template <typename T>
__device__ LineHull<T> hull_centre_lds(const T* wl, const T* wr, int c, T wc, int* capped) {
  const int lane = lane_id();
  T maxL = -inf_v<T>(), minR = inf_v<T>();
  for (int m = 1 + lane; m <= c; m += kWave) {
    T inv = T(1.0 / double(m));
    maxL = fmax(maxL, (wc - wl[m - 1]) * inv);
    minR = fmin(minR, (wr[m - 1] - wc) * inv);
  }
  maxL = seg_max<kWave>(maxL);
  minR = seg_min<kWave>(minR);
  LineHull<T> r = {wc, 0, 0};
  *capped = 0;
  if (!(maxL >= minR)) return r;      // wave-uniform
  Cand<T> p = {-inf_v<T>(), 0, T(0)};
  for (int m = 1 + lane; m <= c; m += kWave) {
    T key = (wc - wl[m - 1]) * T(1.0 / double(m));
    bool take = key >= p.key;
    p.key = take ? key : p.key; p.m = take ? m : p.m; p.w = take ? wl[m - 1] : p.w;
  }
  p = seg_arg<kWave, true>(p);
  Cand<T> q = {inf_v<T>(), 0, T(0)};
  for (int it = 0; it < kBridgeCap; ++it) {
    T nb = inf_v<T>(), db = T(1), wb = T(0);
    int mb = 0;
    for (int m = 1 + lane; m <= c; m += kWave) {
      T num = wr[m - 1] - p.w, den = T(m + p.m);
      bool take = num * db <= nb * den;
      nb = take ? num : nb; db = take ? den : db; mb = take ? m : mb; wb = take ? wr[m - 1] : wb;
    }
    Cand<T> qc = {nb / db, mb, wb};
    q = seg_arg<kWave, false>(qc);
    nb = -inf_v<T>(); db = T(1); wb = T(0); mb = 0;
    for (int m = 1 + lane; m <= c; m += kWave) {
      T num = q.w - wl[m - 1], den = T(q.m + m);
      bool take = num * db >= nb * den;
      nb = take ? num : nb; db = take ? den : db; mb = take ? m : mb; wb = take ? wl[m - 1] : wb;
    }
    Cand<T> pc = {nb / db, mb, wb};
    pc = seg_arg<kWave, true>(pc);
    if (pc.m == p.m) {
      r.h = (T(q.m) * p.w + T(p.m) * q.w) / T(q.m + p.m);
      r.mp = p.m; r.mq = q.m;
      return r;
    }
    p = pc;
  }
  r.h = (T(q.m) * p.w + T(p.m) * q.w) / T(q.m + p.m);
  r.mp = p.m; r.mq = q.m; *capped = 1;
  return r;
}

// Inner directions whose line coefficients are tabulated in LDS per outer line.
constexpr int kMaxTabDirs = 512;

// Waves of an outer-line block (blocks are 256 threads).
constexpr int kOuterWaves = 4;

// Tabulated coefficients per inner direction: 5 for the neo-Hooke family (affine
// in the outer t), 10 for St. Venant-Kirchhoff (p1 cubic, p2 quadratic, p3 affine,
// p4 constant in the outer t).
__host__ __device__ constexpr int tab_coefs(int model) { return model == 2 ? 10 : 5; }

// Bytes of dynamic LDS an outer line needs for samples of elem_bytes bytes:
// the outer line's samples and, when the inner level is tabulated, its
// coefficient table, each wave's warm-start bridge slopes (the last two per
// direction) and each wave's direction visiting order (int).
__host__ __device__ inline size_t outer_lds_bytes(size_t elem_bytes, int n_t_outer, int n_dir_inner, int model) {
  const bool tab = n_dir_inner <= kMaxTabDirs;
  return elem_bytes * (size_t(n_t_outer - 1) +
                       (tab ? size_t(tab_coefs(model) + 2 * kOuterWaves) * size_t(n_dir_inner) : 0)) +
         (tab ? sizeof(int) * size_t(kOuterWaves) * size_t(n_dir_inner) : 0);
}

template <typename T>
__host__ __device__ inline size_t outer_lds_bytes(const Level& lo, const Level& li, int model) {
  return outer_lds_bytes(sizeof(T), lo.n_t, li.n_dir, model);
}

// St. Venant-Kirchhoff inner line along the outer line G(t) = F + t R: its
// coefficients c1 .. c4 (stvk_line) are polynomials in t of degree 3, 2, 1 and 0
// (E(t) of G(t) is quadratic in t).  Their monomial coefficients are fitted in
// double from exact evaluations at t = tau {-1, 0, 1, 2}:
// coef = (c1: t^0..t^3, c2: t^0..t^2, c3: t^0, t^1, c4).
template <typename T, int D>
__device__ __forceinline__ void stvk_inner_coef(double lam, double mu, double k, const double* F, const double* R,
                                                double tau, const double* a, const double* b, T* coef) {
  double y1[4], y2[4], y3[4], c4 = 0.0;
  const double u[4] = {-1.0, 0.0, 1.0, 2.0};
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    double G[D * D];
#pragma unroll
    for (int r = 0; r < D * D; ++r) G[r] = F[r] + u[s] * tau * R[r];
    Line<double> L = stvk_line_g<double, D>(lam, mu, k, make_stvk_geom<D>(G), a, b);
    y1[s] = L.c1; y2[s] = L.c2; y3[s] = L.c3;
    if (s == 1) c4 = L.c4;
  }
  // y(u) = a0 + a1 u + a2 u^2 + a3 u^3 through u = -1, 0, 1, 2; then t = tau u
  const double a0 = y1[1], a2 = 0.5 * (y1[2] + y1[0]) - y1[1], s1 = 0.5 * (y1[2] - y1[0]);
  const double a3 = (y1[3] - a0 - 4.0 * a2 - 2.0 * s1) / 6.0, a1 = s1 - a3;
  const double it = 1.0 / tau;
  coef[0] = T(a0); coef[1] = T(a1 * it); coef[2] = T(a2 * it * it); coef[3] = T(a3 * it * it * it);
  coef[4] = T(y2[1]); coef[5] = T(0.5 * (y2[2] - y2[0]) * it); coef[6] = T((0.5 * (y2[2] + y2[0]) - y2[1]) * it * it);
  coef[7] = T(y3[1]); coef[8] = T(0.5 * (y3[2] - y3[0]) * it);
  coef[9] = T(c4);
}

// What the inner level of one outer sample starts from.
template <typename T>
struct OuterSample {
  Centre<T> c;
  T wc, t;
  ProofPoint<T> pf;
};

// Outer samples a wave sets up at a time, one per lane, into LDS: the FP64 geometry, the
// centre and the vertex bound of a sample then cost a lane's share and hold no registers
// during the line scan (64 x 1025 / 32 x 257, with the centre's logarithm and exponential
// taken once instead of three times: FP32 96 points 23.2 -> 22.2 ms, FP64 37 points 41.4
// -> 38.2, an uneven FP32 plan of 384 points 62.0 -> 58.6).
constexpr int kOuterBatch = 16;

// One outer line (block-level, every thread calls it): the samples W^1(F + t_i R_mo)
// are inner envelopes computed by the block's waves into LDS; wave 0 takes the
// outer hull at the centre.  w1f = W^1(F) is the centre sample.  Thread 0 writes
// the result to *out.  kProve: proven inner lines may be left out (outer_proves_lines).
template <typename T, int D, int S, int K, int M, bool kProve = true>
__device__ __forceinline__ void outer_line(const KArgs& a, int64_t p, int mo, const Level& lo, const Level& li, T w1f,
                                           OuterRes<T>* out, char* smem_raw) {
  const int co = (lo.n_t - 1) / 2;
  // Up to kMaxTabDirs inner directions the waves keep warm-start bridge slopes,
  // visiting orders and the inner lines' coefficients as polynomials in the outer t
  // (tab_coefs) in LDS.
  const bool lds_lines = li.n_dir <= kMaxTabDirs;
  const bool tab = lds_lines;
  constexpr int NC = tab_coefs(M);
  T* coef = reinterpret_cast<T*>(smem_raw);                 // NC * n_dir_i (tab)
  T* warm = coef + (tab ? NC * li.n_dir : 0);                   // 2 kOuterWaves n_dir_i (lds_lines)
  T* wl = warm + (lds_lines ? 2 * kOuterWaves * li.n_dir : 0);  // outer samples at -m
  T* wr = wl + co;                                          // outer samples at +m
  int* order = reinterpret_cast<int*>(wr + co);             // kOuterWaves * n_dir_i (lds_lines)
  __shared__ int capped_any;
  __shared__ OuterSample<T> samples[kOuterWaves][kOuterBatch];
  __shared__ Point<T> sq;                     // for the samples' set-up: what the line scan does not use
  __shared__ double sF[D * D], sR[D * D];     // F and R where the samples read them (not in registers)
  double F[D * D], bn;
  load_point<T, D>(a, p, F, bn);
  double R[D * D];
#pragma unroll
  for (int i = 0; i < D; ++i)
#pragma unroll
    for (int j = 0; j < D; ++j) R[i * D + j] = lo.a[mo * D + i] * lo.b[mo * D + j];
  if (threadIdx.x == 0) {
    capped_any = 0;
#pragma unroll
    for (int k = 0; k < D * D; ++k) { sF[k] = F[k]; sR[k] = R[k]; }
  }
  if (tab) {
    if constexpr (M == kFamSTVK) {
      const double k = line_scale<T, M>(a.mat);
      for (int i = threadIdx.x; i < li.n_dir; i += blockDim.x)
        stvk_inner_coef<T, D>(a.mat.lambda, a.mat.mu, k, F, R, lo.tau, li.a + i * D, li.b + i * D, coef + NC * i);
    } else {
      double cofF[D * D], C1[D * D];
      cofactor<D>(F, cofF);
      cof_derivative<D>(F, R, C1);
      for (int i = threadIdx.x; i < li.n_dir; i += blockDim.x)
        inner_line_coef<T, D>(a.mat.model, line_scale<T>(a.mat), F, cofF, R, C1, li.a + i * D, li.b + i * D,
                              coef + NC * i);
    }
  }
  if (threadIdx.x == 0) sq = make_point<T, M>(a.mat, bn);
  if (lds_lines)
    for (int i = threadIdx.x; i < 2 * kOuterWaves * li.n_dir; i += blockDim.x) warm[i] = T(__builtin_nan(""));
  __syncthreads();
  Layout<T, S, K> lay = make_layout<T, S, K>(li);
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) / kWave), nwave = blockDim.x / kWave;
  int cap = 0;
  // outer samples, interleaved left/right so the waves share both sides; a
  // wave walks one side outwards in even steps of two samples, so the inner
  // bridge slopes of its last two samples (warm, per inner direction),
  // extrapolated, start the next
  T* warm_w = warm + 2 * wave * li.n_dir;      // blocks have kOuterWaves waves
  int* order_w = order + wave * li.n_dir;
  const Point<T> q = sq;
  const T c2u = T(q.kq * li.ab2);
  const bool prove = kProve && M == kFamNH && q.model == 0 && c2u == c2u && outer_proves_lines<T, S>(li.n_dir);
  const auto sample_t = [&](int s) { return (s & 1) ? t_of(lo, 1 + (s >> 1)) : -t_of(lo, 1 + (s >> 1)); };
  for (int s0 = wave; s0 < 2 * co; s0 += nwave * kOuterBatch) {
    wave_lds_fence();                          // reads of the samples before are done
    if (tab && lane_id() < kOuterBatch && s0 + lane_id() * nwave < 2 * co) {
      const double t = sample_t(s0 + lane_id() * nwave);
      double G[D * D], cof[D * D];
#pragma unroll
      for (int k = 0; k < D * D; ++k) G[k] = sF[k] + t * sR[k];
      cofactor<D>(G, cof);
      // W(G) and the part of the inner lines they share: c0 = k psi0(G) (St. Venant-
      // Kirchhoff), J0 = det G and c0 = kq (|G|^2 - d) (neo-Hooke), G11 and the rest
      // (double well)
      const double zero[D] = {};
      const Line<T> L0 = line_setup<T, D, M>(sq, G, cof, zero, zero);
      OuterSample<T>& o = samples[wave][lane_id()];
      o.t = T(t);
      if (M == kFamSTVK || q.model == 0) {
        const Centre<T> c = make_centre<T, M>(sq, L0.J0, L0.c0);
        o.c = c;
        o.wc = fma(c.ws, sq.sc, sq.B);
        if constexpr (M == kFamNH)
          if (prove) o.pf = proof_point<T>(sq, c, c2u, lay.c, float(li.tau));
      } else {
        o.c = Centre<T>{L0.J0, L0.c0, T(0), T(0), T(0)};
        o.wc = w_sample_doublewell<T>(T(0), L0);
      }
    }
    wave_lds_fence();
    for (int j = 0; j < kOuterBatch; ++j) {
      const int s = s0 + j * nwave;
      if (s >= 2 * co) break;                  // wave-uniform
      T v;
      if (tab) {
        const OuterSample<T>& o = samples[wave][j];
        v = o.wc;
        if (o.wc < inf_v<T>()) {
          const T tt = o.t;
          const T J0 = o.c.J0, c0 = o.c.c0;
          const Env<T> e = envelope_next<T, S, K, M>(q, o.wc, li.n_dir, lay, [&](int dd) {
            const T* cf = coef + NC * dd;
            if constexpr (M == kFamSTVK)
              return Line<T>{T(0), T(0), c0, T(fma(tt, fma(tt, fma(tt, cf[3], cf[2]), cf[1]), cf[0])),
                             T(fma(tt, fma(tt, cf[6], cf[5]), cf[4])), T(fma(tt, cf[8], cf[7])), cf[9]};
            else
              return Line<T>{J0, T(fma(tt, cf[1], cf[0])), c0, T(fma(tt, cf[3], cf[2])), cf[4]};
          }, warm_w, order_w, o.c, prove ? &o.pf : nullptr, float(li.tau), c2u);
          v = e.h;
          cap |= e.cap < inf_v<T>();
        }
      } else {
        const double t = sample_t(s);
        double G[D * D], cof[D * D];
#pragma unroll
        for (int k = 0; k < D * D; ++k) G[k] = sF[k] + t * sR[k];
        cofactor<D>(G, cof);
        const T wc = w_point<T, D, M>(q, G, cof);
        v = wc;
        if (wc < inf_v<T>()) {
          const Env<T> e = envelope_at<T, D, S, K, M>(q, G, wc, li, lay);
          v = e.h;
          cap |= capped(e);
        }
      }
      if (lane_id() == 0) ((s & 1) ? wr : wl)[s >> 1] = v;
    }
  }
  if (cap && lane_id() == 0) atomicOr(&capped_any, 1);
  __syncthreads();
  if (wave == 0) {
    int own;
    LineHull<T> r = hull_centre_lds<T>(wl, wr, co, w1f, &own);
    if (threadIdx.x == 0) *out = OuterRes<T>{r.h, r.mp, r.mq, own | capped_any};
  }
  __syncthreads();                            // LDS reused by the caller's next item
}

// Waves per SIMD k_outer is held to: three for up to 16 FP32 or 8 FP64 samples per lane
// (168 registers; two left free), where dependent chains of log, exp and lane reductions
// leave issue slots empty and what spills is reloaded once per outer sample or seldom.
// 40 points, 32 x 153 outer, 32 inner directions, two / three waves: FP32 3D 45 inner
// samples 670 / 549 us, 129 866 / 721, 257 (one wave, 256 registers) 1842 / 1112; FP64
// 2D 45 1338 / 1237, 129 2191 / 2152, 3D 45 1260 / 1130.  A launch of at most two blocks
// per CU (kFewBlocks) has no third wave to take, so there the spills only cost: it is held
// to two waves, and in FP32 it samples every line, since the bound's latency is then not
// hidden either (64 x 513 outer, four points, three waves with the bound / two without:
// 2D 32 x 257 1603 / 1553 us, 3D 32 x 129 887 / 843, 16 x 91 543 / 499; FP64 3D 32 x 65,
// with the bound, 1475 / 1371).
template <typename T, int K>
constexpr int outer_waves(bool few) {
  return K <= (sizeof(T) == 8 ? 8 : 16) ? (few ? 2 : 3) : 1;
}
constexpr int64_t kFewBlocks = 512;

template <typename T, int D, int S, int K, int M, bool kFew>
__global__ __launch_bounds__(256, (outer_waves<T, K>(kFew))) void k_outer(KArgs a) {
  extern __shared__ char smem_raw[];
  const int n_dir_o = a.lv0.n_dir;
  const int64_t p = int64_t(blockIdx.x) / n_dir_o;
  const int mo = int(int64_t(blockIdx.x) % n_dir_o);
  OuterRes<T>* out = static_cast<OuterRes<T>*>(a.scratch_outer) + p * n_dir_o + mo;
  T w1f = static_cast<const T*>(a.scratch_w1f)[p];
  if (!(w1f < inf_v<T>())) {                  // det F <= 0 or non-finite input: block-uniform
    if (threadIdx.x == 0) *out = OuterRes<T>{w1f, 0, 0, 0};
    return;
  }
  outer_line<T, D, S, K, M, !(kFew && sizeof(T) == 4)>(a, p, mo, a.lv0, a.lv1, w1f, out, smem_raw);
}

// Two-level result of point p from its outer-line results res[0 .. n_dir_o):
// min over outer directions, then stress and tree through Algorithm 3 on the
// binary tree (wave-level).
template <typename T, int D, int S, int K, int M>
__device__ __forceinline__ void finalize_point(const KArgs& a, int64_t p, const Level& lo, const Level& li,
                               const OuterRes<T>* res) {
  const int n_dir_o = lo.n_dir;
  double F[D * D], bn;
  bool fin = load_point<T, D>(a, p, F, bn);
  Point<T> q0 = make_point<T, M>(a.mat, bn);
  double cof0[D * D];
  cofactor<D>(F, cof0);
  if (!fin || !(w_point<T, D, M>(q0, F, cof0) < inf_v<T>())) {
    if (lane_id() == 0) write_bad_point<T, D>(a, p, !fin, a.want_stress);
    return;
  }
  T bh = inf_v<T>(), bs = inf_v<T>();
  int bd = 0x7fffffff, bp = 0, bq = 0, cap = 0;
  for (int m = lane_id(); m < n_dir_o; m += kWave) {
    OuterRes<T> r = res[m];
    cap |= r.capped;
    if (r.h < bh) { bs = bh; bh = r.h; bd = m; bp = r.mp; bq = r.mq; }
    else bs = fmin(bs, r.h);
  }
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    T oh = __shfl_xor(bh, off), os = __shfl_xor(bs, off);
    int od = __shfl_xor(bd, off), op = __shfl_xor(bp, off), oq = __shfl_xor(bq, off);
    cap |= __shfl_xor(cap, off);
    bool take = oh < bh || (oh == bh && od < bd);
    bs = take ? fmin(os, bh) : fmin(bs, oh);
    bh = take ? oh : bh; bd = take ? od : bd; bp = take ? op : bp; bq = take ? oq : bq;
  }
  bool tie = near_tie(Env<T>{bh, bd, bp, bq, inf_v<T>(), bs});
  const int c = (lo.n_t - 1) / 2, ci = (li.n_t - 1) / 2;
  r1_laminate node[3];
  double Pout[D * D];
  if (a.want_stress || a.tree) {
    Layout<T, S, K> lay = make_layout<T, S, K>(li);
    double Gm[D * D], Gp[D * D], Pm[D * D], Pp[D * D];
    line_point<D>(F, lo, bd, -t_of(lo, bp), Gm);
    line_point<D>(F, lo, bd, t_of(lo, bq), Gp);
    Env<T> em = envelope_with_stress<T, D, S, K, M>(a, li, lay, bn, Gm, Pm);
    cap |= capped(em);
    tie = tie || near_tie(em);
    Env<T> ep = em;
    if (bp + bq) {
      ep = envelope_with_stress<T, D, S, K, M>(a, li, lay, bn, Gp, Pp);
      cap |= capped(ep);
      tie = tie || near_tie(ep);
    } else {
#pragma unroll
      for (int k = 0; k < D * D; ++k) Pp[k] = Pm[k];
    }
    double xi = (bp + bq) ? double(bp) / double(bp + bq) : 1.0;
#pragma unroll
    for (int k = 0; k < D * D; ++k) Pout[k] = xi * Pp[k] + (1.0 - xi) * Pm[k];
    node[0] = r1_laminate{bd, c - bp, c + bq, float(xi)};
    node[1] = r1_laminate{em.dir, ci - em.mp, ci + em.mq,
                          (em.mp + em.mq) ? float(double(em.mp) / double(em.mp + em.mq)) : 1.0f};
    node[2] = r1_laminate{ep.dir, ci - ep.mp, ci + ep.mq,
                          (ep.mp + ep.mq) ? float(double(ep.mp) / double(ep.mp + ep.mq)) : 1.0f};
  }
  if (lane_id() == 0) {
    static_cast<T*>(a.W)[p] = bh;
    if (a.want_stress && a.P)
#pragma unroll
      for (int k = 0; k < D * D; ++k) static_cast<T*>(a.P)[int64_t(k) * a.n + p] = T(Pout[k]);
    if (a.tree)
      for (int k = 0; k < R1_TREE_NODES; ++k) a.tree[p * R1_TREE_NODES + k] = node[k];
    if (a.flags) a.flags[p] = (cap ? R1_PT_ITERCAP : 0) | (tie ? R1_PT_TIE : 0);
  }
}

template <typename T, int D, int S, int K, int M>
__global__ __launch_bounds__(256) void k_finalize(KArgs a) {
  const int64_t p = int64_t(blockIdx.x) * (blockDim.x / kWave) + threadIdx.x / kWave;
  if (p >= a.n) return;
  finalize_point<T, D, S, K, M>(a, p, a.lv0, a.lv1,
                             static_cast<const OuterRes<T>*>(a.scratch_outer) + p * a.lv0.n_dir);
}

// ---- dispatch ------------------------------------------------------------------

template <typename T, int D, int S, int K, int M>
hipError_t launch_T(const KArgs& a, int depth, hipStream_t st, KTimer* tm) {
  dim3 blk(256);
  unsigned per = 256 / kWave;
  const int ppw = one_level_points_per_wave(a.n);
  const dim3 grd1(unsigned((a.n + 4 * ppw - 1) / (4 * ppw)));
  if (depth == 1) {
    KArgs a1 = a;
    a1.pts_per_wave = ppw;
    const int wpp = one_level_waves<T, D, S, K, M>(a.n, a.lv0.n_dir);
    if (tm) tm->begin("depth1", st);
    if (wpp > 1) {
      hipLaunchKernelGGL((k_depth1_split<T, D, S, K, M>), dim3(unsigned(a.n)), dim3(kWave * wpp), 0, st, a);
      if (tm) tm->end(st);
      return hipGetLastError();
    }
    hipLaunchKernelGGL((k_depth1<T, D, S, K, M>), grd1, blk, 0, st, a1);
    if (a.want_stress && a.P)
      hipLaunchKernelGGL((k_stress1<T, D, M>), dim3(unsigned((a.n + 255) / 256)), blk, 0, st, a);
    if (tm) tm->end(st);
    return hipGetLastError();
  }
  // depth 2: W^1 at every point (the outer lines' centre), outer lines, finalize
  KArgs pre = a;
  pre.lv0 = a.lv1;
  pre.W = a.scratch_w1f;
  pre.P = nullptr;
  pre.tree = nullptr;
  pre.flags = nullptr;
  pre.want_stress = 0;
  pre.pts_per_wave = ppw;
  dim3 grd(unsigned((a.n + per - 1) / per));
  const int wpp = one_level_waves<T, D, S, K, M>(a.n, a.lv1.n_dir);
  if (tm) tm->begin("depth2_centre", st);
  if (wpp > 1)
    hipLaunchKernelGGL((k_depth1_split<T, D, S, K, M>), dim3(unsigned(a.n)), dim3(kWave * wpp), 0, st, pre);
  else
    hipLaunchKernelGGL((k_depth1<T, D, S, K, M>), grd1, blk, 0, st, pre);
  if (tm) tm->end(st);
  size_t lds = outer_lds_bytes<T>(a.lv0, a.lv1, M);
  dim3 grd_o(unsigned(a.n * a.lv0.n_dir));
  if (tm) tm->begin("outer", st);
  constexpr bool has_few = outer_waves<T, K>(true) < outer_waves<T, K>(false);
  if (has_few && a.n * a.lv0.n_dir <= kFewBlocks)
    hipLaunchKernelGGL((k_outer<T, D, S, K, M, has_few>), grd_o, blk, lds, st, a);
  else
    hipLaunchKernelGGL((k_outer<T, D, S, K, M, false>), grd_o, blk, lds, st, a);
  if (tm) tm->end(st);
  if (tm) tm->begin("finalize", st);
  hipLaunchKernelGGL((k_finalize<T, D, S, K, M>), grd, blk, 0, st, a);
  if (tm) tm->end(st);
  return hipGetLastError();
}

template <typename T, int D, int M>
hipError_t launch_TD(const KArgs& a, int depth, int S, int K, hipStream_t st, KTimer* tm) {
#define R1_CASE(SS, KK) \
  if (S == SS && K == KK) return launch_T<T, D, SS, KK, M>(a, depth, st, tm);
  R1_CASE(8, 2) R1_CASE(8, 4) R1_CASE(8, 8) R1_CASE(8, 16) R1_CASE(8, 32)
  R1_CASE(16, 2) R1_CASE(16, 4) R1_CASE(16, 8) R1_CASE(16, 14) R1_CASE(16, 16) R1_CASE(16, 32)
  R1_CASE(32, 2) R1_CASE(32, 4) R1_CASE(32, 8) R1_CASE(32, 16) R1_CASE(32, 32)
  R1_CASE(64, 2) R1_CASE(64, 4) R1_CASE(64, 8) R1_CASE(64, 16) R1_CASE(64, 32)
#undef R1_CASE
  return hipErrorInvalidValue;
}

}  // namespace r1k
