// Global rank-one lamination on a deformation-gradient mesh (Section 4.1 of
// arXiv 2211.14318): node values W^0 = W on the mesh of Section 5.2 (one mesh
// width for every component), then iterations of eq. 4.3 -- every node takes
// the minimum over the directions of the lower hull (Algorithm 1) of the line
// of eq. 4.4 through it, clipped to the mesh's box -- until the maximal decrease
// of an iteration is at most the tolerance or k_max iterations are done
// (Section 6); off-mesh values by multilinear interpolation.  Node stresses and
// tangent moduli, when requested, follow the laminates that lower the nodes
// (eq. 5.2, first case; Algorithm 3's moduli with the same weights);
// interpolating them gives the off-mesh values (eq. 5.2, second case).
//
// A direction is an integer step s in Z^{d x d}; its lines advance the node
// index by a constant stride and partition the mesh.  The directions of an
// iteration all read the previous iterate, so their hulls are independent; only
// the choice among them is ordered (a later direction replaces a node's value
// only when lower by more than a rounding margin).  An iteration therefore runs,
// per group of up to 16 directions with lines of more than three nodes, a hull
// launch -- one thread per line of every such direction; the line starts (nodes
// whose predecessor lies outside the box) form at most d*d disjoint boxes and are
// decoded from the thread index; the thread stages its line in its own LDS
// column, builds the lower hull with a monotone chain and writes every node's
// candidate value (and, when stresses or moduli are carried, its laminate's
// offsets) -- then a pick launch, one thread per node, that takes the candidates
// in direction order.  Directions whose lines hold at most three nodes (166 of
// the 169 of the paper's 3D mesh) need no hull launch: the pick forms their
// candidate, the midpoint of a node's two neighbours, in place.  The last
// pick of an iteration also takes the maximal decrease and writes the carried
// stresses and moduli, so nothing is copied between iterations.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <utility>
#include <vector>

#include "r1.h"
#include "r1_device.hpp"
#include "r1_grid_lines.hpp"
#include "r1_handle.hpp"

namespace {

using namespace r1g;

constexpr int kLineThreads = 64;        // lines per wave of the hull kernels
constexpr int kStageBytes = 56 * 1024;  // LDS of a block that stages its lines

__device__ __forceinline__ void node_multi(const GridArgs& g, int64_t p, int* I) {
  for (int c = g.dd - 1; c >= 0; --c) {
    I[c] = int(p % g.n[c]);
    p /= g.n[c];
  }
}

template <typename T>
__device__ __forceinline__ T inf_t() { return T(__builtin_inf()); }

// Unit roundoff of T: a hull value lowers a node only by more than 4 of these
// relative to max(|W|, 1e-3) -- a node on a straight hull run reads its own value
// back up to rounding, which is no lamination, and of directions that tie to
// rounding the first keeps the node.
template <typename T>
__device__ __forceinline__ T eps_t() { return sizeof(T) == 4 ? T(1.1920928955078125e-07) : T(2.220446049250313e-16); }

// W^0 at every node: the library's W (neo-Hooke: +inf where det F <= 0); with P,
// also P^0 = dW/dF, with A the moduli d^2W/dFdF (component-major, NaN where W is
// +inf).
template <typename T, int D>
__global__ __launch_bounds__(256) void k_grid_energy(GridArgs g, r1d::Material mat, double bn, T* W, T* P, T* A) {
  const int64_t p = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (p >= g.size) return;
  int I[9];
  node_multi(g, p, I);
  double F[D * D];
#pragma unroll
  for (int c = 0; c < D * D; ++c) F[c] = g.lo[c] + I[c] * g.delta;
  const r1d::Point<T> q = r1d::make_point_any<T>(mat, bn);
  double cof[D * D];
  r1d::cofactor<D>(F, cof);
  const T w = r1d::w_point_any<T, D>(q, F, cof);
  W[p] = w < inf_t<T>() ? w : inf_t<T>();
  if (P) {
    double S[D * D];
    r1d::stress0_any<D>(mat, bn, F, S);
#pragma unroll
    for (int c = 0; c < D * D; ++c) P[int64_t(c) * g.size + p] = T(S[c]);
  }
  if (A) r1d::tangent0_store<D>(mat, bn, F, A + p, g.size);
}

// Hulls of some directions of a group of up to kGroupMax directions of one
// iteration, one thread per line, 64 consecutive line starts of one direction per
// wave (so accesses coalesce).  The blocks of the launch's i-th direction, group
// slot slot[i], are block_end[i-1] .. block_end[i]-1, so a block's direction (and
// its Step, read through scalar loads) is uniform.  Only the lines of at least 3
// nodes are covered (shorter ones hold no node strictly inside a segment).
// A node's candidate is the hull value ((b - q) w_a + (q - a) w_b) / (b - a)
// where it lies strictly inside a hull segment [a, b] and its own value is finite;
// with offs, also the offsets (q - a) | (b - q) << 16 of its laminate.  Non-finite
// values are absent from a hull.  Only candidates that the pick could take (lower
// than the node's own value by more than its margin: the running value it is
// compared with is never above the node's own) are written, and marked in the
// node's mark byte of the group slot; unmarked slots hold no value.  A node has 4
// mark bytes when no group has more than 4 hull directions, else 16 (each written
// by one thread, so plain stores do: an atomic bit mask took the 5.8M-node mesh's
// hulls from 0.10 to 0.13 ms).
constexpr int kGroupMax = 16;
constexpr int kBitLine = 64;   // lines of at most this many nodes keep their hull as a bit mask

// Ends an iteration's launches when the iteration before met the tolerance (its
// maximal decrease is at prev; null: no iteration before): an iteration is enqueued
// before the host has read the one before, and must then do nothing.
struct Guard {
  const unsigned long long* prev;
  double tol;
  __device__ __forceinline__ bool stop() const {
    return prev && __longlong_as_double((long long)(*prev)) <= tol;
  }
};

struct Group {
  int n;                       // directions of this launch ...
  int dir[kGroupMax];          // ... their indices
  int slot[kGroupMax];         // ... their candidate slots in the group
  int waves[kGroupMax];        // ... the waves of a block that take lines of it (their LDS is a block's share)
  int block_end[kGroupMax];    // prefix sums of their blocks
};

// What a candidate has to stay below to lower a node of value w (see k_grid_pick).
template <typename T>
__device__ __forceinline__ T pick_limit(T w) { return w - T(4) * eps_t<T>() * fmax(fabs(w), T(1e-3)); }

// The direction of a block, its wave's share of the block's LDS, and this thread's
// line start of the direction.
struct LineRef {
  int slot, dir, waves;
  int64_t t;
};
__device__ __forceinline__ LineRef line_of_block(const Group& grp, int blk, int tid) {
  int i = 0;
#pragma unroll
  for (int k = 0; k < kGroupMax; ++k) i += (k < grp.n && blk >= grp.block_end[k]) ? 1 : 0;
  return LineRef{grp.slot[i], grp.dir[i], grp.waves[i],
                 int64_t(blk - (i ? grp.block_end[i - 1] : 0)) * grp.waves[i] * kLineThreads + tid};
}

// Lines of at most 64 nodes.  A block of 4 waves shares lds_bytes of LDS: 4 or 2 of
// its waves take lines, as many as their columns fit (entry q of a thread's line
// at [q * kLineThreads] of its wave's share), so that one launch holds the short
// lines at full occupancy and the few long ones beside them.
//   ch (nullable): nodes that the previous iteration changed.  A line without one
// has the candidates it had then, and none of them lowers its node: the node was
// offered it and kept a value that it does not lie below by the margin, or has
// taken a lower one since.  A wave without such a line ends before it reads a value.
//   A line whose consecutive differences grow strictly pops nothing from the
// monotone chain and has no candidate; a wave of such lines ends when it has read
// them.  Otherwise each line runs the chain through its LDS column from its first
// pop on (from its start where a value is absent): the top vertex is popped while
// the slope into it is at least the slope from it to the new point (collinear
// points are not kept), in one flat loop of pops and pushes, the vertices a bit
// mask, the next value and the third vertex read ahead.
//   What bounds it is instruction issue in the reading (about 10 per node) and the
// latency of the chains that are left.  672,400-node 2D mesh, 14 directions of
// 20-node and 2 of 41-node lines, FP64: 64 us an iteration, against 135 us with a
// launch per length class, index stacks in LDS, every candidate written and every
// chain run (of which writing only useful candidates and ending convex and unchanged
// waves gave 52 us, the one launch and the cheaper reading 19 us); 13-24% of the
// nodes change in an iteration and 31-53% of the lines hold one.  5.8M-node 3D mesh,
// three directions of 20-node lines: 86 us, 100 us before.
template <typename T, int DD, int CHUNK>
__global__ __launch_bounds__(4 * kLineThreads) void k_grid_hulls(GridArgs g, const Step* __restrict__ steps, Group grp,
                                                                Guard guard, int lds_bytes, const T* __restrict__ Win,
                                                                const uint8_t* __restrict__ ch,
                                                                T* __restrict__ cand, uint32_t* __restrict__ offs,
                                                                uint8_t* __restrict__ marks, int mark_bytes) {
  extern __shared__ __align__(8) unsigned char line_mem[];
  if (guard.stop()) return;
  const LineRef ref = line_of_block(grp, blockIdx.x, threadIdx.x);
  const int wave = threadIdx.x / kLineThreads;
  if (wave >= ref.waves) return;                  // waves are independent: no barrier below
  const Step& s = steps[ref.dir];
  const bool live = ref.t < s.count;
  if (!__any(live)) return;
  int I[9];
  const uint32_t p = uint32_t(line_start<DD>(g, s, live ? ref.t : s.count - 1, I));
  const uint32_t ds = uint32_t(s.ds);             // node indices are below 2^31: 32-bit steps wrap correctly
  const int L = line_length<DD>(g, s, I);         // 3 .. 64
  bool act = live;
  if (ch) {
    uint32_t any = 0;
    uint32_t node = p;
    for (int q0 = 0; q0 < L; q0 += CHUNK) {
#pragma unroll
      for (int i = 0; i < CHUNK; ++i) {
        any |= ch[node];
        node += q0 + i + 1 < L ? ds : 0u;         // the last node again beyond the end
      }
    }
    act = act && any != 0;
    if (!__any(act)) return;
  }
  T* const vin = reinterpret_cast<T*>(line_mem + wave * (lds_bytes / ref.waves)) + threadIdx.x % kLineThreads;
  auto win = [&](int q) -> T { return vin[q * kLineThreads]; };
  // pop: the first node whose step is not above the one before; gap: an absent value
  // between present ones (differences across absent ends compare false)
  int pop = kBitLine, beg = 0;                    // beg: absent values before the first present one
  bool seen = false, ended = false, gap = false;
  {
    T w1 = inf_t<T>(), d1 = T(__builtin_nan(""));
    uint32_t node = p;
    for (int q0 = 0; q0 < L; q0 += CHUNK) {
      T a[CHUNK];                                 // independent loads: one memory round trip
#pragma unroll
      for (int i = 0; i < CHUNK; ++i) {
        a[i] = Win[node];
        node += q0 + i + 1 < L ? ds : 0u;
      }
#pragma unroll
      for (int i = 0; i < CHUNK; ++i) {
        const int q = q0 + i;
        const bool in = q < L;
        const T w = a[i], d = w - w1;
        const bool f = w < inf_t<T>();
        if (in) vin[q * kLineThreads] = w;
        if (in && d1 >= d) pop = min(pop, q);
        seen = seen || f;
        beg = seen ? beg : q + 1;
        gap = gap || (in && f && ended);
        ended = ended || (!f && seen);
        w1 = w;
        d1 = d;
      }
    }
  }
  act = act && (pop < kBitLine || gap);
  if (!__any(act)) return;
  if (!act) return;
  // from the first pop with the vertices before it (without a gap: nodes beg .. pop - 1),
  // or from the start
  int q = gap ? 0 : pop;
  unsigned long long fin = gap ? 0ull : ((1ull << q) - 1ull) & ~((1ull << beg) - 1ull);   // present nodes
  unsigned long long hm = fin;                                                            // vertices
  // the top three vertices, i2 the top (values of fewer vertices are not looked at)
  int i2 = max(q - 1, 0), i1 = max(q - 2, 0), i0 = max(q - 3, 0);
  T v2 = win(i2), v1 = win(i1), v0 = win(i0), w = win(q), wn = win(min(q + 1, L - 1));
  while (q < L) {
    const bool f = w < inf_t<T>();
    if (f && (hm & (hm - 1)) && (v2 - v1) * T(q - i2) >= (w - v2) * T(i2 - i1)) {
      hm &= ~(1ull << i2);
      i2 = i1;
      v2 = v1;
      i1 = i0;
      v1 = v0;
      const unsigned long long below = hm & ((1ull << i1) - 1ull);
      i0 = below ? 63 - __builtin_clzll(below) : 0;
      v0 = win(i0);
      continue;
    }
    if (f) {
      fin |= 1ull << q;
      hm |= 1ull << q;
      i0 = i1;
      v0 = v1;
      i1 = i2;
      v1 = v2;
      i2 = q;
      v2 = w;
    }
    ++q;
    w = wn;
    wn = win(min(q + 1, L - 1));
  }
  // the first and the last finite node are vertices, so every other finite node
  // that is not one lies inside a segment
  T* const cd = cand + int64_t(ref.slot) * g.size;
  for (unsigned long long rest = fin & ~hm; rest; rest &= rest - 1) {
    const int c = __builtin_ctzll(rest);
    const int a = 63 - __builtin_clzll(hm & ((1ull << c) - 1ull));
    const int b = c + __builtin_ctzll(hm >> c);
    const T val = (T(b - c) * win(a) + T(c - a) * win(b)) / T(b - a);
    if (val < pick_limit(win(c))) {
      const uint32_t node = p + uint32_t(c) * ds;
      cd[node] = val;
      if (offs) offs[int64_t(ref.slot) * g.size + node] = uint32_t(c - a) | (uint32_t(b - c) << 16);
      marks[int64_t(node) * mark_bytes + ref.slot] = 1;
    }
  }
}

// Longer lines: the chain's vertices are a stack of offsets in LDS.  STAGED: the
// values sit in the thread's LDS column; otherwise they are read in place.  Staged
// where columns and stacks fit kStageBytes (FP64 89, FP32 149 nodes): 140 x 2 x 2 x 140
// nodes, FP32, random values, four iterations: 500 us, 724 read in place.
template <typename T, bool STAGED>
__global__ __launch_bounds__(kLineThreads) void k_grid_hulls_long(GridArgs g, const Step* __restrict__ steps, Group grp,
                                                                 Guard guard, const T* __restrict__ Win, T* __restrict__ cand,
                                                                 uint32_t* __restrict__ offs,
                                                                 uint8_t* __restrict__ marks, int mark_bytes, int len) {
  extern __shared__ __align__(8) unsigned char line_mem[];
  const int tid = threadIdx.x;
  if (guard.stop()) return;
  const LineRef ref = line_of_block(grp, blockIdx.x, tid);
  const Step& s = steps[ref.dir];
  if (ref.t >= s.count) return;
  int I[9];
  const int64_t p = line_start<9>(g, s, ref.t, I);
  const int64_t ds = s.ds;
  const int L = line_length<9>(g, s, I);
  T* const vin = reinterpret_cast<T*>(line_mem) + tid;  // STAGED only
  uint16_t* const st = reinterpret_cast<uint16_t*>(reinterpret_cast<T*>(line_mem) +
                                                   (STAGED ? len * kLineThreads : 0)) + tid;
  auto win = [&](int q) -> T { return STAGED ? vin[q * kLineThreads] : Win[p + q * ds]; };
  if constexpr (STAGED) {
    // chunks of independent loads: a line costs a few memory round trips, not L
    constexpr int CHUNK = 32;
    for (int q0 = 0; q0 < L; q0 += CHUNK) {
      T a[CHUNK];
#pragma unroll
      for (int i = 0; i < CHUNK; ++i) a[i] = Win[p + min(q0 + i, L - 1) * ds];
#pragma unroll
      for (int i = 0; i < CHUNK; ++i)
        if (q0 + i < L) vin[(q0 + i) * kLineThreads] = a[i];
    }
  }
  int h = 0, i1 = 0, i2 = 0;
  T v1 = T(0), v2 = T(0);
  {
    int q = 0;
    T w = win(0);
    while (q < L) {
      const bool fin = w < inf_t<T>();
      if (fin && h >= 2 && (v2 - v1) * T(q - i2) >= (w - v2) * T(i2 - i1)) {
        --h;
        i2 = i1;
        v2 = v1;
        if (h >= 2) {
          i1 = st[(h - 2) * kLineThreads];
          v1 = win(i1);
        }
        continue;
      }
      if (fin) {
        st[h * kLineThreads] = uint16_t(q);
        ++h;
        i1 = i2;
        v1 = v2;
        i2 = q;
        v2 = w;
      }
      ++q;
      if (q < L) w = win(q);
    }
  }
  if (h < 2) return;
  // candidates along the line, one flat loop; (a, b) is the segment holding q
  T* const cd = cand + int64_t(ref.slot) * g.size;
  int k = 1, a = st[0], b = st[kLineThreads];
  T wa = win(a), wb = win(b);
  const int last = st[(h - 1) * kLineThreads];
  for (int q = a + 1; q < last; ++q) {
    if (q == b) {
      a = b;
      wa = wb;
      ++k;
      b = st[k * kLineThreads];
      wb = win(b);
      continue;
    }
    const T own = win(q);
    if (!(own < inf_t<T>())) continue;
    const T val = (T(b - q) * wa + T(q - a) * wb) / T(b - a);
    if (val < pick_limit(own)) {
      const int64_t node = p + q * ds;
      cd[node] = val;
      if (offs) offs[int64_t(ref.slot) * g.size + node] = uint32_t(q - a) | (uint32_t(b - q) << 16);
      marks[int64_t(node) * mark_bytes + ref.slot] = 1;
    }
  }
}

// What the pick launch needs of a direction: the node index step; the slot of
// its candidates, or -1 where the pick forms them itself (lines of at most three
// nodes, steps of -1, 0, 1: only a node with both neighbours inside the box is
// the middle of such a line); the bit mask of the components it steps.
struct PickDir {
  int32_t ds;
  uint32_t need;
  int32_t slot;
  int32_t dir;
};

// Bit c set: node p has both neighbours in component c.
template <int DD>
__device__ __forceinline__ uint32_t interior_mask(const GridArgs& g, uint32_t p) {
  uint32_t m = 0;
#pragma unroll
  for (int c = DD - 1; c >= 0; --c) {
    // p / n through FP64: (p + 1/2) / n is at least 1 / 1024 from an integer, and
    // p < 2^31 leaves the product's rounding far below that
    const uint32_t n = uint32_t(g.n[c]), q = uint32_t((double(p) + 0.5) * g.inv_n[c]), i = p - q * n;
    m |= (i >= 1 && i + 1 < n) ? 1u << c : 0u;
    p = q;
  }
  return m;
}

// The candidates of ne directions, in order, per node: a candidate replaces the
// running value only when lower by more than 4 units of rounding relative to
// max(|W|, 1e-3), so directions that tie to rounding leave the node to the first.
// kFirst: the running value starts from Win (else Wout, and with sel the running
// laminate) and every node is written.  Only the marked slots of a node count
// (with kNb a slot is loaded with its mark still under way, and dropped where there is
// none), and its marks go back to 0.
// The maximal decrease Win - W over nodes with finite Win goes to *dec (atomic
// maximum of the non-negative doubles' bit patterns; W only decreases over the
// groups, so the maximum over the nodes the groups lower is the iteration's).
// kLast: the node stresses / moduli of the laminate that lowered a node, with the
// weights of its value (eq. 5.2, first case), or the node's own, go to Pout / Aout;
// whether the iteration changed the node goes to ch.
//
// kNb: some directions have slot -1; the node reads its two neighbours for those.
// Which of them concern a node depends only on its interior mask, so k_grid_lists
// writes for each of the 2^(d*d) masks the directions to look at, in order (once
// per call), and each lane works off its own mask's list, four directions at a
// time so that eight loads are in flight: on the 5.8M-node 3D mesh 18 of the 169
// directions per node on average, 30 per wave.  What bounds it is the issue of
// those steps (FP64 compares and 64-bit addresses, about 45 instructions each) and
// the latency of the neighbour reads.  On that mesh an iteration takes 0.45 ms
// (pick 0.35, the three long directions' hulls 0.10) against 2.2 ms when every
// direction had a hull launch and a candidate array; testing all 169 directions
// per wave in scalar code instead of the lists took 1.33 ms.  The blocks take
// contiguous node ranges, an eighth of the mesh per XCD, so that the neighbours
// (up to 400,000 nodes away there) are found in that XCD's L2; 4096 blocks rather
// than 2048 keep the 2D meshes at one strip of 256 nodes a block (pick 32 against
// 42 us, 3D 0.35 against 0.45 ms).
enum : int { kFirst = 1, kLast = 2 };
constexpr unsigned kPickBlocks = 4096;  // 16 blocks per CU, each a contiguous range of nodes
constexpr int kPickBatch = 4;

template <typename T>
struct Carry {
  const T* Pin;
  T* Pout;
  const T* Ain;
  T* Aout;
  int32_t* sel;            // running laminate: direction (-1: none) ...
  uint32_t* soff;          // ... and its offsets, kept between groups
};

// An entry of a mask's list: the node index step (0 where a slot holds the
// candidate), and direction << 5 | slot + 1.
__device__ __forceinline__ long long list_entry(const PickDir& d) {
  const uint32_t ds = d.slot < 0 ? uint32_t(d.ds) : 0u;
  return (long long)((unsigned long long)ds | (unsigned long long)uint32_t(d.dir << 5 | (d.slot + 1)) << 32);
}

// lists[M * pitch ..]: the entries of dirs that a node with interior mask M looks
// at, in order, filled up to a multiple of kPickBatch with the last of them (whose
// candidate, once taken, does not lie below the value it gave; a step of 0 would make the
// node its own neighbour, whose midpoint is -inf where the node's double overflows);
// counts[M] their number.  One wave per mask.
__global__ __launch_bounds__(64) void k_grid_lists(const PickDir* __restrict__ dirs, int ne, int pitch,
                                                   long long* __restrict__ lists, int* __restrict__ counts) {
  const uint32_t M = blockIdx.x;
  const int lane = threadIdx.x;
  long long* const list = lists + int64_t(M) * pitch;
  int at = 0;
  long long last = 0;
  for (int e0 = 0; e0 < ne; e0 += 64) {
    const int e = e0 + lane;
    const PickDir d = dirs[e < ne ? e : 0];
    const bool v = e < ne && (d.slot >= 0 || (d.need & ~M) == 0u);
    const unsigned long long b = __ballot(v);
    const long long entry = list_entry(d);
    if (v) list[at + __popcll(b & ((1ull << lane) - 1ull))] = entry;
    if (b) last = __shfl(entry, 63 - __builtin_clzll(b), 64);
    at += __popcll(b);
  }
  const int full = (at + kPickBatch - 1) / kPickBatch * kPickBatch;
  if (at + lane < full) list[at + lane] = last;
  if (lane == 0) counts[M] = full;
}

// The node's marks as a bit mask (bit = slot); they go back to 0.
template <int BYTES>
__device__ __forceinline__ uint32_t take_marks(uint8_t* marks, int64_t node) {
  auto bits = [](uint32_t w) { return (w | w >> 7 | w >> 14 | w >> 21) & 15u; };
  if constexpr (BYTES == 4) {
    uint32_t* const at = reinterpret_cast<uint32_t*>(marks) + node;
    const uint32_t w = *at;
    if (w) *at = 0u;
    return bits(w);
  } else {
    uint4* const at = reinterpret_cast<uint4*>(marks) + node;
    const uint4 w = *at;
    if (w.x | w.y | w.z | w.w) *at = make_uint4(0u, 0u, 0u, 0u);
    return bits(w.x) | bits(w.y) << 4 | bits(w.z) << 8 | bits(w.w) << 12;
  }
}

template <typename T, int DD, bool kNb, int BYTES>
__global__ __launch_bounds__(256) void k_grid_pick(GridArgs g, Guard guard, int strips,
                                                   const Step* __restrict__ steps,
                                                   const PickDir* __restrict__ dirs, int ne,
                                                   int pitch, const longlong2* __restrict__ lists,
                                                   const int* __restrict__ counts,
                                                   const T* __restrict__ Win, T* __restrict__ Wout,
                                                   const T* __restrict__ cand, const uint32_t* __restrict__ offs,
                                                   uint8_t* __restrict__ marks, uint8_t* __restrict__ ch,
                                                   Carry<T> cy, int flags, unsigned long long* dec) {
  if (guard.stop()) return;
  const int64_t n = g.size;
  const bool first = flags & kFirst;
  const bool carry = cy.Pout || cy.Aout;
  // gridDim.x is a multiple of 8; blocks go to the 8 XCDs in turn
  const int64_t blk = int64_t(blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  double m = 0.0;
  for (int strip = 0; strip < strips; ++strip) {
    const int64_t p0 = (blk * strips + strip) * 256;
    if (p0 >= n) break;                          // block-uniform
    const int64_t node = p0 + threadIdx.x;
    const bool live = node < n;
    const T w0 = live ? Win[node] : inf_t<T>();
    const uint32_t mk = live ? take_marks<BYTES>(marks, node) : 0u;
    T cur = first || !live ? w0 : Wout[node];
    int32_t sl = -1;
    uint32_t so = 0;
    if (carry && !first && live) {
      sl = cy.sel[node];
      so = cy.soff[node];
    }
    bool changed = false;
    int sslot = -1;                              // candidate slot of the laminate taken here
    T lim = pick_limit(cur);
    auto take = [&](T c, int dir, int slot) {
      cur = c;
      lim = pick_limit(c);
      sl = dir;
      sslot = slot;
      changed = true;
    };
    if constexpr (kNb) {
      // a node with no finite value of its own is the middle of nothing
      const uint32_t in = live && w0 < inf_t<T>() ? interior_mask<DD>(g, uint32_t(node)) : 0u;
      const int cnt = live ? counts[in] : 0;
      const longlong2* const list = lists + int64_t(in) * (pitch / 2);
      const T* const wn = Win + node;
      const T* const cn = cand + node;
      for (int k0 = 0; k0 < cnt; k0 += kPickBatch) {
        const longlong2 e01 = list[k0 / 2], e23 = list[k0 / 2 + 1];
        const long long e[kPickBatch] = {e01.x, e01.y, e23.x, e23.y};
        T a[kPickBatch], b[kPickBatch];
#pragma unroll
        for (int j = 0; j < kPickBatch; ++j) {
          const int64_t ds = int32_t(e[j]);
          const uint32_t slot1 = uint32_t(e[j] >> 32) & 31u;      // slot + 1
          a[j] = *(slot1 ? cn + uint64_t(slot1 - 1u) * uint32_t(n) : wn - ds);
          b[j] = wn[ds];
        }
#pragma unroll
        for (int j = 0; j < kPickBatch; ++j) {
          const uint32_t code = uint32_t(e[j] >> 32), slot1 = code & 31u;
          // the monotone chain on three nodes: the middle one is popped exactly when
          // it lies on or above the chord, and its candidate is the chord's midpoint
          // (an absent neighbour, +inf or NaN, fails the comparisons)
          const bool cut = w0 - a[j] >= b[j] - w0;
          const bool ok = slot1 ? ((mk >> (slot1 - 1u)) & 1u) != 0u : cut;
          const T c = slot1 ? a[j] : (a[j] + b[j]) / T(2);
          if (ok && c < lim) take(c, int(code >> 5), int(slot1) - 1);
        }
      }
    } else {
      T v[kGroupMax];                            // all loads first, then the ordered choice
#pragma unroll
      for (int j = 0; j < kGroupMax; ++j)
        v[j] = (mk >> j) & 1u ? cand[int64_t(j) * n + node] : inf_t<T>();
#pragma unroll
      for (int j = 0; j < kGroupMax; ++j)
        if (v[j] < lim) take(v[j], dirs[j].dir, j);
    }
    if (!live) continue;
    if (changed) so = sslot < 0 ? 1u | (1u << 16) : offs ? offs[int64_t(sslot) * n + node] : 0u;
    if (flags & kLast) ch[node] = cur == w0 ? 0 : 1;
    if (first || changed) Wout[node] = cur;
    if (changed && w0 < inf_t<T>()) m = fmax(m, double(w0) - double(cur));
    if (carry && !(flags & kLast) && (first || changed)) {
      cy.sel[node] = sl;
      cy.soff[node] = so;
    }
    if (carry && (flags & kLast)) {
      int64_t ia = node, ib = node;
      int qa = 0, bq = 0;
      if (sl >= 0) {
        qa = int(so & 0xffffu);
        bq = int(so >> 16);
        ia = node - qa * steps[sl].ds;
        ib = node + bq * steps[sl].ds;
      }
      if (cy.Pout)
        for (int c = 0; c < DD; ++c)
          cy.Pout[c * n + node] = sl < 0 ? cy.Pin[c * n + node]
                                         : (T(bq) * cy.Pin[c * n + ia] + T(qa) * cy.Pin[c * n + ib]) / T(qa + bq);
      if (cy.Aout)
        for (int c = 0; c < DD * DD; ++c)
          cy.Aout[c * n + node] = sl < 0 ? cy.Ain[c * n + node]
                                         : (T(bq) * cy.Ain[c * n + ia] + T(qa) * cy.Ain[c * n + ib]) / T(qa + bq);
    }
  }
  // one atomic per block (the launch has a bounded number of blocks)
  __shared__ double red[4];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    m = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
    if (m > 0.0) atomicMax(dec, static_cast<unsigned long long>(__double_as_longlong(m)));
  }
}

__global__ __launch_bounds__(256) void k_grid_zero(int64_t n, uint32_t* a) {
  const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (i < n) a[i] = 0u;
}

// Multilinear interpolation of the node values at n points F (SoA, d*d x n):
// corners of zero weight do not take part; NaN outside the box (beyond a
// rounding margin of 1e-9 mesh widths).  LP lanes share a point: lane sub of them
// takes the corners whose leading log2(LP) bits (one per component, the slowest
// first) are sub, so its own corners are the nearest in memory, and the lanes'
// sums meet in a butterfly.
template <typename T, int D, int LP>
__global__ __launch_bounds__(256) void k_grid_interp(GridArgs g, const T* W, int64_t n, const T* F, T* out) {
  const int64_t t = int64_t(blockIdx.x) * 256 + threadIdx.x;
  const int64_t p = t / LP;
  const int sub = int(t % LP);
  if (p >= n) return;                            // whole groups of LP lanes
  constexpr int DD = D * D;
  constexpr int kLead = LP == 64 ? 6 : 0;
  static_assert((1 << kLead) == LP && kLead <= DD, "lanes per point");
  int base[DD];
  double frac[DD];
  bool inside = true;
#pragma unroll
  for (int c = 0; c < DD; ++c) {
    double u = (double(F[int64_t(c) * n + p]) - g.lo[c]) / g.delta;
    const double top = double(g.n[c] - 1);
    inside = inside && u >= -1e-9 && u <= top + 1e-9;
    u = u < 0.0 ? 0.0 : (u > top ? top : u);
    int i = int(floor(u));
    i = i > g.n[c] - 2 ? g.n[c] - 2 : i;
    i = i < 0 ? 0 : i;
    base[c] = i;
    frac[c] = g.n[c] > 1 ? u - i : 0.0;
  }
  if (!inside) {
    if (sub == 0) out[p] = T(__builtin_nan(""));
    return;
  }
  double lead = 1.0;                             // weight and node index of the lane's leading bits
  int64_t at = 0;
#pragma unroll
  for (int c = 0; c < kLead; ++c) {
    const int up = (sub >> (kLead - 1 - c)) & 1;
    if (up && g.n[c] == 1) lead = 0.0;
    lead *= up ? frac[c] : 1.0 - frac[c];
    at += int64_t(base[c] + up) * g.stride[c];
  }
  double sum = 0.0;
#pragma unroll 8
  for (int corner = 0; corner < (1 << (DD - kLead)); ++corner) {
    double wgt = lead;
    int64_t idx = at;
#pragma unroll
    for (int c = kLead; c < DD; ++c) {
      const int up = (corner >> (DD - 1 - c)) & 1;
      if (up && g.n[c] == 1) wgt = 0.0;
      wgt *= up ? frac[c] : 1.0 - frac[c];
      idx += int64_t(base[c] + up) * g.stride[c];
    }
    if (wgt != 0.0) sum += wgt * double(W[idx]);
  }
#pragma unroll
  for (int o = LP / 2; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
  if (sub == 0) out[p] = T(sum);
}

inline unsigned blocks_of(int64_t n, int b) { return unsigned((n + b - 1) / b); }

// Device scratch of one laminate call: the other iterate (and stress / moduli
// iterates), the per-iteration decreases, the steps, and one group's candidates.
template <typename T>
struct GridWork {
  T* W2 = nullptr;
  T* P2 = nullptr;
  T* A2 = nullptr;
  unsigned long long* dec = nullptr;
  Step* steps = nullptr;
  PickDir* dirs = nullptr;
  long long* lists = nullptr;  // k_grid_lists, 2^(d*d) masks per group with neighbour directions
  int* counts = nullptr;
  T* cand = nullptr;
  uint32_t* offs = nullptr;
  uint8_t* marks = nullptr;
  int mark_bytes = 0;          // per node
  uint8_t* ch = nullptr;
  int32_t* sel = nullptr;
  uint32_t* soff = nullptr;
};

inline size_t round256(size_t b) { return (b + 255) & ~size_t(255); }


// The direction's candidates are formed by the pick launch: lines of at most three
// nodes, at consecutive mesh nodes.
inline bool by_neighbours(const GridArgs& g, const Step& s) {
  for (int c = 0; c < g.dd; ++c)
    if (s.s[c] < -1 || s.s[c] > 1) return false;
  return s.len <= 3;
}

// The iteration's work list: the directions in order without those whose lines
// hold fewer than three nodes (no node strictly inside a segment), cut into
// groups with at most kGroupMax hull directions each.
struct Segment {
  int e0, n;               // entries of the pick launch
  bool neighbours;         // some entry is formed from neighbours ...
  int pitch;               // ... then the entries per interior mask in its lists
  int64_t list0;           // ... and the lists' offset
};

inline void plan_groups(const GridArgs& g, const std::vector<Step>& steps, std::vector<PickDir>* dirs,
                        std::vector<Segment>* segs) {
  int slots = 0;
  segs->push_back(Segment{});
  for (size_t d = 0; d < steps.size(); ++d) {
    const Step& s = steps[d];
    if (s.len < 3) continue;
    const bool nb = by_neighbours(g, s);
    if (!nb && slots == kGroupMax) {
      segs->push_back(Segment{int(dirs->size())});
      slots = 0;
    }
    PickDir p{};
    p.ds = int32_t(s.ds);
    p.slot = nb ? -1 : slots++;
    p.dir = int32_t(d);
    for (int c = 0; c < g.dd; ++c) p.need |= s.s[c] != 0 ? 1u << c : 0u;
    dirs->push_back(p);
    segs->back().n += 1;
    segs->back().neighbours |= nb;
  }
  int64_t at = 0;
  for (Segment& sg : *segs) {
    sg.pitch = (sg.n + kPickBatch - 1) / kPickBatch * kPickBatch;
    sg.list0 = at;
    if (sg.neighbours) at += int64_t(sg.pitch) << g.dd;
  }
}

// One iteration: for each group of directions, the hull launches then the pick
// launch.  ch: the previous iteration's changed nodes (null on the first); guard:
// whether there is anything left to do.
template <typename T>
hipError_t grid_sweep(const GridArgs& g, const std::vector<Step>& steps, const std::vector<PickDir>& dirs,
                      const std::vector<Segment>& segs, const GridWork<T>& wk, const T* Win,
                      const uint8_t* ch, T* Wout, Carry<T> cy, Guard guard, unsigned long long* dec, hipStream_t st,
                      KTimer* tm) {
  const bool carry = cy.Pout || cy.Aout;
  for (size_t sg = 0; sg < segs.size(); ++sg) {
    const Segment& seg = segs[sg];
    uint32_t* offs = carry ? wk.offs : nullptr;
    // the hull directions with lines of at most kBitLine nodes in one launch, then
    // those of at most 128 and longer ones
    for (int part = 0; part < 3; ++part) {
      Group grp{};
      int len = 1, main_len = 1;
      int64_t main_lines = 0;
      for (int j = 0; j < seg.n; ++j) {
        const PickDir& p = dirs[size_t(seg.e0 + j)];
        if (p.slot < 0) continue;
        const Step& s = steps[size_t(p.dir)];
        if ((s.len <= kBitLine ? 0 : s.len <= 128 ? 1 : 2) != part || s.count == 0) continue;
        grp.dir[grp.n] = p.dir;
        grp.slot[grp.n] = p.slot;
        ++grp.n;
        len = std::max(len, s.len);
        int64_t lines = 0;                     // lines of the directions of this length
        for (int i = 0; i < grp.n; ++i)
          if (steps[size_t(grp.dir[i])].len == s.len) lines += steps[size_t(grp.dir[i])].count;
        if (lines > main_lines) {
          main_lines = lines;
          main_len = s.len;
        }
      }
      if (grp.n == 0) continue;
      // LDS of a 4-wave block: the columns of 4 waves of the most frequent length (2 if
      // that passes 64 KB), or of 2 of the longest if those need more
      const size_t column = sizeof(T) * size_t(kLineThreads);
      const int main_waves = column * 4 * size_t(main_len) <= size_t(64) * 1024 ? 4 : 2;
      const size_t share = column * size_t(std::max(main_waves * main_len, 2 * len));
      int blocks = 0;
      for (int i = 0; i < grp.n; ++i) {
        const Step& s = steps[size_t(grp.dir[i])];
        grp.waves[i] = part > 0 ? 1 : column * 4 * size_t(s.len) <= share ? 4 : 2;
        blocks += int(blocks_of(s.count, kLineThreads * grp.waves[i]));
        grp.block_end[i] = blocks;
      }
      if (tm) tm->begin("grid_lines", st);
      if (part == 0) {
        const auto hulls = g.dd == 4 ? (main_len <= 8    ? k_grid_hulls<T, 4, 8>
                                        : main_len <= 16 ? k_grid_hulls<T, 4, 16>
                                        : main_len <= 24 ? k_grid_hulls<T, 4, 24>
                                                         : k_grid_hulls<T, 4, 32>)
                                     : (main_len <= 8    ? k_grid_hulls<T, 9, 8>
                                        : main_len <= 16 ? k_grid_hulls<T, 9, 16>
                                        : main_len <= 24 ? k_grid_hulls<T, 9, 24>
                                                         : k_grid_hulls<T, 9, 32>);
        hipLaunchKernelGGL(hulls, dim3(blocks), dim3(4 * kLineThreads), share, st, g, wk.steps, grp, guard, int(share), Win,
                           ch, wk.cand, offs, wk.marks, wk.mark_bytes);
      } else {
        const size_t stack = sizeof(uint16_t) * size_t(kLineThreads) * size_t(len);
        const bool staged = column * size_t(len) + stack <= size_t(kStageBytes);
        const auto hulls = staged ? k_grid_hulls_long<T, true> : k_grid_hulls_long<T, false>;
        hipLaunchKernelGGL(hulls, dim3(blocks), dim3(kLineThreads), staged ? column * size_t(len) + stack : stack, st,
                           g, wk.steps, grp, guard, Win, wk.cand, offs, wk.marks, wk.mark_bytes, len);
      }
      if (tm) tm->end(st);
    }
    const int flags = (sg == 0 ? kFirst : 0) | (sg + 1 == segs.size() ? kLast : 0);
    Carry<T> c = cy;
    c.sel = carry ? wk.sel : nullptr;
    c.soff = carry ? wk.soff : nullptr;
    if (tm) tm->begin("grid_pick", st);
    const unsigned pick_blocks = std::min<unsigned>((blocks_of(g.size, 256) + 7u) & ~7u, kPickBlocks);
    const unsigned strips = (blocks_of(g.size, 256) + pick_blocks - 1) / pick_blocks;   // of 256 nodes, per block
    const bool m4 = wk.mark_bytes == 4;
    const auto pick =
        g.dd == 4 ? (seg.neighbours ? (m4 ? k_grid_pick<T, 4, true, 4> : k_grid_pick<T, 4, true, 16>)
                                    : (m4 ? k_grid_pick<T, 4, false, 4> : k_grid_pick<T, 4, false, 16>))
                  : (seg.neighbours ? (m4 ? k_grid_pick<T, 9, true, 4> : k_grid_pick<T, 9, true, 16>)
                                    : (m4 ? k_grid_pick<T, 9, false, 4> : k_grid_pick<T, 9, false, 16>));
    hipLaunchKernelGGL(pick, dim3(pick_blocks), dim3(256), 0, st, g, guard, int(strips), wk.steps, wk.dirs + seg.e0, seg.n,
                       seg.pitch, reinterpret_cast<const longlong2*>(wk.lists + seg.list0),
                       wk.counts + (int64_t(sg) << g.dd), Win, Wout, wk.cand, carry ? wk.offs : nullptr, wk.marks,
                       wk.ch, c, flags, dec);
    if (tm) tm->end(st);
  }
  return hipGetLastError();
}

// steps enumerate the lines of at least 3 nodes.
template <typename T>
r1_status grid_laminate_T(r1_handle h, const GridArgs& g, const std::vector<Step>& steps, T* W, T* P, T* A,
                          int k_max, double tol, int32_t* iterations, double* decrease, hipStream_t st) {
  const size_t n = size_t(g.size);
  const bool carry = P || A;
  std::vector<PickDir> dirs;
  std::vector<Segment> segs;
  plan_groups(g, steps, &dirs, &segs);
  int G = 0;                                  // candidate slots
  for (const PickDir& p : dirs) G = std::max(G, p.slot + 1);
  size_t list_len = 0;
  for (const Segment& sg : segs)
    if (sg.neighbours) list_len = size_t(sg.list0) + (size_t(sg.pitch) << g.dd);
  const int mark_bytes = G <= 4 ? 4 : kGroupMax;
  const size_t step_bytes = round256(sizeof(Step) * steps.size());
  const size_t dir_bytes = round256(sizeof(PickDir) * std::max<size_t>(dirs.size(), 1));
  const size_t dec_bytes = round256(sizeof(unsigned long long) * size_t(k_max));
  const size_t mark_total = round256(size_t(mark_bytes) * n);
  size_t total = 0;
  auto place = [&](size_t bytes) { return std::exchange(total, total + round256(bytes)); };
  const size_t at_tables = place(step_bytes + dir_bytes), at_zeros = place(dec_bytes + mark_total),
               at_w2 = place(sizeof(T) * n), at_p2 = place(P ? sizeof(T) * n * size_t(g.dd) : 0),
               at_a2 = place(A ? sizeof(T) * n * size_t(g.dd * g.dd) : 0), at_cand = place(sizeof(T) * n * size_t(G)),
               at_offs = place(carry ? sizeof(uint32_t) * n * size_t(G) : 0),
               at_sel = place(carry ? sizeof(int32_t) * n : 0), at_soff = place(carry ? sizeof(uint32_t) * n : 0),
               at_lists = place(sizeof(long long) * list_len),
               at_counts = place(list_len ? sizeof(int) * (segs.size() << g.dd) : 0), at_ch = place(n);
  void* base = nullptr;
  r1_status s = r1h::scratch(h, total, &base);
  if (s) return s;
  auto at = [&](size_t off) -> void* { return static_cast<char*>(base) + off; };
  GridWork<T> wk;
  wk.steps = static_cast<Step*>(at(at_tables));
  wk.dirs = static_cast<PickDir*>(at(at_tables + step_bytes));
  wk.dec = static_cast<unsigned long long*>(at(at_zeros));
  wk.marks = static_cast<uint8_t*>(at(at_zeros + dec_bytes));
  wk.mark_bytes = mark_bytes;
  wk.W2 = static_cast<T*>(at(at_w2));
  wk.P2 = P ? static_cast<T*>(at(at_p2)) : nullptr;
  wk.A2 = A ? static_cast<T*>(at(at_a2)) : nullptr;
  wk.cand = static_cast<T*>(at(at_cand));
  wk.offs = static_cast<uint32_t*>(at(at_offs));
  wk.sel = static_cast<int32_t*>(at(at_sel));
  wk.soff = static_cast<uint32_t*>(at(at_soff));
  wk.lists = static_cast<long long*>(at(at_lists));
  wk.counts = static_cast<int*>(at(at_counts));
  wk.ch = static_cast<uint8_t*>(at(at_ch));
  std::vector<char> tables(step_bytes + dir_bytes);
  std::memcpy(tables.data(), steps.data(), sizeof(Step) * steps.size());
  if (!dirs.empty()) std::memcpy(tables.data() + step_bytes, dirs.data(), sizeof(PickDir) * dirs.size());
  hipError_t e = hipMemcpyAsync(wk.steps, tables.data(), tables.size(), hipMemcpyHostToDevice, st);
  if (e != hipSuccess) return r1h::fail(h, e, "grid steps");
  // the decreases, and the marks (the invariant the pick launches keep: none between groups)
  const int64_t words = int64_t((dec_bytes + mark_total) / 4);
  hipLaunchKernelGGL(k_grid_zero, dim3(blocks_of(words, 256)), dim3(256), 0, st, words,
                     static_cast<uint32_t*>(at(at_zeros)));
  for (size_t k = 0; k < segs.size(); ++k)
    if (segs[k].neighbours)
      hipLaunchKernelGGL(k_grid_lists, dim3(1u << g.dd), dim3(64), 0, st, wk.dirs + segs[k].e0, segs[k].n,
                         segs[k].pitch, wk.lists + segs[k].list0, wk.counts + (int64_t(k) << g.dd));
  KTimer* tm = h->timer.on ? &h->timer : nullptr;
  double* seen = nullptr;                      // two pinned words for the decreases read back ...
  hipEvent_t* ready = nullptr;                 // ... and the events after their copies
  s = r1h::readback(h, &seen, &ready);
  if (s) return s;
  // iteration i reads the iterate in W (even i) or W2 (odd i) and writes the other
  auto enqueue = [&](int i) -> hipError_t {
    const bool odd = i & 1;
    Carry<T> cy{odd ? wk.P2 : P, odd ? P : wk.P2, odd ? wk.A2 : A, odd ? A : wk.A2, nullptr, nullptr};
    const Guard guard{i ? wk.dec + (i - 1) : nullptr, tol};
    hipError_t r = grid_sweep<T>(g, steps, dirs, segs, wk, odd ? wk.W2 : W, i ? wk.ch : nullptr, odd ? W : wk.W2, cy,
                                 guard, wk.dec + i, st, tm);
    if (r == hipSuccess) r = hipMemcpyAsync(seen + (i & 1), wk.dec + i, sizeof(double), hipMemcpyDeviceToHost, st);
    if (r == hipSuccess) r = hipEventRecord(ready[i & 1], st);
    return r;
  };
  // one iteration ahead of the host's reading of the decreases, so that the device
  // does not wait for the host between iterations (with launch timing on, none ahead:
  // an iteration that turns out to be one too many would count as launches)
  const int ahead = tm ? 1 : 2;
  int k = 0, queued = 0;
  for (;;) {
    while (queued < k_max && queued - k < ahead) {
      e = enqueue(queued);
      if (e != hipSuccess) break;
      ++queued;
    }
    if (e == hipSuccess) e = hipEventSynchronize(ready[k & 1]);
    if (e != hipSuccess) {
      (void)hipStreamSynchronize(st);          // nothing of this call stays in flight
      return r1h::fail(h, e, "grid iteration");
    }
    const double md = seen[k & 1];
    if (decrease) decrease[k] = md;
    ++k;
    if (md <= tol || k == k_max) break;
  }
  if (k & 1) {
    e = hipMemcpyAsync(W, wk.W2, sizeof(T) * n, hipMemcpyDeviceToDevice, st);
    if (e == hipSuccess && P)
      e = hipMemcpyAsync(P, wk.P2, sizeof(T) * n * size_t(g.dd), hipMemcpyDeviceToDevice, st);
    if (e == hipSuccess && A)
      e = hipMemcpyAsync(A, wk.A2, sizeof(T) * n * size_t(g.dd * g.dd), hipMemcpyDeviceToDevice, st);
  }
  if ((k & 1) || queued > k) {                 // the workspace is the handle's: leave nothing using it
    const hipError_t e2 = hipStreamSynchronize(st);
    if (e == hipSuccess) e = e2;
    if (e != hipSuccess) return r1h::fail(h, e, "grid copy");
  }
  if (iterations) *iterations = k;
  return R1_OK;
}

template <typename T>
void launch_energy(int dim, dim3 grd, hipStream_t st, const GridArgs& g, const r1d::Material& m, double beta_n,
                   void* W, void* P, void* A) {
  T* w = static_cast<T*>(W);
  T* p = static_cast<T*>(P);
  T* a = static_cast<T*>(A);
  if (dim == 2)
    hipLaunchKernelGGL((k_grid_energy<T, 2>), grd, dim3(256), 0, st, g, m, beta_n, w, p, a);
  else
    hipLaunchKernelGGL((k_grid_energy<T, 3>), grd, dim3(256), 0, st, g, m, beta_n, w, p, a);
}

// Lanes per point: in 3D a point reads 512 corners, and one lane each for a few
// thousand points leaves the chip idle behind long chains of loads; a whole wave
// per point repeats the point's set-up on every lane and fills the chip earlier.
// FP64 on the 5.8M-node mesh, a lane / a wave per point: 2003 points 357 / 14 us,
// 32767 points 353 / 166 us, equal near 65,000 points (0.34 ms), beyond which the
// wave per point grows with the points and the lane per point does not yet.  In 2D
// the 16 corners are one round of loads.
template <typename T>
void launch_interp(int dim, const GridArgs& g, const void* W, int64_t n, const void* F, void* out, hipStream_t st) {
  const T* w = static_cast<const T*>(W);
  const T* f = static_cast<const T*>(F);
  T* o = static_cast<T*>(out);
  if (dim == 2)
    hipLaunchKernelGGL((k_grid_interp<T, 2, 1>), dim3(blocks_of(n, 256)), dim3(256), 0, st, g, w, n, f, o);
  else if (n < 65536)
    hipLaunchKernelGGL((k_grid_interp<T, 3, 64>), dim3(blocks_of(n * 64, 256)), dim3(256), 0, st, g, w, n, f, o);
  else
    hipLaunchKernelGGL((k_grid_interp<T, 3, 1>), dim3(blocks_of(n, 256)), dim3(256), 0, st, g, w, n, f, o);
}

}  // namespace

extern "C" {

r1_status r1_grid_r11(int32_t dim, int32_t* steps, int32_t* n_dir) {
  if ((dim != 2 && dim != 3) || !steps || !n_dir) return R1_EINVAL;
  const int dd = dim * dim;
  int count = 0;
  // a (x) b for a, b in {-1, 0, 1}^dim \ {0}; s ~ -s, kept with a positive first non-zero entry
  const int na = dim == 2 ? 9 : 27;
  for (int ia = 0; ia < na; ++ia)
    for (int ib = 0; ib < na; ++ib) {
      int a[3], b[3];
      bool az = true, bz = true;
      for (int i = 0, ra = ia, rb = ib; i < dim; ++i, ra /= 3, rb /= 3) {
        a[dim - 1 - i] = ra % 3 - 1;
        b[dim - 1 - i] = rb % 3 - 1;
      }
      for (int i = 0; i < dim; ++i) {
        az = az && a[i] == 0;
        bz = bz && b[i] == 0;
      }
      if (az || bz) continue;
      int s[9];
      int sign = 0;
      for (int i = 0; i < dim; ++i)
        for (int j = 0; j < dim; ++j) {
          s[i * dim + j] = a[i] * b[j];
          if (!sign && s[i * dim + j]) sign = s[i * dim + j];
        }
      for (int c = 0; c < dd; ++c) s[c] *= sign;
      bool dup = false;
      for (int m = 0; m < count && !dup; ++m) dup = std::memcmp(steps + m * dd, s, sizeof(int) * dd) == 0;
      if (!dup) {
        std::memcpy(steps + count * dd, s, sizeof(int) * dd);
        ++count;
      }
    }
  *n_dir = count;
  return R1_OK;
}

r1_status r1_grid_energy(r1_handle h, const r1_material* mat, const r1_grid* grid, double beta_n, r1_dtype dtype,
                         void* W, void* P, void* A, void* stream) {
  if (!h || !W) return R1_EINVAL;
  r1_status s = r1h::check_material(mat);
  if (s) return s;
  GridArgs g;
  s = grid_args(grid, &g);
  if (s) return s;
  if (mat->dim != grid->dim || !std::isfinite(beta_n) || (dtype != R1_F32 && dtype != R1_F64)) return R1_EINVAL;
  hipError_t e = hipSetDevice(h->device);
  if (e != hipSuccess) return r1h::fail(h, e, "hipSetDevice");
  const r1d::Material m{mat->dim, mat->model, mat->mu, mat->lambda, mat->D_inf, mat->D0};
  hipStream_t st = static_cast<hipStream_t>(stream);
  const dim3 grd(blocks_of(g.size, 256));
  if (dtype == R1_F32)
    launch_energy<float>(grid->dim, grd, st, g, m, beta_n, W, P, A);
  else
    launch_energy<double>(grid->dim, grd, st, g, m, beta_n, W, P, A);
  e = hipGetLastError();
  return e == hipSuccess ? R1_OK : r1h::fail(h, e, "kernel launch");
}

r1_status r1_grid_laminate(r1_handle h, const r1_grid* grid, int32_t n_dir, const int32_t* steps, r1_dtype dtype,
                           void* W, void* P, void* A, int32_t k_max, double tol, int32_t* iterations,
                           double* decrease, void* stream) {
  if (!h || !W || !steps || n_dir < 1 || n_dir > R1_MAX_DIRS || k_max < 1 || !(tol >= 0.0)) return R1_EINVAL;
  if (dtype != R1_F32 && dtype != R1_F64) return R1_EINVAL;
  GridArgs g;
  r1_status s = grid_args(grid, &g);
  if (s) return s;
  std::vector<Step> st_list(static_cast<size_t>(n_dir));
  for (int m = 0; m < n_dir; ++m) {
    bool zero = true;
    for (int c = 0; c < 9; ++c) st_list[m].s[c] = c < g.dd ? steps[m * g.dd + c] : 0;
    for (int c = 0; c < g.dd; ++c) {
      if (st_list[m].s[c] < -kGridMaxLen || st_list[m].s[c] > kGridMaxLen) return R1_EINVAL;
      zero = zero && st_list[m].s[c] == 0;
    }
    if (zero) return R1_EINVAL;
  }
  for (int m = 0; m < n_dir; ++m) step_slabs(g, &st_list[m], 3);
  hipError_t e = hipSetDevice(h->device);
  if (e != hipSuccess) return r1h::fail(h, e, "hipSetDevice");
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (dtype == R1_F32)
    return grid_laminate_T<float>(h, g, st_list, static_cast<float*>(W), static_cast<float*>(P),
                                  static_cast<float*>(A), k_max, tol, iterations, decrease, st);
  return grid_laminate_T<double>(h, g, st_list, static_cast<double*>(W), static_cast<double*>(P),
                                 static_cast<double*>(A), k_max, tol, iterations, decrease, st);
}

r1_status r1_grid_interpolate(r1_handle h, const r1_grid* grid, r1_dtype dtype, const void* W, int64_t n,
                              const void* F, void* out, void* stream) {
  if (!h) return R1_EINVAL;
  GridArgs g;
  r1_status s = grid_args(grid, &g);
  if (s) return s;
  if (n < 0 || n > (int64_t(1) << 31) || (dtype != R1_F32 && dtype != R1_F64)) return R1_EINVAL;
  if (n == 0) return R1_OK;
  if (!W || !F || !out) return R1_EINVAL;
  hipError_t e = hipSetDevice(h->device);
  if (e != hipSuccess) return r1h::fail(h, e, "hipSetDevice");
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (dtype == R1_F32)
    launch_interp<float>(grid->dim, g, W, n, F, out, st);
  else
    launch_interp<double>(grid->dim, g, W, n, F, out, st);
  e = hipGetLastError();
  return e == hipSuccess ? R1_OK : r1h::fail(h, e, "kernel launch");
}

}  // extern "C"
