// Device-side search machinery shared by the single-problem and the batched
// sweep kernels: node terms from the per-axis tables, the tabulated scan,
// the golden section, the seeded local search, the foot descriptors of the
// chosen control, and the factorised thrust evaluation.
//
// Paper: arXiv 2407.14675, Section 3 (eq:schema; minimisation by tabulation
// and golden-section refinement).
#pragma once

#include <type_traits>

#include "dpo_kernels.h"
#include "dpo_window.h"

namespace dpo {

// Node terms from the packed coordinates of a free node and the per-axis
// tables: FP64 for the control-independent drift, float for the rest.
// Node coordinates are formed as lo + i*h with the product rounded before the
// sum (no fused multiply-add), the plain definition of the grid: a node whose
// coordinate is exactly zero (the middle v_r node of an odd grid) then gets
// exactly zero, and its feet on a face stay on the face.
//
// The r displacement dt*v_r/h_r (cells) of nodes in v_r row i1.
__device__ inline float drift_r(const SweepArgs& a, int i1) {
#pragma clang fp contract(off)
  if (a.P.model == 1) return 0.0f;
  const double vr = a.G.lo[1] + (double)i1 * a.G.h[1];
  return (float)(a.c0 * vr);
}

// Node terms of the node whose grid coordinates are already in T.i, by the
// formulas (what the context's tables are filled with).
__device__ inline void node_terms_calc(const SweepArgs& a, const float* g1tab, const float* g2tab, NodeTerms& T) {
#pragma clang fp contract(off)
  T.drift[3] = 0.0f;
  if (a.P.model != 1) {
    const double ri = a.rinv[T.i[0]];
    const double vr = a.G.lo[1] + (double)T.i[1] * a.G.h[1];
    const double vt = a.G.lo[2] + (double)T.i[2] * a.G.h[2];
    T.drift[0] = drift_r(a, T.i[1]);
    T.drift[1] = (float)(a.c1 * (vt * vt * ri - a.P.mu * ri * ri));
    T.drift[2] = (float)(-a.c2 * vr * vt * ri);
    // crown: theta' = v_t / r along axis 3
    if (a.P.model == 2) T.drift[3] = (float)(a.c3 * vt * ri);
  } else {
    T.drift[0] = T.drift[1] = T.drift[2] = 0.0f;
  }
  T.g1 = g1tab[T.i[3]];
  T.g2 = g2tab[T.i[3]];
  T.gm = a.gm;
}

// The same from the context's tables: every term depends on one or two of the
// coordinates only (the drift along v_t is one FP64 product of two of them),
// so a node reads a few cached entries instead of some twenty FP64 operations.
// m: the node's mass plane's row, for feet_cells.
__device__ inline void node_terms_at(const SweepArgs& a, NodeTerms& T, float4& m) {
#pragma clang fp contract(off)
  T.drift[0] = a.drift0[T.i[1]];
  T.drift[1] = a.drift1[__umul24(T.i[2], a.G.n[0]) + T.i[0]];
  T.drift[2] = (float)(a.drift2[__umul24(T.i[2], a.G.n[1]) + T.i[1]] * a.rinv[T.i[0]]);
  T.drift[3] = a.drift3 ? a.drift3[__umul24(T.i[2], a.G.n[0]) + T.i[0]] : 0.0f;
  m = a.mrow[T.i[3]];
  T.g1 = m.x;
  T.g2 = m.y;
  T.gm = a.gm;
}

__device__ inline void node_terms_at(const SweepArgs& a, NodeTerms& T) {
  float4 m;
  node_terms_at(a, T, m);
}

__device__ inline int node_terms_tab(const SweepArgs& a, uint32_t packed, NodeTerms& T, float4& m) {
  const int j = unpack_node(a.G, packed, T.i);
  node_terms_at(a, T, m);
  return j;
}
__device__ inline int node_terms_tab(const SweepArgs& a, uint32_t packed, NodeTerms& T) {
  float4 m;
  return node_terms_tab(a, packed, T, m);
}

// A table that no kernel of the launch writes, read at an index all lanes
// share: through the constant address space, so that the loads are scalar
// also where the kernel has stored to memory before (the compiler must
// otherwise take any store as one that may change the table).
typedef const __attribute__((address_space(4))) float* ConstTable;
__device__ inline ConstTable const_table(const float* p) { return (ConstTable)p; }

// Golden-section refinement around the centre angle u0 (sin/cos s0, c0) on
// [u0 - half, u0 + half]: two interior points u0 -+ half*rho^3, then one new
// point per step; the best evaluated point is kept (strict <, evaluation
// order).  The new point of step k is the previous point on the kept side
// moved by L0*rho^(k+4) (L0 = 2*half), because 2*rho - 1 = rho^3 and
// rho^2 - rho^3 = rho^4; its sin/cos are formed by rotating the previous
// point's sin/cos with the per-step constants rot = (sin, cos) of
// half*rho^3, then of L0*rho^(k+4) for k = 0, 1, ...  qf(sin, cos) returns
// the thrust Q at that angle.  Offsets from u0 are tracked in float for the
// stored angle.
struct GoldenState {
  float best_q, best_d;  // best Q and its offset from u0
  float best_s, best_c;  // its sin/cos as evaluated
};

template <class QF>
__device__ inline void golden(const QF& qf, float s0, float c0, float half, int steps, const float* rot_table,
                              GoldenState& g) {
  const ConstTable rot = const_table(rot_table);
  const float rho = 0.6180339887498949f;
  const float sp = rot[0], cp = rot[1];
  // the two interior points u0 -+ half*rho^3 (rho^3 = 2 rho - 1)
  const float x0 = half * 0.2360679774997897f;
  float xN = -x0, sN = fmaf(s0, cp, -c0 * sp), cN = fmaf(c0, cp, s0 * sp);  // left point
  float xK = x0, sK = fmaf(s0, cp, c0 * sp), cK = fmaf(c0, cp, -s0 * sp);   // right point
  float fN = qf(sN, cN);
  if (fN < g.best_q) {
    g.best_q = fN;
    g.best_d = xN;
    g.best_s = sN;
    g.best_c = cN;
  }
  float fK = qf(sK, cK);
  if (fK < g.best_q) {
    g.best_q = fK;
    g.best_d = xK;
    g.best_s = sK;
    g.best_c = cK;
  }
  // K: the interior point kept from the previous step; N: the point just
  // evaluated, on the left of K when nl.  Each step keeps the lower interior
  // point (the right one unless the left is strictly lower) and places the
  // new one symmetrically, at distance 2*half*rho^(k+4) from it, by rotating
  // (sin, cos) of the kept point.  The decision is two compares and lane-mask
  // logic on the scalar unit; no value is selected for it.
  bool nl = true;
  float delta = 2.0f * half * 0.1458980337503155f;  // 2*half*rho^4
  for (int it = 0; it < steps; it++) {
    const float sd = rot[2 + 2 * it], cd = rot[3 + 2 * it];
    const bool n_lower = fN < fK, k_lower = fK < fN;
    const bool keepN = (nl & n_lower) | (!nl & !k_lower);
    const bool left = keepN == nl;  // the left point is the lower one
    const float xk = keepN ? xN : xK, sk = keepN ? sN : sK, ck = keepN ? cN : cK, fk = keepN ? fN : fK;
    const float sdd = left ? -sd : sd;
    sN = fmaf(sk, cd, ck * sdd);
    cN = fmaf(ck, cd, -sk * sdd);
    xN = xk + (left ? -delta : delta);
    delta *= rho;
    xK = xk;
    sK = sk;
    cK = ck;
    fK = fk;
    nl = left;
    fN = qf(sN, cN);
    if (fN < g.best_q) {
      g.best_q = fN;
      g.best_d = xN;
      g.best_s = sN;
      g.best_c = cN;
    }
  }
}

// Exhaustive pass over the n_ang tabulated angles: first strict minimum.
// kWave: the 64 lanes of a wave search for one state together, lane l taking
// the entries l, l + 64, ...; the wave then keeps the smallest value with
// the lowest index among equal values, which is the same first strict
// minimum (entries whose Q is not below +inf are never taken, and with none
// taken the index is 0, as in the one-lane pass).  Every lane ends with the
// result; the caller's lanes must all be active.
// kUnroll: evaluations in flight per lane.
template <bool kWave = false, int kUnroll = 8, class QF>
__device__ inline void scan_table(const QF& qf, const SweepArgs& a, float& bq, int& bk) {
  bq = INFINITY;
  bk = 0;
  if (!kWave) {
    const ConstTable ts = const_table(a.tab_sin), tc = const_table(a.tab_cos);
#pragma unroll kUnroll
    for (int k = 0; k < a.n_ang; k++) {
      const float q = qf(ts[k], tc[k]);
      if (q < bq) {
        bq = q;
        bk = k;
      }
    }
    return;
  }
  int k_best = 0x7fffffff;
  for (int k = (int)(threadIdx.x & 63); k < a.n_ang; k += 64) {
    const float q = qf(a.tab_sin[k], a.tab_cos[k]);
    if (q < bq) {
      bq = q;
      k_best = k;
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    const float q2 = __shfl_xor(bq, o, 64);
    const int k2 = __shfl_xor(k_best, o, 64);
    if (q2 < bq || (q2 == bq && k2 < k_best)) {
      bq = q2;
      k_best = k2;
    }
  }
  bk = k_best == 0x7fffffff ? 0 : k_best;
}

// The outcome of the search at one node.
struct Choice {
  float v;       // min Q
  float ang;     // best thrust angle in [-pi, pi)
  float sn, cs;  // sin/cos of the best thrust angle as evaluated
  int thr;       // 1 = thrust
};

// Full search: scan, golden section around the best sample bk of value bq (if
// n_golden > 0), then thrust iff strictly below the coast value qc.
template <class QF>
__device__ inline void refine_search(const QF& qf, const SweepArgs& a, float bq, int bk, float qc, Choice& ch) {
  GoldenState g{bq, 0.0f, a.tab_sin[bk], a.tab_cos[bk]};
  if (a.n_golden > 0) golden(qf, a.tab_sin[bk], a.tab_cos[bk], a.half_width, a.n_golden, a.rot_scan, g);
  ch.thr = g.best_q < qc ? 1 : 0;
  ch.v = ch.thr ? g.best_q : qc;
  ch.ang = wrap_pi(a.tab_ang[bk] + g.best_d);
  ch.sn = g.best_s;
  ch.cs = g.best_c;
}

template <bool kWave = false, int kUnroll = 8, class QF>
__device__ inline void full_search(const QF& qf, const SweepArgs& a, float qc, Choice& ch) {
  float bq;
  int bk;
  scan_table<kWave, kUnroll>(qf, a, bq, bk);
  refine_search(qf, a, bq, bk, qc, ch);
}

// Tabulated search: first strict minimum over the table, coast on ties.
__device__ inline void table_choice(const SweepArgs& a, float bq, int bk, float qc, Choice& ch) {
  ch.thr = bq < qc ? 1 : 0;
  ch.v = ch.thr ? bq : qc;
  ch.ang = a.tab_ang[bk];
  ch.sn = a.tab_sin[bk];
  ch.cs = a.tab_cos[bk];
}

template <bool kWave = false, int kUnroll = 8, class QF>
__device__ inline void table_search(const QF& qf, const SweepArgs& a, float qc, Choice& ch) {
  float bq;
  int bk;
  scan_table<kWave, kUnroll>(qf, a, bq, bk);
  table_choice(a, bq, bk, qc, ch);
}

// Seeded local search: the seed angle, then a golden section with n_local - 3
// steps on [seed - w, seed + w] (n_local thrust evaluations), then coast.
// Returns true when the result differs from the node's current value by more
// than fallback_tol * max(1, |V|): the node must repeat the full search.
template <class QF>
__device__ inline bool seeded_local(const QF& qf, const SweepArgs& a, float seed, float qc, float vin, Choice& ch) {
  float s0, c0;
  sincosf(seed, &s0, &c0);
  GoldenState g{qf(s0, c0), 0.0f, s0, c0};
  golden(qf, s0, c0, a.local_half_width, a.n_local - 3, a.rot_local, g);
  ch.thr = g.best_q < qc ? 1 : 0;
  ch.v = ch.thr ? g.best_q : qc;
  ch.ang = wrap_pi(seed + g.best_d);
  ch.sn = g.best_s;
  ch.cs = g.best_c;
  return fabsf(ch.v - vin) > a.fallback_tol * fmaxf(1.0f, fabsf(vin));
}

// Table index nearest to the angle u on the circle (halves round up); 0 for
// a non-finite u.  Exact for the table's own angles, whose distance to an
// index is ~1e-6 of a step.
__device__ inline int table_index(float u, int K) {
  if (!(fabsf(u) <= 1.0e30f)) return 0;
  const float t = floorf((u + 3.14159265358979f) * ((float)K * 0.159154943091895f) + 0.5f);
  const int k = (int)(t - (float)K * floorf(t / (float)K));
  return (k >= 0 && k < K) ? k : 0;
}

// sin/cos of a stored policy angle, as the greedy step formed them: an angle
// that is one of the tabulated controls (or scan samples) takes the table's
// values, which the search evaluated it with; any other angle (golden-section
// and seeded points, formed there by rotation recurrences) takes sincosf.
__device__ inline void policy_sincos(const SweepArgs& a, float u, float& sn, float& cs) {
  if (a.n_ang > 0) {
    const int k = table_index(u, a.n_ang);
    if (a.tab_ang[k] == u) {
      sn = a.tab_sin[k];
      cs = a.tab_cos[k];
      return;
    }
  }
  sincosf(u, &sn, &cs);
}

// Walk over the tabulated angles from the previous optimum (paper Section 3,
// "Efficient computation of the minimum"): start at the table angle nearest
// to u_prev, look at both cyclic neighbours, move to the lower one if it is
// strictly below (the k-1 side when the two are equal), then keep moving the
// same way while the next angle is strictly lower (the angle just left is
// higher, so it never needs another look).  Thrust iff the walk's Q is
// strictly below the coast value.  At most K + 2 evaluations; returns their
// number.
template <class QF>
__device__ inline int walk_search(const QF& qf, const SweepArgs& a, float u_prev, float qc, Choice& ch) {
  const int K = a.n_ang;
  int k = table_index(u_prev, K);
  const int km = k == 0 ? K - 1 : k - 1, kp = k == K - 1 ? 0 : k + 1;
  float qk = qf(a.tab_sin[k], a.tab_cos[k]);
  const float qm = qf(a.tab_sin[km], a.tab_cos[km]);
  const float qp = qf(a.tab_sin[kp], a.tab_cos[kp]);
  int n = 3;
  int d = 0;
  if (qm < qk && qm <= qp) d = -1;
  else if (qp < qk) d = 1;
  if (d != 0) {
    k = d < 0 ? km : kp;
    qk = d < 0 ? qm : qp;
    for (int it = 0; it < K; it++) {
      int kn = k + d;
      kn = kn < 0 ? K - 1 : (kn >= K ? 0 : kn);
      const float qn = qf(a.tab_sin[kn], a.tab_cos[kn]);
      n++;
      if (!(qn < qk)) break;
      k = kn;
      qk = qn;
    }
  }
  ch.thr = qk < qc ? 1 : 0;
  ch.v = ch.thr ? qk : qc;
  ch.ang = a.tab_ang[k];
  ch.sn = a.tab_sin[k];
  ch.cs = a.tab_cos[k];
  return n;
}

// Adds the workgroup's sum of v to acc[blockIdx.x] (each workgroup owns its
// entry, so successive sweeps on one stream accumulate without atomics).
// Every thread of the workgroup must call it.
__device__ inline void block_add_count(int v, unsigned long long* acc) {
  __shared__ int wsum[kMaxBlock / 64];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) wsum[w] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    long long s = 0;
    for (int i = 0; i < (int)(blockDim.x >> 6); i++) s += wsum[i];
    acc[blockIdx.x] += (unsigned long long)s;
  }
}


// Seeded search with the fallback done in place.
template <int kUnroll, class QF>
__device__ inline int seeded_search(const QF& qf, const SweepArgs& a, float seed, float qc, float vin, Choice& ch) {
  if (seeded_local(qf, a, seed, qc, vin, ch)) {
    full_search<false, kUnroll>(qf, a, qc, ch);
    return 1;
  }
  return 0;
}

// Policy iteration's greedy step also evaluates the node's current control
// (pol_thr_in / pol_ang_in, read before the node's outputs are written) and
// keeps it unless the search found a strictly smaller Q.  The scan + golden
// search is only approximately the argmin; with the incumbent as a candidate
// the greedy value never exceeds the current policy's, so policy iteration
// from above decreases monotonically instead of alternating between two
// nearly tied basins.
template <class QF>
__device__ inline void keep_incumbent(const QF& qf, const SweepArgs& a, int j, float qc, Choice& ch) {
  if (!a.pol_thr_in) return;
  const int thr0 = a.pol_thr_in[j] ? 1 : 0;
  const float u0 = a.pol_ang_in[j];
  float s0 = 0.0f, c0 = 1.0f, q0 = qc;
  if (thr0) {
    policy_sincos(a, u0, s0, c0);
    q0 = qf(s0, c0);
  }
  if (q0 <= ch.v) {
    ch.v = q0;
    ch.ang = u0;
    ch.sn = s0;
    ch.cs = c0;
    ch.thr = thr0;
  }
}

// Foot descriptor of the chosen control (see SweepArgs::desc_code).
__device__ inline void write_desc(const SweepArgs& a, int t, int j, const NodeTerms& T, const Choice& ch) {
  float off[4];
  off[0] = T.drift[0];
  off[1] = ch.thr ? fmaf(T.g1, ch.sn, T.drift[1]) : T.drift[1];
  off[2] = ch.thr ? fmaf(T.g2, ch.cs, T.drift[2]) : T.drift[2];
  off[3] = T.drift[3] + (ch.thr ? T.gm : 0.0f);
  int base[4];
  float w[4];
  const bool inside = foot_cell(a.G, T.i, off, base, w);
  const float2 wv = inside ? make_float2(w[1], w[2]) : make_float2(0.0f, 0.0f);
  if (a.desc_pk) {
    uint32_t code = ch.thr ? kDescThr : 0;
    if (inside) code |= (uint32_t)((base[1] - T.i[1] + 32) | ((base[2] - T.i[2] + 32) << 6));
    else code |= kDescOut;
    a.desc_pk[j] = desc_pack(code, wv.x, wv.y);
    return;
  }
  if (a.desc16) {
    const int k = a.desc_dense ? j : t;
    uint16_t code = ch.thr ? kDescThr : 0;
    if (inside) code |= (uint16_t)((base[1] - T.i[1] + 32) | ((base[2] - T.i[2] + 32) << 6));
    else code |= kDescOut;
    a.desc16[k] = code;
    a.desc_w[k] = wv;
    return;
  }
  const unsigned flat = inside ? (unsigned)(base[0] + base[1] * a.G.st[1] + base[2] * a.G.st[2] + base[3] * a.G.st[3])
                               : (1u << 30);
  a.desc_code[t] = (int)(flat | ((unsigned)ch.thr << 31));
  a.desc_w[t] = wv;
}

// ---- fast path for thrust controls.
// Under thrust the r displacement (v_r * dt) and the m displacement (-c*dt)
// do not depend on the angle, so every thrust foot of a node shares its r and
// m cell and weights; only the v_r and v_t displacements move, by at most
// |g| < 0.5 cell around the coast foot.  The node therefore collapses its
// neighbourhood over r and m once (36 corner values, 27 lerps) into a 3 x 3
// patch over (v_r, v_t), and every thrust evaluation is the bilinear
// interpolant of the patch cell its foot falls in: the same Q1 value as the
// 16-corner sum, with the lerps reordered.  Along each of v_r, v_t the feet
// span at most two regions split at one threshold (a node or a domain face);
// a region outside the domain has the constant value M.  The four region
// pairs are stored per thread in LDS as Q = A + B dv + C dt + D dv dt in the
// displacements dv = g1 sin u, dt = g2 cos u from the coast foot.
struct Regions {
  int b0;     // first cell (node index) of region 0; region 1 is cell b0 + 1
  float bnd;  // region 1 <=> displacement offset >= bnd (node offsets)
  bool ok0, ok1;
};

__device__ inline Regions axis_regions(int i, int n, float d, float g) {
  Regions R;
  const float ag = fabsf(g) + 1e-6f;  // margin over the rounding of d + g*s
  const float lo = d - ag, hi = d + ag;
  const float top = (float)(n - 1 - i), bot = (float)(-i);
  if (hi < bot || lo > top) {  // every foot outside
    R.b0 = 0;
    R.bnd = INFINITY;
    R.ok0 = R.ok1 = false;
    return R;
  }
  const float k = floorf(hi);
  const int kk = i + (int)k;
  if (kk >= n - 1) {  // reaches the top face: last cell, then outside (the face itself is inside)
    R.b0 = n - 2;
    R.bnd = next_up(top);
    R.ok0 = true;
    R.ok1 = false;
  } else if (k > lo) {  // crosses node kk (kk == 0: the bottom face)
    R.b0 = kk - 1;
    R.bnd = k;
    R.ok0 = kk - 1 >= 0;
    R.ok1 = true;
  } else {  // one cell
    R.b0 = kk;
    R.bnd = INFINITY;
    R.ok0 = true;
    R.ok1 = false;
  }
  return R;
}

struct FastNode {
  float g1, g2;  // thrust displacement per unit sin u (v_r) and cos u (v_t), cells
  float d1, d2;  // coast displacements along v_r and v_t
  float bv, bt;  // region 1 <=> offset >= threshold (the same float test as foot_cell)
  const char* coef;  // this thread's first region pair in LDS
  int offv, offt;    // byte offsets of the region pairs with v_r region 1 / v_t region 1
};

__device__ inline float fast_q(const FastNode& F, float sn, float cs) {
  const float ov = fmaf(F.g1, sn, F.d1), ot = fmaf(F.g2, cs, F.d2);
  const int off = (ov >= F.bv ? F.offv : 0) + (ot >= F.bt ? F.offt : 0);
  const float4 c = *reinterpret_cast<const float4*>(F.coef + off);
  const float dv = ov - F.d1, dt = ot - F.d2;
  return fmaf(fmaf(c.w, dt, c.y), dv, fmaf(c.z, dt, c.x));
}

// Lerp along r of the corner pair (p[0], p[1]), fetched by one 8-byte load.
__device__ inline float lerp_pair(const float* p, float t) {
  const CornerPair v = *reinterpret_cast<const CornerPair*>(p);
  return lerp(v.lo, v.hi, t);
}

// The cells a node's thrust feet fall in.
struct FeetCells {
  bool ok_r, ok_m;    // inside along r; under thrust, along m
  bool coast_lo;      // the coast foot's plane i_m is the lower plane of the thrust feet
  int br;             // r cell, shared by every control
  uint32_t plane;     // byte offset of the thrust feet's lower mass plane (i_m outside)
  float tr, tm;       // cell coordinates along r and (thrust) m
  Regions Rv, Rt;
  // every thrust foot (and the coast foot, which lies between them) in one cell, or outside
  __device__ bool one_cell() const { return Rv.bnd == INFINITY && Rt.bnd == INFINITY; }
};

// axis_regions of a node known to have one region.
__device__ inline Regions axis_one_region(int i, int n, float d, float g) {
  const float ag = fabsf(g) + 1e-6f;
  const float lo = d - ag, hi = d + ag;
  Regions R;
  R.ok0 = !(hi < (float)(-i) || lo > (float)(n - 1 - i));
  R.ok1 = false;
  R.b0 = R.ok0 ? i + (int)floorf(hi) : 0;
  R.bnd = INFINITY;
  return R;
}

template <bool kOne>
__device__ inline void feet_cells(const SweepArgs& a, const NodeTerms& T, const float4& m, FeetCells& C) {
  const Grid& G = a.G;
  C.br = 0;
  C.tr = 0.0f;
  C.ok_r = axis_cell(T.i[0], G.n[0], T.drift[0], C.br, C.tr);
  // m cell under thrust; the coast foot stays on plane i_m
  const uint32_t w = __float_as_uint(m.w);
  C.tm = m.z;
  C.plane = w & ~3u;
  C.ok_m = w & 1u;
  C.coast_lo = w & 2u;
  C.Rv = kOne ? axis_one_region(T.i[1], G.n[1], T.drift[1], T.g1) : axis_regions(T.i[1], G.n[1], T.drift[1], T.g1);
  C.Rt = kOne ? axis_one_region(T.i[2], G.n[2], T.drift[2], T.g2) : axis_regions(T.i[2], G.n[2], T.drift[2], T.g2);
}

// A corner pair at a byte offset from V (below 2^32: at most 2^30 nodes), so
// that the load takes a scalar base and one 32-bit offset.
__device__ inline CornerPair pair_at(const float* __restrict__ V, uint32_t byte_off) {
  return *reinterpret_cast<const CornerPair*>(reinterpret_cast<const char*>(V) + byte_off);
}

// Per-node set-up of the thrust evaluations; returns the coast Q, which is
// the same Q1 value read from the patch (plane i_m, coast cell).
// lds: 4 * blockDim.x float4, laid out [region pair][thread].
__device__ inline float fast_setup(const SweepArgs& a, const NodeTerms& T, const FeetCells& C, float4* lds, FastNode& F) {
  const Grid& G = a.G;
  F.g1 = T.g1;
  F.g2 = T.g2;
  F.d1 = T.drift[1];
  F.d2 = T.drift[2];
  F.offv = 2 * (int)blockDim.x * (int)sizeof(float4);
  F.offt = (int)blockDim.x * (int)sizeof(float4);
  F.coef = reinterpret_cast<const char*>(lds + threadIdx.x);
  const bool ok_r = C.ok_r, ok_m = C.ok_m;
  const float tr = C.tr, tm = C.tm;
  const Regions& Rv = C.Rv;
  const Regions& Rt = C.Rt;
  F.bv = Rv.bnd;
  F.bt = Rt.bnd;
  const float qM = fmaf(a.P.gamma, a.P.M, a.P.q_thr);
  float W[3][3], Wc[3][3];
  if (ok_r) {
    const uint32_t base = C.plane + 4u * (uint32_t)C.br, so = ok_m ? 4u * (uint32_t)G.st[3] : 0u;
#pragma unroll
    for (int p = 0; p < 3; p++) {
      const uint32_t v = base + __umul24(min(max(Rv.b0 + p, 0), G.n[1] - 1), 4 * G.st[1]);
      // the row's six corner pairs are loaded before any of them is used,
      // so that their latencies overlap
      CornerPair lo[3], hi[3];
#pragma unroll
      for (int q = 0; q < 3; q++) {
        const uint32_t o = v + __umul24(min(max(Rt.b0 + q, 0), G.n[2] - 1), 4 * G.st[2]);
        lo[q] = pair_at(a.V_in, o);
        hi[q] = pair_at(a.V_in, o + so);
      }
#pragma unroll
      for (int q = 0; q < 3; q++) {
        const float l = lerp(lo[q].lo, lo[q].hi, tr), h = lerp(hi[q].lo, hi[q].hi, tr);
        W[p][q] = lerp(l, h, tm);
        Wc[p][q] = C.coast_lo ? l : h;
      }
    }
  }
  const float gam = a.P.gamma, q0 = a.P.q_thr;
#pragma unroll
  for (int av = 0; av < 2; av++) {
#pragma unroll
    for (int bt = 0; bt < 2; bt++) {
      float4 c = make_float4(qM, 0.0f, 0.0f, 0.0f);
      const bool valid = ok_r && ok_m && (av ? Rv.ok1 : Rv.ok0) && (bt ? Rt.ok1 : Rt.ok0);
      if (valid) {
        const float w00 = W[av][bt], w10 = W[av + 1][bt], w01 = W[av][bt + 1], w11 = W[av + 1][bt + 1];
        // local coordinates of the coast foot in this cell
        const float tv = T.drift[1] - (float)(Rv.b0 + av - T.i[1]);
        const float tt = T.drift[2] - (float)(Rt.b0 + bt - T.i[2]);
        const float cv = w10 - w00, ct = w01 - w00, dd = (w11 - w10) - (w01 - w00);
        const float A = lerp(lerp(w00, w10, tv), lerp(w01, w11, tv), tt);
        c.x = fmaf(gam, A, q0);
        c.y = gam * fmaf(dd, tt, cv);
        c.z = gam * fmaf(dd, tv, ct);
        c.w = gam * dd;
      }
      lds[(av * 2 + bt) * blockDim.x + threadIdx.x] = c;
    }
  }
  // coast: the cell of (d1, d2) on plane i_m, by the same region tests
  const int av = T.drift[1] >= Rv.bnd ? 1 : 0;
  const int bt = T.drift[2] >= Rt.bnd ? 1 : 0;
  const bool cvalid = ok_r && (av ? Rv.ok1 : Rv.ok0) && (bt ? Rt.ok1 : Rt.ok0);
  float Ic = a.P.M;
  if (cvalid) {
    const float tv = T.drift[1] - (float)(Rv.b0 + av - T.i[1]);
    const float tt = T.drift[2] - (float)(Rt.b0 + bt - T.i[2]);
    float w00, w10, w01, w11;
    // select the coast cell of the 3 x 3 patch (av, bt in {0, 1})
    w00 = av ? (bt ? Wc[1][1] : Wc[1][0]) : (bt ? Wc[0][1] : Wc[0][0]);
    w10 = av ? (bt ? Wc[2][1] : Wc[2][0]) : (bt ? Wc[1][1] : Wc[1][0]);
    w01 = av ? (bt ? Wc[1][2] : Wc[1][1]) : (bt ? Wc[0][2] : Wc[0][1]);
    w11 = av ? (bt ? Wc[2][2] : Wc[2][1]) : (bt ? Wc[1][2] : Wc[1][1]);
    Ic = lerp(lerp(w00, w10, tv), lerp(w01, w11, tv), tt);
  }
  return fmaf(a.P.gamma, Ic, a.P.q_coast);
}


// ---- nodes whose thrust feet all fall in one cell (one region along v_r and
// one along v_t): 92 % of the nodes of the 96^3 x 64 problem, 88 % of 48^4, 82 to 99 %
// of the sixteen batched problems.  The four coefficients of the bilinear form stay in
// registers (CellNode), 8 corner pairs are gathered instead of 18, and an evaluation is
// 7 instructions with no region test and no LDS read.
//
// Set-up of such a node: the operations of fast_setup on its one region pair,
// in the same order, so the values are the same bit for bit.  Returns the
// coast Q.
__device__ inline float cell_setup(const SweepArgs& a, const NodeTerms& T, const FeetCells& C, CellNode& F) {
  const Grid& G = a.G;
  F.g1 = T.g1;
  F.g2 = T.g2;
  F.d1 = T.drift[1];
  F.d2 = T.drift[2];
  F.x = fmaf(a.P.gamma, a.P.M, a.P.q_thr);
  F.y = F.z = F.w = 0.0f;
  float Ic = a.P.M;
  if (C.ok_r && C.Rv.ok0 && C.Rt.ok0) {
    const uint32_t s1 = 4u * (uint32_t)G.st[1], s2 = 4u * (uint32_t)G.st[2], so = C.ok_m ? 4u * (uint32_t)G.st[3] : 0u;
    const uint32_t p = C.plane + __umul24(__umul24(C.Rt.b0, G.n[1]) + C.Rv.b0, s1) + 4u * (uint32_t)C.br;
    CornerPair lo[4], hi[4];
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const uint32_t o = p + ((e & 1) ? s1 : 0u) + ((e & 2) ? s2 : 0u);
      lo[e] = pair_at(a.V_in, o);
      hi[e] = pair_at(a.V_in, o + so);
    }
    float W[4], Wc[4];
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const float l = lerp(lo[e].lo, lo[e].hi, C.tr), h = lerp(hi[e].lo, hi[e].hi, C.tr);
      W[e] = lerp(l, h, C.tm);
      Wc[e] = C.coast_lo ? l : h;
    }
    // local coordinates of the coast foot in the cell
    const float tv = T.drift[1] - (float)(C.Rv.b0 - T.i[1]);
    const float tt = T.drift[2] - (float)(C.Rt.b0 - T.i[2]);
    if (C.ok_m) {
      const float gam = a.P.gamma;
      const float cv = W[1] - W[0], ct = W[2] - W[0], dd = (W[3] - W[1]) - (W[2] - W[0]);
      const float A = lerp(lerp(W[0], W[1], tv), lerp(W[2], W[3], tv), tt);
      F.x = fmaf(gam, A, a.P.q_thr);
      F.y = gam * fmaf(dd, tt, cv);
      F.z = gam * fmaf(dd, tv, ct);
      F.w = gam * dd;
    }
    Ic = lerp(lerp(Wc[0], Wc[1], tv), lerp(Wc[2], Wc[3], tv), tt);
  }
  return fmaf(a.P.gamma, Ic, a.P.q_coast);
}

// The angle table as a one-cell wave reads it, each lane at its own entry: in
// LDS, in the region pairs' place, which such a wave leaves unused (four runs
// of 64 float4, a workgroup's width apart).  Every wave fills its own, so that
// no other waits for it: a table of the whole workgroup's behind the region pairs
// held up the general waves too and took LDS in all modes (scan 64 + golden 12,
// 12^4: 15.8 us a sweep with it, 15.6 now; seeded 9.7 and 9.1).  Tables of more than
// kWaveAngles entries do not fit and are read from memory (1024 samples, 32^4: 302 us
// with the workgroup's table, 299 now).
constexpr int kWaveAngles = 512;

struct WaveAngles {
  float2* run;  // the wave's first run
  int stride;   // float2 from one run to the next
  float2 own;   // the lane's entry of the first 64, on its way from memory
  __device__ float2& at(int k) const { return run[(k >> 7) * stride + (k & 127)]; }
};

__device__ inline void load_angles(const SweepArgs& a, float4* lds, WaveAngles& W) {
  const int k = min((int)(threadIdx.x & 63), a.n_ang - 1);
  W.run = reinterpret_cast<float2*>(lds + ((int)threadIdx.x & ~63));
  W.stride = 2 * (int)blockDim.x;
  W.own = make_float2(a.tab_sin[k], a.tab_cos[k]);
}

// All lanes of the wave call it.
__device__ inline void store_angles(const SweepArgs& a, const WaveAngles& W) {
  if (a.n_ang > kWaveAngles) return;
  int k = threadIdx.x & 63;
  W.at(k) = W.own;  // entries past the table's end are not read
  for (k += 64; k < a.n_ang; k += 64) W.at(k) = make_float2(a.tab_sin[k], a.tab_cos[k]);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// scan_table for a one-cell node: the window where every active lane of the
// wave has one (lanes in step through their own windows), else the whole
// table.
__device__ inline void scan_cell(const SweepArgs& a, const CellNode& F, const WaveAngles& W, float& bq, int& bk) {
  int k;
  const int n = scan_window(F, a.n_ang, a.scan_y0, a.scan_k, k);
  if (!__all(n > 0)) scan_table([&](float sn, float cs) { return cell_q(F, sn, cs); }, a, bq, bk);
  else if (a.n_ang <= kWaveAngles) scan_entries(F, a.n_ang, [&](int e) { return W.at(e); }, k, n, bq, bk);
  else scan_entries(F, a.n_ang, [&](int e) { return make_float2(a.tab_sin[e], a.tab_cos[e]); }, k, n, bq, bk);
}

// write_desc for a one-cell node: the cell of every foot is known, and its
// coordinates are the offsets from it (what axis_cell forms).
__device__ inline void write_desc_cell(const SweepArgs& a, int t, int j, const NodeTerms& T, const FeetCells& C,
                                       const Choice& ch) {
  if (!a.desc_pk && !a.desc16) {
    write_desc(a, t, j, T, ch);
    return;
  }
  const bool inside = C.ok_r && C.Rv.ok0 && C.Rt.ok0 && (!ch.thr || C.ok_m);
  const float o1 = ch.thr ? fmaf(T.g1, ch.sn, T.drift[1]) : T.drift[1];
  const float o2 = ch.thr ? fmaf(T.g2, ch.cs, T.drift[2]) : T.drift[2];
  const int k1 = C.Rv.b0 - T.i[1], k2 = C.Rt.b0 - T.i[2];
  const float w1 = inside ? o1 - (float)k1 : 0.0f, w2 = inside ? o2 - (float)k2 : 0.0f;
  const uint32_t code = (ch.thr ? kDescThr : 0u) | (inside ? (uint32_t)((k1 + 32) | ((k2 + 32) << 6)) : kDescOut);
  if (a.desc_pk) {
    a.desc_pk[j] = desc_pack(code, w1, w2);
    return;
  }
  const int k = a.desc_dense ? j : t;
  a.desc16[k] = (uint16_t)code;
  a.desc_w[k] = make_float2(w1, w2);
}

// Sums of a thread over its nodes: residual contributions, seeded fallbacks,
// thrust evaluations of the table walk.
struct NodeSums {
  double rel = 0, sum = 0, mabs = 0, bad = 0;
  int fell_back = 0, evals = 0;
};

// The sweep's arguments where they lie in constant memory (the kernel's
// argument block, or a record of the batched sweep).
typedef const __attribute__((address_space(4))) SweepArgs* ConstArgs;

// The same address, of which the compiler knows nothing: what is read through
// it is loaded there and not ahead of it.
__device__ inline ConstArgs anew(ConstArgs p) {
  asm volatile("" : "+s"(p));
  return p;
}

// Brings the cache lines of the arguments in, all at once: read piece by piece
// later, each would be a trip to memory of its own.
__device__ inline void touch_args(ConstArgs p) {
  static_assert(sizeof(SweepArgs) > 9 * 64 && sizeof(SweepArgs) <= 10 * 64, "one word of every 64 bytes");
  const auto* w = (const __attribute__((address_space(4))) int*)p;
  asm volatile("" ::"s"(w[0]), "s"(w[16]), "s"(w[32]), "s"(w[48]), "s"(w[64]), "s"(w[80]), "s"(w[96]), "s"(w[112]),
               "s"(w[128]), "s"(w[144]));
}

// The arguments through p, each loaded where it is first used.  The pointers
// are read one by one through the constant address space: only such a load is
// known to give global memory (a pointer copied as part of the struct, or cast to global
// memory and back, is accessed by flat instructions).  kBatch: without what
// a batched sweep does not have.
template <bool kBatch>
__device__ inline SweepArgs sweep_args(ConstArgs p) {
  SweepArgs a = *(const SweepArgs*)p;
  a.V_in = p->V_in;
  a.V_out = p->V_out;
  a.pol_ang = p->pol_ang;
  a.pol_thr = p->pol_thr;
  a.sweep_node = p->sweep_node;
  a.sweep_pos = p->sweep_pos;
  a.one_cell = p->one_cell;
  a.rinv = p->rinv;
  a.drift0 = p->drift0;
  a.drift1 = p->drift1;
  a.drift2 = p->drift2;
  a.drift3 = nullptr;  // the crown problem takes the direct path
  a.mrow = p->mrow;
  a.tab_sin = p->tab_sin;
  a.tab_cos = p->tab_cos;
  a.tab_ang = p->tab_ang;
  a.rot_scan = p->rot_scan;
  a.rot_local = p->rot_local;
  a.seed = kBatch ? nullptr : p->seed;
  a.walk_from = kBatch ? nullptr : p->walk_from;
  a.pol_ang_in = kBatch ? nullptr : p->pol_ang_in;
  a.pol_thr_in = kBatch ? nullptr : p->pol_thr_in;
  a.desc_code = kBatch ? nullptr : p->desc_code;
  a.desc16 = kBatch ? nullptr : p->desc16;
  a.desc_pk = kBatch ? nullptr : p->desc_pk;
  a.desc_w = kBatch ? nullptr : p->desc_w;
  return a;
}

// Search of one node with its set-up done: the choice in ch.  kMode: 0
// tabulated, 1 scan + golden, 2 seeded, 3 table walk.  scan(bq, bk): the
// table's first minimum.
template <int kMode, class QF, class Scan>
__device__ inline void search_node(const QF& qf, const Scan& scan, const SweepArgs& a, int j, float qc, float vin,
                                   Choice& ch, NodeSums& S) {
  float bq;
  int bk;
  if (kMode == 0) {
    scan(bq, bk);
    table_choice(a, bq, bk, qc, ch);
  } else if (kMode == 1) {
    scan(bq, bk);
    refine_search(qf, a, bq, bk, qc, ch);
  } else if (kMode == 3) {
    S.evals += walk_search(qf, a, a.walk_from[j], qc, ch);
  } else {
    // The full search of a lane that falls back holds up its wave.  Listing
    // such nodes for a second launch was dearer at every size and share of them
    // measured: the set-up is formed twice, there in mixed waves, while here it
    // stands in registers and a one-cell wave's scan is short (96^3 x 64, 19 % of
    // the nodes: 2.40 ms then, 1.33 now, with hardly any 1.38 and 1.02; 64 x 60 x 56
    // x 48: 0.32 and 0.22; 10 x 27 x 12 x 10: 42 us and 16).
    if (seeded_local(qf, a, a.seed[j], qc, vin, ch)) {
      S.fell_back++;
      scan(bq, bk);
      refine_search(qf, a, bq, bk, qc, ch);
    }
  }
}

// Outputs of a node whose choice is made, and its residual contribution.
// policy: whether anyone reads this sweep's policy.
__device__ inline void store_node(const SweepArgs& a, int j, float vin, const Choice& ch, bool policy, bool resid,
                                  NodeSums& S) {
  a.V_out[j] = ch.v;
  if (a.pol_ang && policy) a.pol_ang[j] = ch.ang;
  if (a.pol_thr && policy) a.pol_thr[j] = (uint8_t)ch.thr;
  if (resid) node_residual(vin, ch.v, S.rel, S.sum, S.mabs, S.bad);
}

// One free node of a sweep on the factorised path.  kOne: its thrust feet
// share one cell.  live: not a lane beyond the list's end.  lds: 4 * blockDim.x
// float4 (general form: the region pairs; one-cell form: the wave's angles).
// The arguments of the set-up, the search and the outputs are loaded each at
// its place: both forms' together do not fit the scalar registers (23-49 of them
// were spilled to lanes of vector registers, stored one by one ahead of every node;
// 12^4, scan 64 + golden 12: 15.5 -> 14.7 us a sweep, 17 controls 9.3 -> 8.8; 96^3 x
// 64: 1646 -> 1596).  The row of the mass plane is read once, with the other terms
// of the node: read again for the feet's cells it was a trip to memory of its own.
template <int kMode, bool kOne, bool kBatch>
__device__ inline void fast_node(ConstArgs p, int t, bool live, uint32_t packed, float4* lds, bool resid, NodeSums& S) {
  const SweepArgs a = sweep_args<kBatch>(anew(p));
  NodeTerms T;
  float4 m;
  const int j = node_terms_tab(a, packed, T, m);
  // the table search evaluates every entry: its window costs more than it saves with 16
  // angles (32^4: 24.9 us without, 27.5 with) and gains little with 72 (38.4, 38.5;
  // 96^3 x 64: 1426, 1349)
  constexpr bool kAngles = kOne && (kMode == 1 || kMode == 2);
  WaveAngles W;
  if constexpr (kAngles) load_angles(a, lds, W);
  FeetCells C;
  feet_cells<kOne>(a, T, m, C);
  typename std::conditional<kOne, CellNode, FastNode>::type F;
  float qc;
  if constexpr (kOne) qc = cell_setup(a, T, C, F);
  else qc = fast_setup(a, T, C, lds, F);
  auto qf = [&](float sn, float cs) {
    if constexpr (kOne) return cell_q(F, sn, cs);
    else return fast_q(F, sn, cs);
  };
  const float vin = a.V_in[j];
  const SweepArgs b = sweep_args<kBatch>(anew(p));
  if constexpr (kAngles) store_angles(b, W);
  auto scan = [&](float& bq, int& bk) {
    if constexpr (kAngles) scan_cell(b, F, W, bq, bk);
    else scan_table(qf, b, bq, bk);
  };
  Choice ch;
  search_node<kMode>(qf, scan, b, j, qc, vin, ch, S);
  if (!live) {
    S = NodeSums();
    return;
  }
  const SweepArgs c = sweep_args<kBatch>(anew(p));
  keep_incumbent(qf, c, j, qc, ch);
  if (c.desc_code || c.desc16 || c.desc_pk) {
    // formats by free-list position: the node's place in node order
    const int at = c.desc_pk ? 0 : (t & ~(kOrderChunk - 1)) + c.sweep_pos[t];
    if (kOne) write_desc_cell(c, at, j, T, C, ch);
    else write_desc(c, at, j, T, ch);
  }
  // a batch may stop after the sweeps that feed its stop decision only: the others'
  // policies are overwritten unread, 5 bytes a node to memory that the batch's values
  // do not leave in the caches (16 problems of 24 to 64 nodes a side: 2.54 s with them,
  // 2.26 without, 2.36 one after another)
  store_node(c, j, vin, ch, !kBatch || resid, resid, S);
}

// A workgroup's nodes, one per thread.  A wave whose nodes are all one-cell
// nodes (sweep_node keeps the two kinds apart, see k_order_free) takes the
// short form, any other the general one.  Vector instruction issue bounds the
// sweep with many controls (96^3 x 64, coast + scan 64 + golden 12, value
// iteration: 1.99 -> 1.37 ms a sweep with the two forms, the scan's window and
// the tables of the node terms; 2007 -> 1458 vector instructions per wave),
// and the latency of its loads the one with few (40^4, 17 controls: 58 -> 45 us).
// Splitting the nodes inside the kernel instead (listing the others in LDS, per
// workgroup or per wave, and running them together) took 1.96-2.8 ms: the second
// phase leaves lanes and waves idle.
template <int kMode, bool kBatch>
__device__ inline void sweep_nodes(ConstArgs p, int tile, float4* lds, bool resid, NodeSums& S) {
  const SweepArgs a = sweep_args<kBatch>(p);
  touch_args(p);
  const int bd = (int)blockDim.x, tid = (int)threadIdx.x;
  const int first = __builtin_amdgcn_readfirstlane(tile * bd + (tid & ~63));
  const int t = first + (tid & 63);
  if (first >= a.n_free) return;
  // the node and the kind of its wave are loaded together: a sweep of few
  // controls waits on memory, not on arithmetic.  Lanes beyond the list's end
  // go with its last node and store nothing.
  const bool live = t < a.n_free;
  const uint32_t packed = a.sweep_node[live ? t : a.n_free - 1];
  typedef const __attribute__((address_space(4))) unsigned long long* ConstBits;
  const bool one = (((ConstBits)a.one_cell)[first / kOrderChunk] >> ((first / 64) & 63)) & 1;
  if (one) fast_node<kMode, true, kBatch>(p, t, live, packed, lds, resid, S);
  else fast_node<kMode, false, kBatch>(p, t, live, packed, lds, resid, S);
}

// Dynamic LDS of sweep_nodes.
inline size_t sweep_lds_bytes(int block) { return sizeof(float4) * 4 * (size_t)block; }

}  // namespace dpo
