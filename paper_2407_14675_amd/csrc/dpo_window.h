// The one-cell nodes' thrust evaluation and the window of the angle table that
// can hold its minimum (host and device).
#pragma once

#include <cmath>

#include "dpo_order.h"

// Root and reciprocal of the window's rule, which allows for a relative error of
// 2e-7 in either; a host build brings its own.
#ifndef DPO_SQRT
#define DPO_SQRT(x) __builtin_amdgcn_sqrtf(x)
#define DPO_RCP(x) __builtin_amdgcn_rcpf(x)
#endif

namespace dpo {

struct CellNode {
  float g1, g2, d1, d2;
  float x, y, z, w;  // Q = x + y dv + z dt + w dv dt
};

DPO_HOST_DEVICE inline float cell_q(const CellNode& F, float sn, float cs) {
  const float ov = fmaf(F.g1, sn, F.d1), ot = fmaf(F.g2, cs, F.d2);
  const float dv = ov - F.d1, dt = ot - F.d2;
  return fmaf(fmaf(F.w, dt, F.y), dv, fmaf(F.z, dt, F.x));
}

// The part of the table that can hold its minimum.  On one cell Q(u) = x +
// b sin u + c cos u + d sin u cos u with b = y g1, c = z g2, d = w g1 g2, so
// every tabulated Q is x - R cos(u - u*) up to E = |d|/2 plus the rounding of
// the evaluation, R = hypot(b, c), u* = atan2(b, c) + pi.  The sample nearest
// to u* lies within pi/K of it, so a sample farther than theta,
//     1 - cos(theta) = 1 - cos(pi/K) + 2 E / R,
// is above that one and cannot be the first minimum; the samples within theta are
// evaluated exactly as the full scan evaluates them.  The number of samples
// is at most kWindow, else 0 (the caller scans the whole table): nodes with R = 0,
// non-finite or huge coefficients, and those so flat that the rounding of Q
// hides the minimum.
constexpr int kWindow = 24;

DPO_HOST_DEVICE inline int scan_window(const CellNode& F, int entries, float scan_y0, float scan_k, int& k0) {
  k0 = 0;
  // all coefficients zero (a plateau): every sample has the same Q
  if (F.y == 0.0f && F.z == 0.0f && F.w == 0.0f) return 1;
  const float g1 = fabsf(F.g1), g2 = fabsf(F.g2);
  const float b = F.y * F.g1, c = F.z * F.g2;
  const float P = fmaf(fabsf(F.w), g2, fabsf(F.y)), Q = fmaf(fabsf(F.w), g1, fabsf(F.z));
  // the largest |Q|; its unit in the last place bounds the half-units of the two
  // outer operations, the foot's displacements are half a unit of drift and thrust off each
  const float top = fmaf(P, g1, fmaf(Q, g2, fabsf(F.x)));
  const float ulp = __builtin_bit_cast(float, __builtin_bit_cast(int, top) & 0x7f800000) * 1.1920929e-7f;
  const float E = 1.05f * fmaf(0.5f * fabsf(F.w) * g1, g2,
                               fmaf(5.9604645e-8f, fmaf(P, fmaf(6.0f, g1, fabsf(F.d1)), Q * fmaf(6.0f, g2, fabsf(F.d2))), ulp));
  // the approximate root and reciprocals below are within 2e-7 of the exact ones, the
  // table steps' margin of 0.02 and the 5 % on the rounding bound cover them
  const float R = DPO_SQRT(fmaf(b, b, c * c));
  // 1 - cos(theta) = 2 s^2 with s = sin(theta / 2); asin(s) <= s + (pi/2 - 1) s^3 on [0, 1]
  const float h = fmaf(E, DPO_RCP(R), 0.5f * scan_y0);
  if (!(R > 1e-18f && R < 1e18f && h <= 1.0f)) return 0;
  const float s = DPO_SQRT(h);
  const float wid = fmaf(2.0f * scan_k, s * fmaf(0.5708f, h, 1.0f), 0.02f);
  // atan2(b, c) by Abramowitz and Stegun 4.4.49 (error below 1e-5 rad), in table steps:
  // u* is entry K (atan2(b, c) / (2 pi)) mod K
  const float ab = fabsf(b), ac = fabsf(c);
  const float t = fminf(ab, ac) * DPO_RCP(fmaxf(ab, ac)), t2 = t * t;
  float at = t * fmaf(t2, fmaf(t2, fmaf(t2, fmaf(t2, 0.0208351f, -0.0851330f), 0.1801410f), -0.3302995f), 0.9998660f);
  at = ab > ac ? 1.5707964f - at : at;
  at = c < 0.0f ? 3.1415927f - at : at;
  at = b < 0.0f ? -at : at;
  const float kc = at * scan_k;
  const float lo = ceilf(kc - wid);
  const int n = (int)(floorf(kc + wid) - lo) + 1;
  if (n > kWindow || n > entries) return 0;
  int k = (int)lo;
  k = k < 0 ? k + entries : k;
  k0 = k >= entries ? k - entries : k;
  return n;
}

// Constants of scan_window for a table of K angles, the first rounded up.
inline float scan_y0_for(int K) { return std::nextafterf((float)(1.0 - std::cos(3.14159265358979323846 / K)), 4.0f); }
inline float scan_k_for(int K) { return (float)(K / (2.0 * 3.14159265358979323846)); }

// The first minimum of the n table entries from k on, in table order also
// where they wrap around the table's end; at(k): an entry's sin and cos.
template <class At>
DPO_HOST_DEVICE inline void scan_entries(const CellNode& F, int entries, const At& at, int k, int n, float& bq, int& bk) {
  bq = INFINITY;
  bk = 0;
  for (int i = 0; i < n; i++) {
    const auto sc = at(k);
    const float q = cell_q(F, sc.x, sc.y);
    if (q < bq || (q == bq && k < bk)) {
      bq = q;
      bk = k;
    }
    k = k + 1 == entries ? 0 : k + 1;
  }
}

}  // namespace dpo
