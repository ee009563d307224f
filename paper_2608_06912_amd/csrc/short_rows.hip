// Forward of short rows (n <= kRowWaveMax), one wave per row, four rows per
// workgroup: the row in registers, LapSum evaluated at points x until no
// score is left strictly between the two tightest ones (from about the
// budget's quantile; Newton steps, longer while the root stays on one side,
// kept inside the ends; where the temperature is too small for them, between
// the ends in proportion to LapSum), the sums of both
// sides then taken relative to the nearest score on each side and the gap
// solved in closed form; p from the registers.  No LDS and no barriers: the
// bucketed row kernel spends about 8 us of a workgroup clearing and scanning
// 2048 buckets whatever the row's length, two workgroups to a CU.
//
// Bound: vector issue, about 200 instructions per point and wave at four
// scores per lane (half of them the float64 sums over the wave) and five to
// eight points.  4096 rows of 256 scores (k = 8, t = 1): 140 -> 18 us.  At
// t = 0.02 the start and the proportional points took 256 rows of 256 with
// k = 0.26 from 24.5 to 15.2 us (backward included, bisection before).  Rows
// with a sentinel among the scores (-3.4e38, -1e9) take 8-15 points; without
// the middles of the keys 25-40 (4096 rows of 200, 30% masked, forward, us:
// 49-82, with them 25-33, plain rows 20; the 2048 buckets 120-170).
#include <math.h>

#include "kernels.hpp"
#include "narrow.hpp"

namespace lapsum {

namespace {
constexpr int RT = 256;
constexpr int RW = RT / kWave;   // rows per workgroup
}  // namespace

// Lane l holds scores l, l + 64, ...
template <int ITEMS>
__global__ __launch_bounds__(RT) void row_wave_forward_kernel(const float* __restrict__ scores,
                                                              int64_t batch, int n, double k,
                                                              double t, float cut,
                                                              float* __restrict__ probs,
                                                              double* __restrict__ b_out) {
  const int lane = lane_id();
  const int64_t row = static_cast<int64_t>(blockIdx.x) * RW + threadIdx.x / kWave;
  if (row >= batch) return;   // (whole waves; no barrier below)
  const float* r = scores + row * n;
  const double c2 = kLog2e / t;
  float v[ITEMS];
  float mn = INFINITY, mx = -INFINITY;
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const int at = i * kWave + lane;
    v[i] = r[at < n ? at : 0];
  }
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    mn = fminf(mn, v[i]);
    mx = fmaxf(mx, v[i]);
    // past the row: no score (every comparison is false, every term is 0)
    if (i * kWave + lane >= n) v[i] = __int_as_float(0x7fc00000);
  }
  mn = wave_min(mn, INFINITY);
  mx = wave_max(mx, -INFINITY);
  float lo = -INFINITY, hi = INFINITY;
  // from about the quantile of the budget's share in a bell-shaped row
  float x = mx - (mx - mn) * cut;
  if (!(x > mn && x < mx)) x = 0.5f * mn + 0.5f * mx;
  double flo = n, fhi = 0.0;   // LapSum at the ends (about, until they are points)
  int same = 0, last = 0;
  uint32_t left = static_cast<uint32_t>(n);
  uint32_t stuck = 0u;   // points in a row that left nearly every score between the ends
  for (int it = 0; it < 96; ++it) {
    const double xd = x;
    double P = 0.0, E = 0.0;
    uint32_t c = 0u, na = 0u, ng = 0u;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      const bool up = v[i] >= x, dn = v[i] < x;
      const double e = exp2_neg(-fabs(static_cast<double>(v[i]) - xd) * c2);
      P = fma(e, up ? 1.0 : 0.0, P);
      E = fma(e, dn ? 1.0 : 0.0, E);
      c += static_cast<uint32_t>(__popcll(__ballot(up)));
      na += static_cast<uint32_t>(__popcll(__ballot(dn & (v[i] > lo))));
      ng += static_cast<uint32_t>(__popcll(__ballot((v[i] > x) & (v[i] < hi))));
    }
    P = wave_sum(P);
    E = wave_sum(E);
    const double f = static_cast<double>(c) - 0.5 * P + 0.5 * E;
    const uint32_t old = left;
    int side;
    if (f <= k) {
      hi = x;
      fhi = f;
      left = na;
      side = 1;
    } else {
      lo = x;
      flo = f;
      left = ng;
      side = -1;
    }
    if (left == 0u) break;
    same = side == last ? same + 1 : 0;
    last = side;
    float xn = x;
    const double F = 0.5 * (P + E);
    if (it < 12 && F > 0.0)
      xn = static_cast<float>(xd + t * (f - k) / F * static_cast<double>(1 << (same < 6 ? same : 6)));
    if (it >= 3) stuck = left > old - old / 10u ? stuck + 1u : 0u;
    if ((left <= 4u && !(xn > lo && xn < hi)) || (stuck != 0u && (stuck & 3u) == 0u)) {
      // few scores left and no Newton step, or many equal ones that no point
      // between the ends parts: one of them, which settles it and all on one
      // side of it
      float m = -INFINITY;
#pragma unroll
      for (int i = 0; i < ITEMS; ++i) m = fmaxf(m, (v[i] > lo) & (v[i] < hi) ? v[i] : -INFINITY);
      xn = wave_max(m, -INFINITY);
    }
    if (!(xn > lo && xn < hi) && (it & 1) == 0) {
      // where the temperature is too small for a Newton step, between the ends
      // in proportion to LapSum; every second time their middle
      const float l = fmaxf(lo, mn), h = fminf(hi, mx);
      const float s = static_cast<float>((flo - k) / (flo - fhi));
      xn = l + (h - l) * fminf(fmaxf(s, 0.05f), 0.95f);
    }
    if (!(xn > lo && xn < hi)) xn = middle(fmaxf(lo, mn), fminf(hi, mx), it);
    // after a point that left nearly every score between the ends, the middle
    // of the keys: rows masked with a sentinel, heavy tails
    if ((stuck & 1u) != 0u && left > 4u) xn = key_mid(fmaxf(lo, mn), fminf(hi, mx));
    if (!(xn > lo && xn < hi)) xn = key_mid(lo, hi);
    x = xn;
    if (!(x > lo && x < hi)) break;   // no float between the ends
  }
  // the nearest score on each side, then the sums relative to it (scores at
  // or above hi, or below it: none lies strictly between the ends)
  const bool has_hi = hi < INFINITY;
  float u = INFINITY, w = -INFINITY;
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const bool up = has_hi ? v[i] >= hi : v[i] > lo;
    const bool dn = has_hi ? v[i] < hi : v[i] <= lo;
    if (up) u = fminf(u, v[i]);
    if (dn) w = fmaxf(w, v[i]);
  }
  u = wave_min(u, INFINITY);
  w = wave_max(w, -INFINITY);
  double P = 0.0, E = 0.0;
  uint32_t c = 0u;
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const bool up = v[i] >= u, dn = v[i] <= w;
    const double e = exp2_neg(-fabs(static_cast<double>(v[i]) - static_cast<double>(up ? u : w)) * c2);
    P = fma(e, up ? 1.0 : 0.0, P);
    E = fma(e, dn ? 1.0 : 0.0, E);
    c += static_cast<uint32_t>(__popcll(__ballot(up)));
  }
  P = wave_sum(P);
  E = wave_sum(E);
  // the logarithms of the two sums side by side (even and odd lanes)
  const bool has_u = u < INFINITY, has_w = w > -INFINITY;
  const double arg = (lane & 1) == 0 ? (has_u ? P : 1.0) : (has_w ? E : 1.0);
  const double lg = log(arg);
  const double b = gap_root(k, t, static_cast<double>(c), has_u, u, readlane_as(lg, 0), has_w, w,
                            readlane_as(lg, 1));
  if (lane == 0) b_out[row] = b;
  const double inv_t = 1.0 / t;
  float* p = probs + row * n;
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const int at = i * kWave + lane;
    if (at < n) p[at] = laplace_p(v[i], b, inv_t);
  }
}

hipError_t launch_row_wave_forward(const float* scores, int64_t batch, int64_t n, double k, double t,
                                   float* p, double* b, hipStream_t s) {
  if (n < 1 || n > kRowWaveMax || batch < 1) return hipErrorInvalidValue;
  const dim3 grid(static_cast<unsigned>((batch + RW - 1) / RW)), block(RT);
  const int ni = static_cast<int>(n);
  const double q = k / static_cast<double>(n);
  const float cut = static_cast<float>(q < 0.5 ? 0.66 * pow(q, 0.4) : 1.0 - 0.66 * pow(1.0 - q, 0.4));
  { ProfScope ps_("row_wave_forward", s);
#define LAPSUM_ROWW(IT) \
  hipLaunchKernelGGL(row_wave_forward_kernel<IT>, grid, block, 0, s, scores, batch, ni, k, t, cut, p, b)
  if (n <= 64) {
    LAPSUM_ROWW(1);
  } else if (n <= 128) {
    LAPSUM_ROWW(2);
  } else if (n <= 256) {
    LAPSUM_ROWW(4);
  } else if (n <= 512) {
    LAPSUM_ROWW(8);
  } else {
    LAPSUM_ROWW(16);
  }
#undef LAPSUM_ROWW
  }
  return hipGetLastError();
}

}  // namespace lapsum
