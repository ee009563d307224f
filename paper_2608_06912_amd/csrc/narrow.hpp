// Root finding by narrowing, for one workgroup: the threshold of Eq. (1) over
// a set of weighted scores (a row, or the members of a window of a row) with
// the scores outside the set as carries.
//
// LapSum is evaluated at points x (each score contributes 1 - e^{-(r-x)/t}/2
// above x and e^{-(x-r)/t}/2 below), which says on which side of x the root
// lies, until at most kNarrowMax scores are left between the two tightest
// points.  Everything outside is then summarised relative to the nearest
// score on each side (so neither sum can underflow, however flat LapSum is
// around the root), LapSum is formed at each score left, and the gap that
// holds the root is solved in closed form (gap_root).
//
// A point taken on the wrong side by rounding (LapSum(x) within rounding of
// k) moves no score across the root by more than that rounding: where LapSum
// is flat no score lies near x, and where it is not, the root is as close to
// x as the rounding.  So the points need not be scores, and the result does
// not depend on which points were tried.  The sums outside are taken in fixed
// point and the scores left are put in order first, so the result does not
// depend on the order of the set either.
#pragma once

#include "common.hpp"

namespace lapsum {

// Scores left for the last, pairwise step.  64 of them cost 16 terms per
// thread of a 256-thread workgroup; one more point costs about as much as
// the step from 64 to 128 would.
constexpr int kNarrowMax = 64;

// Scores outside the set: rank0 of them above it with their prefix pair
// (anchor at or above every score of the set), and the suffix pair of those
// below.
struct Carry {
  double rank0;
  Pre pre;
  Suf suf;
};

template <int BLOCK>
struct NarrowSmem {
  static constexpr int W = BLOCK / kWave;
  double P[2][W], E[2][W];
  uint32_t c[2][W], a[2][W], g[2][W];
  float um[W], vm[W];
  unsigned long long S[W], T[W];
  uint32_t fill;
  float ev[kNarrowMax], sv[kNarrowMax];
  uint32_t ew[kNarrowMax], sw[kNarrowMax];
  double pa[kNarrowMax], ea[kNarrowMax], ca[kNarrowMax];
  uint32_t le;
  double b;
};

// Descending-key midpoint of the open interval (lo, hi); equals an end when
// no float lies between.
__device__ __forceinline__ float key_mid(float lo, float hi) {
  const uint32_t kh = desc_key(fminf(hi, 3.402823466e38f));
  const uint32_t kl = desc_key(fmaxf(lo, -3.402823466e38f));
  return key_float(kh + (kl - kh) / 2u);
}

// The next point when a Newton step leaves (lo, hi): the arithmetic middle,
// and after twenty points (or with an end still open) the middle of the
// keys.  Taken at least every second time from there on, it reaches every gap
// within 2 x 32 more.
__device__ __forceinline__ float middle(float lo, float hi, int it) {
  const float m = 0.5f * lo + 0.5f * hi;
  return it < 20 && m > lo && m < hi ? m : key_mid(lo, hi);
}

// Each(f) calls f(value, weight) for every score of this thread's share of
// the set, held by the BLOCK threads of the workgroup still running (higher
// waves may have ended); `total` is the number of scores (weighted entries)
// in the set and `weight` their total weight (fewer than 2^31).  x0: the first point, inside
// the carries' anchors.  Returns b in every thread.
template <int BLOCK, class Each>
__device__ double narrow_solve(Each&& each, uint32_t total, uint32_t weight, const Carry& ext,
                               float lo, float hi, float x0, double k, double t,
                               NarrowSmem<BLOCK>& sm) {
  constexpr int W = BLOCK / kWave;
  const int tid = threadIdx.x;
  const int lane = lane_id();
  const int wid = tid / kWave;
  const double c2 = kLog2e / t;
  uint32_t left = total;
  float x = x0 == x0 ? x0 : 0.0f;   // (a NaN point would end the search at once)
  int same = 0, last = 0;
  bool key = false;   // the last point was a middle of the keys
  // LapSum at the ends (about, until they are points)
  double flo = ext.rank0 + static_cast<double>(weight), fhi = ext.rank0;
  const double noise = 1e-14 * flo;
  // the set's range, where the middle of an end still open is taken
  float mn = INFINITY, mx = -INFINITY;
  if (left > static_cast<uint32_t>(kNarrowMax)) {
    each([&](float v, uint32_t) {
      mn = fminf(mn, v);
      mx = fmaxf(mx, v);
    });
    mn = wave_min(mn, INFINITY);
    mx = wave_max(mx, -INFINITY);
    if (lane == 0) {
      sm.um[wid] = mn;
      sm.vm[wid] = mx;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < W; ++w) {
      mn = fminf(mn, sm.um[w]);
      mx = fmaxf(mx, sm.vm[w]);
    }
  }
  for (int it = 0; left > static_cast<uint32_t>(kNarrowMax) && it < 96; ++it) {
    const int pb = it & 1;   // two sets of partials: one barrier per point
    double P = 0.0, E = 0.0;
    uint32_t c = 0u, na = 0u, ng = 0u;
    const double xd = x;
    each([&](float v, uint32_t w) {
      const double d = static_cast<double>(v) - xd;
      const double e = static_cast<double>(w) * exp2_neg(-fabs(d) * c2);
      const bool up = v >= x;
      P += up ? e : 0.0;
      E += up ? 0.0 : e;
      c += up ? w : 0u;
      na += (v > lo && v < x) ? 1u : 0u;
      ng += (v > x && v < hi) ? 1u : 0u;
    });
    P = wave_sum(P);
    E = wave_sum(E);
    c = wave_sum(c);
    na = wave_sum(na);
    ng = wave_sum(ng);
    if (lane == 0) {
      sm.P[pb][wid] = P;
      sm.E[pb][wid] = E;
      sm.c[pb][wid] = c;
      sm.a[pb][wid] = na;
      sm.g[pb][wid] = ng;
    }
    __syncthreads();
    P = E = 0.0;
    c = na = ng = 0u;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      P += sm.P[pb][w];
      E += sm.E[pb][w];
      c += sm.c[pb][w];
      na += sm.a[pb][w];
      ng += sm.g[pb][w];
    }
    P += ext.pre.S * exp2_neg(fmin(xd - static_cast<double>(ext.pre.u), 0.0) * c2);
    E += ext.suf.T * exp2_neg(fmin(static_cast<double>(ext.suf.v) - xd, 0.0) * c2);
    const double f = ext.rank0 + static_cast<double>(c) - 0.5 * P + 0.5 * E;
    const uint32_t old = left;
    int side;
    // (LapSum within its sums' rounding of the budget counts as equal to it, so
    // that their order does not decide where LapSum is flat around the root)
    if (f - k <= noise) {
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
    same = side == last ? same + 1 : 0;
    last = side;
    // the next point: a Newton step, longer each time the root stayed on the
    // same side so that both ends close in; when that leaves them (a
    // temperature too small for it), and after a dozen points always, between
    // the ends in proportion to LapSum, every second time their middle
    float xn = x;
    const double F = 0.5 * (P + E);
    if (it < 12 && F > 0.0 && fabs(f - k) > noise) {
      const double step = t * (f - k) / F * static_cast<double>(1 << (same < 6 ? same : 6));
      xn = static_cast<float>(xd + step);
    }
    if (!(xn > lo && xn < hi) && (it & 1) == 0) {
      const float l = fmaxf(lo, mn), h = fminf(hi, mx);
      const float q = static_cast<float>((flo - k) / (flo - fhi));
      xn = l + (h - l) * fminf(fmaxf(q, 0.05f), 0.95f);
    }
    if (!(xn > lo && xn < hi)) xn = middle(fmaxf(lo, mn), fminf(hi, mx), it);
    // a set that spans many orders of magnitude (a sentinel, heavy tails): the
    // middle of the keys after a point that left most of it between the ends
    if (it >= 4) {
      key = !key && left > old - old / 4u;
      if (key) xn = key_mid(fmaxf(lo, mn), fminf(hi, mx));
    }
    if (!(xn > lo && xn < hi)) xn = key_mid(lo, hi);
    x = xn;
    if (!(x > lo && x < hi)) break;   // no float between the ends
  }

  // the nearest scores outside (lo, hi), then the sums relative to them
  float um = INFINITY, vm = -INFINITY;
  uint32_t cu = 0u, cd = 0u;
  if (tid == 0) {
    sm.fill = 0u;
    sm.le = 0u;
  }
  each([&](float v, uint32_t w) {
    if (v >= hi) {
      um = fminf(um, v);
      cu += w;
    } else if (v <= lo) {
      vm = fmaxf(vm, v);
      cd += w;
    }
  });
  um = wave_min(um, INFINITY);
  vm = wave_max(vm, -INFINITY);
  cu = wave_sum(cu);
  cd = wave_sum(cd);
  __syncthreads();   // the last point's partials have been read
  if (lane == 0) {
    sm.um[wid] = um;
    sm.vm[wid] = vm;
    sm.c[0][wid] = cu;
    sm.a[0][wid] = cd;
  }
  __syncthreads();
  cu = cd = 0u;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    um = fminf(um, sm.um[w]);
    vm = fmaxf(vm, sm.vm[w]);
    cu += sm.c[0][w];
    cd += sm.a[0][w];
  }
  const int fbits = 62 - (64 - __clzll(static_cast<long long>(weight) | 1ll));
  const double fscale = ldexp(1.0, fbits);
  unsigned long long S = 0ull, T = 0ull;
  each([&](float v, uint32_t w) {
    if (v >= hi) {
      const double e = exp2_neg((static_cast<double>(um) - static_cast<double>(v)) * c2);
      S += static_cast<unsigned long long>(w) * __double2ull_rn(e * fscale);
    } else if (v <= lo) {
      const double e = exp2_neg((static_cast<double>(v) - static_cast<double>(vm)) * c2);
      T += static_cast<unsigned long long>(w) * __double2ull_rn(e * fscale);
    } else {
      const uint32_t at = atomicAdd(&sm.fill, 1u);
      if (at < static_cast<uint32_t>(kNarrowMax)) {
        sm.ev[at] = v;
        sm.ew[at] = w;
      }
    }
  });
  S = wave_sum(S);
  T = wave_sum(T);
  if (lane == 0) {
    sm.S[wid] = S;
    sm.T[wid] = T;
  }
  __syncthreads();
  S = T = 0ull;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    S += sm.S[w];
    T += sm.T[w];
  }
  Pre pre = ext.pre;
  Suf suf = ext.suf;
  if (cu != 0u) {
    double s = static_cast<double>(S) * ldexp(1.0, -fbits);
    s += pre.S * exp2_neg(fmin(static_cast<double>(um) - static_cast<double>(pre.u), 0.0) * c2);
    pre = Pre{um, s};
  }
  if (cd != 0u) {
    double s = static_cast<double>(T) * ldexp(1.0, -fbits);
    s += suf.T * exp2_neg(fmin(static_cast<double>(suf.v) - static_cast<double>(vm), 0.0) * c2);
    suf = Suf{vm, s};
  }
  const double rank0 = ext.rank0 + static_cast<double>(cu);
  // (the points end with at most kNarrowMax scores left, or with no float
  // between the ends; anything else is no result)
  if (sm.fill > static_cast<uint32_t>(kNarrowMax)) return NAN;
  const int ne = static_cast<int>(sm.fill);

  // the scores left, in descending order (equal scores by weight): ranks by
  // counting, TPK adjacent threads to an entry
  constexpr int TPK = BLOCK / kNarrowMax;
  static_assert(TPK >= 1 && TPK * kNarrowMax == BLOCK, "threads per entry");
  const int i = tid / TPK, q = tid % TPK;
  const bool active = i < ne;
  if (active) {
    const float v = sm.ev[i];
    const uint32_t w = sm.ew[i];
    uint32_t rk = 0u;
#pragma unroll 4
    for (int j = q; j < ne; j += TPK) {
      const float vj = sm.ev[j];
      const uint32_t wj = sm.ew[j];
      rk += (vj > v || (vj == v && (wj > w || (wj == w && j < i)))) ? 1u : 0u;
    }
#pragma unroll
    for (int o = 1; o < TPK; o <<= 1) rk += __shfl_xor(rk, o, kWave);
    if (q == 0) {
      sm.sv[rk] = v;
      sm.sw[rk] = w;
    }
  }
  __syncthreads();
  if (active) {
    const float v = sm.sv[i];
    const double vd = v;
    double Pg = 0.0, El = 0.0;
    uint32_t gt = 0u, eq = 0u;
#pragma unroll 4
    for (int j = q; j < ne; j += TPK) {
      const double d = static_cast<double>(sm.sv[j]) - vd;
      const uint32_t wj = sm.sw[j];
      const double e = static_cast<double>(wj) * exp2_neg(-fabs(d) * c2);
      Pg += d > 0.0 ? e : 0.0;
      El += d < 0.0 ? e : 0.0;
      gt += d > 0.0 ? wj : 0u;
      eq += d == 0.0 ? wj : 0u;
    }
#pragma unroll
    for (int o = 1; o < TPK; o <<= 1) {
      Pg += __shfl_xor(Pg, o, kWave);
      El += __shfl_xor(El, o, kWave);
      gt += __shfl_xor(gt, o, kWave);
      eq += __shfl_xor(eq, o, kWave);
    }
    const double Pc = pre.S * exp2_neg(fmin(vd - static_cast<double>(pre.u), 0.0) * c2);
    const double Ec = suf.T * exp2_neg(fmin(static_cast<double>(suf.v) - vd, 0.0) * c2);
    const double N = rank0 + gt + 0.5 * eq - 0.5 * (Pg + Pc) + 0.5 * (El + Ec);
    if (q == 0) {
      sm.pa[i] = Pg + eq + Pc;
      sm.ea[i] = El + eq + Ec;
      sm.ca[i] = static_cast<double>(gt) + static_cast<double>(eq);
      if (N <= k) atomicMax(&sm.le, static_cast<uint32_t>(i) + 1u);
    }
  }
  __syncthreads();
  if (tid < 2) {
    // the gap: u the lowest score with LapSum <= k, v the highest above it;
    // the logarithms of its two sums side by side (lanes 0 and 1)
    const int m = static_cast<int>(sm.le);
    const bool has_u = m > 0, has_v = m < ne;
    const bool up = has_u || pre.S > 0.0, dn = has_v || suf.T > 0.0;
    double arg;
    if (tid == 0)
      arg = has_u ? sm.pa[m - 1] : (up ? pre.S : 1.0);
    else
      arg = has_v ? sm.ea[m] : (dn ? suf.T : 1.0);
    const double lg = log(arg);
    const double lnB = __shfl(lg, 1, kWave);
    if (tid == 0) {
      const double c_up = rank0 + (has_u ? sm.ca[m - 1] : 0.0);
      const double u = has_u ? sm.sv[m - 1] : pre.u;
      const double v = has_v ? sm.sv[m] : suf.v;
      sm.b = gap_root(k, t, c_up, up, u, lg, dn, v, lnB);
    }
  }
  __syncthreads();
  const double b = sm.b;
  __syncthreads();
  return b;
}

}  // namespace lapsum
