// The full-sort forward's threshold for long rows without sorting them, many
// rows at a time (used for every row that one workgroup does not hold on
// chip; the sort remains for the permutation).
//
// Three launches, four past 2^18 scores (long_merge), one row per grid.y:
//   long_window   one workgroup per row: a stratified random sample of the
//                 row (4096 scores, 16384 past 2^24) gives a window [xlo, xhi)
//                 that holds b in all but about 2 e^{-z^2/2} = 5e-7 of samples
//                 (z = 5.5; for independent positions and a known variance,
//                 an estimate here): LapSum of the sample, less (plus) a
//                 Bernstein margin, still lies above (below) the budget at its
//                 ends
//   long_pass     the one streaming pass over the row: scores at or above
//                 xhi and below xlo are summed as the tails of Suppl. B, the
//                 members of the window are sorted into cells (count, the two
//                 exponential sums, and the members themselves, per block)
//   long_root     one workgroup per row: the blocks' cells merged, LapSum at
//                 every cell edge, and the members of the cell that holds b
//                 and of its two neighbours narrowed down to the root
//                 (narrow.hpp).  The tails give LapSum at the window's ends
//                 exactly; where the root lies outside them, the whole row
//                 is divided and narrowed by this workgroup, and where the
//                 three cells hold more than LDS, their entries are (slower,
//                 and always right).
// The sample decides only which scores are looked at one by one: b is the
// root of the same equation, from the sums of every score.
//
// Bound: long_pass by reading the row (4 B/score) and, where t is wide, by
// one float64 exponential per score; the other two by latency.  Sorting moves
// 48 B/score in twelve launches and a row at a time for the same b.  Kernels
// of one forward (rocprofv3, the sort's first, without the emit): one row of
// 1e5 68 -> 30 us, of 1e6 (k = 1000, t = 0.05) 77 -> 40 us, of 1e7 (k = 2000,
// t = 0.01) 217 -> 61 us, 48 rows of 131073 (k = n/16, t = 1) 2.8 ms -> 49 us.
#include <math.h>

#include "kernels.hpp"
#include "block_sort.hpp"
#include "narrow.hpp"

namespace lapsum {

namespace {

// One wave per SIMD in the latency-bound kernels: what every wave computes
// for itself (the sums over the waves' partials, the carries) is issued once
// per SIMD instead of four times (1024 threads: 1.7 us a point of long_window
// and 6 us a point of long_root, against 0.7 and 0.9).
constexpr int WT = 256;
constexpr int MT = 1024;   // long_root threads while it merges or divides cells
constexpr int LT = 512;    // long_pass threads
constexpr int LW = LT / kWave;
constexpr int kStage = 512;               // members a wave of long_pass stages
constexpr int kLongQuads = 4;             // 16-byte loads in flight per thread
constexpr int64_t kLongTile = static_cast<int64_t>(LT) * 4;   // scores per step of a block
constexpr int kWindowPoints = 16;
constexpr float kMaxScore = 3.402823466e38f;
constexpr float kFewSamples = 3.0f;       // (b past the sample's last score: e^-3)
constexpr int kRootCap = 24576;           // entries long_root narrows in LDS (half with weights)

// A window of one row.  Cells run downwards: cell 0 above xcap (the sample's
// largest score, past it for small budgets, or xhi), cells 1 .. NC-2 equal steps of value down to
// xfloor, cell NC-1 below xfloor.
struct Window {
  float xlo, xhi;      // -inf / +inf: unbounded
  float xcap, xfloor;
  float scale;         // cells per unit of value; negative: cells by a table
  float x0;            // the sample's estimate of b
};

// Where equal steps would leave one cell with most of the members (many equal
// scores, clusters, a sentinel inside the window), the cells follow the
// sample instead: bound[c], non-increasing, is the least score of cell c for
// c < NC - 1, every bound the same share of the sample's members apart (one
// row of 1e6 scores, forward, us, equal steps / by the sample: two clusters
// 18000 / 260, 30% of the scores -3.4e38 and k = 0.69 n 4800 / 120, a third of
// the row 1e-6 wide 1700 / 95; the sort 70-160); a value met by several
// bounds has a cell to itself (see long_window).
template <int NC>
__device__ __forceinline__ int cell_of(const Window& w, float v) {
  if (v > w.xcap) return 0;
  if (v < w.xfloor) return NC - 1;
  const int c = static_cast<int>((w.xcap - v) * w.scale);   // non-increasing in v
  return 1 + (c < NC - 3 ? c : NC - 3);
}
// Upper edge of cell c (the window's lower end for c = NC), a float32 value.
// A member can lie beyond its edge by the rounding of cell_of; exponents are
// clamped at 0 there, and the last step takes the members themselves.
template <int NC>
__device__ __forceinline__ double edge_of(const Window& w, const float* __restrict__ bound, int c) {
  if (c == 0) return w.xhi < INFINITY ? w.xhi : w.xcap;
  if (c == NC) return w.xlo > -INFINITY ? w.xlo : w.xfloor;
  if (w.scale < 0.0f) return bound[c - 1];
  const double cap = w.xcap, fl = w.xfloor;
  return static_cast<float>(cap - static_cast<double>(c - 1) * ((cap - fl) / static_cast<double>(NC - 2)));
}

// The cell of v from the cells' upper edges (in a fixed number of steps, so
// that several searches run side by side).
template <int NC>
__device__ __forceinline__ int cell_by_edges(const double* edge, float v) {
  const double x = v;
  int c = 0;
#pragma unroll
  for (int step = NC / 2; step > 0; step >>= 1) c += x < edge[c + step] ? step : 0;
  return c;
}
template <int NC>
__device__ __forceinline__ int cell_at(const Window& w, const double* edge, float v) {
  return w.scale >= 0.0f ? cell_of<NC>(w, v) : cell_by_edges<NC>(edge, v);
}

// One block's share of a row.
struct LongBlock {
  double TR, TL;     // tails at xhi and xlo
  uint32_t nR;       // scores at or above xhi
  uint32_t merged;   // a cell's equal members are written once (weight = its count)
};

// One block's cells, each NC long (offs NC + 1).
struct LongCells {
  LongBlock* blk;   // [rows][G]
  double* U;        // [rows][G][NC] sum e^{-(edge(c) - r)/t}
  double* D;        // [rows][G][NC] sum e^{-(r - edge(c+1))/t}
  uint32_t* cnt;    // [rows][G][NC] members
  uint32_t* off;    // [rows][G][NC + 1] first entry of the cell in the block's list
  float* list;      // [rows][G * chunk] entries of each block in cell order
  Window* win;      // [rows]
  float* bound;     // [rows][NC] the cells' table, where the window says so
  double *mU, *mD;  // [rows][NC] the merged cells (rows of many blocks)
  uint32_t* mcnt;
};

// Chris Wellons' 32-bit mixer "lowbias32" (its shifts and two multipliers, from
// his search for integer hashes of low bias, "hash prospector", 2018): every
// input bit flips every output bit in close to half of the cases.
__device__ __forceinline__ uint32_t mix32(uint32_t x) {
  x ^= x >> 16;
  x *= 0x7feb352du;
  x ^= x >> 15;
  x *= 0x846ca68bu;
  x ^= x >> 16;
  return x;
}

}  // namespace

// ---------------------------------------------------------------- window ---
// ITEMS samples per thread, one from each of WT * ITEMS equal strata of the
// row at a hashed position (a plain stride would repeat the period of data
// laid out in columns).  With S = sum p, V = sum p^2 - S^2/m and
// F = sum min(p, 1 - p) over the m samples at a point x (p the Laplace CDF
// term, in [0, 1]) and mu = k m / n the sample's share of the budget, x lies
// below b when S - mu exceeds z sqrt(V mu/S) + z^2/3 and above it when mu - S
// does (Bernstein's bound for a sum whose mean is mu, z = 5.5; V mu/S the
// variance scaled to that mean).  Both ends are found together, by Newton
// steps on S (dS/dx = -F/t) kept inside a bracket, by interpolating the logit
// of S between the bracket's ends where a step leaves it (bisection every
// third time); a point is taken once the margin is the larger part of its
// distance, so the window is at most about a third wider than it must be.
// Points by value do not come near the root where the row spans many orders
// of magnitude (scores masked with a sentinel, heavy tails): from the fifth
// point on, one that leaves more than three quarters of the samples between
// the ends is followed by the middle of the keys, which is sensitive to
// magnitudes.  Rows with 30% of the scores at -3.4e38 take 7-12 points, without
// it all 28 that there were; bell-shaped and exponential rows take 2-6 as
// before (taken from the third point on, exponential ones took up to 9).
// Where no point qualifies after kWindowPoints, the ends are what they are:
// the cells (and not b) depend on them.
// Each point costs about 0.7 us of one workgroup's latency: the start by the
// logit instead of in the middle takes three points instead of four to six
// (kernel 13.5 -> 12.8 us at 1e6 scores, 15.6 -> 13.3 for 48 rows of 131073).
// The sums are float32: they only place the window.
template <int ITEMS, int NC>
__global__ __launch_bounds__(WT) void long_window_kernel(const float* __restrict__ scores,
                                                         int64_t n, double k, double t,
                                                         Window* __restrict__ win,
                                                         float* __restrict__ bounds) {
  constexpr int M = WT * ITEMS;
  constexpr int W = WT / kWave;
  constexpr float Z = 5.5f, Z2 = Z * Z / 3.0f;
  __shared__ float red[2][6][W];
  __shared__ float mm[2][W];
  __shared__ uint32_t cnt[NC + 2], crowd[2][W];
  __shared__ uint32_t sorted[sort_buf_words<WT, 16>()];
  __shared__ SortSmem<WT> ssm;
  const int tid = threadIdx.x;
  const int lane = lane_id();
  const int wid = tid / kWave;
  const float* r = scores + static_cast<int64_t>(blockIdx.y) * n;
  float v[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const uint32_t s = static_cast<uint32_t>(i * WT + tid);
    const uint64_t a = static_cast<uint64_t>(s) * static_cast<uint64_t>(n) / M;
    const uint64_t e = static_cast<uint64_t>(s + 1) * static_cast<uint64_t>(n) / M;
    v[i] = r[a + ((static_cast<uint64_t>(mix32(s)) * (e - a)) >> 32)];
    v[i] = fminf(fmaxf(v[i], -kMaxScore), kMaxScore);   // (every point stays finite)
  }
  float mn = v[0], mx = v[0];
#pragma unroll
  for (int i = 1; i < ITEMS; ++i) {
    mn = fminf(mn, v[i]);
    mx = fmaxf(mx, v[i]);
  }
  mn = wave_min(mn, INFINITY);
  mx = wave_max(mx, -INFINITY);
  if (lane == 0) {
    mm[0][wid] = mn;
    mm[1][wid] = mx;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < W; ++w) {
    mn = fminf(mn, mm[0][w]);
    mx = fmaxf(mx, mm[1][w]);
  }
  const float mu = static_cast<float>(k * static_cast<double>(M) / static_cast<double>(n));
  const float c2 = static_cast<float>(fmin(kLog2e / t, 3.0e38));
  const float tf = static_cast<float>(t);
  // S, V and F at two points at once
  struct At {
    float S, m, F;   // m: the margin
  };
  auto eval = [&](float xa, float xb, int pb, At& A, At& B) {
    float s[6] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      const float ea = 0.5f * exp2_fast(-fabsf(v[i] - xa) * c2);
      const float eb = 0.5f * exp2_fast(-fabsf(v[i] - xb) * c2);
      const float pa = v[i] >= xa ? 1.0f - ea : ea;
      const float pp = v[i] >= xb ? 1.0f - eb : eb;
      s[0] += pa;
      s[1] = fmaf(pa, pa, s[1]);
      s[2] += ea;
      s[3] += pp;
      s[4] = fmaf(pp, pp, s[4]);
      s[5] += eb;
    }
#pragma unroll
    for (int q = 0; q < 6; ++q) s[q] = wave_sum(s[q]);
    if (lane == 0) {
#pragma unroll
      for (int q = 0; q < 6; ++q) red[pb][q][wid] = s[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 6; ++q) {
      s[q] = 0.0f;
#pragma unroll
      for (int w = 0; w < W; ++w) s[q] += red[pb][q][w];
    }
    auto margin = [&](float S, float Q) {
      return Z * sqrtf(fmaxf(Q - S * S * (1.0f / M), 0.0f) * (mu / fmaxf(S, 1e-30f))) + Z2;
    };
    A = At{s[0], margin(s[0], s[1]), s[2]};
    B = At{s[3], margin(s[3], s[4]), s[5]};
  };
  // the lower end between la (surely below b) and lb, the upper end between
  // ha (surely above b) and hb
  At A, B;
  eval(mn, mx, 0, A, B);
  float la = mn, lb = mx, ha = mx, hb = mn;
  const bool has_lo = A.S - A.m >= mu, has_hi = B.S + B.m <= mu;
  // a root surely past the sample's last score (rows much narrower than t):
  // the sample has no better end than that score
  const bool above = has_lo && B.S - B.m >= mu, under = has_hi && A.S + A.m <= mu;
  if (above) la = mx;
  if (under) ha = mn;
  bool lo_on = has_lo && !above, hi_on = has_hi && !under;
  // a point between p and q where the sum's logit, nearly straight over a
  // bell-shaped row, passes the wanted one's
  auto logit = [&](float S) {
    const float c = fminf(fmaxf(S, 0.25f), M - 0.25f);
    return __log2f(c / (M - c));
  };
  auto between = [&](float p, float Lp, float q, float Lq, float want) {
    const float s = (Lp - logit(want)) / (Lp - Lq);
    const float x = p + (q - p) * fminf(fmaxf(s, 0.02f), 0.98f);
    return x > fminf(p, q) && x < fmaxf(p, q) ? x : 0.5f * p + 0.5f * q;
  };
  // a Newton step from x that goes at most a quarter of the way to an end of
  // (l, h): from where few scores are left it can throw far past the root
  auto near = [](float nx, float x, float l, float h) {
    return nx > l && nx < h && nx >= l + 0.75f * (x - l) && nx <= h - 0.75f * (h - x);
  };
  float Lla = logit(A.S), Llb = logit(B.S), Lha = Llb, Lhb = Lla;
  float Sla = above ? B.S : A.S, Slb = B.S, Sha = under ? A.S : B.S, Shb = A.S;
  bool lo_key = false, hi_key = false;   // the last point was a middle of the keys
  const float m0 = 1.15f * (Z * sqrtf(mu * fmaxf(1.0f - mu / M, 0.0f)) + Z2);
  float xa = between(la, Lla, lb, Llb, mu + m0), xb = between(ha, Lha, hb, Lhb, mu - m0);
  for (int it = 1; it <= kWindowPoints && (lo_on || hi_on); ++it) {
    eval(xa, xb, it & 1, A, B);
    if (lo_on) {
      const float old = Sla - Slb;
      if (A.S - A.m >= mu) {
        la = xa;
        Sla = A.S;
        Lla = logit(A.S);
        lo_on = A.S - mu > 1.35f * A.m;
      } else {
        lb = xa;
        Slb = A.S;
        Llb = logit(A.S);
      }
      const float nx = xa + tf * (A.S - mu - 1.15f * A.m) / A.F;
      xa = (it < 12 && near(nx, xa, la, lb)) ? nx
           : (it % 3 != 0)                  ? between(la, Lla, lb, Llb, mu + 1.15f * A.m)
                                            : 0.5f * la + 0.5f * lb;
      if (it >= 5) {
        lo_key = !lo_key && Sla - Slb > 0.75f * old;
        if (lo_key) xa = key_mid(la, lb);
      }
    }
    if (hi_on) {
      const float old = Shb - Sha;
      if (B.S + B.m <= mu) {
        ha = xb;
        Sha = B.S;
        Lha = logit(B.S);
        hi_on = mu - B.S > 1.35f * B.m;
      } else {
        hb = xb;
        Shb = B.S;
        Lhb = logit(B.S);
      }
      const float nx = xb + tf * (B.S - mu + 1.15f * B.m) / B.F;
      xb = (it < 12 && near(nx, xb, hb, ha)) ? nx
           : (it % 3 != 0)                  ? between(ha, Lha, hb, Lhb, mu - 1.15f * B.m)
                                            : 0.5f * ha + 0.5f * hb;
      if (it >= 5) {
        hi_key = !hi_key && Shb - Sha > 0.75f * old;
        if (hi_key) xb = key_mid(hb, ha);
      }
    }
  }
  Window w;
  w.xlo = has_lo ? la : -INFINITY;
  w.xhi = has_hi ? ha : INFINITY;
  // rounding can only cross the ends of a window without scores; keep both
  // sides well formed
  if (!(w.xlo < w.xhi)) {
    w.xlo = -INFINITY;
    w.xhi = INFINITY;
  }
  w.xcap = fminf(mx, w.xhi);
  w.xfloor = fmaxf(mn, w.xlo);
  if (!(w.xfloor <= w.xcap)) w.xfloor = w.xcap;
  // a budget of fewer than kFewSamples of the sample's scores can have b
  // beyond its last score, where all the row's scores would be one cell:
  // cells for as much again (likewise below).  1e7 Laplace scores, k = 2000,
  // t = 0.01, eight rows: forward 65-170 us, mean 105, without, 64-80, mean
  // 70, with.  With more of them b is seldom there, and the steps would be
  // twice as wide for nothing.
  const float span = w.xcap - w.xfloor;
  if (!has_hi && has_lo && mu < kFewSamples && w.xcap + span < INFINITY) w.xcap += span;
  if (!has_lo && has_hi && M - mu < kFewSamples && w.xfloor - span > -INFINITY) w.xfloor -= span;
  const float width = w.xcap - w.xfloor;
  w.scale = (width > 0.0f && width < INFINITY) ? static_cast<float>(NC - 2) / width : 0.0f;
  if (!(w.scale < INFINITY)) w.scale = 0.0f;
  w.x0 = 0.5f * w.xcap + 0.5f * w.xfloor;
  // the cells by the sample where equal steps would crowd three neighbouring
  // ones past what long_root keeps on chip, several times their share.  The
  // sample is looked at where the window can hold a quarter of the row, or
  // four times what long_root keeps (with fewer members long_root divides a
  // crowded cell itself, in 0.1-0.2 ms; the look costs 1.5 us, which ordinary
  // rows with wide windows would pay).  A member's term differs between the
  // ends by (1 - e^{-width/t})/2 next to one of them up to nearly 1 halfway,
  // which tells about how many there are.
  auto member = [&](float x) { return x >= w.xlo && x < w.xhi; };
  const float per = static_cast<float>(static_cast<double>(n) / M);   // scores per sample
  const float ends = fminf(mx, w.xhi) - fmaxf(mn, w.xlo);
  const float most = 1.25f * (Sla - Sha) / (1.0f - exp2_fast(-ends * c2));   // (NaN: no width)
  uint32_t in = 0u, top = 0u;
  if (most * per > 4.0f * kRootCap || (most * per > kRootCap && 4.0f * most > M)) {
    for (int c = tid; c < NC + 2; c += WT) cnt[c] = 0u;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
      if (member(v[i])) atomicAdd(&cnt[1 + cell_of<NC>(w, v[i])], 1u);
    __syncthreads();
    if (tid < NC) {
      in = cnt[tid + 1];
      top = in + cnt[tid] + cnt[tid + 2];
    }
    in = wave_sum(in);
    top = wave_max_u32(top);
    if (lane == 0) {
      crowd[0][wid] = in;
      crowd[1][wid] = top;
    }
    __syncthreads();
    in = 0u;
#pragma unroll
    for (int i = 0; i < W; ++i) {
      in += crowd[0][i];
      top = max(top, crowd[1][i]);
    }
  }
  if (static_cast<float>(top) * per > kRootCap && top > 12u * in / NC + 24u) {
    // 4096 of the samples, the members among them in descending order
    constexpr int STEP = ITEMS / 16;
    uint32_t key[16];
    int32_t none[16];
    uint32_t m = 0u;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float x = v[i * STEP];
      key[i] = member(x) ? desc_key(x + 0.0f) : 0xffffffffu;   // (one zero)
      m += member(x) ? 1u : 0u;
    }
    m = wave_sum(m);
    __syncthreads();
    if (lane == 0) crowd[0][wid] = m;
    __syncthreads();
    m = 0u;
#pragma unroll
    for (int i = 0; i < W; ++i) m += crowd[0][i];
    block_sort_u32<WT, 16, false>(key, none, sorted, ssm);   // (leaves the order in `sorted`)
    if (m > 0u) {
      auto at = [&](int c) {
        const uint32_t q = static_cast<uint32_t>(c) * m / (NC - 2);
        return sorted[buf_at(static_cast<int>(q < m ? q : m - 1u))];
      };
      // of equal bounds the last is the value, those before it the next
      // float above: one cell of that value alone, the others empty
      if (tid < NC - 1) {
        const uint32_t key0 = at(tid);
        const bool again = tid < NC - 2 && at(tid + 1) == key0;
        bounds[static_cast<int64_t>(blockIdx.y) * NC + tid] = key_float(key0 - (again ? 1u : 0u));
      }
      w.scale = -1.0f;
    }
  }
  if (tid == 0) win[blockIdx.y] = w;
}

// ------------------------------------------------------------------ pass ---
// Block g streams scores [g chunk, (g + 1) chunk) of its row.  One
// exponential per score, for whichever tail holds it.  Members are staged per
// wave in LDS, then summed into the cells by LDS atomics (64-bit fixed point: integer additions commute) and
// written out in cell order.  A cell whose members are all equal (quantised
// scores) is written as one entry.  A block whose members outgrow the staging
// streams its chunk twice more instead (from the caches): once for the cells,
// taking equal neighbours together, and once to write the members.
template <int NC>
__global__ __launch_bounds__(LT) void long_pass_kernel(const float* __restrict__ scores, int64_t n,
                                                       int64_t chunk, double t, LongCells o) {
  __shared__ float stage[LW][kStage];
  __shared__ uint32_t cn[NC], kmin[NC], kmax[NC], cur[NC + 1];
  __shared__ unsigned long long cu[NC], cd[NC];
  __shared__ double edge[NC + 1];
  __shared__ double red[2][LW];
  __shared__ uint32_t rn[LW], over_s[LW];
  const int tid = threadIdx.x;
  const int lane = lane_id();
  const int wid = tid / kWave;
  const int64_t row = blockIdx.y;
  const int G = gridDim.x;
  const int g = blockIdx.x;
  const float* r = scores + row * n;
  const Window w = o.win[row];
  const int64_t c0 = static_cast<int64_t>(g) * chunk;
  const int64_t c1 = c0 + chunk < n ? c0 + chunk : n;
  const double c2 = kLog2e / t;
  for (int e = tid; e < NC; e += LT) {
    cn[e] = 0u;
    kmin[e] = 0xffffffffu;
    kmax[e] = 0u;
    cu[e] = 0ull;
    cd[e] = 0ull;
  }
  for (int e = tid; e <= NC; e += LT) edge[e] = edge_of<NC>(w, o.bound + row * NC, e);
  const double xhi = w.xhi, xlo = w.xlo;
  const float farf = static_cast<float>(fmin(fmax(150.0 / c2, 1e-37), 3.0e38));   // beyond: 2^-150, no part of the sums
  double TR = 0.0, TL = 0.0;
  uint32_t nR = 0u;
  int staged = 0;   // members this wave has met (wave-uniform)
  // one quad per lane, without branches inside a lane (a NaN is no score);
  // a wave skips the exponentials when every tail score of its quads is far,
  // and the staging when no score is a member
  auto take4 = [&](const float (&v)[4]) {
    bool up[4], dn[4], in[4];
    float dmin = INFINITY;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      up[e] = v[e] >= w.xhi;
      dn[e] = v[e] < w.xlo;
      in[e] = (v[e] < w.xhi) & (v[e] >= w.xlo);
      const float d = fmaxf(v[e] - w.xhi, w.xlo - v[e]);
      dmin = fminf(dmin, in[e] ? INFINITY : d);
      nR += up[e] ? 1u : 0u;
    }
    if (__any(dmin < farf)) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double d = static_cast<double>(v[e]) - (up[e] ? xhi : xlo);
        const double x = exp2_neg(-fabs(d) * c2);
        TR = fma(x, up[e] ? 1.0 : 0.0, TR);
        TL = fma(x, dn[e] ? 1.0 : 0.0, TL);
      }
    }
    // members, one per lane and turn (a lane seldom holds two)
    uint32_t mem = (in[0] ? 1u : 0u) | (in[1] ? 2u : 0u) | (in[2] ? 4u : 0u) | (in[3] ? 8u : 0u);
    for (uint64_t m = __ballot(mem != 0u); m != 0ull; m = __ballot(mem != 0u)) {
      const int at = staged + static_cast<int>(__builtin_amdgcn_mbcnt_hi(
                                  static_cast<uint32_t>(m >> 32),
                                  __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0u)));
      const float x = (mem & 1u) ? v[0] : ((mem & 2u) ? v[1] : ((mem & 4u) ? v[2] : v[3]));
      if ((mem != 0u) & (at < kStage)) stage[wid][at] = x;
      mem &= mem - 1u;
      staged += __popcll(m);
    }
  };
  // steps of kLongQuads 16-byte loads per thread, the next step's issued
  // before a step is taken; loads past the end read the chunk's first quad
  {
    const int len = static_cast<int>(c1 - c0);
    const int nq = len / 4;
    const float* rc = r + c0;
    auto load = [&](float4 (&q)[kLongQuads], int s) {
#pragma unroll
      for (int j = 0; j < kLongQuads; ++j) {
        const int i = (s * kLongQuads + j) * LT + tid;
        q[j] = load_quad(rc + 4 * (i < nq ? i : 0));
      }
    };
    auto take = [&](const float4 (&q)[kLongQuads], int s) {
#pragma unroll
      for (int j = 0; j < kLongQuads; ++j) {
        const int i0 = (s * kLongQuads + j) * LT;
        if (i0 < nq) {   // uniform
          const bool on = i0 + tid < nq;
          const float none = __int_as_float(0x7fc00000);
          const float v[4] = {on ? q[j].x : none, on ? q[j].y : none, on ? q[j].z : none,
                              on ? q[j].w : none};
          take4(v);
        }
      }
    };
    const int steps = (nq + kLongQuads * LT - 1) / (kLongQuads * LT);
    if (steps > 0) {
      float4 qa[kLongQuads], qb[kLongQuads];
      load(qa, 0);
      for (int s = 0;; s += 2) {
        if (s + 1 < steps) load(qb, s + 1);
        take(qa, s);
        if (s + 1 >= steps) break;
        if (s + 2 < steps) load(qa, s + 2);
        take(qb, s + 1);
        if (s + 2 >= steps) break;
      }
    }
    if (wid == 0 && 4 * nq < len) {   // the row's last one to three scores
      const int i = 4 * nq + lane;
      const float none = __int_as_float(0x7fc00000);
      const float v[4] = {i < len ? rc[i] : none, none, none, none};
      take4(v);
    }
  }
  TR = wave_sum(TR);
  TL = wave_sum(TL);
  nR = wave_sum(nR);
  if (lane == 0) {
    red[0][wid] = TR;
    red[1][wid] = TL;
    rn[wid] = nR;
    over_s[wid] = staged > kStage ? 1u : 0u;
  }
  __syncthreads();
  bool over = false;
#pragma unroll
  for (int i = 0; i < LW; ++i) over = over || over_s[i] != 0u;
  const int fbits = 62 - (64 - __clzll(static_cast<long long>(chunk)));
  const double fscale = ldexp(1.0, fbits);
  auto terms = [&](float v, int c, unsigned long long& U, unsigned long long& D) {
    const double vd = v;
    U = __double2ull_rn(exp2_neg(fmin(vd - edge[c], 0.0) * c2) * fscale);
    D = __double2ull_rn(exp2_neg(fmin(edge[c + 1] - vd, 0.0) * c2) * fscale);
  };
  auto add = [&](float v, int c, uint32_t cnt, unsigned long long U, unsigned long long D) {
    const uint32_t key = desc_key(v + 0.0f);   // (one zero)
    atomicMin(&kmin[c], key);
    atomicMax(&kmax[c], key);
    if (U) atomicAdd(&cu[c], U * cnt);
    if (D) atomicAdd(&cd[c], D * cnt);
    return atomicAdd(&cn[c], cnt);
  };
  constexpr int PER = kStage / kWave;
  float mv[PER];
  int mc[PER];
  uint32_t mr[PER];
  if (!over) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      mc[i] = -1;
      if (i * kWave < staged) {   // wave-uniform
        const int at = i * kWave + lane;
        if (at < staged) {
          mv[i] = stage[wid][at];
          mc[i] = cell_at<NC>(w, edge, mv[i]);
          unsigned long long U, D;
          terms(mv[i], mc[i], U, D);
          mr[i] = add(mv[i], mc[i], 1u, U, D);
        }
      }
    }
  } else {
    for (int64_t b = c0; b < c1; b += LT) {   // every lane of a wave takes part
      const int64_t at = b + tid;
      const float v = at < c1 ? r[at] : 0.0f;
      bool in = at < c1 && v < w.xhi && v >= w.xlo;
      // up to four groups of equal members of the wave are added once each
      for (int q = 0; q < 4; ++q) {
        const uint64_t m = __ballot(in);
        if (m == 0ull) break;
        const float v0 = readlane_as(v, __ffsll(static_cast<long long>(m)) - 1);
        const uint64_t eq = __ballot(in && v == v0);
        if (lane == __ffsll(static_cast<long long>(m)) - 1) {
          const int c = cell_at<NC>(w, edge, v);
          unsigned long long U, D;
          terms(v, c, U, D);
          add(v, c, static_cast<uint32_t>(__popcll(eq)), U, D);
        }
        in = in && v != v0;
      }
      if (in) {
        const int c = cell_at<NC>(w, edge, v);
        unsigned long long U, D;
        terms(v, c, U, D);
        add(v, c, 1u, U, D);
      }
    }
  }
  __syncthreads();
  const int64_t slot = row * G + g;
  // entries per cell (one for equal members), their offsets, and the cells
  if (wid == 0) {
    uint32_t run = 0u;
    uint32_t merged = 0u;
#pragma unroll
    for (int q = 0; q < NC / kWave; ++q) {
      const int c = q * kWave + lane;
      const uint32_t cnt = cn[c];
      const bool one = cnt > 1u && kmin[c] == kmax[c];
      const uint32_t ent = one ? 1u : cnt;
      merged |= one ? 1u : 0u;
      const uint32_t incl = wave_incl_add<uint32_t>(ent);
      cur[c] = run + incl - ent;
      o.off[slot * (NC + 1) + c] = run + incl - ent;
      run += readlane_as(incl, kWave - 1);
    }
    merged = wave_or(merged);
    if (lane == 0) {
      o.off[slot * (NC + 1) + NC] = run;
      LongBlock b;
      b.TR = b.TL = 0.0;
      b.nR = 0u;
#pragma unroll
      for (int i = 0; i < LW; ++i) {
        b.TR += red[0][i];
        b.TL += red[1][i];
        b.nR += rn[i];
      }
      b.merged = merged;
      o.blk[slot] = b;
    }
  }
  const double inv_f = ldexp(1.0, -fbits);
  for (int c = tid; c < NC; c += LT) {
    o.cnt[slot * NC + c] = cn[c];
    o.U[slot * NC + c] = static_cast<double>(cu[c]) * inv_f;
    o.D[slot * NC + c] = static_cast<double>(cd[c]) * inv_f;
  }
  __syncthreads();
  float* list = o.list + (row * G + g) * chunk;
  auto single = [&](int c) { return cn[c] > 1u && kmin[c] == kmax[c]; };
  for (int c = tid; c < NC; c += LT)
    if (single(c)) list[cur[c]] = key_float(kmin[c]);
  if (!over) {
#pragma unroll
    for (int i = 0; i < PER; ++i)
      if (mc[i] >= 0 && !single(mc[i])) list[cur[mc[i]] + mr[i]] = mv[i];
  } else {
    __syncthreads();   // the single cells' offsets have been read
    for (int64_t at = c0 + tid; at < c1; at += LT) {
      const float v = r[at];
      if (v < w.xhi && v >= w.xlo) {
        const int c = cell_at<NC>(w, edge, v);
        if (!single(c)) list[atomicAdd(&cur[c], 1u)] = v;
      }
    }
  }
}

// The cells of a row of many blocks, merged by NC / 16 workgroups per row
// (16 cells each, the blocks in a fixed order);
// long_root of a shorter row merges them itself.
template <int NC>
__global__ __launch_bounds__(256) void long_merge_kernel(int G, LongCells o) {
  __shared__ double pU[16][17], pD[16][17];
  __shared__ uint32_t pc[16][17];
  const int64_t s0 = static_cast<int64_t>(blockIdx.y) * G;
  const int lc = threadIdx.x % 16, gi = threadIdx.x / 16;
  const int c = static_cast<int>(blockIdx.x) * 16 + lc;
  double su = 0.0, sd = 0.0;
  uint32_t sc = 0u;
  for (int b0 = gi; b0 < G; b0 += 16 * 8) {
    double vu[8], vd[8];
    uint32_t vc[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int bb = b0 + q * 16;
      const int64_t at = (s0 + (bb < G ? bb : b0)) * NC + c;
      vu[q] = o.U[at];
      vd[q] = o.D[at];
      vc[q] = o.cnt[at];
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      if (b0 + q * 16 < G) {
        su += vu[q];
        sd += vd[q];
        sc += vc[q];
      }
    }
  }
  pU[gi][lc] = su;
  pD[gi][lc] = sd;
  pc[gi][lc] = sc;
  __syncthreads();
  if (threadIdx.x < 16) {
    su = sd = 0.0;
    sc = 0u;
#pragma unroll
    for (int g = 0; g < 16; ++g) {
      su += pU[g][lc];
      sd += pD[g][lc];
      sc += pc[g][lc];
    }
    const int64_t at = static_cast<int64_t>(blockIdx.y) * NC + c;
    o.mU[at] = su;
    o.mD[at] = sd;
    o.mcnt[at] = sc;
  }
}

// ------------------------------------------------------------------ root ---
namespace {
// LapSum at every edge of NC cells (cn members each, the two sums U and D):
// P, the scores above an edge, and T, those below, move from edge to edge by
// the cells' links e^{-(edge(c) - edge(c+1))/t} (affine scans over the lanes of
// one wave, NC / 64 cells each).  above, TR, TL: the scores above the cells
// and the sums at their two ends.  ab[c]: members in the cells before c.
template <int NC>
__device__ void edge_sums(const uint32_t* cn, const double* U, const double* D, const double* edge,
                          double above, double TR, double TL, double c2, uint32_t* ab, double* eP,
                          double* eT, double* lap) {
  const int lane = lane_id();
  uint32_t run = 0u;
#pragma unroll
  for (int q = 0; q < NC / kWave; ++q) {
    const uint32_t v = cn[q * kWave + lane];
    const uint32_t incl = wave_incl_add<uint32_t>(v);
    ab[q * kWave + lane] = run + incl - v;
    run += readlane_as(incl, kWave - 1);
  }
  if (lane == 0) ab[NC] = run;
  constexpr int PER = NC / kWave;
  const int c0 = PER * lane;
  double lk[PER], T[PER + 1];
  double Au = 1.0, Bu = 0.0, Ad = 1.0, Bd = 0.0;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    lk[q] = exp2_neg(fmin(edge[c0 + q + 1] - edge[c0 + q], 0.0) * c2);
    Bu = fma(lk[q], Bu, D[c0 + q]);
    Au *= lk[q];
  }
#pragma unroll
  for (int q = PER - 1; q >= 0; --q) Bd = fma(lk[q], Bd, U[c0 + q]);
  Ad = Au;
  wave_affine_up(Au, Bu);
  wave_affine_down(Ad, Bd);
  double P = __shfl_up(fma(Au, TR, Bu), 1, kWave);
  if (lane == 0) P = TR;
  T[PER] = __shfl_down(fma(Ad, TL, Bd), 1, kWave);
  if (lane == kWave - 1) T[PER] = TL;
#pragma unroll
  for (int q = PER - 1; q >= 0; --q) T[q] = fma(lk[q], T[q + 1], U[c0 + q]);
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    eP[c0 + q] = P;
    eT[c0 + q] = T[q];
    lap[c0 + q] = above + static_cast<double>(ab[c0 + q]) - 0.5 * P + 0.5 * T[q];
    P = fma(lk[q], P, D[c0 + q]);
  }
  if (lane == kWave - 1) {
    eP[NC] = P;
    eT[NC] = TL;
    lap[NC] = above + static_cast<double>(ab[NC]) - 0.5 * P + 0.5 * TL;
  }
}

// js[0]: the cell holding b, the last one whose upper edge has LapSum <= k
// (cell 0 when none has); js[1], js[2]: its nearest non-empty neighbours.  One
// wave.
template <int NC>
__device__ void root_cell(const uint32_t* cn, const double* lap, double k, int* js) {
  const int lane = lane_id();
  int js_ = 0;
#pragma unroll
  for (int q = 0; q < NC / kWave; ++q) {
    const int c = q * kWave + lane;
    if (c > 0 && lap[c] <= k) js_ = c;
  }
  js_ = static_cast<int>(wave_max_u32(static_cast<uint32_t>(js_)));
  uint32_t jp = 0u, jn = NC - 1;   // (the last cell kept if none is non-empty)
#pragma unroll
  for (int q = 0; q < NC / kWave; ++q) {
    const int c = q * kWave + lane;
    if (cn[c] != 0u && c < js_) jp = static_cast<uint32_t>(c);
    if (cn[NC - 1 - c] != 0u && NC - 1 - c > js_) jn = static_cast<uint32_t>(NC - 1 - c);
  }
  jp = wave_max_u32(jp);
  jn = wave_min_u32(jn);
  if (lane == 0) {
    js[0] = js_;
    js[1] = static_cast<int>(jp);
    js[2] = static_cast<int>(jn);
  }
}

// More entries than LDS holds (each(f) over all of them): 256 cells by a
// sample of the row's scores in their range, one pass over the entries for the
// cells' sums, one to collect those of the root's cell and its neighbours in
// LDS.  A cell of equal entries is collected as one.  Two passes of 16 waves
// instead of one of four waves for each of 10 to 20 points (1e6 scores of
// which 1% are -3.4e38, k = 0.99 n, forward: 2300 -> 150 us; two passes of
// four waves 300).  (The sample is
// the row's and not the entries', whose order in a list is not always the
// same: every call takes the same cells.)
constexpr int kSub = 256;
constexpr int kSubCap = 8192;   // entries collected, then their weights
struct SubCells {
  uint32_t cn[kSub], en[kSub], kmin[kSub], kmax[kSub], ab[kSub + 1];
  uint32_t fill;
  unsigned long long cu[kSub], cd[kSub];
  double U[kSub], D[kSub], edge[kSub + 1], lap[kSub + 1], eP[kSub + 1], eT[kSub + 1];
};
static_assert(4 * (2 * kSubCap) + sizeof(SubCells) <= 4 * kRootCap, "the cells lie behind the entries");
static_assert(sort_buf_words<MT, 4>() <= kSubCap && sizeof(SortSmem<MT>) <= 4 * kSubCap, "sample");

// What is narrowed: `count` entries of the total weight, the scores outside
// them as carries, and the first point.
struct Crowd {
  uint32_t count, weight;
  Carry ext;
  float x0;
};

// top, bottom: the entries' range (infinite: open).  buf: kRootCap words;
// true: the entries are in buf[0 .. count), their weights kSubCap words behind
// them, and q says the rest; false (too many left): nothing has changed.
template <int BT, class Each>
__device__ bool divide_crowd(Each&& each, const float* __restrict__ r, int64_t n, double top,
                             double bottom, double k, double t, float* buf, int* js, Crowd& q) {
  constexpr int M = 4096;   // scores sampled, at most
  constexpr int SI = M / BT;
  uint32_t* sorted = reinterpret_cast<uint32_t*>(buf);
  SortSmem<BT>& ssm = *reinterpret_cast<SortSmem<BT>*>(buf + kSubCap);
  SubCells& S = *reinterpret_cast<SubCells*>(buf + 2 * kSubCap);
  const int tid = threadIdx.x;
  const double c2 = kLog2e / t;
  // 1. the cells' bounds: hashed positions of the row, up to 65536 of them or
  //    until 3072 scores in the range have been met, in order
  for (int c = tid; c < kSub; c += BT) {
    S.cn[c] = S.en[c] = 0u;
    S.kmin[c] = 0xffffffffu;
    S.kmax[c] = 0u;
    S.cu[c] = S.cd[c] = 0ull;
  }
  if (tid == 0) S.fill = 0u;
  __syncthreads();
  int m = 0;
  for (int i = 0; i < 64 && m <= M - BT; ++i) {
    const uint64_t h = mix32(static_cast<uint32_t>(i * BT + tid) + 0x51ed2700u);
    const float x = fminf(fmaxf(r[(h * static_cast<uint64_t>(n)) >> 32], -kMaxScore), kMaxScore);
    const bool in = x < top && x >= bottom;   // (so that no bound lies above top)
    const uint64_t b = __ballot(in);
    uint32_t at = 0u;
    if (lane_id() == 0) at = atomicAdd(&S.fill, static_cast<uint32_t>(__popcll(b)));
    at = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(at)));
    if (in) sorted[at + __popcll(b & ((1ull << lane_id()) - 1ull))] = desc_key(x + 0.0f);
    __syncthreads();
    m = static_cast<int>(S.fill);
    __syncthreads();
  }
  if (m == 0) return false;
  {
    uint32_t key[SI];
    int32_t none[SI];
#pragma unroll
    for (int i = 0; i < SI; ++i) key[i] = i * BT + tid < m ? sorted[i * BT + tid] : 0xffffffffu;
    if (tid == 0) S.fill = 0u;
    block_sort_u32<BT, SI, false>(key, none, sorted, ssm);   // (leaves the order in `sorted`)
  }
  for (int c = tid; c < kSub - 1; c += BT) {
    auto key_at = [&](int b) {
      const int i = b * m / (kSub - 2);
      return sorted[buf_at(i < m ? i : m - 1)];
    };
    const uint32_t key0 = key_at(c);
    const bool again = c < kSub - 2 && key_at(c + 1) == key0;   // (as in long_window)
    const double e = key_float(key0 - (again ? 1u : 0u));
    S.edge[c + 1] = e;
    // (an open end: the sample's own last score)
    if (c == 0) S.edge[0] = top < INFINITY ? fmax(e, top) : e;
    if (c == kSub - 2) S.edge[kSub] = bottom > -INFINITY ? fmin(e, bottom) : e;
  }
  __syncthreads();
  auto cell = [&](float v) { return cell_by_edges<kSub>(S.edge, v); };
  // 2. their sums, in fixed point
  const int fbits = 62 - (64 - __clzll(static_cast<long long>(q.weight) | 1ll));
  const double fscale = ldexp(1.0, fbits), inv_f = ldexp(1.0, -fbits);
  each([&](float v, uint32_t w) {
    const int c = cell(v);
    const double vd = v;
    const unsigned long long U = __double2ull_rn(exp2_neg(fmin(vd - S.edge[c], 0.0) * c2) * fscale);
    const unsigned long long D = __double2ull_rn(exp2_neg(fmin(S.edge[c + 1] - vd, 0.0) * c2) * fscale);
    const uint32_t kv = desc_key(v + 0.0f);
    atomicMin(&S.kmin[c], kv);
    atomicMax(&S.kmax[c], kv);
    atomicAdd(&S.cu[c], U * w);
    atomicAdd(&S.cd[c], D * w);
    atomicAdd(&S.cn[c], w);
    atomicAdd(&S.en[c], 1u);
  });
  __syncthreads();
  for (int c = tid; c < kSub; c += BT) {
    S.U[c] = static_cast<double>(S.cu[c]) * inv_f;
    S.D[c] = static_cast<double>(S.cd[c]) * inv_f;
  }
  __syncthreads();
  if (tid < kWave) {
    const Carry& x = q.ext;
    const double TR = x.pre.S * exp2_neg(fmin(S.edge[0] - static_cast<double>(x.pre.u), 0.0) * c2);
    const double TL = x.suf.T * exp2_neg(fmin(static_cast<double>(x.suf.v) - S.edge[kSub], 0.0) * c2);
    edge_sums<kSub>(S.cn, S.U, S.D, S.edge, x.rank0, TR, TL, c2, S.ab, S.eP, S.eT, S.lap);
    root_cell<kSub>(S.cn, S.lap, k, js);
  }
  __syncthreads();
  const int j = js[0], jp = js[1], jn = js[2];
  auto single = [&](int c) { return S.en[c] > 1u && S.kmin[c] == S.kmax[c]; };
  auto left_of = [&](int c) { return single(c) ? 1u : S.en[c]; };
  // (only these three of the cells jp .. jn hold entries)
  const uint32_t left = left_of(j) + (jp != j ? left_of(jp) : 0u) + (jn != j && jn != jp ? left_of(jn) : 0u);
  if (left > static_cast<uint32_t>(kSubCap)) return false;
  // 3. the entries of cells jp .. jn, everything else as carries
  uint32_t* bw = reinterpret_cast<uint32_t*>(buf) + kSubCap;
  auto keep = [&](float v, uint32_t w) {
    const uint32_t e = atomicAdd(&S.fill, 1u);
    if (e < static_cast<uint32_t>(kSubCap)) {
      buf[e] = v;
      bw[e] = w;
    }
  };
  each([&](float v, uint32_t w) {
    const int c = cell(v);
    if (c >= jp && c <= jn && !single(c)) keep(v, w);
  });
  for (int c = jp + tid; c <= jn; c += BT)
    if (single(c)) keep(key_float(S.kmin[c]), S.cn[c]);
  q.ext.rank0 += static_cast<double>(S.ab[jp]);
  if (jp > 0)
    q.ext.pre = S.eP[jp] > 0.0 ? Pre{static_cast<float>(S.edge[jp]), S.eP[jp]} : pre_empty();
  if (jn < kSub - 1)
    q.ext.suf = S.eT[jn + 1] > 0.0 ? Suf{static_cast<float>(S.edge[jn + 1]), S.eT[jn + 1]} : suf_empty();
  q.weight = S.ab[jn + 1] - S.ab[jp];
  q.x0 = static_cast<float>(0.5 * (S.edge[j] + S.edge[j + 1]));
  q.count = left;
  __syncthreads();
  return true;
}
}  // namespace

// MERGED: long_merge has run.
template <int NC, bool MERGED>
__global__ __launch_bounds__(MT) void long_root_kernel(
    const float* __restrict__ scores, int64_t n, int64_t chunk, int G, double k, double t,
    LongCells o, double* __restrict__ b_out) {
  constexpr int W = WT / kWave;
  constexpr int T0 = MT;
  constexpr int GR = MERGED ? 1 : MT / NC;   // groups of threads, each merging every GR-th block
  static_assert(NC <= WT && WT % NC == 0, "cells are spread over the threads");
  __shared__ NarrowSmem<WT> nsm;
  __shared__ __align__(16) float lv[kRootCap];
  __shared__ double pU[GR][NC], pD[GR][NC];
  __shared__ uint32_t pc[GR][NC];
  __shared__ double U[NC], D[NC];
  __shared__ uint32_t cn[NC], ab[NC + 1];   // ab[c]: members in cells before c
  __shared__ double edge[NC + 1], lap[NC + 1];
  __shared__ double eP[NC + 1], eT[NC + 1];
  __shared__ int64_t at_n[kLongMaxBlocks];   // a block's first entry of cell jp
  __shared__ uint32_t pre_n[kLongMaxBlocks + 1];
  __shared__ double red[2][W];
  __shared__ uint32_t rn[W], wt[W], mg[W];
  __shared__ int js[3];
  const int tid = threadIdx.x;
  const int lane = lane_id();
  const int wid = tid / kWave;
  const int64_t row = blockIdx.y;
  const float* r = scores + row * n;
  const Window w = o.win[row];
  const int64_t s0 = row * G;
  const double c2 = kLog2e / t;
  // 1. tails and cells over the blocks, in a fixed order
  for (int e = tid; e <= NC; e += T0) edge[e] = edge_of<NC>(w, o.bound + row * NC, e);
  if (tid < WT) {
    double TR = 0.0, TL = 0.0;
    uint32_t nR = 0u, m = 0u;
#pragma unroll
    for (int q = 0; q < kLongMaxBlocks / WT; ++q) {
      const int bb = q * WT + tid;
      const LongBlock b = o.blk[s0 + (bb < G ? bb : 0)];
      if (bb < G) {
        TR += b.TR;
        TL += b.TL;
        nR += b.nR;
        m |= b.merged;
      }
    }
    TR = wave_sum(TR);
    TL = wave_sum(TL);
    nR = wave_sum(nR);
    m = wave_or(m);
    if (lane == 0) {
      red[0][wid] = TR;
      red[1][wid] = TL;
      rn[wid] = nR;
      mg[wid] = m;
    }
  }
  if constexpr (MERGED) {
    if (tid < NC) {
      U[tid] = o.mU[row * NC + tid];
      D[tid] = o.mD[row * NC + tid];
      cn[tid] = o.mcnt[row * NC + tid];
    }
    __syncthreads();
  } else {
    const int c = tid % NC, gi = tid / NC;
    double su = 0.0, sd = 0.0;
    uint32_t sc = 0u;
    for (int b0 = gi; b0 < G; b0 += 8 * GR) {
      double vu[8], vd[8];
      uint32_t vc[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int bb = b0 + q * GR;
        const int64_t at = (s0 + (bb < G ? bb : b0)) * NC + c;
        vu[q] = o.U[at];
        vd[q] = o.D[at];
        vc[q] = o.cnt[at];
      }
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        if (b0 + q * GR < G) {
          su += vu[q];
          sd += vd[q];
          sc += vc[q];
        }
      }
    }
    pU[gi][c] = su;
    pD[gi][c] = sd;
    pc[gi][c] = sc;
    __syncthreads();
    if (tid < NC) {
      su = sd = 0.0;
      sc = 0u;
#pragma unroll 4
      for (int g = 0; g < GR; ++g) {
        su += pU[g][tid];
        sd += pD[g][tid];
        sc += pc[g][tid];
      }
      U[tid] = su;
      D[tid] = sd;
      cn[tid] = sc;
    }
    __syncthreads();
  }
  double TR = 0.0, TL = 0.0;
  uint32_t nR = 0u, merged = 0u;
#pragma unroll
  for (int i = 0; i < W; ++i) {
    TR += red[0][i];
    TL += red[1][i];
    nR += rn[i];
    merged |= mg[i];
  }
  const bool bounded_hi = w.xhi < INFINITY, bounded_lo = w.xlo > -INFINITY;
  // 2. LapSum at every edge, and the cell holding b with its neighbours
  if (wid == 0) {
    edge_sums<NC>(cn, U, D, edge, nR, TR, TL, c2, ab, eP, eT, lap);
    root_cell<NC>(cn, lap, k, js);
  }
  __syncthreads();
  const int jp = js[1], jn = js[2];
  const bool direct = !(bounded_hi && lap[0] > k) && !(bounded_lo && lap[NC] < k);
  // 3. carries: everything above cell jp and below cell jn (at cell 0 and
  //    cell NC-1 the edge is the window's own end)
  Carry ext;
  ext.rank0 = static_cast<double>(nR) + static_cast<double>(ab[jp]);
  ext.pre = eP[jp] > 0.0 ? Pre{static_cast<float>(edge[jp]), eP[jp]} : pre_empty();
  ext.suf = eT[jn + 1] > 0.0 ? Suf{static_cast<float>(edge[jn + 1]), eT[jn + 1]} : suf_empty();
  // 4. the entries of cells jp .. jn of every block
  {
    constexpr int PB = kLongMaxBlocks / WT;   // consecutive blocks per thread
    uint32_t mine[PB], loc = 0u;
#pragma unroll
    for (int q = 0; q < PB; ++q) {
      const int bb = tid * PB + q;
      mine[q] = 0u;
      if (tid < WT && bb < G) {
        const uint32_t first = o.off[(s0 + bb) * (NC + 1) + jp];
        mine[q] = o.off[(s0 + bb) * (NC + 1) + jn + 1] - first;
        at_n[bb] = (s0 + bb) * chunk + first;
      }
      loc += mine[q];
    }
    const uint32_t incl = wave_incl_add<uint32_t>(loc);
    if (lane == kWave - 1 && wid < W) wt[wid] = incl;
    __syncthreads();
    uint32_t run = incl - loc;
#pragma unroll
    for (int i = 0; i < W; ++i)
      if (i < wid) run += wt[i];
    if (tid < WT) {
#pragma unroll
      for (int q = 0; q < PB; ++q) {
        pre_n[tid * PB + q] = run;   // blocks past G hold the total
        run += mine[q];
      }
    }
    if (tid == WT - 1) pre_n[kLongMaxBlocks] = run;
  }
  __syncthreads();
  const uint32_t total = pre_n[kLongMaxBlocks];
  // entry e of them: its block, its score, and its weight (a merged cell
  // stands for its count)
  auto block_of = [&](uint32_t e) {
    int lo = 0;   // the last with pre_n[lo] <= e (blocks past G hold the total)
#pragma unroll
    for (int step = kLongMaxBlocks / 2; step > 0; step >>= 1) lo += pre_n[lo + step] <= e ? step : 0;
    return lo;
  };
  auto entry = [&](int bb, uint32_t e) { return o.list[at_n[bb] + (e - pre_n[bb])]; };
  auto weight_of = [&](int bb, float x) -> uint32_t {
    const int c = cell_at<NC>(w, edge, x);
    const uint32_t* off = o.off + (s0 + bb) * (NC + 1);
    return off[c + 1] - off[c] == 1u ? o.cnt[(s0 + bb) * NC + c] : 1u;
  };
  double b;
  if (direct && total <= static_cast<uint32_t>(merged ? kRootCap / 2 : kRootCap)) {
    if (wid >= W) return;   // one wave per SIMD from here on (ended waves
                            // take no part in the barriers below)
    uint32_t* lw = reinterpret_cast<uint32_t*>(lv) + kRootCap / 2;   // with merged cells
#pragma unroll 2
    for (uint32_t e = tid; e < total; e += WT) {
      const int bb = block_of(e);
      const float x = entry(bb, e);
      lv[e] = x;
      if (merged) lw[e] = weight_of(bb, x);
    }
    // (each thread reads back only what it wrote)
    auto each = [&](auto&& f) {
      for (uint32_t e = tid; e < total; e += WT) f(lv[e], merged ? lw[e] : 1u);
    };
    // (from the middle of the cell)
    const float x0 = static_cast<float>(0.5 * (edge[js[0]] + edge[js[0] + 1]));
    b = narrow_solve<WT>(each, total, ab[jn + 1] - ab[jp], ext, -INFINITY, INFINITY, x0, k, t, nsm);
  } else {
    // more entries than LDS holds, in the blocks' lists, or a root outside the
    // window, anywhere in the row
    enum { kOnChip, kLists, kRow };
    int from = direct ? kLists : kRow;
    int T = T0;   // threads that take part
    Crowd q;
    q.count = direct ? total : static_cast<uint32_t>(n);
    q.weight = direct ? ab[jn + 1] - ab[jp] : static_cast<uint32_t>(n);
    q.ext = direct ? ext : Carry{0.0, pre_empty(), suf_empty()};
    q.x0 = direct ? static_cast<float>(0.5 * (edge[js[0]] + edge[js[0] + 1])) : w.x0;
    auto each = [&](auto&& f) {
      if (from == kOnChip) {
        const uint32_t* lw = reinterpret_cast<const uint32_t*>(lv) + kSubCap;
        for (uint32_t e = tid; e < q.count; e += T) f(lv[e], lw[e]);
      } else if (from == kLists) {
        for (uint32_t e0 = 0u; e0 < total; e0 += 4 * T) {
          float x[4];
          uint32_t xw[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const uint32_t e = e0 + i * T + tid;
            const uint32_t ee = e < total ? e : 0u;
            const int bb = block_of(ee);
            x[i] = entry(bb, ee);
            xw[i] = merged ? weight_of(bb, x[i]) : 1u;
          }
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (e0 + i * T + tid < total) f(x[i], xw[i]);
        }
      } else {
        for (int64_t i0 = 0; i0 < n; i0 += 4 * T) {
          float x[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) x[i] = r[i0 + i * T + tid < n ? i0 + i * T + tid : 0];
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (i0 + i * T + tid < n) f(x[i], 1u);
        }
      }
    };
    // (a first or last cell that is not bounded has no end)
    const double top = direct && (jp > 0 || bounded_hi) ? edge[jp] : INFINITY;
    const double bottom = direct && (jn < NC - 1 || bounded_lo) ? edge[jn + 1] : -INFINITY;
    if (divide_crowd<T0>(each, r, n, top, bottom, k, t, lv, js, q)) from = kOnChip;
    if (wid >= W) return;
    T = WT;
    b = narrow_solve<WT>(each, q.count, q.weight, q.ext, -INFINITY, INFINITY, q.x0, k, t, nsm);
  }
  if (tid == 0) b_out[row] = b;
}

// --------------------------------------------------------------- launches --
namespace {
// Rows past 2^24 scores take four times the sample, which halves the window.
// Rows past 2^18 scores take 256 cells and the separate merge (a window can
// hold several percent of the row, of which long_root takes three cells: at
// 2^20 with 64 cells up to 2900 members, 35 us of narrowing instead of 12),
// and past 2^22 up to 512 blocks; shorter rows 64 cells, merged in long_root.
bool long_wide(int64_t n) { return n > (int64_t(1) << 18); }
int long_cells(int64_t n) { return long_wide(n) ? 256 : 64; }

struct LongGrid {
  int G;
  int64_t chunk;
};
// Blocks per row: one step of a block (2048 scores) up to the most blocks; a
// batch takes fewer and longer chunks per row, so that the grid stays a few
// rounds of the device and long_root has fewer blocks to merge.
LongGrid long_grid(int64_t rows, int64_t n) {
  const int64_t most = n > (int64_t(1) << 22) ? kLongMaxBlocks : kLongMaxBlocks / 2;
  int64_t cap = rows > 1 ? 768 / rows : most;
  cap = cap < 8 ? 8 : (cap > most ? most : cap);
  int64_t chunk = (n + cap - 1) / cap;
  chunk = (chunk + kLongTile - 1) / kLongTile * kLongTile;
  return LongGrid{static_cast<int>((n + chunk - 1) / chunk), chunk};
}

template <typename T>
T* carve(char* base, size_t& off, size_t count) {
  off = (off + 255) / 256 * 256;
  T* p = base ? reinterpret_cast<T*>(base + off) : nullptr;
  off += count * sizeof(T);
  return p;
}

// Laid out for `rows` rows of the grid `lg`.
LongCells long_view(void* ws, int64_t rows, const LongGrid& lg, int64_t n, size_t* bytes) {
  const size_t slots = static_cast<size_t>(rows) * static_cast<size_t>(lg.G);
  const size_t NC = static_cast<size_t>(long_cells(n));
  char* base = static_cast<char*>(ws);
  size_t off = 0;
  LongCells o;
  o.win = carve<Window>(base, off, static_cast<size_t>(rows));
  o.bound = carve<float>(base, off, static_cast<size_t>(rows) * NC);
  o.mU = carve<double>(base, off, static_cast<size_t>(rows) * NC);
  o.mD = carve<double>(base, off, static_cast<size_t>(rows) * NC);
  o.mcnt = carve<uint32_t>(base, off, static_cast<size_t>(rows) * NC);
  o.blk = carve<LongBlock>(base, off, slots);
  o.U = carve<double>(base, off, slots * NC);
  o.D = carve<double>(base, off, slots * NC);
  o.cnt = carve<uint32_t>(base, off, slots * NC);
  o.off = carve<uint32_t>(base, off, slots * (NC + 1));
  o.list = carve<float>(base, off, slots * static_cast<size_t>(lg.chunk));
  *bytes = (off + 255) / 256 * 256;
  return o;
}
}  // namespace

size_t long_solve_bytes(int64_t rows, int64_t n) {
  size_t bytes = 0;
  long_view(nullptr, rows, long_grid(rows, n), n, &bytes);
  return bytes;
}

int64_t long_rows(int64_t batch, int64_t n) {
  constexpr size_t most = size_t(48) << 20;
  int64_t rows = batch < 1024 ? batch : 1024;
  while (rows > 1 && long_solve_bytes(rows, n) > most) rows -= (rows + 15) / 16;
  return rows < 1 ? 1 : rows;
}

size_t long_group_bytes(int64_t group, int64_t rows, int64_t n) {
  const LongGrid lg = long_grid(group, n);
  // (the lists come last, and a row's follow the row's before it)
  const size_t unused = static_cast<size_t>(group - rows) * static_cast<size_t>(lg.G) *
                        static_cast<size_t>(lg.chunk) * sizeof(float);
  return long_solve_bytes(group, n) - unused;
}

hipError_t launch_long_solve(const float* scores, int64_t rows, int64_t group, int64_t n, double k,
                             double t, void* ws, size_t ws_bytes, double* b, hipStream_t s) {
  if (rows < 1 || rows > group || group > 65535 || n < 1) return hipErrorInvalidValue;
  if (long_group_bytes(group, rows, n) > ws_bytes) return hipErrorInvalidValue;
  const LongGrid lg = long_grid(group, n);
  size_t bytes = 0;
  const LongCells o = long_view(ws, group, lg, n, &bytes);
  const unsigned ry = static_cast<unsigned>(rows);
  const bool wide = long_wide(n);
  { ProfScope ps_("long_window", s);
  if (n > (int64_t(1) << 24))
    hipLaunchKernelGGL((long_window_kernel<64, 256>), dim3(1, ry), dim3(WT), 0, s, scores, n, k, t, o.win,
                       o.bound);
  else if (wide)
    hipLaunchKernelGGL((long_window_kernel<16, 256>), dim3(1, ry), dim3(WT), 0, s, scores, n, k, t, o.win,
                       o.bound);
  else
    hipLaunchKernelGGL((long_window_kernel<16, 64>), dim3(1, ry), dim3(WT), 0, s, scores, n, k, t, o.win,
                       o.bound); }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  { ProfScope ps_("long_pass", s);
  const dim3 grid(static_cast<unsigned>(lg.G), ry);
  if (wide)
    hipLaunchKernelGGL(long_pass_kernel<256>, grid, dim3(LT), 0, s, scores, n, lg.chunk, t, o);
  else
    hipLaunchKernelGGL(long_pass_kernel<64>, grid, dim3(LT), 0, s, scores, n, lg.chunk, t, o); }
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (wide) {
    ProfScope ps_("long_merge", s);
    hipLaunchKernelGGL(long_merge_kernel<256>, dim3(256 / 16, ry), dim3(256), 0, s, lg.G, o);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  { ProfScope ps_("long_root", s);
  if (wide)
    hipLaunchKernelGGL((long_root_kernel<256, true>), dim3(1, ry), dim3(MT), 0, s, scores, n,
                       lg.chunk, lg.G, k, t, o, b);
  else
    hipLaunchKernelGGL((long_root_kernel<64, false>), dim3(1, ry), dim3(MT), 0, s, scores, n,
                       lg.chunk, lg.G, k, t, o, b); }
  return hipGetLastError();
}

}  // namespace lapsum
