// Hard top-k mask straight from the scores (the forward of the straight-
// through estimator): m_i = 1 for the k largest of the row in the order of
// the sort's keys, equal keys by index, without sorting the row.
//
// A radix select on the order-preserving key: the digits of the k-th smallest
// descending key (11, 11 and 10 bits, the largest first) from histograms of
// the keys that share the digits before.  Integers only, so every layout of
// the row costs about the same and infinities (masked scores), the lowest
// float and zeros of both signs take their place in the order.  (A threshold
// search on values costs less where the scores are bell-shaped, and
// milliseconds where half of them are one value or -inf.)
//
//   n <= 1024     one wave per row, the keys in registers: the key bit by bit
//                 from counts over the wave, no LDS and no barriers
//   n <= 32768    one workgroup per row, the keys in registers, histograms in
//                 LDS
//   longer        four launches, one row per grid.y:
//                 select_hist    histogram of the first digit
//                 select_gather  every block finds the first digit; histogram
//                                of the second, and the keys that share the
//                                first are kept per block
//                 select_last    the second digit; histogram of the third over
//                                the kept keys only, in total and per block
//                 select_write   the third digit, and the mask: equal keys cut
//                                by the budget are counted across the blocks
//                                before from their histograms
//
// Bound: the row read three times and the mask written (4 B/score each), and
// for rows in the caches the launches (hard_topk_mask of one row of 2^17 or
// 1e6 scores 27 us, of 8e6 37-49 us; with 30% of the scores -3.4e38, 28, 27
// and 47-67 us; through the sort with indices 72, 101 and 357 us; as the
// threshold of a vanishing temperature 45, 56 and 102-169 us, and with the
// masked scores 1.4, 11 and 180 ms).  Equal scores share an LDS counter: 64
// rows of 20000 take 15 us, with 90% of each equal 27-65.
#include "kernels.hpp"
#include "common.hpp"

namespace lapsum {

namespace {
constexpr int kBins = 2048;            // first and second digit, 11 bits each
constexpr int kLastBins = 1024;        // third digit, 10 bits
constexpr int kShift1 = 21, kShift2 = 10;

// Histogram bin that holds the kk-th key (kk from 1, at most the total), and
// how many keys lie in the bins before it.
struct Digit {
  uint32_t d, below;
};
struct DigitSmem {
  uint32_t wsum[16];
  Digit out;
};

template <int T, int BINS>
__device__ __forceinline__ Digit find_digit(const uint32_t* bins, uint32_t kk, DigitSmem& sm) {
  constexpr int B = BINS / T;
  static_assert(B * T == BINS && T / kWave <= 16, "bins per thread");
  const int tid = threadIdx.x;
  uint32_t v[B], s = 0u;
#pragma unroll
  for (int q = 0; q < B; ++q) {
    v[q] = bins[B * tid + q];
    s += v[q];
  }
  const uint32_t incl = wave_incl_add<uint32_t>(s);
  if (lane_id() == kWave - 1) sm.wsum[tid / kWave] = incl;
  __syncthreads();
  uint32_t run = incl - s;
#pragma unroll
  for (int w = 0; w < T / kWave; ++w)
    if (w < tid / kWave) run += sm.wsum[w];
  if (run < kk && kk <= run + s) {
    bool found = false;
#pragma unroll
    for (int q = 0; q < B; ++q) {
      if (!found && kk <= run + v[q]) {
        sm.out = Digit{static_cast<uint32_t>(B * tid + q), run};
        found = true;
      }
      run += v[q];
    }
  }
  __syncthreads();
  return sm.out;
}
}  // namespace

// ------------------------------------------------------------ short rows ---
namespace {
constexpr int RT = 256;
constexpr int RW = RT / kWave;   // rows per workgroup
constexpr int64_t kWaveRowMax = 1024;
}  // namespace

// Lane l holds scores l, l + 64, ...: the largest key with fewer than k keys
// below it, one bit at a time.
template <int ITEMS>
__global__ __launch_bounds__(RT) void mask_wave_kernel(const float* __restrict__ scores,
                                                       int64_t batch, int n, uint32_t k,
                                                       float* __restrict__ masks) {
  const int lane = lane_id();
  const int64_t row = static_cast<int64_t>(blockIdx.x) * RW + threadIdx.x / kWave;
  if (row >= batch) return;   // (whole waves; no barrier below)
  const float* r = scores + row * n;
  uint32_t key[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const int at = i * kWave + lane;
    key[i] = desc_key(r[at < n ? at : 0]);
  }
#pragma unroll
  for (int i = 0; i < ITEMS; ++i)
    if (i * kWave + lane >= n) key[i] = 0xffffffffu;   // past the row: after every score
  uint32_t K = 0u, below = 0u;
  for (int bit = 31; bit >= 0; --bit) {
    const uint32_t cand = K | (1u << bit);
    uint32_t c = 0u;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) c += static_cast<uint32_t>(__popcll(__ballot(key[i] < cand)));
    if (c < k) {
      K = cand;
      below = c;
    }
  }
  // (below counts the keys below K: the last candidate taken is K itself, or
  // K = 0 with none below)
  uint32_t seen = 0u;
  const uint32_t need = k - below;
  const uint64_t before = (1ull << lane) - 1ull;
  float* mask = masks + row * n;
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const int at = i * kWave + lane;
    const uint64_t eq = __ballot(key[i] == K);
    const uint32_t rank = seen + static_cast<uint32_t>(__popcll(eq & before));
    seen += static_cast<uint32_t>(__popcll(eq));
    if (at < n) mask[at] = (key[i] < K || (key[i] == K && rank < need)) ? 1.0f : 0.0f;
  }
}

// ---------------------------------------------------------- rows on chip ---
// Item i of thread tid is score tid + T i.
template <int T, int ITEMS>
__global__ __launch_bounds__(T) void mask_row_kernel(const float* __restrict__ scores, int n,
                                                     uint32_t k, float* __restrict__ masks) {
  constexpr int W = T / kWave;
  __shared__ uint32_t bins[kBins];
  __shared__ DigitSmem sm;
  __shared__ uint32_t wc[ITEMS][W];
  const int tid = threadIdx.x;
  const int lane = lane_id();
  const int wid = tid / kWave;
  const float* r = scores + static_cast<int64_t>(blockIdx.x) * n;
  float* mask = masks + static_cast<int64_t>(blockIdx.x) * n;
  uint32_t key[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const int e = tid + T * i;
    key[i] = desc_key(r[e < n ? e : 0]);
  }
  uint32_t kk = k, prefix = 0u, eq = 0u;
#pragma unroll
  for (int pass = 0; pass < 3; ++pass) {
    const int shift = pass == 0 ? kShift1 : (pass == 1 ? kShift2 : 0);
    const int above = pass == 0 ? 32 : (pass == 1 ? kShift1 : kShift2);
    const uint32_t dmask = pass == 2 ? kLastBins - 1 : kBins - 1;
    for (int e = tid; e < kBins; e += T) bins[e] = 0u;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
      if (tid + T * i < n && (pass == 0 || (key[i] >> (above & 31)) == prefix))
        atomicAdd(&bins[(key[i] >> shift) & dmask], 1u);
    __syncthreads();
    const Digit g = find_digit<T, kBins>(bins, kk, sm);
    kk -= g.below;
    prefix = pass == 2 ? (prefix << 10) | g.d : (prefix << 11) | g.d;
    eq = bins[g.d];
    __syncthreads();   // the bins and the digit have been read
  }
  const uint32_t K = prefix;
  if (kk == eq) {   // every key equal to the k-th is wanted
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
      if (tid + T * i < n) mask[tid + T * i] = key[i] <= K ? 1.0f : 0.0f;
    return;
  }
  uint64_t me[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    me[i] = __ballot(tid + T * i < n && key[i] == K);
    if (lane == 0) wc[i][wid] = static_cast<uint32_t>(__popcll(me[i]));
  }
  __syncthreads();
  const uint64_t before = (1ull << lane) - 1ull;
  uint32_t seen = 0u;
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    uint32_t rank = seen + static_cast<uint32_t>(__popcll(me[i] & before));
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const uint32_t c = wc[i][w];
      if (w < wid) rank += c;
      seen += c;
    }
    if (tid + T * i < n)
      mask[tid + T * i] = (key[i] < K || (key[i] == K && rank < kk)) ? 1.0f : 0.0f;
  }
}

// ------------------------------------------------------------- long rows ---
namespace {
constexpr int HT = 512;
constexpr int HW = HT / kWave;
constexpr int HI = 8;                                          // scores per thread and tile
constexpr int64_t kMaskTile = static_cast<int64_t>(HT) * HI;   // 4096
constexpr int kQuads = 4;                                      // 16-byte loads in flight per thread

// What the launches of a group of rows share.
struct Select {
  uint32_t* hist;     // [rows][kBins + kBins + kLastBins], zero before select_hist
  Digit* first;       // [rows] the first digit, and the keys before it
  Digit* second;      // [rows] the first two digits, and the keys before them
  uint32_t* cnt;      // [rows][G] keys kept per block
  uint32_t* bhist;    // [rows][G][kLastBins] the third digit's histogram per block
  uint32_t* list;     // [rows][G][chunk] keys kept
};
constexpr int64_t kHistWords = 2 * kBins + kLastBins;

struct SelectGrid {
  int G;
  int64_t chunk;
};
// Blocks per row for groups of `rows` rows: tiles of 4096 up to 512 blocks of
// one row, fewer and longer chunks per row in a batch (a few rounds of the
// device in all).
SelectGrid select_grid(int64_t rows, int64_t n) {
  int64_t cap = 1024 / rows;
  cap = cap < 4 ? 4 : (cap > 512 ? 512 : cap);
  int64_t chunk = (n + cap - 1) / cap;
  chunk = (chunk + kMaskTile - 1) / kMaskTile * kMaskTile;
  return SelectGrid{static_cast<int>((n + chunk - 1) / chunk), chunk};
}

// f(x0, x1, x2, x3, on) for the quads of [c0, c1), on = false in lanes past
// the last, then g(x, on) for the up to three scores after them (wave 0).
template <class F, class G>
__device__ __forceinline__ void stream_chunk(const float* __restrict__ rc, int64_t len, F&& f, G&& g) {
  const int64_t nq = len / 4;
  const int tid = threadIdx.x;
  for (int64_t q0 = 0; q0 < nq; q0 += kQuads * HT) {
    float4 x[kQuads];
#pragma unroll
    for (int j = 0; j < kQuads; ++j) {
      const int64_t i = q0 + j * HT + tid;
      x[j] = load_quad(rc + 4 * (i < nq ? i : 0));
    }
#pragma unroll
    for (int j = 0; j < kQuads; ++j) f(x[j], q0 + j * HT + tid < nq);
  }
  if (tid < kWave && 4 * nq < len) {
    const int64_t i = 4 * nq + tid;
    g(rc[i < len ? i : 4 * nq], i < len);
  }
}
}  // namespace

__global__ __launch_bounds__(HT) void select_hist_kernel(const float* __restrict__ scores, int64_t n,
                                                         int64_t chunk, Select o) {
  __shared__ uint32_t bins[kBins];
  const int tid = threadIdx.x;
  const int64_t row = blockIdx.y;
  const int64_t c0 = static_cast<int64_t>(blockIdx.x) * chunk;
  const int64_t len = c0 + chunk < n ? chunk : n - c0;
  for (int e = tid; e < kBins; e += HT) bins[e] = 0u;
  __syncthreads();
  auto take = [&](float x) { atomicAdd(&bins[desc_key(x) >> kShift1], 1u); };
  stream_chunk(
      scores + row * n + c0, len,
      [&](const float4& x, bool on) {
        if (on) {
          take(x.x);
          take(x.y);
          take(x.z);
          take(x.w);
        }
      },
      [&](float x, bool on) {
        if (on) take(x);
      });
  __syncthreads();
  uint32_t* hist = o.hist + row * kHistWords;
  for (int e = tid; e < kBins; e += HT)
    if (bins[e]) atomicAdd(&hist[e], bins[e]);
}

__global__ __launch_bounds__(HT) void select_gather_kernel(const float* __restrict__ scores,
                                                           int64_t n, int64_t chunk, uint32_t k,
                                                           Select o) {
  __shared__ uint32_t bins[kBins];
  __shared__ DigitSmem sm;
  __shared__ uint32_t fill;
  const int tid = threadIdx.x;
  const int lane = lane_id();
  const int64_t row = blockIdx.y;
  const int64_t slot = row * gridDim.x + blockIdx.x;
  const int64_t c0 = static_cast<int64_t>(blockIdx.x) * chunk;
  const int64_t len = c0 + chunk < n ? chunk : n - c0;
  uint32_t* hist = o.hist + row * kHistWords;
  const Digit one = find_digit<HT, kBins>(hist, k, sm);
  if (tid == 0) {
    fill = 0u;
    if (blockIdx.x == 0) o.first[row] = one;
  }
  for (int e = tid; e < kBins; e += HT) bins[e] = 0u;
  __syncthreads();
  uint32_t* list = o.list + slot * chunk;   // (at most len keys)
  // the lanes of a wave together: room for all of them, then each lane's own
  auto keep = [&](uint32_t key, bool in, uint32_t at) {
    if (in) {
      atomicAdd(&bins[(key >> kShift2) & (kBins - 1)], 1u);
      list[at] = key;
    }
  };
  const uint64_t before = (1ull << lane) - 1ull;
  auto rank = [&](uint64_t m) { return static_cast<uint32_t>(__popcll(m & before)); };
  auto room = [&](uint32_t total) {
    uint32_t at = 0u;
    if (lane == 0) at = atomicAdd(&fill, total);
    return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(at)));
  };
  stream_chunk(
      scores + row * n + c0, len,
      [&](const float4& x, bool on) {
        const uint32_t key[4] = {desc_key(x.x), desc_key(x.y), desc_key(x.z), desc_key(x.w)};
        bool in[4];
        uint64_t m[4];
        uint32_t total = 0u;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          in[e] = on && (key[e] >> kShift1) == one.d;
          m[e] = __ballot(in[e]);
          total += static_cast<uint32_t>(__popcll(m[e]));
        }
        if (total == 0u) return;   // wave-uniform
        uint32_t at = room(total);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          keep(key[e], in[e], at + rank(m[e]));
          at += static_cast<uint32_t>(__popcll(m[e]));
        }
      },
      [&](float x, bool on) {
        const uint32_t key = desc_key(x);
        const bool in = on && (key >> kShift1) == one.d;
        const uint64_t m = __ballot(in);
        if (m != 0ull) keep(key, in, room(static_cast<uint32_t>(__popcll(m))) + rank(m));
      });
  __syncthreads();
  if (tid == 0) o.cnt[slot] = fill;
  for (int e = tid; e < kBins; e += HT)
    if (bins[e]) atomicAdd(&hist[kBins + e], bins[e]);
}

__global__ __launch_bounds__(HT) void select_last_kernel(int64_t chunk, uint32_t k, Select o) {
  __shared__ uint32_t bins[kLastBins];
  __shared__ DigitSmem sm;
  const int tid = threadIdx.x;
  const int64_t row = blockIdx.y;
  const int64_t slot = row * gridDim.x + blockIdx.x;
  uint32_t* hist = o.hist + row * kHistWords;
  const Digit one = o.first[row];
  const Digit two = find_digit<HT, kBins>(hist + kBins, k - one.below, sm);
  const uint32_t prefix = (one.d << 11) | two.d;
  if (tid == 0 && blockIdx.x == 0) o.second[row] = Digit{prefix, one.below + two.below};
  for (int e = tid; e < kLastBins; e += HT) bins[e] = 0u;
  __syncthreads();
  const uint32_t* list = o.list + slot * chunk;
  const uint32_t cnt = o.cnt[slot];
  for (uint32_t i = tid; i < cnt; i += HT) {
    const uint32_t key = list[i];
    if ((key >> kShift2) == prefix) atomicAdd(&bins[key & (kLastBins - 1)], 1u);
  }
  __syncthreads();
  for (int e = tid; e < kLastBins; e += HT) {
    o.bhist[slot * kLastBins + e] = bins[e];
    if (bins[e]) atomicAdd(&hist[2 * kBins + e], bins[e]);
  }
}

__global__ __launch_bounds__(HT) void select_write_kernel(const float* __restrict__ scores,
                                                          int64_t n, int64_t chunk, uint32_t k,
                                                          Select o, float* __restrict__ masks) {
  __shared__ DigitSmem sm;
  __shared__ uint32_t red[HW];
  __shared__ uint32_t wc[HI][HW];
  const int tid = threadIdx.x;
  const int lane = lane_id();
  const int wid = tid / kWave;
  const int64_t row = blockIdx.y;
  const float* r = scores + row * n;
  float* mask = masks + row * n;
  const int64_t c0 = static_cast<int64_t>(blockIdx.x) * chunk;
  const int64_t c1 = c0 + chunk < n ? c0 + chunk : n;
  const uint32_t* hist = o.hist + row * kHistWords + 2 * kBins;
  const Digit two = o.second[row];
  const Digit three = find_digit<HT, kLastBins>(hist, k - two.below, sm);
  const uint32_t K = (two.d << 10) | three.d;
  const uint32_t need = k - two.below - three.below;   // equal keys wanted, by index
  if (need == hist[three.d]) {                         // all of them
    const int64_t nq = (c1 - c0) / 4;
    auto on = [&](float x) { return desc_key(x) <= K ? 1.0f : 0.0f; };
    for (int64_t q = tid; q < nq; q += HT) {
      const float4 x = load_quad(r + c0 + 4 * q);
      store_quad(mask + c0 + 4 * q, make_float4(on(x.x), on(x.y), on(x.z), on(x.w)));
    }
    for (int64_t i = c0 + 4 * nq + tid; i < c1; i += HT) mask[i] = on(r[i]);
    return;
  }
  // equal keys in the blocks before this one
  uint32_t seen = 0u;
  const uint32_t* bh = o.bhist + row * gridDim.x * kLastBins + three.d;
  for (uint32_t b = tid; b < blockIdx.x; b += HT) seen += bh[static_cast<int64_t>(b) * kLastBins];
  seen = wave_sum(seen);
  if (lane == 0) red[wid] = seen;
  __syncthreads();
  seen = 0u;
#pragma unroll
  for (int w = 0; w < HW; ++w) seen += red[w];
  const uint64_t before = (1ull << lane) - 1ull;
  for (int64_t base = c0; base < c1; base += kMaskTile) {
    uint32_t key[HI];
    uint64_t me[HI];
#pragma unroll
    for (int j = 0; j < HI; ++j) {
      const int64_t at = base + j * HT + tid;
      key[j] = desc_key(r[at < c1 ? at : c0]);
    }
#pragma unroll
    for (int j = 0; j < HI; ++j) {
      me[j] = __ballot(base + j * HT + tid < c1 && key[j] == K);
      if (lane == 0) wc[j][wid] = static_cast<uint32_t>(__popcll(me[j]));
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < HI; ++j) {
      uint32_t rank = seen + static_cast<uint32_t>(__popcll(me[j] & before));
#pragma unroll
      for (int w = 0; w < HW; ++w) {
        const uint32_t c = wc[j][w];
        if (w < wid) rank += c;
        seen += c;
      }
      const int64_t at = base + j * HT + tid;
      if (at < c1) mask[at] = (key[j] < K || (key[j] == K && rank < need)) ? 1.0f : 0.0f;
    }
    __syncthreads();
  }
}

// --------------------------------------------------------------- launches --
namespace {
template <typename T>
T* carve(char* base, size_t& off, size_t count) {
  off = (off + 255) / 256 * 256;
  T* p = base ? reinterpret_cast<T*>(base + off) : nullptr;
  off += count * sizeof(T);
  return p;
}

Select select_view(void* ws, int64_t rows, int64_t n, size_t* bytes) {
  const SelectGrid g = select_grid(rows, n);
  const size_t slots = static_cast<size_t>(rows) * static_cast<size_t>(g.G);
  char* base = static_cast<char*>(ws);
  size_t off = 0;
  Select o;
  o.hist = carve<uint32_t>(base, off, static_cast<size_t>(rows) * kHistWords);
  o.first = carve<Digit>(base, off, static_cast<size_t>(rows));
  o.second = carve<Digit>(base, off, static_cast<size_t>(rows));
  o.cnt = carve<uint32_t>(base, off, slots);
  o.bhist = carve<uint32_t>(base, off, slots * kLastBins);
  o.list = carve<uint32_t>(base, off, slots * static_cast<size_t>(g.chunk));
  *bytes = (off + 255) / 256 * 256;
  return o;
}

size_t select_bytes(int64_t rows, int64_t n) {
  size_t bytes = 0;
  select_view(nullptr, rows, n, &bytes);
  return bytes;
}

// Long rows taken by one set of launches: as many as fit in 48 MiB of
// workspace, one row always.  Every group of a batch, the last one too, is
// laid out for this many rows.
int64_t select_rows(int64_t batch, int64_t n) {
  constexpr size_t most = size_t(48) << 20;
  int64_t rows = batch < 1024 ? batch : 1024;
  while (rows > 1 && select_bytes(rows, n) > most) rows -= (rows + 15) / 16;
  return rows < 1 ? 1 : rows;
}

hipError_t launch_select(const float* scores, int64_t rows, int64_t group, int64_t n, uint32_t k,
                         float* mask, void* ws, hipStream_t s) {
  size_t bytes = 0;
  const Select o = select_view(ws, group, n, &bytes);
  const SelectGrid g = select_grid(group, n);
  const dim3 grid(static_cast<unsigned>(g.G), static_cast<unsigned>(rows)), block(HT);
  hipError_t e = launch_fill_u32(o.hist, rows * kHistWords, 0u, s);
  if (e != hipSuccess) return e;
  { ProfScope ps_("select_hist", s);
  hipLaunchKernelGGL(select_hist_kernel, grid, block, 0, s, scores, n, g.chunk, o); }
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  { ProfScope ps_("select_gather", s);
  hipLaunchKernelGGL(select_gather_kernel, grid, block, 0, s, scores, n, g.chunk, k, o); }
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  { ProfScope ps_("select_last", s);
  hipLaunchKernelGGL(select_last_kernel, grid, block, 0, s, g.chunk, k, o); }
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  { ProfScope ps_("select_write", s);
  hipLaunchKernelGGL(select_write_kernel, grid, block, 0, s, scores, n, g.chunk, k, o, mask); }
  return hipGetLastError();
}
}  // namespace

size_t hard_mask_bytes(int64_t batch, int64_t n) {
  // (rows on chip need none; a call has always been given some)
  if (n <= kRowOnChipMax) return 256;
  return select_bytes(select_rows(batch, n), n);
}

hipError_t launch_hard_mask(const float* scores, int64_t batch, int64_t n, int64_t k, float* mask,
                            void* ws, hipStream_t s) {
  if (batch < 1 || n < 1 || n > 2147483647LL || k < 1 || k > n) return hipErrorInvalidValue;
  const uint32_t ku = static_cast<uint32_t>(k);
  if (n > kRowOnChipMax) {
    const int64_t step = select_rows(batch, n);
    for (int64_t row = 0; row < batch; row += step) {
      const int64_t rows = batch - row < step ? batch - row : step;
      const hipError_t e = launch_select(scores + row * n, rows, step, n, ku, mask + row * n, ws, s);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  const int ni = static_cast<int>(n);
  constexpr int64_t kStep = int64_t(1) << 20;   // rows per launch (a grid's threads are 32-bit)
  for (int64_t row = 0; row < batch; row += kStep) {
    const int64_t rows = batch - row < kStep ? batch - row : kStep;
    const float* r = scores + row * n;
    float* m = mask + row * n;
    { ProfScope ps_("mask_row", s);
#define LAPSUM_MASKW(IT)                                                                         \
  hipLaunchKernelGGL(mask_wave_kernel<IT>, dim3(static_cast<unsigned>((rows + RW - 1) / RW)),    \
                     dim3(RT), 0, s, r, rows, ni, ku, m)
#define LAPSUM_MASKR(T, IT)                                                                      \
  hipLaunchKernelGGL((mask_row_kernel<T, IT>), dim3(static_cast<unsigned>(rows)), dim3(T), 0, s, \
                     r, ni, ku, m)
    if (n <= 64) {
      LAPSUM_MASKW(1);
    } else if (n <= 256) {
      LAPSUM_MASKW(4);
    } else if (n <= 512) {
      LAPSUM_MASKW(8);
    } else if (n <= kWaveRowMax) {
      LAPSUM_MASKW(16);
    } else if (n <= 2048) {
      LAPSUM_MASKR(256, 8);
    } else if (n <= 4096) {
      LAPSUM_MASKR(256, 16);
    } else if (n <= 8192) {
      LAPSUM_MASKR(1024, 8);
    } else if (n <= 16384) {
      LAPSUM_MASKR(1024, 16);
    } else {
      LAPSUM_MASKR(1024, 32);
    }
#undef LAPSUM_MASKW
#undef LAPSUM_MASKR
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace lapsum
