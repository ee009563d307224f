// Hard top-k mask straight from the scores (the forward of the straight-
// through estimator): m_i = 1 for the k largest of the row, equal scores by
// index, without sorting the row.
//
// The k-th largest score is the threshold of Eq. (1) in the limit t -> 0 with
// the budget k - 1/2 (LapSum there is the count above plus half the ties), so
// the row solvers find it with a temperature no two float32 scores resolve;
// b rounded to float32 is that score.  Two passes then write the mask: counts
// of larger and equal scores per block, and the mask with the blocks' counts
// before it.  Bound: 4 B/score read twice, 4 B/score written; a row of 2^20
// took 85 us through the sort with indices and the scatter.
#include "kernels.hpp"
#include "common.hpp"

namespace lapsum {

namespace {
constexpr int HT = 256;
constexpr int HW = HT / kWave;
constexpr int HI = 16;                           // scores per thread and tile
constexpr int64_t kMaskTile = static_cast<int64_t>(HT) * HI;
constexpr int kMaskBlocks = 512;                 // blocks per row

int64_t mask_chunk(int64_t n) {
  const int64_t c = (n + kMaskBlocks - 1) / kMaskBlocks;
  return (c + kMaskTile - 1) / kMaskTile * kMaskTile;
}
int mask_blocks(int64_t n) { return static_cast<int>((n + mask_chunk(n) - 1) / mask_chunk(n)); }

// Per block: scores larger than the k-th, equal to it, and equal to it with
// the larger key (-0 where the k-th is zero: +0 ranks before -0).
struct MaskCount {
  uint32_t gt, eq, late;
};
}  // namespace

__global__ __launch_bounds__(HT) void mask_count_kernel(const float* __restrict__ scores, int64_t n,
                                                        int64_t chunk, const double* __restrict__ b,
                                                        MaskCount* __restrict__ out) {
  __shared__ uint32_t red[3][HW];
  const int64_t row = blockIdx.y;
  const float* r = scores + row * n;
  const float v = static_cast<float>(b[row]);
  const int64_t c0 = static_cast<int64_t>(blockIdx.x) * chunk;
  const int64_t c1 = c0 + chunk < n ? c0 + chunk : n;
  uint32_t gt = 0u, eq = 0u, late = 0u;
  auto take = [&](float x) {
    gt += x > v ? 1u : 0u;
    const bool neg = v == 0.0f && __float_as_uint(x) == 0x80000000u;
    eq += (x == v && !neg) ? 1u : 0u;
    late += neg ? 1u : 0u;
  };
  const int64_t nq = (c1 - c0) / 4;
  for (int64_t q = threadIdx.x; q < nq; q += HT) {
    const float4 x = load_quad(r + c0 + 4 * q);
    take(x.x);
    take(x.y);
    take(x.z);
    take(x.w);
  }
  for (int64_t i = c0 + 4 * nq + threadIdx.x; i < c1; i += HT) take(r[i]);
  gt = wave_sum(gt);
  eq = wave_sum(eq);
  late = wave_sum(late);
  const int wid = threadIdx.x / kWave;
  if (lane_id() == 0) {
    red[0][wid] = gt;
    red[1][wid] = eq;
    red[2][wid] = late;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    MaskCount m{0u, 0u, 0u};
#pragma unroll
    for (int w = 0; w < HW; ++w) {
      m.gt += red[0][w];
      m.eq += red[1][w];
      m.late += red[2][w];
    }
    out[row * gridDim.x + blockIdx.x] = m;
  }
}

__global__ __launch_bounds__(HT) void mask_write_kernel(const float* __restrict__ scores, int64_t n,
                                                        int64_t chunk, int64_t k,
                                                        const double* __restrict__ b,
                                                        const MaskCount* __restrict__ counts,
                                                        float* __restrict__ masks) {
  __shared__ uint32_t red[5][HW];
  __shared__ uint32_t wc[2][HI][HW];
  const int64_t row = blockIdx.y;
  const float* r = scores + row * n;
  float* mask = masks + row * n;
  const float v = static_cast<float>(b[row]);
  const int tid = threadIdx.x;
  const int lane = lane_id();
  const int wid = tid / kWave;
  const int G = gridDim.x;
  const int g = blockIdx.x;
  // totals over the row, and the ties before this block
  uint32_t gt = 0u, eq = 0u, late = 0u, eq0 = 0u, late0 = 0u;
  for (int i = tid; i < G; i += HT) {
    const MaskCount m = counts[row * G + i];
    gt += m.gt;
    eq += m.eq;
    late += m.late;
    if (i < g) {
      eq0 += m.eq;
      late0 += m.late;
    }
  }
  gt = wave_sum(gt);
  eq = wave_sum(eq);
  late = wave_sum(late);
  eq0 = wave_sum(eq0);
  late0 = wave_sum(late0);
  if (lane == 0) {
    red[0][wid] = gt;
    red[1][wid] = eq;
    red[2][wid] = late;
    red[3][wid] = eq0;
    red[4][wid] = late0;
  }
  __syncthreads();
  gt = eq = late = eq0 = late0 = 0u;
#pragma unroll
  for (int w = 0; w < HW; ++w) {
    gt += red[0][w];
    eq += red[1][w];
    late += red[2][w];
    eq0 += red[3][w];
    late0 += red[4][w];
  }
  // ties wanted: the first `need` by index, +0 before -0
  const int64_t need_all = k - static_cast<int64_t>(gt);
  const int64_t need = need_all < static_cast<int64_t>(eq) ? need_all : static_cast<int64_t>(eq);
  const int64_t need_late = need_all - need;
  const bool plain = need == static_cast<int64_t>(eq) && need_late == static_cast<int64_t>(late);
  const int64_t c0 = static_cast<int64_t>(g) * chunk;
  const int64_t c1 = c0 + chunk < n ? c0 + chunk : n;
  if (plain) {   // every tie is wanted
    const int64_t nq = (c1 - c0) / 4;
    for (int64_t q = tid; q < nq; q += HT) {
      const float4 x = load_quad(r + c0 + 4 * q);
      store_quad(mask + c0 + 4 * q, make_float4(x.x >= v ? 1.0f : 0.0f, x.y >= v ? 1.0f : 0.0f,
                                                x.z >= v ? 1.0f : 0.0f, x.w >= v ? 1.0f : 0.0f));
    }
    for (int64_t i = c0 + 4 * nq + tid; i < c1; i += HT) mask[i] = r[i] >= v ? 1.0f : 0.0f;
    return;
  }
  int64_t seen = eq0, seen_late = late0;
  for (int64_t base = c0; base < c1; base += kMaskTile) {
    float x[HI];
    uint64_t me[HI], ml[HI];
#pragma unroll
    for (int j = 0; j < HI; ++j) {
      const int64_t at = base + j * HT + tid;
      x[j] = at < c1 ? r[at] : -INFINITY;
    }
#pragma unroll
    for (int j = 0; j < HI; ++j) {
      const bool on = base + j * HT + tid < c1;
      const bool neg = v == 0.0f && __float_as_uint(x[j]) == 0x80000000u;
      me[j] = __ballot(on && x[j] == v && !neg);
      ml[j] = __ballot(on && neg);
      if (lane == 0) {
        wc[0][j][wid] = static_cast<uint32_t>(__popcll(me[j]));
        wc[1][j][wid] = static_cast<uint32_t>(__popcll(ml[j]));
      }
    }
    __syncthreads();
    const uint64_t below = (1ull << lane) - 1ull;
    for (int j = 0; j < HI; ++j) {
      int64_t re = seen, rl = seen_late;
#pragma unroll
      for (int w = 0; w < HW; ++w) {
        const uint32_t ce = wc[0][j][w], cl = wc[1][j][w];
        if (w < wid) {
          re += ce;
          rl += cl;
        }
        seen += ce;
        seen_late += cl;
      }
      const int64_t at = base + j * HT + tid;
      if (at < c1) {
        bool on = x[j] > v;
        if ((me[j] >> lane) & 1ull) on = re + __popcll(me[j] & below) < need;
        if ((ml[j] >> lane) & 1ull) on = rl + __popcll(ml[j] & below) < need_late;
        mask[at] = on ? 1.0f : 0.0f;
      }
    }
    __syncthreads();
  }
}

size_t hard_mask_bytes(int64_t rows, int64_t n) {
  return static_cast<size_t>(rows) * static_cast<size_t>(mask_blocks(n)) * sizeof(MaskCount);
}

hipError_t launch_hard_mask(const float* scores, int64_t rows, int64_t n, int64_t k,
                            const double* b, void* counts, float* mask, hipStream_t s) {
  if (rows < 1 || rows > 65535) return hipErrorInvalidValue;
  const dim3 grid(static_cast<unsigned>(mask_blocks(n)), static_cast<unsigned>(rows)), block(HT);
  const int64_t chunk = mask_chunk(n);
  MaskCount* c = static_cast<MaskCount*>(counts);
  { ProfScope ps_("mask_count", s);
  hipLaunchKernelGGL(mask_count_kernel, grid, block, 0, s, scores, n, chunk, b, c); }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  { ProfScope ps_("mask_write", s);
  hipLaunchKernelGGL(mask_write_kernel, grid, block, 0, s, scores, n, chunk, k, b, c, mask); }
  return hipGetLastError();
}

}  // namespace lapsum
