// Planning and summation of split contractions (gemm_split.h).
#include <algorithm>
#include <cmath>

#include "gemm_dev.h"
#include "gemm_split.h"

namespace fdh {

// Picks the part length that gives the shortest estimated launch: rounds of
// workgroups over the 256 CUs, each `len` slices and a fixed cost, and the
// write and read of the parts (which mostly stay in the caches behind the
// L2s, about 6 TB/s) with the summation's own launch.  Causal products are
// never cut (their tiles differ in length and come in large batches), nor
// outputs that the summation cannot take as aligned vectors of four.
// Contractions longer than c.longest slices are cut into parts of at most that
// length whatever the estimate says, in as many as that takes; where the scratch
// does not hold so many, the estimate decides among those that it holds.  Up to
// 32 parts are tried for time alone.  (fp32 product with a 128,256-word head, 512
// tokens of 512 columns: 11.1 ms with the head's input gradient whole, 4.5 cut.)
GemmPlan plan_splits(const GemmArgs* g, int n, const GemmCost& c, size_t scratch) {
  const int64_t tiles = (int64_t)ceil_div(g[0].M, c.BM) * ceil_div(g[0].N, c.BN) * g[0].nbatch;
  const int nkt = (g[0].K + c.KT - 1) / c.KT;
  // (rows in whole tiles of 128: one plan for every M of a tile count)
  const size_t out = (size_t)ceil_div(g[0].M, 128) * 128 * g[0].N * g[0].nbatch * 4;
  int tot[2] = {0, 0}, top = 0;
  bool cut = scratch > 0;
  for (int p = 0; p < n; ++p) {
    tot[p] = nkt * g[p].npairs;
    top = std::max(top, tot[p]);
    const size_t ob = g[p].out_type == OUT_F32 ? 16 : 8;
    cut = cut && g[p].causal == CAUSAL_NONE && g[p].N % 4 == 0 && g[p].ldc % 4 == 0 && g[p].c_outer % 4 == 0 &&
          g[p].c_inner % 4 == 0 && (uintptr_t)g[p].C % ob == 0 && (uintptr_t)g[p].resid % 16 == 0;
  }
  // a CU with one workgroup runs it at the lone rate, one with several (or a
  // full chip) at the busy rate
  const double whole_chip = 256.0 * c.per_cu;
  auto rounds_us = [&](int64_t wgs, int len) {
    const double busy = std::min(1.0, std::max(0.0, (double)wgs / whole_chip));
    const double slice = c.per_cu == 1 ? c.alone + (c.slice - c.alone) * busy : wgs <= 256 ? c.alone : c.slice;
    return (double)((wgs + 255) / 256) * len * slice + c.fixed * std::ceil((double)wgs / whole_chip);
  };
  // no cut takes less than all slices at the better rate, spread evenly
  double least = 0.0;
  for (int q = 0; q < n; ++q) least += (double)tiles * tot[q] / 256.0 * std::min(c.alone, c.slice);
  GemmPlan best;
  const int most = std::max(32, c.longest ? (top + c.longest - 1) / c.longest : 0);
  for (int k = 1; k <= most; ++k) {
    if (k > 1 && !cut) break;
    GemmPlan p;
    p.len = std::max(1, (top + k - 1) / k);
    if (k > 1 && p.len < 4) break;
    int64_t wgs = 0;
    double moved = 0.0;
    for (int q = 0; q < n; ++q) {
      p.splits[q] = std::max(1, (tot[q] + p.len - 1) / p.len);
      wgs += tiles * p.splits[q];
      if (p.splits[q] > 1) {
        p.bytes += ((size_t)p.splits[q] * out + 255) / 256 * 256;
        moved += 2.0 * p.splits[q] * (double)out;
      }
    }
    if (p.bytes > scratch) break;
    const bool best_fits = c.longest == 0 || best.len <= c.longest;
    if (k > 1 && best_fits && least + moved / 6e6 >= best.us) break;   // (moved grows with k)
    if (k == 1) {
      // every product whole (a one-pair product ends after half of its workgroup's run)
      double work = 0.0;
      for (int q = 0; q < n; ++q) work += (double)tiles * tot[q];
      p.us = std::max(rounds_us(tiles, top), work / 256.0 * c.slice + c.fixed);
    } else {
      p.us = rounds_us(wgs, p.len) + (p.bytes ? moved / 6e6 + 4.0 : 0.0);
    }
    const bool fits = c.longest == 0 || p.len <= c.longest;
    if (k == 1 || (fits && !best_fits) || (fits == best_fits && p.us < best.us)) best = p;
  }
  return best;
}

int make_job(GemmJob& j, const GemmArgs* g, int n, const GemmPlan& pl, const GemmCost& c, float* scratch) {
  const int tiles = (int)(ceil_div(g[0].M, c.BM) * ceil_div(g[0].N, c.BN)) * g[0].nbatch;
  j.len = pl.len;
  int blocks = 0;
  char* at = reinterpret_cast<char*>(scratch);
  for (int p = 0; p < n; ++p) {
    j.g[p] = g[p];
    j.splits[p] = pl.splits[p];
    blocks += tiles * pl.splits[p];
    if (p == 0) j.nblk0 = blocks;
    if (pl.splits[p] > 1) {
      j.part[p] = reinterpret_cast<float*>(at);
      at += ((size_t)pl.splits[p] * g[p].M * g[p].N * g[p].nbatch * 4 + 255) / 256 * 256;
    }
  }
  return blocks;
}

namespace {
// grid.y = product; four consecutive outputs per thread
template <typename T>
__global__ void reduce_splits_kernel(GemmJob j) {
  const int prod = blockIdx.y;
  const int ns = j.splits[prod];
  if (ns <= 1) return;
  const GemmArgs& a = j.g[prod];
  const int64_t mn = (int64_t)a.M * a.N, n4 = mn * a.nbatch / 4;
  const float4* part = reinterpret_cast<const float4*>(j.part[prod]);
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n4; i += (int64_t)gridDim.x * blockDim.x) {
    double t[4] = {0.0, 0.0, 0.0, 0.0};
    for (int s = 0; s < ns; ++s) {
      const float4 p = part[s * n4 + i];
      t[0] += p.x; t[1] += p.y; t[2] += p.z; t[3] += p.w;
    }
    const int64_t e = 4 * i;
    const int z = (int)(e / mn);
    const int r = (int)(e - z * mn);
    const int row = r / a.N, col = r - row * a.N;
    float x[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float b = 0.f;
      if (a.bias_theta) b += a.bias_theta_scale * ldf(reinterpret_cast<const T*>(a.bias_theta), col + q);
      if (a.bias_v) b += a.bias_v_scale * a.bias_v[col + q];
      x[q] = a.alpha * (float)t[q] + b;
    }
    store_quad<T>(a, x, batch_off(z, a.inner_count, a.c_outer, a.c_inner, a.c_div) + (int64_t)row * a.ldc + col);
  }
}
}  // namespace

template <typename T>
hipError_t reduce_splits(const GemmJob& j, int n, hipStream_t s) {
  if (j.splits[0] <= 1 && (n < 2 || j.splits[1] <= 1)) return hipSuccess;
  const int64_t n4 = (int64_t)j.g[0].M * j.g[0].N * j.g[0].nbatch / 4;
  hipLaunchKernelGGL(reduce_splits_kernel<T>, dim3((unsigned)std::min<int64_t>((n4 + 255) / 256, 8192), n), dim3(256), 0, s, j);
  return hipGetLastError();
}
template hipError_t reduce_splits<float>(const GemmJob&, int, hipStream_t);
template hipError_t reduce_splits<bf16_t>(const GemmJob&, int, hipStream_t);

}  // namespace fdh
