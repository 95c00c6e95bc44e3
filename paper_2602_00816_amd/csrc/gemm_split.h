// Split contractions and two products per launch, shared by the fp32 and bf16 GEMM kernels.
//
// A launch takes one or two products of the same shape and layouts (the mean
// and the half-difference channel of a linear layer: one and two operand
// pairs).  A product's contraction is a run of slices over its pairs, one
// after the other; where the output tiles alone do not fill the chip it is cut
// into parts of job.len slices, one workgroup each, whose fp32 results go to
// the scratch and are added in part order (fp64 sums) by reduce_splits, which
// also applies the epilogue.  With parts of equal length the one-pair product
// gets half as many as the two-pair one, and all workgroups take equal time.
#pragma once
#include "gemm.h"

namespace fdh {

struct GemmPlan {
  int len = 0;              // slices per part
  int splits[2] = {1, 1};   // parts of each product
  size_t bytes = 0;         // scratch
  double us = 0.0;          // estimated time
};

struct GemmJob {
  GemmArgs g[2];
  int nblk0 = 0;            // workgroups of the first product
  int len = 0;
  int splits[2] = {1, 1};
  float* part[2] = {nullptr, nullptr};
};

// cost model of one kernel variant (microseconds; see the plan functions)
struct GemmCost {
  int BM, BN, KT;
  double slice;             // one slice of one tile on a CU that is kept busy
  double alone;             // the same when the CU holds one workgroup
  double fixed;             // prologue and epilogue of a workgroup
  int per_cu;               // workgroups resident on a CU
  int longest;              // most slices in a part, for the accuracy of its sum (0: no limit)
};

GemmPlan plan_splits(const GemmArgs* g, int n, const GemmCost& c, size_t scratch);

// fills the launch description; returns the number of workgroups
int make_job(GemmJob& j, const GemmArgs* g, int n, const GemmPlan& pl, const GemmCost& c, float* scratch);

// adds the parts of every product that was cut, with its epilogue
template <typename T>
hipError_t reduce_splits(const GemmJob& j, int n, hipStream_t s);

#ifdef __HIPCC__
// accumulator block (rb, cb) of part `row` (part * nbatch + batch entry) of product prod
template <typename ACC>
__device__ inline void store_partial(const GemmJob& j, int prod, const ACC& acc, int part, int rb, int cb, int lane) {
  const int M = j.g[prod].M, N = j.g[prod].N;
  const int row = rb + (lane & 31);
  if (row >= M) return;
  float* p = j.part[prod] + ((int64_t)part * M + row) * N;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int col = cb + 8 * g + 4 * (lane >> 5);
    if (col < N) *reinterpret_cast<float4*>(p + col) = make_float4(acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]);
  }
}
#endif

}  // namespace fdh
