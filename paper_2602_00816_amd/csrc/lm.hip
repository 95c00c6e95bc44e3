// Transformer kernels for the two gradient passes, run in lockstep.
//
// Every activation is carried as a pair of fp32 tensors: m = (x+ + x-)/2 and
// d = (x+ - x-)/2, where x+ and x- are the activation at theta + eps v and at
// theta - eps v.  The bilinear contractions run on MFMA (gemm.hip); every
// other operation here reconstructs the two points x+- = m +- d in fp64,
// evaluates the operation at each point in fp64, and stores the mean and half
// difference of the two results.  The half difference therefore keeps full
// relative precision however small the step eps is.
#include "kernels.h"

namespace fdh {

namespace {

constexpr int NT = 256;

unsigned grid_for(int64_t n) {
  int64_t g = (n + NT - 1) / NT;
  if (g > 262144) g = 262144;
  if (g < 1) g = 1;
  return (unsigned)g;
}

#define GRID_LOOP(i, n) for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < (n); i += (int64_t)gridDim.x * blockDim.x)

template <typename T>
__device__ inline void put_pair(PairT<T> o, int64_t i, double p, double q) {
  stf(o.m, i, (float)(0.5 * (p + q)));
  stf(o.d, i, (float)(0.5 * (p - q)));
}

template <typename T>
__global__ void cast_pair_kernel(PairT<T> o, const float* m, const float* d, int64_t n) {
  GRID_LOOP(i, n) {
    stf(o.m, i, m[i]);
    stf(o.d, i, d[i]);
  }
}

// ---- embedding ----------------------------------------------------------------
// token ids outside [0, V) are clamped so that no access leaves the tables;
// the embedding forward reports them (bad_tok[0] = 1) and the call that
// launched it turns that into an invalid-argument error
__device__ inline int clamp_tok(int t, int V) { return t < 0 ? 0 : (t >= V ? V - 1 : t); }

template <typename T>
__global__ void embed_fwd_kernel(PairF x, const int32_t* tok, int T_, int S, int dm, int V, const T* the, const float* ve,
                                 const T* thp, const float* vp, double eps, int* bad_tok) {
  const int64_t n = (int64_t)T_ * dm;
  GRID_LOOP(i, n) {
    const int t = (int)(i / dm), j = (int)(i % dm);
    const int tk = tok[t];
    if ((tk < 0 || tk >= V) && bad_tok && j == 0) bad_tok[0] = 1;
    const int64_t r = (int64_t)clamp_tok(tk, V) * dm + j;
    double xp = (double)ldf(the, r) + eps * (double)ve[r];
    double xm = (double)ldf(the, r) - eps * (double)ve[r];
    if (thp) {
      const int64_t pr = (int64_t)(t % S) * dm + j;
      xp += (double)ldf(thp, pr) + eps * (double)vp[pr];
      xm += (double)ldf(thp, pr) - eps * (double)vp[pr];
    }
    x.m[i] = (float)(0.5 * (xp + xm));
    x.d[i] = (float)(0.5 * (xp - xm));
  }
}

// ---- LayerNorm / RMSNorm ---------------------------------------------------------
// one workgroup per row
template <typename T>
__global__ __launch_bounds__(NT) void norm_fwd_kernel(PairT<T> y, const float* xm, const float* xd, int dm, bool ln,
                                                      const T* thg, const float* vg, const T* thb, const float* vb,
                                                      double eps, double neps) {
  __shared__ double sh[NT / 64];
  const int64_t row = blockIdx.x;
  const float* rm = xm + row * dm;
  const float* rd = xd + row * dm;
  double mup = 0.0, mum = 0.0;
  if (ln) {
    double sp = 0.0, sm = 0.0;
    for (int j = threadIdx.x; j < dm; j += NT) {
      sp += (double)rm[j] + (double)rd[j];
      sm += (double)rm[j] - (double)rd[j];
    }
    mup = block_sum<NT>(sp, sh) / dm;
    mum = block_sum<NT>(sm, sh) / dm;
  }
  double qp = 0.0, qm = 0.0;
  for (int j = threadIdx.x; j < dm; j += NT) {
    const double a = (double)rm[j] + (double)rd[j] - mup;
    const double b = (double)rm[j] - (double)rd[j] - mum;
    qp += a * a;
    qm += b * b;
  }
  const double rp = 1.0 / sqrt(block_sum<NT>(qp, sh) / dm + neps);
  const double rmi = 1.0 / sqrt(block_sum<NT>(qm, sh) / dm + neps);
  for (int j = threadIdx.x; j < dm; j += NT) {
    const double g = ldf(thg, j), dg = eps * (double)vg[j];
    double op = ((double)rm[j] + (double)rd[j] - mup) * rp * (g + dg);
    double om = ((double)rm[j] - (double)rd[j] - mum) * rmi * (g - dg);
    if (thb) {
      const double b = ldf(thb, j), db = eps * (double)vb[j];
      op += b + db;
      om += b - db;
    }
    put_pair(y, row * dm + j, op, om);
  }
}

template <typename T>
__device__ inline float4 ld4f(const T* p, int64_t i) {
  if constexpr (sizeof(T) == 4) {
    return *reinterpret_cast<const float4*>(p + i);
  } else {
    const uint2 u = *reinterpret_cast<const uint2*>(p + i);
    return make_float4(bf16_to_f32((bf16_t)(u.x & 0xFFFF)), bf16_to_f32((bf16_t)(u.x >> 16)),
                       bf16_to_f32((bf16_t)(u.y & 0xFFFF)), bf16_to_f32((bf16_t)(u.y >> 16)));
  }
}
template <typename T>
__device__ inline void st4f(T* p, int64_t i, float a, float b, float c, float d) {
  if constexpr (sizeof(T) == 4) {
    *reinterpret_cast<float4*>(p + i) = make_float4(a, b, c, d);
  } else {
    *reinterpret_cast<uint2*>(p + i) = make_uint2((uint32_t)f32_to_bf16(a) | ((uint32_t)f32_to_bf16(b) << 16),
                                                  (uint32_t)f32_to_bf16(c) | ((uint32_t)f32_to_bf16(d) << 16));
  }
}
__device__ inline float f4e(const float4& v, int e) { return e == 0 ? v.x : (e == 1 ? v.y : (e == 2 ? v.z : v.w)); }

// Norm forward with one wavefront per row (rows of 256 CPL columns, lane l
// at columns 256 c + 4 l), NORM_FWD_ROWS rows per workgroup: wavefront
// reductions, x reread from the caches between the passes.  Same arithmetic
// as norm_fwd_kernel.
constexpr int NORM_FWD_ROWS = 4;
// An empty statement that claims to modify the cached row values, so that the
// compiler recomputes their fp64 conversions in each pass instead of keeping
// them live (twice the registers) from the previous one.  No instruction.
template <int CPL>
__device__ inline void reload_barrier(float4 (&a)[CPL], float4 (&b)[CPL]) {
#pragma unroll
  for (int c = 0; c < CPL; ++c) {
    asm volatile("" : "+v"(a[c].x), "+v"(a[c].y), "+v"(a[c].z), "+v"(a[c].w));
    asm volatile("" : "+v"(b[c].x), "+v"(b[c].y), "+v"(b[c].z), "+v"(b[c].w));
  }
}

template <typename T, int CPL>
__global__ __launch_bounds__(NT) void norm_fwd_wave_kernel(PairT<T> y, const float* xm, const float* xd, int rows, bool ln,
                                                           const T* thg, const float* vg, const T* thb, const float* vb,
                                                           double eps, double neps) {
  constexpr int DM = 256 * CPL;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  auto ld = [](const float* p, int64_t i) { return *reinterpret_cast<const float4*>(p + i); };
  const int r0 = blockIdx.x * NORM_FWD_ROWS;
  for (int i = wave; i < NORM_FWD_ROWS; i += 4) {
    const int row = r0 + i;
    if (row >= rows) break;
    const int64_t o = (int64_t)row * DM + 4 * lane;
    // the lane's 4 CPL elements of both channels, loaded once (all loads in flight together)
    float4 xa[CPL], xb[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
      xa[c] = ld(xm, o + 256 * c);
      xb[c] = ld(xd, o + 256 * c);
    }
    double mup = 0.0, mum = 0.0;
    if (ln) {
      double sp = 0.0, sm = 0.0;
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        const float4 a = xa[c], b = xb[c];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          sp += (double)f4e(a, e) + (double)f4e(b, e);
          sm += (double)f4e(a, e) - (double)f4e(b, e);
        }
      }
      mup = wave_sum(sp) / DM;
      mum = wave_sum(sm) / DM;
    }
    // keep the fp32 values, not their fp64 conversions, live across the passes
    reload_barrier<CPL>(xa, xb);
    double qp = 0.0, qm = 0.0;
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
      const float4 a = xa[c], b = xb[c];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double p = (double)f4e(a, e) + (double)f4e(b, e) - mup;
        const double q = (double)f4e(a, e) - (double)f4e(b, e) - mum;
        qp += p * p;
        qm += q * q;
      }
    }
    const double rp = 1.0 / sqrt(wave_sum(qp) / DM + neps);
    const double rmi = 1.0 / sqrt(wave_sum(qm) / DM + neps);
    reload_barrier<CPL>(xa, xb);
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
      const int col = 256 * c + 4 * lane;
      const float4 a = xa[c], b = xb[c];
      const float4 g4 = ld4f(thg, col), v4 = ld(vg, col);
      float4 b4 = make_float4(0.f, 0.f, 0.f, 0.f), w4 = b4;
      if (thb) {
        b4 = ld4f(thb, col);
        w4 = ld(vb, col);
      }
      float om[4], od[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double g = f4e(g4, e), dg = eps * (double)f4e(v4, e);
        double op = ((double)f4e(a, e) + (double)f4e(b, e) - mup) * rp * (g + dg);
        double on = ((double)f4e(a, e) - (double)f4e(b, e) - mum) * rmi * (g - dg);
        if (thb) {
          const double bb = f4e(b4, e), db = eps * (double)f4e(w4, e);
          op += bb + db;
          on += bb - db;
        }
        om[e] = (float)(0.5 * (op + on));
        od[e] = (float)(0.5 * (op - on));
      }
      st4f(y.m, o + 256 * c, om[0], om[1], om[2], om[3]);
      st4f(y.d, o + 256 * c, od[0], od[1], od[2], od[3]);
    }
  }
}

// Sums of K values over the workgroup, the same for every thread (wavefront sums,
// then the wavefronts in order).  sh: two slots of K * waves doubles used in
// turn, so that one barrier per call is enough.
template <int NTH, int K>
__device__ inline void block_sums(double (&x)[K], double* sh, int& slot) {
  constexpr int NWV = NTH / 64;
#pragma unroll
  for (int k = 0; k < K; ++k) x[k] = wave_sum(x[k]);
  if constexpr (NWV > 1) {
    double* q = sh + slot * K * NWV;
    slot ^= 1;
    if ((threadIdx.x & 63) == 0)
#pragma unroll
      for (int k = 0; k < K; ++k) q[k * NWV + (threadIdx.x >> 6)] = x[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) {
      double t = q[k * NWV];
#pragma unroll
      for (int w = 1; w < NWV; ++w) t += q[k * NWV + w];
      x[k] = t;
    }
  }
}

// Norm backward, HBM-bound (three pairs read, one written, with its operand-type
// copy): a workgroup takes norm_bwd_rows consecutive rows one after the other,
// thread t the float4 chunks at columns 4 (t + c NTH).  The row of x and dy is
// read once into registers; both row statistics come from it (RMSNorm: sum x^2
// and sum dxhat x in one reduction, mean(dxhat xhat) = r mean(dxhat x);
// LayerNorm: the mean first, then the variance, sum dxhat and sum dxhat (x - mu)
// in one).  Each thread adds the gain terms of its columns, the LayerNorm bias
// terms (dy.d) and, with osum, the outputs' half differences (the bias gradient
// of the linear layer before this norm) over the rows in fp64 registers and
// writes them as one row of part.  2048 x 4096: 482 -> 90 us, 512 x 64: 69 -> 6 us
// (16 rows per workgroup, three passes over each before).
template <typename T, int NTH, int C, bool LN>
__global__ __launch_bounds__(NTH) void norm_bwd_kernel(PairF dx, PairT<T> dxo, const float* dresm, const float* dresd,
                                                       const float* xm, const float* xd, const float* dym,
                                                       const float* dyd, int rows, int per, int dm, const T* thg,
                                                       const float* vg, double eps, double neps, double* part, int ncol,
                                                       bool osum) {
  __shared__ double sh1[2 * 2 * (NTH / 64)], sh2[2 * 6 * (NTH / 64)];
  int slot1 = 0, slot2 = 0;
  auto ld = [](const float* p, int64_t i) { return *reinterpret_cast<const float4*>(p + i); };
  int col[C];
  bool on[C];
  float4 g4[C], v4[C];
  double sg[4 * C], sb[4 * C], so[4 * C];
  const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int c = 0; c < C; ++c) {
    col[c] = 4 * ((int)threadIdx.x + c * NTH);
    on[c] = col[c] < dm;
    g4[c] = on[c] ? ld4f(thg, col[c]) : zero;
    v4[c] = on[c] ? ld(vg, col[c]) : zero;
#pragma unroll
    for (int e = 0; e < 4; ++e) sg[4 * c + e] = sb[4 * c + e] = so[4 * c + e] = 0.0;
  }
  const int r0 = blockIdx.x * per, r1 = min(rows, r0 + per);
  for (int row = r0; row < r1; ++row) {
    const int64_t o = (int64_t)row * dm;
    float4 xa[C], xb[C], ya[C], yb[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
      xa[c] = on[c] ? ld(xm, o + col[c]) : zero;
      xb[c] = on[c] ? ld(xd, o + col[c]) : zero;
      ya[c] = on[c] ? ld(dym, o + col[c]) : zero;
      yb[c] = on[c] ? ld(dyd, o + col[c]) : zero;
    }
    double mup = 0.0, mum = 0.0, rp, rmi, a1p = 0.0, a1m = 0.0, a2p, a2m;
    if constexpr (LN) {
      double t[2] = {0.0, 0.0};
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          t[0] += (double)f4e(xa[c], e) + (double)f4e(xb[c], e);
          t[1] += (double)f4e(xa[c], e) - (double)f4e(xb[c], e);
        }
      block_sums<NTH, 2>(t, sh1, slot1);
      mup = t[0] / dm;
      mum = t[1] / dm;
    }
    {
      double t[LN ? 6 : 4];
#pragma unroll
      for (int k = 0; k < (LN ? 6 : 4); ++k) t[k] = 0.0;
#pragma unroll
      for (int c = 0; c < C; ++c) {
        if (!on[c]) continue;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const double g = f4e(g4[c], e), dg = eps * (double)f4e(v4[c], e);
          const double p = (double)f4e(xa[c], e) + (double)f4e(xb[c], e) - mup;
          const double q = (double)f4e(xa[c], e) - (double)f4e(xb[c], e) - mum;
          const double dhp = ((double)f4e(ya[c], e) + (double)f4e(yb[c], e)) * (g + dg);
          const double dhm = ((double)f4e(ya[c], e) - (double)f4e(yb[c], e)) * (g - dg);
          t[0] += p * p;
          t[1] += q * q;
          t[2] += dhp * p;
          t[3] += dhm * q;
          if constexpr (LN) {
            t[4] += dhp;
            t[5] += dhm;
          }
        }
      }
      block_sums<NTH, LN ? 6 : 4>(t, sh2, slot2);
      rp = 1.0 / sqrt(t[0] / dm + neps);
      rmi = 1.0 / sqrt(t[1] / dm + neps);
      a2p = rp * (t[2] / dm);
      a2m = rmi * (t[3] / dm);
      if constexpr (LN) {
        a1p = t[4] / dm;
        a1m = t[5] / dm;
      }
    }
#pragma unroll
    for (int c = 0; c < C; ++c) {
      if (!on[c]) continue;
      const float4 ra = dresm ? ld(dresm, o + col[c]) : zero, rb = dresd ? ld(dresd, o + col[c]) : zero;
      float om[4], od[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double g = f4e(g4[c], e), dg = eps * (double)f4e(v4[c], e);
        const double xhp = ((double)f4e(xa[c], e) + (double)f4e(xb[c], e) - mup) * rp;
        const double xhm = ((double)f4e(xa[c], e) - (double)f4e(xb[c], e) - mum) * rmi;
        const double dyp = (double)f4e(ya[c], e) + (double)f4e(yb[c], e);
        const double dyn = (double)f4e(ya[c], e) - (double)f4e(yb[c], e);
        const double dxp = rp * (dyp * (g + dg) - a1p - xhp * a2p);
        const double dxn = rmi * (dyn * (g - dg) - a1m - xhm * a2m);
        om[e] = (float)((double)f4e(ra, e) + 0.5 * (dxp + dxn));
        od[e] = (float)((double)f4e(rb, e) + 0.5 * (dxp - dxn));
        sg[4 * c + e] += 0.5 * (dyp * xhp - dyn * xhm);
        if constexpr (LN) sb[4 * c + e] += (double)f4e(yb[c], e);
        so[4 * c + e] += (double)od[e];
      }
      *reinterpret_cast<float4*>(dx.m + o + col[c]) = make_float4(om[0], om[1], om[2], om[3]);
      *reinterpret_cast<float4*>(dx.d + o + col[c]) = make_float4(od[0], od[1], od[2], od[3]);
      if (dxo.m) {
        st4f(dxo.m, o + col[c], om[0], om[1], om[2], om[3]);
        st4f(dxo.d, o + col[c], od[0], od[1], od[2], od[3]);
      }
    }
  }
  double* p = part + (int64_t)blockIdx.x * ncol;
#pragma unroll
  for (int c = 0; c < C; ++c) {
    if (!on[c]) continue;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      p[col[c] + e] = sg[4 * c + e];
      if constexpr (LN) p[dm + col[c] + e] = sb[4 * c + e];
      if (osum) p[(LN ? 2 : 1) * dm + col[c] + e] = so[4 * c + e];
    }
  }
}

// The same with one wavefront per row (rows of 256 CPL columns, lane l at columns
// 256 c + 4 l) and 4 rows per wavefront, 16 per workgroup, for many rows: no
// barrier per row and a quarter of the reductions per element.  x is kept in
// registers, dy read again from the caches.  Column sums in LDS, at most 4 rows per
// wavefront: gain and bias terms in fp32, the outputs' half differences in fp64 (as
// the pass over the stored outputs, which they replace, added them).
// 8192 x 1024 with LayerNorm and output sums: 65 us per call; the kernel above 118,
// dy kept in registers too 100.
// 8192 x 2048 without LayerNorm: 126 to 130 us, 604 MB at 4.7 TB/s;
// the kernel above 148, dy kept in registers too 188, the registers that the
// compiler takes without a bound (one wavefront per SIMD) 168, more than two
// workgroups per CU (the second read of dy then misses the L2) 158.
template <typename T, int CPL, bool LN, bool OS>
__global__ __launch_bounds__(NT, 2) void norm_bwd_wave_kernel(PairF dx, PairT<T> dxo, const float* dresm, const float* dresd,
                                                           const float* xm, const float* xd, const float* dym,
                                                           const float* dyd, int rows, const T* thg,
                                                           const float* vg, double eps, double neps, double* part) {
  constexpr int DM = 256 * CPL;
  // per-wavefront column sums (gain, bias, outputs); a lane only touches its own columns
  constexpr int NF = 1 + (LN ? 1 : 0), NS = NF + (OS ? 1 : 0);
  // (rows of 2048: two workgroups per CU by LDS)
  constexpr int NL = DM >= 2048 && NS < 2 ? 2 : NF;
  __shared__ float cs[NL][4][DM];
  __shared__ __attribute__((aligned(16))) double so[OS ? 4 : 1][OS ? DM : 2];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int n = 0; n < NF; ++n)
    for (int c = 0; c < CPL; ++c)
      *reinterpret_cast<float4*>(&cs[n][wave][256 * c + 4 * lane]) = make_float4(0.f, 0.f, 0.f, 0.f);
  if constexpr (OS)
    for (int c = 0; c < CPL; ++c)
      for (int e = 0; e < 4; e += 2)
        *reinterpret_cast<double2*>(&so[wave][256 * c + 4 * lane + e]) = make_double2(0.0, 0.0);
  auto ld = [](const float* p, int64_t i) { return *reinterpret_cast<const float4*>(p + i); };
  const int r0 = blockIdx.x * NORM_WAVE_ROWS;
  for (int i = wave; i < NORM_WAVE_ROWS; i += 4) {
    const int row = r0 + i;
    if (row >= rows) break;
    const int64_t o = (int64_t)row * DM + 4 * lane;
    double mup = 0.0, mum = 0.0;
    float4 xac[CPL], xbc[CPL];   // the row of x, kept in registers for the later passes
    if constexpr (LN) {
      double sp = 0.0, sm = 0.0;
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        const float4 xa = ld(xm, o + 256 * c), xb = ld(xd, o + 256 * c);
        xac[c] = xa;
        xbc[c] = xb;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          sp += (double)f4e(xa, e) + (double)f4e(xb, e);
          sm += (double)f4e(xa, e) - (double)f4e(xb, e);
        }
      }
      mup = wave_sum(sp) / DM;
      mum = wave_sum(sm) / DM;
    }
    double rp, rmi, a1p = 0.0, a1m = 0.0, a2p, a2m;
    if constexpr (!LN) {
      // RMSNorm (no mean): sum x^2 and sum dxhat * x in one pass over x and
      // dy; mean(dxhat * xhat) = r * mean(dxhat * x)
      double qp = 0.0, qm = 0.0, tp = 0.0, tm = 0.0;
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        const int col = 256 * c + 4 * lane;
        const float4 xa = ld(xm, o + 256 * c), xb = ld(xd, o + 256 * c);
        xac[c] = xa;
        xbc[c] = xb;
        const float4 ya = ld(dym, o + 256 * c), yb = ld(dyd, o + 256 * c);
        const float4 g4 = ld4f(thg, col), v4 = ld(vg, col);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const double g = f4e(g4, e), dg = eps * (double)f4e(v4, e);
          const double p = (double)f4e(xa, e) + (double)f4e(xb, e);
          const double q = (double)f4e(xa, e) - (double)f4e(xb, e);
          qp += p * p;
          qm += q * q;
          tp += ((double)f4e(ya, e) + (double)f4e(yb, e)) * (g + dg) * p;
          tm += ((double)f4e(ya, e) - (double)f4e(yb, e)) * (g - dg) * q;
        }
      }
      rp = 1.0 / sqrt(wave_sum(qp) / DM + neps);
      rmi = 1.0 / sqrt(wave_sum(qm) / DM + neps);
      a2p = rp * (wave_sum(tp) / DM);
      a2m = rmi * (wave_sum(tm) / DM);
    } else {
      // LayerNorm: the variance, sum dxhat and sum dxhat * (x - mu) in one
      // pass over dy, x from the registers; mean(dxhat * xhat) =
      // r * mean(dxhat * (x - mu))
      double qp = 0.0, qm = 0.0, s1p = 0.0, s1m = 0.0, tp = 0.0, tm = 0.0;
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        const int col = 256 * c + 4 * lane;
        const float4 xa = xac[c], xb = xbc[c];
        const float4 ya = ld(dym, o + 256 * c), yb = ld(dyd, o + 256 * c);
        const float4 g4 = ld4f(thg, col), v4 = ld(vg, col);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const double g = f4e(g4, e), dg = eps * (double)f4e(v4, e);
          const double p = (double)f4e(xa, e) + (double)f4e(xb, e) - mup;
          const double q = (double)f4e(xa, e) - (double)f4e(xb, e) - mum;
          const double dhp = ((double)f4e(ya, e) + (double)f4e(yb, e)) * (g + dg);
          const double dhm = ((double)f4e(ya, e) - (double)f4e(yb, e)) * (g - dg);
          qp += p * p;
          qm += q * q;
          s1p += dhp;
          s1m += dhm;
          tp += dhp * p;
          tm += dhm * q;
        }
      }
      rp = 1.0 / sqrt(wave_sum(qp) / DM + neps);
      rmi = 1.0 / sqrt(wave_sum(qm) / DM + neps);
      a1p = wave_sum(s1p) / DM;
      a1m = wave_sum(s1m) / DM;
      a2p = rp * (wave_sum(tp) / DM);
      a2m = rmi * (wave_sum(tm) / DM);
    }
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
      const int col = 256 * c + 4 * lane;
      const float4 xa = xac[c], xb = xbc[c];
      const float4 ya = ld(dym, o + 256 * c), yb = ld(dyd, o + 256 * c);
      const float4 g4 = ld4f(thg, col), v4 = ld(vg, col);
      const float4 ra = dresm ? ld(dresm, o + 256 * c) : make_float4(0.f, 0.f, 0.f, 0.f);
      const float4 rb = dresd ? ld(dresd, o + 256 * c) : make_float4(0.f, 0.f, 0.f, 0.f);
      float om[4], od[4], tg[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double g = f4e(g4, e), dg = eps * (double)f4e(v4, e);
        const double xhp = ((double)f4e(xa, e) + (double)f4e(xb, e) - mup) * rp;
        const double xhm = ((double)f4e(xa, e) - (double)f4e(xb, e) - mum) * rmi;
        const double dyp = (double)f4e(ya, e) + (double)f4e(yb, e);
        const double dymi = (double)f4e(ya, e) - (double)f4e(yb, e);
        const double dhp = dyp * (g + dg), dhm = dymi * (g - dg);
        const double dxp = rp * (dhp - a1p - xhp * a2p);
        const double dxm = rmi * (dhm - a1m - xhm * a2m);
        om[e] = (float)((double)f4e(ra, e) + 0.5 * (dxp + dxm));
        od[e] = (float)((double)f4e(rb, e) + 0.5 * (dxp - dxm));
        tg[e] = (float)(0.5 * (dyp * xhp - dymi * xhm));
      }
      *reinterpret_cast<float4*>(dx.m + o + 256 * c) = make_float4(om[0], om[1], om[2], om[3]);
      *reinterpret_cast<float4*>(dx.d + o + 256 * c) = make_float4(od[0], od[1], od[2], od[3]);
      if (dxo.m) {
        st4f(dxo.m, o + 256 * c, om[0], om[1], om[2], om[3]);
        st4f(dxo.d, o + 256 * c, od[0], od[1], od[2], od[3]);
      }
      auto add = [&](int n, float a, float b, float c, float e) {
        float4* p = reinterpret_cast<float4*>(&cs[n][wave][col]);
        const float4 v = *p;
        *p = make_float4(v.x + a, v.y + b, v.z + c, v.w + e);
      };
      add(0, tg[0], tg[1], tg[2], tg[3]);
      if constexpr (LN) add(1, yb.x, yb.y, yb.z, yb.w);
      if constexpr (OS)
#pragma unroll
        for (int e = 0; e < 4; e += 2) {
          double2* q = reinterpret_cast<double2*>(&so[wave][col + e]);
          const double2 v = *q;
          *q = make_double2(v.x + (double)od[e], v.y + (double)od[e + 1]);
        }
    }
  }
  // the four wavefronts' column sums, added in fp64 in wavefront order
  __syncthreads();
  double* p = part + (int64_t)blockIdx.x * NS * DM;
  for (int j = threadIdx.x; j < DM; j += NT) {
#pragma unroll
    for (int n = 0; n < NF; ++n)
      p[n * DM + j] = (double)cs[n][0][j] + (double)cs[n][1][j] + (double)cs[n][2][j] + (double)cs[n][3][j];
    if constexpr (OS) p[NF * DM + j] = so[0][j] + so[1][j] + so[2][j] + so[3][j];
  }
}

// ---- column sums ---------------------------------------------------------------
// out[s][j] (+)= scale * sum_r part[r][s C + j] for the sums s that have an
// output.  16 columns and 64 row groups per workgroup: a thread adds every 64th
// row, lanes and then wavefronts are added in a fixed order.
__global__ __launch_bounds__(1024) void colsum_part_kernel(ColSums o, const double* part, int rows, int ncol, int C,
                                                           double scale, bool acc) {
  __shared__ double sh[16][16];
  const int cl = threadIdx.x & 15, j = blockIdx.x * 16 + cl;
  double s = 0.0;
  if (j < ncol)
    for (int r = threadIdx.x >> 4; r < rows; r += 64) s += part[(int64_t)r * ncol + j];
  s += __shfl_xor(s, 16, 64);
  s += __shfl_xor(s, 32, 64);
  if ((threadIdx.x & 63) < 16) sh[threadIdx.x >> 6][cl] = s;
  __syncthreads();
  if (threadIdx.x >= 16 || j >= ncol) return;
  s = 0.0;
#pragma unroll
  for (int w = 0; w < 16; ++w) s += sh[w][cl];
  s *= scale;
  float* out = o.out[j / C];
  if (!out) return;
  out += j % C;
  *out = acc ? (float)((double)*out + s) : (float)s;
}

// ---- RoPE ----------------------------------------------------------------------
__global__ void rope_table_kernel(double* cs, int S, int dh, double base) {
  const int half = dh / 2;
  GRID_LOOP(i, (int64_t)S * half) {
    const int s = (int)(i / half), f = (int)(i % half);
    const double inv = pow(base, -(double)(2 * f) / (double)dh);
    const double ang = (double)s * inv;
    cs[(int64_t)s * dh + 2 * f] = cos(ang);
    cs[(int64_t)s * dh + 2 * f + 1] = sin(ang);
  }
}

// Both channels in one pass.  A thread takes 4 consecutive columns f0..f0+3
// of the first half of a q or k head together with their rotate-half
// partners f0+dh/2.., reads each once and writes both rotated quadruples
// (packed); v columns are cast 4 at a time.
template <typename T, typename TI>
__global__ void qkv_rope_kernel(PairT<T> out, const TI* inm, const TI* ind, int S, int ncols, int nqk, int dh,
                                const double* cs, bool inverse, bool copy_v) {
  const int t = blockIdx.y;
  const int u = blockIdx.x * blockDim.x + threadIdx.x;
  const int half = dh / 2, qpu = half / 4;      // units per q/k head
  const int qu = nqk * qpu;                     // rotated units
  const int vu = copy_v ? (ncols - nqk * dh) / 4 : 0;
  const int64_t o = (int64_t)t * ncols;
  if (u < qu) {
    const int head = u / qpu, f0 = 4 * (u % qpu);
    const int c = head * dh + f0;
    const double* row = cs + (int64_t)(t % S) * dh;
    double co[4], si[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      co[e] = row[2 * (f0 + e)];
      si[e] = inverse ? -row[2 * (f0 + e) + 1] : row[2 * (f0 + e) + 1];
    }
    const TI* ins[2] = {inm, ind};
    T* outs[2] = {out.m, out.d};
#pragma unroll
    for (int ch = 0; ch < 2; ++ch) {
      // (in place when ins == outs: this thread alone reads and writes these 8 elements)
      const float4 x = ld4f(ins[ch], o + c);
      const float4 y = ld4f(ins[ch], o + c + half);
      float lo[4], hi[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double xe = f4e(x, e), ye = f4e(y, e);
        lo[e] = (float)(xe * co[e] - ye * si[e]);
        hi[e] = (float)(ye * co[e] + xe * si[e]);
      }
      st4f(outs[ch], o + c, lo[0], lo[1], lo[2], lo[3]);
      st4f(outs[ch], o + c + half, hi[0], hi[1], hi[2], hi[3]);
    }
  } else if (u < qu + vu) {
    const int c = nqk * dh + 4 * (u - qu);
    const float4 a = ld4f(inm, o + c), b = ld4f(ind, o + c);
    st4f(out.m, o + c, a.x, a.y, a.z, a.w);
    st4f(out.d, o + c, b.x, b.y, b.z, b.w);
  }
}

// Without RoPE: the operand-type copy of both channels (out.m not null) and the
// q/k/v bias gradient: a thread takes 4 columns of `per` rows and writes the sums
// of their half differences as its workgroup row of part.
template <typename T>
__global__ __launch_bounds__(NT) void qkv_bias_kernel(PairT<T> out, const float* gm, const float* gd, int rows, int per,
                                                      int ncols, double* part) {
  const int c = 4 * (blockIdx.x * NT + threadIdx.x);
  if (c >= ncols) return;
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  const int r0 = blockIdx.y * per, r1 = min(rows, r0 + per);
  for (int r = r0; r < r1; ++r) {
    const int64_t i = (int64_t)r * ncols + c;
    const float4 b = *reinterpret_cast<const float4*>(gd + i);
    if (out.m) {
      const float4 a = *reinterpret_cast<const float4*>(gm + i);
      st4f(out.m, i, a.x, a.y, a.z, a.w);
      st4f(out.d, i, b.x, b.y, b.z, b.w);
    }
    s[0] += b.x; s[1] += b.y; s[2] += b.z; s[3] += b.w;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) part[(int64_t)blockIdx.y * ncols + c + e] = s[e];
}

// ---- causal softmax and its backward, both points ---------------------------------------
// One wavefront per row, 4 rows per workgroup.  Row i of a causal score
// matrix has i+1 live entries; entries i < j < roundup(i+1, 256) are written
// as zeros, because the MFMA tiles that contract over a row read exactly up
// to that boundary; entries beyond it are never read and not written.
// The softmax at both points uses exp(Sm - c +- Sd) = exp(Sm - c) (cosh Sd +- sinh Sd):
// per live entry a = exp(Sm - c) cosh(Sd) and b = exp(Sm - c) sinh(Sd), both
// with full relative precision however small Sd is, so that e+- = a +- b and
//   P.m = (a Zm - b Zd) / (Z+ Z-),  P.d = (b Zm - a Zd) / (Z+ Z-),
// with Zm = sum a and Zd = sum b (fp64 sums) the mean and half difference of
// Z+- = sum e+-.  exp(Sm - c) is formed in fp32: its rounding is common to the
// two points.
__device__ inline int zero_end(int i, int S) { return min(S, ((i + 256) / 256) * 256); }

template <typename T, int PER>
__global__ __launch_bounds__(256) void attn_softmax_w(PairT<T> P, const float* Sm, const float* Sd, int nrows, int S) {
  const int lane = threadIdx.x & 63;
  const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= nrows) return;
  const int i = (int)(r % S);
  const int64_t base = r * (int64_t)S;
  const int len = i + 1;
  float av[PER], bv[PER];
  float mx = -3.0e38f;
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int j = lane + 64 * e;
    av[e] = (j < len) ? Sm[base + j] : -3.0e38f;
    bv[e] = (j < len) ? Sd[base + j] : 0.f;
    mx = fmaxf(mx, av[e]);
  }
  mx = wave_max(mx);
  double Zm = 0.0, Zd = 0.0;
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int j = lane + 64 * e;
    if (j < len) {
      const float ea = expf(av[e] - mx);
      const float b = bv[e];
      av[e] = ea * coshf(b);
      bv[e] = ea * sinhf(b);
      Zm += (double)av[e];
      Zd += (double)bv[e];
    } else {
      av[e] = bv[e] = 0.f;
    }
  }
  Zm = wave_sum(Zm);
  Zd = wave_sum(Zd);
  const double inv = 1.0 / ((Zm + Zd) * (Zm - Zd));
  const int ze = zero_end(i, S);
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int j = lane + 64 * e;
    if (j < ze) {
      const double a = av[e], b = bv[e];
      stf(P.m, base + j, (float)((a * Zm - b * Zd) * inv));
      stf(P.d, base + j, (float)((b * Zm - a * Zd) * inv));
    }
  }
}

template <typename T, int PER>
__global__ __launch_bounds__(256) void attn_dsoftmax_w(PairT<T> dS, const T* Pm, const T* Pd, const float* dPm,
                                                       const float* dPd, int nrows, int S) {
  const int lane = threadIdx.x & 63;
  const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= nrows) return;
  const int i = (int)(r % S);
  const int64_t base = r * (int64_t)S;
  const int len = i + 1;
  double dp = 0.0, dm = 0.0;
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int j = lane + 64 * e;
    if (j < len) {
      const double pm = ldf(Pm, base + j), pd = ldf(Pd, base + j);
      const double gm = dPm[base + j], gd = dPd[base + j];
      dp += (pm + pd) * (gm + gd);
      dm += (pm - pd) * (gm - gd);
    }
  }
  dp = wave_sum(dp);
  dm = wave_sum(dm);
  const int ze = zero_end(i, S);
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int j = lane + 64 * e;
    if (j < ze) {
      double sp = 0.0, sn = 0.0;
      if (j < len) {
        const double pm = ldf(Pm, base + j), pd = ldf(Pd, base + j);
        const double gm = dPm[base + j], gd = dPd[base + j];
        sp = (pm + pd) * (gm + gd - dp);
        sn = (pm - pd) * (gm - gd - dm);
      }
      put_pair(dS, base + j, sp, sn);
    }
  }
}

__global__ void group_sum_kernel(float* out, int64_t out_ld, const float* in, int T_, int Hk, int G, int dh) {
  const int64_t n = (int64_t)T_ * Hk * dh;
  GRID_LOOP(i, n) {
    const int t = (int)(i / (Hk * dh)), c = (int)(i % (Hk * dh));
    const int kh = c / dh, e = c % dh;
    double s = 0.0;
    for (int g = 0; g < G; ++g) s += in[(int64_t)t * (Hk * G * dh) + (int64_t)(kh * G + g) * dh + e];
    out[(int64_t)t * out_ld + c] = (float)s;
  }
}

// ---- activations ------------------------------------------------------------------
// GELU (tanh form) is u sigmoid(y), y = 2 k (u + a u^3): tanh t = 2 sigmoid(2t) - 1.
// Both points' sigmoids in fp64 from one exponential and one division:
// e^-y+- = e^-ym e^-+h for ym and h the half sum and half difference of y+-, and
// 1 / (1 + e^-y+) = B / (A B), 1 / (1 + e^-y-) = A / (A B).  (e^-ym is held
// below 1e150, where u sigmoid is already far below the smallest fp32 number.)
__device__ inline void exp_pm(double b, double& ep, double& en);
__device__ inline void sigmoid_pair(double yp, double yn, double& sp, double& sn) {
  const double ym = 0.5 * (yp + yn), h = 0.5 * (yp - yn);
  double ep, en;
  if (fabs(h) < 0.0625) {
    const double E = fmin(exp(-ym), 1e150);
    exp_pm(h, ep, en);
    ep *= E;   // e^-yn
    en *= E;   // e^-yp
  } else {
    en = fmin(exp(-yp), 1e150);
    ep = fmin(exp(-yn), 1e150);
  }
  const double A = 1.0 + en, B = 1.0 + ep;
  const double inv = 1.0 / (A * B);
  sp = B * inv;
  sn = A * inv;
}
constexpr double GELU_K = 2.0 * 0.7978845608028654, GELU_A = 0.044715;
__device__ inline void gelu_pair(double a, double b, float& om, float& od) {
  const double up = a + b, un = a - b;
  double sp, sn;
  sigmoid_pair(GELU_K * (up + GELU_A * up * up * up), GELU_K * (un + GELU_A * un * un * un), sp, sn);
  const double p = up * sp, n = un * sn;
  om = (float)(0.5 * (p + n));
  od = (float)(0.5 * (p - n));
}
// gradient s + u s (1 - s) y'(u) at both points times the upstream gradient
__device__ inline void gelu_bwd_pair(double a, double b, double zm, double zd, float& om, float& od) {
  const double up = a + b, un = a - b;
  double sp, sn;
  sigmoid_pair(GELU_K * (up + GELU_A * up * up * up), GELU_K * (un + GELU_A * un * un * un), sp, sn);
  const double gp = (zm + zd) * (sp + up * sp * (1.0 - sp) * (GELU_K * (1.0 + 3.0 * GELU_A * up * up)));
  const double gn = (zm - zd) * (sn + un * sn * (1.0 - sn) * (GELU_K * (1.0 + 3.0 * GELU_A * un * un)));
  om = (float)(0.5 * (gp + gn));
  od = (float)(0.5 * (gp - gn));
}

// SwiGLU output at both points, (s(a) v_a, s(b) v_b) with s(x) = x sigmoid(x),
// gate a, b = gm +- gd and up u = um +- ud, returned as its half sum om and half
// difference od, in fp32 without forming the two values and subtracting them:
//   (s(a) + s(b)) / 2 is taken directly;
//   (s(a) - s(b)) / 2 = (gd (sig(a) + sig(b)) + gm (sig(a) - sig(b))) / 2, and
//   sig(a) - sig(b) = sig(a) sig(-b) (1 - e^(-2 gd)) with expm1 for the last
//   factor, so the difference channel keeps fp32 relative accuracy for any gd
//   (no loss of order gd / gm);
//   om = S um + D ud and od = S ud + D um for the gate's half sum S and half
//   difference D.
__device__ inline void swiglu_pair(float gm, float gd, float um, float ud, float& om, float& od) {
  const float a = gm + gd, b = gm - gd;
  const float eb = expf(-b);
  const float sa = 1.f / (1.f + expf(-a)), sb = 1.f / (1.f + eb);
  const float snb = b < 0.f ? 1.f - sb : eb * sb;   // sig(-b), accurate on both sides
  const float dsig = sa * snb * -expm1f(-2.f * gd);
  const float S = 0.5f * (a * sa + b * sb), D = 0.5f * (gd * (sa + sb) + gm * dsig);
  om = S * um + D * ud;
  od = S * ud + D * um;
}

// SwiGLU backward at both points in the same channel form: for the upstream
// gradient z = zm +- zd, the gate gradient z v s'(g) and the up gradient
// z s(g), with s'(x) = sig(x) (1 + x sig(-x)).  Every factor is split into its
// half sum and half difference and a product of two split factors is formed as
// (xm ym + xd yd, xm yd + xd ym), which is exact before rounding.  The half
// difference of s' is (sig(a) - sig(b) + h(a) - h(b)) / 2 with
// h(x) = x sig'(x), sig' = sig(x) sig(-x), and
//   h(a) - h(b) = gd (sig'(a) + sig'(b)) + gm (sig'(a) - sig'(b)),
//   sig'(a) - sig'(b) = (sig(a) - sig(b)) (1 - sig(a) - sig(b)),
// so no term subtracts two values of the full size of s'.
__device__ inline void swiglu_bwd_pair(float gm, float gd, float um, float ud, float zm, float zd, float& am,
                                       float& ad, float& bm, float& bd) {
  const float a = gm + gd, b = gm - gd;
  const float ea = expf(-a), eb = expf(-b);
  const float sa = 1.f / (1.f + ea), sb = 1.f / (1.f + eb);
  const float sna = a < 0.f ? 1.f - sa : ea * sa, snb = b < 0.f ? 1.f - sb : eb * sb;
  const float dsig = sa * snb * -expm1f(-2.f * gd);
  const float pa = sa * sna, pb = sb * snb;   // sig'(a), sig'(b)
  const float S1 = 0.5f * (sa * (1.f + a * sna) + sb * (1.f + b * snb));
  const float D1 = 0.5f * (dsig + gd * (pa + pb) + gm * dsig * (1.f - sa - sb));
  const float S0 = 0.5f * (a * sa + b * sb), D0 = 0.5f * (gd * (sa + sb) + gm * dsig);
  const float xm = zm * um + zd * ud, xd = zm * ud + zd * um;   // z v
  am = xm * S1 + xd * D1;
  ad = xm * D1 + xd * S1;
  bm = zm * S0 + zd * D0;
  bd = zm * D0 + zd * S0;
}

// four consecutive elements per thread (n is a multiple of 4)
template <typename T>
__global__ __launch_bounds__(NT) void gelu_fwd_kernel(PairT<T> z, const T* um, const T* ud, int64_t n4) {
  GRID_LOOP(i, n4) {
    const float4 a = ld4f(um, 4 * i), b = ld4f(ud, 4 * i);
    float om[4], od[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) gelu_pair(f4e(a, e), f4e(b, e), om[e], od[e]);
    st4f(z.m, 4 * i, om[0], om[1], om[2], om[3]);
    st4f(z.d, 4 * i, od[0], od[1], od[2], od[3]);
  }
}
// A thread takes 4 columns of `per` rows; the sums of the half differences (the
// bias gradient of the MLP input layer, from the fp32 values) go to part.
template <typename T>
__global__ __launch_bounds__(NT) void gelu_bwd_kernel(PairT<T> du, const T* um, const T* ud, const float* dzm,
                                                      const float* dzd, int rows, int per, int F, double* part) {
  const int c = 4 * (blockIdx.x * NT + threadIdx.x);
  if (c >= F) return;
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  const int r0 = blockIdx.y * per, r1 = min(rows, r0 + per);
  for (int r = r0; r < r1; ++r) {
    const int64_t i = (int64_t)r * F + c;
    const float4 a = ld4f(um, i), b = ld4f(ud, i);
    const float4 zm = *reinterpret_cast<const float4*>(dzm + i), zd = *reinterpret_cast<const float4*>(dzd + i);
    float om[4], od[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      gelu_bwd_pair(f4e(a, e), f4e(b, e), f4e(zm, e), f4e(zd, e), om[e], od[e]);
      s[e] += (double)od[e];
    }
    st4f(du.m, i, om[0], om[1], om[2], om[3]);
    st4f(du.d, i, od[0], od[1], od[2], od[3]);
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) part[(int64_t)blockIdx.y * F + c + e] = s[e];
}
// Vectorised forms: grid.y = row, each thread 4 consecutive columns of the
// F gate (and F up) columns; F % 4 == 0.  Same arithmetic as the scalar forms.
template <typename T>
__global__ void swiglu_fwd4_kernel(PairT<T> z, const T* gum, const T* gud, int F) {
  const int c = 4 * (blockIdx.x * blockDim.x + threadIdx.x);
  if (c >= F) return;
  const int64_t t = blockIdx.y;
  const int64_t ig = t * 2 * F + c, iu = ig + F, io = t * F + c;
  const float4 gm = ld4f(gum, ig), gd = ld4f(gud, ig);
  const float4 um = ld4f(gum, iu), ud = ld4f(gud, iu);
  float om[4], od[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) swiglu_pair(f4e(gm, e), f4e(gd, e), f4e(um, e), f4e(ud, e), om[e], od[e]);
  st4f(z.m, io, om[0], om[1], om[2], om[3]);
  st4f(z.d, io, od[0], od[1], od[2], od[3]);
}
template <typename T>
__global__ void swiglu_bwd4_kernel(PairT<T> dgu, const T* gum, const T* gud, const float* dzm, const float* dzd,
                                   int F) {
  const int c = 4 * (blockIdx.x * blockDim.x + threadIdx.x);
  if (c >= F) return;
  const int64_t t = blockIdx.y;
  const int64_t ig = t * 2 * F + c, iu = ig + F, io = t * F + c;
  const float4 gm = ld4f(gum, ig), gd = ld4f(gud, ig);
  const float4 um = ld4f(gum, iu), ud = ld4f(gud, iu);
  const float4 zm = *reinterpret_cast<const float4*>(dzm + io), zd = *reinterpret_cast<const float4*>(dzd + io);
  float am[4], ad[4], bm[4], bd[4];
#pragma unroll
  for (int e = 0; e < 4; ++e)
    swiglu_bwd_pair(f4e(gm, e), f4e(gd, e), f4e(um, e), f4e(ud, e), f4e(zm, e), f4e(zd, e), am[e], ad[e], bm[e], bd[e]);
  st4f(dgu.m, ig, am[0], am[1], am[2], am[3]);
  st4f(dgu.d, ig, ad[0], ad[1], ad[2], ad[3]);
  st4f(dgu.m, iu, bm[0], bm[1], bm[2], bm[3]);
  st4f(dgu.d, iu, bd[0], bd[1], bd[2], bd[3]);
}

template <typename T>
__global__ void swiglu_fwd_kernel(PairT<T> z, const T* gum, const T* gud, int rows, int F) {
  const int64_t n = (int64_t)rows * F;
  GRID_LOOP(i, n) {
    const int64_t t = i / F, c = i % F;
    const int64_t ig = t * 2 * F + c, iu = ig + F;
    float om, od;
    swiglu_pair(ldf(gum, ig), ldf(gud, ig), ldf(gum, iu), ldf(gud, iu), om, od);
    stf(z.m, i, om);
    stf(z.d, i, od);
  }
}
template <typename T>
__global__ void swiglu_bwd_kernel(PairT<T> dgu, const T* gum, const T* gud, const float* dzm, const float* dzd,
                                  int rows, int F) {
  const int64_t n = (int64_t)rows * F;
  GRID_LOOP(i, n) {
    const int64_t t = i / F, c = i % F;
    const int64_t ig = t * 2 * F + c, iu = ig + F;
    float am, ad, bm, bd;
    swiglu_bwd_pair(ldf(gum, ig), ldf(gud, ig), ldf(gum, iu), ldf(gud, iu), dzm[i], dzd[i], am, ad, bm, bd);
    stf(dgu.m, ig, am);
    stf(dgu.d, ig, ad);
    stf(dgu.m, iu, bm);
    stf(dgu.d, iu, bd);
  }
}

// ---- cross-entropy, both points -------------------------------------------------------------
// The logits of position t predict the label of position t + 1: the next token,
// or lab[t + 1] when labels are given; a label of IGNORE_LABEL (padding,
// masked prompt) leaves the row out.  inv_n scales every kept row.
// e^b and e^-b as c + s and c - s with c = cosh b and s = sinh b: for
// |b| < 1/16 their Taylor series to b^8 and b^9 (the first omitted terms are
// below 2^-40 / 10! of the sum), otherwise from exp.
constexpr double EXP_PM_SERIES = 0.0625;
__device__ inline void exp_pm(double b, double& ep, double& en) {
  if (fabs(b) < EXP_PM_SERIES) {
    const double b2 = b * b;
    const double c = 1.0 + b2 * (1.0 / 2 + b2 * (1.0 / 24 + b2 * (1.0 / 720 + b2 * (1.0 / 40320))));
    const double sn = b * (1.0 + b2 * (1.0 / 6 + b2 * (1.0 / 120 + b2 * (1.0 / 5040 + b2 * (1.0 / 362880)))));
    ep = c + sn;
    en = c - sn;
  } else {
    ep = exp(b);
    en = exp(-b);
  }
}

// One workgroup per row, four consecutive logits per thread and step, two passes.
// Large workgroups keep few rows in flight, so that the second pass over a row
// finds it in the last-level cache (256 KB per row of 32000 logits: 512 rows in
// flight are 128 MB, the 2048 rows of 256-thread workgroups do not fit).
// 8192 x 32000: 1250 -> 1020 us.
template <typename T, int NTH>
__global__ __launch_bounds__(NTH) void ce_kernel(PairT<T> dl, double* rowloss, const float* lm, const float* ld,
                                                 const int32_t* tok, const int32_t* lab, int T_, int S, int V,
                                                 double inv_n) {
  __shared__ double sh[NTH / 64];
  const int64_t t = blockIdx.x;
  const int64_t o = t * (int64_t)V;
  const int n4 = V / 4;   // V is a multiple of 8
  const bool last = (t % S) == (S - 1);
  const int raw = last ? IGNORE_LABEL : (lab ? lab[t + 1] : tok[t + 1]);
  if (raw == IGNORE_LABEL) {
    for (int j = threadIdx.x; j < n4; j += NTH) {
      st4f(dl.m, o + 4 * j, 0.f, 0.f, 0.f, 0.f);
      st4f(dl.d, o + 4 * j, 0.f, 0.f, 0.f, 0.f);
    }
    if (threadIdx.x == 0) { rowloss[t] = 0.0; rowloss[T_ + t] = 0.0; }
    return;
  }
  const int y = clamp_tok(raw, V);
  auto ld4 = [](const float* p, int64_t i) { return *reinterpret_cast<const float4*>(p + i); };
  // exp(a +- b) = E e^+-b with E = exp(a) shared by both points and e^+-b from
  // exp_pm.  For bf16 models E is taken in fp32 (a common factor of the two
  // channels, so its rounding never cancels in their half difference).  fp32
  // models share E within the series only, and take the maximum over a + |b|
  // beyond it: a far smaller E with a far larger e^b would be 0 times infinity.
  auto expa = [&](double a) {
    if constexpr (sizeof(T) == 2) return (double)__expf((float)a);
    else return exp(a);
  };
  auto both = [&](double E, double a, double b, double& xp, double& xn) {
    if (sizeof(T) == 2 || fabs(b) < EXP_PM_SERIES) {
      double ep, en;
      exp_pm(b, ep, en);
      xp = E * ep;
      xn = E * en;
    } else {
      xp = exp(a + b);
      xn = exp(a - b);
    }
  };
  // one pass for the row maximum and the sums: each thread keeps its sums
  // relative to its own running maximum mt, rescaled by exp(old mt - new mt)
  // when mt rises, then relative to the row maximum mx.  The rescale factors
  // are common to both points.
  double mt = -1e300, zp = 0.0, zm = 0.0;
  for (int j = threadIdx.x; j < n4; j += NTH) {
    const float4 a = ld4(lm, o + 4 * j), b = ld4(ld, o + 4 * j);
    auto high = [](float x, float y) { return sizeof(T) == 4 && fabsf(y) >= (float)EXP_PM_SERIES ? x + fabsf(y) : x; };
    const double top = (double)fmaxf(fmaxf(high(a.x, b.x), high(a.y, b.y)), fmaxf(high(a.z, b.z), high(a.w, b.w)));
    if (top > mt) {
      const double f = mt > -1e300 ? expa(mt - top) : 0.0;
      zp *= f;
      zm *= f;
      mt = top;
    }
    double E[4];   // (ahead of the branches, so that the four exponentials overlap)
#pragma unroll
    for (int e = 0; e < 4; ++e) E[e] = expa((double)f4e(a, e) - mt);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      double xp, xn;
      both(E[e], (double)f4e(a, e) - mt, f4e(b, e), xp, xn);
      zp += xp;
      zm += xn;
    }
  }
  const double mx = block_max<NTH>(mt, sh);
  const double fr = mt > -1e300 ? expa(mt - mx) : 0.0;
  zp = block_sum<NTH>(zp * fr, sh);
  zm = block_sum<NTH>(zm * fr, sh);
  const double izp = inv_n / zp, izm = inv_n / zm;
  // (last logits first: they are still in the L2)
  for (int j = ((n4 - 1) / NTH) * NTH + threadIdx.x; j >= 0; j -= NTH) {
    if (j >= n4) continue;
    const float4 a = ld4(lm, o + 4 * j), b = ld4(ld, o + 4 * j);
    float om[4], od[4];
    double E[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) E[e] = expa((double)f4e(a, e) - mx);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      double xp, xn;
      both(E[e], (double)f4e(a, e) - mx, f4e(b, e), xp, xn);
      const double pp = xp * izp, pn = xn * izm;
      om[e] = (float)(0.5 * (pp + pn) - (4 * j + e == y ? inv_n : 0.0));
      od[e] = (float)(0.5 * (pp - pn));
    }
    st4f(dl.m, o + 4 * j, om[0], om[1], om[2], om[3]);
    st4f(dl.d, o + 4 * j, od[0], od[1], od[2], od[3]);
  }
  if (threadIdx.x == 0) {
    const double a = (double)lm[o + y] - mx, b = (double)ld[o + y];
    rowloss[t] = (log(zp) - (a + b)) * inv_n;
    rowloss[T_ + t] = (log(zm) - (a - b)) * inv_n;
  }
}

__global__ void loss_sum_kernel(double* out2, const double* rowloss, int T_, bool acc) {
  __shared__ double sh[NT / 64];
  double a = 0.0, b = 0.0;
  // fixed assignment of rows to threads, fixed reduction tree
  for (int t0 = threadIdx.x; t0 < T_; t0 += 8 * NT) {
    double x[8], y[8];   // sixteen loads in flight
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int t = t0 + u * NT;
      x[u] = t < T_ ? rowloss[t] : 0.0;
      y[u] = t < T_ ? rowloss[T_ + t] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) { a += x[u]; b += y[u]; }
  }
  a = block_sum<NT>(a, sh);
  b = block_sum<NT>(b, sh);
  if (threadIdx.x == 0) {
    out2[0] = acc ? out2[0] + a : a;
    out2[1] = acc ? out2[1] + b : b;
  }
}

// out[0] += number of targets of one [B, S] batch (positions t % S < S - 1
// whose label at t + 1 is not IGNORE_LABEL; all of them without labels),
// out[1] += number of labels outside [0, V) other than IGNORE_LABEL,
// out[2] += number of tokens outside [0, V).
__global__ void count_targets_kernel(int64_t* out, const int32_t* tok, const int32_t* lab, int B, int S, int V) {
  __shared__ double sh[NT / 64];
  const int64_t n = (int64_t)B * S;
  double c = 0.0, bad = 0.0, badt = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += NT) {
    const int x = tok[i];
    if (x < 0 || x >= V) badt += 1.0;
    const int64_t t = i % S;
    if (t == S - 1) continue;
    const int y = lab ? lab[i + 1] : 0;
    if (y == IGNORE_LABEL) continue;
    if (y < 0 || y >= V) bad += 1.0;
    else c += 1.0;
  }
  // counts below 2^53 are exact in fp64
  c = block_sum<NT>(c, sh);
  bad = block_sum<NT>(bad, sh);
  badt = block_sum<NT>(badt, sh);
  if (threadIdx.x == 0) {
    out[0] += (int64_t)c;
    out[1] += (int64_t)bad;
    out[2] += (int64_t)badt;
  }
}

// ---- embedding backward --------------------------------------------------------------
// Sorted keys by rank: keys = token << 14 | position (positions < 2^14) are
// distinct, so the rank of a key is the number of smaller ones.  A workgroup
// holds all keys in LDS and ranks 32 of them, 8 lanes each (T^2 / 8 comparisons
// per lane group over the whole chip; one workgroup's bitonic sort of 8192 keys
// took 100 us, this 26).
constexpr int SORT_N = 16384;
__global__ __launch_bounds__(NT) void token_sort_kernel(uint32_t* keys, const int32_t* tok, int T_, int V) {
  extern __shared__ uint32_t k[];   // [round_up(T, 4)]
  const int n4 = (T_ + 3) / 4;
  for (int i0 = threadIdx.x; i0 < 4 * n4; i0 += 8 * NT) {
    int t[8];   // eight loads in flight
#pragma unroll
    for (int u = 0; u < 8; ++u) t[u] = tok[min(i0 + u * NT, T_ - 1)];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = i0 + u * NT;
      if (i < 4 * n4) k[i] = i < T_ ? (((uint32_t)clamp_tok(t[u], V) << 14) | (uint32_t)i) : 0xFFFFFFFFu;
    }
  }
  __syncthreads();
  const int i = blockIdx.x * (NT / 8) + (threadIdx.x >> 3);
  const uint32_t own = k[min(i, T_ - 1)];
  int rank = 0;
  for (int q = threadIdx.x & 7; q < n4; q += 8) {
    const uint4 x = *reinterpret_cast<const uint4*>(k + 4 * q);
    rank += (int)(x.x < own) + (int)(x.y < own) + (int)(x.z < own) + (int)(x.w < own);
  }
  rank += __shfl_xor(rank, 1, 64);
  rank += __shfl_xor(rank, 2, 64);
  rank += __shfl_xor(rank, 4, 64);
  if ((threadIdx.x & 7) == 0 && i < T_) keys[rank] = own;
}

// One workgroup per (sorted position, NT-column chunk); only segment starts
// work.  The segment end is found by binary search in the sorted keys, and the
// segment's rows are summed with 16 partial sums (row q of the segment into
// partial q % 16, combined in a fixed order), the next rows' keys loaded ahead:
// a frequent token (hundreds of rows under a Zipf distribution) is a chain of
// loads, which bounds the kernel.  8192 x 512: 81 -> 70 us (8 rows in flight).
__global__ void embed_bwd_kernel(float* hv, const uint32_t* keys, const float* dxd, int T_, int dm, double inv_eps,
                                 bool acc) {
  const int j = blockIdx.x;
  const uint32_t tk = keys[j] >> 14;
  if (j > 0 && (keys[j - 1] >> 14) == tk) return;
  int lo = j + 1, hi = T_;   // first position with a larger token
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if ((keys[mid] >> 14) == tk) lo = mid + 1;
    else hi = mid;
  }
  const int e = lo;
  const int c = blockIdx.y * NT + threadIdx.x;
  if (c >= dm) return;
  constexpr int U = 16;
  double s[U];
  uint32_t pos[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    s[u] = 0.0;
    pos[u] = keys[min(j + u, T_ - 1)] & 0x3FFFu;
  }
  int q = j;
  for (; q + U <= e; q += U) {
    float x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = dxd[(int64_t)pos[u] * dm + c];
#pragma unroll
    for (int u = 0; u < U; ++u) pos[u] = keys[min(q + U + u, T_ - 1)] & 0x3FFFu;
#pragma unroll
    for (int u = 0; u < U; ++u) s[u] += (double)x[u];
  }
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (q + u < e) s[u] += (double)dxd[(int64_t)pos[u] * dm + c];
#pragma unroll
  for (int w = U / 2; w > 0; w /= 2)
#pragma unroll
    for (int u = 0; u < w; ++u) s[u] += s[u + w];
  const int64_t idx = (int64_t)tk * dm + c;
  hv[idx] = acc ? (float)((double)hv[idx] + s[0] * inv_eps) : (float)(s[0] * inv_eps);
}

__global__ void pos_bwd_kernel(float* hv, const float* dxd, int B, int S, int dm, double inv_eps, bool acc) {
  const int64_t n = (int64_t)S * dm;
  GRID_LOOP(i, n) {
    const int s = (int)(i / dm), c = (int)(i % dm);
    double a = 0.0;
    for (int b = 0; b < B; ++b) a += (double)dxd[((int64_t)b * S + s) * dm + c];
    const float x = (float)(a * inv_eps);
    hv[i] = acc ? hv[i] + x : x;
  }
}

}  // namespace

// ================================ launchers ==============================================
template <typename T>
hipError_t launch_cast_pair(PairT<T> out, const float* m, const float* d, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(cast_pair_kernel<T>, dim3(grid_for(n)), dim3(NT), 0, s, out, m, d, n);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_embed_fwd(PairF x, const int32_t* tok, int T_, int S, int dm, int V, const T* the, const float* ve,
                            const T* thp, const float* vp, double eps, int* bad_tok, hipStream_t s) {
  hipLaunchKernelGGL(embed_fwd_kernel<T>, dim3(grid_for((int64_t)T_ * dm)), dim3(NT), 0, s, x, tok, T_, S, dm, V, the,
                     ve, thp, vp, eps, bad_tok);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_norm_fwd(PairT<T> y, const float* xm, const float* xd, int rows, int dm, bool ln, const T* thg,
                           const float* vg, const T* thb, const float* vb, double eps, float neps, hipStream_t s) {
  const dim3 g(ceil_div(rows, NORM_FWD_ROWS));
#define NFW(C) hipLaunchKernelGGL((norm_fwd_wave_kernel<T, C>), g, dim3(NT), 0, s, y, xm, xd, rows, ln, thg, vg, thb, vb, eps, \
                                  (double)neps)
  if (dm == 512) NFW(2);
  else if (dm == 1024) NFW(4);
  else if (dm == 2048) NFW(8);
  else hipLaunchKernelGGL(norm_fwd_kernel<T>, dim3(rows), dim3(NT), 0, s, y, xm, xd, dm, ln, thg, vg, thb, vb, eps, (double)neps);
#undef NFW
  return hipGetLastError();
}

template <typename T>
hipError_t launch_norm_bwd(PairF dx, PairT<T> dxo, const float* dresm, const float* dresd, const float* xm, const float* xd,
                           const float* dym, const float* dyd, int rows, int dm, bool ln, const T* thg,
                           const float* vg, double eps, float neps, double* part, bool osum, hipStream_t s) {
  // (wider rows were never supported)
  if ((size_t)dm * (ln ? 2 : 1) > 8192) return hipErrorInvalidValue;
  if (norm_bwd_waves(rows, dm)) {
    const dim3 g(norm_bwd_groups(rows, dm));
#define NW(C, L, O)                                                                                                    \
  hipLaunchKernelGGL((norm_bwd_wave_kernel<T, C, L, O>), g, dim3(NT), 0, s, dx, dxo, dresm, dresd, xm, xd, dym, dyd,    \
                     rows, thg, vg, eps, (double)neps, part)
#define NWD(C)                    \
  do {                            \
    if (ln && osum) NW(C, true, true);  \
    else if (ln) NW(C, true, false);    \
    else if (osum) NW(C, false, true);  \
    else NW(C, false, false);     \
  } while (0)
    if (dm == 512) NWD(2);
    else if (dm == 1024) NWD(4);
    else NWD(8);
#undef NWD
#undef NW
    return hipGetLastError();
  }
  const int per = norm_bwd_rows(rows), ncol = dm * (1 + (ln ? 1 : 0) + (osum ? 1 : 0));
  const dim3 g(norm_bwd_groups(rows, dm));
#define NB(N, C)                                                                                                        \
  do {                                                                                                                  \
    if (ln) hipLaunchKernelGGL((norm_bwd_kernel<T, N, C, true>), g, dim3(N), 0, s, dx, dxo, dresm, dresd, xm, xd, dym,  \
                               dyd, rows, per, dm, thg, vg, eps, (double)neps, part, ncol, osum);                       \
    else hipLaunchKernelGGL((norm_bwd_kernel<T, N, C, false>), g, dim3(N), 0, s, dx, dxo, dresm, dresd, xm, xd, dym,    \
                            dyd, rows, per, dm, thg, vg, eps, (double)neps, part, ncol, osum);                          \
  } while (0)
  // as few chunks per thread as the registers of the column sums allow
  if (dm <= 256) NB(64, 1);
  else if (dm <= 512) NB(128, 1);
  else if (dm <= 1024) NB(256, 1);
  else if (dm <= 2048) NB(256, 2);
  else if (dm <= 4096) NB(512, 2);
  else NB(1024, 2);
#undef NB
  return hipGetLastError();
}

hipError_t launch_colsum_part(const ColSums& o, const double* part, int rows, int ncol, int C, double scale, bool acc,
                              hipStream_t s) {
  hipLaunchKernelGGL(colsum_part_kernel, dim3(ceil_div(ncol, 16)), dim3(1024), 0, s, o, part, rows, ncol, C, scale, acc);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_qkv_bias(PairT<T> out, const float* gm, const float* gd, int rows, int ncols, double* part, hipStream_t s) {
  const int groups = bias_groups(rows, ncols), per = (rows + groups - 1) / groups;
  hipLaunchKernelGGL(qkv_bias_kernel<T>, dim3(ceil_div(ncols / 4, NT), groups), dim3(NT), 0, s, out, gm, gd, rows, per,
                     ncols, part);
  return hipGetLastError();
}

hipError_t launch_rope_table(double* cs, int S, int dh, double base, hipStream_t s) {
  hipLaunchKernelGGL(rope_table_kernel, dim3(grid_for((int64_t)S * dh / 2)), dim3(NT), 0, s, cs, S, dh, base);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_rope_inplace(PairT<T> qkv, int T_, int S, int Hq, int Hk, int dh, const double* cs, hipStream_t s) {
  const int ncols = (Hq + 2 * Hk) * dh;
  const int units = (Hq + Hk) * dh / 8;
  const dim3 g(ceil_div(units, NT), T_);
  hipLaunchKernelGGL((qkv_rope_kernel<T, T>), g, dim3(NT), 0, s, qkv, (const T*)qkv.m, (const T*)qkv.d, S, ncols, Hq + Hk, dh,
                     cs, false, false);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_qkv_bwd_post(PairT<T> out, float* gm, float* gd, int T_, int S, int Hq, int Hk, int dh,
                               const double* cs, hipStream_t s) {
  const int ncols = (Hq + 2 * Hk) * dh;
  const int units = (Hq + Hk) * dh / 8 + (ncols - (Hq + Hk) * dh) / 4;
  const dim3 g(ceil_div(units, NT), T_);
  hipLaunchKernelGGL((qkv_rope_kernel<T, float>), g, dim3(NT), 0, s, out, (const float*)gm, (const float*)gd, S, ncols,
                     Hq + Hk, dh, cs, true, true);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_attn_softmax(PairT<T> P, const float* Sm, const float* Sd, int nrows, int S, hipStream_t s) {
  if (S > 4096) return hipErrorInvalidValue;
  const dim3 g(ceil_div(nrows, 4)), b(256);
  if (S <= 512) hipLaunchKernelGGL((attn_softmax_w<T, 8>), g, b, 0, s, P, Sm, Sd, nrows, S);
  else if (S <= 1024) hipLaunchKernelGGL((attn_softmax_w<T, 16>), g, b, 0, s, P, Sm, Sd, nrows, S);
  else if (S <= 2048) hipLaunchKernelGGL((attn_softmax_w<T, 32>), g, b, 0, s, P, Sm, Sd, nrows, S);
  else hipLaunchKernelGGL((attn_softmax_w<T, 64>), g, b, 0, s, P, Sm, Sd, nrows, S);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_attn_dsoftmax(PairT<T> dS, const T* Pm, const T* Pd, const float* dPm, const float* dPd, int nrows,
                                int S, hipStream_t s) {
  if (S > 4096) return hipErrorInvalidValue;
  const dim3 g(ceil_div(nrows, 4)), b(256);
  if (S <= 512) hipLaunchKernelGGL((attn_dsoftmax_w<T, 8>), g, b, 0, s, dS, Pm, Pd, dPm, dPd, nrows, S);
  else if (S <= 1024) hipLaunchKernelGGL((attn_dsoftmax_w<T, 16>), g, b, 0, s, dS, Pm, Pd, dPm, dPd, nrows, S);
  else if (S <= 2048) hipLaunchKernelGGL((attn_dsoftmax_w<T, 32>), g, b, 0, s, dS, Pm, Pd, dPm, dPd, nrows, S);
  else hipLaunchKernelGGL((attn_dsoftmax_w<T, 64>), g, b, 0, s, dS, Pm, Pd, dPm, dPd, nrows, S);
  return hipGetLastError();
}

hipError_t launch_group_sum(float* out, int64_t out_ld, const float* in, int T_, int Hk, int G, int dh, hipStream_t s) {
  hipLaunchKernelGGL(group_sum_kernel, dim3(grid_for((int64_t)T_ * Hk * dh)), dim3(NT), 0, s, out, out_ld, in, T_, Hk, G, dh);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_gelu_fwd(PairT<T> z, const T* um, const T* ud, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(gelu_fwd_kernel<T>, dim3(grid_for(n / 4)), dim3(NT), 0, s, z, um, ud, n / 4);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_gelu_bwd(PairT<T> du, const T* um, const T* ud, const float* dzm, const float* dzd, int rows, int F,
                           double* part, hipStream_t s) {
  const int groups = bias_groups(rows, F), per = (rows + groups - 1) / groups;
  hipLaunchKernelGGL(gelu_bwd_kernel<T>, dim3(ceil_div(F / 4, NT), groups), dim3(NT), 0, s, du, um, ud, dzm, dzd, rows, per,
                     F, part);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_swiglu_fwd(PairT<T> z, const T* gum, const T* gud, int rows, int F, hipStream_t s) {
  if (F % 4 == 0 && rows <= 65535) {
    // workgroups of 128 threads divide the 1.3B row (1408 groups of 4) exactly
    const int nt = (F / 4) % 128 == 0 ? 128 : NT;
    hipLaunchKernelGGL(swiglu_fwd4_kernel<T>, dim3(ceil_div(F / 4, nt), rows), dim3(nt), 0, s, z, gum, gud, F);
  }
  else
    hipLaunchKernelGGL(swiglu_fwd_kernel<T>, dim3(grid_for((int64_t)rows * F)), dim3(NT), 0, s, z, gum, gud, rows, F);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_swiglu_bwd(PairT<T> dgu, const T* gum, const T* gud, const float* dzm, const float* dzd, int rows,
                             int F, hipStream_t s) {
  if (F % 4 == 0 && rows <= 65535) {
    const int nt = (F / 4) % 128 == 0 ? 128 : NT;
    hipLaunchKernelGGL(swiglu_bwd4_kernel<T>, dim3(ceil_div(F / 4, nt), rows), dim3(nt), 0, s, dgu, gum, gud, dzm, dzd, F);
  }
  else
    hipLaunchKernelGGL(swiglu_bwd_kernel<T>, dim3(grid_for((int64_t)rows * F)), dim3(NT), 0, s, dgu, gum, gud, dzm, dzd, rows,
                       F);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_ce(PairT<T> dl, double* rowloss, const float* lm, const float* ld, const int32_t* tok,
                     const int32_t* lab, int T_, int S, int V, double inv_n, hipStream_t s) {
  // one step of the row loop over the whole workgroup is 4 NTH logits
  if (V >= 8192) hipLaunchKernelGGL((ce_kernel<T, 1024>), dim3(T_), dim3(1024), 0, s, dl, rowloss, lm, ld, tok, lab, T_, S, V, inv_n);
  else hipLaunchKernelGGL((ce_kernel<T, NT>), dim3(T_), dim3(NT), 0, s, dl, rowloss, lm, ld, tok, lab, T_, S, V, inv_n);
  return hipGetLastError();
}
hipError_t launch_loss_sum(double* out2, const double* rowloss, int T_, bool acc, hipStream_t s) {
  hipLaunchKernelGGL(loss_sum_kernel, dim3(1), dim3(NT), 0, s, out2, rowloss, T_, acc);
  return hipGetLastError();
}
hipError_t launch_count_targets(int64_t* out3, const int32_t* tok, const int32_t* lab, int B, int S, int V, hipStream_t s) {
  hipLaunchKernelGGL(count_targets_kernel, dim3(1), dim3(NT), 0, s, out3, tok, lab, B, S, V);
  return hipGetLastError();
}

hipError_t launch_token_sort(uint32_t* keys, const int32_t* tok, int T_, int V, hipStream_t s) {
  if (T_ > SORT_N) return hipErrorInvalidValue;
  hipLaunchKernelGGL(token_sort_kernel, dim3(ceil_div(T_, NT / 8)), dim3(NT), (size_t)(T_ + 3) / 4 * 16, s, keys, tok, T_, V);
  return hipGetLastError();
}
hipError_t launch_embed_bwd(float* hv, const uint32_t* keys, const float* dxd, int T_, int dm, double inv_eps, bool acc,
                            hipStream_t s) {
  hipLaunchKernelGGL(embed_bwd_kernel, dim3(T_, (dm + NT - 1) / NT), dim3(NT), 0, s, hv, keys, dxd, T_, dm, inv_eps,
                     acc);
  return hipGetLastError();
}
hipError_t launch_pos_bwd(float* hv, const float* dxd, int B, int S, int dm, double inv_eps, bool acc, hipStream_t s) {
  hipLaunchKernelGGL(pos_bwd_kernel, dim3(grid_for((int64_t)S * dm)), dim3(NT), 0, s, hv, dxd, B, S, dm, inv_eps, acc);
  return hipGetLastError();
}

#define INST_T(T)                                                                                                     \
  template hipError_t launch_cast_pair<T>(PairT<T>, const float*, const float*, int64_t, hipStream_t);                 \
  template hipError_t launch_embed_fwd<T>(PairF, const int32_t*, int, int, int, int, const T*, const float*, const T*, \
                                          const float*, double, int*, hipStream_t);                                    \
  template hipError_t launch_norm_fwd<T>(PairT<T>, const float*, const float*, int, int, bool, const T*, const float*, \
                                         const T*, const float*, double, float, hipStream_t);                          \
  template hipError_t launch_norm_bwd<T>(PairF, PairT<T>, const float*, const float*, const float*, const float*,      \
                                         const float*, const float*, int, int, bool, const T*, const float*, double,    \
                                         float, double*, bool, hipStream_t);                                           \
  template hipError_t launch_qkv_bias<T>(PairT<T>, const float*, const float*, int, int, double*, hipStream_t);        \
  template hipError_t launch_rope_inplace<T>(PairT<T>, int, int, int, int, int, const double*, hipStream_t);          \
  template hipError_t launch_qkv_bwd_post<T>(PairT<T>, float*, float*, int, int, int, int, int, const double*,         \
                                             hipStream_t);                                                             \
  template hipError_t launch_attn_softmax<T>(PairT<T>, const float*, const float*, int, int, hipStream_t);             \
  template hipError_t launch_attn_dsoftmax<T>(PairT<T>, const T*, const T*, const float*, const float*, int, int,      \
                                              hipStream_t);                                                            \
  template hipError_t launch_gelu_fwd<T>(PairT<T>, const T*, const T*, int64_t, hipStream_t);                          \
  template hipError_t launch_gelu_bwd<T>(PairT<T>, const T*, const T*, const float*, const float*, int, int, double*,  \
                                         hipStream_t);                                                                 \
  template hipError_t launch_swiglu_fwd<T>(PairT<T>, const T*, const T*, int, int, hipStream_t);                       \
  template hipError_t launch_swiglu_bwd<T>(PairT<T>, const T*, const T*, const float*, const float*, int, int,         \
                                           hipStream_t);                                                               \
  template hipError_t launch_ce<T>(PairT<T>, double*, const float*, const float*, const int32_t*, const int32_t*, int, \
                                   int, int, double, hipStream_t);
INST_T(float)
INST_T(bf16_t)

}  // namespace fdh
