// fp32 GEMM on the bf16 matrix cores:  C[z] = alpha * sum_p A_p[z] B_p[z]^T (+ epilogue).
//
// Each fp32 operand element is taken as the exact sum of three bf16 numbers
// x = h + m + l (8 significant bits each), and a product of two elements as
// the six partial products of weight 2^-16 and above,
//     hh + hm + mh + hl + mm + lh,
// accumulated in fp32.  The three left out (ml, lm, ll) are below 2^-23 of the
// product, with random signs, under the rounding of the fp32 accumulation
// itself.  gfx950 multiplies bf16 at sixteen times the rate of
// v_mfma_f32_32x32x2_f32, so six products leave 2.7 times the fp32 rate.
//
// Workgroup tile 128 x BN (BN = 128 or 64), four wavefronts of 64 x BN/2.  The
// fp32 tiles go straight from memory to LDS (buffer_load_dwordx4 ... lds) in
// slices of 32 k through a two-stage ring, two workgroups per CU; a wavefront
// splits the fragments it reads in registers (11 vector operations for two
// elements) between the matrix operations of the step before.  Splitting on
// the way into LDS instead would write 6 bytes per element through the LDS
// port (ds_write_b128 moves about a fifth of what ds_read_b128 does per clock).
// 8192 x 2048 x 512, both channels: 302 to 341 us (170 to 151 TFLOP/s, by the
// clock held under load); the fp32 matrix instructions with register-staged tiles
// took 1080 us for the two launches.
// Lanes outside the operand read past the buffer resource's range and get
// zeros, so K needs no alignment beyond the 16-byte chunk.
// An infinite element splits into inf and a NaN remainder: its products are NaN.
// (Through a model's norms and softmax every infinity ends as NaN, and the
// product is refused as non-finite.)  Elements below about 1e-33 keep fewer bits,
// as the remainders reach bf16's smallest number, 2^-133: relative errors of 5e-7
// at 1e-34, 3e-5 at 1e-36.
//
// LDS layouts (64 banks of 4 bytes; a 16-byte read is served 16 lanes at a time):
//   K-major: rows of 32 k = 128 bytes, 16-byte chunk c of row r at c ^ ((r >> 1) & 7);
//   MN-major: rows of BM or BN floats along m/n, chunk c of k-row k at
//     c ^ (8 ((k >> 2) & 1)); a fragment is eight 4-byte reads, whose two half
//     wavefronts (k-rows 4 apart) fall on different halves of the banks.
// Element e (0..7) of lane half h in a 16-deep step holds k = 8 (e >> 2) + 4 h + (e & 3)
// for both operands; the order within the step is free as long as they agree.
#include "gemm_dev.h"
#include "gemm_split.h"

namespace fdh {

namespace {

constexpr int BM = 128, KT = 32;
constexpr uint32_t OOB = 0x80000000u;   // byte offset at which the buffer resources end

__device__ inline i32x4_t rsrc_of(const float* base) {
  const uint64_t b = (uint64_t)(uintptr_t)base;
  return i32x4_t{(int)(uint32_t)b, (int)((b >> 32) & 0xffffu), (int)OOB, 0x00020000};
}

// 1 KB from the buffer at per-lane byte offset vo to LDS (64 lanes x 16 bytes, contiguous)
__device__ inline void dma16(uint32_t lds, i32x4_t rs, uint32_t vo) {
  asm volatile(
      "s_mov_b32 m0, %0\n\t"
      "s_nop 0\n\t"
      "buffer_load_dwordx4 %1, %2, 0 offen lds"
      :
      : "s"(lds), "v"(vo), "s"(rs)
      : "memory", "m0");
}

// One operand's tile of R rows x 32 k: source offsets of this wavefront's loads.
template <int R, bool KMAJ>
struct Tile {
  static constexpr int NI = R * KT * 4 / 1024;   // 1 KB loads per slice
  static constexpr int PER = NI / 4;             // per wavefront
  uint32_t vo[PER];                              // byte offsets from the slice origin
  int kq[PER];                                   // k of the lane's chunk within the slice

  __device__ inline void init(const GemmOperand& o, int rows, int row0, int wave, int lane) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int q = wave + 4 * u;
      if (KMAJ) {
        const int r = q * 8 + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
        kq[u] = 4 * c;
        vo[u] = 4u * (uint32_t)((int64_t)(min(row0 + r, rows - 1) - row0) * o.s_row + 4 * c);
      } else {
        constexpr int CPR = R / 4, RPI = 64 / CPR;   // chunks per k-row, k-rows per load
        const int k = q * RPI + lane / CPR, c = (lane % CPR) ^ (8 * ((k >> 2) & 1));
        kq[u] = k;
        vo[u] = 4u * (uint32_t)((int64_t)k * o.s_k + (min(row0 + 4 * c, rows - 4) - row0));
      }
    }
  }
  // loads of the slice at k0 (left = k's remaining in the contraction from k0)
  __device__ inline void issue(const float* base, int left, uint32_t lds, int wave) const {
    const i32x4_t rs = rsrc_of(base);
#pragma unroll
    for (int u = 0; u < PER; ++u) dma16(lds + (wave + 4 * u) * 1024, rs, kq[u] < left ? vo[u] : OOB);
  }
};

// the eight fp32 elements of one 32-row fragment at k step kk (0 or 16)
template <int R, bool KMAJ>
__device__ inline void read8(float (&x)[8], const float* t, int r0, int kk, int lane) {
  const int h = lane >> 5;
  if (KMAJ) {
    const int r = r0 + (lane & 31);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const float4 v = *reinterpret_cast<const float4*>(t + r * KT + (((kk >> 2) + 2 * j + h) ^ ((r >> 1) & 7)) * 4);
      x[4 * j] = v.x; x[4 * j + 1] = v.y; x[4 * j + 2] = v.z; x[4 * j + 3] = v.w;
    }
  } else {
    const float* p = t + (kk + 4 * h) * R + ((r0 + (lane & 31)) ^ (32 * h));
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = p[(8 * (e >> 2) + (e & 3)) * R];
  }
}

struct Frag { bf16x8_t h, m, l; };

typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2_t;
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// x = h + m + l exactly: h the upper half of the word (truncated), m the
// remainder rounded to bf16, l what is left (at most 8 bits: its word's lower
// half is zero).  (Remainders by v_dot2_f32_bf16, which needs no unpacking,
// take seven operations instead of eleven, but that instruction does not run
// beside matrix operations.)
__device__ inline Frag split3(const float (&x)[8]) {
  u32x4_t h, m, l;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t a = __builtin_bit_cast(uint32_t, x[2 * i]), b = __builtin_bit_cast(uint32_t, x[2 * i + 1]);
    const float ra = x[2 * i] - __builtin_bit_cast(float, a & 0xFFFF0000u);
    const float rb = x[2 * i + 1] - __builtin_bit_cast(float, b & 0xFFFF0000u);
    h[i] = __builtin_amdgcn_perm(b, a, 0x07060302u);
    uint32_t mm;
    asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(mm) : "v"(ra), "v"(rb));
    m[i] = mm;
    const float sa = ra - __builtin_bit_cast(float, mm << 16);
    const float sb = rb - __builtin_bit_cast(float, mm & 0xFFFF0000u);
    l[i] = __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, sb), __builtin_bit_cast(uint32_t, sa), 0x07060302u);
  }
  return {__builtin_bit_cast(bf16x8_t, h), __builtin_bit_cast(bf16x8_t, m), __builtin_bit_cast(bf16x8_t, l)};
}

// What a workgroup computes: its product, output tile, slices and operand loads.
template <int BN, bool AK, bool BKM>
struct Work {
  static constexpr int SSZ = (BM + BN) * KT;                            // floats per ring stage
  static constexpr int PERT = Tile<BM, AK>::PER + Tile<BN, BKM>::PER;   // loads per slice and wavefront
  int prod, part, z, m0, n0, kmin, kmax, nkt, t0, t1, wave, lane;
  const float* pa[2];
  const float* pb[2];
  int64_t ska, skb;
  uint32_t lds0;
  Tile<BM, AK> ta;
  Tile<BN, BKM> tb;

  // false: an output tile that a causal product leaves out
  __device__ inline bool init(const GemmJob& job, const float* ring) {
    prod = (int)blockIdx.x >= job.nblk0 ? 1 : 0;
    const GemmArgs& a = job.g[prod];
    const int nblk = prod ? (int)gridDim.x - job.nblk0 : job.nblk0;
    const int lin = xcd_order((int)blockIdx.x - (prod ? job.nblk0 : 0), nblk);
    const int gx = (a.N + BN - 1) / BN, gy = (a.M + BM - 1) / BM;
    const int tiles = gx * gy;
    const int sp = lin / (tiles * a.nbatch), rest = lin % (tiles * a.nbatch);
    const int tl = rest % tiles;
    z = rest / tiles;
    part = sp * a.nbatch + z;
    constexpr int GM = 8;
    const int gsize = GM * gx, first_m = (tl / gsize) * GM;
    const int gm_rows = min(gy - first_m, GM);
    m0 = (first_m + (tl % gsize) % gm_rows) * BM;
    n0 = ((tl % gsize) / gm_rows) * BN;
    if (a.causal == CAUSAL_SKIP_UPPER && n0 > m0 + BM - 1) return false;
    lane = threadIdx.x & 63;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    kmin = 0;
    kmax = a.K;
    if (a.causal == CAUSAL_K_LE_M) kmax = min(a.K, m0 + BM);
    if (a.causal == CAUSAL_K_GE_M) kmin = (min(m0, a.K) / KT) * KT;
    nkt = kmax > kmin ? (kmax - kmin + KT - 1) / KT : 0;
    // this workgroup's slices of the pair-concatenated contraction
    t0 = sp * job.len;
    t1 = min(nkt * a.npairs, t0 + job.len);
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const GemmOperand& A = a.A[p < a.npairs ? p : 0];
      const GemmOperand& B = a.B[p < a.npairs ? p : 0];
      pa[p] = reinterpret_cast<const float*>(A.ptr) + batch_off(z, a.inner_count, A.s_outer, A.s_inner, A.inner_div) +
              (AK ? (int64_t)m0 * A.s_row : (int64_t)m0);
      pb[p] = reinterpret_cast<const float*>(B.ptr) + batch_off(z, a.inner_count, B.s_outer, B.s_inner, B.inner_div) +
              (BKM ? (int64_t)n0 * B.s_row : (int64_t)n0);
    }
    // both pairs share the lane offsets (equal strides: checked on the host)
    ta.init(a.A[0], a.M, m0, wave, lane);
    tb.init(a.B[0], a.N, n0, wave, lane);
    ska = a.A[0].s_k;
    skb = a.B[0].s_k;
    lds0 = (uint32_t)(uintptr_t)(lds_void_t*)ring;
    return true;
  }
  // loads of slice t into stage t & 1 (past the last slice every lane reads
  // out of range: no branch in the loop)
  __device__ inline void issue(int t) const {
    const uint32_t lds = lds0 + (uint32_t)((t & 1) * SSZ * 4);
    const int tc = min(t, t1 - 1);
    const int p = tc >= nkt ? 1 : 0;
    const int k0 = kmin + (tc - p * nkt) * KT;
    const int left = t < t1 ? kmax - k0 : 0;
    ta.issue((p ? pa[1] : pa[0]) + k0 * ska, left, lds, wave);
    tb.issue((p ? pb[1] : pb[0]) + k0 * skb, left, lds + BM * KT * 4, wave);
  }
  template <typename ACC>
  __device__ inline void store(const GemmJob& job, const ACC& acc, int i, int j) const {
    const GemmArgs& a = job.g[prod];
    const int rb = m0 + (wave >> 1) * 64 + i * 32, cb = n0 + (wave & 1) * (BN / 2) + j * 32;
    if (job.splits[prod] > 1) store_partial(job, prod, acc, part, rb, cb, lane);
    else store_block<float>(a, acc, batch_off(z, a.inner_count, a.c_outer, a.c_inner, a.c_div), rb, cb, lane);
  }
};

template <int BN, bool AK, bool BKM>
__global__ __launch_bounds__(256, 2) void gemm_f32_kernel(GemmJob job) {
  typedef Work<BN, AK, BKM> W;
  constexpr int IM = 2, JN = BN / 64;
  __shared__ __attribute__((aligned(1024))) float ring[2][W::SSZ];
  W w;
  if (!w.init(job, &ring[0][0])) return;
  const int lane = w.lane, wm = w.wave >> 1, wn = w.wave & 1;

  // The leading products hh have accumulators of their own: a matrix operation
  // rounds into its accumulator once per 16 k, and the five others, 2^-8 and
  // less of it, would round there five times more (at K = 8192 that is
  // 1.8e-6 of an HVP's result against 3e-7).
  f32x16_t acc[IM][JN], low[IM][JN];
#pragma unroll
  for (int i = 0; i < IM; ++i)
#pragma unroll
    for (int j = 0; j < JN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = low[i][j][r] = 0.f;

  // One 16-deep step: the 6 IM JN matrix operations on the fragments cur, and
  // between them the reads and splits of the next step's fragments into nxt
  // (issued by themselves ahead of the matrix operations, the splits left the
  // matrix cores idle for half of the time).  The products with l come first,
  // so that its registers are free early.
  constexpr int NF = IM + JN, NM = 6 * IM * JN;
  auto mma = [&](const Frag (&f)[NF], int e) {
    const int i = (e % (IM * JN)) / JN, j = e % JN;
    const Frag &A = f[i], &B = f[IM + j];
    // B first: a lane then holds four consecutive columns of one row of C
#define MM(ACC, X, Y) ACC[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(B.Y, A.X, ACC[i][j], 0, 0, 0)
    switch (e / (IM * JN)) {
      case 0: MM(low, h, l); break;
      case 1: MM(low, l, h); break;
      case 2: MM(low, m, m); break;
      case 3: MM(low, h, m); break;
      case 4: MM(low, m, h); break;
      default: MM(acc, h, h); break;
    }
#undef MM
  };
  auto rd = [&](float (&x)[8], const float* st, int f, int kk) {
    if (f < IM) read8<BM, AK>(x, st, wm * 64 + f * 32, kk, lane);
    else read8<BN, BKM>(x, st + BM * KT, wn * (BN / 2) + (f - IM) * 32, kk, lane);
  };
  auto step = [&](const Frag (&cur)[NF], Frag (&nxt)[NF], const float* st, int kk) {
    float x[2][8];
    rd(x[0], st, 0, kk);
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      if (f + 1 < NF) rd(x[(f + 1) & 1], st, f + 1, kk);
#pragma unroll
      for (int e = f * NM / NF; e < (f + 1) * NM / NF; ++e) mma(cur, e);
      nxt[f] = split3(x[f & 1]);
      // (formed here: without this the compiler sinks the split to the next step)
      asm volatile("" : "+v"(nxt[f].h), "+v"(nxt[f].m), "+v"(nxt[f].l));
#pragma unroll
      for (int e = 0; e < NM / NF; ++e) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one matrix operation,
        __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);   // eight vector ones
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  Frag f0[NF], f1[NF];
  if (w.t0 < w.t1) {
    w.issue(w.t0);
    w.issue(w.t0 + 1);
    wait_vm<W::PERT>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      float x[8];
      rd(x, ring[w.t0 & 1], f, 0);
      f0[f] = split3(x);
    }
    for (int t = w.t0; t < w.t1; ++t) {
      step(f0, f1, ring[t & 1], 16);
      // own loads of slice t + 1 and own reads of this stage done, then
      // everyone's: the stage is free for slice t + 2
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      w.issue(t + 2);
      step(f1, f0, ring[(t + 1) & 1], 0);   // (after the last slice: zeros, not used)
    }
    wait_vm<0>();   // no load may land in LDS after the workgroup ends
  }
#pragma unroll
  for (int i = 0; i < IM; ++i)
#pragma unroll
    for (int j = 0; j < JN; ++j) {
      acc[i][j] += low[i][j];
      w.store(job, acc[i][j], i, j);
    }
}

template <int BN, bool AK, bool BKM>
void launch_t(const GemmJob& j, int blocks, hipStream_t s) {
  hipLaunchKernelGGL((gemm_f32_kernel<BN, AK, BKM>), dim3(blocks), dim3(256), 0, s, j);
}
template <int BN>
void launch_bn(const GemmJob& j, int blocks, hipStream_t s) {
  const bool ak = j.g[0].A[0].s_k == 1, bk = j.g[0].B[0].s_k == 1;
  if (ak && bk) launch_t<BN, true, true>(j, blocks, s);
  else if (ak && !bk) launch_t<BN, true, false>(j, blocks, s);
  else if (!ak && bk) launch_t<BN, false, true>(j, blocks, s);
  else launch_t<BN, false, false>(j, blocks, s);
}

}  // namespace

// Costs of the two tile widths, measured: 8192^3 with two pairs runs at 198
// TFLOP/s, 1.38 us per slice and CU, power-bound (1.6 GHz, matrix cores 70%
// busy); 64 workgroups alone on their CUs take 0.95 us per slice.
// The leading accumulator rounds once per 16 k, so a part of 128 slices (4096
// k) keeps the error of its sum near 2e-7 of the magnitudes.
static const GemmCost COST128{BM, 128, KT, 1.38, 0.95, 7.0, 2, 128}, COST64{BM, 64, KT, 0.8, 0.62, 6.0, 2, 128};

static const GemmCost& pick(const GemmArgs* g, int n, size_t scratch, GemmPlan& pl) {
  pl = plan_splits(g, n, COST64, scratch);
  if (g[0].N <= 64) return COST64;
  const GemmPlan wide = plan_splits(g, n, COST128, scratch);
  if (pl.us < wide.us) return COST64;
  pl = wide;
  return COST128;
}

size_t gemm_f32_scratch(const GemmArgs* g, int n, size_t most) {
  GemmPlan pl;
  pick(g, n, most, pl);
  return pl.bytes;
}

void gemm_f32_plan(const GemmArgs* g, int n, size_t scratch, int32_t (&out)[4]) {
  GemmPlan pl;
  out[0] = pick(g, n, scratch, pl).BN;
  out[1] = pl.len;
  out[2] = pl.splits[0];
  out[3] = pl.splits[1];
}

hipError_t gemm_f32(const GemmArgs* g, int n, const GemmScratch& ws, hipStream_t stream) {
  if (g[0].M == 0 || g[0].N == 0) return hipSuccess;
  GemmJob j;
  GemmPlan pl;
  const GemmCost& c = pick(g, n, ws.bytes, pl);
  if (pl.bytes > ws.held) return hipErrorInvalidValue;
  const int blocks = make_job(j, g, n, pl, c, ws.p);
  if (c.BN == 64) launch_bn<64>(j, blocks, stream);
  else launch_bn<128>(j, blocks, stream);
  const hipError_t r = hipGetLastError();
  return r != hipSuccess ? r : reduce_splits<float>(j, n, stream);
}

}  // namespace fdh
