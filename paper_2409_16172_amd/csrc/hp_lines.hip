// Mixed-radix lines (N = 2^a 3^b 5^c, not a power of two; the grids of Example 1,
// Section 5.1) held in registers: the four transform passes of the preconditioner
// apply (Eqn. 403) with two to four stages of radix up to 16 per line.
//
// A line of N = r_0 r_1 .. points is transformed by T = N / min r threads.  In a stage
// of radix r, N/r of them hold one butterfly each in registers; stages exchange through
// LDS.  Before stage s the line is the matrix [k < K][j < J r] (K the product of the
// earlier radices, J of the later ones); butterfly (k, j) takes its inputs J apart and
// leaves its outputs at [k + K t][j].  The first stage takes its inputs from the pass
// itself (global loads, or the symbol multiply on the spectrum kept in registers) and
// the last gives its outputs back to it (stores, or the weighted sum), so a three-stage
// transform touches LDS four times per element; the LDS-resident stages of
// hp_kernels.hip (which remain for the lengths make_line_plan refuses) touch it eight
// times and more, and keep a fixed wavefront multiple of threads busy however short the
// line.  Any number of lines shares a workgroup: thread = (line, butterfly) for rows,
// (butterfly, column) for columns, so short lines fill the wavefronts.
//
// LDS layout: the exchange before the last stage is stored [j][k] with an odd row pitch,
// the earlier ones [k][j] with a pitch equal to the next stage's J modulo the elements
// of one 128-byte LDS access, so that consecutive lanes meet distinct banks on both
// sides of every exchange, and every index advances by a constant.
#include <algorithm>

#include "hp_device.h"

namespace hp {

// Workgroup barrier ordering LDS only (global loads and stores stay in flight).
__device__ __forceinline__ void line_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Waves per SIMD the kernels of passes B and C are compiled for.  FP64: three (168 VGPRs)
// with radices up to kLineRadixLo, two above.  FP32: four and, in pass C with radices up
// to 16, three (pass B takes its 29 spilled registers for the fourth wave: 1920 x 1500,
// K = 19, 268 -> 233 us; pass C does not: 2400^2, K = 8, 52 us with three, 71 with four).
// FP64 pass C in the other interpolation modes, whose records and weights take more
// registers, gives a wave up where it would spill 172 to 288 bytes a lane (Lagrange 576^2,
// K = 15, sixteen fields: 1450 -> 900 us; FP32 spills 32 to 148 and is better off so: 320 x
// 486, K = 8, 14 us, 18 with a wave less).
__host__ __device__ constexpr int line_waves(bool fp64, int rm, int kind, int im = kInterpLinear) {
  const bool less = kind == kLineComb && im != kInterpLinear;
  return fp64 ? (rm <= kLineRadixLo && !less ? 3 : 2) : (rm <= kLineRadixLo || kind == kLineSym ? 4 : 3);
}
#define HP_LINE_WAVES(R, RM, ...) __attribute__((amdgpu_waves_per_eu(line_waves(sizeof(R) == 8, RM, __VA_ARGS__))))

enum LineStageKind { kStageFirst = 0, kStageMid = 1, kStageLast = 2 };

// Where a transform's exchanges live: element a of this thread's line at buf[a * mul],
// in two alternating regions reg_elems apart (one when the plan has no second buffer).
template <typename R>
struct LineBuf {
  cpx<R>* buf;
  int mul, reg_elems, cur;
};

// One stage of radix RAD for the thread of index tl of its line (live: the line exists
// and takes part).  The pass's context c fills the inputs of the first stage (in) and
// takes the outputs of the last (out); it is one struct handed down by reference, with
// its register arrays as members, so that the compiler keeps them in registers through
// the radix switches.  tw: this stage's part of the plan's stage table in LDS (TWL), entry
// (t - 1) K + k, else the line's table exp(-2 pi i m / N) in global memory.
template <typename R, int RAD, int DIR, int KIND, bool TWL, typename Ctx>
__device__ __forceinline__ void line_stage(const LinePlan& p, int s, LineBuf<R>& b, int tl, int mk, bool live,
                                           const cpx<R>* __restrict__ tw, Ctx& c) {
  const int J = p.J[s], K = p.K[s], mul = b.mul;
  const bool act = live && tl < J * K;
  int j = 0, k = 0;
  if constexpr (KIND == kStageFirst) {
    j = tl;
  } else if constexpr (KIND == kStageMid) {
    k = mk;
    j = tl - k * J;
  } else {
    k = tl;
  }
  cpx<R> v[RAD];
  if (act) {
    if constexpr (KIND == kStageFirst) {
      c.template in<DIR>(v);
    } else {
      const int pitch = p.pitch[s - 1];
      const cpx<R>* rd = b.buf + b.cur * b.reg_elems;
      int a = KIND == kStageLast ? k * mul : (k * pitch + j) * mul;
      const int da = (KIND == kStageLast ? pitch : J) * mul;
#pragma unroll
      for (int t = 0; t < RAD; ++t, a += da) v[t] = rd[a];
      int q = TWL ? k : k * J;
      const int dq = TWL ? K : k * J;
#pragma unroll
      for (int t = 1; t < RAD; ++t, q += dq) {
        const cpx<R> w = tw[q];
        v[t] = DIR < 0 ? cmul(v[t], w) : cmulc(v[t], w);
      }
    }
    dft_radix<R, RAD, DIR>(v);
  }
  if constexpr (KIND == kStageLast) {
    if (act) c.template out<DIR>(v);
  } else {
    if (p.two_buf) {
      if (KIND == kStageMid) b.cur ^= 1;
    } else {
      line_barrier();   // the readers of the region are done
    }
    if (act) {
      const int pitch = p.pitch[s];
      cpx<R>* wr = b.buf + b.cur * b.reg_elems;
      const bool to_last = s + 2 == p.nst;
      int a = (to_last ? j * pitch + k : k * pitch + j) * mul;
      const int da = (to_last ? K : K * pitch) * mul;
#pragma unroll
      for (int t = 0; t < RAD; ++t, a += da) wr[a] = v[t];
    }
  }
}

template <typename R, int DIR, int KIND, bool TWL, int RM, typename Ctx>
__device__ __forceinline__ void line_stage_any(const LinePlan& p, int s, LineBuf<R>& b, int tl, int mk, bool live,
                                               const cpx<R>* __restrict__ tw, Ctx& c) {
  switch (p.r[s]) {   // the plan's radices are at most RM
#define HP_LINE_CASE(RAD)                                                                     \
  case RAD:                                                                                   \
    if constexpr (RAD <= RM) line_stage<R, RAD, DIR, KIND, TWL>(p, s, b, tl, mk, live, tw, c); \
    break;
    HP_LINE_CASE(2)
    HP_LINE_CASE(3)
    HP_LINE_CASE(4)
    HP_LINE_CASE(5)
    HP_LINE_CASE(6)
    HP_LINE_CASE(8)
    HP_LINE_CASE(9)
    HP_LINE_CASE(10)
    HP_LINE_CASE(12)
    HP_LINE_CASE(15)
    HP_LINE_CASE(16)
    default: break;
#undef HP_LINE_CASE
  }
}

// The k of this thread's butterfly in each middle stage (j = tl - k J), once per kernel.
__device__ __forceinline__ void line_mid_k(const LinePlan& p, int tl, int (&mk)[2]) {
  mk[0] = p.nst > 2 ? tl / p.J[1] : 0;
  mk[1] = p.nst > 3 ? tl / p.J[2] : 0;
}

// The transform of one line; every thread of the workgroup calls it together.  TWL: tw is
// the stage table, else the line's table.
template <typename R, int DIR, bool TWL, int RM, typename Ctx>
__device__ __forceinline__ void line_fft(const LinePlan& p, LineBuf<R>& b, int tl, const int (&mk)[2], bool live,
                                         const cpx<R>* __restrict__ tw, Ctx& c) {
  line_stage_any<R, DIR, kStageFirst, TWL, RM>(p, 0, b, tl, 0, live, tw, c);
  const cpx<R>* t = tw;
  for (int s = 1; s + 1 < p.nst; ++s) {
    line_barrier();
    line_stage_any<R, DIR, kStageMid, TWL, RM>(p, s, b, tl, s == 1 ? mk[0] : mk[1], live, t, c);
    if (TWL) t += p.K[s] * (p.r[s] - 1);
  }
  line_barrier();
  line_stage_any<R, DIR, kStageLast, TWL, RM>(p, p.nst - 1, b, tl, 0, live, t, c);
  if (p.two_buf) b.cur ^= 1;   // the next transform writes the other region
}

// The plan's stage table (p.twn entries) into LDS.
template <typename R>
__device__ __forceinline__ void line_tables(const LinePlan& p, cpx<R>* dst, const cpx<R>* __restrict__ stw) {
  for (int q = threadIdx.x; q < p.twn; q += blockDim.x) dst[q] = stw[q];
}

// Lines read from and written to global memory, elements step apart.
template <typename R, typename TI>
struct CopyCtx {
  const cpx<TI>* src;
  cpx<R>* dst;
  size_t in_step, out_step;
  template <int DIR, int RAD>
  __device__ __forceinline__ void in(cpx<R> (&v)[RAD]) const {
#pragma unroll
    for (int t = 0; t < RAD; ++t) v[t] = cvt<R>(src[t * in_step]);
  }
  template <int DIR, int RAD>
  __device__ __forceinline__ void out(const cpx<R> (&v)[RAD]) const {
#pragma unroll
    for (int t = 0; t < RAD; ++t) dst[t * out_step] = v[t];
  }
};

// ---------------------------------------------------------------- pass A
template <typename R, typename TI>
__global__ __launch_bounds__(kLineMaxThr) void k_line_rows(const cpx<TI>* __restrict__ in, cpx<R>* __restrict__ out,
                                                           int rows, size_t in_rs, size_t out_rs, LinePlan p,
                                                           const cpx<R>* __restrict__ tw,
                                                           const int* __restrict__ skip) {
  extern __shared__ char dyn_lds[];
  const int rhs = blockIdx.y;
  if (skip != nullptr && skip[rhs] != 0) return;
  const int line = (int)threadIdx.x / p.T, tl = (int)threadIdx.x - line * p.T;
  const int row = (int)blockIdx.x * p.L + line;
  const bool live = line < p.L && row < rows;
  LineBuf<R> b{reinterpret_cast<cpx<R>*>(dyn_lds) + line * p.slots, 1, p.L * p.slots, 0};
  int mk[2];
  line_mid_k(p, tl, mk);
  CopyCtx<R, TI> c{in + (size_t)rhs * in_rs + (size_t)row * p.n + tl,
                   out + (size_t)rhs * out_rs + (size_t)row * p.n + tl, (size_t)p.J[0], (size_t)p.K[p.nst - 1]};
  line_fft<R, -1, false, kLineRadixMax>(p, b, tl, mk, live, tw, c);
}

// ---------------------------------------------------------------- strided passes
// Plain transform of L adjacent columns per workgroup (element (o, p, c) at
// o n S + p S + c); slabs that no point of node field `fld` uses are skipped.
template <typename R, int DIR>
__global__ __launch_bounds__(kLineMaxThr) void k_line_cols(const cpx<R>* __restrict__ in, cpx<R>* __restrict__ out,
                                                           int S, int nfields, size_t in_rs, size_t out_rs,
                                                           size_t in_fs, size_t out_fs, LinePlan p,
                                                           const cpx<R>* __restrict__ tw,
                                                           const int* __restrict__ skip,
                                                           const uint8_t* __restrict__ need) {
  extern __shared__ char dyn_lds[];
  const int rhs = (int)blockIdx.z / nfields, fld = (int)blockIdx.z % nfields;
  if (skip != nullptr && skip[rhs] != 0) return;
  int tile, slab;
  xcd_tile(blockIdx.x, blockIdx.y, gridDim.x, gridDim.y, &tile, &slab);
  if (need != nullptr && need[(size_t)fld * gridDim.y + slab] == 0) return;
  const int tl = (int)threadIdx.x / p.L, g = (int)threadIdx.x - tl * p.L;
  const int c = tile * p.L + g;
  const bool live = c < S;
  const size_t base = (size_t)slab * p.n * S + (size_t)tl * S + c;
  LineBuf<R> b{reinterpret_cast<cpx<R>*>(dyn_lds) + g, p.L, p.L * p.slots, 0};
  int mk[2];
  line_mid_k(p, tl, mk);
  CopyCtx<R, R> ctx{in + (size_t)rhs * in_rs + (size_t)fld * in_fs + base,
                    out + (size_t)rhs * out_rs + (size_t)fld * out_fs + base, (size_t)p.J[0] * S,
                    (size_t)p.K[p.nst - 1] * S};
  line_fft<R, DIR, false, kLineRadixMax>(p, b, tl, mk, live, tw, ctx);
}

// What pass B holds of a column: forward, its loads and then the spectrum; inverse, the
// symbol multiply and the stores of the axis-0 indices in the mask.
template <typename R, int RM>
struct SymCtx {
  static constexpr int E = line_spectrum_max<R, RM>();
  cpx<R> vh[E];
  double lam[E];
  NodeConst nc;
  R scale;
  unsigned mask;
  const cpx<R>* src;
  cpx<R>* dst;
  size_t in_step, out_step;
  // (the plan's last forward radix, its first inverse one, is at most E)
  template <int DIR, int RAD>
  __device__ __forceinline__ void in(cpx<R> (&v)[RAD]) {
    if constexpr (DIR < 0) {
#pragma unroll
      for (int t = 0; t < RAD; ++t) v[t] = src[t * in_step];
    } else if constexpr (RAD <= E) {
      symbol_mul(vh, v, lam, nc);
    }
  }
  template <int DIR, int RAD>
  __device__ __forceinline__ void out(const cpx<R> (&v)[RAD]) {
    if constexpr (DIR > 0) {
#pragma unroll
      for (int t = 0; t < RAD; ++t)
        if ((mask >> t) & 1u) dst[t * out_step] = v[t];
    } else if constexpr (RAD <= E) {
#pragma unroll
      for (int t = 0; t < RAD; ++t) vh[t] = cscale(v[t], scale);
    }
  }
};

// Pass B: forward transform of L adjacent columns (plan fw), then for every node of this
// workgroup's group the symbol multiply and the inverse transform (plan iv, the radices
// of fw reversed, so that the spectrum a thread holds is the input of its own first
// butterfly), storing the axis-0 indices whose rows use the node.
template <typename R, int RM>
__global__ __launch_bounds__(kLineMaxThr) HP_LINE_WAVES(R, RM, kLineSym) void k_line_sym(const cpx<R>* __restrict__ in, cpx<R>* __restrict__ out,
                                                          int S, size_t in_rs, size_t out_rs, size_t out_fs,
                                                          LinePlan fw, LinePlan iv, const cpx<R>* __restrict__ tw,
                                                          const cpx<R>* __restrict__ stw,
                                                          const int* __restrict__ skip,
                                                          const double* __restrict__ lam_ax,
                                                          const double* __restrict__ lam_in,
                                                          const NodeConst* __restrict__ nodes, int K, double scale,
                                                          const uint16_t* __restrict__ smask) {
  extern __shared__ char dyn_lds[];
  const int rhs = blockIdx.z;
  if (skip != nullptr && skip[rhs] != 0) return;
  const int L = fw.L, tl = (int)threadIdx.x / L, g = (int)threadIdx.x - tl * L;
  int tile, grp;
  xcd_tile(blockIdx.x, blockIdx.y, gridDim.x, gridDim.y, &tile, &grp);
  const int c = tile * L + g;
  const bool live = c < S;
  cpx<R>* lds = reinterpret_cast<cpx<R>*>(dyn_lds);
  const int reg = L * fw.slots;
  cpx<R>* tab = lds + reg * (fw.two_buf ? 2 : 1);
  LineBuf<R> b{lds + g, L, reg, 0};
  line_tables<R>(iv, tab, stw);   // the transform's barriers come before their first use
  int mk[2];
  line_mid_k(fw, tl, mk);
  const int J0 = iv.J[0], KL = iv.K[iv.nst - 1];
  SymCtx<R, RM> ctx;
  ctx.scale = (R)scale;
  ctx.src = in + (size_t)rhs * in_rs + (size_t)tl * S + c;
  ctx.in_step = (size_t)fw.J[0] * S;
  ctx.out_step = (size_t)KL * S;
  line_fft<R, -1, false, RM>(fw, b, tl, mk, live, tw, ctx);
  const double lc = live ? lam_in[c] : 0.0;
#pragma unroll
  for (int t = 0; t < SymCtx<R, RM>::E; ++t) ctx.lam[t] = (t < iv.r[0] && tl < J0 ? lam_ax[tl + t * J0] : 0.0) + lc;
  line_mid_k(iv, tl, mk);
  const bool stores = live && tl < KL;
  const int n_lo = (int)(((long)grp * K) / gridDim.y), n_hi = (int)(((long)(grp + 1) * K) / gridDim.y);
  for (int n = n_lo; n < n_hi; ++n) {
    ctx.nc = nodes[n];
    ctx.mask = stores ? smask[(size_t)n * KL + tl] : 0u;
    ctx.dst = out + (size_t)rhs * out_rs + (size_t)n * out_fs + (size_t)tl * S + c;
    line_fft<R, +1, true, RM>(iv, b, tl, mk, live, tab, ctx);
  }
}

// ---------------------------------------------------------------- pass C
// What pass C holds of a row: its points' records and sums.
template <typename R, int IM, int RM>
struct CombCtx {
  static constexpr int E = line_spectrum_max<R, RM>();
  CombPoint<R, IM> pt[E];
  cpx<R> acc[E];
  const cpx<R>* src;
  size_t in_step;
  int n, M, mo, ord;
  const double* lag;
  template <int DIR, int RAD>
  __device__ __forceinline__ void in(cpx<R> (&v)[RAD]) const {
#pragma unroll
    for (int t = 0; t < RAD; ++t) v[t] = src[t * in_step];
  }
  template <int DIR, int RAD>
  __device__ __forceinline__ void out(const cpx<R> (&v)[RAD]) {
    if constexpr (RAD <= E) {
#pragma unroll
      for (int t = 0; t < RAD; ++t) {
        const R w = pt[t].weight(n, M, mo, ord, lag);
        acc[t].re += w * v[t].re;
        acc[t].im += w * v[t].im;
      }
    }
  }
};

// Inverse transform of every node row some row of the workgroup uses and the weighted
// sum of each point, L rows per workgroup (SPLIT: L / splits rows, each shared by
// `splits` lines that take its nodes in turn, where the rows alone are too few).
template <typename R, typename TO, bool ACC, int IM, int RM, bool SPLIT>
__global__ __launch_bounds__(kLineMaxThr) HP_LINE_WAVES(R, RM, kLineComb, IM) void k_line_combine(const cpx<R>* __restrict__ fields, size_t fs,
                                                              size_t frs, const double* __restrict__ pos,
                                                              const uint64_t* __restrict__ rowmask,
                                                              cpx<TO>* __restrict__ out, size_t out_rs, int rows,
                                                              int M, int Mt, int mo, LinePlan p,
                                                              const cpx<R>* __restrict__ stw,
                                                              const int* __restrict__ skip, int ord,
                                                              const double* __restrict__ lag,
                                                              const double* __restrict__ posa, int Ma) {
  constexpr int E = CombCtx<R, IM, RM>::E;
  constexpr bool LAG = IM == kInterpLagrange;
  extern __shared__ char dyn_lds[];
  __shared__ double slag[LAG ? kLagTable : 1];
  const int rhs = blockIdx.y;
  if (skip != nullptr && skip[rhs] != 0) return;
  if constexpr (LAG) {
    for (int i = threadIdx.x; i < kLagTable; i += blockDim.x) slag[i] = lag[i];
    __syncthreads();
  }
  // SPLIT: line sp * nrow + i takes every p.splits-th node of row i from its sp-th on
  const int line = (int)threadIdx.x / p.T, tl = (int)threadIdx.x - line * p.T;
  const int nrow = SPLIT ? p.L / p.splits : p.L;
  const int sp = SPLIT ? line / nrow : 0;
  const int row0 = (int)blockIdx.x * nrow, row = row0 + (SPLIT ? line - sp * nrow : line);
  const bool live = line < p.L && row < rows;
  cpx<R>* lds = reinterpret_cast<cpx<R>*>(dyn_lds);
  const int reg = p.L * p.slots;
  cpx<R>* tab = lds + reg * (p.two_buf ? 2 : 1);
  LineBuf<R> b{lds + line * p.slots, 1, reg, 0};
  line_tables<R>(p, tab, stw);
  int mk[2];
  line_mid_k(p, tl, mk);
  const int KL = p.K[p.nst - 1], RL = p.r[p.nst - 1];
  const size_t rbase = (size_t)row * p.n + tl;
  const bool mine = live && tl < KL;
  CombCtx<R, IM, RM> c;
  c.in_step = (size_t)p.J[0];
  c.M = M;
  c.mo = mo;
  c.ord = ord;
  c.lag = slag;
#pragma unroll
  for (int t = 0; t < E; ++t) {
    c.pt[t].clear();
    if (t < RL && mine) {
      const size_t i = rbase + (size_t)t * KL;
      c.pt[t].load(pos[i], IM == kInterpBilinear ? posa[i] : 0.0, M, Mt, mo, Ma, ord, slag);
    }
    c.acc[t] = {0, 0};
  }
  const uint64_t rm = live ? rowmask[row] : 0ull;
  if constexpr (SPLIT) {
    // every line walks its share of its own row's nodes (so that the order of a row's sum
    // does not depend on the rows beside it); all make the same number of transforms
    int most = 0;
    for (int i = 0; i < nrow; ++i)
      most = max(most, row0 + i < rows ? (int)__builtin_popcountll(rowmask[row0 + i]) : 0);
    uint64_t left = rm;
    for (int q = 0; q < sp; ++q) left &= left - 1;
    for (int i = 0; i < most; i += p.splits) {
      const bool on = left != 0;
      c.n = on ? __builtin_ctzll(left) : 0;
      c.src = fields + (size_t)rhs * frs + (size_t)c.n * fs + rbase;
      line_fft<R, +1, true, RM>(p, b, tl, mk, on, tab, c);
      for (int q = 0; q < p.splits; ++q) left &= left - 1;   // 0 stays 0
    }
    // the splits' sums, added by the first in a fixed order
    line_barrier();
    cpx<R>* own = lds + line * p.slots + tl;
    if (mine && sp > 0) {
#pragma unroll
      for (int t = 0; t < E; ++t)
        if (t < RL) own[t * KL] = c.acc[t];
    }
    line_barrier();
    if (!mine || sp > 0) return;
    for (int q = 1; q < p.splits; ++q) {
      const cpx<R>* o = own + (size_t)q * nrow * p.slots;
#pragma unroll
      for (int t = 0; t < E; ++t)
        if (t < RL) c.acc[t] = cadd(c.acc[t], o[t * KL]);
    }
  } else {
    uint64_t left = 0;
    for (int i = 0; i < nrow; ++i) left |= row0 + i < rows ? rowmask[row0 + i] : 0ull;
    while (left != 0) {
      c.n = __builtin_ctzll(left);
      left &= left - 1;
      c.src = fields + (size_t)rhs * frs + (size_t)c.n * fs + rbase;
      line_fft<R, +1, true, RM>(p, b, tl, mk, live && ((rm >> c.n) & 1ull) != 0, tab, c);
    }
    if (!mine) return;
  }
  cpx<TO>* dst = out + (size_t)rhs * out_rs + rbase;
#pragma unroll
  for (int t = 0; t < E; ++t) {
    if (t < RL) {
      if constexpr (ACC) {
        const cpx<TO> o = dst[t * KL];
        dst[t * KL] = {o.re + (TO)c.acc[t].re, o.im + (TO)c.acc[t].im};
      } else {
        dst[t * KL] = cvt<TO>(c.acc[t]);
      }
    }
  }
}

// ---------------------------------------------------------------- plans
namespace {

constexpr int kLineRadices[] = {16, 15, 12, 10, 9, 8, 6, 5, 4, 3, 2};

// The factors of n into `left` radices of at most `cap` with the largest smallest radix
// (fewest threads per line), then the smallest largest one; descending.
bool best_factors(int n, int left, int cap, int (&cur)[kLineStages], int at, int (&best)[kLineStages], int total) {
  if (left == 0) {
    if (n != 1) return false;
    if (best[0] == 0 || cur[total - 1] > best[total - 1] ||
        (cur[total - 1] == best[total - 1] && cur[0] < best[0]))
      for (int i = 0; i < total; ++i) best[i] = cur[i];
    return true;
  }
  bool any = false;
  for (int r : kLineRadices) {
    if (r > cap || n % r != 0) continue;
    cur[at] = r;
    any = best_factors(n / r, left - 1, r, cur, at + 1, best, total) || any;
  }
  return any;
}

// Stages, exchange pitches and LDS sizes for the radices in p->r (lines interleaved
// `ilv` fold in LDS).
void lay_out(LinePlan* p, int elem_bytes, int ilv) {
  int K = 1;
  const int q = std::max(1, 128 / elem_bytes / ilv);   // elements of a line per LDS access
  p->slots = 0;
  p->twn = 0;
  for (int s = 0; s < p->nst; ++s) {
    p->K[s] = K;
    p->J[s] = p->n / (K * p->r[s]);
    if (s > 0) p->twn += K * (p->r[s] - 1);
    K *= p->r[s];
  }
  for (int s = 0; s + 1 < p->nst; ++s) {
    const int Kn = p->K[s + 1], J = p->J[s];   // the exchange holds [k < Kn][j < J]
    if (s + 2 == p->nst) {
      p->pitch[s] = q > 1 ? (Kn | 1) : Kn;
      p->slots = std::max(p->slots, J * p->pitch[s]);
    } else {
      int pi = J;
      while (pi % q != p->J[s + 1] % q) ++pi;
      p->pitch[s] = pi;
      p->slots = std::max(p->slots, Kn * pi);
    }
  }
}

size_t line_lds(const LinePlan& p, int elem_bytes, bool table) {
  return ((size_t)p.slots * p.L * (p.two_buf ? 2 : 1) + (table ? p.twn : 0)) * elem_bytes;
}

constexpr size_t kLineLdsMax = (size_t)150 * 1024;

}  // namespace

static bool find_line_plan(int real_kind, int n, int kind, int across, int groups, int lines_req, LinePlan* out) {
  if (is_pow2_len(n) || n < 8) return false;
  const int eb = real_kind == 0 ? 16 : 8;
  const bool keeps = kind == kLineSym || kind == kLineComb, table = keeps;
  const bool cols = kind == kLineCols || kind == kLineSym;
  LinePlan p{};
  p.n = n;
  // The fewest stages, with radices up to 10 in passes B and C where that takes no more
  // (600^2 FP64, 10 10 6 either way: pass B 50 -> 38 us with the smaller kernel; 1440^2,
  // 12 12 10 or 8 6 6 5: 191 us with three stages, 270 with four).
  for (int k = 2; k <= kLineStages && p.nst == 0; ++k)
    for (int rm : {kLineRadixLo, kLineRadixMax}) {
      if (rm == kLineRadixLo && !keeps) continue;
      const int spec = rm == kLineRadixLo ? line_spectrum_max<double, kLineRadixLo>()
                       : real_kind == 0   ? line_spectrum_max<double, kLineRadixMax>()
                                          : line_spectrum_max<float, kLineRadixMax>();
      int cur[kLineStages] = {}, best[kLineStages] = {};
      if (!best_factors(n, k, rm, cur, 0, best, k)) continue;
      if (n / best[k - 1] > kLineMaxThr || (keeps && best[k - 1] > spec)) continue;
      p.nst = k;
      p.rm = rm;
      for (int i = 0; i < k; ++i) p.r[i] = best[i];
      break;
    }
  if (p.nst == 0) return false;
  p.T = n / p.r[p.nst - 1];
  p.splits = 1;
  auto fits = [&](int L) {
    if (L < 1 || L * p.T > kLineMaxThr || (cols && (L > 32 || (L & (L - 1)) != 0 || L > across))) return false;
    LinePlan t = p;
    t.L = L;
    lay_out(&t, eb, cols ? L : 1);
    if (line_lds(t, eb, table) > kLineLdsMax) return false;
    p = t;
    return true;
  };
  if (!fits(1)) return false;
  if (kind == kLineComb && across < 1024) {
    // few rows: up to four lines share a row's nodes
    int sp = groups >= 8 ? kLineSplits : groups >= 2 ? 2 : 1;
    while (sp > 1 && (sp * p.T > 384 || (real_kind == 0 && sp * p.T > 320) || !fits(sp))) sp /= 2;
    p.splits = sp;
  }
  if (lines_req > 0 && fits(lines_req * p.splits)) {
    // the caller's choice
  } else if (cols) {
    // adjacent columns up to 256 threads (more to reach two, which makes a store's row
    // segment 32 bytes in FP64: 1440^2, T = 144, 191 -> 166 us; but not where two columns
    // leave a CU one workgroup: 2400^2, T = 240, 268 -> 286 us) and half a CU's LDS, as
    // long as tiles and groups give every CU two workgroups
    const long total = (long)across * groups;
    for (int L = 2; L <= 32 && L * p.T <= (L > 2 ? 256 : real_kind == 0 ? 384 : 512) && total / L >= 512 && L * eb <= 256; L *= 2) {
      const LinePlan keep = p;
      if (!fits(L)) break;
      if (line_lds(p, eb, table) > 80 * 1024) {
        p = keep;
        break;
      }
    }
  } else {
    const int most = std::max(1, std::min(256 / std::max(1, p.T * p.splits), across / 512));
    for (int L = most; L > 1; --L) {
      const LinePlan keep = p;
      if (!fits(L * p.splits)) continue;
      if (line_lds(p, eb, table) <= 64 * 1024) break;
      p = keep;
    }
  }
  // a second exchange region where it costs no occupancy: one barrier per exchange
  const int waves = (p.T * p.L + 63) / 64;
  const int by_regs = std::max(1, 4 * (keeps ? line_waves(real_kind == 0, p.rm, kind) : real_kind == 0 ? 4 : 6) / waves);
  auto held = [&] { return std::min(by_regs, (int)((size_t)160 * 1024 / line_lds(p, eb, table))); };
  const int one = held();
  p.two_buf = 1;
  if (line_lds(p, eb, table) > kLineLdsMax || held() < one) p.two_buf = 0;
  *out = p;
  return true;
}

// The launches of one apply ask for the same few plans every time: each thread remembers
// the last ones it found (a search costs about as much host time as a launch).
bool make_line_plan(int real_kind, int n, int kind, int across, int groups, int lines_req, LinePlan* out) {
  struct Entry {
    int key[6];
    bool ok;
    LinePlan plan;
  };
  constexpr unsigned kEntries = 32;
  static thread_local Entry memo[kEntries] = {};
  const int key[6] = {real_kind + 1, n, kind, across, groups, lines_req};
  unsigned h = 0;
  for (int v : key) h = h * 31 + (unsigned)v;
  Entry& e = memo[(h ^ (h >> 7)) % kEntries];
  if (!std::equal(key, key + 6, e.key)) {
    e.ok = find_line_plan(real_kind, n, kind, across, groups, lines_req, &e.plan);
    std::copy(key, key + 6, e.key);
  }
  if (e.ok) *out = e.plan;
  return e.ok;
}

// The plan of the inverse transform of pass B: the radices reversed.
static LinePlan reversed(const LinePlan& fw, int elem_bytes) {
  LinePlan p = fw;
  for (int s = 0; s < fw.nst; ++s) p.r[s] = fw.r[fw.nst - 1 - s];
  lay_out(&p, elem_bytes, fw.L);
  return p;
}

int line_symbol_threads(int real_kind, int n, int* elems) {
  LinePlan p;
  if (!make_line_plan(real_kind, n, kLineSym, 1 << 20, 1, 0, &p)) return 0;
  *elems = p.r[0];
  return n / p.r[0];
}

int line_stage_table(int real_kind, int n, int kind, std::vector<int>* index) {
  LinePlan p;
  index->clear();
  if (!make_line_plan(real_kind, n, kind, 1 << 20, 1, 0, &p)) return 0;
  if (kind == kLineSym) p = reversed(p, real_kind == 0 ? 16 : 8);
  for (int s = 1; s < p.nst; ++s)
    for (int t = 1; t < p.r[s]; ++t)
      for (int k = 0; k < p.K[s]; ++k) index->push_back(k * t * p.J[s]);
  return (int)index->size();
}

// ---------------------------------------------------------------- launchers
static unsigned line_block(const LinePlan& p) { return (unsigned)((p.T * p.L + 63) / 64 * 64); }

template <typename R, typename TI>
static hipError_t rows_go(const LinePlan& p, const void* in, void* out, int rows, size_t in_rs, size_t out_rs, int nrhs,
                          const void* tw, const int* skip, hipStream_t st, const hipEvent_t* tev) {
  const size_t lds = line_lds(p, sizeof(cpx<R>), false);
  allow_dynamic_lds(k_line_rows<R, TI>, lds);
  HP_PASS_LAUNCH(tev, (k_line_rows<R, TI>), dim3((rows + p.L - 1) / p.L, nrhs), dim3(line_block(p)), lds, st,
                 (const cpx<TI>*)in, (cpx<R>*)out, rows, in_rs, out_rs, p, (const cpx<R>*)tw, skip);
  return hipGetLastError();
}

hipError_t launch_line_rows(int real_kind, int in_kind, const LinePlan& p, const void* in, void* out, int rows,
                            size_t in_rs, size_t out_rs, int nrhs, const void* tw, const int* skip, hipStream_t st,
                            const hipEvent_t* tev) {
  if (real_kind == 0) {
    if (in_kind != 0) return hipErrorInvalidValue;
    return rows_go<double, double>(p, in, out, rows, in_rs, out_rs, nrhs, tw, skip, st, tev);
  }
  if (in_kind == 0) return rows_go<float, double>(p, in, out, rows, in_rs, out_rs, nrhs, tw, skip, st, tev);
  return rows_go<float, float>(p, in, out, rows, in_rs, out_rs, nrhs, tw, skip, st, tev);
}

// Node groups of pass B: every group repeats the forward transform, so the ones that
// need the fewest rounds of (forward + nodes) transforms, counting how many workgroups
// the chip holds at once; a tie goes to fewer groups.
static int node_groups(const LinePlan& p, size_t lds, bool fp64, int tiles, int K, int nrhs) {
  const int waves = (p.T * p.L + 63) / 64;
  const long held = 256l * std::max(1, std::min(4 * line_waves(fp64, p.rm, kLineSym) / waves, (int)((size_t)160 * 1024 / lds)));
  int best = 1;
  long cost = 0;
  for (int ng = 1; ng <= K; ++ng) {
    const long wgs = (long)tiles * ng * nrhs, c = ((wgs + held - 1) / held) * (1 + (K + ng - 1) / ng);
    if (cost == 0 || c < cost) {
      cost = c;
      best = ng;
    }
    if (wgs > 2 * held) break;
  }
  return best;
}

template <typename R>
static hipError_t cols_go(const LinePlan& p, const ColsArgs& a, hipStream_t st) {
  const cpx<R>* in = (const cpx<R>*)a.in;
  cpx<R>* out = (cpx<R>*)a.out;
  const cpx<R>* tw = (const cpx<R>*)a.tw;
  const unsigned tiles = (unsigned)((a.S + p.L - 1) / p.L);
  if (a.mode == 1) {
    LinePlan fw = p, iv = reversed(p, sizeof(cpx<R>));
    fw.slots = iv.slots = std::max(fw.slots, iv.slots);
    const size_t lds = ((size_t)fw.slots * p.L * (p.two_buf ? 2 : 1) + iv.twn) * sizeof(cpx<R>);
    if (lds > kLineLdsMax + 8 * 1024) return hipErrorInvalidValue;
    const unsigned ng = (unsigned)node_groups(p, lds, sizeof(R) == 8, (int)tiles, a.K, a.nrhs);
    auto go = [&](auto kern) {
      allow_dynamic_lds(kern, lds);
      HP_PASS_LAUNCH(a.tev, kern, dim3(tiles, ng, a.nrhs), dim3(line_block(p)), lds, st, in, out, a.S, a.in_rs,
                     a.out_rs, a.out_fs, fw, iv, tw, (const cpx<R>*)a.stw, a.skip, a.lam_ax, a.lam_in, a.nodes, a.K, a.scale, a.store_mask);
      return hipGetLastError();
    };
    return p.rm == kLineRadixLo ? go(k_line_sym<R, kLineRadixLo>) : go(k_line_sym<R, kLineRadixMax>);
  }
  const size_t lds = line_lds(p, sizeof(cpx<R>), false);
  const dim3 grid(tiles, a.outer, a.nrhs * a.nfields);
  auto go = [&](auto kern) {
    allow_dynamic_lds(kern, lds);
    HP_PASS_LAUNCH(a.tev, kern, grid, dim3(line_block(p)), lds, st, in, out, a.S, a.nfields, a.in_rs, a.out_rs,
                   a.in_fs, a.out_fs, p, tw, a.skip, a.slab_need);
    return hipGetLastError();
  };
  return a.dir < 0 ? go(k_line_cols<R, -1>) : go(k_line_cols<R, +1>);
}

hipError_t launch_line_cols(const LinePlan& p, const ColsArgs& a, hipStream_t st) {
  return a.real_kind == 0 ? cols_go<double>(p, a, st) : cols_go<float>(p, a, st);
}

template <typename R, typename TO, bool ACC, int IM>
static hipError_t combine_go(const LinePlan& plan, const CombineArgs& a, hipStream_t st) {
  LinePlan p = plan;
  if constexpr (IM == kInterpLagrange) {
    // the weights' table beside the lines may cost a workgroup that the plan's second
    // exchange region did not (1620 points FP64: one on a CU instead of two)
    auto held = [&] { return (size_t)160 * 1024 / (line_lds(p, sizeof(cpx<R>), true) + kLagTable * sizeof(double)); };
    const size_t two = held();
    p.two_buf = 0;
    const size_t waves = (p.T * p.L + 63) / 64, regs = 4 * line_waves(sizeof(R) == 8, p.rm, kLineComb, IM) / waves;
    if (std::min(held(), std::max<size_t>(1, regs)) <= two) p.two_buf = plan.two_buf;
  }
  const size_t lds = line_lds(p, sizeof(cpx<R>), true);
  const int nrow = p.L / p.splits;
  auto go = [&](auto kern) {
    allow_dynamic_lds(kern, lds);
    HP_PASS_LAUNCH(a.tev, kern, dim3((a.rows + nrow - 1) / nrow, a.nrhs), dim3(line_block(p)), lds, st,
                   (const cpx<R>*)a.fields, a.fs, a.frs, a.pos, a.rowmask, (cpx<TO>*)a.out, a.out_rs, a.rows, a.M,
                   a.Mt, a.mo, p, (const cpx<R>*)a.stw, a.skip, a.order, a.lag, a.posa, a.Ma);
    return hipGetLastError();
  };
  if (p.rm == kLineRadixLo)
    return p.splits > 1 ? go(k_line_combine<R, TO, ACC, IM, kLineRadixLo, true>)
                        : go(k_line_combine<R, TO, ACC, IM, kLineRadixLo, false>);
  return p.splits > 1 ? go(k_line_combine<R, TO, ACC, IM, kLineRadixMax, true>)
                      : go(k_line_combine<R, TO, ACC, IM, kLineRadixMax, false>);
}
template <typename R, typename TO, bool ACC>
static hipError_t combine_any(const LinePlan& p, const CombineArgs& a, hipStream_t st) {
  switch (interp_mode(a)) {
    case kInterpLagrange: return combine_go<R, TO, ACC, kInterpLagrange>(p, a, st);
    case kInterpBilinear: return combine_go<R, TO, ACC, kInterpBilinear>(p, a, st);
    default: return combine_go<R, TO, ACC, kInterpLinear>(p, a, st);
  }
}

hipError_t launch_line_combine(const LinePlan& p, const CombineArgs& a, hipStream_t st) {
  if (a.real_kind == 0) {
    if (a.out_kind != 0) return hipErrorInvalidValue;
    return a.accumulate ? combine_any<double, double, true>(p, a, st) : combine_any<double, double, false>(p, a, st);
  }
  if (a.out_kind == 0)
    return a.accumulate ? combine_any<float, double, true>(p, a, st) : combine_any<float, double, false>(p, a, st);
  if (a.accumulate) return hipErrorInvalidValue;
  return combine_any<float, float, false>(p, a, st);
}

}  // namespace hp
