// Device code shared by the kernel files: conversions, the symbol reciprocal, the
// interpolation records and weights of the combine, and the small-radix DFTs of the
// mixed-radix lines.
#pragma once
#include <hip/hip_ext.h>

#include "hp_internal.h"

// Launch of a pass kernel; with timing events (tev non-null) through
// hipExtLaunchKernelGGL, which stores the kernel's own start and end times in
// tev[0] and tev[1] (no marker packets around it).
#define HP_PASS_LAUNCH(tev, kernel, grid, block, shm, st, ...)                                         \
  do {                                                                                                 \
    if ((tev) != nullptr)                                                                              \
      hipExtLaunchKernelGGL(kernel, grid, block, (std::uint32_t)(shm), st, (tev)[0], (tev)[1], 0, __VA_ARGS__); \
    else                                                                                               \
      hipLaunchKernelGGL(kernel, grid, block, shm, st, __VA_ARGS__);                                    \
  } while (0)

namespace hp {

template <typename R, typename S>
__device__ __forceinline__ cpx<R> cvt(cpx<S> a) {
  return {(R)a.re, (R)a.im};
}

// Workgroups are dispatched round-robin over the 8 XCDs, each with its own L2.  Over the
// gx x gy workgroups of a grid slice, the ones of one XCD take consecutive (tile, group)
// pairs, tiles fastest, so that tiles sharing cache lines meet in one L2.
__device__ __forceinline__ void xcd_tile(int bx, int by, int gx, int gy, int* tile, int* group) {
  const int id = bx + gx * by, total = gx * gy, x = id & 7, rest = total & 7;
  const int at = x * (total >> 3) + (x < rest ? x : rest) + (id >> 3);
  *group = at / gx;
  *tile = at - *group * gx;
}

// 1/x for finite x > 0: hardware reciprocal estimate r with residual e = 1 - x r, refined
// in FP64 (e about 2^-24) by the cubic step r <- r + r (e + e^2), whose own error e^3 is
// below rounding, in FP32 by one Newton-Raphson step.
__device__ __forceinline__ double recip(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  const double e = __builtin_fma(-x, r, 1.0);
  return __builtin_fma(r, __builtin_fma(e, e, e), r);
}
__device__ __forceinline__ float recip(float x) {
  float r = __builtin_amdgcn_rcpf(x);
  const float e = __builtin_fmaf(-x, r, 1.0f);
  return __builtin_fmaf(r, e, r);
}

// Interpolation record of one point: pos >= 0 encodes the real-axis segment
// seg + t (weights 1-t on node seg, t on node seg+1); pos < 0 encodes the layer
// segment, -(1 + j + t): weights 1-t on the lower layer node (c_o itself for
// j = 0) and t on layer node j+1 (Eqn. 405 with Re gamma = c_o in the layer).
__device__ __forceinline__ void decode_pos(double p, int M, int Mt, int mo, int& A, int& B, double& t) {
  if (p >= 0.0) {
    if (M == 1) {
      A = 0; B = 0; t = 0.0;
      return;
    }
    int s = (int)p;
    if (s > M - 2) s = M - 2;
    A = s; B = s + 1; t = p - (double)s;
  } else {
    const double q = -p - 1.0;
    int s = (int)q;
    if (s > Mt - 1) s = Mt - 1;
    A = (s == 0) ? mo : M + s - 1; B = M + s; t = q - (double)s;
  }
}

// Interpolation modes of the combine: piecewise linear along Re gamma (the
// paper's), piecewise Lagrange of degree >= 2 along the real axis, and bilinear in
// (c, a) (one damping node axis; no layer).
enum InterpMode { kInterpLinear = 0, kInterpLagrange = 1, kInterpBilinear = 2 };

// Per-point record for the combine: `ab` packs nodes A, B (piecewise linear:
// weights 1-t, t) or, for a real-axis point under Lagrange interpolation of degree
// ord >= 2, the first node A of its ord+1-node stencil and a flag; `tt` holds t,
// or the point's speed x for the Lagrange weights.  Bilinear: `ab` packs the four
// nodes (s, r), (s+1, r), (s, r+1), (s+1, r+1) of node index m + M r, `tt` and `uu`
// the fractions along c and along a.  lag: the table of CombineArgs.
template <typename R, int IM>
__device__ __forceinline__ void interp_record(double pv, double pa, int M, int Mt, int mo, int Ma, int ord,
                                              const double* lag, int& ab, R& tt, R& uu) {
  int A = -1, B = -1;
  double t = 0.0;
  decode_pos(pv, M, Mt, mo, A, B, t);
  if (IM == kInterpBilinear) {
    int r = (int)pa;
    if (r > Ma - 2) r = Ma - 2;
    if (r < 0) r = 0;
    const double u = pa - (double)r;
    A += M * r;
    B += M * r;
    ab = A | (B << 8) | ((A + M) << 16) | ((B + M) << 24);
    tt = (R)t;
    uu = (R)u;
  } else if (IM == kInterpLagrange && pv >= 0.0 && M > 1) {
    int a = A - (ord - 1) / 2;
    a = a < 0 ? 0 : (a > M - 1 - ord ? M - 1 - ord : a);
    ab = a | (1 << 16);
    tt = (R)(lag[A] + t * (lag[A + 1] - lag[A]));
  } else {
    ab = (A & 0xff) | ((B & 0xff) << 8);
    tt = (R)t;
  }
}

// Weight of node n at a point with record (ab, tt, uu).
template <typename R, int IM>
__device__ __forceinline__ R interp_weight(int ab, R tt, R uu, int n, int ord, const double* lag) {
  const int A = ab & 0xff;
  if (IM == kInterpBilinear) {
    const int B = (ab >> 8) & 0xff, Cn = (ab >> 16) & 0xff, D = (ab >> 24) & 0xff;
    const R lo = (R)1 - uu;
    return (A == n ? ((R)1 - tt) * lo : (R)0) + (B == n ? tt * lo : (R)0) + (Cn == n ? ((R)1 - tt) * uu : (R)0) +
           (D == n ? tt * uu : (R)0);
  }
  if (IM == kInterpLagrange && (ab >> 16)) {
    if (n < A || n > A + ord) return (R)0;
    R w = (R)lag[kMaxNodes + 4 * n + (n - A)];
    for (int k = A; k <= A + ord; ++k)
      if (k != n) w *= tt - (R)lag[k];
    return w;
  }
  const int B = (ab >> 8) & 0xff;
  return (A == n ? (R)1 - tt : (R)0) + (B == n ? tt : (R)0);
}

// Spectrum elements v (the 1/N^d of the inverse transform already in them) times the
// symbol of a node, x_s = v_s / (A_n - g_n lambda_s).  The denominator is formed in FP64
// (it cancels near |xi| = omega/|gamma_n|), then reciprocated in the working precision.
// A node of real speed has a constant imaginary part (most nodes: 16 of 19 at 16 + 3);
// SPLIT: such nodes take a loop of their own.
template <bool SPLIT = true, typename R, int E, int CNT>
__device__ __forceinline__ void symbol_mul(const cpx<R> (&v)[E], cpx<R> (&x)[CNT], const double (&lam)[E],
                                           const NodeConst& nc) {
  static_assert(CNT <= E, "outputs within the elements held");
  if (SPLIT && nc.gim == 0.0) {
    const R fi = (R)nc.aim, fi2 = fi * fi;
#pragma unroll
    for (int s = 0; s < CNT; ++s) {
      const R fr = (R)(nc.are - nc.gre * lam[s]);
      const R inv = recip(fr * fr + fi2);
      x[s] = cmul(v[s], cpx<R>{fr * inv, -fi * inv});
    }
  } else {
#pragma unroll
    for (int s = 0; s < CNT; ++s) {
      const R fr = (R)(nc.are - nc.gre * lam[s]), fi = (R)(nc.aim - nc.gim * lam[s]);
      const R inv = recip(fr * fr + fi * fi);
      x[s] = cmul(v[s], cpx<R>{fr * inv, -fi * inv});
    }
  }
}

// What the combine keeps of a point, and the point's weight on
// node n.  Piecewise linear: the record p itself; the weight is the hat of width 1 around
// the node's centre on the record's axis, n for a real node, -(i + 2) for layer node i,
// and -1 beside its own for the background node mo, where the layer's leg starts (record
// -(1 + j + t), see decode_pos).  The weights are those of decode_pos to rounding, without
// a search or a compare per node: the differences and 1 - |d| are exact in FP64 but in the
// first segment, where p - 1 rounds by at most 2^-54; FP32 weights are rounded from FP64
// one by one, not as a rounded t and 1 - t.
// (FP32 rows above 1024 points keep the select: their combine has no registers left for
// the FP64 temporaries, 2048^2 mixed 190 us with selects before, 208 with hats, 173 with
// selects and the reordered loads)
template <typename R>
constexpr bool hat_weights(int n) { return sizeof(R) == 8 || n <= 1024; }
template <typename R, int IM, bool HAT = true>
struct CombPoint {
  int ab;
  R tt, uu;
  __device__ __forceinline__ void clear() { ab = 0xffff; tt = (R)0; uu = (R)0; }
  __device__ __forceinline__ void load(double pv, double pa, int M, int Mt, int mo, int Ma, int ord, const double* lag) {
    interp_record<R, IM>(pv, pa, M, Mt, mo, Ma, ord, lag, ab, tt, uu);
  }
  __device__ __forceinline__ R weight(int n, int M, int mo, int ord, const double* lag) const {
    return interp_weight<R, IM>(ab, tt, uu, n, ord, lag);
  }
};
__device__ __forceinline__ double hat(double d) { return __builtin_fmin(__builtin_fmax(1.0 - __builtin_fabs(d), 0.0), 1.0); }
template <typename R>
struct CombPoint<R, kInterpLinear, true> {
  double p;
  __device__ __forceinline__ void clear() { p = 1e9; }   // no node is near
  __device__ __forceinline__ void load(double pv, double, int, int, int, int, int, const double*) { p = pv; }
  __device__ __forceinline__ R weight(int n, int M, int mo, int, const double*) const {
    double w = hat(p - (n < M ? (double)n : (double)(M - 2 - n)));
    if (n == mo) w += hat(p + 1.0);
    return (R)w;
  }
};

// cos and sin of 2 pi m / r, evaluated at compile time for the butterflies' fixed
// roots: the angle is reduced to [0, pi/4] by the octant symmetries (exactly, in
// integers), then summed as a Taylor series.
constexpr double kPiD = 3.14159265358979323846;
constexpr double taylor_sin(double x) {
  double t = x, s = x;
  for (int k = 1; k < 14; ++k) { t *= -x * x / ((2.0 * k) * (2.0 * k + 1.0)); s += t; }
  return s;
}
constexpr double taylor_cos(double x) {
  double t = 1.0, s = 1.0;
  for (int k = 1; k < 14; ++k) { t *= -x * x / ((2.0 * k - 1.0) * (2.0 * k)); s += t; }
  return s;
}
// angle 2 pi m / r with 0 <= m <= r/8 (at most pi/4)
constexpr void small_cs(long m, long r, double& c, double& s) {
  const double x = 2.0 * kPiD * (double)m / (double)r;
  c = taylor_cos(x);
  s = taylor_sin(x);
}
constexpr void root_cs(long m, long r, double& c, double& s) {
  m %= r;
  double sg = 1.0;
  if (2 * m > r) { m = r - m; sg = -1.0; }           // sin(2 pi - x) = -sin x
  double cg = 1.0;                                   // now x in [0, pi]
  if (4 * m > r) { m = r - 2 * m; cg = -1.0; r *= 2; }  // x -> pi - x: cos flips; m/r -> (r/2 - m)/r
  // now x = 2 pi m / r in [0, pi/2]
  double cc = 0.0, ss = 0.0;
  if (8 * m > r) {                                   // x -> pi/2 - x swaps cos and sin
    small_cs(r - 4 * m, 4 * r, ss, cc);
  } else {
    small_cs(m, r, cc, ss);
  }
  c = cg * cc;
  s = sg * ss;
}
template <int RAD>
struct RootTab {
  double c[RAD], s[RAD];
};
template <int RAD>
constexpr RootTab<RAD> make_roots() {
  RootTab<RAD> t{};
  for (int m = 0; m < RAD; ++m) root_cs(m, RAD, t.c[m], t.s[m]);
  return t;
}
template <int RAD>
constexpr RootTab<RAD> kRoots = make_roots<RAD>();

// x exp(DIR 2 pi i m / RAD) for a fixed m (the quarter turns without multiplies)
template <typename R, int RAD, int DIR>
__device__ __forceinline__ cpx<R> mul_root(cpx<R> x, int m) {
  m %= RAD;
  if (m == 0) return x;
  if (2 * m == RAD) return {-x.re, -x.im};
  if (4 * m == RAD) return DIR > 0 ? cpx<R>{-x.im, x.re} : cpx<R>{x.im, -x.re};
  if (4 * m == 3 * RAD) return DIR > 0 ? cpx<R>{x.im, -x.re} : cpx<R>{-x.im, x.re};
  const R c = (R)kRoots<RAD>.c[m], sn = (R)(DIR * kRoots<RAD>.s[m]);
  return {x.re * c - x.im * sn, x.re * sn + x.im * c};
}

// DFTs of length 2, 3, 4 and 5 in place: out[k] = sum_t v[t] exp(DIR 2 pi i t k / RAD),
// with the symmetric pairs of terms combined.
template <typename R, int DIR>
__device__ __forceinline__ void dft2(cpx<R>& a, cpx<R>& b) {
  const cpx<R> s = cadd(a, b), d = csub(a, b);
  a = s;
  b = d;
}
template <typename R, int DIR>
__device__ __forceinline__ cpx<R> times_dir_i(cpx<R> x) {   // DIR i x
  return DIR > 0 ? cpx<R>{-x.im, x.re} : cpx<R>{x.im, -x.re};
}
template <typename R, int RAD, int DIR>
__device__ __forceinline__ void dft_prime(cpx<R> (&v)[RAD]) {
  if constexpr (RAD == 2) {
    dft2<R, DIR>(v[0], v[1]);
  } else if constexpr (RAD == 3) {
    constexpr double s3 = 0.86602540378443864676;   // sin(2 pi / 3)
    const cpx<R> a = cadd(v[1], v[2]);
    const cpx<R> d = csub(v[1], v[2]);
    const cpx<R> m = {v[0].re - (R)0.5 * a.re, v[0].im - (R)0.5 * a.im};
    const cpx<R> j = times_dir_i<R, DIR>(cpx<R>{(R)s3 * d.re, (R)s3 * d.im});
    v[0] = cadd(v[0], a);
    v[1] = cadd(m, j);
    v[2] = csub(m, j);
  } else if constexpr (RAD == 4) {
    const cpx<R> s02 = cadd(v[0], v[2]), d02 = csub(v[0], v[2]);
    const cpx<R> s13 = cadd(v[1], v[3]), d13 = times_dir_i<R, DIR>(csub(v[1], v[3]));
    v[0] = cadd(s02, s13);
    v[2] = csub(s02, s13);
    v[1] = cadd(d02, d13);
    v[3] = csub(d02, d13);
  } else {
    static_assert(RAD == 5, "radix 2, 3, 4 or 5");
    constexpr double c1 = 0.30901699437494742410, s1 = 0.95105651629515357212;   // 2 pi / 5
    constexpr double c2 = -0.80901699437494742410, s2 = 0.58778525229247312917;  // 4 pi / 5
    const cpx<R> a1 = cadd(v[1], v[4]), b1 = csub(v[1], v[4]);
    const cpx<R> a2 = cadd(v[2], v[3]), b2 = csub(v[2], v[3]);
    const cpx<R> m1 = {v[0].re + (R)c1 * a1.re + (R)c2 * a2.re, v[0].im + (R)c1 * a1.im + (R)c2 * a2.im};
    const cpx<R> m2 = {v[0].re + (R)c2 * a1.re + (R)c1 * a2.re, v[0].im + (R)c2 * a1.im + (R)c1 * a2.im};
    const cpx<R> j1 = times_dir_i<R, DIR>(cpx<R>{(R)s1 * b1.re + (R)s2 * b2.re, (R)s1 * b1.im + (R)s2 * b2.im});
    const cpx<R> j2 = times_dir_i<R, DIR>(cpx<R>{(R)s2 * b1.re - (R)s1 * b2.re, (R)s2 * b1.im - (R)s1 * b2.im});
    v[0] = cadd(v[0], cadd(a1, a2));
    v[1] = cadd(m1, j1);
    v[4] = csub(m1, j1);
    v[2] = cadd(m2, j2);
    v[3] = csub(m2, j2);
  }
}

// first factor of a stage radix: the DFT of length RAD = F·(RAD/F) runs as RAD/F
// DFTs of length F, fixed roots, then F DFTs of length RAD/F
constexpr int radix_first(int r) { return r % 5 == 0 ? 5 : r % 4 == 0 ? 4 : r % 3 == 0 ? 3 : 2; }

template <typename R, int RAD, int DIR>
__device__ __forceinline__ void dft_radix(cpx<R> (&v)[RAD]) {
  constexpr int F = radix_first(RAD), G = RAD / F;
  if constexpr (G == 1) {
    dft_prime<R, RAD, DIR>(v);
  } else {
    // input index t = tf G + tg, output index kf + F kg
    cpx<R> a[G][F];
#pragma unroll
    for (int tg = 0; tg < G; ++tg) {
      cpx<R> u[F];
#pragma unroll
      for (int tf = 0; tf < F; ++tf) u[tf] = v[tf * G + tg];
      dft_prime<R, F, DIR>(u);
#pragma unroll
      for (int kf = 0; kf < F; ++kf) a[tg][kf] = mul_root<R, RAD, DIR>(u[kf], tg * kf);
    }
#pragma unroll
    for (int kf = 0; kf < F; ++kf) {
      cpx<R> u[G];
#pragma unroll
      for (int tg = 0; tg < G; ++tg) u[tg] = a[tg][kf];
      dft_radix<R, G, DIR>(u);
#pragma unroll
      for (int kg = 0; kg < G; ++kg) v[kf + F * kg] = u[kg];
    }
  }
}

template <typename K>
inline void allow_dynamic_lds(K kernel, size_t bytes) {
  // lines longer than 64 KiB of LDS need the limit raised once per kernel
  if (bytes > 65536) (void)hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

inline int interp_mode(const CombineArgs& a) {
  return a.order >= 2 ? kInterpLagrange : (a.Ma >= 2 ? kInterpBilinear : kInterpLinear);
}

}  // namespace hp
