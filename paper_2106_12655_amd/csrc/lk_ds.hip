// lk_ds.hip -- the direct-summation hot loop for CDNA4 (gfx950).
//
// Computes, for every work item (pair p, a block of 64 segments of loop B, a
// chunk of segments of loop A), the partial sum of the Eq. 4 segment-pair term
// and adds it into the pair's 128-bit fixed-point accumulator.
//
// Layout of the work (one 64-lane wavefront = one workgroup = one item; calls with
// few pairs give an item to a workgroup of several waves, ds_team below):
//   * each lane owns one segment (k_i, k_{i+1}) of loop B in registers;
//   * the item's vertices of loop A are staged through LDS in tiles and every
//     lane walks them in order (a broadcast read: all lanes read the same
//     vertex at the same step);
//   * when loop B has fewer than 64 segments left, the lanes split loop A's
//     range into groups instead (both loops parallel, as the paper does for
//     small pairs).
// The kernel is persistent: a fixed grid of waves pulls items from device
// counters until the device-side item total is reached, so the launch shape
// does not depend on the data and the whole pass can live in a HIP graph.
//
// Per term (Eq. 4, Sec. 2.1): a = l_j - k_i, b = l_j - k_{i+1},
// c = l_{j+1} - k_{i+1}, d = l_{j+1} - k_i.  Walking j in order, a and b of
// segment j+1 are d and c of segment j, so each step needs only the new
// vertex-pair vectors v_r = l_{j+1} - k_r of the lane's vertices, their norms
// and their dot products with the previous ones; the other dot products of
// Eq. 4 follow from carried ones and the lane's segment vectors s_r:
//   c . a = (d - s_r) . a = a . d - s_r . a      (s_r . a carried from the
//                                                  previous step's s_r . d)
//   d . c = d . (d - s_r) = |d|^2 - s_r . d
// The common numerator of both arctangents is p = a . (s_j x s_r) (equal to
// a . (b x c) and c . (d x a) in exact arithmetic, Sec. 3.4.2).  With the
// lane's first vertex k_0 as a local origin, a = V_0 - delta_r where
// V_0 = l_j - k_0 and delta_r = k_r - k_0, so
//   p = s_r . (V_0 x s_j) - s_j . (s_r x delta_r)
// with one cross product per step shared by the lane's R segments and a
// per-lane constant s_r x delta_r; both pieces are built from short vectors,
// which keeps FP32 accurate for distant pairs.  The two arctangents are merged
// into one: (d1 + i p)(d2 + i p) has the angle atan2(p, d1) + atan2(p, d2)
// (the angle-addition idea of the appendix, Alg. 7, applied per term).  Every
// difference vector l(s) - k(t) of the two segments has the same component p
// along s_j x s_r, so the pair's quadrilateral lies in one open hemisphere:
// the angle stays inside (-pi, pi) and has the sign of p, which makes
// d1 + d2 > 0 in exact arithmetic.  Near contact with the crossing close to
// the diagonal a-c both d1 and d2 shrink and their FP32 sum carries no sign,
// so the sign is taken from p (which stays accurate there) and only the
// magnitude from the merged form:
//   theta = atan2(p |d1 + d2|, d1 d2 - p^2),  term = theta / (2 pi)
// The magnitude's error near contact grows like eps |s| / h (h the distance
// of the segments); it stays below 0.5 per term and is caught by the refit
// rule long before h reaches the resolution of the coordinates.
#include "lk_internal.h"
#include "atan_poly.h"

namespace lk {
namespace {

template <typename T>
struct V3 {
  T x, y, z;
};
template <typename T>
__device__ __forceinline__ V3<T> operator-(const V3<T>& a, const V3<T>& b) {
  return {a.x - b.x, a.y - b.y, a.z - b.z};
}
template <typename T>
__device__ __forceinline__ T dot(const V3<T>& a, const V3<T>& b) {
  return a.x * b.x + a.y * b.y + a.z * b.z;
}
template <typename T>
__device__ __forceinline__ V3<T> cross(const V3<T>& a, const V3<T>& b) {
  return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}

__device__ __forceinline__ float fabs_t(float a) { return __builtin_fabsf(a); }
__device__ __forceinline__ double fabs_t(double a) { return __builtin_fabs(a); }
__device__ __forceinline__ float fmad(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fmad(double a, double b, double c) { return __builtin_fma(a, b, c); }

// The walk's products, with each rounding spelled out: where a sum of products is
// fused is otherwise the compiler's choice, which changes the last bits with
// the code around it.
template <typename T>
__device__ __forceinline__ T dot_r(const V3<T>& a, const V3<T>& b) {
  return fmad(a.z, b.z, fmad(a.x, b.x, a.y * b.y));
}
template <typename T>
__device__ __forceinline__ V3<T> cross_r(const V3<T>& a, const V3<T>& b) {
  return {fmad(a.y, b.z, -(a.z * b.y)), fmad(a.z, b.x, -(a.x * b.z)),
          fmad(a.x, b.y, -(a.y * b.x))};
}

// The FP32 square roots and reciprocals of a step, as blocks between two changes
// of the wave's priority.  A SIMD issues two VALU instructions of two of its
// waves at once (FP32 adds, products and fused products, unless all three
// source registers have one parity), 2.2 cycles each instead of 4.3, but only
// while the two stay in step, and a transcendental (8 cycles) leaves them out
// of step.  Raised priority brings them back: this walk's instructions, 9
// of 159 a step transcendental, took 4.4 cycles each without it, 3.4 with a
// no-op around each transcendental, 2.7 with the priority around each and 2.65
// around blocks of 5 and 4 (four waves a SIMD; 2.5 is the sum of the issue
// times).  The closing s_setprio is also the wait state that a use of the last
// result needs.
template <int N>
__device__ __forceinline__ void sqrt_n(const float (&x)[N], float (&y)[N]) {
  static_assert(N == 1 || N == 2 || N == 3 || N == 5, "vertices of a lane");
  if constexpr (N == 1)
    asm("s_setprio 1\n\tv_sqrt_f32 %0, %1\n\ts_setprio 0" : "=&v"(y[0]) : "v"(x[0]));
  if constexpr (N == 2)
    asm("s_setprio 1\n\tv_sqrt_f32 %0, %2\n\tv_sqrt_f32 %1, %3\n\ts_setprio 0"
        : "=&v"(y[0]), "=&v"(y[1])
        : "v"(x[0]), "v"(x[1]));
  if constexpr (N == 3)
    asm("s_setprio 1\n\tv_sqrt_f32 %0, %3\n\tv_sqrt_f32 %1, %4\n\tv_sqrt_f32 %2, %5\n\ts_setprio 0"
        : "=&v"(y[0]), "=&v"(y[1]), "=&v"(y[2])
        : "v"(x[0]), "v"(x[1]), "v"(x[2]));
  if constexpr (N == 5)
    asm("s_setprio 1\n\tv_sqrt_f32 %0, %5\n\tv_sqrt_f32 %1, %6\n\tv_sqrt_f32 %2, %7\n\t"
        "v_sqrt_f32 %3, %8\n\tv_sqrt_f32 %4, %9\n\ts_setprio 0"
        : "=&v"(y[0]), "=&v"(y[1]), "=&v"(y[2]), "=&v"(y[3]), "=&v"(y[4])
        : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]));
}
template <int N>
__device__ __forceinline__ void rcp_n(const float (&x)[N], float (&y)[N]) {
  static_assert(N == 1 || N == 2 || N == 4, "segments of a lane");
  if constexpr (N == 1)
    asm("s_setprio 1\n\tv_rcp_f32 %0, %1\n\ts_setprio 0" : "=&v"(y[0]) : "v"(x[0]));
  if constexpr (N == 2)
    asm("s_setprio 1\n\tv_rcp_f32 %0, %2\n\tv_rcp_f32 %1, %3\n\ts_setprio 0"
        : "=&v"(y[0]), "=&v"(y[1])
        : "v"(x[0]), "v"(x[1]));
  if constexpr (N == 4)
    asm("s_setprio 1\n\tv_rcp_f32 %0, %4\n\tv_rcp_f32 %1, %5\n\tv_rcp_f32 %2, %6\n\t"
        "v_rcp_f32 %3, %7\n\ts_setprio 0"
        : "=&v"(y[0]), "=&v"(y[1]), "=&v"(y[2]), "=&v"(y[3])
        : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]));
}

// FP64 square root from the hardware reciprocal-square-root estimate and two
// Goldschmidt iterations (s -> sqrt(x), h -> 1 / (2 sqrt(x))), then one
// Newton correction on the residual x - s^2.  No range scaling: arguments
// are squared distances of geometry, far from the FP64 limits; x = 0 gives
// NaN, which only happens for coincident vertices (a degenerate pair, flagged).
__device__ __forceinline__ double fsqrt(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  double s = x * y, h = 0.5 * y;
  double r = fma(-s, h, 0.5);
  s = fma(s, r, s);
  h = fma(h, r, h);
  r = fma(-s, h, 0.5);
  s = fma(s, r, s);
  h = fma(h, r, h);
  return fma(fma(-s, s, x), h, s);
}

template <int N>
__device__ __forceinline__ void sqrt_n(const double (&x)[N], double (&y)[N]) {
#pragma unroll
  for (int r = 0; r < N; ++r) y[r] = fsqrt(x[r]);
}

// Own FP32 arctangent: octant reduction to t = min/max in [0, 1], then
// atan(t) = t q(t^2) with q the Remez minimax polynomial of atan_poly.h.
// (0, 0) gives NaN on purpose: it only arises for touching segments.  inv: the
// hardware reciprocal of max(|x|, |y|).
__device__ __forceinline__ float atan2_minimax(float y, float x, float inv) {
  const float ax = fabsf(x), ay = fabsf(y);
  const float t = fminf(ax, ay) * inv;
  const float s = t * t;
  float q = kAtanQ[LK_ATAN_DEG];
#pragma unroll
  for (int k = LK_ATAN_DEG - 1; k >= 0; --k) q = fmaf(q, s, kAtanQ[k]);
  float r = t * q;
  r = (ay > ax) ? (1.57079632679489662f - r) : r;
  r = (x < 0.0f) ? (3.14159265358979324f - r) : r;
  return copysignf(r, y);
}

// Own FP64 arctangent: the same octant reduction, t = min/max from the
// hardware reciprocal estimate with two Newton steps and a residual
// correction (no IEEE division sequence), and the degree-19 polynomial of
// atan_poly.h (relative error 2.5e-16 in FP64 Horner form).
__device__ __forceinline__ double atan2_f64(double y, double x) {
  const double ax = fabs(x), ay = fabs(y);
  const double mx = fmax(ax, ay), mn = fmin(ax, ay);
  double r = __builtin_amdgcn_rcp(mx);
  r = fma(r, fma(-mx, r, 1.0), r);
  r = fma(r, fma(-mx, r, 1.0), r);
  const double q = mn * r;
  const double t = fma(fma(-mx, q, mn), r, q);
  const double s = t * t;
  double p = kAtanQ64[LK_ATAN_DEG64];
#pragma unroll
  for (int k = LK_ATAN_DEG64 - 1; k >= 0; --k) p = fma(p, s, kAtanQ64[k]);
  double a = t * p;
  a = (ay > ax) ? (1.57079632679489661923 - a) : a;
  a = (x < 0.0) ? (3.14159265358979323846 - a) : a;
  return copysign(a, y);
}

// AT, the arctangent: FP32 1 = HIP's, 2 = own with short forms for small angles,
// kFullForm = own without them; FP64 0 = own with short forms.
constexpr int kFullForm = 4;
template <typename T, int AT>
__device__ __forceinline__ T angle(T y, T x);
template <>
__device__ __forceinline__ float angle<float, 1>(float y, float x) {
  return atan2f(y, x);
}
template <>
__device__ __forceinline__ double angle<double, 0>(double y, double x) {
  return atan2_f64(y, x);
}
template <>
__device__ __forceinline__ float angle<float, 2>(float y, float x) {
  return atan2_minimax(y, x, __builtin_amdgcn_rcpf(fmaxf(fabsf(x), fabsf(y))));
}
template <>
__device__ __forceinline__ float angle<float, kFullForm>(float y, float x) {
  return angle<float, 2>(y, x);
}

// LDS vertex record: 16 bytes for float (one ds_read_b128), 32 for double.
template <typename T>
struct alignas(4 * sizeof(T)) Vtx {
  T x, y, z, w;
};

template <typename Tc, typename Tin>
__device__ __forceinline__ V3<Tc> load_vertex(const Tin* X, int64_t v) {
  return {(Tc)X[3 * v], (Tc)X[3 * v + 1], (Tc)X[3 * v + 2]};
}

// A value that is the same in every lane, moved to scalar registers (the
// compiler cannot tell for values that come from memory or a shuffle).
__device__ __forceinline__ int32_t uniform(int32_t x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ int64_t uniform(int64_t x) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)x);
  const int32_t hi = __builtin_amdgcn_readfirstlane((int32_t)(x >> 32));
  return ((int64_t)hi << 32) | lo;
}
__device__ __forceinline__ double uniform(double x) {
  return __longlong_as_double(uniform((int64_t)__double_as_longlong(x)));
}
__device__ __forceinline__ WorkRec uniform(const WorkRec& r) {
  return {uniform(r.oa), uniform(r.ob), uniform(r.na), uniform(r.nb), uniform(r.p), uniform(r.items)};
}

// Vertex loads of one work item.  An FP32 pass over FP64 input takes every
// coordinate relative to an origin inside the item (a vertex of its loop-B
// block), subtracted in FP64 before the rounding to FP32: the FP32 values
// then carry relative precision against the item's own extent, not against
// the distance from the coordinate origin (2^-24 of 1e3 is 6e-5, enough to
// move a near contact across its partner).  The terms only use differences
// of vertices, which the shift leaves unchanged in exact arithmetic.  FP32
// input, and FP64 passes, load the values as stored.
template <typename Tin, typename Tc>
struct Frame {
  static constexpr bool kShift = sizeof(Tin) > sizeof(Tc);
  Tin ox = 0, oy = 0, oz = 0;
  __device__ __forceinline__ void set(const Tin* X, int64_t v) {
    if constexpr (kShift) {
      ox = X[3 * v];
      oy = X[3 * v + 1];
      oz = X[3 * v + 2];
    }
  }
  // the same origin in every lane: to scalar registers
  __device__ __forceinline__ void to_scalar() {
    if constexpr (kShift) {
      ox = uniform(ox);
      oy = uniform(oy);
      oz = uniform(oz);
    }
  }
  __device__ __forceinline__ V3<Tc> load(const Tin* X, int64_t v) const {
    if constexpr (kShift)
      return {(Tc)(X[3 * v] - ox), (Tc)(X[3 * v + 1] - oy), (Tc)(X[3 * v + 2] - oz)};
    else
      return load_vertex<Tc>(X, v);
  }
};

// The R consecutive segments of loop B owned by a lane: vertices k_0..k_R,
// segment vectors s_r = k_{r+1} - k_r and the constants s_r x (k_r - k_0) of
// the numerator p.  Segments past the end of the item have zero length
// (repeated vertices) and add exactly 0.
template <typename T, int R>
struct Segs {
  V3<T> k[R + 1];
  V3<T> s[R];
  V3<T> m[R];
};

// Walk state at vertex l_j of loop A, for all R + 1 vertices of the lane:
// V_r = l_j - k_r, N_r = |V_r|, E_r = N_r N_{r+1} + V_r . V_{r+1},
// G_r = s_r . V_r.
template <typename T, int R>
struct Walk {
  V3<T> l;
  V3<T> V[R + 1];
  T N[R + 1];
  T E[R];
  T G[R];
};

// `first`: the lane's walk starts at l.  Otherwise the state is, bit for bit,
// what the steps up to l leave there: it depends on l only, and only E_r is
// another rounding of the same value (|d|^2 - s_r . d in the place of d . c).
template <typename T, int R>
__device__ __forceinline__ void walk_init(Walk<T, R>& w, const V3<T>& l, const Segs<T, R>& g,
                                          bool first) {
  w.l = l;
  T n2[R + 1];
#pragma unroll
  for (int r = 0; r <= R; ++r) {
    w.V[r] = l - g.k[r];
    n2[r] = dot_r(w.V[r], w.V[r]);
  }
  sqrt_n<R + 1>(n2, w.N);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    w.G[r] = dot_r(g.s[r], w.V[r]);
    w.E[r] = fmad(w.N[r], w.N[r + 1], first ? dot_r(w.V[r], w.V[r + 1]) : n2[r] - w.G[r]);
  }
}

// One step of the walk, segment (l_j, l_{j+1}) against the lane's R segments:
// the merged arctangents' arguments (term r is atan2(Y[r], X[r]) / (2 pi)),
// and the walk advanced to l_{j+1}.  For segment r: a = V_r, b = V_{r+1} (at
// l_j), c = v_{r+1}, d = v_r (at l_{j+1}); a.b enters through E_r, and the
// "vertical" products V_r . v_r are shared by segments r - 1 and r.
template <typename T, int R>
__device__ __forceinline__ void walk_xy(Walk<T, R>& w, const V3<T>& l1, const Segs<T, R>& g,
                                        T (&X)[R], T (&Y)[R]) {
  const V3<T> sj = l1 - w.l;
  const V3<T> M = cross_r(w.V[0], sj);
  w.l = l1;
  T n2[R + 1], n[R + 1], vert[R + 1];
#pragma unroll
  for (int r = 0; r <= R; ++r) {
    const V3<T> v = l1 - g.k[r];
    n2[r] = dot_r(v, v);
    vert[r] = dot_r(w.V[r], v);
    w.V[r] = v;
  }
  sqrt_n<R + 1>(n2, n);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const T na = w.N[r], nb = w.N[r + 1], nc = n[r + 1], nd = n[r];
    const T gr = dot_r(g.s[r], w.V[r]);
    T p = dot_r(g.s[r], M);
    if (r > 0) {
      const V3<T>& m = g.m[r];
      p = fmad(g.s[r].x, M.x, fmad(g.s[r].y, M.y, fmad(g.s[r].z, M.z, -dot_r(sj, m))));
    }
    const T ca = vert[r] - w.G[r];
    const T f = fmad(nd, nc, n2[r] - gr);
    const T d1 = fmad(ca, nb, fmad(vert[r + 1], na, nc * w.E[r]));
    const T d2 = fmad(ca, nd, fmad(vert[r], nc, na * f));
    Y[r] = p * fabs_t(d1 + d2);  // |.| is a free source modifier
    X[r] = fmad(d1, d2, -(p * p));
    w.E[r] = f;
    w.G[r] = gr;
  }
#pragma unroll
  for (int r = 0; r <= R; ++r) w.N[r] = n[r];
}

// 2 pi times the sum of the step's R terms, by the arctangent of the full range.
// RUN: in a run of such steps, where FP32's reciprocals are a block (rcp_n).
template <typename T, int AT, int R, bool RUN = false>
__device__ __forceinline__ T full_angles(const T (&X)[R], const T (&Y)[R]) {
  T sum = 0;
  if constexpr (RUN && sizeof(T) == 4 && AT == 2) {
    T mx[R], inv[R];
#pragma unroll
    for (int r = 0; r < R; ++r) mx[r] = fmaxf(fabsf(X[r]), fabsf(Y[r]));
    rcp_n<R>(mx, inv);
#pragma unroll
    for (int r = 0; r < R; ++r) sum += atan2_minimax(Y[r], X[r], inv[r]);
  } else {
#pragma unroll
    for (int r = 0; r < R; ++r) sum += angle<T, AT>(Y[r], X[r]);
  }
  return sum;
}

// The tangent t = Y / X of a term, by the same operations as the full-range
// arctangent takes where 0 < X and |Y| <= X (its octant reduction is then the
// identity).  That holds for t below SmallAngle::octant, which is below 1 by more
// than a reciprocal that is off by its last place can move t: an |Y| just above X
// can give a t just below 1.
template <int R>
__device__ __forceinline__ void tangents(const float (&X)[R], const float (&Y)[R], float (&t)[R]) {
  float i[R];
  rcp_n<R>(X, i);
#pragma unroll
  for (int r = 0; r < R; ++r) t[r] = Y[r] * i[r];
}
template <int R>
__device__ __forceinline__ void tangents(const double (&X)[R], const double (&Y)[R],
                                         double (&t)[R]) {
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const double x = X[r], y = Y[r];
    double i = __builtin_amdgcn_rcp(x);
    i = fma(i, fma(-x, i, 1.0), i);
    i = fma(i, fma(-x, i, 1.0), i);
    const double q = y * i;
    t[r] = fma(fma(-x, q, y), i, q);
  }
}

// The arctangent of a small t: the full range's polynomial and Horner order from
// a lower coefficient D on.  For |t| < lim[k] the rounded polynomial is the full
// range's.  Where D[k] > 0 (FP32 s = t^2 below 2^-12, FP64 2^-20 and 2^-12) the
// coefficients above D[k] change the sum before its last rounding by less than
// 2^-36 of its last place (FP64 2^-40); no difference in 2e8 random t (a CPU test
// tries a part of them).  FP32's D = 0 takes 1 for 1 - s/3 + ..: below the limit
// s/3 is less than 2^-25, half the place below 1, so the full chain rounds to 1
// (the limit could be sqrt(3) 2^-12.5 = 2.99e-4), and t times 1 is t.
// The angle of a term is about |s_j| |s_r| / h^2 for segments at distance h,
// so a polyline that follows its curve has small ones: of the steps of
// 256 terms in chainmail of 64 segments a ring, 1% have one above 1/32 and
// none one above 1/16; nearly all of the knit and long-loop workloads' terms
// are below 2.9e-4.  The class tests the tangents of a step: `worst` is not
// below a limit if any |t| is not, if a t is NaN, or unless every X > 0.
template <typename T>
struct SmallAngle;
template <>
struct SmallAngle<float> {
  static constexpr int kFull = LK_ATAN_DEG;
  static constexpr int D[2] = {0, 4};
  static constexpr float lim[2] = {2.9e-4f, 0.015625f};
  static constexpr float octant = 0.5f;  // (of the values that an instruction holds)
  float lo = INFINITY, worst = 0.0f;
  __device__ __forceinline__ void add(float x, float t) {
    lo = fminf(lo, x);
    worst = __builtin_elementwise_maximum(worst, fabsf(t));  // keeps a NaN, as t is for an X that is
  }
  __device__ __forceinline__ bool below(float limit) const { return lo > 0.0f && worst < limit; }
  template <int N>
  static __device__ __forceinline__ float eval(float t) {
#pragma clang fp contract(off)  // t * q is rounded before it is summed
    const float s = t * t;
    float q = kAtanQ[N];
#pragma unroll
    for (int k = N - 1; k >= 0; --k) q = fmaf(q, s, kAtanQ[k]);
    return N == 0 ? t : t * q;
  }
};
// (FP64: on the upper words, whose order is the values' and whose minimum and
// maximum are cheaper; a word above 0x7ff00000 is a NaN's)
template <>
struct SmallAngle<double> {
  static constexpr int kFull = LK_ATAN_DEG64;
  static constexpr int D[2] = {4, 7};
  static constexpr uint32_t lim[2] = {0x3f500000u, 0x3f900000u};  // 2^-10, 2^-6
  static constexpr uint32_t octant = 0x3fefffffu;  // 1 - 2^-21
  int32_t lo = 0x7fffffff;
  uint32_t worst = 0u;
  __device__ __forceinline__ void add(double x, double t) {
    const int32_t hx = __double2hiint(x);
    const uint32_t ht = (uint32_t)__double2hiint(t) & 0x7fffffffu;
    lo = hx < lo ? hx : lo;
    worst = ht > worst ? ht : worst;
  }
  __device__ __forceinline__ bool below(uint32_t limit) const { return lo > 0 && worst < limit; }
  template <int N>
  static __device__ __forceinline__ double eval(double t) {
#pragma clang fp contract(off)
    const double s = t * t;
    double q = kAtanQ64[N];
#pragma unroll
    for (int k = N - 1; k >= 0; --k) q = fma(q, s, kAtanQ64[k]);
    return t * q;
  }
};

// 2 pi times the sum of one step's R terms.  Each wave takes the shortest
// arctangent that serves all its lanes; every choice gives the same value, so
// a lane's sum does not depend on what shares its wave.  Vector instructions
// a term after X and Y, tangent and tests included: 4 (all below 2.9e-4), 10
// (2^-6), 14 (below 1/2, FP64 1: the octant reduction left out) and 26, against 22
// for the full form alone; FP64 20, 23, 35 and 55 against 38.  `full` counts the
// steps that took the full form, for the walk to leave the tests out (kFullRun).
template <typename T, int N, int R>
__device__ __forceinline__ T sum_small(const T (&t)[R]) {
  T sum = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) sum += SmallAngle<T>::template eval<N>(t[r]);
  return sum;
}
template <typename T, int AT, int R>
__device__ __forceinline__ T step_angles(const T (&X)[R], const T (&Y)[R], int& full) {
  using A = SmallAngle<T>;
  if constexpr (AT == 1 || AT == kFullForm) {
    return full_angles<T, AT, R>(X, Y);
  } else {
    T t[R];
    tangents<R>(X, Y, t);
    A a;
#pragma unroll
    for (int r = 0; r < R; ++r) a.add(X[r], t[r]);
    if (!__any(!a.below(A::lim[0]))) return sum_small<T, A::D[0], R>(t);
    if (!__any(!a.below(A::lim[1]))) return sum_small<T, A::D[1], R>(t);
    if (!__any(!a.below(A::octant))) return sum_small<T, A::kFull, R>(t);
    ++full;
    return full_angles<T, AT, R>(X, Y);
  }
}

// Where the lanes of one work item sit: B block [b0, b0 + nbh) of loop B split
// into `slots` lanes of R segments; if that leaves lanes over, they form
// `groups` that split the item's A range [a0, a0 + nah) into [js, je).
struct Layout {
  int b0, a0, nbh, nah, bi, js, je;
  bool active;
};

// 32-bit arithmetic throughout: the plan guarantees fewer than 2^31 items per
// pair and 2^31 vertices per loop, and js/je products stay below 2^30
// (chunk <= 2^24, 64 groups).  `width`: lanes given to the item (a power of
// two dividing 64; `lane` counts within them).
template <int R>
__device__ __forceinline__ Layout layout(const WorkRec& r, int64_t local, int chunk, int lane,
                                         unsigned width = kWave) {
  constexpr unsigned kB = kWave * R;
  Layout L;
  const unsigned nbb = ((unsigned)r.nb + kB - 1) / kB;
  const unsigned loc = (unsigned)local;
  const unsigned bq = loc / nbb;
  L.b0 = (int)((loc - bq * nbb) * kB);
  L.a0 = (int)(bq * (unsigned)chunk);
  L.nbh = (int)((r.nb - L.b0) < kB ? (r.nb - L.b0) : kB);
  L.nah = (int)((r.na - L.a0) < chunk ? (r.na - L.a0) : chunk);
  const unsigned slots = ((unsigned)L.nbh + R - 1) / R;
  const unsigned groups = slots <= width ? width / slots : 1u;
  const unsigned g = (unsigned)lane / slots;
  L.bi = (int)((unsigned)lane - g * slots);
  L.active = g < groups;
  L.js = (int)(((unsigned)L.nah * g) / groups);
  L.je = (int)(((unsigned)L.nah * (g + 1)) / groups);
  return L;
}

// Vertex k_{b0 + bi R + r} of loop B for r = 0..R (cyclic).  Past the end
// of the block the lane repeats the block's end vertex, so its padding
// segments have zero length: their Eq. 4 term is exactly 0 (p = 0 and
// d1 d2 > 0 unless a vertex of loop A sits on that vertex, which only
// touching loops do), and the sum needs no mask.  The crossing count still
// masks them (Segs::valid), since a zero-length segment has no certain side.
template <typename Tin, typename Tc, int R>
__device__ __forceinline__ void load_b(const Tin* X, const WorkRec& w, const Layout& L,
                                       const Frame<Tin, Tc>& F, V3<Tc>* k) {
  const int first = L.bi * R;
#pragma unroll
  for (int r = 0; r <= R; ++r) {
    int i = L.b0 + (first + r < L.nbh ? first + r : L.nbh);
    if (i >= w.nb) i -= w.nb;
    k[r] = F.load(X, w.ob + i);
  }
}

template <typename Tc, int R>
__device__ __forceinline__ void make_segs(const V3<Tc>* k, Segs<Tc, R>& sg) {
#pragma unroll
  for (int r = 0; r <= R; ++r) sg.k[r] = k[r];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    sg.s[r] = sg.k[r + 1] - sg.k[r];
    sg.m[r] = cross_r(sg.s[r], sg.k[r] - sg.k[0]);
  }
}

// Walk the segments l[0] l[1], .. up to le[0] of the item's A range, in LDS
// (le[1] is read too); `first`: the lane's walk starts at l.  The walk state is
// made afresh at l and at the remainder (the same bits), so no registers hold
// it across tiles and loops.  ALU-bound: 139 vector instructions and 5 square
// roots a step of R = 4 before the arctangents.  The chainmail workload's
// kernel went from 428 to 320 us (to 268 with the work queues), that of three
// pairs of 90,000 segments from 33.7 to 18.3 ms (73 to 127 TFLOP/s at 90 FLOP a
// term).
// After four steps that all took the full arctangent, the next kFullRun groups of
// four take it without a test: where all angles are large (random polygons) the
// tests cost a fifth of an FP64 walk.  1,770 pairs of 1,000 random segments took
// 6,520 us in FP64 and 2,930 mixed without such runs, now 5,510 and 2,580 (5,430
// and 2,500 with the full form alone); smooth curves never get there.  A branch in
// each step, in the place of one around groups, cost those 3-11%.  FP32 runs are
// not unrolled: its registers are all in use.
// `sink` takes the sums of four steps in the compute type, then those of the
// last steps one by one; added up in that order in FP64 they are the lane's sum.
// EACH: it takes the steps' sums instead.
constexpr int kFullRun = 16;
template <typename Tc, int AT, int R, bool EACH = false, typename Sink>
__device__ __forceinline__ void walk(const Vtx<Tc>* l, const Vtx<Tc>* le, bool first,
                                     const Segs<Tc, R>& sg, const Sink& sink) {
  if (l + 4 <= le) {
    Walk<Tc, R> wk;
    walk_init(wk, V3<Tc>{l[0].x, l[0].y, l[0].z}, sg, first);
    first = false;
    V3<Tc> vn{l[1].x, l[1].y, l[1].z};
    // one step to vn; `next` is the vertex after it
    const auto step = [&](const Vtx<Tc>* next, const auto& angles,
                          Tc& s4) __attribute__((always_inline)) {
      const V3<Tc> v1 = vn;
      Tc X[R], Y[R];
      vn = {next->x, next->y, next->z};
      walk_xy(wk, v1, sg, X, Y);
      if constexpr (EACH)
        sink(angles(X, Y));
      else
        s4 += angles(X, Y);
    };
    using Args = const Tc(&)[R];
    do {
      int full;
      do {
        Tc s4 = 0;
        full = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q)
          step(l + q + 2, [&](Args X, Args Y) { return step_angles<Tc, AT, R>(X, Y, full); }, s4);
        if constexpr (!EACH) sink(s4);
        l += 4;
      } while (full < 4 && l + 4 <= le);
      if (__builtin_expect(full == 4, 0)) {
        for (int k = 0; k < kFullRun && l + 4 <= le; ++k) {
          const auto angles = [](Args X, Args Y) { return full_angles<Tc, AT, R, true>(X, Y); };
          Tc s4 = 0;
          if constexpr (sizeof(Tc) == 8) {
#pragma unroll
            for (int q = 0; q < 4; ++q) step(l + q + 2, angles, s4);
            l += 4;
          } else {
#pragma unroll 1
            for (int q = 0; q < 4; ++q) step(++l + 1, angles, s4);
          }
          if constexpr (!EACH) sink(s4);
        }
      }
    } while (l + 4 <= le);
  }
  if (l < le) {
    Walk<Tc, R> wk;
    walk_init(wk, V3<Tc>{l[0].x, l[0].y, l[0].z}, sg, first);
    do {
      ++l;
      Tc X[R], Y[R];
      walk_xy(wk, V3<Tc>{l[0].x, l[0].y, l[0].z}, sg, X, Y);
      int full = 0;
      sink(step_angles<Tc, AT, R>(X, Y, full));
    } while (l < le);
  }
}

template <typename Tc, int AT, int R>
__device__ __forceinline__ void walk_tile(const Vtx<Tc>* l, const Vtx<Tc>* le, bool first,
                                          const Segs<Tc, R>& sg, double& acc) {
  walk<Tc, AT, R>(l, le, first, sg, [&](Tc sum) { acc += (double)sum; });
}

// ---------------------------------------------------------------------------
// Count Crossings (Sec. 2.1, Alg. 4): the linking number is half the signed
// number of crossings of a regular projection.  The projection is along a view
// direction n (uniform over the launch).  Two projected segments cross iff the
// endpoints of each lie strictly on opposite sides of the other's line.  The
// side of a point x relative to the projected line through y with direction e
// is the sign of (x - y) . (n x e), so no coordinate is rotated: a step forms
// u = n x s_j once and every lane holds t_r = n x s_r.  With v_r = l_{j+1} - k_r:
//   side of k_r      w.r.t. segment j's line:  w_r = v_r . u
//   side of l_{j+1}  w.r.t. segment r's line:  q_r = v_r . t_r
// (the side of l_j is the previous step's q_r).  At a crossing the points of
// the two segments over the crossing differ by h n, so the Eq. 4 numerator
// p = a . (s_j x s_r) = v_r . (s_j x s_r) = h n . (s_j x s_r) has the sign of
// the crossing (over tangent x under tangent, against n); the count sums
// sign(p) and the pair's value is half of it.
//
// Every predicate is certified in FP32 on the vertices as given: a value
// counts only when its magnitude exceeds a forward error bound of the form
// tau |first|_inf |second|_inf (about 63 u for w and q, 216 u for p with the
// unit roundoff u = 2^-24, from first-order error analysis of the differences,
// the cross products and the dot products; tau defaults to twice that).  A
// term that is neither certainly crossing nor certainly not crossing, or an
// odd total, makes the pair's value NaN or a half-integer, and the pair is
// counted again by this kernel in FP64 (Tc = double, bounds at u = 2^-53):
// the depth separation of two segments enters |v| but not the side values,
// so at shallow crossings of curves far apart in depth the FP32 bound is
// loose while FP64 decides.  Only a pair that FP64 cannot decide either -- a
// crossing within about 1e-16 of a vertex, overlapping projected segments,
// segments that touch in space -- goes to the FP64 direct sum.  Needs
// |n|_inf <= 1 (the runtime scales n so).
constexpr int kCrossings = 3;  // term form of the kernel's template: crossing count

template <typename T, int R>
struct CcSegs {
  V3<T> k[R + 1];
  V3<T> t[R];    // n x s_r
  T cq[R];       // tau |s_r|_inf: certainty scale of q_r
  T sn[R];       // |s_r|_inf
  V3<T> n;       // view direction
  T tau, tau_p;
  bool valid[R];
};

// Walk state at l_j: the vertex and the certified sides of l_j relative to
// the lane's R segment lines (0 = uncertain).
template <typename T, int R>
struct CcWalk {
  V3<T> l;
  T Q[R];
};

template <typename T>
__device__ __forceinline__ T inf_norm(const V3<T>& a) {
  return fmax(fmax(fabs(a.x), fabs(a.y)), fabs(a.z));
}

// x if |x| > tol, else 0 (the sign survives only when it is certain; NaN -> 0)
template <typename T>
__device__ __forceinline__ T certain(T x, T tol) {
  return fabs(x) > tol ? x : (T)0;
}

template <typename Tc, int R>
__device__ __forceinline__ void make_lane(const V3<Tc>* k, const Layout& L, const DsArgs& A,
                                          CcSegs<Tc, R>& sg) {
  const int first = L.bi * R;
  sg.n = V3<Tc>{A.view[0], A.view[1], A.view[2]};
  sg.tau = (Tc)A.cc_tau;
  sg.tau_p = (Tc)A.cc_tau_p;
#pragma unroll
  for (int r = 0; r <= R; ++r) sg.k[r] = k[r];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const V3<Tc> s = sg.k[r + 1] - sg.k[r];
    sg.t[r] = cross(sg.n, s);
    sg.sn[r] = inf_norm(s);
    sg.cq[r] = sg.tau * sg.sn[r];
    sg.valid[r] = first + r < L.nbh;
  }
}

template <typename Tc, int R>
__device__ __forceinline__ void cc_init(CcWalk<Tc, R>& w, const V3<Tc>& l, const CcSegs<Tc, R>& g) {
  w.l = l;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const V3<Tc> V = l - g.k[r];
    w.Q[r] = certain(dot(V, g.t[r]), g.cq[r] * inf_norm(V));
  }
}

// One step l_j -> l_{j+1} against the lane's R segments: adds the certified
// crossing signs to cnt, sets bad when a term is undecided.
template <typename Tc, int R>
__device__ __forceinline__ void cc_step(CcWalk<Tc, R>& w, const V3<Tc>& l1, const CcSegs<Tc, R>& g,
                                        int& cnt, bool& bad) {
  const V3<Tc> sj = l1 - w.l;
  const V3<Tc> u = cross(g.n, sj);
  const Tc sjn = inf_norm(sj);
  const Tc cw = g.tau * sjn;
  V3<Tc> v[R + 1];
  Tc nv[R + 1], wc[R + 1];
#pragma unroll
  for (int r = 0; r <= R; ++r) {
    v[r] = l1 - g.k[r];
    nv[r] = inf_norm(v[r]);
    wc[r] = certain(dot(v[r], u), cw * nv[r]);
  }
  Tc Wp[R], Qp[R];
  bool cand[R];
  bool any = false;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const Tc qc = certain(dot(v[r], g.t[r]), g.cq[r] * nv[r]);
    Wp[r] = wc[r] * wc[r + 1];  // < 0: k_r, k_{r+1} certainly on opposite sides
    Qp[r] = w.Q[r] * qc;        // < 0: l_j, l_{j+1} certainly on opposite sides
    w.Q[r] = qc;
    // either product certainly positive: certainly no crossing
    cand[r] = g.valid[r] && !(fmax(Wp[r], Qp[r]) > (Tc)0);
    any = any || cand[r];
  }
  w.l = l1;
  if (any) {  // rare: a crossing or an undecided term somewhere in the lane
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (!cand[r]) continue;
      const V3<Tc> s = g.k[r + 1] - g.k[r];
      const Tc p = dot(v[r], cross(sj, s));
      const Tc tp = g.tau_p * g.sn[r] * sjn * nv[r];
      if (Wp[r] < (Tc)0 && Qp[r] < (Tc)0 && fabs(p) > tp) {
        cnt += p > (Tc)0 ? 1 : -1;
      } else {
        bad = true;
      }
    }
  }
}

template <typename Tc, int AT, int R>
__device__ __forceinline__ void walk_tile(const Vtx<Tc>* l, const Vtx<Tc>* le, bool,
                                          const CcSegs<Tc, R>& sg, double& acc) {
  CcWalk<Tc, R> wk;
  cc_init(wk, V3<Tc>{l[0].x, l[0].y, l[0].z}, sg);
  int cnt = 0;
  bool bad = false;
  V3<Tc> next{l[1].x, l[1].y, l[1].z};  // read a step ahead
#pragma unroll 2
  for (; l < le; ++l) {
    const V3<Tc> l1 = next;
    next = {l[2].x, l[2].y, l[2].z};
    cc_step(wk, l1, sg, cnt, bad);
  }
  acc += bad ? __builtin_nan("") : (double)cnt;
}

// One work item of the crossing count with culling: the item's B block (R
// blocks of 64 segments) has a projected box; loop A's superblocks and then
// blocks whose boxes are disjoint from it are skipped, and every other block
// is staged (65 vertices) and walked from a fresh start.  The box tests are
// uniform over the wave.
template <typename Tin, typename Tc, int R>
__device__ __forceinline__ void cc_item_culled(const DsArgs& A, const Tin* X,
                                               const Frame<Tin, Tc>& F, Vtx<Tc>* lds,
                                               const WorkRec& r, const Layout& L, int lane,
                                               const CcSegs<Tc, R>& sg, double& acc) {
  const int32_t ia = A.pairs[2 * (int64_t)r.p], ib = A.pairs[2 * (int64_t)r.p + 1];
  const int64_t o0 = A.off[0];
  const int64_t bslot = (r.ob - o0) / kCcBlock + ib + L.b0 / kCcBlock;
  float4 bb = float4{INFINITY, -INFINITY, INFINITY, -INFINITY};
  bool bok = true;
#pragma unroll
  for (int c = 0; c < R; ++c) {
    if (L.b0 + (int64_t)c * kCcBlock < r.nb) {
      if ((uint64_t)(bslot + c) < (uint64_t)A.cc_nblk) {
        const float4 q = A.cc_blk[bslot + c];
        bb = float4{fminf(bb.x, q.x), fmaxf(bb.y, q.y), fminf(bb.z, q.z), fmaxf(bb.w, q.w)};
      } else {
        bok = false;
      }
    }
  }
  if (!bok) bb = float4{-INFINITY, INFINITY, -INFINITY, INFINITY};  // no box: cull nothing
  const int64_t ablk = (r.oa - o0) / kCcBlock + ia;
  const int64_t asup = (r.oa - o0) / kCcSuper + ia;
  const int a0 = (int)L.a0, a_end = (int)L.a0 + L.nah;
  const int lo_l = a0 + L.js, hi_l = a0 + L.je;  // this lane's segments of A
  for (int sp = a0 / kCcSuper; sp * kCcSuper < a_end; ++sp) {
    if ((uint64_t)(asup + sp) < (uint64_t)A.cc_nsup && boxes_disjoint(A.cc_sup[asup + sp], bb))
      continue;
    const int k0 = max(sp * (kCcSuper / kCcBlock), a0 / kCcBlock);
    const int k1 = min((sp + 1) * (kCcSuper / kCcBlock), (a_end + kCcBlock - 1) / kCcBlock);
    for (int k = k0; k < k1; ++k) {
      if ((uint64_t)(ablk + k) < (uint64_t)A.cc_nblk && boxes_disjoint(A.cc_blk[ablk + k], bb))
        continue;
      const int v0 = k * kCcBlock;
      __syncthreads();
      for (int t = lane; t <= kCcBlock; t += kWave) {
        const int idx = (v0 + t) % r.na;  // the block's vertices, cyclic
        const V3<Tc> x = F.load(X, r.oa + idx);
        lds[t] = Vtx<Tc>{x.x, x.y, x.z, (Tc)0};
      }
      __syncthreads();
      const int jlo = max(v0, lo_l), jhi = min(v0 + kCcBlock, hi_l);
      if (L.active && jlo < jhi)
        walk_tile<Tc, kCrossings, R>(lds + (jlo - v0), lds + (jhi - v0), true, sg, acc);
    }
  }
}

// Per-lane state of the term form AT (the direct sum's, or the crossing count's).
template <typename Tc, int AT, int R>
struct LaneOf {
  using S = Segs<Tc, R>;
};
template <typename Tc, int R>
struct LaneOf<Tc, kCrossings, R> {
  using S = CcSegs<Tc, R>;
};

template <typename Tc, int R>
__device__ __forceinline__ void make_lane(const V3<Tc>* k, const Layout& L, const DsArgs&,
                                          Segs<Tc, R>& sg) {
  make_segs<Tc, R>(k, sg);
}

// Scale from the lane sums to the pair's value: 1 / (2 pi) for the direct
// sum's angles, 1/2 for crossing signs.
template <int AT>
__device__ __forceinline__ double value_scale() {
  return AT == kCrossings ? 0.5 : kInvTwoPi;
}

// Wave sum of the lanes' partials.  `whole`: this item is the pair's only one,
// so its value is final and the pair is finalised at once (`fpre`: the pair's
// flags as the plan left them, loaded when the item started so that finishing
// does not wait on a load).  Otherwise the sum goes into the pair's fixed-point
// accumulator, and the pair is finalised after this kernel, from the big list.
template <int AT>
__device__ __forceinline__ void finish_item(double acc, int32_t p, int lane, const DsArgs& A,
                                            bool whole, uint32_t fpre) {
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
  if (lane != 0) return;
  const double v = acc * value_scale<AT>();
  const bool ok = fabs(v) < 1.0e14;  // false for NaN / Inf / absurd magnitude
  if (whole)
    finalize_pair(A.out, p, v, fpre | (ok ? 0u : kFlagNonfinite));
  else if (ok)
    fixed_add(&A.acc[2 * (int64_t)p], v);
  else
    atomicOr(&A.out.flags[p], kFlagNonfinite);
}

// Code placement of the walk loops of the FP32 kernel (R = 4, FP32 input): each
// starts 4 bytes past an 8-byte boundary of the kernel and the big items' one
// 12 bytes past a 32-byte boundary, which these no-ops (4 bytes each) arrange.
// While transcendentals left the waves out of step (sqrt_n), the placement moved
// a call's time by 7-10%; now offsets of 0-16 bytes give 349.3-350.4 us on the
// chainmail workload.  A CPU test checks the placements.
constexpr int kPadPacked = 4, kPadWhole = 1, kPadBig = 5;
template <typename Tin, typename Tc, int AT, int R, bool PK, int N>
__device__ __forceinline__ void place_code() {
  if constexpr (PK && sizeof(Tin) == 4 && sizeof(Tc) == 4 && AT == 2 && R == 4 && N > 0)
    asm volatile(".rept %0\n s_nop 0\n.endr" ::"n"(N));
}

// Waves per SIMD that a variant is compiled for (0: the compiler's choice).  The
// default FP32 kernel gets four (128 registers, which the walk leaves free by
// keeping no state across loops): the SIMD pairs instructions of two waves, so
// an even number runs better than three (chainmail kernel 415 us at 168
// registers and three waves, 363 us at four, before the transcendentals were
// put in blocks; the start of that change had 241 registers, two waves, 428 us).
template <typename Tc, int AT, int R>
constexpr int waves_per_simd() {
  return sizeof(Tc) == 4 && AT == 2 && R == 4 ? 4 : 0;
}

// Every variant must fit in 256 registers per lane (two waves per SIMD); a
// test checks the compiled register counts.
// R small pairs whose loop B fits one wave's lanes share a wave (PK, true in every
// variant: part of the symbol that records of measurements name).
template <typename Tin, typename Tc, int AT, int R, bool PK = true>
__global__ __launch_bounds__(kWave, (waves_per_simd<Tc, AT, R>())) void ds_persistent(DsArgs A) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  Vtx<Tc>* lds = reinterpret_cast<Vtx<Tc>*>(lds_raw);
  const int lane = threadIdx.x;
  const Tin* X = static_cast<const Tin*>(A.xyz);
  const int64_t big_total = uniform(*A.s.big_total);
  const int64_t n_big = uniform(A.s.counts[1]);
  const int64_t n_small = uniform(A.s.counts[0]);
  const int64_t total = big_total + (n_small + A.batch - 1) / A.batch;

  // A wave's first work index is its workgroup index, so a launch with fewer
  // items than waves costs no atomic at all; later indices, offset by the grid,
  // come from a device counter.  An atomic on one counter takes 5 ns, so many
  // short items get kQueues of them: queue q hands out the indices that are q
  // modulo the number of queues, to the waves whose index is.  Split pairs' items
  // are long and differ, and their list starts with the largest: below eight per
  // wave they stay in one queue.  With one queue / 16, us per call on one MI355X:
  // 69,041 pairs of 64 x 64 segments, mixed 347 / 283, crossings 294 / 186; 13,000
  // of 61 x 61 in FP64 267 / 248; 20,000 of 128 x 3 366 / 167, of 150 x 150 808 /
  // 730; 700 pairs of 1,500 x 1,500 in FP64 (8,400 items) 4,085 / 4,210.
  // The next index is fetched one item ahead so the atomic's latency overlaps
  // the current item's arithmetic; a fused check's stop flag is read with it
  // (device-scope load, so another wave's store is seen).
  const bool spread = total >= 8 * (int64_t)gridDim.x || 4 * big_total <= total ||
                      uniform(A.s.big[0].items) == 1;  // then no pair is split
  const unsigned n_queues = !spread ? 1u : gridDim.x < kQueues ? gridDim.x : kQueues;
  const unsigned queue = blockIdx.x % n_queues;
  unsigned long long* const my_counter = A.s.counter + queue * kQueueStride;
  unsigned long long wnext = blockIdx.x;
  int stopnext = 0;
  if (lane == 0 && A.out.stop)
    stopnext = __hip_atomic_load(A.out.stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  for (;;) {
    const int64_t w = uniform((int64_t)wnext);  // lane 0's
    if (w >= total || uniform(stopnext)) break;
    if (lane == 0) {
      wnext = gridDim.x + queue + (unsigned long long)n_queues * atomicAdd(my_counter, 1ull);
      if (A.out.stop)
        stopnext = __hip_atomic_load(A.out.stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }

    if (w < big_total) {
      // one item of a big pair: position with big_prefix[pos] <= w < big_prefix[pos + 1]
      int64_t lo = 0, hi = n_big;
      while (hi - lo > 1) {
        const int64_t mid = (lo + hi) >> 1;
        if (uniform(A.s.big_prefix[mid]) <= w)
          lo = mid;
        else
          hi = mid;
      }
      const WorkRec r = uniform(A.s.big[lo]);
      const uint32_t fpre = r.items == 1 ? A.out.flags[r.p] : 0u;
      const Layout L = layout<R>(r, w - uniform(A.s.big_prefix[lo]), A.chunk, lane);
      Frame<Tin, Tc> F;
      F.set(X, r.ob + L.b0);
      F.to_scalar();
      V3<Tc> kv[R + 1];
      load_b<Tin, Tc, R>(X, r, L, F, kv);
      typename LaneOf<Tc, AT, R>::S sg;
      make_lane<Tc, R>(kv, L, A, sg);
      double acc = 0.0;
      bool culled = false;
      if constexpr (AT == kCrossings) {
        if (A.cc_blk) {
          cc_item_culled<Tin, Tc, R>(A, X, F, lds, r, L, lane, sg, acc);
          culled = true;
        }
      }
      place_code<Tin, Tc, AT, R, PK, kPadBig>();
      if (!culled)
      for (int t0 = 0; t0 < L.nah; t0 += A.tile) {
        const int tl = (L.nah - t0) < A.tile ? (L.nah - t0) : A.tile;
        __syncthreads();
        for (int v = lane; v <= tl; v += kWave) {
          unsigned idx = (unsigned)L.a0 + (unsigned)t0 + (unsigned)v;
          if (idx >= (unsigned)r.na) idx -= (unsigned)r.na;  // closing vertex of the loop
          const V3<Tc> x = F.load(X, r.oa + idx);
          lds[v] = Vtx<Tc>{x.x, x.y, x.z, (Tc)0};
        }
        __syncthreads();
        const int jlo = L.js > t0 ? L.js : t0;
        const int jhi = L.je < t0 + tl ? L.je : t0 + tl;
        if (L.active && jlo < jhi)
          walk_tile<Tc, AT, R>(lds + (jlo - t0), lds + (jhi - t0), jlo == L.js, sg, acc);
      }
      finish_item<AT>(acc, r.p, lane, A, r.items == 1, fpre);
    } else {
      // a batch of small pairs (one item each, loop A of at most kSmallA - 1
      // segments).  Pairs whose loop B has at most 64 segments run R at a
      // time when R > 1, 64 / R lanes each (each lane walks more of loop A,
      // and the per-pair setup, reduction and finalisation are shared); the
      // others run one at a time on the whole wave.  Which way a pair runs
      // depends only on the pair, so results are reproducible.  Records are
      // re-read from the list where needed rather than held in registers
      // across the walks.
      const int64_t m0 = (w - big_total) * (int64_t)A.batch;
      const int cnt = (int)((n_small - m0) < A.batch ? (n_small - m0) : A.batch);
      const WorkRec* recs = A.s.small + m0;
      const int32_t nb_l = lane < cnt ? recs[lane].nb : 0;
      const unsigned long long pmask = __ballot(PK && R > 1 && lane < cnt && nb_l <= kWave);
      unsigned long long smask = __ballot(lane < cnt) & ~pmask;
      const int npk = __popcll(pmask);
      if (npk > 0) {
        constexpr int K = R, S = kWave / R;
        for (int r0 = 0; r0 < npk; r0 += K) {
          // what comes from the lane index is computed again in each round:
          // kept, it would cost the FP32 walk registers that it has not got
          int ln = lane;
          if constexpr (sizeof(Tc) == 4) asm volatile("" : "+v"(ln));
          const int seg = ln / S, sl = ln - seg * S;
          Vtx<Tc>* myl = lds + seg * kSmallA;
          const bool has = r0 + seg < npk;
          // batch position of the (r0 + seg)-th packed pair
          unsigned long long mm = pmask;
          for (int t = has ? r0 + seg : r0; t > 0; --t) mm &= mm - 1ull;
          const WorkRec cur = recs[__ffsll((long long)mm) - 1];
          const uint32_t fm = A.out.flags[cur.p];
          Frame<Tin, Tc> F;
          F.set(X, cur.ob);
          __syncthreads();
          if (has)
            for (int v = sl; v <= cur.na; v += S) {
              const V3<Tc> x = F.load(X, cur.oa + (v < cur.na ? v : 0));
              myl[v] = Vtx<Tc>{x.x, x.y, x.z, (Tc)0};
            }
          const Layout L = layout<R>(cur, 0, A.chunk, sl, S);
          V3<Tc> kv[R + 1];
          load_b<Tin, Tc, R>(X, cur, L, F, kv);
          typename LaneOf<Tc, AT, R>::S sg;
          make_lane<Tc, R>(kv, L, A, sg);
          __syncthreads();
          double acc = 0.0;
          place_code<Tin, Tc, AT, R, PK, kPadPacked>();
          if (has && L.active && L.js < L.je)
            walk_tile<Tc, AT, R>(myl + L.js, myl + L.je, true, sg, acc);
#pragma unroll
          for (int o = S / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
          if (has && sl == 0) {
            const double v = acc * value_scale<AT>();
            finalize_pair(A.out, cur.p, v, fm | (fabs(v) < 1.0e14 ? 0u : kFlagNonfinite));
          }
        }
      }
      while (smask) {
        const int m = __ffsll((long long)smask) - 1;
        smask &= smask - 1ull;
        const WorkRec cur = uniform(recs[m]);
        const uint32_t fm = A.out.flags[cur.p];
        const Layout L = layout<R>(cur, 0, A.chunk, lane);
        Frame<Tin, Tc> F;
        F.set(X, cur.ob);
        F.to_scalar();
        V3<Tc> kv[R + 1];
        load_b<Tin, Tc, R>(X, cur, L, F, kv);
        const V3<Tc> a_lo = F.load(X, cur.oa + (lane < cur.na ? lane : 0));
        const V3<Tc> a_hi = F.load(X, cur.oa + (lane + kWave < cur.na ? lane + kWave : 0));
        __syncthreads();
        if (lane <= cur.na) lds[lane] = Vtx<Tc>{a_lo.x, a_lo.y, a_lo.z, (Tc)0};
        if (lane + kWave <= cur.na) lds[lane + kWave] = Vtx<Tc>{a_hi.x, a_hi.y, a_hi.z, (Tc)0};
        typename LaneOf<Tc, AT, R>::S sg;
        make_lane<Tc, R>(kv, L, A, sg);
        __syncthreads();
        double acc = 0.0;
        place_code<Tin, Tc, AT, R, PK, kPadWhole>();
        if (L.active && L.js < L.je)
          walk_tile<Tc, AT, R>(lds + L.js, lds + L.je, true, sg, acc);
        finish_item<AT>(acc, cur.p, lane, A, true, fm);
      }
    }
  }
}

// The direct sum of a call with few pairs: one item per workgroup of kTeam waves
// (a team).  With an item per wave such a call leaves most of the chip idle, or
// waits for the longest items: an item's walk is up to 4,096 steps long.  A team
// takes an item's tile in pieces of U steps, a wave each.  The lane sums keep
// their order to the last bit: a piece's sums of four steps go to LDS in the
// compute type, and the first wave adds them up in FP64 in the order of the walk
// while the others stage the next tile.  The pieces start every U steps (a
// multiple of four) from where the lane's walk of the tile starts, so the groups
// of four are those of ds_persistent, and a big pair's value is the same in both.
// A small pair is summed by one wave, all 64 lanes (each walks less of loop A than
// in a packed round), a work index taking up to kTeam of them: one in the main
// pass, which spreads them, kTeam in the refit pass, whose teams are few (with one
// a team 500 pairs of 100 segments that all need a refit took 370 us a call, now
// 148; 151 with an item per wave).  ALU-bound as ds_persistent is.
// Eight waves (FP64: four, which its registers let a compute unit hold two teams
// of) and U = 64 share the default tile; the LDS of two teams is 2 x 47 KB.  An
// FP64 tile of fewer steps is shared out in shorter pieces: with 64 the last waves
// of a team had none, and 512 pairs of 130 segments took 140 us, 107 so (an item
// per wave 108; 400 of 200 segments 132, 115, 138).  FP32 keeps pieces of 64: it
// starts a walk for each, which costs where the chip is full (neighbours of 100
// yarns 2,157 us, in shorter pieces 2,240).
// Against an item per wave, us per call on one MI355X: 276 pairs of 5 to 5,000
// segments 1,610 -> 546, neighbours of 100 yarns of up to 16,384 segments 3,330 ->
// 2,460, of 60 yarns in FP64 3,930 -> 2,560, three pairs of 90,000 segments 21,290
// -> 21,000 (such pairs fill the chip with items by themselves).  FP32 teams of
// four waves took 659 and 2,620 us, FP64 teams of eight 2,730.
template <typename Tc>
constexpr int kTeam = sizeof(Tc) == 4 ? 8 : 4;
template <typename Tc>
constexpr int team_piece(int tile) {
  const int u = (tile / kTeam<Tc>) & ~3;
  return u < 4 ? 4 : (u > 64 ? 64 : u);
}
template <typename Tc>
constexpr int team_slots(int tile) { return team_piece<Tc>(tile) / 4 + 3; }

template <typename Tin, typename Tc, int R>
__global__ __launch_bounds__(kWave * kTeam<Tc>, (sizeof(Tc) == 4 ? 4 : 2)) void ds_team(DsArgs A) {
  constexpr int AT = sizeof(Tc) == 4 ? 2 : 0;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  __shared__ unsigned long long next_w;
  __shared__ int next_stop;
  Vtx<Tc>* lds = reinterpret_cast<Vtx<Tc>*>(lds_raw);
  const int n_vtx = A.tile + 2 > kSmallA + 1 ? A.tile + 2 : kSmallA + 1;
  Tc* slots = reinterpret_cast<Tc*>(lds + n_vtx);
  const int U_max = uniform((int32_t)team_piece<Tc>(A.tile)), E = U_max / 4 + 3;
  const int wv = uniform((int32_t)(threadIdx.x >> 6));
  // The thread's index, read again wherever it is used: what comes from it,
  // kept across the walk, would cost FP32 registers that it has not got.
  const auto tid = [] {
    int t = threadIdx.x;
    if constexpr (sizeof(Tc) == 4) asm volatile("" : "+v"(t));
    return t;
  };
  const Tin* X = static_cast<const Tin*>(A.xyz);
  const int64_t big_total = uniform(*A.s.big_total);
  const int64_t n_big = uniform(A.s.counts[1]);
  const int64_t n_small = uniform(A.s.counts[0]);
  // small pairs a work index (FP32 teams run no refits)
  const int per = sizeof(Tc) == 4 ? 1 : A.batch < kTeam<Tc> ? A.batch : kTeam<Tc>;
  const int64_t total = big_total + (n_small + per - 1) / per;

  // work indices as in ds_persistent, one ahead, in the first thread
  int64_t w = blockIdx.x;
  int stop = 0;
  if (A.out.stop) {
    if (tid() == 0)
      next_stop = __hip_atomic_load(A.out.stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    stop = uniform(next_stop);
    __syncthreads();
  }
  while (w < total && !stop) {  // the same in every thread
    unsigned long long wn = 0ull;
    int sn = 0;
    if (tid() == 0) {
      wn = gridDim.x + atomicAdd(A.s.counter, 1ull);
      if (A.out.stop)
        sn = __hip_atomic_load(A.out.stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (w < big_total) {
      int64_t lo = 0, hi = n_big;
      while (hi - lo > 1) {
        const int64_t mid = (lo + hi) >> 1;
        if (uniform(A.s.big_prefix[mid]) <= w)
          lo = mid;
        else
          hi = mid;
      }
      const WorkRec r = uniform(A.s.big[lo]);
      const uint32_t fpre = r.items == 1 ? A.out.flags[r.p] : 0u;
      const int lane = tid() & 63;
      const int64_t local = w - uniform(A.s.big_prefix[lo]);
      const Layout L = layout<R>(r, local, A.chunk, lane);
      Frame<Tin, Tc> F;
      F.set(X, r.ob + L.b0);
      F.to_scalar();
      V3<Tc> kv[R + 1];
      load_b<Tin, Tc, R>(X, r, L, F, kv);
      Segs<Tc, R> sg;
      make_segs<Tc, R>(kv, sg);
      double acc = 0.0;  // the first wave's
      int per_lane = 0;  // FP64: a lane's steps at most
      if constexpr (sizeof(Tc) == 8) {
        const int n_slots = uniform((L.nbh + R - 1) / R);
        const int n_groups = n_slots <= kWave ? kWave / n_slots : 1;
        per_lane = (uniform(L.nah) + n_groups - 1) / n_groups;
      }
      for (int t0 = 0; t0 < L.nah; t0 += A.tile) {
        const int tl = (L.nah - t0) < A.tile ? (L.nah - t0) : A.tile;
        int steps = tl, U = U_max;
        if constexpr (sizeof(Tc) == 8) {
          if (per_lane < steps) steps = per_lane;
          const int share = ((steps + kTeam<Tc> - 1) / kTeam<Tc> + 3) & ~3;
          if (share < U) U = share;
        }
        for (int v = tid(); v <= tl; v += kWave * kTeam<Tc>) {
          unsigned idx = (unsigned)L.a0 + (unsigned)t0 + (unsigned)v;
          if (idx >= (unsigned)r.na) idx -= (unsigned)r.na;  // closing vertex of the loop
          const V3<Tc> x = F.load(X, r.oa + idx);
          lds[v] = Vtx<Tc>{x.x, x.y, x.z, (Tc)0};
        }
        __syncthreads();  // the tile is there, and the slots are read
        for (int u0 = 0; u0 * U < steps; u0 += kTeam<Tc>) {
          if (u0 > 0) __syncthreads();  // the slots are read
          const int ln = tid() & 63;
          const Layout M = layout<R>(r, local, A.chunk, ln);
          const int jlo = M.js > t0 ? M.js : t0;
          const int jhi = M.je < t0 + tl ? M.je : t0 + tl;
          const int n = M.active && jlo < jhi ? jhi - jlo : 0;  // the lane's steps in this tile
          const int b = (u0 + wv) * U;
          const int m = n - b < U ? n - b : U;
          if (m > 0) {
            const Vtx<Tc>* l = lds + (jlo - t0 + b);
            Tc* to = slots + (wv * E) * kWave + ln;
            walk<Tc, AT, R>(l, l + m, jlo + b == M.js, sg, [&](Tc sum) {
              *to = sum;
              to += kWave;
            });
          }
          __syncthreads();
          if (wv == 0) {
#pragma unroll 1
            for (int q = 0; q < kTeam<Tc>; ++q) {
              const int c = n - (u0 + q) * U < U ? n - (u0 + q) * U : U;
              const int k = c > 0 ? (c >> 2) + (c & 3) : 0;
              const Tc* from = slots + (q * E) * kWave + ln;
#pragma unroll 4
              for (int e = 0; e < k; ++e) acc += (double)from[e * kWave];
            }
          }
        }
      }
      if (wv == 0) finish_item<AT>(acc, r.p, lane, A, r.items == 1, fpre);
    } else if (wv < per && (w - big_total) * per + wv < n_small) {
      // a small pair on this wave (one wave: LDS accesses stay in order)
      const int lane = tid() & 63;
      Vtx<Tc>* const own = per == 1 ? lds : lds + wv * (kSmallA + 1);
      const WorkRec cur = uniform(A.s.small[(w - big_total) * per + wv]);
      const uint32_t fm = A.out.flags[cur.p];
      const Layout L = layout<R>(cur, 0, A.chunk, lane);
      Frame<Tin, Tc> F;
      F.set(X, cur.ob);
      F.to_scalar();
      V3<Tc> kv[R + 1];
      load_b<Tin, Tc, R>(X, cur, L, F, kv);
      const V3<Tc> a_lo = F.load(X, cur.oa + (lane < cur.na ? lane : 0));
      const V3<Tc> a_hi = F.load(X, cur.oa + (lane + kWave < cur.na ? lane + kWave : 0));
      if (lane <= cur.na) own[lane] = Vtx<Tc>{a_lo.x, a_lo.y, a_lo.z, (Tc)0};
      if (lane + kWave <= cur.na) own[lane + kWave] = Vtx<Tc>{a_hi.x, a_hi.y, a_hi.z, (Tc)0};
      Segs<Tc, R> sg;
      make_segs<Tc, R>(kv, sg);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      double acc = 0.0;
      if (L.active && L.js < L.je)
        walk_tile<Tc, AT, R>(own + L.js, own + L.je, true, sg, acc);
      finish_item<AT>(acc, cur.p, lane, A, true, fm);
    }
    if (tid() == 0) {
      next_w = wn;
      next_stop = sn;
    }
    __syncthreads();
    w = uniform((int64_t)next_w);
    stop = uniform(next_stop);
    __syncthreads();
  }
}

// Leaf pairs of the Barnes-Hut traversal (Alg. 6, both nodes leaves): Eq. 4
// over their kBhLeaf x kBhLeaf segment pairs with the walk above.  Like the
// packed small pairs of the direct sum, a wave takes four leaf pairs at a
// time, 16 lanes each: a lane holds 4 consecutive segments of the B leaf, the
// A leaf's vertices are in LDS (FP32 terms, FP64 sums).  A wave takes eight
// consecutive entries of the list at a time from sixteen queues (as
// ds_persistent: on a fixed stride the waves ended at very different times, at
// 73% of their seats) and adds one sum per run of entries of the same pair into
// its fixed-point accumulator.  ALU-bound: 11,000 vector instructions a wave and
// round at 2.5 cycles a SIMD.  840,000 leaf pairs (knit, 200 yarns) took 5,270 us
// with the walk of two waves a SIMD, 3,800 with its parts of four steps not
// unrolled, 3,320 on a fixed stride of 32 entries, 3,070 so.
template <typename Tin>
__global__ __launch_bounds__(kWave, 4) void bh_near_k(BhArgs A) {
  constexpr int K = 4, S = kWave / K, R = 4;  // S * R == kBhLeaf
  static_assert(S * R == kBhLeaf, "a segment of S lanes covers one leaf");
  __shared__ Vtx<float> lds[K][kBhLeaf + 2];  // the walk reads a vertex ahead
  const int lane = threadIdx.x, seg = lane / S, sl = lane - seg * S;
  const Tin* X = static_cast<const Tin*>(A.xyz);
  const int64_t cnt = A.counts[kBhMaxIters + 1];
  const int64_t n = cnt < A.near_cap ? cnt : A.near_cap;
  constexpr int kChunk = 8;
  const unsigned queue = blockIdx.x % kQueues;  // the grid is a multiple of kQueues
  int32_t* const my_counter = A.counts + kBhQueues + queue * kBhQueueStride;
  int64_t next = blockIdx.x;
  for (;;) {
    const int64_t c0 = uniform(next) * kChunk;  // lane 0's
    if (c0 >= n) break;
    if (lane == 0) next = gridDim.x + queue + (int64_t)kQueues * atomicAdd(my_counter, 1);
    const int64_t c1 = (c0 + kChunk) < n ? c0 + kChunk : n;
    double run = 0.0;  // uniform over the wave
    int32_t pr = -1;
    for (int64_t e0 = c0; e0 < c1; e0 += K) {
      const int64_t e = e0 + seg;
      const bool has = e < c1;
      const BhPair w = A.near[has ? e : e0];
      const int32_t i = A.pairs[2 * (int64_t)w.p], j = A.pairs[2 * (int64_t)w.p + 1];
      const int64_t oa = A.off[i], na = A.off[i + 1] - oa;
      const int64_t ob = A.off[j], nb = A.off[j + 1] - ob;
      const int64_t a0 = (int64_t)w.ka * kBhLeaf, b0 = (int64_t)w.kb * kBhLeaf;
      const int ma = (int)((na - a0) < kBhLeaf ? (na - a0) : kBhLeaf);
      const int mb = (int)((nb - b0) < kBhLeaf ? (nb - b0) : kBhLeaf);
      Frame<Tin, float> F;
      F.set(X, ob + b0);
      __syncthreads();
      for (int t = sl; t <= ma; t += S) {
        int64_t idx = a0 + t;
        if (idx >= na) idx -= na;  // closing vertex of the loop
        const V3<float> x = F.load(X, oa + idx);
        lds[seg][t] = Vtx<float>{x.x, x.y, x.z, 0.0f};
      }
      Segs<float, R> sg;
      {
        const int first = sl * R;
        V3<float> kv[R + 1];
#pragma unroll
        for (int r = 0; r <= R; ++r) {
          int64_t ib = b0 + (first + r < mb ? first + r : mb);  // vertex b0 + mb closes the leaf
          if (ib >= nb) ib -= nb;
          kv[r] = F.load(X, ob + ib);
        }
#pragma unroll
        for (int r = 0; r <= R; ++r) sg.k[r] = kv[r];
#pragma unroll
        for (int r = 0; r < R; ++r) {
          sg.s[r] = sg.k[r + 1] - sg.k[r];
          sg.m[r] = cross_r(sg.s[r], sg.k[r] - sg.k[0]);
        }
      }
      __syncthreads();
      double acc = 0.0;
      if (has)
        walk<float, 2, R, true>(lds[seg], lds[seg] + ma, true, sg,
                                [&](float sum) { acc += (double)sum; });
#pragma unroll
      for (int o = S / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
      // the K entries in order: extend the run or flush it (uniform logic)
#pragma unroll
      for (int q = 0; q < K; ++q) {
        if (e0 + q >= c1) break;
        const int32_t pq = __shfl(w.p, q * S);
        const double vq = __shfl(acc, q * S);
        if (pq != pr) {
          if (pr >= 0 && lane == 0) {
            const double v = run * kInvTwoPi;
            if (fabs(v) < 1.0e14)
              fixed_add(&A.acc[2 * (int64_t)pr], v);
            else
              atomicOr(&A.out.flags[pr], kFlagNonfinite);
          }
          pr = pq;
          run = 0.0;
        }
        run += vq;
      }
    }
    if (pr >= 0 && lane == 0) {
      const double v = run * kInvTwoPi;
      if (fabs(v) < 1.0e14)
        fixed_add(&A.acc[2 * (int64_t)pr], v);
      else
        atomicOr(&A.out.flags[pr], kFlagNonfinite);
    }
  }
}

// A tile plus its closing vertex, or R small pairs' loops A side by side.
template <typename Tc, int R>
size_t lds_bytes(int tile) {
  const int n = tile + 1 > R * kSmallA ? tile + 1 : R * kSmallA;
  return (size_t)(n + 1) * sizeof(Vtx<Tc>);
}

template <typename Tin, typename Tc, int AT, int R>
hipError_t launch_t(const DsArgs& a, int grid, hipStream_t s) {
  ds_persistent<Tin, Tc, AT, R><<<dim3(grid), dim3(kWave), lds_bytes<Tc, R>(a.tile), s>>>(a);
  return hipGetLastError();
}

// Workgroups of a kernel that are resident at once, at most `waves_per_cu` waves
// per compute unit (0: no limit), on average over the units where a workgroup has
// more of them.
int resident(hipError_t e, int per_cu, int waves, int n_cu, int waves_per_cu) {
  if (e != hipSuccess || per_cu < 1) per_cu = 1;
  if (waves_per_cu > 0 && waves_per_cu < per_cu * waves) {
    const int g = (int)((int64_t)waves_per_cu * n_cu / waves);
    return g > 0 ? g : 1;
  }
  return per_cu * n_cu;
}

template <typename Tin, typename Tc, int AT, int R>
int grid_t(int tile, int n_cu, int waves_per_cu) {
  int per_cu = 0;
  const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
      &per_cu, ds_persistent<Tin, Tc, AT, R>, kWave, lds_bytes<Tc, R>(tile));
  return resident(e, per_cu, 1, n_cu, waves_per_cu);
}

// The team kernel's tile and the waves' slots, or small pairs' loops A.
template <typename Tc>
size_t team_lds(int tile) {
  const int n = tile + 2 > kSmallA + 1 ? tile + 2 : kSmallA + 1;
  const size_t big =
      (size_t)n * sizeof(Vtx<Tc>) + (size_t)kTeam<Tc> * team_slots<Tc>(tile) * kWave * sizeof(Tc);
  const size_t small = (size_t)kTeam<Tc> * (kSmallA + 1) * sizeof(Vtx<Tc>);
  return big > small ? big : small;
}
template <typename Tin, typename Tc, int R>
hipError_t launch_team(const DsArgs& a, int grid, hipStream_t s) {
  ds_team<Tin, Tc, R><<<dim3(grid), dim3(kWave * kTeam<Tc>), team_lds<Tc>(a.tile), s>>>(a);
  return hipGetLastError();
}
template <typename Tin, typename Tc, int R>
int grid_team(int tile, int n_cu, int waves_per_cu) {
  int per_cu = 0;
  const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
      &per_cu, ds_team<Tin, Tc, R>, kWave * kTeam<Tc>, team_lds<Tc>(tile));
  return resident(e, per_cu, kTeam<Tc>, n_cu, waves_per_cu);
}

// Kernel variants: input type x arithmetic x arctangent form x segments per lane.
struct Variant {
  hipError_t (*launch)(const DsArgs&, int, hipStream_t);
  int (*grid)(int, int, int);
  int waves;  // per workgroup
};

template <typename Tin, typename Tc, int AT, int R>
constexpr Variant variant() {
  return Variant{launch_t<Tin, Tc, AT, R>, grid_t<Tin, Tc, AT, R>, 1};
}
template <typename Tin, typename Tc, int R>
constexpr Variant team() {
  return Variant{launch_team<Tin, Tc, R>, grid_team<Tin, Tc, R>, kTeam<Tc>};
}

// The team kernel, for calls with few pairs: the direct-sum forms with the own
// arctangent and R > 1 only.
bool pick_team(bool in_f64, bool compute_f64, int atan_form, int segs, Variant* v) {
  if (atan_form == kCrossings || segs < 2) return false;
  if (compute_f64) {
    *v = in_f64 ? team<double, double, 2>() : team<float, double, 2>();
    return true;
  }
  if (atan_form == 1) return false;
  if (segs >= 4)
    *v = in_f64 ? team<double, float, 4>() : team<float, float, 4>();
  else
    *v = in_f64 ? team<double, float, 2>() : team<float, float, 2>();
  return true;
}

// With one segment per lane an FP32 pass of few pairs is bound by the latency of its
// steps, which the tests for small angles lengthen: 56 pairs of 100-2,048 segments
// take 184 us with them, 176 without, 512 of 100 75 and 70 (23,441 pairs of 64
// segments 197 and 265).
Variant pick(bool in_f64, bool compute_f64, int atan_form, int segs, bool unpacked = false) {
  Variant u;
  if (unpacked && pick_team(in_f64, compute_f64, atan_form, segs, &u)) return u;
  if (unpacked && !compute_f64 && segs < 2 && (atan_form == 0 || atan_form == 2))
    return in_f64 ? variant<double, float, kFullForm, 1>() : variant<float, float, kFullForm, 1>();
  if (compute_f64 && atan_form == kCrossings) {
    constexpr int C = kCrossings;
    if (segs >= 2) return in_f64 ? variant<double, double, C, 2>() : variant<float, double, C, 2>();
    return in_f64 ? variant<double, double, C, 1>() : variant<float, double, C, 1>();
  }
  if (compute_f64) {
    if (segs >= 2) return in_f64 ? variant<double, double, 0, 2>() : variant<float, double, 0, 2>();
    return in_f64 ? variant<double, double, 0, 1>() : variant<float, double, 0, 1>();
  }
  if (atan_form == 1) {
    if (segs >= 4) return in_f64 ? variant<double, float, 1, 4>() : variant<float, float, 1, 4>();
    if (segs >= 2) return in_f64 ? variant<double, float, 1, 2>() : variant<float, float, 1, 2>();
    return in_f64 ? variant<double, float, 1, 1>() : variant<float, float, 1, 1>();
  }
  if (atan_form == kCrossings) {
    constexpr int C = kCrossings;
    if (segs >= 8) return in_f64 ? variant<double, float, C, 8>() : variant<float, float, C, 8>();
    if (segs >= 4) return in_f64 ? variant<double, float, C, 4>() : variant<float, float, C, 4>();
    if (segs >= 2) return in_f64 ? variant<double, float, C, 2>() : variant<float, float, C, 2>();
    return in_f64 ? variant<double, float, C, 1>() : variant<float, float, C, 1>();
  }
  // forms 0 and 2 give the same values and run the same kernel
  if (segs >= 4) return in_f64 ? variant<double, float, 2, 4>() : variant<float, float, 2, 4>();
  if (segs >= 2) return in_f64 ? variant<double, float, 2, 2>() : variant<float, float, 2, 2>();
  return in_f64 ? variant<double, float, 2, 1>() : variant<float, float, 2, 1>();
}

}  // namespace

int segs_supported(bool compute_f64, int segs, bool crossings) {
  if (compute_f64) return segs >= 2 ? 2 : 1;
  if (crossings && segs >= 8) return 8;
  return segs >= 4 ? 4 : (segs >= 2 ? 2 : 1);
}

hipError_t launch_bh_near(const BhArgs& a, bool in_f64, hipStream_t s) {
  if (in_f64)
    bh_near_k<double><<<4096, kWave, 0, s>>>(a);
  else
    bh_near_k<float><<<4096, kWave, 0, s>>>(a);
  return hipGetLastError();
}

hipError_t launch_direct_sum(const DsArgs& a, bool in_f64, bool compute_f64, int atan_form,
                             int segs, int grid, hipStream_t s, bool unpacked) {
  return pick(in_f64, compute_f64, atan_form, segs, unpacked).launch(a, grid, s);
}

int direct_sum_grid(bool in_f64, bool compute_f64, int atan_form, int segs, int tile, int n_cu,
                    int waves_per_cu, bool unpacked) {
  return pick(in_f64, compute_f64, atan_form, segs, unpacked).grid(tile, n_cu, waves_per_cu);
}

int direct_sum_waves(bool in_f64, bool compute_f64, int atan_form, int segs, bool unpacked) {
  return pick(in_f64, compute_f64, atan_form, segs, unpacked).waves;
}

}  // namespace lk
