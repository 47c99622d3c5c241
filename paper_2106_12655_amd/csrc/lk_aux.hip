// lk_aux.hip -- everything around the direct-sum hot loop: input validation,
// work planning with its device-side schedule, the potential link search
// (Alg. 2) and the verification merge (Sec. 3.1, "Fast Verification").
//
// All sizes that depend on the data (work item totals, the refit count) stay in
// device memory, so every launch here has a host-known shape and the whole
// sequence can be captured in a HIP graph.  No kernel uses float atomics: all
// reductions have a fixed order, and results are bitwise reproducible.
#include <float.h>
#include <math.h>

#include <type_traits>

#include "lk_internal.h"

namespace lk {
namespace {

inline int blocks_for(int64_t n, int threads, int cap = 65535 * 8) {
  int64_t b = (n + threads - 1) / threads;
  if (b < 1) b = 1;
  if (b > cap) b = cap;
  return (int)b;
}

// ------------------------------------------------------------- validation
// Sum of one value per thread of a 256-thread workgroup (a fixed-order tree),
// stored at part[blockIdx.x].
__device__ __forceinline__ void block_sum_to(double v, double* red, double* part) {
  red[threadIdx.x] = v;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// One wavefront per loop: the per-loop bits that do not depend on xi (fewer
// than 3 vertices, non-finite coordinates), each loop's shortest squared
// segment, and one xi partial sum of |coordinate| per workgroup over the
// vertices of its loops.  The zero-length test of Alg. 3 (segment shorter
// than eps * xi) is applied by the plan, which reduces the partials to xi
// itself.  When the crossing count's box kernel does the per-loop scan, this
// kernel sums xi over a flat grid stride and only initialises the per-loop
// entries.  Block 0 also zeroes the main pass's schedule counts.
// One wavefront's scan of loop l: its flags that do not depend on xi (fewer
// than 3 vertices, non-finite coordinates) and its shortest squared segment,
// written by lane 0; returns the lane's sum of |x| + |y| + |z| over the
// vertices it read.
// W: lanes per loop (a power of two up to 64, aligned within the wavefront;
// every lane of the group calls it).
template <typename Tin, int W = 64>
__device__ double scan_loop(const Tin* X, const int64_t* off, int64_t l, int lane, uint32_t* lf,
                            double* minseg2) {
  double s = 0.0;
  const int64_t o = off[l], n = off[l + 1] - o;
  uint32_t f = (n < 3) ? kFlagBadloop : 0u;
  double mn = INFINITY;
  for (int64_t q = lane; q < n; q += W) {
    const int64_t t = (q + 1 == n) ? 0 : q + 1;
    const double x0 = (double)X[3 * (o + q)], y0 = (double)X[3 * (o + q) + 1],
                 z0 = (double)X[3 * (o + q) + 2];
    const double x1 = (double)X[3 * (o + t)], y1 = (double)X[3 * (o + t) + 1],
                 z1 = (double)X[3 * (o + t) + 2];
    if (!isfinite(x0) || !isfinite(y0) || !isfinite(z0)) f |= kFlagNonfinite | kFlagBadloop;
    s += fabs(x0) + fabs(y0) + fabs(z0);
    const double dx = x1 - x0, dy = y1 - y0, dz = z1 - z0;
    mn = fmin(mn, dx * dx + dy * dy + dz * dz);
  }
  for (int o2 = W / 2; o2 > 0; o2 >>= 1) {
    f |= (uint32_t)__shfl_xor((int)f, o2);
    mn = fmin(mn, __shfl_xor(mn, o2));
  }
  if (lane == 0) {
    lf[l] = f;
    minseg2[l] = mn;
  }
  return s;
}

template <typename Tin>
__global__ __launch_bounds__(256) void prep_k(const Tin* X, const int64_t* off, int32_t L,
                                              double* part, uint32_t* lf, double* minseg2,
                                              int32_t* zero_counts,
                                              unsigned long long* zero_mismatch,
                                              int32_t* zero_stop, int scan_loops) {
  __shared__ double red[256];
  if (blockIdx.x == 0 && threadIdx.x < 2) zero_counts[threadIdx.x] = 0;
  if (blockIdx.x == 0 && threadIdx.x == 0 && zero_mismatch) {
    *zero_mismatch = 0ull;
    *zero_stop = 0;
  }
  double s = 0.0;
  if (!scan_loops) {
    const int64_t v0 = off[0], v1 = off[L];
    const int64_t n3 = 3 * (v1 - v0);
    for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < n3;
         k += (int64_t)gridDim.x * 256)
      s += fabs((double)X[3 * v0 + k]);
    block_sum_to(s, red, part);
    // the crossing count's box kernel scans the vertices (in parallel over
    // blocks of long loops) and folds its results into these with atomics
    for (int64_t l = (int64_t)blockIdx.x * 256 + threadIdx.x; l < L; l += (int64_t)gridDim.x * 256) {
      lf[l] = off[l + 1] - off[l] < 3 ? kFlagBadloop : 0u;
      minseg2[l] = INFINITY;
    }
    return;
  }
  // one pass over the loops: each vertex adds |x| + |y| + |z| to the xi
  // partial of the workgroup that scans its loop
  const int lane = threadIdx.x & 63;
  const int64_t wave = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 6;
  const int64_t nwaves = ((int64_t)gridDim.x * 256) >> 6;
  for (int64_t l = wave; l < L; l += nwaves) s += scan_loop(X, off, l, lane, lf, minseg2);
  block_sum_to(s, red, part);
}

// ------------------------------------------------- crossing-count boxes
// One wavefront per superblock slot: the loop that owns the slot comes from a
// binary search over the slot bases, and the wave boxes the superblock's
// blocks one after another (lane t holds vertex 64k + t; lane 0 also the
// vertex that closes the block).  Coordinates are FP32 on the vertices as the
// crossing kernel sees them (FP64 input rounded first).  Each box is widened
// by 8 u (u = 2^-24) times the largest |x|_1 of its vertices, which covers the
// rounding of the two projections and the FP32 directions' deviation from
// exact orthogonality to the view direction.  The slot count comes from the
// device offsets, so every vertex is scanned whatever the buffers hold; boxes
// beyond the buffers are not written.
//
// The same scan does the per-loop validation of the preparation kernel (which
// then only initialises it): non-finite coordinates and the shortest squared
// segment, folded into the loop's entries with atomics (a minimum of
// non-negative doubles is a minimum of their bit patterns).
__device__ __forceinline__ float4 box_join(const float4& a, const float4& b) {
  return float4{fminf(a.x, b.x), fmaxf(a.y, b.y), fminf(a.z, b.z), fmaxf(a.w, b.w)};
}

template <typename Tin>
__global__ __launch_bounds__(256) void cc_boxes_k(const Tin* X, const int64_t* off, int32_t L,
                                                  CcProj pr, float4* blk, int64_t n_blk,
                                                  float4* sup, int64_t n_sup, uint32_t* lf,
                                                  double* minseg2) {
  const int lane = threadIdx.x & 63;
  const int64_t o0 = off[0];
  const int64_t n_slots = (off[L] - o0) / kCcSuper + L + 1;
  const int64_t wave = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 6;
  const int64_t nwaves = ((int64_t)gridDim.x * 256) >> 6;
  for (int64_t slot = wave; slot < n_slots; slot += nwaves) {
    // largest loop i with (off[i] - off[0]) / kCcSuper + i <= slot
    int32_t lo = 0, hi = L;
    while (hi - lo > 1) {
      const int32_t mid = (lo + hi) >> 1;
      if ((off[mid] - o0) / kCcSuper + mid <= slot)
        lo = mid;
      else
        hi = mid;
    }
    const int64_t oi = off[lo], n = off[lo + 1] - oi;
    const int64_t s = slot - ((oi - o0) / kCcSuper + lo);
    const int64_t nblk = n > 0 ? (n + kCcBlock - 1) / kCcBlock : 0;
    constexpr int64_t kPer = kCcSuper / kCcBlock;
    // slot not used by the loop, or offsets that decrease (uniform over the wave)
    if (n <= 0 || s < 0 || s * kPer >= nblk) continue;
    const int64_t bbase = (oi - o0) / kCcBlock + lo;
    float4 acc = float4{INFINITY, -INFINITY, INFINITY, -INFINITY};
    uint32_t f = 0u;
    double mn = INFINITY;
    const int64_t kend = (s + 1) * kPer < nblk ? (s + 1) * kPer : nblk;
    for (int64_t k = s * kPer; k < kend; ++k) {
      const int64_t v0 = k * kCcBlock;
      const int64_t m = (n - v0) < kCcBlock ? (n - v0) : kCcBlock;
      float a0 = INFINITY, a1 = -INFINITY, b0 = INFINITY, b1 = -INFINITY, mag = 0.0f;
      for (int t = lane; t <= m; t += 64) {  // m + 1 vertices: the last closes the block
        int64_t v = v0 + t;
        if (v >= n) v -= n;
        const Tin* p = X + 3 * (oi + v);
        const double x = (double)p[0], y = (double)p[1], z = (double)p[2];
        if (t < m) {
          // the loop's validation: vertex v and its segment to v + 1
          int64_t w = v + 1;
          if (w >= n) w -= n;
          const Tin* q = X + 3 * (oi + w);
          if (!isfinite(x) || !isfinite(y) || !isfinite(z)) f |= kFlagNonfinite | kFlagBadloop;
          const double dx = (double)q[0] - x, dy = (double)q[1] - y, dz = (double)q[2] - z;
          mn = fmin(mn, dx * dx + dy * dy + dz * dz);
        }
        const float xf = (float)x, yf = (float)y, zf = (float)z;
        const float a = fmaf(xf, pr.e1[0], fmaf(yf, pr.e1[1], zf * pr.e1[2]));
        const float b = fmaf(xf, pr.e2[0], fmaf(yf, pr.e2[1], zf * pr.e2[2]));
        a0 = fminf(a0, a);
        a1 = fmaxf(a1, a);
        b0 = fminf(b0, b);
        b1 = fmaxf(b1, b);
        mag = fmaxf(mag, fabsf(xf) + fabsf(yf) + fabsf(zf));
      }
      for (int o = 32; o > 0; o >>= 1) {
        a0 = fminf(a0, __shfl_xor(a0, o));
        a1 = fmaxf(a1, __shfl_xor(a1, o));
        b0 = fminf(b0, __shfl_xor(b0, o));
        b1 = fmaxf(b1, __shfl_xor(b1, o));
        mag = fmaxf(mag, __shfl_xor(mag, o));
      }
      const float pad = 4.76837158203125e-7f * mag;  // 8 * 2^-24
      const float4 box = float4{a0 - pad, a1 + pad, b0 - pad, b1 + pad};
      if (lane == 0 && (uint64_t)(bbase + k) < (uint64_t)n_blk) blk[bbase + k] = box;
      acc = box_join(acc, box);
    }
    for (int o = 32; o > 0; o >>= 1) {
      f |= (uint32_t)__shfl_xor((int)f, o);
      mn = fmin(mn, __shfl_xor(mn, o));
    }
    if (lane == 0) {
      if (slot < n_sup) sup[slot] = acc;
      if (f) atomicOr(&lf[lo], f);
      // the entry only decreases, so a plain read that is not above mn
      // makes the atomic unnecessary (thousands of blocks share one loop)
      if (mn < INFINITY && mn < minseg2[lo])
        atomicMin(reinterpret_cast<unsigned long long*>(&minseg2[lo]),
                  (unsigned long long)__double_as_longlong(mn));
    }
  }
}

// --------------------------------------------------------------- planning
// Workgroup-collective append to two lists at once: one atomic per list per
// workgroup (instead of one per wavefront), so the plan of tens of thousands
// of pairs does not queue thousands of atomics on two counters.  Every
// thread of the workgroup must call it; *pos0 / *pos1 receive the thread's
// slot in list 0 / 1 when it appends there.
__device__ __forceinline__ void block_append2(int32_t* count0, bool pred0, int32_t* pos0,
                                              int32_t* count1, bool pred1, int32_t* pos1) {
  __shared__ int32_t wn[2][16], base[2];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const unsigned long long m0 = __ballot(pred0), m1 = __ballot(pred1);
  if (lane == 0) {
    wn[0][w] = (int32_t)__popcll(m0);
    wn[1][w] = (int32_t)__popcll(m1);
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    const int k = threadIdx.x;
    int32_t t = 0;
    for (int q = 0; q < nw; ++q) t += wn[k][q];
    base[k] = t ? atomicAdd(k ? count1 : count0, t) : 0;
  }
  __syncthreads();
  int32_t b0 = base[0], b1 = base[1];
  for (int q = 0; q < w; ++q) {
    b0 += wn[0][q];
    b1 += wn[1][q];
  }
  const unsigned long long below = lane ? (~0ull >> (64 - lane)) : 0ull;
  *pos0 = b0 + (int32_t)__popcll(m0 & below);
  *pos1 = b1 + (int32_t)__popcll(m1 & below);
  __syncthreads();  // wn and base are reused by the next call
}

// Exclusive scan of one value per thread over a 1024-thread workgroup
// (wavefront shuffles, then the 16 wave totals).  *total receives the sum.
__device__ int64_t block_excl_scan(int64_t v, int64_t* wsum, int64_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int64_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int64_t y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  if (lane == 63) wsum[wave] = x;
  __syncthreads();
  if (wave == 0) {
    int64_t sw = lane < 16 ? wsum[lane] : 0;
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
      const int64_t y = __shfl_up(sw, o);
      if (lane >= o) sw += y;
    }
    if (lane < 16) wsum[lane] = sw;
  }
  __syncthreads();
  const int64_t before = wave ? wsum[wave - 1] : 0;
  *total = wsum[15];
  __syncthreads();
  return before + x - v;
}

// In-place-capable exclusive scan of src[0..n) into dst[0..n], dst[n] = total;
// 4 consecutive elements per thread per round, so loads are coalesced.
__device__ int64_t block_scan_array(const int64_t* src, int64_t n, int64_t* dst, int64_t* wsum) {
  const int t = threadIdx.x;
  int64_t carry = 0;
  for (int64_t base = 0; base < n; base += 4096) {
    const int64_t k0 = base + 4 * (int64_t)t;
    int64_t v[4];
    int64_t sum = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[i] = (k0 + i < n) ? src[k0 + i] : 0;
      sum += v[i];
    }
    int64_t tot = 0;
    int64_t run = carry + block_excl_scan(sum, wsum, &tot);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (k0 + i < n) dst[k0 + i] = run;
      run += v[i];
    }
    carry += tot;
  }
  if (t == 0) dst[n] = carry;
  return carry;
}

__device__ __forceinline__ int cost_bucket(int32_t items) { return 31 - __clz(items); }

// One workgroup (1024 threads): bucket the big pairs by log2(items), largest
// bucket first (an LPT order up to a factor of two), then scan their items.
__device__ void schedule(const Sched& S, int32_t* zero_next) {
  __shared__ int hist[32];
  __shared__ int cur[32];
  __shared__ int64_t wsum[16];
  const int t = threadIdx.x;
  // a device-scope load: in the fused launch below the count was built by
  // atomics of the same kernel
  const int nb = __hip_atomic_load(&S.counts[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (t < 32) hist[t] = 0;
  __syncthreads();
  for (int k = t; k < nb; k += 1024) atomicAdd(&hist[cost_bucket(S.big_in[k].items)], 1);
  __syncthreads();
  if (t == 0) {
    int run = 0;
    for (int b = 31; b >= 0; --b) {
      cur[b] = run;
      run += hist[b];
    }
  }
  __syncthreads();
  for (int k = t; k < nb; k += 1024) {
    const WorkRec r = S.big_in[k];
    const int pos = atomicAdd(&cur[cost_bucket(r.items)], 1);
    S.big[pos] = r;
    S.big_prefix[pos] = r.items;
  }
  __syncthreads();
  const int64_t total = block_scan_array(S.big_prefix, nb, S.big_prefix, wsum);
  if (t < kQueues) S.counter[t * kQueueStride] = 0ull;
  if (t == 0) {
    *S.big_total = total;
    if (zero_next) {
      zero_next[0] = 0;
      zero_next[1] = 0;
      zero_next[2] = 0;
    }
  }
}

// The plan's work over list positions base = first, first + stride, ...
// below n, one thread per position (every thread of the workgroup takes part:
// the appends are workgroup-collective, so n and the loop bounds must be the
// same in every thread).
__device__ void plan_positions(const PlanArgs& A, int32_t L, const LoopInfo& li, const Sched& S,
                               int refit, double xi, int64_t n, int64_t first, int64_t stride) {
  for (int64_t base = first; base < n; base += stride) {
    const int64_t q = base + threadIdx.x;
    bool small = false, big = false;
    WorkRec r{};
    if (q < n) {
      const int32_t p = A.list ? A.list[q] : (int32_t)q;
      const int32_t i = A.pairs[2 * p], j = A.pairs[2 * p + 1];
      const bool valid = i >= 0 && j >= 0 && i < L && j < L && i != j;
      int64_t items = 0;
      if (valid) {
        r.oa = A.off[i];
        r.ob = A.off[j];
        const int64_t na = A.off[i + 1] - r.oa, nb = A.off[j + 1] - r.ob;
        r.na = (int32_t)na;
        r.nb = (int32_t)nb;
        if (na >= 1 && nb >= 1)
          items = ((nb + A.bblock - 1) / A.bblock) * ((na + A.chunk - 1) / A.chunk);
      }
      // loops beyond 2^31 vertices or pairs beyond 2^31 work items are not handled
      const bool too_big = valid && (A.off[i + 1] - A.off[i] > 0x7fffffffLL ||
                                     A.off[j + 1] - A.off[j] > 0x7fffffffLL ||
                                     items > 0x7fffffffLL);
      if (too_big) items = 0;
      // crossing count: two loops of one superblock each whose projected
      // boxes are disjoint have no crossing, so the pair is 0 without work
      if (A.cc_sup && valid && !too_big && items > 0 && r.na <= kCcSuper && r.nb <= kCcSuper) {
        const int64_t o0 = A.off[0];
        const int64_t si = (r.oa - o0) / kCcSuper + i, sj = (r.ob - o0) / kCcSuper + j;
        if ((uint64_t)si < (uint64_t)A.cc_nsup && (uint64_t)sj < (uint64_t)A.cc_nsup &&
            boxes_disjoint(A.cc_sup[si], A.cc_sup[sj]))
          items = 0;
      }
      uint32_t f;
      if (refit) {
        // a non-finite value of the previous pass may become finite in FP64;
        // non-finite coordinates stay non-finite
        const uint32_t coords = valid ? (li.lf[i] | li.lf[j]) & kFlagNonfinite : 0u;
        f = (A.out.flags[p] & ~kFlagNonfinite) | coords | (too_big ? kFlagNonfinite : 0u);
      } else if (valid) {
        // Alg. 3's zero-length test: a segment shorter than eps * xi
        const double lim = li.eps * xi;
        const double lim2 = lim * lim;
        const uint32_t fi = li.lf[i] | (li.minseg2[i] < lim2 ? kFlagBadloop : 0u);
        const uint32_t fj = li.lf[j] | (li.minseg2[j] < lim2 ? kFlagBadloop : 0u);
        f = fi | fj | (too_big ? kFlagBadloop | kFlagNonfinite : 0u);
      } else {
        f = kFlagBadpair;
      }
      A.acc[2 * (int64_t)p] = 0ull;
      A.acc[2 * (int64_t)p + 1] = 0ull;
      r.p = p;
      r.items = (int32_t)items;
      small = items == 1 && r.na < kSmallA;
      big = items > 0 && !small;
      if (!valid) {
        A.out.flags[p] = f;
        A.out.lk_real[p] = __builtin_nan("");
        A.out.lk_int[p] = kIntInvalid;
        check_pair(A.out, p, kIntInvalid, f);
      } else if (items == 0) {
        // nothing to sum (an empty loop, or beyond the supported sizes)
        Outs o = A.out;
        o.refit_list = nullptr;
        finalize_pair(o, p, 0.0, f);
      } else {
        if (A.out.expected && !refit) {
          // a fused check marks every pair SKIPPED until it is finalised
          f |= kFlagSkipped;
          A.out.lk_real[p] = __builtin_nan("");
          A.out.lk_int[p] = kIntInvalid;
        }
        A.out.flags[p] = f;
      }
    }
    int32_t ps, pb;
    block_append2(&S.counts[0], small, &ps, &S.counts[1], big, &pb);
    if (small) S.small[ps] = r;
    if (big) S.big_in[pb] = r;
  }
}

// One thread per list position, 1024-thread workgroups.  The schedule is a
// separate single-workgroup launch: handing it to the plan's last workgroup
// (a fence and a ticket in every workgroup) measured slower on MI355X, where
// a device-scope fence writes back the XCD's L2.
__global__ __launch_bounds__(1024) void plan_k(PlanArgs A, int32_t L, LoopInfo li, Sched S,
                                               int refit) {
  // xi = mean |coordinate|: every block reduces the preparation kernel's
  // partials in the same fixed order (cheaper than another launch); a refit
  // pass validates nothing and skips it
  __shared__ double red[1024];
  double xi = 0.0;
  if (!refit) {
    double part = 0.0;
    for (int k = threadIdx.x; k < li.n_part; k += 1024) part += li.part[k];
    red[threadIdx.x] = part;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
      if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
      __syncthreads();
    }
    const int64_t nv = A.off[L] - A.off[0];
    xi = nv > 0 ? red[0] / (3.0 * (double)nv) : 0.0;
  }
  int64_t n = A.n_list;
  if (A.n_list_dev) {
    const int64_t nd = __hip_atomic_load(A.n_list_dev, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    n = nd < n ? nd : n;
  }
  // grid stride over the list's length on the device (the same in every
  // thread), so an empty refit list costs each workgroup one load
  plan_positions(A, L, li, S, refit, xi, n, (int64_t)blockIdx.x * 1024, (int64_t)gridDim.x * 1024);
}

// Finalises the big-list pairs that were split over several work items,
// positions first, first + stride, ...
__device__ void finalize_split_range(const Sched& S, const unsigned long long* acc, const Outs& o,
                                     int32_t first, int32_t stride) {
  if (o.stop && *o.stop) return;  // a fused check stopped early: sums may be partial
  const int32_t nb = S.counts[1];
  for (int32_t k = first; k < nb; k += stride) {
    const WorkRec r = S.big[k];
    if (r.items < 2) continue;  // single-item pairs were finalised by their wave
    const int32_t p = r.p;
    finalize_pair(o, p, from_fixed(acc[2 * (int64_t)p], acc[2 * (int64_t)p + 1]), o.flags[p]);
  }
}

__global__ __launch_bounds__(256) void finalize_split_k(Sched S, const unsigned long long* acc,
                                                        Outs o) {
  finalize_split_range(S, acc, o, blockIdx.x * 256 + threadIdx.x, gridDim.x * 256);
}

// The end of one pass and the start of the next in one launch of a single
// workgroup: the pass's split pairs are finalised (queuing their refits), then
// the refit list is planned and scheduled.  Every write that a later step
// reads comes from the same workgroup, so barriers order the three steps and
// no grid-wide synchronisation is needed.  This saves two kernel boundaries
// per call (each a few microseconds on MI355X); the steps are short (a refit
// list is usually empty, and the split pairs number a few thousand at most).
__global__ __launch_bounds__(1024) void finalize_replan_k(Sched S, const unsigned long long* acc,
                                                          Outs o, PlanArgs R, int32_t L,
                                                          LoopInfo li, Sched SR,
                                                          int32_t* zero_next) {
  finalize_split_range(S, acc, o, threadIdx.x, 1024);
  __syncthreads();
  int64_t n = R.n_list;
  const int64_t nd = __hip_atomic_load(R.n_list_dev, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  n = nd < n ? nd : n;
  plan_positions(R, L, li, SR, 1, 0.0, n, 0, 1024);
  __syncthreads();
  schedule(SR, zero_next);
}

__global__ __launch_bounds__(1024) void sched_k(Sched S, int32_t* zero_next) {
  schedule(S, zero_next);
}

// Single-workgroup exclusive scan (tiles of the pair search, verification).
__global__ __launch_bounds__(1024) void scan_k(const int64_t* counts, int64_t n, int64_t* prefix,
                                               int64_t* host_total) {
  __shared__ int64_t wsum[16];
  const int64_t total = block_scan_array(counts, n, prefix, wsum);
  if (threadIdx.x == 0)
    __hip_atomic_store(host_total, total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ------------------------------------------------------ potential link search
// Boxes: W lanes per loop (a power of two up to 64), or a workgroup per loop
// for few loops, which may be long (below).  Minima and maxima are exact, so
// they are taken in the input type.  The tiles' pair counts start at 0 here.
template <typename Tin>
struct MinMax {
  Tin lo[3], hi[3];
  __device__ __forceinline__ void clear() {
    for (int q = 0; q < 3; ++q) {
      lo[q] = (Tin)INFINITY;
      hi[q] = (Tin)-INFINITY;
    }
  }
  __device__ __forceinline__ void add(const Tin* p) {
    for (int q = 0; q < 3; ++q) {
      lo[q] = fmin(lo[q], p[q]);
      hi[q] = fmax(hi[q], p[q]);
    }
  }
  template <int W>
  __device__ __forceinline__ void reduce() {
    for (int o = W / 2; o > 0; o >>= 1)
      for (int q = 0; q < 3; ++q) {
        lo[q] = fmin(lo[q], __shfl_xor(lo[q], o));
        hi[q] = fmax(hi[q], __shfl_xor(hi[q], o));
      }
  }
  __device__ __forceinline__ void store(double* b) const {
    for (int q = 0; q < 3; ++q) {
      b[q] = (double)lo[q];
      b[3 + q] = (double)hi[q];
    }
  }
};

__device__ __forceinline__ void clear_tiles(unsigned long long* tiles, int32_t L) {
  const int32_t n = (L + kRowTile - 1) / kRowTile;
  for (int32_t k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += gridDim.x * blockDim.x)
    tiles[k] = 0ull;
}

// A loop of more than kBoxNarrow vertices is left by its 16 lanes to the whole wave:
// 10,000 loops of 32 vertices and one of a million took 15,100 us by 16 lanes,
// 3,940 so (4,320 with a wave for every loop).  Loops of some hundred vertices are
// better side by side: 10,000 of 2,000 take 112 us a search, by waves in turn 116.
constexpr int64_t kBoxNarrow = 2048;
template <typename Tin, int W>
__global__ __launch_bounds__(256) void boxes_k(const Tin* X, const int64_t* off, int32_t L,
                                               double* box, unsigned long long* tiles) {
  clear_tiles(tiles, L);
  const int sub = threadIdx.x & (W - 1);
  const int64_t first = ((int64_t)blockIdx.x * 256 + threadIdx.x) / W;
  const int64_t stride = (int64_t)gridDim.x * 256 / W;
  // the same trip count in every lane (the reduction is wavefront-collective)
  const int64_t trips = (L + stride - 1) / stride;
  for (int64_t t = 0; t < trips; ++t) {
    const int64_t l = first + t * stride;
    MinMax<Tin> m;
    m.clear();
    const int64_t v0 = l < L ? off[l] : 0, v1 = l < L ? off[l + 1] : 0;
    const bool wide = W < 64 && v1 - v0 > kBoxNarrow;
    if (!wide)
      for (int64_t v = v0 + sub; v < v1; v += W) m.add(X + 3 * v);
    m.template reduce<W>();
    if (l < L && sub == 0 && !wide) m.store(box + 6 * l);
    if constexpr (W < 64) {
      for (unsigned long long left = __ballot(wide && sub == 0); left; left &= left - 1ull) {
        const int from = __ffsll((long long)left) - 1;  // the loop's first lane
        const int64_t a = __shfl(v0, from), b = __shfl(v1, from), to = __shfl(l, from);
        MinMax<Tin> all;
        all.clear();
        for (int64_t v = a + (int)(threadIdx.x & 63); v < b; v += 64) all.add(X + 3 * v);
        all.template reduce<64>();
        if ((threadIdx.x & 63) == 0) all.store(box + 6 * to);
      }
    }
  }
}

template <typename Tin>
__global__ __launch_bounds__(1024) void boxes_wide_k(const Tin* X, const int64_t* off, int32_t L,
                                                     double* box, unsigned long long* tiles) {
  __shared__ MinMax<Tin> part[16];
  clear_tiles(tiles, L);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  for (int64_t l = blockIdx.x; l < L; l += gridDim.x) {
    MinMax<Tin> m;
    m.clear();
    for (int64_t v = off[l] + threadIdx.x; v < off[l + 1]; v += blockDim.x) m.add(X + 3 * v);
    m.template reduce<64>();
    if (lane == 0) part[w] = m;
    __syncthreads();
    if (w == 0) {
      MinMax<Tin> t;
      t.clear();
      if (lane < nw) t = part[lane];
      t.template reduce<16>();
      if (lane == 0) t.store(box + 6 * l);
    }
    __syncthreads();
  }
}

// All six bounds are loaded before the first comparison (a chain of || would wait
// for them one after the other).
__device__ __forceinline__ bool overlap(const double* P, const double* Q) {
  const double q0 = Q[0], q1 = Q[1], q2 = Q[2], q3 = Q[3], q4 = Q[4], q5 = Q[5];
  return !((P[0] > q3) | (q0 > P[3]) | (P[1] > q4) | (q1 > P[4]) | (P[2] > q5) | (q2 > P[5]));
}

// ------------------------------------- potential link search on a hashed grid
// A box is "regular" when it is finite, no side is longer than `side` (the cell
// size h is 17/16 of that) and its cell coordinates are below 2^40; regular
// boxes are binned by the cell of their min corner.  Two overlapping regular
// boxes have min corners at most 16/17 of a cell apart on every axis, so with
// the rounding of the coordinates (below 2^-11 of a cell) their cells differ
// by at most one: a regular box only meets the regular boxes of the 27 cells
// around its own.  (Cells of twice the side gave 3.5 times the candidates on a
// sheet.)  Cells are hashed into a table of buckets, so the scene's extent does
// not matter; boxes of other cells that share a bucket are candidates the box
// test rejects.  Every other box (large, empty, far off or non-finite) is
// tested against all boxes with the same predicate as the all-pairs scan, so
// both give exactly the same pairs.  Each pair is found once, from its smaller
// index; a row's pairs are sorted by j, so the output is lexicographic.
__device__ __forceinline__ double grid_cell(const GridParams& g, const double* b, int q) {
  return floor((b[q] - g.lo[q]) * g.inv_h);
}

__device__ __forceinline__ bool box_regular(const GridParams& g, const double* b) {
  bool ok = true;
  for (int q = 0; q < 3; ++q) {
    const double e = b[3 + q] - b[q];
    ok = ok && isfinite(b[q]) && isfinite(b[3 + q]) && e >= 0.0 && e <= g.side &&
         fabs(grid_cell(g, b, q)) < 1.0e12;
  }
  return ok;
}

// buckets is a power of two, so the hash is masked rather than divided
__device__ __forceinline__ int32_t grid_bucket(const GridParams& g, int64_t x, int64_t y,
                                               int64_t z) {
  const uint64_t k = ((uint64_t)x * 73856093ull) ^ ((uint64_t)y * 19349663ull) ^
                     ((uint64_t)z * 83492791ull);
  return (int32_t)((k ^ (k >> 29)) & (uint64_t)(g.buckets - 1));
}

// The grid parameters in two passes over the boxes.  Every reduction runs in a
// fixed order (64 workgroup partials, each a tree in LDS), so the cell size
// does not depend on scheduling.  Pass 0 sums the box sizes (the largest side
// per box) and clears the bucket counts; pass 1 takes the largest size not above
// 4 x their mean and, over the boxes up to that size, each axis' min corner of
// least magnitude.  That is the grid's origin: with the least corner, one loop
// thrown 1e13 sizes off to the negative side made every other box irregular (20,000
// loops took 359 us, now 113; 87 without it).
__device__ __forceinline__ double grid_box_size(const double* b) {
  double e = -1.0;
  for (int q = 0; q < 3; ++q) e = fmax(e, b[3 + q] - b[q]);
  return e;
}

static_assert(kGridStatBlocks == 64, "one partial per lane");
__device__ __forceinline__ double wave_sum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}
// the one nearer to 0 (of two at one distance the negative one)
__device__ __forceinline__ double nearer(double a, double b) {
  const double x = fabs(a), y = fabs(b);
  return y < x || (y == x && b < a) ? b : a;
}
__device__ __forceinline__ double wave_nearest(double v) {
  for (int o = 32; o > 0; o >>= 1) v = nearer(v, __shfl_xor(v, o));
  return v;
}
__device__ __forceinline__ double wave_max(double v) {
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o));
  return v;
}

template <int PASS>
__global__ __launch_bounds__(256) void grid_stats_k(const double* box, int32_t L, int64_t buckets,
                                                    double* part, uint32_t* cell_count,
                                                    int32_t* n_over, uint32_t* n_binned) {
  __shared__ double red[4][256];
  const int t = threadIdx.x, lane = t & 63;
  double cap = 0.0;
  if (PASS == 1) {
    const double s = wave_sum(part[lane]), c = wave_sum(part[kGridStatBlocks + lane]);
    cap = 4.0 * (c > 0.0 ? s / c : 0.0);
  }
  constexpr int kValues = PASS == 0 ? 2 : 4;  // size sum and count; size, origin
  double v[4] = {0.0, PASS == 0 ? 0.0 : INFINITY, INFINITY, INFINITY};
  for (int64_t i = (int64_t)blockIdx.x * 256 + t; i < L; i += kGridStatBlocks * 256) {
    const double* b = box + 6 * i;
    const double e = grid_box_size(b);
    if (PASS == 0) {
      if (isfinite(e) && e >= 0.0) {
        v[0] += e;
        v[1] += 1.0;
      }
    } else if (isfinite(e) && e <= cap) {
      v[0] = fmax(v[0], e);
      for (int q = 0; q < 3; ++q)
        if (isfinite(b[q])) v[1 + q] = nearer(v[1 + q], b[q]);
    }
  }
  if (PASS == 0) {
    for (int64_t k = (int64_t)blockIdx.x * 256 + t; k < buckets; k += kGridStatBlocks * 256)
      cell_count[k] = 0u;
    if (blockIdx.x == 0 && t == 0) {
      *n_over = 0;
      *n_binned = 0u;
    }
  }
  for (int q = 0; q < kValues; ++q) red[q][t] = v[q];
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (t < w) {
      if (PASS == 0) {
        red[0][t] += red[0][t + w];
        red[1][t] += red[1][t + w];
      } else {
        red[0][t] = fmax(red[0][t], red[0][t + w]);
        for (int q = 1; q < 4; ++q) red[q][t] = nearer(red[q][t], red[q][t + w]);
      }
    }
    __syncthreads();
  }
  if (t < kValues) part[((PASS == 0 ? 0 : 2) + t) * kGridStatBlocks + blockIdx.x] = red[t][0];
}

// Each workgroup finishes the grid parameters from the partials; the first one
// stores them for the later kernels.
__global__ __launch_bounds__(256) void grid_bin_k(const double* box, int32_t L, const double* part,
                                                  int64_t buckets, GridParams* gp,
                                                  uint32_t* cell_count, int32_t* cell_of,
                                                  int32_t* over, int32_t* n_over) {
  const int lane = threadIdx.x & 63;
  GridParams g;
  const double em = wave_max(part[2 * kGridStatBlocks + lane]);
  g.side = em > 0.0 ? em : 1.0;
  g.inv_h = 1.0 / (1.0625 * g.side);
  for (int q = 0; q < 3; ++q) {
    const double m = wave_nearest(part[(3 + q) * kGridStatBlocks + lane]);
    g.lo[q] = isfinite(m) ? m : 0.0;
  }
  g.buckets = buckets;
  if (blockIdx.x == 0 && threadIdx.x == 0) *gp = g;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < L; i += (int64_t)gridDim.x * 256) {
    const double* b = box + 6 * i;
    if (box_regular(g, b)) {
      const int32_t c = grid_bucket(g, (int64_t)grid_cell(g, b, 0), (int64_t)grid_cell(g, b, 1),
                                    (int64_t)grid_cell(g, b, 2));
      cell_of[i] = c;
      atomicAdd(&cell_count[c], 1u);
    } else {
      cell_of[i] = -1;
      over[atomicAdd(n_over, 1)] = (int32_t)i;
    }
  }
}

// Room for every bucket's boxes: buckets in order within a workgroup's 1,024,
// the workgroups' runs in any order (rows are sorted in the end).
__global__ __launch_bounds__(256) void grid_alloc_k(const uint32_t* cell_count, int64_t buckets,
                                                    uint2* cell, uint32_t* n_binned) {
  __shared__ uint32_t wsum[4], base;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t k0 = (int64_t)blockIdx.x * 1024 + 4 * (int64_t)threadIdx.x;
  uint32_t c[4], sum = 0u;
  for (int i = 0; i < 4; ++i) {
    c[i] = k0 + i < buckets ? cell_count[k0 + i] : 0u;
    sum += c[i];
  }
  uint32_t x = sum;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  if (lane == 63) wsum[w] = x;
  __syncthreads();
  if (threadIdx.x == 0) base = atomicAdd(n_binned, wsum[0] + wsum[1] + wsum[2] + wsum[3]);
  __syncthreads();
  uint32_t run = base + x - sum;
  for (int q = 0; q < w; ++q) run += wsum[q];
  for (int i = 0; i < 4; ++i) {
    if (k0 + i < buckets) cell[k0 + i] = uint2{run, run};
    run += c[i];
  }
}

// Each box takes the next place of its bucket (whose .y ends at the bucket's
// end); a copy of the box goes with it, so a bucket's boxes are read
// contiguously.
__global__ __launch_bounds__(256) void grid_scatter_k(const double* box, int32_t L,
                                                      const int32_t* cell_of, uint2* cell,
                                                      int32_t* cell_items, double* cell_box) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < L; i += (int64_t)gridDim.x * 256) {
    const int32_t c = cell_of[i];
    if (c < 0) continue;
    const int64_t pos = atomicAdd(&cell[c].y, 1u);
    cell_items[pos] = (int32_t)i;
    for (int q = 0; q < 6; ++q) cell_box[6 * pos + q] = box[6 * i + q];
  }
}

// The rows of the pair list, one wavefront per row i, the lanes testing 64
// candidates j > i side by side; emit(hit, j) is called by all lanes.  GRID:
// a regular box's candidates are its 27 buckets' boxes as one list (lane t < 27
// reads bucket t's range, a scan makes the ranges one, and lane c of a round
// finds its place in it), so a row waits for five loads in turn, not for three
// in each bucket.  Everything else is tested against all later boxes.
template <bool GRID, typename Emit>
__device__ __forceinline__ void row_candidates(const double* box, int32_t L, int64_t i,
                                               const RowGrid& R, const Emit& emit) {
  const int lane = threadIdx.x & 63;
  double me[6];
  for (int q = 0; q < 6; ++q) me[q] = box[6 * i + q];
  if (GRID && R.cell_of[i] >= 0) {
    const GridParams g = *R.params;
    const int64_t c0 = (int64_t)grid_cell(g, me, 0), c1 = (int64_t)grid_cell(g, me, 1),
                  c2 = (int64_t)grid_cell(g, me, 2);
    const int tl = lane < 27 ? lane : 0;
    const int32_t mine = grid_bucket(g, c0 + tl % 3 - 1, c1 + (tl / 3) % 3 - 1, c2 + tl / 9 - 1);
    // a bucket reached by two neighbour cells is visited once, at its first lane
    bool dup = lane >= 27;
    for (int u = 0; u < 26; ++u)
      dup = dup || (u < lane && __builtin_amdgcn_readlane(mine, u) == mine);
    const uint2 se = dup ? uint2{0u, 0u} : R.cell[mine];
    const int32_t n = (int32_t)(se.y - se.x);
    int32_t x = n;
    for (int o = 1; o < 32; o <<= 1) {
      const int32_t y = __shfl_up(x, o);
      if (lane >= o) x += y;
    }
    const int32_t total = __builtin_amdgcn_readlane(x, 26), before = x - n;
    const int32_t shift = (int32_t)se.x - before;  // a bucket's place of list entry k: k + shift
    const unsigned long long some = __ballot(n > 0);
    for (int32_t k0 = 0; k0 < total; k0 += 64) {
      const int32_t k = k0 + lane;
      int32_t sh = 0;
      for (unsigned long long m = some; m; m &= m - 1ull) {
        const int u = __ffsll((long long)m) - 1;
        sh = k >= __builtin_amdgcn_readlane(before, u) ? __builtin_amdgcn_readlane(shift, u) : sh;
      }
      const bool in = k < total;
      const int64_t at = in ? (int64_t)k + sh : 0;
      const int32_t j = in ? R.cell_items[at] : -1;
      emit(overlap(me, R.cell_box + 6 * at) & (j > i), j);  // (j is -1 beyond the list)
    }
    const int32_t no = *R.n_over;
    for (int32_t k0 = 0; k0 < no; k0 += 64) {
      const int32_t k = k0 + lane;
      const int32_t j = k < no ? R.over[k] : -1;
      emit(k < no && j > i && overlap(me, box + 6 * (int64_t)j), j);
    }
  } else {
    for (int64_t j0 = i + 1; j0 < L; j0 += 256) {
      bool hit[4];  // four rounds' loads in flight
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int64_t j = j0 + 64 * q + lane;
        hit[q] = overlap(me, box + 6 * (j < L ? j : i)) & (j < L);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) emit(hit[q], (int32_t)(j0 + 64 * q + lane));
    }
  }
}

// Counts the rows' pairs, per row and per tile of kRowTile rows, and keeps the
// first kRowSlots of each row for the fill.  16 rows per workgroup, whose sum
// goes to the tile in one atomic (one per row queued 256 of them on each
// tile's count: 104 us instead of 43 for 20,000 loops).
template <bool GRID>
__global__ __launch_bounds__(64 * kFillRows) void rows_count_k(const double* box, int32_t L,
                                                               RowGrid R, RowBufs B) {
  __shared__ int32_t sum[kFillRows];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const unsigned long long below = lane ? (~0ull >> (64 - lane)) : 0ull;
  const int64_t i = (int64_t)blockIdx.x * kFillRows + w;
  int32_t cnt = 0;  // uniform over the wave
  if (i < L) {
    row_candidates<GRID>(box, L, i, R, [&](bool hit, int32_t j) {
      const unsigned long long m = __ballot(hit);
      const int32_t at = cnt + (int32_t)__popcll(m & below);
      if (hit && at < kRowSlots) B.slots[i * kRowSlots + at] = j;
      cnt += (int32_t)__popcll(m);
    });
    if (lane == 0) B.counts[i] = cnt;
  }
  if (lane == 0) sum[w] = cnt;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long t = 0ull;
    for (int q = 0; q < kFillRows; ++q) t += (unsigned long long)sum[q];
    if (t) atomicAdd(&B.tiles[(int64_t)blockIdx.x * kFillRows / kRowTile], t);
  }
}

// Writes the rows, 16 per workgroup.  A row's place is the sum of the earlier
// tiles and of its tile's earlier rows, which each workgroup adds up itself
// (cheaper than a scan in a launch of its own), but for more than kRowTilesDirect
// tiles, which a launch before scans (SCANNED): added up by every workgroup they
// took 90 of the 150 ms of a search of 30 million loops.  (At one million 1,940 us
// so, 1,830 scanned; at 60,000 168 and a launch more.)
// Nothing is written unless all pairs fit; the first workgroup reports the total to the host.  A row whose
// pairs are all in its slots is sorted by counting, lane against lane.  A longer
// one is searched again; if the grid gives it, the wave gathers up to kRowSort
// second indices in LDS and counts for each how many are below it, and a row of
// more is searched without the grid, which gives them in order.  (Sorted in place by
// one lane, a search of 7,000 loops whose 64 first rows have up to 238 pairs took
// 1,740 us, 1,024 rows of up to 1,059 141,000 us, 20,000 loops of 114 pairs a row
// 18,600 us; now 330, 815 and 1,900.  The registers of five waves a SIMD: with four,
// sheets of 20,000 loops took 96 us, with five 90.)
constexpr int kRowSort = 1024;
constexpr int64_t kRowTilesDirect = 1024;
template <bool GRID, bool SCANNED>
__global__ __launch_bounds__(256, 5) void rows_fill_k(const double* box, int32_t L, RowGrid R,
                                                   RowBufs B, int32_t* out, int64_t capacity,
                                                   int64_t* host_total) {
  __shared__ int64_t red[2][4];
  __shared__ int32_t row_n[kFillRows];
  __shared__ __align__(16) int32_t gathered[GRID ? 4 : 1][GRID ? kRowSort : 4];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t base = (int64_t)blockIdx.x * kFillRows;
  const int64_t tile = base / kRowTile, n_tiles = (L + kRowTile - 1) / kRowTile;
  int64_t before = 0, total = 0;
  if (!SCANNED)
    for (int64_t k = threadIdx.x; k < n_tiles; k += 256) {
      const int64_t c = (int64_t)B.tiles[k];
      total += c;
      if (k < tile) before += c;
    }
  const int64_t r = tile * kRowTile + threadIdx.x;  // kRowTile == 256
  const int32_t c = r < L ? B.counts[r] : 0;
  if (r < base) before += c;
  if (r >= base && r < base + kFillRows) row_n[r - base] = c;
  for (int o = 32; o > 0; o >>= 1) {
    before += __shfl_xor(before, o);
    total += __shfl_xor(total, o);
  }
  if (lane == 0) {
    red[0][w] = before;
    red[1][w] = total;
  }
  __syncthreads();
  total = SCANNED ? (int64_t)B.tiles[n_tiles] : red[1][0] + red[1][1] + red[1][2] + red[1][3];
  if (!SCANNED && blockIdx.x == 0 && threadIdx.x == 0)
    __hip_atomic_store(host_total, total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  if (total > capacity) return;
  int64_t pos = red[0][0] + red[0][1] + red[0][2] + red[0][3];
  if (SCANNED) pos += (int64_t)B.tiles[tile];
  const unsigned long long below = lane ? (~0ull >> (64 - lane)) : 0ull;
  for (int q = 0; q < kFillRows; ++q) {
    const int64_t i = base + q;
    const int32_t n = __builtin_amdgcn_readfirstlane(row_n[q]);
    if ((q & 3) == w && i < L && n > 0) {
      if (n <= kRowSlots) {
        const int32_t j = lane < n ? B.slots[i * kRowSlots + lane] : 0;
        int32_t rank = lane;
        if (GRID) {
          rank = 0;
          for (int u = 0; u < n; ++u) rank += __builtin_amdgcn_readlane(j, u) < j ? 1 : 0;
        }
        if (lane < n) {
          out[2 * (pos + rank)] = (int32_t)i;
          out[2 * (pos + rank) + 1] = j;
        }
      } else if (GRID && n <= kRowSort && R.cell_of[i] >= 0) {
        int32_t* const g = gathered[w];
        int32_t to = 0;  // uniform over the wave
        row_candidates<GRID>(box, L, i, R, [&](bool hit, int32_t j) {
          const unsigned long long m = __ballot(hit);
          if (hit) g[to + (int32_t)__popcll(m & below)] = j;
          to += (int32_t)__popcll(m);
        });
        if (lane < 3 && n + lane < kRowSort) g[n + lane] = INT32_MAX;  // up to a multiple of four
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        for (int k = lane; k < n; k += 64) {
          const int32_t j = g[k];
          int32_t rank = 0;
#pragma unroll 4
          for (int u = 0; u < n; u += 4) {
            const int4 v = *reinterpret_cast<const int4*>(g + u);
            rank += (v.x < j) + (v.y < j) + (v.z < j) + (v.w < j);
          }
          out[2 * (pos + rank)] = (int32_t)i;
          out[2 * (pos + rank) + 1] = j;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      } else {
        int64_t to = pos;  // uniform over the wave
        row_candidates<false>(box, L, i, R, [&](bool hit, int32_t j) {
          const unsigned long long m = __ballot(hit);
          if (hit) {
            const int64_t at = to + __popcll(m & below);
            out[2 * at] = (int32_t)i;
            out[2 * at + 1] = j;
          }
          to += __popcll(m);
        });
      }
    }
    pos += n;
  }
}

// ------------------------------------------------------------ verification
__device__ __forceinline__ long long key_of(const int32_t* pr, int64_t k) {
  return ((long long)pr[2 * k] << 32) | (unsigned int)pr[2 * k + 1];
}
// first index in [0, n) whose key is >= x
__device__ __forceinline__ int64_t lower_bound_key(const int32_t* pr, int64_t n, long long x) {
  int64_t lo = 0, hi = n;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (key_of(pr, mid) < x)
      lo = mid + 1;
    else
      hi = mid;
  }
  return lo;
}

// Mismatch indicator per position of the concatenation [current | expected]:
// current c mismatches when lk[c] differs from the expected value (0 if the
// pair is not expected); expected e counts when it is absent from the current
// list and non-zero.
__global__ __launch_bounds__(256) void verify_flag_k(const int32_t* pr, const int32_t* lk,
                                                     int64_t n, const int32_t* ep,
                                                     const int32_t* elk, int64_t ne,
                                                     int64_t* m) {
  const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (k < n) {
    const long long x = key_of(pr, k);
    const int64_t e = lower_bound_key(ep, ne, x);
    const int32_t want = (e < ne && key_of(ep, e) == x) ? elk[e] : 0;
    m[k] = (lk[k] != want) ? 1 : 0;
  } else if (k < n + ne) {
    const int64_t e = k - n;
    const long long x = key_of(ep, e);
    const int64_t c = lower_bound_key(pr, n, x);
    const bool present = c < n && key_of(pr, c) == x;
    m[k] = (!present && elk[e] != 0) ? 1 : 0;
  }
}

// Scatter mismatch records in pair order.  The rank of a mismatch in pair
// order is (mismatches of the other list with a smaller key) + (its rank
// within its own list); keys of the two lists never tie for counted records
// (a key in both lists is counted once, from the current list).
__global__ __launch_bounds__(256) void verify_scatter_k(const int32_t* pr, const int32_t* lk,
                                                        int64_t n, const int32_t* ep,
                                                        const int32_t* elk, int64_t ne,
                                                        const int64_t* mp, int32_t* out,
                                                        int64_t cap) {
  const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (k >= n + ne) return;
  if (mp[k + 1] == mp[k]) return;  // not a mismatch
  const int64_t base_c = 0, base_e = mp[n];
  long long x;
  int64_t rank;
  int32_t got, want;
  if (k < n) {
    x = key_of(pr, k);
    const int64_t e = lower_bound_key(ep, ne, x);
    want = (e < ne && key_of(ep, e) == x) ? elk[e] : 0;
    got = lk[k];
    rank = (mp[k] - base_c) + (mp[n + e] - base_e);
  } else {
    const int64_t e = k - n;
    x = key_of(ep, e);
    const int64_t c = lower_bound_key(pr, n, x);
    want = elk[e];
    got = 0;
    rank = (mp[k] - base_e) + (mp[c] - base_c);
  }
  if (rank < cap) {
    out[4 * rank] = (int32_t)(x >> 32);
    out[4 * rank + 1] = (int32_t)(x & 0xffffffffll);
    out[4 * rank + 2] = got;
    out[4 * rank + 3] = want;
  }
}

// Preparation, plan and schedule of a call with few pairs in one launch: the
// per-loop scan of prep_k, xi in a fixed order, then the plan and the schedule.
// Small scenes are scanned by the first workgroup (16 lanes per loop, so 64 loops
// at once and their loads overlap) and the others leave.  Otherwise the vertices
// are scanned in equal pieces, a wavefront each, whatever the loops' sizes, and
// the workgroup that ends last puts the pieces together, plans and schedules
// (each step reads only what was written before a barrier, or before the ticket).
// A step of 16 lanes takes 0.16 us and the pieces' fences and ticket 12 us, so the
// line lies at some 64 steps: us per call with one workgroup / in pieces at 64
// loops of 32 vertices 23.6 / 36.4, 64 of 512 31.0 / 36.5, 1,000 of 8 32.8 / 34.7,
// 4 of 2,048 41.7 / 36.5, 2 of 8,192 104 / 36.5, 2 of 32,768 364 / 36.4.  Per call
// of 100 yarns of up to 16,384 vertices this launch went from 331 to 25 us, of
// three pairs of 90,000 vertices from 2,200 to 25 us.
constexpr int64_t kPrepAloneVertices = 32768, kPrepAloneLoop = 1024;
constexpr int32_t kPrepAloneLoops = 1024;

// What the pieces leave.  A loop is owned by the piece that its first vertex is
// in; one that ends in there is complete and goes to lf and minseg2 directly.
struct PrepPieces {
  unsigned* ticket;
  double *xi, *head_min, *tail_min;     // sums; minima of the parts below
  uint32_t *head_flags, *tail_flags;
  int32_t *head_owner;  // the piece's first part, of a loop that another piece owns (-1: none)
  int32_t *tail_loop;   // the piece's last part, of an own loop that goes on (-1: none)
  __host__ __device__ explicit PrepPieces(void* p) {
    char* c = static_cast<char*>(p);
    ticket = (unsigned*)c;
    xi = (double*)(c + 256);
    head_min = xi + kPrepPieces;
    tail_min = head_min + kPrepPieces;
    head_flags = (uint32_t*)(tail_min + kPrepPieces);
    tail_flags = head_flags + kPrepPieces;
    head_owner = (int32_t*)(tail_flags + kPrepPieces);
    tail_loop = head_owner + kPrepPieces;
  }
};

// In head_flags: the piece's share of the offsets decreases somewhere.
constexpr uint32_t kPieceDecreases = 1u << 31;

// The first loop that starts at vertex x or later (off[0] = 0), found by a wavefront.
// Whatever the offsets hold, it ends and returns 0 .. L.
__device__ int32_t first_loop_from(const int64_t* off, int32_t L, int64_t x, int lane) {
  int32_t lo = 0, hi = L;  // starts below lo are before x, those from hi on are not
  while (lo < hi) {
    const int32_t step = (hi - lo + 63) / 64;
    const int64_t at = lo + (int64_t)lane * step;
    const bool before = at < hi && off[at] - off[0] < x;
    const int n = __popcll(__ballot(before));  // a prefix of the lanes
    if (n == 0) return lo;
    const int64_t top = lo + (int64_t)n * step;
    lo += (n - 1) * step + 1;
    hi = top < hi ? (int32_t)top : hi;
  }
  return lo;
}

// Vertices a .. b - 1 of loop l (positions from the loop's first, a >= 0; none
// beyond its last): flags and shortest squared segment in every lane, the lane's
// sum of coordinates returned.
template <typename Tin>
__device__ double scan_part(const Tin* X, const int64_t* off, int32_t l, int64_t a, int64_t b,
                            int lane, uint32_t* flags, double* shortest) {
  const int64_t o = off[l], n = off[l + 1] - o;
  if (b > n) b = n;
  uint32_t f = 0u;
  double s = 0.0, mn = INFINITY;
#pragma unroll 4
  for (int64_t q = a + lane; q < b; q += 64) {
    const Tin* P = X + 3 * (o + q);
    const Tin* Q = X + 3 * (o + (q + 1 == n ? 0 : q + 1));
    const double x0 = (double)P[0], y0 = (double)P[1], z0 = (double)P[2];
    const double dx = (double)Q[0] - x0, dy = (double)Q[1] - y0, dz = (double)Q[2] - z0;
    if (!isfinite(x0) || !isfinite(y0) || !isfinite(z0)) f |= kFlagNonfinite | kFlagBadloop;
    s += fabs(x0) + fabs(y0) + fabs(z0);
    mn = fmin(mn, dx * dx + dy * dy + dz * dz);
  }
  for (int w = 32; w > 0; w >>= 1) {
    f |= (uint32_t)__shfl_xor((int)f, w);
    mn = fmin(mn, __shfl_xor(mn, w));
  }
  *flags = f;
  *shortest = mn;
  return s;
}

// Offsets that decrease make a loop of negative size, which is invalid by itself,
// but then the loops' starts are not sorted and pieces miss some of their
// vertices.  So each piece looks through an equal share of the offsets, and where
// one finds a decrease the workgroup that ends last scans loop by loop.  Until
// then every access stays in range: a piece leaves out what does not start where
// sorted offsets would have it.
template <typename Tin>
__device__ void scan_piece(const Tin* X, const int64_t* off, int32_t L, int64_t V, int32_t k,
                           int lane, uint32_t* lf, double* minseg2, const PrepPieces& P) {
  const int64_t share = ((int64_t)L + kPrepPieces - 1) / kPrepPieces;
  const int64_t end = (k + 1) * share < L ? (k + 1) * share : L;
  bool decreases = false;
  for (int64_t l = k * share + lane; l < end; l += 64) decreases |= off[l + 1] < off[l];
  if (__any(decreases)) {
    if (lane == 0) P.head_flags[k] = kPieceDecreases;
    return;
  }
  const int64_t len = V > 0 ? (V + kPrepPieces - 1) / kPrepPieces : 1, o0 = off[0];
  const int64_t s = k * len, e = s + len < V ? s + len : V;
  const bool last = k == kPrepPieces - 1;
  const int32_t l0 = first_loop_from(off, L, s, lane);
  const int32_t l1 = last ? L : first_loop_from(off, L, s + len, lane);
  double sum = 0.0, mn = INFINITY;
  uint32_t f = 0u;
  int32_t owner = -1;
  if (l0 > 0) {
    const int64_t o = off[l0 - 1] - o0, end0 = off[l0] - o0;  // of the loop before l0
    if (0 <= o && o < s && end0 > s) {
      owner = (int32_t)(o / len);  // below k
      sum += scan_part(X, off, l0 - 1, s - o, (end0 < e ? end0 : e) - o, lane, &f, &mn);
    }
  }
  if (lane == 0) {
    P.head_owner[k] = owner;
    P.head_flags[k] = f;
    P.head_min[k] = mn;
  }
  int32_t tail = -1;
  f = 0u;
  mn = INFINITY;
  for (int32_t l = l0; l < l1; ++l) {
    const int64_t o = off[l] - o0, n = off[l + 1] - off[l];
    if (o < s || (o >= s + len && !last)) break;
    const bool on = o + n > e;  // the last of them
    sum += scan_part(X, off, l, 0, on ? e - o : n, lane, &f, &mn);
    if (n < 3) f |= kFlagBadloop;
    if (on) {
      tail = l;
    } else if (lane == 0) {
      lf[l] = f;
      minseg2[l] = mn;
    }
  }
  for (int w = 32; w > 0; w >>= 1) sum += __shfl_xor(sum, w);
  if (lane == 0) {
    P.tail_loop[k] = tail;
    P.tail_flags[k] = f;
    P.tail_min[k] = mn;
    P.xi[k] = sum;
  }
}

// Whether a piece found offsets that decrease (the same in every thread of the one
// workgroup that calls it).
__device__ bool pieces_decrease(const PrepPieces& P) {
  bool d = false;
  for (int k = threadIdx.x; k < kPrepPieces; k += 1024) d |= (P.head_flags[k] & kPieceDecreases) != 0u;
  return __syncthreads_or(d);
}

// The parts of loops that several pieces scanned, one workgroup; returns the
// thread's part of the sum of coordinates.
__device__ double join_pieces(const PrepPieces& P, uint32_t* lf, double* minseg2) {
  __shared__ unsigned long long mn[kPrepPieces];  // of squares: ordered as their bits
  __shared__ uint32_t f[kPrepPieces];
  double s = 0.0;
  for (int k = threadIdx.x; k < kPrepPieces; k += 1024) {
    mn[k] = (unsigned long long)__double_as_longlong(P.tail_min[k]);
    f[k] = P.tail_flags[k];
    s += P.xi[k];
  }
  __syncthreads();
  for (int k = threadIdx.x; k < kPrepPieces; k += 1024) {
    const int32_t o = P.head_owner[k];
    if (o < 0) continue;
    atomicMin(&mn[o], (unsigned long long)__double_as_longlong(P.head_min[k]));
    atomicOr(&f[o], P.head_flags[k]);
  }
  __syncthreads();
  for (int k = threadIdx.x; k < kPrepPieces; k += 1024) {
    const int32_t l = P.tail_loop[k];
    if (l < 0) continue;
    lf[l] = f[k];
    minseg2[l] = __longlong_as_double((long long)mn[k]);
  }
  return s;
}

template <typename Tin>
__global__ __launch_bounds__(1024) void prep_plan_k(const Tin* X, PlanArgs A, int32_t L,
                                                    LoopInfo li, uint32_t* lf, double* minseg2,
                                                    Sched S, PrepPieces P,
                                                    unsigned long long* zero_mismatch,
                                                    int32_t* zero_stop, int32_t* zero_next) {
  __shared__ double red[1024];
  __shared__ unsigned order;
  const int64_t nv = A.off[L] - A.off[0];
  const int64_t ln = threadIdx.x < L ? A.off[threadIdx.x + 1] - A.off[threadIdx.x] : 0;
  const bool alone =
      !__syncthreads_or(ln > kPrepAloneLoop) && nv <= kPrepAloneVertices && L <= kPrepAloneLoops;
  if (alone && blockIdx.x > 0) return;
  double s = 0.0;
  if (!alone) {
    scan_piece(X, A.off, L, nv, (int32_t)(blockIdx.x * 16 + (threadIdx.x >> 6)),
               (int)(threadIdx.x & 63), lf, minseg2, P);
    __syncthreads();
    if (threadIdx.x == 0) {
      __threadfence();  // the workgroup's pieces before its ticket
      // wraps to 0 with the last workgroup: after every whole number of launches
      // the ticket is 0, also after launches that overlapped against the rules
      order = atomicInc(P.ticket, gridDim.x - 1);
    }
    __syncthreads();
    if (order != gridDim.x - 1) return;
    __threadfence();  // every workgroup's pieces
  }
  if (threadIdx.x < 2) S.counts[threadIdx.x] = 0;
  if (threadIdx.x == 0 && zero_mismatch) {
    *zero_mismatch = 0ull;
    *zero_stop = 0;
  }
  if (alone || pieces_decrease(P)) {
    const int sub = threadIdx.x & 15, group = threadIdx.x >> 4;
    for (int64_t l = group; l < L; l += 64)
      s += scan_loop<Tin, 16>(X, A.off, l, sub, lf, minseg2);
  } else {
    s = join_pieces(P, lf, minseg2);
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 512; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  const double xi = nv > 0 ? red[0] / (3.0 * (double)nv) : 0.0;
  plan_positions(A, L, li, S, 0, xi, A.n_list, 0, 1024);
  __syncthreads();
  schedule(S, zero_next);
}

}  // namespace

// ---------------------------------------------------------------- launchers
int prep_blocks(int32_t n_loops, int64_t n_vertices) {
  // one wavefront per loop up to kPrepMaxBlocks * 4 loops, and (when the
  // vertex count is known) enough workgroups to stream the coordinates
  int64_t g = ((int64_t)n_loops + 3) / 4;
  const int64_t gv = n_vertices / 8192;
  if (gv > g) g = gv;
  if (g < kXiBlocks) g = kXiBlocks;
  if (g > kPrepMaxBlocks) g = kPrepMaxBlocks;
  return (int)g;
}

hipError_t launch_prep(const void* xyz, bool in_f64, const int64_t* off, int32_t n_loops,
                       double* xi_partials, uint32_t* lf, double* minseg2, int32_t* zero_counts,
                       unsigned long long* zero_mismatch, int32_t* zero_stop, bool scan_loops,
                       int n_blocks, hipStream_t s) {
  const int g = n_blocks;
  const int sl = scan_loops ? 1 : 0;
  if (in_f64)
    prep_k<double><<<g, 256, 0, s>>>((const double*)xyz, off, n_loops, xi_partials, lf, minseg2,
                                     zero_counts, zero_mismatch, zero_stop, sl);
  else
    prep_k<float><<<g, 256, 0, s>>>((const float*)xyz, off, n_loops, xi_partials, lf, minseg2,
                                    zero_counts, zero_mismatch, zero_stop, sl);
  return hipGetLastError();
}

hipError_t launch_cc_boxes(const void* xyz, bool in_f64, const int64_t* off, int32_t n_loops,
                           const CcProj& pr, float4* blk, int64_t n_blk, float4* sup,
                           int64_t n_sup, uint32_t* lf, double* minseg2, hipStream_t s) {
  // four slots (waves) per workgroup; the grid strides over the device's count
  const int g = blocks_for(n_sup, 4, 16384);
  if (in_f64)
    cc_boxes_k<double><<<g, 256, 0, s>>>((const double*)xyz, off, n_loops, pr, blk, n_blk, sup,
                                         n_sup, lf, minseg2);
  else
    cc_boxes_k<float><<<g, 256, 0, s>>>((const float*)xyz, off, n_loops, pr, blk, n_blk, sup, n_sup,
                                        lf, minseg2);
  return hipGetLastError();
}

hipError_t launch_plan(const PlanArgs& a, int32_t n_loops, const LoopInfo& li, const Sched& sc,
                       bool refit, hipStream_t s) {
  // a refit list is short (pairs far from an integer): a few workgroups
  plan_k<<<blocks_for(a.n_list, 1024, refit ? 16 : 8192), 1024, 0, s>>>(a, n_loops, li, sc,
                                                                       refit ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_finalize_split(const Sched& sc, const unsigned long long* acc, const Outs& o,
                                 int64_t n_pairs, hipStream_t s) {
  // only multi-item pairs remain, at most a few thousand: grid stride
  finalize_split_k<<<blocks_for(n_pairs, 256, 64), 256, 0, s>>>(sc, acc, o);
  return hipGetLastError();
}

hipError_t launch_sched(const Sched& sc, int32_t* zero_next, hipStream_t s) {
  sched_k<<<1, 1024, 0, s>>>(sc, zero_next);
  return hipGetLastError();
}

hipError_t launch_prep_plan(const void* xyz, bool in_f64, const PlanArgs& a, int32_t n_loops,
                            const LoopInfo& li, uint32_t* lf, double* minseg2, const Sched& sc,
                            void* pieces, unsigned long long* zero_mismatch, int32_t* zero_stop,
                            int32_t* zero_next, hipStream_t s) {
  if (a.list || a.n_list_dev) return hipErrorInvalidValue;  // the main pass only
  const PrepPieces pc(pieces);
  if (in_f64)
    prep_plan_k<double><<<kPrepGroups, 1024, 0, s>>>((const double*)xyz, a, n_loops, li, lf,
                                                    minseg2, sc, pc, zero_mismatch, zero_stop, zero_next);
  else
    prep_plan_k<float><<<kPrepGroups, 1024, 0, s>>>((const float*)xyz, a, n_loops, li, lf,
                                                   minseg2, sc, pc, zero_mismatch, zero_stop, zero_next);
  return hipGetLastError();
}

hipError_t launch_finalize_replan(const Sched& sc, const unsigned long long* acc, const Outs& o,
                                  const PlanArgs& r, int32_t n_loops, const LoopInfo& li,
                                  const Sched& sr, int32_t* zero_next, hipStream_t s) {
  if (!r.n_list_dev) return hipErrorInvalidValue;
  finalize_replan_k<<<1, 1024, 0, s>>>(sc, acc, o, r, n_loops, li, sr, zero_next);
  return hipGetLastError();
}

__global__ void zero_i64_k(int64_t* p) { *p = 0; }

hipError_t launch_zero_i64(int64_t* p, hipStream_t s) {
  zero_i64_k<<<1, 1, 0, s>>>(p);
  return hipGetLastError();
}

hipError_t launch_scan(const int64_t* counts, int64_t n, int64_t* prefix, int64_t* host_total,
                       hipStream_t s) {
  scan_k<<<1, 1024, 0, s>>>(counts, n, prefix, host_total);
  return hipGetLastError();
}

// A workgroup per loop below 2,048 loops (of 1,024 threads below 256, where
// loops may be long: 100 knit rows of 8,000 vertices took 77 us with a
// wavefront each, 14 us so), a wavefront per loop below 8,192, 16 lanes above
// (20,000 loops of 32 vertices: 19.8 us with a wavefront each, 5.6 us so) for
// loops of up to kBoxNarrow vertices.
hipError_t launch_boxes(const void* xyz, bool in_f64, const int64_t* off, int32_t n_loops,
                        double* boxes, unsigned long long* tiles, hipStream_t s) {
  auto go = [&](auto* X) {
    using Tin = std::remove_const_t<std::remove_pointer_t<decltype(X)>>;
    if (n_loops < 2048)
      boxes_wide_k<Tin><<<n_loops, n_loops < 256 ? 1024 : 128, 0, s>>>(X, off, n_loops, boxes, tiles);
    else if (n_loops < 8192)
      boxes_k<Tin, 64><<<blocks_for((int64_t)n_loops * 64, 256, 8192), 256, 0, s>>>(X, off, n_loops,
                                                                                    boxes, tiles);
    else
      boxes_k<Tin, 16><<<blocks_for((int64_t)n_loops * 16, 256, 8192), 256, 0, s>>>(X, off, n_loops,
                                                                                    boxes, tiles);
  };
  if (in_f64)
    go((const double*)xyz);
  else
    go((const float*)xyz);
  return hipGetLastError();
}

hipError_t launch_grid(const double* boxes, int32_t n_loops, const GridBufs& b, hipStream_t s) {
  const int g = blocks_for(n_loops, 256, 4096);
  grid_stats_k<0><<<kGridStatBlocks, 256, 0, s>>>(boxes, n_loops, b.buckets, b.part, b.cell_count,
                                                  b.rows.n_over, b.n_binned);
  grid_stats_k<1><<<kGridStatBlocks, 256, 0, s>>>(boxes, n_loops, b.buckets, b.part, nullptr,
                                                  nullptr, nullptr);
  grid_bin_k<<<g, 256, 0, s>>>(boxes, n_loops, b.part, b.buckets, b.rows.params, b.cell_count,
                               b.rows.cell_of, b.rows.over, b.rows.n_over);
  grid_alloc_k<<<(unsigned)((b.buckets + 1023) / 1024), 256, 0, s>>>(b.cell_count, b.buckets,
                                                                     b.rows.cell, b.n_binned);
  grid_scatter_k<<<g, 256, 0, s>>>(boxes, n_loops, b.rows.cell_of, b.rows.cell, b.rows.cell_items,
                                   b.rows.cell_box);
  return hipGetLastError();
}

hipError_t launch_pair_rows(const double* boxes, int32_t n_loops, const RowGrid* grid,
                            const RowBufs& b, int32_t* pairs_out, int64_t capacity,
                            int64_t* host_total, hipStream_t s) {
  const unsigned gf = (unsigned)(((int64_t)n_loops + kFillRows - 1) / kFillRows);
  const int64_t n_tiles = ((int64_t)n_loops + kRowTile - 1) / kRowTile;
  const RowGrid g = grid ? *grid : RowGrid{};
  auto go = [&](auto with_grid, auto scanned) {
    constexpr bool G = decltype(with_grid)::value, S = decltype(scanned)::value;
    rows_count_k<G><<<gf, 64 * kFillRows, 0, s>>>(boxes, n_loops, g, b);
    if (S)
      scan_k<<<1, 1024, 0, s>>>((const int64_t*)b.tiles, n_tiles, (int64_t*)b.tiles, host_total);
    rows_fill_k<G, S><<<gf, 256, 0, s>>>(boxes, n_loops, g, b, pairs_out, capacity, host_total);
  };
  const std::true_type yes;
  const std::false_type no;
  if (n_tiles > kRowTilesDirect)
    grid ? go(yes, yes) : go(no, yes);
  else
    grid ? go(yes, no) : go(no, no);
  return hipGetLastError();
}

hipError_t launch_verify(const int32_t* pairs, const int32_t* lk, int64_t n,
                         const int32_t* exp_pairs, const int32_t* exp_lk, int64_t n_exp,
                         int64_t* mism_counts, hipStream_t s) {
  verify_flag_k<<<blocks_for(n + n_exp, 256), 256, 0, s>>>(pairs, lk, n, exp_pairs, exp_lk, n_exp,
                                                           mism_counts);
  return hipGetLastError();
}

hipError_t launch_verify_scatter(const int32_t* pairs, const int32_t* lk, int64_t n,
                                 const int32_t* exp_pairs, const int32_t* exp_lk, int64_t n_exp,
                                 const int64_t* mism_prefix, int32_t* out, int64_t cap,
                                 hipStream_t s) {
  verify_scatter_k<<<blocks_for(n + n_exp, 256), 256, 0, s>>>(pairs, lk, n, exp_pairs, exp_lk,
                                                              n_exp, mism_prefix, out, cap);
  return hipGetLastError();
}

}  // namespace lk
