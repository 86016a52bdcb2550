// Householder tridiagonalisation with the matrix held on the chip.
//
// A reflector needs the product of the whole trailing matrix with the
// reflector before it, so the columns are a serial chain; with a launch per
// stage of a step (npga_sketch.hip) a column costs a read and a write of the
// trailing matrix and three launches.  Here up to 256 workgroups hold the
// last kTriMax columns' trailing matrix in registers, whole rows (both
// triangles) dealt out cyclically, and run the whole chain in one launch:
//
//   step i: every workgroup has p = tau_{i-1} A v_{i-1} and row i of the
//   matrix, both before the rank-2 update of step i - 1.  Each one forms w =
//   p - (tau/2)(p^T v) v, the updated row i, and from it the reflector v_i
//   (the same arithmetic on the same numbers everywhere, so nothing else has
//   to be sent), updates its own rows, and sends its entries of p and, the
//   owner of row i + 1, that row.
//
// A step has one exchange and no barrier between workgroups.  The exchanged
// vectors have a slot of their own in every step, filled beforehand with a
// word that no arithmetic produces; a reader waits for the entries it needs.
// Entries are stored and read at device scope.  Every wait is bounded: a
// workgroup whose wait runs out raises the abort word and all leave; the
// upper triangle still holds the trailing matrix (the reflectors go to the
// lower one), and the caller goes on with a launch per stage.
//
// Bound by the exchange (about 2 us) and by the redundant vector work of a
// step (its reductions over the workgroup).  The operations are those of
// npga_sketch.hip, all in float64.  Measured, all columns: k = 403 4.9 ms by
// launches, 2.25 ms here (5.6 us a column); k = 4096 80 ms by launches, 59.5
// ms here, of which the last 3072 columns 28 ms.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "npga_device.h"
#include "npga_internal.h"
#include "npga_sketch.h"

namespace npga {

namespace {

constexpr int kTriT = 512;  // threads of a workgroup: eight wavefronts
constexpr unsigned long long kTriUnset = 0xFFFFDEAD5EAF0001ull;

struct TriRun {
  int64_t i0;        // first column
  int64_t m;         // order of the trailing matrix: k - i0
  int64_t lds;       // doubles between slots (whole 256-byte lines: a line never holds two steps)
  unsigned long long *p, *x;  // slots of p and of the next row
  unsigned long long *head;   // abort word
  long long ticks;
};

// Sum over the workgroup; every thread gets the same bits.
__device__ __forceinline__ double tri_sum(double v, double (&buf)[2][8], int &par) {
  v = wave_sum_f64(v);
  if ((threadIdx.x & 63) == 0) buf[par][threadIdx.x >> 6] = v;
  __syncthreads();
  double t = buf[par][0];
#pragma unroll
  for (int w = 1; w < 8; ++w) t += buf[par][w];
  par ^= 1;
  return t;
}

// Sums over the wavefront of N (4 or 8) values per lane; lane l returns the
// total of value l N / 64.
template <int N>
__device__ __forceinline__ double wave_reduce_n(double (&t)[N], int lane) {
  int mask = 32;
#pragma unroll
  for (int half = N / 2; half >= 1; half >>= 1) {
    const bool hi = (lane & mask) != 0;
#pragma unroll
    for (int q = 0; q < N / 2; ++q) {
      if (q < half) {
        const double send = hi ? t[q] : t[q + half];
        const double keep = hi ? t[q + half] : t[q];
        t[q] = keep + __shfl_xor(send, mask);
      }
    }
    mask >>= 1;
  }
  double r = t[0];
#pragma unroll
  for (int off = 64 / (2 * N); off > 2; off >>= 1) r += __shfl_xor(r, off);
  r += dpp_f64<0x4E>(r);  // swap pairs
  r += dpp_f64<0xB1>(r);  // swap neighbours
  return r;
}

__device__ __forceinline__ unsigned long long tri_get(const unsigned long long *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void tri_put(unsigned long long *p, double v) {
  __hip_atomic_store(p, (unsigned long long)__double_as_longlong(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace

// Thread t holds columns t + 512 j (j < SL) of its workgroup's rows me + W q
// (q < ROWS); all indices relative to i0.
template <int SL, int ROWS>
__global__ __launch_bounds__(kTriT) void k_tri_chip(SketchState s, TriRun a) {
  __shared__ double vl[SL * kTriT], wl[SL * kTriT];
  __shared__ double sums[2][8], rowsum[8][16];
  __shared__ double x0s;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int W = gridDim.x, me = blockIdx.x, m = (int)a.m;
  const int64_t k = s.k, i0 = a.i0;
  int par = 0;
  double A[ROWS][SL], v[SL];
#pragma unroll
  for (int q = 0; q < ROWS; ++q) {
    const int64_t lr = std::min(me + W * q, m - 1);
#pragma unroll
    for (int j = 0; j < SL; ++j) {
      const int64_t c = std::min(tid + kTriT * j, m - 1);
      A[q][j] = s.A[(i0 + c) + (i0 + lr) * k];
    }
  }
#pragma unroll
  for (int j = 0; j < SL; ++j) {
    const int c = tid + kTriT * j;
    v[j] = (i0 > 0 && c < m) ? s.vcur[i0 + c] : 0.0;
  }
  double tau = i0 > 0 ? s.tau[i0 - 1] : 0.0;

  for (int st = 0; st < m; ++st) {
    const int js = st >> 9;  // slots below are finished
    const unsigned long long *ps = a.p + (int64_t)st * a.lds, *xs = a.x + (int64_t)st * a.lds;
    unsigned long long pb[SL], xb[SL], pd;
    bool lost = false;
    for (long long t0 = 0;;) {
      pd = tri_get(ps + st);
      bool ok = pd != kTriUnset;
#pragma unroll
      for (int j = 0; j < SL; ++j) {
        if (j < js) continue;
        const int c = std::max(st, std::min(tid + kTriT * j, m - 1));
        pb[j] = tri_get(ps + c);
        xb[j] = tri_get(xs + c);
      }
#pragma unroll
      for (int j = 0; j < SL; ++j)
        if (j >= js) ok = ok && pb[j] != kTriUnset && xb[j] != kTriUnset;
      if (ok) break;
      if (t0 == 0) {
        t0 = wall_clock64();
      } else if (tri_get(a.head) != 0ull || wall_clock64() - t0 >= a.ticks) {
        lost = true;
        break;
      }
    }
    double w[SL], x[SL], dot = 0.0;
#pragma unroll
    for (int j = 0; j < SL; ++j) {
      if (j < js) continue;
      w[j] = __longlong_as_double((long long)pb[j]);
      x[j] = __longlong_as_double((long long)xb[j]);
      const int c = tid + kTriT * j;
      if (c >= st && c < m) dot = fma(w[j], v[j], dot);
    }
    if (lost) dot = __longlong_as_double(0x7FF8000000000000ll);
    const double pv = tri_sum(dot, sums, par);
    if (!(pv == pv)) {  // a wait ran out here (or the data are not numbers): everybody leaves
      if (tid == 0) __hip_atomic_store(a.head, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return;
    }
    const double half = 0.5 * tau * pv;
    const double ws = __longlong_as_double((long long)pd) - half;  // w at row i, where v is 1
    double xn = 0.0;
#pragma unroll
    for (int j = 0; j < SL; ++j) {
      if (j < js) continue;
      const int c = tid + kTriT * j;
      const bool in = c >= st && c < m;
      w[j] = in ? w[j] - half * v[j] : 0.0;
      x[j] = in ? x[j] - (v[j] * ws + w[j]) : 0.0;
      vl[c] = v[j];
      wl[c] = w[j];
      if (c == st && me == 0) s.d[i0 + st] = x[j];
      if (c == st + 1) x0s = x[j];
      if (c >= st + 2) xn = fma(x[j], x[j], xn);
    }
    if (st + 1 == m) break;
    const double xn2 = tri_sum(xn, sums, par);  // its barrier also publishes vl, wl and x0s
    const double x0 = x0s;
    double beta = x0, scale = 0.0;
    tau = 0.0;
    if (xn2 > 0.0) {
      beta = -copysign(sqrt(x0 * x0 + xn2), x0);
      tau = (beta - x0) / beta;
      scale = 1.0 / (x0 - beta);
    }
    double vn[SL];
    const bool writes = me == st % W;
#pragma unroll
    for (int j = 0; j < SL; ++j) {
      if (j < js) {
        vn[j] = 0.0;
        continue;
      }
      const int c = tid + kTriT * j;
      vn[j] = (c == st + 1) ? 1.0 : ((c >= st + 2 && tau != 0.0) ? x[j] * scale : 0.0);
      if (writes && c > st && c < m) s.A[(i0 + c) + (i0 + st) * k] = vn[j];
    }
    if (me == 0 && tid == 0) {
      s.e[i0 + st] = beta;
      s.tau[i0 + st] = tau;
    }
    // own rows, RB at a time: the update, the product with v_i, its sum
    constexpr int RB = ROWS % 8 ? 4 : 8;
#pragma unroll
    for (int q0 = 0; q0 < ROWS; q0 += RB) {
      if (me + W * (q0 + RB - 1) <= st) continue;  // finished rows (their sums are not read)
      double acc[RB];
#pragma unroll
      for (int u = 0; u < RB; ++u) {
        const int q = q0 + u, lr = me + W * q;
        acc[u] = 0.0;
        if (lr <= st || lr >= m) continue;
        const double vr = vl[lr], wr = wl[lr];
#pragma unroll
        for (int j = 0; j < SL; ++j) {
          if (j < js) continue;
          A[q][j] -= vr * w[j] + wr * v[j];
          acc[u] = fma(A[q][j], vn[j], acc[u]);
        }
        if (lr == st + 1) {
          unsigned long long *xo = a.x + (int64_t)(st + 1) * a.lds;
#pragma unroll
          for (int j = 0; j < SL; ++j) {
            const int c = tid + kTriT * j;
            if (j >= js && c > st && c < m) tri_put(xo + c, A[q][j]);
          }
        }
      }
      const double r = wave_reduce_n<RB>(acc, lane);
      if (lane % (64 / RB) == 0) rowsum[wave][q0 + lane / (64 / RB)] = r;
    }
    __syncthreads();
    if (tid < ROWS) {
      const int lr = me + W * tid;
      double t = rowsum[0][tid];
#pragma unroll
      for (int u = 1; u < 8; ++u) t += rowsum[u][tid];
      if (lr > st && lr < m) tri_put(a.p + (int64_t)(st + 1) * a.lds + lr, tau * t);
    }
#pragma unroll
    for (int j = 0; j < SL; ++j) v[j] = vn[j];
  }
}

// Slots unset but the first (p of the step before and row i0; no step before:
// zeros), the abort word cleared.
__global__ __launch_bounds__(256) void k_tri_slots(SketchState s, TriRun a) {
  const int64_t total = a.m * a.lds;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
    unsigned long long pv = kTriUnset, xv = kTriUnset;
    if (e < a.m) {
      pv = a.i0 > 0 ? (unsigned long long)__double_as_longlong(s.p[a.i0 + e]) : 0ull;
      xv = (unsigned long long)__double_as_longlong(s.A[(a.i0 + e) + a.i0 * s.k]);
    }
    a.p[e] = pv;
    a.x[e] = xv;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) *a.head = 0ull;
}

// One triangle of the trailing matrix copied onto the other, 64 x 64 tiles
// (grid: tiles x tiles); up: the lower onto the upper.
__global__ __launch_bounds__(256) void k_tri_mirror(SketchState s, int64_t i0, int up) {
  if (blockIdx.y < blockIdx.x) return;
  __shared__ double tile[64][65];
  const int64_t k = s.k, r0 = i0 + 64 * (int64_t)blockIdx.y, c0 = i0 + 64 * (int64_t)blockIdx.x;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  for (int q = ty; q < 64; q += 4) {
    // lower tile: rows r0.., columns c0..; upper tile: rows c0.., columns r0..
    const int64_t r = up ? r0 + tx : c0 + tx, c = up ? c0 + q : r0 + q;
    tile[q][tx] = (r < k && c < k) ? s.A[r + c * k] : 0.0;
  }
  __syncthreads();
  for (int q = ty; q < 64; q += 4) {
    const int64_t r = up ? c0 + tx : r0 + tx, c = up ? r0 + q : c0 + q;
    if (r < k && c < k && (up ? r < c : r > c)) s.A[r + c * k] = tile[tx][q];
  }
}

namespace {

struct TriPlan {
  int64_t i0, m;
  int sl, rows, groups;
};

// Registers per thread: SL x ROWS doubles of the matrix, at most 72 of the
// 128 a thread can hold beside a step's vectors; so 512 columns a slot, and
// the rows that 256 workgroups need.
TriPlan tri_plan(int64_t k) {
  TriPlan p{};
  p.m = std::min<int64_t>(k, kTriMax);
  p.i0 = k - p.m;
  p.sl = p.m <= 512 ? 1 : p.m <= 1024 ? 2 : p.m <= 2048 ? 4 : 6;
  p.rows = p.sl == 6 ? 12 : 16;
  p.groups = (int)((p.m + p.rows - 1) / p.rows);
  return p;
}

TriRun tri_run(const TriPlan &p, void *slots) {
  TriRun a{};
  a.i0 = p.i0;
  a.m = p.m;
  a.lds = (p.m + 31) / 32 * 32;
  a.head = static_cast<unsigned long long *>(slots);
  a.p = a.head + 32;
  a.x = a.p + p.m * a.lds;
  return a;
}

int mirror(const SketchState &s, int64_t i0, int up, hipStream_t st) {
  const unsigned t = (unsigned)((s.k - i0 + 63) / 64);
  hipLaunchKernelGGL(k_tri_mirror, dim3(t, t), dim3(256), 0, st, s, i0, up);
  return (int)hipGetLastError();
}

}  // namespace

size_t tri_chip_bytes(int64_t k) {
  const TriPlan p = tri_plan(k);
  return sizeof(double) * (size_t)(32 + 2 * p.m * ((p.m + 31) / 32 * 32));
}

int launch_tridiag_chip(const SketchState &s, void *slots, long long ticks, hipStream_t st) {
  const TriPlan p = tri_plan(s.k);
  TriRun a = tri_run(p, slots);
  a.ticks = ticks;
  if (p.i0 > 0) {
    if (launch_tridiag(s, 0, p.i0, st)) return (int)hipErrorLaunchFailure;
    if (mirror(s, p.i0, 1, st)) return (int)hipErrorLaunchFailure;
  }
  hipLaunchKernelGGL(k_tri_slots, dim3(2048), dim3(256), 0, st, s, a);
  if (hipGetLastError() != hipSuccess) return (int)hipErrorLaunchFailure;
  switch (p.sl) {
    case 1: hipLaunchKernelGGL((k_tri_chip<1, 16>), dim3(p.groups), dim3(kTriT), 0, st, s, a); break;
    case 2: hipLaunchKernelGGL((k_tri_chip<2, 16>), dim3(p.groups), dim3(kTriT), 0, st, s, a); break;
    case 4: hipLaunchKernelGGL((k_tri_chip<4, 16>), dim3(p.groups), dim3(kTriT), 0, st, s, a); break;
    default: hipLaunchKernelGGL((k_tri_chip<6, 12>), dim3(p.groups), dim3(kTriT), 0, st, s, a); break;
  }
  return (int)hipGetLastError();
}

int launch_tridiag_resume(const SketchState &s, hipStream_t st) {
  const TriPlan p = tri_plan(s.k);
  if (mirror(s, p.i0, 0, st)) return (int)hipErrorLaunchFailure;
  return launch_tridiag(s, p.i0, s.k, st);
}

}  // namespace npga
