// Householder tridiagonalisation with the matrix held on the chip.
//
// A reflector needs the product of the whole trailing matrix with the
// reflector before it, so the columns are a serial chain; with a launch per
// stage of a step (npga_sketch.hip) a column costs a read and a write of the
// trailing matrix and three launches.  Here up to 256 workgroups hold the
// last kTriMax columns' trailing matrix, whole rows (both triangles) dealt out
// cyclically: in registers up to order 2048, five rows of a workgroup's
// fourteen in LDS up to 3584, two rows more and the first columns in memory up
// to 4096.  The chain of an order is one launch, which goes on in a launch of
// the next smaller kind when what is left fits that:
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
// upper triangle (or what the launch before left) still holds the trailing
// matrix, and the caller goes on with a launch per stage.  A stream whose
// compute units do not hold a launch's workgroups together takes those
// launches at once (tri_chip_fits), and the streams of a process take turns
// (ChipTurn).
//
// The operations are those of npga_sketch.hip, all in float64.  Bound by a
// step's latency: the exchange (about 1.2 us) and three sums over the
// workgroup, one after the other.  Measured, us a column: 2.2 up to order
// 512, 2.3 to 1024, 2.9 to 2048, 5.6 from 3584 to 2048 (the registers do not
// hold those, and some rows stand in LDS), 17 from 4096 to 3584 (a quarter
// of the elements stands in memory); by launches 12 at order 403 and 16 to 33
// at 2048 to 4096.  Without the wait before the first look at the slots (kNap)
// the same columns took 3.9, 4.5, 5.0 and 7.7.  All columns of a k = 403
// sketch: 4.9 ms by launches, 0.87 ms here; k = 4096: 80 ms and 23 ms.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <mutex>
#include <type_traits>

#include "npga_device.h"
#include "npga_internal.h"
#include "npga_sketch.h"

namespace npga {

namespace {

constexpr int kTriT = 512;  // threads of a workgroup: eight wavefronts
constexpr unsigned long long kTriUnset = 0xFFFFDEAD5EAF0001ull;

// One launch: the first n columns of a symmetric matrix of order m that
// stands at row and column i0 of the whole.
struct TriRun {
  int64_t i0, m, n;
  const double *src;  // its rows (m of them, lsrc apart)
  int64_t lsrc;
  const double *p0, *v0;  // p and v of the column before (i0 > 0)
  unsigned long long *p, *x;  // slots of p and of the next row, one for each column
  int64_t lds;  // words between slots (a multiple of 32: no 256-byte line holds two columns' words)
  double *edge;  // the elements that have no place on the chip (kTriEdge each thread)
  double *rest, *vrest;  // n < m: the trailing matrix of order m - n and its v afterwards
  unsigned long long *head;  // abort word: 0, or 1 + the number of the launch that gave up
  unsigned long long stage;
  long long ticks;
};

constexpr int kTriEdge = 30;  // two rows of eight slots, slot 0 of fourteen

// Sum over the workgroup; every thread gets the same bits.  buf: its own
// eight words for each of a step's sums, so one barrier is enough.
__device__ __forceinline__ double tri_sum(double v, double *buf) {
  v = wave_sum_f64(v);
  if ((threadIdx.x & 63) == 0) buf[threadIdx.x >> 6] = v;
  __syncthreads();
  return ((buf[0] + buf[1]) + (buf[2] + buf[3])) + ((buf[4] + buf[5]) + (buf[6] + buf[7]));
}

__device__ __forceinline__ unsigned long long tri_get(const unsigned long long *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// p plus off bytes
__device__ __forceinline__ const unsigned long long *tri_at(const unsigned long long *p, unsigned off) {
  return reinterpret_cast<const unsigned long long *>(reinterpret_cast<const char *>(p) + off);
}
__device__ __forceinline__ unsigned long long *tri_at(unsigned long long *p, unsigned off) {
  return reinterpret_cast<unsigned long long *>(reinterpret_cast<char *>(p) + off);
}
__device__ __forceinline__ void tri_put(unsigned long long *p, double v) {
  __hip_atomic_store(p, (unsigned long long)__double_as_longlong(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace

// Thread t holds columns t + 512 j (j < SL) of its workgroup's rows me + W q
// (q < LR + RR), W a power of two up to 256; all indices relative to i0.  The
// first LR rows, which are finished first, stand in LDS, the others in
// registers.  A loop for each 512 columns: slots and rows that are finished
// before it begins are left out of it.
//
// EDGE (orders above 3584, up to 512 columns of it): slot 0 and the first two
// rows stay in memory, kTriEdge doubles a thread, read and written once a
// step (31 MB over the chip); all of them are finished when 3584 are left.
template <int SL, int RR, int LR, int W, int JEND, bool EDGE = false>
__global__ __launch_bounds__(kTriT) void k_tri_chip(SketchState s, TriRun a) {
  constexpr int QB = EDGE ? 2 : 0, JB = EDGE ? 1 : 0, SC = SL - JB;  // first row and slot on the chip, slots
  constexpr int ROWS = RR + LR + QB;
  constexpr int ROWS4 = (ROWS + 3) / 4 * 4;
  // x 64 clocks, see below; the best of 12 to 40, flat within 2 around it
  constexpr int kNap = SL <= 2 ? 13 : SL == 4 ? 16 : 18;
  static_assert(!EDGE || (W == 256 && ROWS == 16 && JEND == 1), "");
  extern __shared__ double alds[];  // LR x SC x 512
  __shared__ double sums[2][8], rowsum[ROWS4][8];
  __shared__ double2 own[ROWS4];  // v and w at the own rows
  __shared__ double pds, x0s;
  int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int me = blockIdx.x, m = (int)a.m;
  const int64_t k = s.k, i0 = a.i0;
  if (__syncthreads_or(tri_get(a.head) != 0ull)) return;
  double A[RR][SC], v[SL];
  double *em = EDGE ? a.edge + (int64_t)me * kTriEdge * kTriT : nullptr;
  auto in_memory = [](int q, int j) { return EDGE && (q < QB || j < JB); };
  auto memory_at = [](int q, int j) { return (q < QB ? q * SL + j : QB * SL + q - QB) * kTriT; };
  auto lds_at = [](int q, int j) { return ((q - QB) * SC + j - JB) * kTriT; };
  // element (q, j); the indexes are constants wherever it is used
  auto get = [&](int q, int j) __attribute__((always_inline)) -> double {
    if (in_memory(q, j)) return em[memory_at(q, j) + (unsigned)tid];
    if (q - QB < LR) return alds[lds_at(q, j) + tid];
    return A[q - QB < LR ? 0 : q - QB - LR][j < JB ? 0 : j - JB];
  };
  auto put = [&](int q, int j, double e) __attribute__((always_inline)) {
    if (in_memory(q, j)) em[memory_at(q, j) + (unsigned)tid] = e;
    else if (q - QB < LR) alds[lds_at(q, j) + tid] = e;
    else A[q - QB < LR ? 0 : q - QB - LR][j < JB ? 0 : j - JB] = e;
  };
#pragma unroll
  for (int q = 0; q < ROWS; ++q) {
    const double *row = a.src + std::min(me + W * q, m - 1) * a.lsrc;
    asm volatile("" : "+v"(tid));
#pragma unroll
    for (int j = 0; j < SL; ++j) {
      put(q, j, row[(unsigned)std::min(tid + kTriT * j, m - 1)]);
    }
  }
  if (tid < ROWS4) own[tid] = double2{0.0, 0.0};
#pragma unroll
  for (int j = 0; j < SL; ++j) {
    const int c = tid + kTriT * j;
    v[j] = (i0 > 0 && c < m) ? a.v0[c] : 0.0;
  }
  double tau = i0 > 0 ? s.tau[i0 - 1] : 0.0;
  __syncthreads();                          // own

  // columns 512 JS .. 512 JS + 511
  auto columns = [&](auto js_) __attribute__((always_inline)) {
    constexpr int JS = decltype(js_)::value;
    constexpr int Q0 = kTriT / W * JS / 4 * 4;  // rows below are finished
    const int end = std::min((int)a.n, kTriT * (JS + 1));
    for (int st = kTriT * JS; st < end; ++st) {
      // nothing derived from tid is worth a register for longer than a step
      asm volatile("" : "+v"(tid));
      const unsigned long long *ps = a.p + (int64_t)st * a.lds, *xs = a.x + (int64_t)st * a.lds;
      unsigned long long pb[SL], xb[SL];
      bool lost = st > 0 && a.ticks == 0;  // no time to wait: the first exchange is where it ends
      // A look that comes too early costs a round trip and holds up the words
      // on their way, so the first one is made when they are due.
      __builtin_amdgcn_s_sleep(kNap);
      for (long long t0 = 0;;) {  // (a lost wait looks once more, and leaves)
        unsigned off = (unsigned)tid * 8u;
        asm volatile("" : "+v"(off));  // keeps the addresses out of registers
#pragma unroll
        for (int j = JS; j < SL; ++j) {
          pb[j] = tri_get(tri_at(ps + kTriT * j, off));
          xb[j] = tri_get(tri_at(xs + kTriT * j, off));
        }
        unsigned wait = 0;
#pragma unroll
        for (int j = JS; j < SL; ++j) {
          const int c = tid + kTriT * j;
          wait |= (unsigned)(c >= st) & (unsigned)(c < m) & ((unsigned)(pb[j] == kTriUnset) | (unsigned)(xb[j] == kTriUnset));
        }
        if (lost || !__any((int)wait)) break;
        if (t0 == 0) {
          t0 = wall_clock64();
        } else if (tri_get(a.head) != 0ull || wall_clock64() - t0 >= a.ticks) {
          lost = true;
          break;
        }
      }
      double w[SL], x[SL], dot = lost ? __longlong_as_double(0x7FF8000000000000ll) : 0.0;
#pragma unroll
      for (int j = JS; j < SL; ++j) {
        const int c = tid + kTriT * j;
        w[j] = __longlong_as_double((long long)pb[j]);
        x[j] = __longlong_as_double((long long)xb[j]);
        if (j == JS && c == st) pds = w[j];
        dot = fma((c >= st && c < m) ? w[j] : 0.0, v[j], dot);
      }
      const double pv = tri_sum(dot, sums[0]);  // its barrier also publishes pds
      if (__builtin_amdgcn_readfirstlane(!(pv == pv))) {  // a wait ran out here (or the data are not numbers): everybody leaves
        if (tid == 0) __hip_atomic_store(a.head, 1 + a.stage, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_endpgm();  // (a return would have the matrix live on both ways)
      }
      const double half = 0.5 * tau * pv;
      const double ws = pds - half;  // w at row i, where v is 1
      double xn = 0.0;
#pragma unroll
      for (int j = JS; j < SL; ++j) {
        const int c = tid + kTriT * j;
        const bool in = c >= st && c < m;
        w[j] = in ? w[j] - half * v[j] : 0.0;
        x[j] = in ? x[j] - (v[j] * ws + w[j]) : 0.0;
        if ((tid & (W - 1)) == me) {  // a column of an own row
          const int q = tid / W + kTriT / W * j;
          if (q < ROWS) own[q] = double2{v[j], w[j]};
        }
        if (j == JS && c == st && me == 0) s.d[i0 + st] = x[j];
        if (j <= JS + 1 && c == st + 1) x0s = x[j];
        const double xt = c >= st + 2 ? x[j] : 0.0;
        xn = fma(xt, xt, xn);
      }
      if (st + 1 == m) __builtin_amdgcn_endpgm();
      const double xn2 = tri_sum(xn, sums[1]);  // its barrier also publishes own and x0s
      const double x0 = x0s;
      const bool refl = xn2 > 0.0;
      const double nrm = -copysign(sqrt(x0 * x0 + xn2), x0);
      const double beta = refl ? nrm : x0;
      tau = refl ? (nrm - x0) / nrm : 0.0;
      const double scale = refl ? 1.0 / (x0 - nrm) : 0.0;
#pragma unroll
      for (int j = JS; j < SL; ++j) {  // v_i
        const int c = tid + kTriT * j;
        x[j] = (c == st + 1) ? 1.0 : ((c >= st + 2 && refl) ? x[j] * scale : 0.0);
      }
      if (me == st % W) {
        double *vo = s.A + i0 + (i0 + st) * k;
#pragma unroll
        for (int j = JS; j < SL; ++j) {
          const int c = tid + kTriT * j;
          if (c > st && c < m) vo[kTriT * j + (unsigned)tid] = x[j];
        }
      }
      if (me == 0 && tid == 0) {
        s.e[i0 + st] = beta;
        s.tau[i0 + st] = tau;
      }
      // own rows, four at a time: the update, the product with v_i, its sum.
      // (Rows that are finished or beyond m are carried along; nothing reads
      // them.)  What stands in memory is asked for some groups ahead; the two
      // rows there come last.
      double m0[EDGE ? ROWS - QB : 1], mr[1][EDGE ? SL : 1];
      if constexpr (EDGE) {
#pragma unroll
        for (int q = QB; q < QB + 4; ++q) m0[q - QB] = get(q, 0);
      }
#pragma unroll
      for (int q0 = Q0; q0 < ROWS; q0 += 4) {
        if constexpr (EDGE) {
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int q = q0 + QB + 4; q < q0 + QB + 8 && q < ROWS; ++q) m0[q - QB] = get(q, 0);
          if (q0 == 12) {
#pragma unroll
            for (int j = 0; j < SL; ++j) mr[0][j] = get(0, j);
          }
        }
        double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int q = EDGE ? (q0 + u + QB) % ROWS : q0 + u;
          if (q >= ROWS) continue;
          // (two rows' loads from LDS in flight: more cost registers)
          if (LR > 0 && u % 2 == 0) __builtin_amdgcn_sched_barrier(0);
          const double2 vw = own[q];
#pragma unroll
          for (int j = JS; j < SL; ++j) {
            double e;
            if constexpr (EDGE)
              e = q == 0 ? mr[0][j] : (j < JB && q >= QB) ? m0[q < QB ? 0 : q - QB] : get(q, j);
            else
              e = get(q, j);
            e -= vw.x * w[j] + vw.y * v[j];
            put(q, j, e);
            acc[u] = fma(e, x[j], acc[u]);
          }
        }
        const double r = wave_sum4_f64(acc[0], acc[1], acc[2], acc[3]);
        const int qr = EDGE ? (q0 + (lane >> 4) + QB) % ROWS : q0 + (lane >> 4);
        if ((lane & 15) == 0) rowsum[qr][wave] = r;
      }
      if (me == (st + 1) % W) {  // row st + 1 goes out
        const int qs = (st + 1) / W;
        unsigned long long *xo = a.x + (int64_t)(st + 1) * a.lds;
        unsigned off = (unsigned)tid * 8u;
        asm volatile("" : "+v"(off)::"memory");  // what stands in LDS is read from there again
#pragma unroll
        for (int q = Q0; q < (EDGE ? QB : ROWS); ++q) {  // (EDGE: row 512, the next launch's first, is in `rest`)
          if (q != qs) continue;
#pragma unroll
          for (int j = JS; j < SL; ++j) {
            const int c = tid + kTriT * j;
            const double e = get(q, j);
            if (c > st && c < m) tri_put(tri_at(xo + kTriT * j, off), e);
          }
        }
      }
      __syncthreads();
      if (tid < 8 * ROWS4) {
        const int q = tid >> 3, lr = me + W * q;
        double t = rowsum[q][tid & 7];
        t += dpp_f64<0x141>(t);  // mirror the half row (lanes 7 - l)
        t += dpp_f64<0x4E>(t);
        t += dpp_f64<0xB1>(t);
        if ((tid & 7) == 0 && q < ROWS && lr > st && lr < m) tri_put(a.p + (int64_t)(st + 1) * a.lds + lr, tau * t);
      }
#pragma unroll
      for (int j = JS; j < SL; ++j) v[j] = x[j];
    }
  };
  columns(std::integral_constant<int, 0>{});
  if constexpr (JEND > 1) columns(std::integral_constant<int, 1>{});
  if constexpr (JEND > 2) columns(std::integral_constant<int, 2>{});
  if constexpr (JEND > 3) columns(std::integral_constant<int, 3>{});
  if constexpr (JEND < SL) {
    const int n = (int)a.n;
    const int64_t mr = m - n;
#pragma unroll
    for (int j = 0; j < SL; ++j) {
      const int c = tid + kTriT * j;
      if (c < n || c >= m) continue;
      if (me == 0) a.vrest[c - n] = v[j];
#pragma unroll
      for (int q = 0; q < ROWS; ++q) {
        const int lr = me + W * q;
        if (lr >= n && lr < m)
          a.rest[(c - n) + (lr - n) * mr] = get(q, j);
      }
    }
  }
}

// Slots unset but the first (p of the column before and row i0; no column
// before: zeros), the abort word cleared before the first launch.
__global__ __launch_bounds__(256) void k_tri_slots(TriRun a) {
  const int64_t total = (a.n + (a.n < a.m ? 1 : 0)) * a.lds;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
    unsigned long long pv = kTriUnset, xv = kTriUnset;
    if (e < a.m) {
      pv = a.i0 > 0 ? (unsigned long long)__double_as_longlong(a.p0[e]) : 0ull;
      xv = (unsigned long long)__double_as_longlong(a.src[e]);
    }
    a.p[e] = pv;
    a.x[e] = xv;
  }
  if (a.stage == 0 && blockIdx.x == 0 && threadIdx.x == 0) *a.head = 0ull;
}

// The trailing matrix that a launch left, with its p and v, back where a
// launch per stage looks for them.
__global__ __launch_bounds__(256) void k_tri_restore(SketchState s, TriRun a) {
  const int64_t r = blockIdx.x;
  for (int64_t c = threadIdx.x; c <= r; c += 256) s.A[(a.i0 + r) + (a.i0 + c) * s.k] = a.src[c + r * a.lsrc];
  if (threadIdx.x == 0) {
    s.p[a.i0 + r] = a.p0[r];
    s.vcur[a.i0 + r] = a.v0[r];
  }
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

int64_t round32(int64_t v) { return (v + 31) / 32 * 32; }

// The launches for order k.  512 columns a slot, and as few rows to a
// workgroup as 256 workgroups allow (four are summed together).  Above 2048
// the registers do not hold everything and a column takes 6 us against 3, and
// above 3584 not the LDS either (17 us, 33 by launches): as soon as fewer columns are left the
// matrix is dealt out again.
struct TriPlan {
  int launches;
  TriRun run[3];
  int sl[3];
  size_t words;
};

TriPlan tri_plan(const SketchState &s, void *slots, long long ticks) {
  TriPlan p{};
  int64_t m = std::min(s.k, kTriMax), i0 = s.k - m;
  unsigned long long *w = static_cast<unsigned long long *>(slots), *head = w;
  w += 32;
  const double *src = s.A + i0 * (s.k + 1), *p0 = s.p + i0, *v0 = s.vcur + i0;
  int64_t lsrc = s.k;
  for (;;) {
    TriRun &a = p.run[p.launches];
    const int sl = m <= 512 ? 1 : m <= 1024 ? 2 : m <= 2048 ? 4 : m <= 3584 ? 7 : 8;
    p.sl[p.launches] = sl;
    a.i0 = i0;
    a.m = m;
    a.n = sl == 8 ? m - 3584 : sl == 7 ? m - 2048 : m;
    a.src = src;
    a.lsrc = lsrc;
    a.p0 = p0;
    a.v0 = v0;
    a.lds = (int64_t)kTriT * sl;
    a.head = head;
    a.stage = (unsigned long long)p.launches;
    a.ticks = ticks;
    ++p.launches;
    const int64_t steps = a.n + (a.n < m ? 1 : 0), mr = m - a.n;
    a.p = w;
    a.x = w + steps * a.lds;
    w += 2 * steps * a.lds;
    if (sl == 8) {
      a.edge = reinterpret_cast<double *>(w);
      w += (int64_t)256 * kTriEdge * kTriT;
    }
    if (mr == 0) break;
    a.rest = reinterpret_cast<double *>(w);
    a.vrest = a.rest + round32(mr * mr);
    w += round32(mr * mr) + round32(mr);
    src = a.rest;
    lsrc = mr;
    p0 = reinterpret_cast<const double *>(a.p + a.n * (a.lds + 1));
    v0 = a.vrest;
    i0 += a.n;
    m = mr;
  }
  p.words = (size_t)(w - static_cast<unsigned long long *>(slots));
  return p;
}

int mirror(const SketchState &s, int64_t i0, int up, hipStream_t st) {
  const unsigned t = (unsigned)((s.k - i0 + 63) / 64);
  hipLaunchKernelGGL(k_tri_mirror, dim3(t, t), dim3(256), 0, st, s, i0, up);
  return (int)hipGetLastError();
}

}  // namespace

size_t tri_chip_bytes(int64_t k) {
  SketchState s{};
  s.k = k;
  return sizeof(double) * tri_plan(s, nullptr, 0).words;
}

namespace {

struct TriKernel {
  void (*fn)(SketchState, TriRun);
  unsigned groups, lds;
};
TriKernel tri_kernel(int sl, int64_t m) {
  constexpr int kRows7 = 5, kRows8 = 5;  // rows in LDS
  constexpr unsigned row = (unsigned)sizeof(double) * 7 * kTriT;
  switch (sl) {
    case 1: return {k_tri_chip<1, 4, 0, 128, 1>, (unsigned)std::min<int64_t>(128, m), 0};
    case 2: return {k_tri_chip<2, 4, 0, 256, 2>, 256, 0};
    case 4: return {k_tri_chip<4, 8, 0, 256, 4>, 256, 0};
    case 8: return {k_tri_chip<8, 14 - kRows8, kRows8, 256, 1, true>, 256, kRows8 * row};
    default: return {k_tri_chip<7, 14 - kRows7, kRows7, 256, 3>, 256, kRows7 * row};
  }
}

// The launches of two streams do not run side by side: each would hold a part
// of the chip and wait for workgroups that the other keeps from starting.  A
// stream's turn begins when the launches of the turn before it have ended
// (an event the stream waits for; the host does not).
class ChipTurn {
  static constexpr int kDevices = 64;
  static std::mutex lock_;
  static hipEvent_t last_[kDevices];
  std::lock_guard<std::mutex> held_;
  hipStream_t st_;
  int dev_ = -1;

 public:
  explicit ChipTurn(hipStream_t st) : held_(lock_), st_(st) {}
  int begin() {
    int d = 0;
    if (hipGetDevice(&d) != hipSuccess || d < 0 || d >= kDevices) return 1;
    if (last_[d]) {
      if (hipStreamWaitEvent(st_, last_[d], 0) != hipSuccess) return 1;
    } else if (hipEventCreateWithFlags(&last_[d], hipEventDisableTiming | hipEventDisableSystemFence) != hipSuccess) {
      last_[d] = nullptr;
      return 1;
    }
    dev_ = d;
    return 0;
  }
  int end() { return hipEventRecord(last_[dev_], st_) == hipSuccess ? 0 : 1; }
};
std::mutex ChipTurn::lock_;
hipEvent_t ChipTurn::last_[ChipTurn::kDevices] = {};

}  // namespace

bool tri_chip_fits(int64_t k, hipStream_t st) {
  SketchState s{};
  s.k = k;
  const TriPlan p = tri_plan(s, nullptr, 0);
  const int cus = stream_compute_units(st);
  for (int l = 0; l < p.launches; ++l) {
    const TriKernel t = tri_kernel(p.sl[l], p.run[l].m);
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void *>(t.fn), kTriT, t.lds) !=
        hipSuccess) {
      (void)hipGetLastError();
      return false;
    }
    if ((int64_t)per_cu * cus < (int64_t)t.groups) return false;
  }
  return true;
}

int launch_tridiag_chip(const SketchState &s, void *slots, long long ticks, hipStream_t st) {
  const TriPlan p = tri_plan(s, slots, ticks);
  if (p.run[0].i0 > 0) {
    if (launch_tridiag(s, 0, p.run[0].i0, st)) return (int)hipErrorLaunchFailure;
    if (mirror(s, p.run[0].i0, 1, st)) return (int)hipErrorLaunchFailure;
  }
  ChipTurn turn(st);
  if (turn.begin()) return (int)hipErrorUnknown;
  for (int l = 0; l < p.launches; ++l) {
    const TriRun &a = p.run[l];
    hipLaunchKernelGGL(k_tri_slots, dim3(2048), dim3(256), 0, st, a);
    if (hipGetLastError() != hipSuccess) return (int)hipErrorLaunchFailure;
    const TriKernel t = tri_kernel(p.sl[l], a.m);
    hipLaunchKernelGGL(t.fn, dim3(t.groups), dim3(kTriT), t.lds, st, s, a);
    if (hipGetLastError() != hipSuccess) return (int)hipErrorLaunchFailure;
  }
  return turn.end() ? (int)hipErrorUnknown : 0;
}

int launch_tridiag_resume(const SketchState &s, void *slots, uint64_t flag, hipStream_t st) {
  const TriPlan p = tri_plan(s, slots, 0);
  const int l = flag >= 1 && flag <= (uint64_t)p.launches ? (int)flag - 1 : 0;
  const TriRun &a = p.run[l];
  if (l == 0) {
    if (mirror(s, a.i0, 0, st)) return (int)hipErrorLaunchFailure;
  } else {
    hipLaunchKernelGGL(k_tri_restore, dim3((unsigned)a.m), dim3(256), 0, st, s, a);
    if (hipGetLastError() != hipSuccess) return (int)hipErrorLaunchFailure;
  }
  return launch_tridiag(s, a.i0, s.k, st);
}

}  // namespace npga
