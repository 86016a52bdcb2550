// A whole phase of a small solve in one launch.
//
// An iteration is a gradient and a serial tail.  For a few hundred assets
// both are a few microseconds of arithmetic, and separate launches spend
// more on starting, draining and re-reading their vectors than on it.  Here
// up to kLoopMaxGroups workgroups stay for the phase:
//   * each wavefront owns items (rows of Sigma on the covariance path,
//     columns of L on the factor path), the first of them held in registers
//     or LDS from the start, the rest streamed;
//   * every workgroup keeps its own copy of the iterate, the gradients and
//     the solver state in LDS and runs the serial tail on it, all of them
//     the same arithmetic on the same numbers, so that an iteration needs
//     one exchange (the gradient's pieces) and no broadcast of the new point;
//   * the exchange has no barrier: words of 8 bytes stored and read at device
//     scope, and a reader waits for the words it needs.  On the covariance
//     path a word is one float and a 32-bit sequence number; a word cannot be
//     overwritten before it is read: a workgroup writes step s + 2's words
//     (same half of the double buffer) only after it has read step s + 1's,
//     which the others write after reading step s's.  On the factor path,
//     where every workgroup reads all the others' vectors, a word is all
//     data, and a word that no arithmetic produces stands for one that has
//     not arrived (fewer words than with a number in each, and one round of
//     looks for 14 to 16 workgroups).
// Bound by latency: the exchange, the tail's reductions and a barrier or two.
// Per NPGA step, a launch per step and one launch: n = 64 on Sigma 12 and 3.8
// us, n = 501 on Sigma 11 and 4.9 us (16 workgroups), n = 1001, T = 403 on L
// 19 and 10.0 us (14 workgroups; CG 11.0); whole solves 3.4 -> 1.25 ms, 4.6 -> 2.0
// ms, 15.2 -> 9.65 ms.  (Waiting before the first look at the others' words, which
// halves a column of the tridiagonalisation, gains nothing here: 1 % at n =
// 501, and a loss on L, where the looks are many and spread.)
// With one workgroup there is no exchange.  Every wait is bounded: after
// LoopArgs::wait_ticks a workgroup raises the abort word and leaves, the others
// follow, the state is that of the last whole iteration, and the host goes
// on with the launch-per-step path.  An estimate that ended so leaves the
// state kStalled, at which the phase after it does not begin, and the host
// starts again with that path.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>

#include "npga_device.h"
#include "npga_internal.h"
#include "npga_tail.h"

namespace npga {

namespace {

// Items of a wavefront kept on the compute unit: on the covariance path in
// registers (32 float4 per lane beside the tails), on the factor path, whose
// gradient accumulators and piece reads need those, in what the vectors
// leave of the LDS.
constexpr int loop_resident(int E, bool symv) { return symv ? 32 / E : (E == 1 ? 16 : E == 2 ? 12 : 4); }

// Words of one workgroup's piece of the factor path's exchange, and ||u||^2.
// A piece is a float64 sum over the workgroup's columns, and no float32
// rounding may come between it and the total: with few pieces, each of many
// columns, it would weigh more than in the launches' sums of four columns
// each.  Up to two entries a thread go as float64; four as their float32
// values, two to a word, and a word of the four remainders in bfloat16 (32
// bits in all).  Error of L L^T x against float64, relative, n = 1001, T =
// 403 / n = 300, T = 1400: the launches 2.0e-8 / 0.9e-8, float32 sums and
// pieces 2.4e-8 / 1.4e-8, float32 pieces alone 2.0e-8 / 0.94e-8, so 1.8e-8 /
// 0.8e-8.  At n = 1001, T = 403 the solve takes 8.9, 9.4 and 9.65 ms.
constexpr int kLoopWords(int E) { return E <= 2 ? E : 3; }
constexpr int kLoopPiece(int E) { return 256 * kLoopWords(E) + 8; }
constexpr unsigned long long kLoopUnset = 0xFFFFDEAD5EAF0001ull;  // (no arithmetic produces these NaN)

enum LoopKind { kLoopSymv = 0, kLoopSweep = 1, kLoopSweep16 = 2 };

__device__ __forceinline__ void put_word(unsigned long long *p, uint32_t value, uint32_t tag) {
  __hip_atomic_store(p, ((unsigned long long)tag << 32) | value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void set_word(unsigned long long *p, unsigned long long v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long get_word(const unsigned long long *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Bounded wait: true when the caller has to give up.
struct Waiter {
  unsigned long long *abort_word;
  uint32_t id;
  long long ticks, t0;
  bool started;
  __device__ __forceinline__ bool give_up() {
    if (!started) {
      started = true;
      t0 = wall_clock64();
      return false;
    }
    if (get_word(abort_word) == id) return true;
    if (wall_clock64() - t0 < ticks) return false;
    __hip_atomic_store(abort_word, (unsigned long long)id, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return true;
  }
};

// A x B words p[i + a_stride a + b_stride b] (a clamped to a_last), all in
// flight at once, until every one carries `tag`; values into out.
template <int A, int B>
__device__ __forceinline__ bool get_words(const unsigned long long *p, uint32_t i, uint32_t a_stride, int a_last,
                                          uint32_t b_stride, uint32_t tag, float (&out)[A][B], Waiter &w) {
  if (w.ticks == 0) return false;  // no time to wait: the first exchange is where it ends
  for (;;) {
    unsigned long long v[A][B];
#pragma unroll
    for (int x = 0; x < A; ++x)
#pragma unroll
      for (int y = 0; y < B; ++y)
        v[x][y] = get_word(p + (i + (uint32_t)(x < a_last ? x : a_last) * a_stride + (uint32_t)y * b_stride));
    uint32_t miss = 0u;
#pragma unroll
    for (int x = 0; x < A; ++x)
#pragma unroll
      for (int y = 0; y < B; ++y) {
        miss |= (uint32_t)(v[x][y] >> 32) ^ tag;
        out[x][y] = __uint_as_float((uint32_t)v[x][y]);
      }
    if (miss == 0u) return true;
    if (w.give_up()) return false;
  }
}

// A x B words p[i + a_stride a + b_stride b] (a clamped to a_last), all in
// flight at once, until none of them is unset.
template <int A, int B>
__device__ __forceinline__ bool get_set_words(const unsigned long long *p, uint32_t i, uint32_t a_stride, int a_last,
                                              uint32_t b_stride, unsigned long long (&v)[A][B], Waiter &w) {
  if (w.ticks == 0) return false;
  for (;;) {
#pragma unroll
    for (int x = 0; x < A; ++x)
#pragma unroll
      for (int y = 0; y < B; ++y)
        v[x][y] = get_word(p + (i + (uint32_t)(x < a_last ? x : a_last) * a_stride + (uint32_t)y * b_stride));
    uint32_t miss = 0u;
#pragma unroll
    for (int x = 0; x < A; ++x)
#pragma unroll
      for (int y = 0; y < B; ++y) miss |= v[x][y] == kLoopUnset ? 1u : 0u;
    if (miss == 0u) return true;
    if (w.give_up()) return false;
  }
}

template <int KIND>
struct LoopElem {
  typedef float type;
};
template <>
struct LoopElem<kLoopSweep16> {
  typedef bf16_t type;
};

// Four consecutive entries of an item (cached loads: the matrix is read
// again in the next iteration).
__device__ __forceinline__ f4 load4(const float *p) { return *reinterpret_cast<const f4 *>(p); }
__device__ __forceinline__ f4 load4(const bf16_t *p) {
  typedef unsigned int u2 __attribute__((ext_vector_type(2)));
  const u2 w = *reinterpret_cast<const u2 *>(p);
  return f4{__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u), __uint_as_float(w.y << 16),
            __uint_as_float(w.y & 0xffff0000u)};
}

}  // namespace

// MODE: the tail (one instantiation per mode, so that each carries its own
// tail's registers only).
template <int E, int KIND, int MODE>
__global__ __launch_bounds__(256, 1) void k_loop(SolveArgs m, LoopArgs la) {
  constexpr int NP = 256 * E;  // padded length of a vector
  constexpr int R = loop_resident(E, KIND == kLoopSymv);
  typedef typename LoopElem<KIND>::type TL;
  __shared__ DevState st;
  __shared__ double vec[8][NP];
  __shared__ __attribute__((aligned(16))) float xs[NP];
  constexpr int CW = E <= 2 ? 4 : 2;  // wavefronts' sums that fit beside the rest
  typedef double d4 __attribute__((ext_vector_type(4)));
  __shared__ __attribute__((aligned(32))) double comb[KIND == kLoopSymv ? 4 : CW * NP];
  __shared__ f4 slab_lds[KIND == kLoopSymv ? 1 : 4 * R * E * 64];
  __shared__ float dsh[KIND == kLoopSymv ? NP : 1];
  __shared__ double redbuf[red_buf_doubles<4>()], mbuf[8], ush[4 + kLoopMaxPieces];
  __shared__ int64_t ibuf[8];
  if (m.st->done != kRunning) {  // (nobody changes it before the first exchange)
    // the phase was over before it began (an estimate that overflowed, a start
    // projection that was not bracketed): the host waits for the code
    if (blockIdx.x == 0 && threadIdx.x == 0 && m.host_done) {
      m.host_done[1] = 0;
      m.host_done[0] = m.st->done;
    }
    return;
  }

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t n = m.n;
  const int W = gridDim.x, me = blockIdx.x;
  const int64_t items = KIND == kLoopSymv ? n : m.cols;
  const int64_t nwv = 4 * (int64_t)W, gw = 4 * (int64_t)me + wave;

  // this workgroup's copies
  SolveArgs a = m;
  {
    const double *src[8] = {m.xbuf0, m.xbuf1, m.gbuf0, m.gbuf1, m.mu, m.pvec, m.fvec, m.gvec};
#pragma unroll
    for (int q = 0; q < 8; ++q)
#pragma unroll
      for (int j = 0; j < E; ++j) {
        const int i = tid + 256 * j;
        vec[q][i] = (src[q] && i < n) ? src[q][i] : 0.0;
      }
#pragma unroll
    for (int j = 0; j < E; ++j) xs[tid + 256 * j] = m.xs[tid + 256 * j];
    const uint32_t *s32 = reinterpret_cast<const uint32_t *>(m.st);
    uint32_t *d32 = reinterpret_cast<uint32_t *>(&st);
    for (int i = tid; i < (int)(sizeof(DevState) / 4); i += 256) d32[i] = s32[i];
  }
  a.st = &st;
  a.xbuf0 = vec[0];
  a.xbuf1 = vec[1];
  a.gbuf0 = vec[2];
  a.gbuf1 = vec[3];
  a.mu = vec[4];
  a.pvec = vec[5];
  a.fvec = vec[6];
  a.gvec = vec[7];
  a.xs = xs;
  a.host_done = nullptr;

  // the resident items; rows n.. of an item read as zeros
  const TL *L = static_cast<const TL *>(la.mat);
  // (an item past the last one reads the last one: its product is dropped)
  uint32_t off[E];
#pragma unroll
  for (int j = 0; j < E; ++j) off[j] = (uint32_t)std::min<int64_t>(4 * lane + 256 * j, la.ld - 4);
  auto load_item = [&](f4(&c)[E], int64_t it) {
    const TL *p = L + (it < items ? it : items - 1) * la.ld;
#pragma unroll
    for (int j = 0; j < E; ++j) c[j] = load4(p + off[j]);
#pragma unroll
    for (int j = E / 2; j < E; ++j) {  // n > 128 E: lower entries are all assets
      const int64_t row0 = 4 * lane + 256 * j;
      c[j].x = (row0 + 0 < n) ? c[j].x : 0.f;
      c[j].y = (row0 + 1 < n) ? c[j].y : 0.f;
      c[j].z = (row0 + 2 < n) ? c[j].z : 0.f;
      c[j].w = (row0 + 3 < n) ? c[j].w : 0.f;
    }
  };
  f4 slab[KIND == kLoopSymv ? R : 1][E];
  if constexpr (KIND == kLoopSymv) {
#pragma unroll
    for (int k = 0; k < R; ++k) load_item(slab[k], gw + k * nwv);
  } else {
    for (int k = 0; k < R; ++k) {
      load_item(slab[0], gw + k * nwv);
#pragma unroll
      for (int j = 0; j < E; ++j) slab_lds[((wave * R + k) * E + j) * 64 + lane] = slab[0][j];
    }
  }
  __syncthreads();

  auto dot_part = [&](const f4(&c)[E], const f4(&x)[E]) {
    float d = 0.f;
#pragma unroll
    for (int j = 0; j < E; ++j) {
      d = fmaf(c[j].x, x[j].x, d);
      d = fmaf(c[j].y, x[j].y, d);
      d = fmaf(c[j].z, x[j].z, d);
      d = fmaf(c[j].w, x[j].w, d);
    }
    return d;
  };
  auto dot = [&](const f4(&c)[E], const f4(&x)[E]) { return wave_sum_f32(dot_part(c, x)); };

  Waiter wait{la.xch, la.seq0 + 1u, la.wait_ticks, 0, false};
  unsigned long long *words = la.xch + 8;
  int s = 0;
  bool stalled = false;
  for (; s < la.steps; ++s) {
    const uint32_t tag = la.seq0 + 1u + (uint32_t)s;
    f4 xr[E];
#pragma unroll
    for (int j = 0; j < E; ++j) xr[j] = *reinterpret_cast<const f4 *>(xs + 4 * lane + 256 * j);
    float sum[E];     // covariance path: (Sigma x)_i of this thread's entries
    double tot[E];    // factor path: (L L^T x)_i
    double usq = -1.0;
    bool bad = false;
    wait.started = false;

    if constexpr (KIND == kLoopSymv) {
      unsigned long long *buf = words + (s & 1) * la.half;
      float mine = 0.f;
#pragma unroll
      for (int k = 0; k < R; ++k) {
        if (k * nwv < items) {
          const float d = dot(slab[k], xr);
          if (lane == k) mine = d;
        }
      }
      const int64_t it = gw + lane * nwv;
      if (lane < R && it < items) {
        if (W == 1)
          dsh[it] = mine;
        else
          put_word(buf + it, __float_as_uint(mine), tag);
      }
      for (int64_t k0 = R; k0 * nwv < items; k0 += 2) {  // streamed items, two in flight
        f4 c0[E], c1[E];
        load_item(c0, gw + k0 * nwv);
        load_item(c1, gw + (k0 + 1) * nwv);
        const float d0 = dot(c0, xr), d1 = dot(c1, xr);
        const int64_t i2 = gw + (k0 + lane) * nwv;
        if (lane < 2 && i2 < items) {
          const float d = lane ? d1 : d0;
          if (W == 1)
            dsh[i2] = d;
          else
            put_word(buf + i2, __float_as_uint(d), tag);
        }
      }
      if (W == 1) {
        __syncthreads();
#pragma unroll
        for (int j = 0; j < E; ++j) sum[j] = dsh[tid + 256 * j];
      } else {
        if (me == 0) {  // the padding, so that a reader needs no bounds
#pragma unroll
          for (int j = E / 2; j < E; ++j)
            if (tid + 256 * j >= n) put_word(buf + tid + 256 * j, 0u, tag);
        }
        float got[1][E];
        bad = !get_words<1, E>(buf, (uint32_t)tid, 0u, 0, 256u, tag, got, wait);
#pragma unroll
        for (int j = 0; j < E; ++j) sum[j] = got[0][j];
      }
    } else {
      d4 g[E];
      double usq_w = 0.0;
#pragma unroll
      for (int j = 0; j < E; ++j) g[j] = d4{0.0, 0.0, 0.0, 0.0};
      // two items at a time: a product is a chain of some fifty dependent
      // instructions.  Their sum leaves float32 (the launches add four
      // columns at least before theirs does).
      auto take2 = [&](const f4(&c0)[E], bool live0, const f4(&c1)[E], bool live1) {
        float d0 = dot_part(c0, xr), d1 = dot_part(c1, xr);
        wave_sum2_f32(d0, d1);
        d0 = live0 ? d0 : 0.f;
        d1 = live1 ? d1 : 0.f;
        usq_w = fma((double)d0, (double)d0, usq_w);
        usq_w = fma((double)d1, (double)d1, usq_w);
#pragma unroll
        for (int j = 0; j < E; ++j) {
          g[j].x += (double)fmaf(c1[j].x, d1, c0[j].x * d0);
          g[j].y += (double)fmaf(c1[j].y, d1, c0[j].y * d0);
          g[j].z += (double)fmaf(c1[j].z, d1, c0[j].z * d0);
          g[j].w += (double)fmaf(c1[j].w, d1, c0[j].w * d0);
        }
      };
      constexpr int F = 4;  // streamed items in flight
      f4 ahead[F][E];
      const bool more = R * nwv < items;
      if (more) {
#pragma unroll
        for (int k = 0; k < F; ++k) load_item(ahead[k], gw + (R + k) * nwv);
      }
      for (int k = 0; k < R && k * nwv < items; k += 2) {
        f4 c[2][E];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int j = 0; j < E; ++j) c[u][j] = slab_lds[((wave * R + k + u) * E + j) * 64 + lane];
        take2(c[0], gw + k * nwv < items, c[1], gw + (k + 1) * nwv < items);
      }
      if (more) {
        for (int64_t k0 = R;;) {
#pragma unroll
          for (int k = 0; k < F; k += 2)
            take2(ahead[k], gw + (k0 + k) * nwv < items, ahead[k + 1], gw + (k0 + k + 1) * nwv < items);
          k0 += F;
          if (k0 * nwv >= items) break;
#pragma unroll
          for (int k = 0; k < F; ++k) load_item(ahead[k], gw + (k0 + k) * nwv);
        }
      }
      if (lane == 0) ush[wave] = usq_w;
      // the wavefronts' sums meet in float64
      double part[E];
      auto sums_at = [&](int w, int j) { return reinterpret_cast<d4 *>(comb + w * NP + 4 * lane + 256 * j); };
      if (wave >= 4 - CW) {
#pragma unroll
        for (int j = 0; j < E; ++j) *sums_at(wave - (4 - CW), j) = g[j];
      }
      __syncthreads();
      if constexpr (CW == 2) {
        if (wave < 2) {
#pragma unroll
          for (int j = 0; j < E; ++j) *sums_at(wave, j) += g[j];
        }
        __syncthreads();
      }
#pragma unroll
      for (int j = 0; j < E; ++j) {
        const double *cf = comb + tid + 256 * j;
        part[j] = CW == 2 ? cf[0] + cf[NP] : (cf[0] + cf[NP]) + (cf[2 * NP % (CW * NP)] + cf[3 * NP % (CW * NP)]);
      }
      const double up = ((ush[0] + ush[1]) + ush[2]) + ush[3];
      usq = up;
      if (W == 1) {
#pragma unroll
        for (int j = 0; j < E; ++j) tot[j] = part[j];
      } else {
        // W pieces.  Three buffers in turn; a step's word is unset again
        // two steps before its next use, when every reader has shown (by its
        // own next piece) that it is done with it, and before this thread's
        // next piece, which a reader of the new word has to see first.
        constexpr int PQ = kLoopWords(E);
        unsigned long long *buf = words + (uint32_t)(s % 3) * (uint32_t)(W * kLoopPiece(E));
        unsigned long long *own = buf + (uint32_t)me * (uint32_t)kLoopPiece(E);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if constexpr (E <= 2) {
#pragma unroll
          for (int j = 0; j < E; ++j) set_word(own + tid + 256 * j, (unsigned long long)__double_as_longlong(part[j]));
        } else {
          unsigned long long w[3] = {0ull, 0ull, 0ull};
#pragma unroll
          for (int j = 0; j < E; ++j) {
            const float hi = (float)part[j];
            const float lo = isfinite(hi) ? (float)(part[j] - (double)hi) : 0.f;
            w[j / 2] |= (unsigned long long)__float_as_uint(hi) << (32 * (j % 2));
            w[2] |= (unsigned long long)(__float_as_uint(lo) >> 16) << (16 * j);
          }
#pragma unroll
          for (int j = 0; j < PQ; ++j) set_word(own + tid + 256 * j, w[j]);
        }
        // ||u||^2 enters the objective of a stopping test only
        const bool wants_usq = MODE == kTailNpga && st.iter % st.check_every == 0;
        if (wants_usq && tid == 0) set_word(own + 256 * PQ, (unsigned long long)__double_as_longlong(up));
#pragma unroll
        for (int j = 0; j < E; ++j) tot[j] = 0.0;
        float rest[E];  // (E = 4: the remainders)
#pragma unroll
        for (int j = 0; j < E; ++j) rest[j] = 0.f;
        // G pieces in flight, added in order; past the last, the last again.
        // The remainders are asked for when the values are there, and arrive
        // while those are added.
        auto pieces = [&](auto g_c, int w0) {
          constexpr int G = decltype(g_c)::value, VQ = E <= 2 ? PQ : PQ - 1;
          unsigned long long v[G][VQ];
          const unsigned long long *from = buf + (uint32_t)w0 * (uint32_t)kLoopPiece(E);
          bad = !get_set_words<G, VQ>(from, (uint32_t)tid, (uint32_t)kLoopPiece(E), W - 1 - w0, 256u, v, wait);
          unsigned long long r[E <= 2 ? 1 : G][1];
          if constexpr (E > 2) {
#pragma unroll
            for (int x = 0; x < G; ++x) {
              const int xc = x < W - 1 - w0 ? x : W - 1 - w0;
              r[x][0] = get_word(from + (tid + 256 * VQ + (uint32_t)xc * (uint32_t)kLoopPiece(E)));
            }
            __builtin_amdgcn_sched_barrier(0);
          }
#pragma unroll
          for (int x = 0; x < G; ++x) {
            const uint32_t keep = w0 + x < W ? 0xffffffffu : 0u;
#pragma unroll
            for (int j = 0; j < E; ++j) {
              if constexpr (E <= 2)
                tot[j] += __longlong_as_double((long long)(v[x][j] & (((unsigned long long)keep << 32) | keep)));
              else
                tot[j] += (double)__uint_as_float((uint32_t)(v[x][j / 2] >> (32 * (j % 2))) & keep);
            }
          }
          if constexpr (E > 2) {
            uint32_t miss = 0u;
#pragma unroll
            for (int x = 0; x < G; ++x) miss |= r[x][0] == kLoopUnset ? 1u : 0u;
            if (miss && !bad)
              bad = !get_set_words<G, 1>(from, (uint32_t)tid + 256u * VQ, (uint32_t)kLoopPiece(E), W - 1 - w0, 0u, r, wait);
#pragma unroll
            for (int x = 0; x < G; ++x) {
              const uint32_t keep = w0 + x < W ? 0xffffffffu : 0u;
#pragma unroll
              for (int j = 0; j < E; ++j) {
                const uint32_t lo = (uint32_t)(r[x][0] >> (32 * (j / 2)));
                rest[j] += __uint_as_float((j % 2 ? lo & 0xffff0000u : lo << 16) & keep);
              }
            }
          }
        };
        // (16 pieces with remainders in flight cost register copies: n = 1001,
        // 14 workgroups, 10.0 ms a solve by rounds of 16, 12, 8 and 4, 9.65 so)
        constexpr int GM = E > 2 ? 14 : 16;
        for (int w0 = 0; w0 < W && !bad; w0 += GM) {
          const int left = W - w0;
          if (left > 14)
            pieces(std::integral_constant<int, GM>{}, w0);
          else if (left > 12)
            pieces(std::integral_constant<int, 14>{}, w0);
          else if (left > 10)
            pieces(std::integral_constant<int, 12>{}, w0);
          else if (left > 8)
            pieces(std::integral_constant<int, 10>{}, w0);
          else if (left > 6)
            pieces(std::integral_constant<int, 8>{}, w0);
          else if (left > 4)
            pieces(std::integral_constant<int, 6>{}, w0);
          else if (left > 2)
            pieces(std::integral_constant<int, 4>{}, w0);
          else
            pieces(std::integral_constant<int, 2>{}, w0);
        }
        if constexpr (E > 2) {
#pragma unroll
          for (int j = 0; j < E; ++j) tot[j] += (double)rest[j];
        }
        if (wants_usq && tid < W && !bad) {
          unsigned long long v[1][1];
          bad = !get_set_words<1, 1>(buf, (uint32_t)(tid * kLoopPiece(E) + 256 * PQ), 0u, 0, 0u, v, wait);
          ush[4 + tid] = __longlong_as_double((long long)v[0][0]);
        }
        if (!bad) {  // the step before's words
          unsigned long long *old = words + ((uint32_t)((s + 2) % 3) * (uint32_t)W + (uint32_t)me) * (uint32_t)kLoopPiece(E);
#pragma unroll
          for (int j = 0; j < PQ; ++j) set_word(old + tid + 256 * j, kLoopUnset);
          if (tid == 0) set_word(old + 256 * PQ, kLoopUnset);
        }
      }
    }
    if (W > 1) {
      if (__syncthreads_or(bad ? 1 : 0)) {
        stalled = true;
        break;
      }
      if constexpr (KIND != kLoopSymv && MODE == kTailNpga) {
        usq = ush[4];
        for (int w = 1; w < W; ++w) usq += ush[4 + w];
      }
    }

    // the gradient of this thread's entries, as the reduce launches form it
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const int64_t i = tid + 256 * j;
      if (i >= n) continue;
      const double d = KIND == kLoopSymv ? (double)sum[j] : tot[j];
      if constexpr (MODE == kTailNpga)
        npga_store_grad_step(a, &st, i, 2.0 * d + (a.ga ? a.ga[i] : 0.0) + 2.0 * st.gamma * vec[st.iter & 1][i]);
      else if constexpr (MODE == kTailLanczos)
        vec[2][i] = d;
      else
        vec[2][i] = 2.0 * d + 2.0 * st.gamma * vec[5][i];
    }
    if constexpr (MODE == kTailNpga)
      tail_npga<E>(a, usq, redbuf);
    else if constexpr (MODE == kTailLanczos)
      tail_lanczos<E>(a, redbuf);
    else if constexpr (MODE == kTailCG)
      tail_cg<E>(a, redbuf, mbuf, ibuf);
    else
      tail_pdas<E>(a, redbuf);
    __syncthreads();
    if (st.done != kRunning) {
      ++s;
      break;
    }
  }

  if (me != 0) return;
  // the first workgroup's copies are the result
  if constexpr (MODE == kTailLanczos) {
    if (stalled) {  // the iterations cannot start from an unfinished estimate
      if (tid == 0) st.done = kStalled;
      __syncthreads();
    }
  }
  double *dst[8] = {m.xbuf0, m.xbuf1, m.gbuf0, m.gbuf1, nullptr, m.pvec, m.fvec, m.gvec};
#pragma unroll
  for (int q = 0; q < 8; ++q)
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const int i = tid + 256 * j;
      if (dst[q] && i < n) dst[q][i] = vec[q][i];
    }
#pragma unroll
  for (int j = 0; j < E; ++j) m.xs[tid + 256 * j] = xs[tid + 256 * j];
  const uint32_t *s32 = reinterpret_cast<const uint32_t *>(&st);
  uint32_t *d32 = reinterpret_cast<uint32_t *>(m.st);
  for (int i = tid; i < (int)(sizeof(DevState) / 4); i += 256) d32[i] = s32[i];
  if (tid == 0 && m.host_done) {
    m.host_done[1] = stalled ? -1 : s;
    m.host_done[0] = st.done;
  }
}

// The factor path's words before a launch.
__global__ __launch_bounds__(256) void k_loop_unset(unsigned long long *p, int64_t words) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < words; i += (int64_t)gridDim.x * 256) p[i] = kLoopUnset;
}

// Columns of L up to which a step of the loop takes no longer than one by
// launches, for the entries a thread has.  A step by launches takes 13 to 14
// us whatever the shape (17 on a host that launches more slowly), the loop's
// grows with the columns of a wavefront.  Measured, us a step, float32 /
// bfloat16: n = 256 12.8 / 13.3 at 8000 columns, 14.7 / 15.3 at 10000; n = 512
// 12.8 / 13.2 at 4000, 14.4 / 15.0 at 5000; n = 1000 12.4 / 15.0 at 1000 (17 by
// launches there), 13.7 / 16.5 at 1200, 15.4 / 18.6 at 2000.
constexpr int64_t kLoopMaxCols(int E) { return E == 1 ? 8192 : E == 2 ? 4096 : 1024; }

// Workgroups of the loop for a shape (0: the launch-per-step path).  One
// workgroup when it holds all the items (its products then take about the
// time of an exchange).  Beyond, eight rows of Sigma a wavefront (n = 2000:
// 10.1 us a step by 63 workgroups, 13.2 by 32, 12.6 by launches; n = 1000: 5.8
// by 32, 9.6 by 16); on the factor path, where every workgroup reads all the
// others' n-vectors, as many as balance that against the columns a workgroup
// works through, or as hold all the columns (n = 1001, T = 403: 14 workgroups
// 9.65 ms a solve, 16 10.7, 12 10.4, 10 10.0, 8 10.9), and at most
// kLoopMaxPieces (n = 300, T = 4000: 12.7 us a step by 32, 12.5 by 45, 17.6 by
// 16).
LoopPlan loop_plan(int64_t n, int64_t cols, int path, int dtype) {
  LoopPlan p{};
  const int e = slots_for(n);
  const bool symv = path == NPGA_PATH_SYRK;
  if (e < 1 || e > (symv ? 8 : 4) || (!symv && cols > kLoopMaxCols(e))) return p;
  const int64_t items = symv ? n : cols;
  const int64_t esz = dtype == NPGA_BF16 ? 2 : 4;
  const int64_t held = 4 * loop_resident(e, symv);
  int64_t w = 1;
  if (items > held) {
    const int64_t balance = std::lround(std::sqrt((double)(cols * esz) / 8.0));
    w = symv ? (items + 31) / 32 : std::max<int64_t>(2, std::min<int64_t>((items + held - 1) / held, balance));
    w = std::min<int64_t>(w, symv ? kLoopMaxGroups : kLoopMaxPieces);
  }
  p.groups = (int)w;
  p.half = w == 1 ? 0 : (symv ? (int64_t)256 * e : (3 * w * kLoopPiece(e) + 1) / 2);
  return p;
}

template <int E, int KIND>
static void launch_loop_mode(const SolveArgs &a, const LoopArgs &la, int groups, hipStream_t s) {
  switch (a.mode) {
    case kTailNpga: hipLaunchKernelGGL((k_loop<E, KIND, kTailNpga>), dim3(groups), dim3(256), 0, s, a, la); break;
    case kTailCG: hipLaunchKernelGGL((k_loop<E, KIND, kTailCG>), dim3(groups), dim3(256), 0, s, a, la); break;
    case kTailPdas: hipLaunchKernelGGL((k_loop<E, KIND, kTailPdas>), dim3(groups), dim3(256), 0, s, a, la); break;
    default: hipLaunchKernelGGL((k_loop<E, KIND, kTailLanczos>), dim3(groups), dim3(256), 0, s, a, la); break;
  }
}

// (the factor path's kernels for eight entries per thread do not fit the
// register file)
template <int E>
static void launch_loop_kind(const SolveArgs &a, const LoopArgs &la, int groups, int path, hipStream_t s) {
  if (path == NPGA_PATH_SYRK)
    launch_loop_mode<E, kLoopSymv>(a, la, groups, s);
  else if constexpr (E <= 4) {
    if (a.dtype == NPGA_BF16)
      launch_loop_mode<E, kLoopSweep16>(a, la, groups, s);
    else
      launch_loop_mode<E, kLoopSweep>(a, la, groups, s);
  }
}

int launch_loop(const SolveArgs &a, const LoopArgs &la, int groups, int slots, int path, hipStream_t s) {
  if (groups < 1 || groups > (path == NPGA_PATH_SYRK ? kLoopMaxGroups : kLoopMaxPieces) || a.dykstra || a.backtrack || a.pre_y ||
      (a.mode != kTailNpga && a.mode != kTailCG && a.mode != kTailPdas && a.mode != kTailLanczos))
    return (int)hipErrorInvalidValue;
  if (path != NPGA_PATH_SYRK && groups > 1)
    hipLaunchKernelGGL(k_loop_unset, dim3(64), dim3(256), 0, s, la.xch + 8, 2 * la.half);
  switch (slots) {
    case 1: launch_loop_kind<1>(a, la, groups, path, s); break;
    case 2: launch_loop_kind<2>(a, la, groups, path, s); break;
    case 4: launch_loop_kind<4>(a, la, groups, path, s); break;
    case 8: launch_loop_kind<8>(a, la, groups, path, s); break;
    default: return (int)hipErrorInvalidValue;
  }
  return (int)hipGetLastError();
}

}  // namespace npga
