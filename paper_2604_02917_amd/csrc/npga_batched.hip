// Batched solves: m targets r_1..r_m on one factor L (points of the
// efficient frontier, Sec. 5), each running Algorithm 1 with its own state.
//
// One iteration of all targets is three launches:
//   k_bgemm_u : U^T = X^T L  (m x T): v_mfma_f32_32x32x2f32 over tiles of
//               periods t x targets j, both operands contiguous along the
//               asset index i (the contraction);
//   k_bgemm_g : P[s] = (L_{:, T_s} U_{T_s, :})^T  (m x n) for the period
//               range T_s of split s: L tiles contiguous along the assets i,
//               U^T tiles contiguous along the targets j;
//   k_btail   : one workgroup per target: g_j = 2 sum_s P[s][j] in a fixed
//               order, the epilogue of its mode (ridge term, anchor, CG
//               direction) and its serial tail (stopping test, momentum,
//               projection; or a face-CG step).
// L is read twice per iteration for all m targets instead of once per
// target, and the arithmetic moves from the vector ALUs to the matrix cores.
// The covariance form (Sigma = L L^T formed once) replaces the GEMM pair by
// one GEMM P[s] = (Sigma[:, K_s] X[K_s, :])^T (k_cov16).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "npga_device.h"
#include "npga_internal.h"
#include "npga_tail.h"

namespace npga {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef unsigned int u2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

const BatchConfig kBatchConfigTable[kBatchConfigs] = {
    {128, 128, 128, 128, 16}, {128, 128, 128, 128, 32}, {64, 128, 128, 128, 32}, {64, 128, 64, 128, 32},
    {128, 64, 128, 64, 16},   {128, 64, 128, 64, 32},   {64, 64, 64, 64, 32},    {64, 64, 128, 64, 64},
    {128, 32, 128, 32, 16},   {128, 32, 128, 32, 32},   {128, 32, 128, 32, 64},  {64, 128, 128, 128, 64},
};

int batch_default_config(int64_t n, int64_t cols, int32_t m) {
  (void)cols;
  // widest target tile that m fills; split count so that the G GEMM has
  // about 2 workgroups per compute unit
  const int bn = m <= 32 ? 32 : (m <= 64 ? 64 : 128);
  const int64_t gt = ((n + 127) / 128) * ((m + bn - 1) / bn);
  const int want = (int)((512 + gt - 1) / gt);
  int best = -1, best_d = 1 << 30;
  for (int c = 0; c < kBatchConfigs; ++c) {
    const BatchConfig &k = kBatchConfigTable[c];
    if (k.u_bn != bn || k.g_bn != bn || k.g_bm != 128 || k.u_bm != 128) continue;
    const int d = k.splits > want ? k.splits - want : want - k.splits;
    if (d < best_d) {
      best_d = d;
      best = c;
    }
  }
  return best < 0 ? 0 : best;
}

// Per-target view of the batch: target j's state and vectors.
__device__ __forceinline__ SolveArgs target_args(const BatchArgs &b, int j) {
  SolveArgs a = b.base;
  const int64_t vs = (int64_t)j * b.vstride;
  const int64_t gs = (int64_t)j * b.gstride;
  a.st = b.base.st + j;
  a.xs = b.base.xs + (int64_t)j * b.ldx;
  a.xbuf0 = b.base.xbuf0 + vs;
  a.xbuf1 = b.base.xbuf1 + vs;
  a.gbuf0 = b.base.gbuf0 + gs;
  a.gbuf1 = b.base.gbuf1 ? b.base.gbuf1 + gs : nullptr;
  a.xa = b.base.xa ? b.base.xa + vs : nullptr;
  a.ga = b.base.ga ? b.base.ga + vs : nullptr;
  a.ua = nullptr;
  if (b.base.pvec) {
    a.pvec = b.base.pvec + vs;
    a.fvec = b.base.fvec + vs;
    a.gvec = b.base.gvec + vs;
  }
  return a;
}

// Four consecutive entries of L kept in their storage format until they are
// written to LDS, so the prefetch of the next tile never waits on its loads.
template <typename TL>
struct Raw4;
template <>
struct Raw4<float> {
  typedef f4 type;
  static __device__ __forceinline__ f4 load(const float *p) { return *reinterpret_cast<const f4 *>(p); }
  static __device__ __forceinline__ f4 zero() { return f4{0.f, 0.f, 0.f, 0.f}; }
  static __device__ __forceinline__ f4 widen(f4 v) { return v; }
};
template <>
struct Raw4<bf16_t> {
  typedef u2v type;
  static __device__ __forceinline__ u2v load(const bf16_t *p) { return *reinterpret_cast<const u2v *>(p); }
  static __device__ __forceinline__ u2v zero() { return u2v{0u, 0u}; }
  static __device__ __forceinline__ f4 widen(u2v w) {
    return f4{__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u), __uint_as_float(w.y << 16),
              __uint_as_float(w.y & 0xffff0000u)};
  }
};

constexpr int KB = 32;       // contraction depth of one LDS stage
constexpr int LDK = KB + 4;  // row length (floats) of contraction-contiguous LDS tiles

// --------------------------------------------------------------------------
// U^T = X^T L.  Tile: BM periods x BN targets; WM x WN wavefronts, each
// PM x PN blocks of 32 x 32.  Lane half h of a wavefront holds contraction
// indices 16h..16h+15 of a stage, read from LDS as four float4, so that MFMA
// step s pairs k = s (lanes 0-31) with k = 16 + s (lanes 32-63) on both
// operands.  Epilogue: U^T and per-tile column sums of U^2 (float64).
// --------------------------------------------------------------------------
template <typename TL, int BM, int BN, int WM, int WN>
__global__ __launch_bounds__(256) void k_bgemm_u(BatchArgs b) {
  constexpr int PM = BM / (32 * WM), PN = BN / (32 * WN);
  constexpr int QA = BM / 32, QB = BN / 32;
  static_assert(WM * WN == 4 && PM >= 1 && PN >= 1, "tile");
  typedef Raw4<TL> R;
  __shared__ float As[2][BM * LDK];
  __shared__ float Bs[2][BN * LDK];
  __shared__ double ush[WM * BN];
  const int64_t T = b.base.cols, n = b.base.n;
  const int m = b.m;
  const int64_t t0 = (int64_t)blockIdx.x * BM;
  const int64_t j0 = (int64_t)blockIdx.y * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = wave / WN, wc = wave % WN;
  const int h = lane >> 5, r = lane & 31;
  const TL *L = static_cast<const TL *>(b.base.L);
  const int64_t ld = b.base.ld;
  const float *X = b.base.xs;
  const int kq = 4 * (tid & 7);
  const int ma = *b.mact;
  if (j0 >= ma) return;
  (void)m;
  const int64_t kbeg = 0, kend = n;
  // targets of this thread's X columns (column c -> target act[c])
  const float *xcol[QB];
#pragma unroll
  for (int q = 0; q < QB; ++q) {
    const int64_t c = j0 + (tid >> 3) + 32 * q;
    xcol[q] = (c < ma) ? X + (int64_t)b.act[c] * b.ldx : nullptr;
  }

  typename R::type ra[QA];
  f4 rb[QB];
  auto gload = [&](int64_t k0) {
    const int64_t k = k0 + kq;
#pragma unroll
    for (int q = 0; q < QA; ++q) {
      const int64_t t = t0 + (tid >> 3) + 32 * q;
      ra[q] = (t < T && k < kend) ? R::load(L + t * ld + k) : R::zero();
    }
#pragma unroll
    for (int q = 0; q < QB; ++q)
      rb[q] = (xcol[q] && k < kend) ? *reinterpret_cast<const f4 *>(xcol[q] + k) : f4{0.f, 0.f, 0.f, 0.f};
  };
  auto sstore = [&](int buf, int64_t k0) {
    const int64_t k = k0 + kq;
#pragma unroll
    for (int q = 0; q < QA; ++q) {
      f4 v = R::widen(ra[q]);
      // rows past n inside the float4 (ld may exceed n): the contraction
      // must not see them
      if (k + 1 >= kend) v.y = 0.f;
      if (k + 2 >= kend) v.z = 0.f;
      if (k + 3 >= kend) v.w = 0.f;
      *reinterpret_cast<f4 *>(&As[buf][((tid >> 3) + 32 * q) * LDK + kq]) = v;
    }
#pragma unroll
    for (int q = 0; q < QB; ++q) *reinterpret_cast<f4 *>(&Bs[buf][((tid >> 3) + 32 * q) * LDK + kq]) = rb[q];
  };

  v16f acc[PM][PN];
#pragma unroll
  for (int p = 0; p < PM; ++p)
#pragma unroll
    for (int q = 0; q < PN; ++q)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[p][q][v] = 0.f;

  const int64_t nk = (kend - kbeg + KB - 1) / KB;
  gload(kbeg);
  sstore(0, kbeg);
  __syncthreads();
  for (int64_t s = 0; s < nk; ++s) {
    const int buf = (int)(s & 1);
    if (s + 1 < nk) gload(kbeg + (s + 1) * KB);
    float av[PM][16], bv[PN][16];
#pragma unroll
    for (int p = 0; p < PM; ++p) {
      const float *src = &As[buf][(wr * 32 * PM + 32 * p + r) * LDK + 16 * h];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const f4 t = *reinterpret_cast<const f4 *>(src + 4 * c);
        av[p][4 * c + 0] = t.x;
        av[p][4 * c + 1] = t.y;
        av[p][4 * c + 2] = t.z;
        av[p][4 * c + 3] = t.w;
      }
    }
#pragma unroll
    for (int q = 0; q < PN; ++q) {
      const float *src = &Bs[buf][(wc * 32 * PN + 32 * q + r) * LDK + 16 * h];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const f4 t = *reinterpret_cast<const f4 *>(src + 4 * c);
        bv[q][4 * c + 0] = t.x;
        bv[q][4 * c + 1] = t.y;
        bv[q][4 * c + 2] = t.z;
        bv[q][4 * c + 3] = t.w;
      }
    }
#pragma unroll
    for (int kk = 0; kk < 16; ++kk)
#pragma unroll
      for (int p = 0; p < PM; ++p)
#pragma unroll
        for (int q = 0; q < PN; ++q)
          acc[p][q] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[p][kk], bv[q][kk], acc[p][q], 0, 0, 0);
    if (s + 1 < nk) sstore(buf ^ 1, kbeg + (s + 1) * KB);
    __syncthreads();
  }

  // epilogue: U^T (coalesced along j) and column sums of U^2 over this tile
  double cs[PN];
#pragma unroll
  for (int q = 0; q < PN; ++q) cs[q] = 0.0;
#pragma unroll
  for (int p = 0; p < PM; ++p)
#pragma unroll
    for (int q = 0; q < PN; ++q) {
      const int64_t j = j0 + wc * 32 * PN + 32 * q + r;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int64_t t = t0 + wr * 32 * PM + 32 * p + 8 * (v >> 2) + 4 * h + (v & 3);
        const float val = acc[p][q][v];
        if (t < T && j < ma) b.Ut[j + t * b.ldut] = val;
        cs[q] = fma((double)val, (double)val, cs[q]);  // rows t >= T are zero
      }
    }
#pragma unroll
  for (int q = 0; q < PN; ++q) cs[q] += __shfl_xor(cs[q], 32, 64);
  if (h == 0) {
#pragma unroll
    for (int q = 0; q < PN; ++q) ush[wr * BN + wc * 32 * PN + 32 * q + r] = cs[q];
  }
  __syncthreads();
  for (int c = tid; c < BN; c += 256) {
    double sum = 0.0;
#pragma unroll
    for (int w = 0; w < WM; ++w) sum += ush[w * BN + c];
    const int64_t cc = j0 + c;
    if (cc < ma) b.usq_part[(int64_t)blockIdx.x * b.ldq + b.act[cc]] = sum;
  }
}

// --------------------------------------------------------------------------
// U^T = X^T L for factors whose tiles would leave most of the chip idle: 32
// periods x 32 targets a workgroup, its eight wavefronts every eighth
// 16-asset step each (operands straight from memory to registers, four steps
// ahead), the eight sums added in float64 in LDS.
// --------------------------------------------------------------------------
template <typename TL>
__global__ __launch_bounds__(512) void k_bgemm_u_split(BatchArgs b) {
  constexpr int D = 4;  // steps in flight
  typedef Raw4<TL> R;
  __shared__ float red[8][16][64];
  const int64_t T = b.base.cols, n = b.base.n, ld = b.base.ld;
  const int ma = *b.mact;
  const int64_t t0 = (int64_t)blockIdx.x * 32;
  const int c0 = (int)blockIdx.y * 32;
  if (c0 >= ma) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = lane >> 5, r = lane & 31;
  // lane: period t0 + r and target c0 + r, assets 8 h .. 8 h + 7 of a step;
  // matrix step q pairs assets q and 8 + q.  Past the last: the last, dropped
  const int c = c0 + r < ma ? c0 + r : ma - 1;
  const float *X = b.base.xs + (int64_t)b.act[c] * b.ldx + 8 * h;
  const TL *L = static_cast<const TL *>(b.base.L) + (t0 + r < T ? t0 + r : T - 1) * ld;
  const int64_t last = ld - 4;
  const int steps = (int)((n + 15) / 16);
  const int cnt = (steps - wave + 7) >> 3;
  f4 xa[D][2];
  typename R::type lb[D][2];
  auto load = [&](int slot, int t) {
    const int64_t k0 = 16 * (int64_t)(wave + 8 * (t < cnt ? t : cnt - 1));
    const int64_t kl = k0 + 8 * h;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      xa[slot][q] = *reinterpret_cast<const f4 *>(X + k0 + 4 * q);  // zero-padded to a multiple of 256
      lb[slot][q] = R::load(L + (kl + 4 * q < last ? kl + 4 * q : last));
    }
  };
  v16f acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  if (cnt > 0) {
#pragma unroll
    for (int t = 0; t < D; ++t) {
      load(t, t);
      __builtin_amdgcn_sched_barrier(0);
    }
    for (int s0 = 0; s0 < cnt; s0 += D) {
#pragma unroll
      for (int u = 0; u < D; ++u) {
        if (s0 + u < cnt) {
          const int64_t k = 16 * (int64_t)(wave + 8 * (s0 + u)) + 8 * h;
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            f4 l = R::widen(lb[u][q]);
            const int64_t row = k + 4 * q;  // asset rows past n (ld may exceed n) are not data
            l.x = row + 0 < n ? l.x : 0.f;
            l.y = row + 1 < n ? l.y : 0.f;
            l.z = row + 2 < n ? l.z : 0.f;
            l.w = row + 3 < n ? l.w : 0.f;
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(l.x, xa[u][q].x, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(l.y, xa[u][q].y, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(l.z, xa[u][q].z, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(l.w, xa[u][q].w, acc, 0, 0, 0);
          }
        }
        load(u, s0 + u + D);
      }
    }
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) red[wave][v][lane] = acc[v];
  __shared__ double qs[8][64];
  __syncthreads();
  // register v of lane (h, r): period t0 + 8 (v / 4) + 4 h + v % 4, target c0 + r
  double q = 0.0;
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int v = 8 * e + wave;
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < 8; ++w) s += (double)red[w][v][lane];
    const int64_t t = t0 + 8 * (v >> 2) + 4 * h + (v & 3);
    const float val = t < T ? (float)s : 0.f;
    q = fma((double)val, (double)val, q);
    if (t < T && c0 + r < ma) b.Ut[c0 + r + t * b.ldut] = val;
  }
  qs[wave][lane] = q;
  __syncthreads();
  if (tid < 32 && c0 + tid < ma) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < 8; ++w) s += qs[w][tid] + qs[w][tid + 32];
    b.usq_part[(int64_t)blockIdx.x * b.ldq + b.act[c0 + tid]] = s;
  }
}

// --------------------------------------------------------------------------
// P[s] = (L_{:, T_s} U_{T_s, :})^T.  Tile: BM assets x BN targets over the
// period range of split s (grid.y).  Both LDS tiles are indexed [k][row];
// MFMA step s takes k = 2s + h.  Output rows i >= n and columns j >= m are
// never stored, so garbage there (padding of L or U^T) stays in unused
// accumulator entries; periods outside the range are zero in both tiles.
// --------------------------------------------------------------------------
template <typename TL, int BM, int BN, int WM, int WN>
__global__ __launch_bounds__(256) void k_bgemm_g(BatchArgs b) {
  constexpr int PM = BM / (32 * WM), PN = BN / (32 * WN);
  constexpr int LDA = BM + 4, LDB = BN + 4;
  constexpr int FA = BM / 4, FB = BN / 4;       // float4 per period row of a tile
  constexpr int QA = KB * FA / 256, QB = KB * FB / 256;
  static_assert(WM * WN == 4 && PM >= 1 && PN >= 1 && QA >= 1 && QB >= 1, "tile");
  typedef Raw4<TL> R;
  __shared__ float As[2][KB * LDA];
  __shared__ float Bs[2][KB * LDB];
  const int64_t T = b.base.cols, n = b.base.n;
  const int m = b.m;
  const int64_t i0 = (int64_t)blockIdx.x * BM;
  const int64_t tb = (int64_t)blockIdx.y * b.kchunk;
  const int64_t te = (tb + b.kchunk < T) ? tb + b.kchunk : T;
  const int64_t j0 = (int64_t)blockIdx.z * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = wave / WN, wc = wave % WN;
  const int h = lane >> 5, r = lane & 31;
  const TL *L = static_cast<const TL *>(b.base.L);
  const int64_t ld = b.base.ld;
  const float *Ut = b.Ut;
  const int ma = *b.mact;
  if (j0 >= ma) return;
  (void)m;

  typename R::type ra[QA];
  f4 rb[QB];
  auto gload = [&](int64_t k0) {
#pragma unroll
    for (int q = 0; q < QA; ++q) {
      const int idx = tid + 256 * q;
      const int64_t t = k0 + idx / FA;
      const int64_t i = i0 + 4 * (idx % FA);
      ra[q] = (t < te && i < n) ? R::load(L + t * ld + i) : R::zero();
    }
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      const int idx = tid + 256 * q;
      const int64_t t = k0 + idx / FB;
      const int64_t j = j0 + 4 * (idx % FB);
      rb[q] = (t < te && j < ma) ? *reinterpret_cast<const f4 *>(Ut + j + t * b.ldut) : f4{0.f, 0.f, 0.f, 0.f};
    }
  };
  auto sstore = [&](int buf) {
#pragma unroll
    for (int q = 0; q < QA; ++q) {
      const int idx = tid + 256 * q;
      *reinterpret_cast<f4 *>(&As[buf][(idx / FA) * LDA + 4 * (idx % FA)]) = R::widen(ra[q]);
    }
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      const int idx = tid + 256 * q;
      *reinterpret_cast<f4 *>(&Bs[buf][(idx / FB) * LDB + 4 * (idx % FB)]) = rb[q];
    }
  };

  v16f acc[PM][PN];
#pragma unroll
  for (int p = 0; p < PM; ++p)
#pragma unroll
    for (int q = 0; q < PN; ++q)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[p][q][v] = 0.f;

  const int64_t nk = (te > tb) ? (te - tb + KB - 1) / KB : 0;
  if (nk > 0) {
    gload(tb);
    sstore(0);
  }
  __syncthreads();
  for (int64_t s = 0; s < nk; ++s) {
    const int buf = (int)(s & 1);
    if (s + 1 < nk) gload(tb + (s + 1) * KB);
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      const int k = 2 * kk + h;
      float av[PM], bv[PN];
#pragma unroll
      for (int p = 0; p < PM; ++p) av[p] = As[buf][k * LDA + wr * 32 * PM + 32 * p + r];
#pragma unroll
      for (int q = 0; q < PN; ++q) bv[q] = Bs[buf][k * LDB + wc * 32 * PN + 32 * q + r];
#pragma unroll
      for (int p = 0; p < PM; ++p)
#pragma unroll
        for (int q = 0; q < PN; ++q)
          acc[p][q] = __builtin_amdgcn_mfma_f32_32x32x2f32(bv[q], av[p], acc[p][q], 0, 0, 0);
    }
    if (s + 1 < nk) sstore(buf ^ 1);
    __syncthreads();
  }

  // targets on the output's rows, assets along the lanes
  float *P = b.P + (int64_t)blockIdx.y * b.ldpm * b.ldpi;
#pragma unroll
  for (int p = 0; p < PM; ++p)
#pragma unroll
    for (int q = 0; q < PN; ++q) {
      const int64_t i = i0 + wr * 32 * PM + 32 * p + r;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int64_t j = j0 + wc * 32 * PN + 32 * q + 8 * (v >> 2) + 4 * h + (v & 3);
        if (i < n && j < ma) P[j * b.ldpi + i] = acc[p][q][v];
      }
    }
}

// --------------------------------------------------------------------------
// One workgroup per running target (GEMM column c): its gradient g = 2 sum_s
// P[s][c] in a fixed order (float64), the element-wise epilogue of its mode,
// and its serial tail.  The partials run along the assets, so a workgroup
// reads its own column's S n floats coalesced (64 KB at n = 2000 and eight
// splits); the gradient and the step input reach the tail through LDS.  A
// separate reduce launch before the tail (5.6 us at n = 2000, 128 targets)
// and its gap are saved.
// --------------------------------------------------------------------------

// Target j's place in the planes of X: a fragment of 32 targets, 16 assets
// and one plane is 64 pieces of 16 bytes, piece 32 h + j % 32 the assets 8 h ..
// 8 h + 7 of target j.
constexpr int kXFrag = 512;
__device__ __forceinline__ uint16_t *x_planes(const BatchArgs &b, int j) {
  return b.Xp + (int64_t)(j >> 5) * 32 * b.xpstride + 8 * (j & 31);
}

// The planes of x (n floats at xs in LDS; zeros past n) into target j's
// pieces: one 16-byte group of each plane a thread.
__device__ __forceinline__ void store_x_planes(const BatchArgs &b, int j, const float *xs) {
  uint16_t *out = x_planes(b, j);
  for (int64_t q = threadIdx.x; 8 * q < b.base.n; q += 256) {
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (8 * q + e < b.base.n) ? xs[8 * q + e] : 0.f;
    u4v w[3];
    split8(v, w);
    uint16_t *o = out + (q >> 1) * 3 * kXFrag + (q & 1) * 256;
#pragma unroll
    for (int pl = 0; pl < 3; ++pl) *reinterpret_cast<u4v *>(o + kXFrag * pl) = w[pl];
  }
}

// Bound by latency: one workgroup's chain of loads, sums and barriers.  So
// everything the tail reads from memory is asked for at once, before the
// target's state says which iterate buffer is the current one, and the tail
// works on copies in LDS (state, mu, both iterates where they fit); a load
// after a barrier or a store would cost its latency each time.  n = 2000,
// 128 targets: 13.1 us with the loads where they are used, 11.2 us so (12.0
// with the planes it writes in k_cov16's fragments); n = 1500, 24
// targets and 22 splits: 14.8 and 13.6 us.
template <int E>
__global__ __launch_bounds__(256) void k_btail(BatchArgs b) {
  constexpr bool HOLD = E <= 8;  // five vectors of 256 E in LDS: 80 KB
  __shared__ __attribute__((aligned(16))) double gl[2][256 * E];  // g_k and the step input (CG: H p)
  __shared__ double xv[HOLD ? 2 : 1][HOLD ? 256 * E : 1], mul[HOLD ? 256 * E : 1];
  __shared__ DevState stl;
  __shared__ double redbuf[64];
  __shared__ double mbuf[8];
  __shared__ int64_t ibuf[8];
  // the new iterate in float32 for its planes: the tails read the step input
  // at their start and write the iterate at their end
  float *xl = reinterpret_cast<float *>(gl[1]);
  const int tid = threadIdx.x, c = blockIdx.x;
  const int64_t n = b.base.n;
  const int ma = *b.mact, j = b.act[c];  // (act has m entries; those past the running ones are not used)
  // Entries past n and splits past the last read the last one and are dropped.
  int off[E];
  double tot[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    off[e] = (int)(tid + 256 * e < n ? tid + 256 * e : n - 1);
    tot[e] = 0.0;
  }
  const float *part = b.P + (int64_t)c * b.ldpi;
  const int64_t split_stride = b.ldpm * b.ldpi;
  constexpr int F = E <= 8 ? 8 : (E <= 16 ? 4 : 2);  // splits in flight
  float pv[F][E];
  auto load_parts = [&](int sp) {
#pragma unroll
    for (int f = 0; f < F; ++f) {
      const float *ps = part + (int64_t)(sp + f < b.splits ? sp + f : b.splits - 1) * split_stride;
#pragma unroll
      for (int e = 0; e < E; ++e) pv[f][e] = ps[off[e]];
    }
  };
  load_parts(0);
  if (c >= ma) return;
  SolveArgs a = target_args(b, j);
  DevState *st_mem = a.st;
  const bool npga = a.mode == kTailNpga;
  constexpr int kStateWords = (int)(sizeof(DevState) / 8);
  static_assert(kStateWords <= 256, "a word per thread");
  const uint64_t sw = reinterpret_cast<const uint64_t *>(st_mem)[tid < kStateWords ? tid : 0];
  // NPGA: x_k, x_{k-1}, g_{k-1}; CG: p; gradient only: x.  (Longer vectors
  // have no registers for the gradient buffer that is not wanted.)
  const double *r0 = npga || a.mode == kTailGrad ? a.xbuf0 : a.pvec;
  double u0[E], u1[E], u2[E], u3[HOLD ? E : 1], um[HOLD ? E : 1];
  const int early = HOLD ? 0 : st_mem->iter & 1;
  const double *r1 = a.xbuf1, *r2 = early ? a.gbuf0 : a.gbuf1;
  if (!HOLD && npga && early) {
    r0 = a.xbuf1;
    r1 = a.xbuf0;
  }
#pragma unroll
  for (int e = 0; e < E; ++e) {
    u0[e] = r0[off[e]];
    if (npga) {
      u1[e] = r1[off[e]];
      u2[e] = r2[off[e]];
    }
    if constexpr (HOLD) {
      if (npga) u3[e] = a.gbuf0[off[e]];
      um[e] = a.mu[off[e]];
    }
  }
  if (tid < kStateWords) reinterpret_cast<uint64_t *>(&stl)[tid] = sw;
  for (int sp = 0;;) {
#pragma unroll
    for (int f = 0; f < F; ++f)
#pragma unroll
      for (int e = 0; e < E; ++e) tot[e] += (sp + f < b.splits) ? (double)pv[f][e] : 0.0;
    sp += F;
    if (sp >= b.splits) break;
    load_parts(sp);
  }
  __syncthreads();  // stl
  if (stl.done != kRunning) return;
  a.st = &stl;
  const int cur = stl.iter & 1;
  const double alpha = stl.alpha, beta = stl.beta, gamma2 = 2.0 * stl.gamma;
  double usq = -1.0;  // covariance form: f = x^T g / 2 in the tails
  if (!b.covariance && (a.mode == kTailGrad || (npga && stl.iter % stl.check_every == 0))) {
    BlockReducer<5> red5{redbuf, 0};
    double acc[5] = {0, 0, 0, 0, 0};
    for (int w = tid; w < b.utiles; w += 256) acc[0] += b.usq_part[(int64_t)w * b.ldq + j];
    red5.sum(acc);
    usq = acc[0];
    __syncthreads();
  }
  double *gk = cur ? a.gbuf1 : a.gbuf0;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int64_t i = tid + 256 * e;
    if constexpr (HOLD) {
      mul[i] = um[e];
      if (npga) {
        xv[0][i] = u0[e];
        xv[1][i] = u1[e];
      }
    }
    if (i >= n) continue;
    const double g = 2.0 * tot[e];
    if (npga) {
      // g_k kept for the next iteration; v = y - alpha grad f(y), as
      // npga_store_grad_step forms it
      const bool swapped = HOLD && cur;
      const double xk = swapped ? u1[e] : u0[e], xp = swapped ? u0[e] : u1[e];
      const double gp = swapped ? u3[HOLD ? e : 0] : u2[e];
      const double gi = g + (a.ga ? a.ga[i] : 0.0) + gamma2 * xk;
      const double y = fma(beta, xk - xp, xk);
      const double gy = fma(beta, gi - gp, gi);
      gk[i] = gi;
      gl[0][i] = gi;
      gl[1][i] = fma(-alpha, gy, y);
    } else if (a.mode == kTailGrad) {
      a.gbuf0[i] = g + gamma2 * u0[e];
    } else {
      gl[0][i] = g + gamma2 * u0[e];
    }
  }
  if (b.covariance) a.xs = xl;
  if constexpr (HOLD) a.mu = mul;
  if (a.mode == kTailNpga) {
    SolveArgs t = a;
    t.gbuf0 = gl[cur];
    t.gbuf1 = gl[1 - cur];
    if constexpr (HOLD) {
      t.xbuf0 = xv[0];
      t.xbuf1 = xv[1];
    }
    tail_npga<E>(t, usq, redbuf);
    if constexpr (HOLD) {  // (an iteration that ended before its step leaves x_{k-1} as it was)
      double *xn = cur ? a.xbuf0 : a.xbuf1;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int64_t i = tid + 256 * e;
        if (i < n) xn[i] = xv[1 - cur][i];
      }
    }
  } else if (a.mode == kTailCG) {
    SolveArgs t = a;
    t.gbuf0 = gl[0];
    tail_cg<E>(t, redbuf, mbuf, ibuf);
  } else if (a.mode == kTailGrad) {
    tail_grad<E>(a, usq, redbuf);
  }
  __syncthreads();
  if (tid < kStateWords) reinterpret_cast<uint64_t *>(st_mem)[tid] = reinterpret_cast<const uint64_t *>(&stl)[tid];
  if (b.covariance) store_x_planes(b, j, xl);
}

template <int E>
__global__ __launch_bounds__(256) void k_bproject_init(BatchArgs b) {
  __shared__ double redbuf[64];
  __shared__ float xl[256 * E];
  SolveArgs a = target_args(b, blockIdx.x);
  if (a.st->done != kRunning) return;
  if (b.covariance) a.xs = xl;
  project_init_body<E>(a, redbuf);
  if (b.covariance) {
    __syncthreads();
    store_x_planes(b, blockIdx.x, xl);
  }
}

template <int E>
__global__ __launch_bounds__(256) void k_bcg_init(BatchArgs b) {
  __shared__ double redbuf[64];
  __shared__ float xl[256 * E];
  SolveArgs a = target_args(b, blockIdx.x);
  if (a.st->done != kRunning) return;
  if (b.covariance) a.xs = xl;
  cg_init_body<E>(a, redbuf);
  if (b.covariance) {
    __syncthreads();
    store_x_planes(b, blockIdx.x, xl);
  }
}

// X[:, j] = x_j (float32); grid (row blocks, m).
__global__ __launch_bounds__(256) void k_bfinalize(BatchArgs b, float *X, int64_t ldo) {
  const SolveArgs a = target_args(b, blockIdx.y);
  const double *x = (a.st->iter & 1) ? a.xbuf1 : a.xbuf0;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < a.n) X[(int64_t)blockIdx.y * ldo + i] = (float)x[i];
}

// x_j = X0[:, j] (or 1/n) in float64, the whole column of X zeroed first
// (rows n..ldx-1 stay zero for the U GEMM); grid (row blocks, m).
__global__ __launch_bounds__(256) void k_bset_x0(BatchArgs b, const float *X0, int64_t ldx0) {
  const SolveArgs a = target_args(b, blockIdx.y);
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < b.ldx) a.xs[i] = 0.0f;
  if (i < a.n) {
    const double v = X0 ? (double)X0[(int64_t)blockIdx.y * ldx0 + i] : 1.0 / (double)a.n;
    a.xbuf0[i] = v;
  }
}

// Float32 copy of X into the GEMM input and float64 copy into xbuf0 (the
// batched gradient entry point); grid (row blocks, m).
__global__ __launch_bounds__(256) void k_bload_x(BatchArgs b, const float *X, int64_t ldx_in) {
  const SolveArgs a = target_args(b, blockIdx.y);
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < b.ldx) {
    const float v = (i < a.n) ? X[(int64_t)blockIdx.y * ldx_in + i] : 0.0f;
    a.xs[i] = v;
    if (i < a.n) a.xbuf0[i] = (double)v;
  }
}

// Step size of the shared factor: alpha and L_f from the power-method state.
__global__ void k_bcopy_step(BatchArgs b, const DevState *src) {
  for (int j = threadIdx.x; j < b.m; j += blockDim.x) {
    b.base.st[j].alpha = src->alpha;
    b.base.st[j].lipschitz = src->lipschitz;
    b.base.st[j].rho2 = src->rho2;
    b.base.st[j].beta_const = src->beta_const;
    b.base.st[j].lz_m = src->lz_m;
  }
}

// Refinement phase: every target whose last phase converged runs again.
__global__ void k_bphase_reset(BatchArgs b, double tol, int32_t max_iter) {
  for (int j = threadIdx.x; j < b.m; j += blockDim.x) {
    DevState *st = b.base.st + j;
    if (st->done != kConverged) continue;
    st->done = kRunning;
    st->cg_window = 60;
    st->tol = tol;
    st->max_iter = max_iter;
    st->restart = 1;
    st->t = 1.0;
    st->beta = 0.0;
  }
}

// x_a = x_k for every target about to be refined (converged last phase).
__global__ __launch_bounds__(256) void k_bcopy_anchor(BatchArgs b) {
  const SolveArgs a = target_args(b, blockIdx.y);
  if (a.st->done != kConverged) return;
  const double *x = (a.st->iter & 1) ? a.xbuf1 : a.xbuf0;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < a.n) const_cast<double *>(a.xa)[i] = x[i];
}

// out[0] = number of running targets, out[1 + j] = done code of target j;
// act[0..mact) = the running targets in ascending order (GEMM columns of the
// next iterations).  One workgroup; target j = 4 tid + e (m <= 1024).
__global__ __launch_bounds__(256) void k_bstatus(BatchArgs b, int32_t *out, int32_t *act, int32_t *mact) {
  __shared__ int scan[256];
  const int tid = threadIdx.x;
  int run[4];
  int c = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int j = 4 * tid + e;
    run[e] = 0;
    if (j < b.m) {
      const int32_t d = b.base.st[j].done;
      out[1 + j] = d;
      run[e] = (d == kRunning) ? 1 : 0;
      c += run[e];
    }
  }
  // inclusive scan of the per-thread counts (Hillis-Steele)
  scan[tid] = c;
  __syncthreads();
  for (int off = 1; off < 256; off <<= 1) {
    const int v = (tid >= off) ? scan[tid - off] : 0;
    __syncthreads();
    scan[tid] += v;
    __syncthreads();
  }
  int pos = scan[tid] - c;
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (run[e]) act[pos++] = 4 * tid + e;
  if (tid == 255) {
    out[0] = scan[255];
    *mact = scan[255];
  }
}

// Every target is a GEMM column (batched gradient, tuning).
__global__ __launch_bounds__(256) void k_bact_all(int32_t m, int32_t *act, int32_t *mact) {
  for (int j = threadIdx.x; j < m; j += 256) act[j] = j;
  if (threadIdx.x == 0) *mact = m;
}

// L32 = float32 values of a bfloat16 factor (the covariance form's SYRK
// reads float32); rows n..ld32-1 are written as zeros.
__global__ __launch_bounds__(256) void k_widen_bf16(const uint16_t *L, int64_t ld, int64_t n, int64_t T, float *L32,
                                                    int64_t ld32) {
  const int64_t total = ld32 * T;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
    const int64_t t = e / ld32, i = e - t * ld32;
    L32[e] = (i < n) ? __uint_as_float((uint32_t)L[i + t * ld] << 16) : 0.f;
  }
}

int launch_widen_bf16(const uint16_t *L, int64_t ld, int64_t n, int64_t T, float *L32, int64_t ld32, hipStream_t s) {
  hipLaunchKernelGGL(k_widen_bf16, dim3(2048), dim3(256), 0, s, L, ld, n, T, L32, ld32);
  return (int)hipGetLastError();
}

__global__ __launch_bounds__(256) void k_zero_f32(float *p, int64_t count) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (int64_t)gridDim.x * 256)
    p[i] = 0.0f;
}

// --------------------------------------------------------------------------
// launchers
// --------------------------------------------------------------------------
#define BATCH_SLOT_SWITCH(slots, CALL)     \
  switch (slots) {                         \
    case 1: CALL(1); break;                \
    case 2: CALL(2); break;                \
    case 4: CALL(4); break;                \
    case 8: CALL(8); break;                \
    case 12: CALL(12); break;              \
    case 16: CALL(16); break;              \
    case 22: CALL(22); break;              \
    case 28: CALL(28); break;              \
    case 32: CALL(32); break;              \
    default: return (int)hipErrorInvalidValue; \
  }

template <typename TL>
static int launch_bgemm_t(const BatchArgs &b, const BatchConfig &c, hipStream_t s) {
  const int64_t T = b.base.cols, n = b.base.n;
  const dim3 gu((unsigned)((T + c.u_bm - 1) / c.u_bm), (unsigned)((b.m + c.u_bn - 1) / c.u_bn));
  if (b.u_split)
    hipLaunchKernelGGL(k_bgemm_u_split<TL>, dim3((unsigned)((T + 31) / 32), (unsigned)((b.running + 31) / 32)),
                       dim3(512), 0, s, b);
  else if (c.u_bm == 128 && c.u_bn == 128)
    hipLaunchKernelGGL((k_bgemm_u<TL, 128, 128, 2, 2>), gu, dim3(256), 0, s, b);
  else if (c.u_bm == 64 && c.u_bn == 128)
    hipLaunchKernelGGL((k_bgemm_u<TL, 64, 128, 1, 4>), gu, dim3(256), 0, s, b);
  else if (c.u_bm == 128 && c.u_bn == 64)
    hipLaunchKernelGGL((k_bgemm_u<TL, 128, 64, 2, 2>), gu, dim3(256), 0, s, b);
  else if (c.u_bm == 64 && c.u_bn == 64)
    hipLaunchKernelGGL((k_bgemm_u<TL, 64, 64, 2, 2>), gu, dim3(256), 0, s, b);
  else if (c.u_bm == 128 && c.u_bn == 32)
    hipLaunchKernelGGL((k_bgemm_u<TL, 128, 32, 4, 1>), gu, dim3(256), 0, s, b);
  else
    return (int)hipErrorInvalidValue;
  if (hipGetLastError() != hipSuccess) return (int)hipErrorLaunchFailure;
  const dim3 gg((unsigned)((n + c.g_bm - 1) / c.g_bm), (unsigned)b.splits, (unsigned)((b.m + c.g_bn - 1) / c.g_bn));
  if (c.g_bm == 128 && c.g_bn == 128)
    hipLaunchKernelGGL((k_bgemm_g<TL, 128, 128, 2, 2>), gg, dim3(256), 0, s, b);
  else if (c.g_bm == 64 && c.g_bn == 128)
    hipLaunchKernelGGL((k_bgemm_g<TL, 64, 128, 1, 4>), gg, dim3(256), 0, s, b);
  else if (c.g_bm == 128 && c.g_bn == 64)
    hipLaunchKernelGGL((k_bgemm_g<TL, 128, 64, 2, 2>), gg, dim3(256), 0, s, b);
  else if (c.g_bm == 64 && c.g_bn == 64)
    hipLaunchKernelGGL((k_bgemm_g<TL, 64, 64, 2, 2>), gg, dim3(256), 0, s, b);
  else if (c.g_bm == 128 && c.g_bn == 32)
    hipLaunchKernelGGL((k_bgemm_g<TL, 128, 32, 4, 1>), gg, dim3(256), 0, s, b);
  else
    return (int)hipErrorInvalidValue;
  return (int)hipGetLastError();
}

// Covariance form on the bfloat16 matrix cores: P_z = (Sigma[:, K_z]
// X[K_z, :])^T for the 16-row stages K_z of range z, both operands as three
// bfloat16 planes (v = v_h + v_m + v_l exactly); the six largest plane
// products (h h, h m, m h, h l, m m, l h: the dropped m l, l m and l l are
// below 2^-24 of the leading one) on v_mfma_f32_32x32x16_bf16 with float32
// accumulation, as the split SYRK does.
//
// Tile: 64 rows of Sigma x 32 NC running targets.  The four wavefronts take
// every fourth stage of the range each, so a fragment is used by one
// wavefront only and comes straight from memory to its registers (Sigma's
// fragments lane-linear, X's gathered from the running targets' pieces), D
// stages ahead; no LDS and no barrier until the four sums meet at the end.
// Bound by the 64 bytes a cycle a compute unit takes from its L2 (12 KiB a
// stage at 64 columns) and by latency: at n = 2000 a compute unit has 32
// stages.  128 targets 10.5 us, 32 or fewer 6.6 us; with each target's planes
// by themselves (a load of X's then touched 32 lines, not eight) 12.5 and 6.8,
// and with loads past the last stage 13.1 and 7.1.
template <int NC>
__global__ __launch_bounds__(256, 1) void k_cov16(BatchArgs b) {
  constexpr int D = 4;  // stages in flight
  __shared__ float red[4][2 * NC][16][64];
  const int64_t n = b.base.n;
  const int ma = *b.mact;
  // workgroups with the same range of the contraction on the same XCDs (and,
  // with fewer than eight ranges, the same part of the rows): what an XCD
  // reads of Sigma and X together is an eighth of Sigma and, at most, that
  // share of X, which its L2 keeps from one iteration to the next
  const int gx = (int)((n + 63) / 64), sx = b.splits < 8 ? b.splits : 8, rx = 8 / sx;
  const int gp = (gx + rx - 1) / rx, xcd = blockIdx.x & 7;
  int loc = blockIdx.x >> 3;
  const int bz = xcd % sx + sx * (loc % (b.splits / sx));
  loc /= b.splits / sx;
  const int bx = (xcd / sx) * gp + loc % gp, by = loc / gp;
  const int c0 = by * 32 * NC;
  if (c0 >= ma || bx >= gx) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = lane >> 5, r = lane & 31;
  const int64_t kb = (int64_t)bz * b.kchunk;
  const int64_t ke = (kb + b.kchunk < b.stages) ? kb + b.kchunk : b.stages;
  const int cnt = (int)((ke - kb - wave + 3) >> 2);  // this wavefront's stages: kb + wave, + 4, ...
  const uint16_t *pa[2], *pb[NC];
#pragma unroll
  for (int g = 0; g < 2; ++g) pa[g] = frag_ptr(b.Sp, 2 * (int64_t)bx + g, kb + wave, b.stages) + 8 * lane;
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const int c = c0 + 32 * q + r;
    const int j = b.act[c < ma ? c : ma - 1];
    pb[q] = x_planes(b, j) + (kb + wave) * 3 * kXFrag + 256 * h;
  }
  typedef bf16x8_t frag_t;
  frag_t fa[D][2][3], fb[D][NC][3];
  auto load = [&](int slot, int t) {
    const int64_t s = 4 * (int64_t)(t < cnt ? t : cnt - 1);  // past the end the last one again, not used
#pragma unroll
    for (int pl = 0; pl < 3; ++pl) {
#pragma unroll
      for (int g = 0; g < 2; ++g)
        fa[slot][g][pl] =
            __builtin_bit_cast(frag_t, *reinterpret_cast<const u4v *>(pa[g] + s * kPanelStage + pl * 4 * kFrag));
#pragma unroll
      for (int q = 0; q < NC; ++q)
        fb[slot][q][pl] = __builtin_bit_cast(frag_t, *reinterpret_cast<const u4v *>(pb[q] + (s * 3 + pl) * kXFrag));
    }
  };
  v16f acc[2][NC];
#pragma unroll
  for (int g = 0; g < 2; ++g)
#pragma unroll
    for (int q = 0; q < NC; ++q)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[g][q][v] = 0.f;
  if (cnt > 0) {
#pragma unroll
    for (int t = 0; t < D; ++t) {
      load(t, t);
      __builtin_amdgcn_sched_barrier(0);  // in the order of use
    }
    for (int t0 = 0; t0 < cnt; t0 += D) {
#pragma unroll
      for (int u = 0; u < D; ++u) {
        if (t0 + u < cnt) {
          // plane products, smallest terms first; targets on the output's
          // rows, so that a lane's results run along the assets
          constexpr int ka[6] = {2, 1, 0, 1, 0, 0}, kx[6] = {0, 1, 2, 0, 1, 0};
#pragma unroll
          for (int k = 0; k < 6; ++k)
#pragma unroll
            for (int g = 0; g < 2; ++g)
#pragma unroll
              for (int q = 0; q < NC; ++q)
                acc[g][q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[u][q][kx[k]], fa[u][g][ka[k]], acc[g][q], 0, 0, 0);
        }
        if (t0 + u + D < cnt) load(u, t0 + u + D);
      }
    }
  }
#pragma unroll
  for (int g = 0; g < 2; ++g)
#pragma unroll
    for (int q = 0; q < NC; ++q)
#pragma unroll
      for (int v = 0; v < 16; ++v) red[wave][g * NC + q][v][lane] = acc[g][q][v];
  __syncthreads();
  // block k = (g, q), register v -> target c0 + 32 q + 8 (v / 4) + 4 h + v % 4,
  // asset 64 x + 32 g + r
  float *out = b.P + (int64_t)bz * b.ldpm * b.ldpi;
#pragma unroll
  for (int e = 0; e < 8 * NC; ++e) {
    const int idx = 4 * e + wave;  // (k, v)
    const int k = idx >> 4, v = idx & 15;
    const double s = ((double)red[0][k][v][lane] + (double)red[1][k][v][lane]) +
                     ((double)red[2][k][v][lane] + (double)red[3][k][v][lane]);
    const int64_t col = c0 + 32 * (k % NC) + 8 * (v >> 2) + 4 * h + (v & 3);
    const int64_t row = (int64_t)bx * 64 + 32 * (k / NC) + r;
    if (row < n && col < ma) out[col * b.ldpi + row] = (float)s;
  }
}

// Ranges and width for `running` targets: 64 columns a workgroup (32 when no
// more run), the contraction split so that a launch has about one workgroup
// per compute unit, with at least four stages (one a wavefront) in a range.
void cov_plan(BatchArgs &b, int running) {
  const int w = running <= 32 ? 32 : 64;
  const int64_t tiles = ((b.base.n + 63) / 64) * ((running + w - 1) / w);
  int64_t want = std::max<int64_t>(1, 256 / tiles);
  want = std::min<int64_t>(std::min<int64_t>(want, kCovMaxSplits), (b.stages + 3) / 4);
  // 1, 2, 4 or a multiple of 8 ranges (the ranges are spread over the XCDs)
  want = want >= 8 ? want / 8 * 8 : (want >= 4 ? 4 : want >= 2 ? 2 : 1);
  b.kchunk = (b.stages + want - 1) / want;
  b.splits = (int32_t)want;  // (a last range may be empty: its sums are zeros)
  b.running = running;
}

static int launch_bcov(const BatchArgs &b, hipStream_t s) {
  if (!b.Sp || !b.Xp || b.splits < 1 || b.running < 1) return (int)hipErrorInvalidValue;
  const int nc = b.running <= 32 ? 1 : 2;
  const int gx = (int)((b.base.n + 63) / 64), gy = (b.running + 32 * nc - 1) / (32 * nc);
  const int sx = std::min(b.splits, 8), rx = 8 / sx;
  const unsigned grid = (unsigned)(8 * (b.splits / sx) * ((gx + rx - 1) / rx) * gy);
  if (nc == 1)
    hipLaunchKernelGGL(k_cov16<1>, dim3(grid), dim3(256), 0, s, b);
  else
    hipLaunchKernelGGL(k_cov16<2>, dim3(grid), dim3(256), 0, s, b);
  return (int)hipGetLastError();
}

int launch_bgemm(const BatchArgs &b, const BatchConfig &c, hipStream_t s) {
  if (b.covariance) return launch_bcov(b, s);
  if (b.Lt) return launch_b16_gemm(b, c, s);
  if (b.base.dtype == NPGA_BF16) return launch_bgemm_t<bf16_t>(b, c, s);
  return launch_bgemm_t<float>(b, c, s);
}

int launch_breduce_tail(const BatchArgs &b, int slots, hipStream_t s) {
#define CALL(E) hipLaunchKernelGGL(k_btail<E>, dim3((unsigned)b.running), dim3(256), 0, s, b)
  BATCH_SLOT_SWITCH(slots, CALL)
#undef CALL
  return (int)hipGetLastError();
}

int launch_bproject_init(const BatchArgs &b, int slots, hipStream_t s) {
#define CALL(E) hipLaunchKernelGGL(k_bproject_init<E>, dim3((unsigned)b.m), dim3(256), 0, s, b)
  BATCH_SLOT_SWITCH(slots, CALL)
#undef CALL
  return (int)hipGetLastError();
}

int launch_bcg_init(const BatchArgs &b, int slots, hipStream_t s) {
#define CALL(E) hipLaunchKernelGGL(k_bcg_init<E>, dim3((unsigned)b.m), dim3(256), 0, s, b)
  BATCH_SLOT_SWITCH(slots, CALL)
#undef CALL
  return (int)hipGetLastError();
}

int launch_bfinalize(const BatchArgs &b, float *X, int64_t ldx_out, hipStream_t s) {
  const dim3 g((unsigned)((b.base.n + 255) / 256), (unsigned)b.m);
  hipLaunchKernelGGL(k_bfinalize, g, dim3(256), 0, s, b, X, ldx_out);
  return (int)hipGetLastError();
}

int launch_bset_x0(const BatchArgs &b, const float *X0, int64_t ldx0, hipStream_t s) {
  const dim3 g((unsigned)((b.ldx + 255) / 256), (unsigned)b.m);
  hipLaunchKernelGGL(k_bset_x0, g, dim3(256), 0, s, b, X0, ldx0);
  return (int)hipGetLastError();
}

int launch_bload_x(const BatchArgs &b, const float *X, int64_t ldx_in, hipStream_t s) {
  const dim3 g((unsigned)((b.ldx + 255) / 256), (unsigned)b.m);
  hipLaunchKernelGGL(k_bload_x, g, dim3(256), 0, s, b, X, ldx_in);
  return (int)hipGetLastError();
}

int launch_bcopy_step(const BatchArgs &b, const DevState *src, hipStream_t s) {
  hipLaunchKernelGGL(k_bcopy_step, dim3(1), dim3(256), 0, s, b, src);
  return (int)hipGetLastError();
}

int launch_bphase_reset(const BatchArgs &b, double tol, int32_t max_iter, hipStream_t s) {
  hipLaunchKernelGGL(k_bphase_reset, dim3(1), dim3(256), 0, s, b, tol, max_iter);
  return (int)hipGetLastError();
}

int launch_bcopy_anchor(const BatchArgs &b, hipStream_t s) {
  const dim3 g((unsigned)((b.base.n + 255) / 256), (unsigned)b.m);
  hipLaunchKernelGGL(k_bcopy_anchor, g, dim3(256), 0, s, b);
  return (int)hipGetLastError();
}

int launch_bstatus(const BatchArgs &b, int32_t *out, int32_t *act, int32_t *mact, hipStream_t s) {
  if (b.m > 1024) return (int)hipErrorInvalidValue;
  hipLaunchKernelGGL(k_bstatus, dim3(1), dim3(256), 0, s, b, out, act, mact);
  return (int)hipGetLastError();
}

int launch_bact_all(const BatchArgs &b, int32_t *act, int32_t *mact, hipStream_t s) {
  hipLaunchKernelGGL(k_bact_all, dim3(1), dim3(256), 0, s, b.m, act, mact);
  return (int)hipGetLastError();
}

int launch_zero_f32(float *p, int64_t count, hipStream_t s) {
  const int64_t blocks = (count + 255) / 256;
  const int g = (int)(blocks < 1024 ? (blocks < 1 ? 1 : blocks) : 1024);
  hipLaunchKernelGGL(k_zero_f32, dim3(g), dim3(256), 0, s, p, count);
  return (int)hipGetLastError();
}

}  // namespace npga
