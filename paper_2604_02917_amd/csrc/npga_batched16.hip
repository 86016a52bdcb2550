// Batched gradient GEMMs for a bfloat16 factor on the bfloat16 matrix cores
// (v_mfma_f32_32x32x16_bf16, float32 accumulation).
//
// The entries of L are exact in bfloat16.  The other operand (the float32
// iterates X, then the float32 product U) is split into three bfloat16
// planes, v = v_h + v_m + v_l with v_h = bf16(v), v_m = bf16(v - v_h),
// v_l = bf16(v - v_h - v_m) (each difference exact in float32), which
// represents v to about 2^-27 relative; three matrix-core products per tile
// then give L^T X and L U to float32 accuracy.  Both GEMMs read their
// operands contiguous along the contraction:
//   k_b16_u : U[c][t] = sum_i X[i][c] L[i][t]     (L column-major, X columns)
//   k_b16_g : P[s][c][i] = sum_{t in T_s} Lt[i][t] U[c][t]
// where Lt is a row-major copy of L made once per batched solve.  U is
// stored directly as its three bfloat16 planes.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "npga_device.h"
#include "npga_internal.h"

namespace npga {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef unsigned int u2v __attribute__((ext_vector_type(2)));

constexpr int KB16 = 32;          // contraction depth of one LDS stage
constexpr int LDH = KB16 + 8;     // LDS row length in bfloat16 (80 bytes)

// Three-plane split of one value.
__device__ __forceinline__ void split3(float v, uint32_t &h, uint32_t &m, uint32_t &l) {
  h = rne_bf16(v);
  const float r1 = v - bf16_f32(h);
  m = rne_bf16(r1);
  l = rne_bf16(r1 - bf16_f32(m));
}

__device__ __forceinline__ bf8 lds_bf8(const uint16_t *p) {
  return __builtin_bit_cast(bf8, *reinterpret_cast<const u4v *>(p));
}

// --------------------------------------------------------------------------
// U = X^T L with X split in three planes.  Tile: BM GEMM columns c (rows of
// the product) x BN periods t; WM x WN wavefronts of PM x PN 32 x 32 blocks.
// Epilogue: U as three bfloat16 planes [c][t] and per-tile sums of U^2.
// --------------------------------------------------------------------------
template <int BM, int BN, int WM, int WN>
__global__ __launch_bounds__(256) void k_b16_u(BatchArgs b) {
  constexpr int PM = BM / (32 * WM), PN = BN / (32 * WN);
  constexpr int QA = BM * KB16 / 4 / 256;  // float4 of X per thread per stage
  constexpr int QB = BN * KB16 / 8 / 256;  // 8 x bfloat16 of L per thread per stage
  static_assert(WM * WN == 4 && PM >= 1 && PN >= 1 && QA >= 1 && QB >= 1, "tile");
  __shared__ __attribute__((aligned(16))) uint16_t Ax[2][3][BM * LDH];
  __shared__ __attribute__((aligned(16))) uint16_t Bl[2][BN * LDH];
  __shared__ double ush[WN * BM];
  const int64_t T = b.base.cols, n = b.base.n;
  const int ma = *b.mact;
  const int64_t t0 = (int64_t)blockIdx.x * BN;
  const int64_t c0 = (int64_t)blockIdx.y * BM;
  if (c0 >= ma) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = wave / WN, wc = wave % WN;
  const int h = lane >> 5, r = lane & 31;
  const uint16_t *L = static_cast<const uint16_t *>(b.base.L);
  const int64_t ld = b.base.ld;

  const float *xcol[QA];
#pragma unroll
  for (int q = 0; q < QA; ++q) {
    const int64_t c = c0 + (tid >> 3) + 32 * q;
    xcol[q] = (c < ma) ? b.base.xs + (int64_t)b.act[c] * b.ldx : nullptr;
  }
  f4 xa[QA];
  u4v lb[QB];
  auto gload = [&](int64_t k0) {
    const int64_t kx = k0 + 4 * (tid & 7);
#pragma unroll
    for (int q = 0; q < QA; ++q)
      xa[q] = (xcol[q] && kx < n) ? *reinterpret_cast<const f4 *>(xcol[q] + kx) : f4{0.f, 0.f, 0.f, 0.f};
    const int64_t kl = k0 + 8 * (tid & 3);
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      const int64_t t = t0 + (tid >> 2) + 64 * q;
      lb[q] = (t < T && kl < n) ? *reinterpret_cast<const u4v *>(L + t * ld + kl) : u4v{0u, 0u, 0u, 0u};
    }
  };
  auto sstore = [&](int buf, int64_t k0) {
    const int kx = 4 * (tid & 7);
#pragma unroll
    for (int q = 0; q < QA; ++q) {
      uint32_t hh[4], mm[4], ll[4];
      split3(xa[q].x, hh[0], mm[0], ll[0]);
      split3(xa[q].y, hh[1], mm[1], ll[1]);
      split3(xa[q].z, hh[2], mm[2], ll[2]);
      split3(xa[q].w, hh[3], mm[3], ll[3]);
      const int off = ((tid >> 3) + 32 * q) * LDH + kx;
      *reinterpret_cast<u2v *>(&Ax[buf][0][off]) = u2v{hh[0] | (hh[1] << 16), hh[2] | (hh[3] << 16)};
      *reinterpret_cast<u2v *>(&Ax[buf][1][off]) = u2v{mm[0] | (mm[1] << 16), mm[2] | (mm[3] << 16)};
      *reinterpret_cast<u2v *>(&Ax[buf][2][off]) = u2v{ll[0] | (ll[1] << 16), ll[2] | (ll[3] << 16)};
    }
    const int64_t kl = k0 + 8 * (tid & 3);
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      u4v v = lb[q];
      // asset rows past n inside the group (ld may exceed n) are not data
      if (kl + 8 > n) {
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const int64_t row = kl + 2 * w;
          const uint32_t keep = row + 1 < n ? 0xffffffffu : (row < n ? 0x0000ffffu : 0u);
          v[w] &= keep;
        }
      }
      *reinterpret_cast<u4v *>(&Bl[buf][((tid >> 2) + 64 * q) * LDH + 8 * (tid & 3)]) = v;
    }
  };

  v16f acc[PM][PN];
#pragma unroll
  for (int p = 0; p < PM; ++p)
#pragma unroll
    for (int q = 0; q < PN; ++q)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[p][q][v] = 0.f;

  const int64_t nk = (n + KB16 - 1) / KB16;
  gload(0);
  sstore(0, 0);
  __syncthreads();
  for (int64_t s = 0; s < nk; ++s) {
    const int buf = (int)(s & 1);
    if (s + 1 < nk) gload((s + 1) * KB16);
#pragma unroll
    for (int ks = 0; ks < KB16 / 16; ++ks) {
      const int koff = 16 * ks + 8 * h;
      bf8 a[PM][3], bb[PN];
#pragma unroll
      for (int p = 0; p < PM; ++p)
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) a[p][pl] = lds_bf8(&Ax[buf][pl][(wr * 32 * PM + 32 * p + r) * LDH + koff]);
#pragma unroll
      for (int q = 0; q < PN; ++q) bb[q] = lds_bf8(&Bl[buf][(wc * 32 * PN + 32 * q + r) * LDH + koff]);
#pragma unroll
      for (int p = 0; p < PM; ++p)
#pragma unroll
        for (int q = 0; q < PN; ++q) {
          acc[p][q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[p][2], bb[q], acc[p][q], 0, 0, 0);
          acc[p][q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[p][1], bb[q], acc[p][q], 0, 0, 0);
          acc[p][q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[p][0], bb[q], acc[p][q], 0, 0, 0);
        }
    }
    if (s + 1 < nk) sstore(buf ^ 1, (s + 1) * KB16);
    __syncthreads();
  }

  // epilogue: U planes (coalesced along t) and row sums of U^2
  double rs[PM][16];
#pragma unroll
  for (int p = 0; p < PM; ++p)
#pragma unroll
    for (int v = 0; v < 16; ++v) rs[p][v] = 0.0;
#pragma unroll
  for (int p = 0; p < PM; ++p)
#pragma unroll
    for (int q = 0; q < PN; ++q) {
      const int64_t t = t0 + wc * 32 * PN + 32 * q + r;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int64_t c = c0 + wr * 32 * PM + 32 * p + 8 * (v >> 2) + 4 * h + (v & 3);
        const float val = acc[p][q][v];
        if (c < ma && t < T) {
          uint32_t hh, mm, ll;
          split3(val, hh, mm, ll);
          uint16_t *u = b.U16 + c * b.ldu16 + t;
          u[0] = (uint16_t)hh;
          u[b.u16plane] = (uint16_t)mm;
          u[2 * b.u16plane] = (uint16_t)ll;
        }
        rs[p][v] = fma((double)val, (double)val, rs[p][v]);  // periods t >= T are zero
      }
    }
#pragma unroll
  for (int p = 0; p < PM; ++p)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      double x = rs[p][v];
#pragma unroll
      for (int off = 1; off < 32; off <<= 1) x += __shfl_xor(x, off, 64);
      if (r == 0) ush[wc * BM + wr * 32 * PM + 32 * p + 8 * (v >> 2) + 4 * h + (v & 3)] = x;
    }
  __syncthreads();
  for (int cl = tid; cl < BM; cl += 256) {
    const int64_t c = c0 + cl;
    if (c >= ma) continue;
    double sum = 0.0;
#pragma unroll
    for (int w = 0; w < WN; ++w) sum += ush[w * BM + cl];
    b.usq_part[(int64_t)blockIdx.x * b.ldq + b.act[c]] = sum;
  }
}

// --------------------------------------------------------------------------
// U = X^T L for factors whose tiles would leave most of the chip idle (701
// periods in 128-period tiles are six workgroups, each a chain of n / 32
// stages at a memory round trip apiece: 43 us at n = 1500).  32 targets x 32
// periods a workgroup; its eight wavefronts take every eighth 16-asset step
// each, so an operand is used by one wavefront only and comes straight from
// memory to its registers, four steps ahead; the eight sums meet in LDS at
// the end (added in float64).  9.6 us at n = 1500, T = 701, 24 targets.
// --------------------------------------------------------------------------
__global__ __launch_bounds__(512) void k_b16_u_split(BatchArgs b) {
  constexpr int D = 4;  // steps in flight
  __shared__ float red[8][16][64];
  const int64_t T = b.base.cols, n = b.base.n, ld = b.base.ld;
  const int ma = *b.mact;
  const int64_t t0 = (int64_t)blockIdx.x * 32;
  const int c0 = (int)blockIdx.y * 32;
  if (c0 >= ma) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = lane >> 5, r = lane & 31;
  // lane: target c0 + r and period t0 + r, assets 8 h .. 8 h + 7 of a step;
  // targets, periods and steps past the last read the last and are dropped
  const int c = c0 + r < ma ? c0 + r : ma - 1;
  const float *X = b.base.xs + (int64_t)b.act[c] * b.ldx + 8 * h;
  const uint16_t *L = static_cast<const uint16_t *>(b.base.L) + (t0 + r < T ? t0 + r : T - 1) * ld;
  const int64_t last = (ld - 8) / 8 * 8;  // columns hold ld >= n entries, ld % 8 == 0
  const int steps = (int)((n + 15) / 16);
  const int cnt = (steps - wave + 7) >> 3;  // this wavefront's steps: wave, wave + 8, ...
  f4 xa[D][2];
  u4v lb[D];
  auto load = [&](int slot, int t) {
    const int64_t k0 = 16 * (int64_t)(wave + 8 * (t < cnt ? t : cnt - 1));
    xa[slot][0] = *reinterpret_cast<const f4 *>(X + k0);  // X columns are padded to a multiple of 256 with zeros
    xa[slot][1] = *reinterpret_cast<const f4 *>(X + k0 + 4);
    const int64_t kl = k0 + 8 * h;
    lb[slot] = *reinterpret_cast<const u4v *>(L + (kl < last ? kl : last));
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
          const float v8[8] = {xa[u][0].x, xa[u][0].y, xa[u][0].z, xa[u][0].w,
                               xa[u][1].x, xa[u][1].y, xa[u][1].z, xa[u][1].w};
          u4v w[3];
          split8(v8, w);
          // asset rows past n (ld may exceed n) are not data
          u4v lv = lb[u];
          if (k + 8 > n) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const int64_t row = k + 2 * q;
              lv[q] &= row + 1 < n ? 0xffffffffu : (row < n ? 0x0000ffffu : 0u);
            }
          }
          const bf8 bb = __builtin_bit_cast(bf8, lv);
#pragma unroll
          for (int pl = 2; pl >= 0; --pl)
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8, w[pl]), bb, acc, 0, 0, 0);
        }
        load(u, s0 + u + D);
      }
    }
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) red[wave][v][lane] = acc[v];
  __syncthreads();
  // register v of lane (h, r): target c0 + 8 (v / 4) + 4 h + v % 4, period t0 + r
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int v = 8 * e + wave;
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < 8; ++w) s += (double)red[w][v][lane];
    const float val = (t0 + r < T) ? (float)s : 0.f;
    const int cc = c0 + 8 * (v >> 2) + 4 * h + (v & 3);
    double q = (double)val * (double)val;
#pragma unroll
    for (int off = 1; off < 32; off <<= 1) q += __shfl_xor(q, off, 64);
    if (cc >= ma) continue;
    if (t0 + r < T) {
      uint32_t hh, mm, ll;
      split3(val, hh, mm, ll);
      uint16_t *u = b.U16 + (int64_t)cc * b.ldu16 + t0 + r;
      u[0] = (uint16_t)hh;
      u[b.u16plane] = (uint16_t)mm;
      u[2 * b.u16plane] = (uint16_t)ll;
    }
    if (r == 0) b.usq_part[(int64_t)blockIdx.x * b.ldq + b.act[cc]] = q;
  }
}

// --------------------------------------------------------------------------
// The same for the smallest products: 16 targets x 16 periods a workgroup,
// 32-asset steps, six ahead.  A compute unit takes the lines of a load's rows
// one after another, so few workgroups are bound by the rows each of them
// reads: n = 1500, T = 701, 24 targets (22 workgroups of 32 x 32, 88 of 16 x
// 16) 9.8 us there and 7.4 us here.  With more tiles than compute units the
// operands read twice as often cost more: n = 2000, T = 1600, 128 targets 16
// us there and 30 us here.
// --------------------------------------------------------------------------
__global__ __launch_bounds__(512) void k_b16_u_small(BatchArgs b) {
  constexpr int D = 6;  // steps in flight
  __shared__ float red[8][4][64];
  const int64_t T = b.base.cols, n = b.base.n, ld = b.base.ld;
  const int ma = *b.mact;
  const int64_t t0 = (int64_t)blockIdx.x * 16;
  const int c0 = (int)blockIdx.y * 16;
  if (c0 >= ma) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = lane >> 4, r = lane & 15;
  // lane: target c0 + r and period t0 + r, assets 8 h .. 8 h + 7 of a step;
  // targets, periods and steps past the last read the last and are dropped
  const int c = c0 + r < ma ? c0 + r : ma - 1;
  const float *X = b.base.xs + (int64_t)b.act[c] * b.ldx + 8 * h;
  const uint16_t *L = static_cast<const uint16_t *>(b.base.L) + (t0 + r < T ? t0 + r : T - 1) * ld;
  const int64_t last = (ld - 8) / 8 * 8;  // columns hold ld >= n entries, ld % 8 == 0
  const int steps = (int)((n + 31) / 32);
  const int cnt = (steps - wave + 7) >> 3;  // this wavefront's steps: wave, wave + 8, ...
  f4 xa[D][2];
  u4v lb[D];
  auto load = [&](int slot, int t) {
    const int64_t k0 = 32 * (int64_t)(wave + 8 * (t < cnt ? t : cnt - 1));
    xa[slot][0] = *reinterpret_cast<const f4 *>(X + k0);  // X columns are padded to a multiple of 256 with zeros
    xa[slot][1] = *reinterpret_cast<const f4 *>(X + k0 + 4);
    const int64_t kl = k0 + 8 * h;
    lb[slot] = *reinterpret_cast<const u4v *>(L + (kl < last ? kl : last));
  };
  f4 acc = f4{0.f, 0.f, 0.f, 0.f};
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
          const int64_t k = 32 * (int64_t)(wave + 8 * (s0 + u)) + 8 * h;
          const float v8[8] = {xa[u][0].x, xa[u][0].y, xa[u][0].z, xa[u][0].w,
                               xa[u][1].x, xa[u][1].y, xa[u][1].z, xa[u][1].w};
          u4v w[3];
          split8(v8, w);
          // asset rows past n (ld may exceed n) are not data
          u4v lv = lb[u];
          if (k + 8 > n) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const int64_t row = k + 2 * q;
              lv[q] &= row + 1 < n ? 0xffffffffu : (row < n ? 0x0000ffffu : 0u);
            }
          }
          const bf8 bb = __builtin_bit_cast(bf8, lv);
#pragma unroll
          for (int pl = 2; pl >= 0; --pl)
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8, w[pl]), bb, acc, 0, 0, 0);
        }
        if (s0 + D < cnt) load(u, s0 + u + D);
      }
    }
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) red[wave][v][lane] = acc[v];
  __syncthreads();
  if (wave >= 4) return;
  // register v = wave of lane (h, r): target c0 + 4 h + v, period t0 + r
  double s = 0.0;
#pragma unroll
  for (int w = 0; w < 8; ++w) s += (double)red[w][wave][lane];
  const float val = (t0 + r < T) ? (float)s : 0.f;
  const int cc = c0 + 4 * h + wave;
  double q = (double)val * (double)val;
#pragma unroll
  for (int off = 1; off < 16; off <<= 1) q += __shfl_xor(q, off, 64);
  if (cc >= ma) return;
  if (t0 + r < T) {
    uint32_t hh, mm, ll;
    split3(val, hh, mm, ll);
    uint16_t *u = b.U16 + (int64_t)cc * b.ldu16 + t0 + r;
    u[0] = (uint16_t)hh;
    u[b.u16plane] = (uint16_t)mm;
    u[2 * b.u16plane] = (uint16_t)ll;
  }
  if (r == 0) b.usq_part[(int64_t)blockIdx.x * b.ldq + b.act[cc]] = q;
}

// --------------------------------------------------------------------------
// P[s] = Lt_{:, T_s} U_{T_s}: BM assets x BN GEMM columns over the period
// range of split s; U's three planes give three products per step.
// --------------------------------------------------------------------------
template <int BM, int BN, int WM, int WN>
__global__ __launch_bounds__(256) void k_b16_g(BatchArgs b) {
  constexpr int PM = BM / (32 * WM), PN = BN / (32 * WN);
  constexpr int NA = BM * KB16 / 8;            // 16-byte groups of an Lt stage
  constexpr int NB = BN * KB16 / 8;            // 16-byte groups of one U plane stage
  constexpr int QA = (NA + 255) / 256, QB = (NB + 255) / 256;
  static_assert(WM * WN == 4 && PM >= 1 && PN >= 1, "tile");
  __shared__ __attribute__((aligned(16))) uint16_t As[2][BM * LDH];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[2][3][BN * LDH];
  const int64_t T = b.base.cols, n = b.base.n;
  const int ma = *b.mact;
  const int64_t i0 = (int64_t)blockIdx.x * BM;
  const int64_t tb = (int64_t)blockIdx.y * b.kchunk;
  const int64_t te = (tb + b.kchunk < T) ? tb + b.kchunk : T;
  const int64_t c0 = (int64_t)blockIdx.z * BN;
  if (c0 >= ma) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = wave / WN, wc = wave % WN;
  const int h = lane >> 5, r = lane & 31;

  u4v ra[QA], rb[3][QB];
  auto gload = [&](int64_t k0) {
#pragma unroll
    for (int q = 0; q < QA; ++q) {
      const int idx = tid + 256 * q;
      const int64_t i = i0 + (idx >> 2);
      const int64_t t = k0 + 8 * (idx & 3);
      ra[q] = (idx < NA && i < n && t < te) ? *reinterpret_cast<const u4v *>(b.Lt + i * b.ldlt + t)
                                           : u4v{0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      const int idx = tid + 256 * q;
      const int64_t c = c0 + (idx >> 2);
      const int64_t t = k0 + 8 * (idx & 3);
      const bool ok = idx < NB && c < ma && t < te;
      const uint16_t *u = b.U16 + c * b.ldu16 + t;
#pragma unroll
      for (int pl = 0; pl < 3; ++pl)
        rb[pl][q] = ok ? *reinterpret_cast<const u4v *>(u + pl * b.u16plane) : u4v{0u, 0u, 0u, 0u};
    }
  };
  auto sstore = [&](int buf) {
#pragma unroll
    for (int q = 0; q < QA; ++q) {
      const int idx = tid + 256 * q;
      if (idx < NA) *reinterpret_cast<u4v *>(&As[buf][(idx >> 2) * LDH + 8 * (idx & 3)]) = ra[q];
    }
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      const int idx = tid + 256 * q;
      if (idx < NB)
#pragma unroll
        for (int pl = 0; pl < 3; ++pl)
          *reinterpret_cast<u4v *>(&Bs[buf][pl][(idx >> 2) * LDH + 8 * (idx & 3)]) = rb[pl][q];
    }
  };

  v16f acc[PM][PN];
#pragma unroll
  for (int p = 0; p < PM; ++p)
#pragma unroll
    for (int q = 0; q < PN; ++q)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[p][q][v] = 0.f;

  const int64_t nk = (te > tb) ? (te - tb + KB16 - 1) / KB16 : 0;
  if (nk > 0) {
    gload(tb);
    sstore(0);
  }
  __syncthreads();
  for (int64_t s = 0; s < nk; ++s) {
    const int buf = (int)(s & 1);
    if (s + 1 < nk) gload(tb + (s + 1) * KB16);
#pragma unroll
    for (int ks = 0; ks < KB16 / 16; ++ks) {
      const int koff = 16 * ks + 8 * h;
      bf8 a[PM], bb[PN][3];
#pragma unroll
      for (int p = 0; p < PM; ++p) a[p] = lds_bf8(&As[buf][(wr * 32 * PM + 32 * p + r) * LDH + koff]);
#pragma unroll
      for (int q = 0; q < PN; ++q)
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) bb[q][pl] = lds_bf8(&Bs[buf][pl][(wc * 32 * PN + 32 * q + r) * LDH + koff]);
#pragma unroll
      for (int p = 0; p < PM; ++p)
#pragma unroll
        for (int q = 0; q < PN; ++q) {
          acc[p][q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bb[q][2], a[p], acc[p][q], 0, 0, 0);
          acc[p][q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bb[q][1], a[p], acc[p][q], 0, 0, 0);
          acc[p][q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bb[q][0], a[p], acc[p][q], 0, 0, 0);
        }
    }
    if (s + 1 < nk) sstore(buf ^ 1);
    __syncthreads();
  }

  // columns of the product on the output's rows, assets along the lanes
  float *P = b.P + (int64_t)blockIdx.y * b.ldpm * b.ldpi;
#pragma unroll
  for (int p = 0; p < PM; ++p)
#pragma unroll
    for (int q = 0; q < PN; ++q) {
      const int64_t i = i0 + wr * 32 * PM + 32 * p + r;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int64_t c = c0 + wc * 32 * PN + 32 * q + 8 * (v >> 2) + 4 * h + (v & 3);
        if (i < n && c < ma) P[c * b.ldpi + i] = acc[p][q][v];
      }
    }
}

// --------------------------------------------------------------------------
// P of the smallest products: 16 assets x 16 columns a workgroup, its eight
// wavefronts every eighth 32-period step each (operands straight from memory,
// four steps ahead).  Sums leave float32 after each step and meet in float64;
// the total goes out as two float32, so that a tail's sum is the float64 one.
// n = 1500, T = 701, 24 targets: 5.3 us against 4.3 us by tiles of 128 x 32 in
// 22 ranges, and a tail 11.2 us against 13.1 us, which reads one sum, not 22.
// --------------------------------------------------------------------------
__global__ __launch_bounds__(512) void k_b16_g_small(BatchArgs b) {
  constexpr int D = 4;  // steps in flight
  __shared__ double red[8][4][64];
  const int64_t T = b.base.cols, n = b.base.n;
  const int ma = *b.mact;
  const int64_t i0 = (int64_t)blockIdx.x * 16;
  const int c0 = (int)blockIdx.y * 16;
  if (c0 >= ma) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = lane >> 4, r = lane & 15;
  // lane: asset i0 + r and column c0 + r, periods 8 h .. 8 h + 7 of a step;
  // assets, columns and periods past the last read the last and are dropped
  const uint16_t *L = b.Lt + (i0 + r < n ? i0 + r : n - 1) * b.ldlt;
  const uint16_t *U = b.U16 + (int64_t)(c0 + r < ma ? c0 + r : ma - 1) * b.ldu16;
  const int64_t last = b.ldlt - 8;  // ldlt = ldu16: a multiple of 8; periods T .. ldlt - 1 are zeros
  const int steps = (int)((T + 31) / 32);
  const int cnt = (steps - wave + 7) >> 3;
  u4v la[D], ub[D][3];
  auto load = [&](int slot, int t) {
    const int64_t k0 = 32 * (int64_t)(wave + 8 * (t < cnt ? t : cnt - 1)) + 8 * h;
    const int64_t k = k0 < last ? k0 : last;
    la[slot] = *reinterpret_cast<const u4v *>(L + k);
#pragma unroll
    for (int pl = 0; pl < 3; ++pl) ub[slot][pl] = *reinterpret_cast<const u4v *>(U + pl * b.u16plane + k);
  };
  double sum[4] = {0.0, 0.0, 0.0, 0.0};
  if (cnt > 0) {
#pragma unroll
    for (int t = 0; t < D; ++t) {
      load(t, t);
      __builtin_amdgcn_sched_barrier(0);
    }
    for (int s0 = 0; s0 < cnt; s0 += D) {
#pragma unroll
      for (int u = 0; u < D; ++u) {
        const bool live = s0 + u < cnt && 32 * (int64_t)(wave + 8 * (s0 + u)) + 8 * h < T;
        u4v lv = la[u];
#pragma unroll
        for (int q = 0; q < 4; ++q) lv[q] = live ? lv[q] : 0u;
        const bf8 a = __builtin_bit_cast(bf8, lv);
        f4 acc = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int pl = 2; pl >= 0; --pl)
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8, ub[u][pl]), a, acc, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) sum[v] += (double)acc[v];
        if (s0 + D < cnt) load(u, s0 + u + D);
      }
    }
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) red[wave][v][lane] = sum[v];
  __syncthreads();
  if (wave >= 4) return;
  // register v = wave of lane (h, r): column c0 + 4 h + v, asset i0 + r
  double s = red[0][wave][lane];
#pragma unroll
  for (int w = 1; w < 8; ++w) s += red[w][wave][lane];
  const int cc = c0 + 4 * h + wave;
  if (cc < ma && i0 + r < n) {
    float *o = b.P + (int64_t)cc * b.ldpi + i0 + r;
    const float hi = (float)s;
    o[0] = hi;
    o[b.ldpm * b.ldpi] = (float)(s - (double)hi);
  }
}

// Lt[i][t] = L[i + t ld] for t < T, zero for T <= t < ldlt (64 x 64 tiles).
__global__ __launch_bounds__(256) void k_transpose16(const uint16_t *L, int64_t ld, int64_t n, int64_t T,
                                                     uint16_t *Lt, int64_t ldlt) {
  __shared__ uint16_t tile[64][66];
  const int64_t t0 = (int64_t)blockIdx.x * 64, i0 = (int64_t)blockIdx.y * 64;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  for (int k = ty; k < 64; k += 4) {
    const int64_t t = t0 + k, i = i0 + tx;
    tile[k][tx] = (t < T && i < n) ? L[t * ld + i] : (uint16_t)0;
  }
  __syncthreads();
  for (int k = ty; k < 64; k += 4) {
    const int64_t i = i0 + k, t = t0 + tx;
    if (i < n && t < ldlt) Lt[i * ldlt + t] = tile[tx][k];
  }
}

int launch_b16_gemm(const BatchArgs &b, const BatchConfig &c, hipStream_t s) {
  const int64_t T = b.base.cols, n = b.base.n;
  const int bn = c.g_bn;  // width of the target tiles
  if (b.u_split) {
    const int w = b.u_split == 2 ? 16 : 32;
    const dim3 gu((unsigned)((T + w - 1) / w), (unsigned)((b.running + w - 1) / w));
    if (w == 16)
      hipLaunchKernelGGL(k_b16_u_small, gu, dim3(512), 0, s, b);
    else
      hipLaunchKernelGGL(k_b16_u_split, gu, dim3(512), 0, s, b);
  } else if (bn == 128) {
    const dim3 gu((unsigned)((T + 63) / 64), (unsigned)((b.m + 127) / 128));
    hipLaunchKernelGGL((k_b16_u<128, 64, 2, 2>), gu, dim3(256), 0, s, b);
  } else if (bn == 64) {
    const dim3 gu((unsigned)((T + 63) / 64), (unsigned)((b.m + 63) / 64));
    hipLaunchKernelGGL((k_b16_u<64, 64, 2, 2>), gu, dim3(256), 0, s, b);
  } else {
    const dim3 gu((unsigned)((T + 127) / 128), (unsigned)((b.m + 31) / 32));
    hipLaunchKernelGGL((k_b16_u<32, 128, 1, 4>), gu, dim3(256), 0, s, b);
  }
  if (hipGetLastError() != hipSuccess) return (int)hipErrorLaunchFailure;
  const dim3 gg((unsigned)((n + 127) / 128), (unsigned)b.splits, (unsigned)((b.m + bn - 1) / bn));
  if (b.g_small)
    hipLaunchKernelGGL(k_b16_g_small, dim3((unsigned)((n + 15) / 16), (unsigned)((b.running + 15) / 16)), dim3(512), 0, s, b);
  else if (bn == 128)
    hipLaunchKernelGGL((k_b16_g<128, 128, 2, 2>), gg, dim3(256), 0, s, b);
  else if (bn == 64)
    hipLaunchKernelGGL((k_b16_g<128, 64, 2, 2>), gg, dim3(256), 0, s, b);
  else
    hipLaunchKernelGGL((k_b16_g<128, 32, 4, 1>), gg, dim3(256), 0, s, b);
  return (int)hipGetLastError();
}

int launch_transpose16(const uint16_t *L, int64_t ld, int64_t n, int64_t T, uint16_t *Lt, int64_t ldlt,
                       hipStream_t s) {
  const dim3 g((unsigned)((ldlt + 63) / 64), (unsigned)((n + 63) / 64));
  hipLaunchKernelGGL(k_transpose16, g, dim3(256), 0, s, L, ld, n, T, Lt, ldlt);
  return (int)hipGetLastError();
}

}  // namespace npga
