// Explicit-covariance path (paper Sec. 3.1: grad f(x) = 2 Sigma x at O(n^2)
// per iteration).
//
// k_syrk: Sigma = L L^T with float32 MFMA (v_mfma_f32_32x32x2_f32).  One
// workgroup computes a 128 x 128 tile of the lower triangle (eight
// wavefronts, 32 x 64 each as 1 x 2 MFMA blocks) and also writes the
// mirrored tile, so Sigma is stored full.  Columns of L (periods) are the
// reduction dimension; 32-period slices of both row panels are staged in
// LDS (double buffered).  The float32 MFMA accumulators are flushed into
// float64 registers every 256 periods, which bounds the float32 rounding
// to partial sums of 256 products.
//
// k_symv: g = 2 Sigma x + 2 gamma x.  Sigma is symmetric, so (Sigma x)_i
// is the dot product of column i with x; every wavefront owns whole columns
// (contiguous) and writes g_i directly, so no partial sums are needed.  The
// serial tail (the same one as the factor path's) is the next launch on the
// stream.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "npga_device.h"
#include "npga_internal.h"

namespace npga {

typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int kTile = 128;
constexpr int kKB = 32;          // periods per LDS stage
constexpr int kFlushStages = 8;  // float32 -> float64 flush every 256 periods

__global__ __launch_bounds__(512) void k_syrk(const float *__restrict__ L, int64_t n, int64_t T, int64_t ld,
                                              float *__restrict__ S, int64_t lds, int nb) {
  __shared__ float As[2][kKB][kTile];
  __shared__ float Bs[2][kKB][kTile];
  // triangular tile index from blockIdx; the eight XCDs receive
  // consecutive workgroups round-robin, so give each XCD a contiguous
  // range of tiles (tiles sharing a row panel) for L2 reuse
  const int ntiles = nb * (nb + 1) / 2;
  const int b = blockIdx.x;
  const int per_xcd = (ntiles + 7) / 8;
  const int tix = (b % 8) * per_xcd + (b / 8);
  if (tix >= ntiles) return;  // the map is a bijection of [0, 8 per_xcd); skip the padding
  int bi = 0;
  while ((bi + 1) * (bi + 2) / 2 <= tix) ++bi;
  const int bj = tix - bi * (bi + 1) / 2;
  const int64_t row_a = (int64_t)bi * kTile;
  const int64_t row_b = (int64_t)bj * kTile;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wr = wave >> 1, wc = wave & 1;  // rows wr*32.., columns wc*64..

  v16f acc[2];
  double acc64[2][16];
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      acc[q][v] = 0.f;
      acc64[q][v] = 0.0;
    }

  // global -> register staging: thread loads float4 index (tid % 32) of
  // columns (tid / 32) + 16 q, q = 0..1, for both panels
  const int f4i = tid & 31;
  const int colq = tid >> 5;
  f4 ra[2], rb[2];
  auto gload = [&](int64_t k0) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int64_t t = k0 + colq + 16 * q;
      const int64_t ra0 = row_a + 4 * f4i;
      const int64_t rb0 = row_b + 4 * f4i;
      f4 za = f4{0.f, 0.f, 0.f, 0.f}, zb = za;
      if (t < T) {
        if (ra0 < n) {
          za = *reinterpret_cast<const f4 *>(L + t * ld + ra0);
          if (ra0 + 1 >= n) za.y = 0.f;
          if (ra0 + 2 >= n) za.z = 0.f;
          if (ra0 + 3 >= n) za.w = 0.f;
        }
        if (rb0 < n) {
          zb = *reinterpret_cast<const f4 *>(L + t * ld + rb0);
          if (rb0 + 1 >= n) zb.y = 0.f;
          if (rb0 + 2 >= n) zb.z = 0.f;
          if (rb0 + 3 >= n) zb.w = 0.f;
        }
      }
      ra[q] = za;
      rb[q] = zb;
    }
  };
  auto sstore = [&](int buf) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      *reinterpret_cast<f4 *>(&As[buf][colq + 16 * q][4 * f4i]) = ra[q];
      *reinterpret_cast<f4 *>(&Bs[buf][colq + 16 * q][4 * f4i]) = rb[q];
    }
  };

  const int64_t nstages = (T + kKB - 1) / kKB;
  gload(0);
  sstore(0);
  __syncthreads();
  for (int64_t s = 0; s < nstages; ++s) {
    const int buf = (int)(s & 1);
    if (s + 1 < nstages) gload((s + 1) * kKB);
#pragma unroll
    for (int kk = 0; kk < kKB; kk += 2) {
      const int kr = kk + (lane >> 5);
      const float av = As[buf][kr][wr * 32 + (lane & 31)];
      float bv[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) bv[q] = Bs[buf][kr][wc * 64 + q * 32 + (lane & 31)];
#pragma unroll
      for (int q = 0; q < 2; ++q) acc[q] = __builtin_amdgcn_mfma_f32_32x32x2f32(av, bv[q], acc[q], 0, 0, 0);
    }
    if (((s + 1) % kFlushStages) == 0 || s + 1 == nstages) {
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          acc64[q][v] += (double)acc[q][v];
          acc[q][v] = 0.f;
        }
    }
    if (s + 1 < nstages) {
      sstore(buf ^ 1);
    }
    __syncthreads();
  }

  // write the tile and its mirror.  MFMA 32x32 output layout: lane l,
  // register v -> row 8 (v/4) + 4 (l/32) + (v%4), column l%32.
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int64_t r = row_a + wr * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
      const int64_t c = row_b + wc * 64 + q * 32 + (lane & 31);
      if (r < n && c < n) {
        const float val = (float)acc64[q][v];
        S[r + c * lds] = val;
        if (bi != bj) S[c + r * lds] = val;
      }
    }
}

// --------------------------------------------------------------------------
// Sigma = L L^T on the bfloat16 matrix cores with three-plane operands.
//
// Every float32 entry is split exactly into three bfloat16 planes,
// v = v_h + v_m + v_l (v_h = bf16(v), v_m = bf16(v - v_h), v_l = bf16(v -
// v_h - v_m); each difference is exact in float32), which carries 24
// significant bits.  A product of two such entries keeps the six plane
// products whose weight is at least 2^-24 of the leading one (h h, h m,
// m h, h l, m m, l h); each is exact in float32, and
// v_mfma_f32_32x32x16_bf16 accumulates them in float32, flushed to float64
// every 256 periods like the float32 kernel.  Six bfloat16 products run at
// 2.5 PFLOP/s against one float32 product at 157 TFLOP/s.
//
// Plane layout.  The planes are stored in the order the matrix instruction
// reads them: a fragment is 32 rows x 16 periods of one plane, 1 KiB, lane
// l = 32 h + r of a wavefront holding row r, periods 8 h .. 8 h + 7; a stage
// is one 16-period step of a 128-row panel, [3 planes][4 row groups] of
// fragments, 12 KiB in one piece; a panel's stages follow each other.  A
// stage goes from memory to LDS by global_load_lds (1 KiB per wavefront
// instruction, lane-linear on both sides) without passing through
// registers, every fragment is then one ds_read_b128 per lane at 16 lane
// bytes (no bank conflicts, no padding), and rows past n and periods past T
// are zeros, so the GEMM has no bounds checks.
//
// k_split_t: L (float32, column-major, ld) -> fragments; one 64 x 64 tile
//   per workgroup, transposed through LDS.
// k_split_k: the same for a matrix whose rows are contiguous along the
//   contraction (the sketch).
// k_mm16<true>: 128 x 128 tiles of the lower triangle; the mirrored tile is
//   written too.  k_mm16<false>: all tiles of C = A B (the sketch Y = L S).
// --------------------------------------------------------------------------
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

constexpr int kSplitTile = 64;
constexpr int kMmStep = 16;                  // periods of a stage
constexpr int kMmGroup = 4;                  // stages per padding unit (64 periods)
constexpr int kMmFlush = 16;                 // stages between float64 flushes (256 periods)
constexpr int kMmRing = 6;                   // stages of both panels in LDS (144 KiB)
constexpr int kTileElems = kTile * kTile;

__global__ __launch_bounds__(256) void k_split_t(const float *__restrict__ L, int64_t n, int64_t T, int64_t ld,
                                                 uint16_t *__restrict__ P, int64_t stages) {
  __shared__ float tile[kSplitTile][kSplitTile + 1];  // [t][i]
  const int tid = threadIdx.x;
  const int64_t t0 = (int64_t)blockIdx.x * kSplitTile, i0 = (int64_t)blockIdx.y * kSplitTile;
  const int il = 4 * (tid & 15);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int tl = (tid >> 4) + 16 * q;
    const int64_t t = t0 + tl, i = i0 + il;
    f4 v = f4{0.f, 0.f, 0.f, 0.f};
    if (t < T && i < n) {
      v = *reinterpret_cast<const f4 *>(L + t * ld + i);
      if (i + 1 >= n) v.y = 0.f;
      if (i + 2 >= n) v.z = 0.f;
      if (i + 3 >= n) v.w = 0.f;
    }
    tile[tl][il + 0] = v.x;
    tile[tl][il + 1] = v.y;
    tile[tl][il + 2] = v.z;
    tile[tl][il + 3] = v.w;
  }
  __syncthreads();
  // the tile's eight fragments (2 row groups x 4 stages), two per wavefront,
  // each plane written as 1 KiB in lane order
  const int lane = tid & 63, wave = tid >> 6, h = lane >> 5, r = lane & 31;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int tl = 16 * wave + 8 * h;
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = tile[tl + e][32 * q + r];
    u4v w[3];
    split8(v, w);
    uint16_t *out = frag_ptr(P, i0 / 32 + q, t0 / kMmStep + wave, stages) + 8 * lane;
#pragma unroll
    for (int pl = 0; pl < 3; ++pl) *reinterpret_cast<u4v *>(out + pl * 4 * kFrag) = w[pl];
  }
}

// Row j of X (j < rows) at X + j ldx, T entries along the contraction.  One
// fragment per wavefront iteration; four stages of one row group in a row,
// so a row's 256 bytes are read together.
__global__ __launch_bounds__(256) void k_split_k(const float *__restrict__ X, int64_t rows, int64_t T, int64_t ldx,
                                                 uint16_t *__restrict__ P, int64_t stages, int vec) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, h = lane >> 5, r = lane & 31;
  const int64_t g = blockIdx.y;
  const int64_t st0 = ((int64_t)blockIdx.x * 4 + wave) * kMmGroup;
  const int64_t j = 32 * g + r;
#pragma unroll
  for (int q = 0; q < kMmGroup; ++q) {
    const int64_t st = st0 + q;
    if (st >= stages) return;
    const int64_t t = st * kMmStep + 8 * h;
    float v[8];
    if (vec && j < rows && t + 8 <= T) {
      const f4 a = *reinterpret_cast<const f4 *>(X + j * ldx + t);
      const f4 b = *reinterpret_cast<const f4 *>(X + j * ldx + t + 4);
      v[0] = a.x, v[1] = a.y, v[2] = a.z, v[3] = a.w, v[4] = b.x, v[5] = b.y, v[6] = b.z, v[7] = b.w;
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = (j < rows && t + e < T) ? X[j * ldx + t + e] : 0.f;
    }
    u4v w[3];
    split8(v, w);
    uint16_t *out = frag_ptr(P, g, st, stages) + 8 * lane;
#pragma unroll
    for (int pl = 0; pl < 3; ++pl) *reinterpret_cast<u4v *>(out + pl * 4 * kFrag) = w[pl];
  }
}

__device__ __forceinline__ bf8 lds_bf8x(const uint16_t *p) {
  return __builtin_bit_cast(bf8, *reinterpret_cast<const u4v *>(p));
}

typedef __attribute__((address_space(1))) const void gmem_t;
typedef __attribute__((address_space(3))) void lmem_t;

// A product C = A B^T of two panel sets (A = B and the lower triangle when
// SYM), its tiles and their split over the contraction.
struct Mm16 {
  const uint16_t *PA, *PB;
  int64_t na, nb, stages;  // rows of A, rows of B, stages (a multiple of kMmGroup)
  int ta, tb;              // 128-row panels of A and B
  int full;                // tiles computed whole by one workgroup (a multiple of 256)
  int rest;                // the remaining tiles, each split into `parts` stage ranges
  int parts;
  int64_t part_stages;     // stages of a range (a multiple of kMmFlush when parts > 1)
  double *partial;         // rest x parts float64 tiles (parts > 1)
  float *C;
  int64_t ldc;
};

// Tile `tix` of the sequence all workgroups follow: four panel rows at a
// time, column by column, so that the ~32 tiles an XCD has in flight lie in
// a 4 x 8 block (12 panels through its L2 instead of 33).
template <bool SYM>
__device__ __forceinline__ void mm16_tile(const Mm16 &m, int tix, int &bi, int &bj) {
  int b0 = 0, g = (m.ta & 3) ? (m.ta & 3) : 4;  // first row and height of the band
  if (SYM) {
    for (;;) {
      const int cnt = g * b0 + g * (g + 1) / 2;
      if (tix < cnt) break;
      tix -= cnt;
      b0 += g;
      g = 4;
    }
    if (tix < g * (b0 + 1)) {
      bj = tix / g;
      bi = b0 + tix % g;
      return;
    }
    tix -= g * (b0 + 1);
    int j = 1;
    while (tix >= g - j) {
      tix -= g - j;
      ++j;
    }
    bj = b0 + j;
    bi = b0 + j + tix;
  } else {
    for (;;) {
      const int cnt = g * m.tb;
      if (tix < cnt) break;
      tix -= cnt;
      b0 += g;
      g = 4;
    }
    bj = tix / g;
    bi = b0 + tix % g;
  }
}

// Element e of a lane's 64 accumulators (block q = (a, b) of 2 x 2, register
// v) in the 128 x 128 tile; 32 x 32 output layout: lane (h, r), register v
// -> row 8 (v/4) + 4 h + (v%4), column r.
template <bool SYM>
__device__ __forceinline__ void mm16_store(const Mm16 &m, int bi, int bj, int wr, int wc, int h, int r, int q, int v,
                                           float val) {
  const int64_t rr = (int64_t)bi * kTile + wr * 64 + 32 * (q >> 1) + 8 * (v >> 2) + 4 * h + (v & 3);
  const int64_t cc = (int64_t)bj * kTile + wc * 64 + 32 * (q & 1) + r;
  if (SYM) {
    // the plane products of (i, j) and (j, i) are summed in different
    // orders, so a diagonal tile keeps its lower half and mirrors it
    if (rr < m.na && cc < m.na && (bi != bj || rr >= cc)) {
      m.C[rr + cc * m.ldc] = val;
      m.C[cc + rr * m.ldc] = val;
    }
  } else if (rr < m.na && cc < m.nb) {
    m.C[rr + cc * m.ldc] = val;
  }
}

// Four wavefronts, one per SIMD, 64 x 64 of the tile each (2 x 2 blocks,
// float32 accumulators with a float64 total: 64 + 128 registers; 64 x 64 is
// the largest block whose totals fit beside two register sets of
// fragments).  Per stage and compute unit: 768 cycles of matrix
// instructions, 384 of LDS reads, 384 of loads at 64 bytes a cycle.  With
// everything but the matrix instructions taken out the loads and LDS reads
// took 4.6 ms at n = 5440, T = 48384, the matrix instructions alone 4.2, the
// kernel 6.5 (1.32 PFLOP/s of plane products) called again and again, 7.4 to
// 7.8 in the trace of a training step (issuing a stage's six loads in one go
// instead of between the products: 7.1 and not 6.5).  Before, with eight
// wavefronts of 32 x 64, register staging and padded LDS rows: 11.1 ms at
// that size (planes and product together, n = 4000, T = 16000: 2.74 ms, now
// 1.32; n = 501, T = 2003: 103 us for the product, now 15 and the join's 12).
template <bool SYM>
__global__ __launch_bounds__(256, 1) void k_mm16(Mm16 m) {
  __shared__ __attribute__((aligned(16))) uint16_t ring[kMmRing * 2 * kPanelStage];
  const int u = blockIdx.x;
  int tix, part = 0;
  if (u < m.full) {
    tix = (u & 7) * (m.full >> 3) + (u >> 3);  // consecutive tiles on one XCD
  } else {
    const int units = m.rest * m.parts;
    const int per_xcd = (units + 7) >> 3;
    const int e = (u & 7) * per_xcd + ((u - m.full) >> 3);
    if (e >= units) return;
    part = e / m.rest;
    tix = m.full + e % m.rest;
  }
  int bi = 0, bj = 0;
  mm16_tile<SYM>(m, tix, bi, bj);
  const bool split = u >= m.full && m.parts > 1;
  const int64_t s0 = split ? part * m.part_stages : 0;
  const int64_t s1 = split ? (s0 + m.part_stages < m.stages ? s0 + m.part_stages : m.stages) : m.stages;
  const int ns = (int)(s1 - s0);

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = wave >> 1, wc = wave & 1;

  // staging: wavefronts 0, 1 bring the A panel's fragments, 2, 3 the B
  // panel's, six each
  const uint16_t *src = (wave < 2 ? m.PA + ((int64_t)bi * m.stages + s0) * kPanelStage
                                  : (SYM ? m.PA : m.PB) + ((int64_t)bj * m.stages + s0) * kPanelStage) +
                        (wave & 1) * 6 * kFrag + 8 * lane;
  const int dst = (wave >> 1) * kPanelStage + (wave & 1) * 6 * kFrag;
  int issued = 0, wbuf = 0;
  // past the last stage the last one is fetched again (never read), so that
  // every step has the same number of loads in flight
  // (a stage's six loads are spread between its products: the compute unit
  // takes 64 bytes a cycle, and a wavefront waits at a load that does not
  // fit in the queue)
  auto issue = [&](auto j_c) {
    constexpr int j = decltype(j_c)::value;
    __builtin_amdgcn_global_load_lds((gmem_t *)(src + (j / 3) * 3 * kFrag),
                                     (lmem_t *)(ring + wbuf + dst + (j / 3) * 3 * kFrag), 16, (j % 3) * 1024, 0);
  };
  auto issued_stage = [&]() {
    if (++issued < ns) src += kPanelStage;
    wbuf += 2 * kPanelStage;
    if (wbuf == kMmRing * 2 * kPanelStage) wbuf = 0;
  };
#define MM16_J(j) std::integral_constant<int, j>{}

  v16f acc[4];
  double tot[4][16];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      acc[q][v] = 0.f;
      tot[q][v] = 0.0;
    }
  auto flush = [&](int q, int v0, int v1) {
#pragma unroll
    for (int v = v0; v < v1; ++v) {
      tot[q][v] += (double)acc[q][v];
      acc[q][v] = 0.f;
    }
  };

  bf8 fa[2][2][3], fb[2][2][3];  // two register sets: this stage's and the next's
  int rbuf = 0;
  const int aoff = 2 * wr * kFrag + 8 * lane, boff = kPanelStage + 2 * wc * kFrag + 8 * lane;
  // pair i = 0..5 of a stage's twelve fragments (plane 2 first: the first
  // products need planes 2 of A and 0 of B)
  auto fetch_pair = [&](int set, int i) {
    const uint16_t *l = ring + rbuf;
    const int g = i & 1, pl = i >> 1;
    fa[set][g][2 - pl] = lds_bf8x(l + aoff + (4 * (2 - pl) + g) * kFrag);
    fb[set][g][pl] = lds_bf8x(l + boff + (4 * pl + g) * kFrag);
  };
  auto fetched = [&]() {
    rbuf += 2 * kPanelStage;
    if (rbuf == kMmRing * 2 * kPanelStage) rbuf = 0;
  };
  auto mma1 = [&](int set, int q, int pa, int pb) {
    acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[set][q >> 1][pa], fb[set][q & 1][pb], acc[q], 0, 0, 0);
  };
  // plane products, smallest terms first
  constexpr int ka[6] = {2, 1, 0, 1, 0, 0}, kb[6] = {0, 1, 2, 0, 1, 0};
  // One stage: wait for the next stage's data (its loads are older than the
  // 6 (kMmRing - 2) newest) and for this stage's LDS reads, meet the other
  // wavefronts; then six groups of products, each with a sixth of the
  // refill of the buffer this stage was read from and of the next stage's
  // reads into the other register set.  fq >= 0: block fq's float32 sums go
  // to its float64 total beside the other three blocks' products, its own
  // products come last.  The scheduling barriers keep this order.
  auto step = [&](auto set_c, auto fq_c) {
    constexpr int set = decltype(set_c)::value, fq = decltype(fq_c)::value;
    asm volatile("s_waitcnt vmcnt(24) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    auto part = [&](auto k_c) {
      constexpr int k = decltype(k_c)::value;
      fetch_pair(set ^ 1, k);
      issue(k_c);
      if constexpr (fq < 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q) mma1(set, q, ka[k], kb[k]);
      } else {
#pragma unroll
        for (int q = 1; q < 4; ++q) mma1(set, (fq + q) & 3, ka[k], kb[k]);
        if constexpr (k > 0) flush(fq, 4 * (k - 1), k < 5 ? 4 * k : 16);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    part(MM16_J(0)), part(MM16_J(1)), part(MM16_J(2)), part(MM16_J(3)), part(MM16_J(4)), part(MM16_J(5));
    if constexpr (fq >= 0) {
#pragma unroll
      for (int k = 0; k < 6; ++k) mma1(set, fq, ka[k], kb[k]);
      __builtin_amdgcn_sched_barrier(0);
    }
    issued_stage();
    fetched();
  };
#define MM16_STEP(set, fq) step(MM16_J(set), MM16_J(fq))
  static_assert(6 * (kMmRing - 2) == 24 && 6 * (kMmRing - 1) == 30, "loads in flight behind a stage");
#pragma unroll
  for (int s = 0; s < kMmRing; ++s) {
    issue(MM16_J(0)), issue(MM16_J(1)), issue(MM16_J(2)), issue(MM16_J(3)), issue(MM16_J(4)), issue(MM16_J(5));
    issued_stage();
  }
  asm volatile("s_waitcnt vmcnt(30)\n\ts_barrier" ::: "memory");
#pragma unroll
  for (int k = 0; k < 6; ++k) fetch_pair(0, k);
  fetched();
  int s = 0;
  for (; s + kMmFlush <= ns; s += kMmFlush) {
    // each block's flush comes at its own quarter of the period
    MM16_STEP(0, 0), MM16_STEP(1, -1), MM16_STEP(0, -1), MM16_STEP(1, -1);
    MM16_STEP(0, 1), MM16_STEP(1, -1), MM16_STEP(0, -1), MM16_STEP(1, -1);
    MM16_STEP(0, 2), MM16_STEP(1, -1), MM16_STEP(0, -1), MM16_STEP(1, -1);
    MM16_STEP(0, 3), MM16_STEP(1, -1), MM16_STEP(0, -1), MM16_STEP(1, -1);
  }
  if (s > 0 && s < ns) {
    // 4, 8 or 12 stages are left.  They begin new sums: block 0 holds a whole
    // period by now, and without this its last sum ran over up to 28 stages.
    // (Flushes at the quarters of the last, shorter period instead: 7.27 ms
    // against 7.11 at n = 5440, T = 48374, more registers live in the loop.)
#pragma unroll
    for (int q = 0; q < 4; ++q) flush(q, 0, 16);
  }
  for (; s < ns; s += 2) MM16_STEP(0, -1), MM16_STEP(1, -1);
#undef MM16_STEP
#undef MM16_J
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no load may still write this workgroup's LDS at its end
#pragma unroll
  for (int q = 0; q < 4; ++q) flush(q, 0, 16);

  if (split) {
    double *out = m.partial + ((int64_t)(tix - m.full) * m.parts + part) * kTileElems + threadIdx.x;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int v = 0; v < 16; ++v) out[(16 * q + v) * 256] = tot[q][v];
    return;
  }
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int v = 0; v < 16; ++v) mm16_store<SYM>(m, bi, bj, wr, wc, lane >> 5, lane & 31, q, v, (float)tot[q][v]);
}

// The split tiles: their ranges' float64 sums added in range order.  Grid:
// (tiles, 4 blocks of a tile).
template <bool SYM>
__global__ __launch_bounds__(256) void k_mm16_join(Mm16 m) {
  const int tix = m.full + blockIdx.x, q = blockIdx.y;
  int bi = 0, bj = 0;
  mm16_tile<SYM>(m, tix, bi, bj);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const double *in = m.partial + (int64_t)blockIdx.x * m.parts * kTileElems + 16 * q * 256 + threadIdx.x;
  double t[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) t[v] = in[v * 256];
  for (int p = 1; p < m.parts; ++p)
#pragma unroll
    for (int v = 0; v < 16; ++v) t[v] += in[(int64_t)p * kTileElems + v * 256];
#pragma unroll
  for (int v = 0; v < 16; ++v)
    mm16_store<SYM>(m, bi, bj, wave >> 1, wave & 1, lane >> 5, lane & 31, q, v, (float)t[v]);
}

namespace {

constexpr int kMmUnits = 256;     // workgroups in flight: one per compute unit
constexpr int kMmMaxParts = 768;  // float64 tiles of split sums (96 MiB)

int64_t mm16_stages(int64_t T) {
  return (T + kMmStep * kMmGroup - 1) / (kMmStep * kMmGroup) * kMmGroup;
}
int64_t panel_elems(int64_t rows, int64_t T) { return (rows + kTile - 1) / kTile * mm16_stages(T) * kPanelStage; }

// Whole tiles in rounds of one per compute unit; what is left over would
// occupy a last round only partly (n = 4000: 16 of 528 tiles, a third
// round as long as the others), so each left-over tile is cut into stage
// ranges, as many as make the extra rounds shortest; a range costs about 30
// stages (its float64 tile written and added again).
void mm16_plan(Mm16 &m, int64_t tiles) {
  m.full = (int)(tiles / kMmUnits * kMmUnits);
  m.rest = (int)(tiles - m.full);
  m.parts = 1;
  m.part_stages = m.stages;
  if (m.rest == 0) return;
  int64_t best = m.stages;
  for (int p = 2; p <= 64 && (int64_t)p * m.rest <= kMmMaxParts; ++p) {
    const int64_t len = ((m.stages + p - 1) / p + kMmFlush - 1) / kMmFlush * kMmFlush;
    const int64_t cnt = (m.stages + len - 1) / len;
    if (cnt != p) continue;
    const int64_t cost = (cnt * m.rest + kMmUnits - 1) / kMmUnits * len + 30;
    if (cost < best) {
      best = cost;
      m.parts = p;
      m.part_stages = len;
    }
  }
}

int64_t mm16_tiles(bool sym, int64_t ta, int64_t tb) { return sym ? ta * (ta + 1) / 2 : ta * tb; }

size_t mm16_partial_bytes(bool sym, int64_t na, int64_t nb, int64_t T) {
  Mm16 m{};
  m.stages = mm16_stages(T);
  mm16_plan(m, mm16_tiles(sym, (na + kTile - 1) / kTile, (nb + kTile - 1) / kTile));
  return m.parts > 1 ? sizeof(double) * (size_t)m.rest * (size_t)m.parts * kTileElems : 0;
}

template <bool SYM>
int launch_mm16(Mm16 m, hipStream_t s) {
  m.ta = (int)((m.na + kTile - 1) / kTile);
  m.tb = (int)((m.nb + kTile - 1) / kTile);
  mm16_plan(m, mm16_tiles(SYM, m.ta, m.tb));
  const int grid = m.full + (m.rest * m.parts + 7) / 8 * 8;
  hipLaunchKernelGGL(k_mm16<SYM>, dim3(grid), dim3(256), 0, s, m);
  if (m.parts > 1) {
    if (hipGetLastError() != hipSuccess) return (int)hipErrorLaunchFailure;
    hipLaunchKernelGGL(k_mm16_join<SYM>, dim3(m.rest, 4), dim3(256), 0, s, m);
  }
  return (int)hipGetLastError();
}

int launch_split_t(const float *A, int64_t n, int64_t T, int64_t ld, uint16_t *P, hipStream_t s) {
  const int64_t stages = mm16_stages(T);
  const int64_t rows = (n + kTile - 1) / kTile * kTile;
  hipLaunchKernelGGL(k_split_t, dim3((unsigned)(stages / kMmGroup), (unsigned)(rows / kSplitTile)), dim3(256), 0, s,
                     A, n, T, ld, P, stages);
  return (int)hipGetLastError();
}

}  // namespace

size_t syrk_split_bytes(int64_t n, int64_t T) {
  return sizeof(uint16_t) * (size_t)panel_elems(n, T) + mm16_partial_bytes(true, n, n, T);
}

int launch_syrk_split(const float *L, int64_t n, int64_t T, int64_t ld, uint16_t *planes, float *Sigma,
                      int64_t lds, hipStream_t s) {
  if (launch_split_t(L, n, T, ld, planes, s)) return (int)hipErrorLaunchFailure;
  Mm16 m{};
  m.PA = m.PB = planes;
  m.na = m.nb = n;
  m.stages = mm16_stages(T);
  m.partial = reinterpret_cast<double *>(planes + panel_elems(n, T));
  m.C = Sigma;
  m.ldc = lds;
  return launch_mm16<true>(m, s);
}

size_t gemm_split_bytes(int64_t m, int64_t ncols, int64_t K) {
  return sizeof(uint16_t) * (size_t)(panel_elems(m, K) + panel_elems(ncols, K)) +
         mm16_partial_bytes(false, m, ncols, K);
}

int64_t split_stages(int64_t T) { return mm16_stages(T); }
int64_t split_k_elems(int64_t rows, int64_t T) { return panel_elems(rows, T); }

int launch_split_k(const float *X, int64_t rows, int64_t T, int64_t ldx, uint16_t *P, hipStream_t s) {
  const int64_t stages = mm16_stages(T);
  const int64_t groups = (rows + kTile - 1) / kTile * (kTile / 32);
  const int vec = (ldx % 4) == 0 && (reinterpret_cast<uintptr_t>(X) % 16) == 0;
  hipLaunchKernelGGL(k_split_k, dim3((unsigned)((stages + 15) / 16), (unsigned)groups), dim3(256), 0, s, X, rows, T,
                     ldx, P, stages, vec);
  return (int)hipGetLastError();
}

int launch_gemm_split(const float *A, int64_t lda, const float *B, int64_t ldb, float *C, int64_t ldc, int64_t M,
                      int64_t N, int64_t K, uint16_t *planes, hipStream_t s) {
  const int64_t stages = mm16_stages(K);
  uint16_t *PB = planes + panel_elems(M, K);
  if (launch_split_t(A, M, K, lda, planes, s)) return (int)hipErrorLaunchFailure;
  if (launch_split_k(B, N, K, ldb, PB, s)) return (int)hipErrorLaunchFailure;
  Mm16 m{};
  m.PA = planes;
  m.PB = PB;
  m.na = M;
  m.nb = N;
  m.stages = stages;
  m.partial = reinterpret_cast<double *>(PB + panel_elems(N, K));
  m.C = C;
  m.ldc = ldc;
  return launch_mm16<false>(m, s);
}

// g = 2 Sigma x (+ 2 gamma x); the serial tail runs as a separate launch.
// A wavefront per column, the next column's loads in flight while the
// current one is reduced (Sigma, 118 MB at n = 5440, stays in the MALL
// between iterations, so the loads are ordinary cached ones).
template <int E>
__global__ __launch_bounds__(256) void k_symv(SolveArgs a, const float *__restrict__ S, int64_t lds) {
  DevState *st = a.st;
  if (st->done != kRunning) return;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int64_t n = a.n;
  const int64_t W = (int64_t)gridDim.x * 4;
  const bool ragged = (n & 3) != 0;
  f4 xr[E];
#pragma unroll
  for (int j = 0; j < E; ++j) xr[j] = *reinterpret_cast<const f4 *>(a.xs + 4 * lane + 256 * j);
  const int cur = (a.mode == kTailNpga) ? (st->iter & 1) : 0;
  const double *xk = cur ? a.xbuf1 : a.xbuf0;
  double *gk = (a.mode == kTailNpga) ? (cur ? a.gbuf1 : a.gbuf0) : a.gbuf0;
  const double *pv = a.pvec;
  auto load = [&](f4(&c)[E], int64_t col) {
    const f4 *p = reinterpret_cast<const f4 *>(S + col * lds) + lane;
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const int64_t row0 = 4 * lane + 256 * j;
      c[j] = (row0 < n) ? p[64 * j] : f4{0.f, 0.f, 0.f, 0.f};
    }
  };
  auto process = [&](f4(&c)[E], int64_t col) {
    float d = 0.f;
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const int64_t row0 = 4 * lane + 256 * j;
      if (ragged) {
        if (row0 + 1 >= n) c[j].y = 0.f;
        if (row0 + 2 >= n) c[j].z = 0.f;
        if (row0 + 3 >= n) c[j].w = 0.f;
      }
      d = fmaf(c[j].x, xr[j].x, d);
      d = fmaf(c[j].y, xr[j].y, d);
      d = fmaf(c[j].z, xr[j].z, d);
      d = fmaf(c[j].w, xr[j].w, d);
    }
    d = wave_sum_f32(d);
    if (lane == 0) {
      if (a.mode == kTailPower || a.mode == kTailLanczos)
        gk[col] = (double)d;
      else if (a.mode == kTailCG || a.mode == kTailPdas || a.mode == kTailAdj)
        gk[col] = 2.0 * (double)d + 2.0 * st->gamma * pv[col];
      else
        npga_store_grad_step(a, st, col, 2.0 * (double)d + (a.ga ? a.ga[col] : 0.0) + 2.0 * st->gamma * xk[col]);
    }
  };
  f4 c0[E], c1[E];
  int64_t col = (int64_t)blockIdx.x * 4 + wave;
  if (col < n) load(c0, col);
  while (col < n) {
    const int64_t col1 = col + W;
    if (col1 < n) load(c1, col1);
    process(c0, col);
    if (col1 >= n) break;
    const int64_t col2 = col1 + W;
    if (col2 < n) load(c0, col2);
    process(c1, col1);
    col = col2;
  }
}

int launch_syrk(const float *L, int64_t n, int64_t T, int64_t ld, float *Sigma, int64_t lds,
                hipStream_t s) {
  const int nb = (int)((n + kTile - 1) / kTile);
  const int ntiles = nb * (nb + 1) / 2;
  const int grid = ((ntiles + 7) / 8) * 8;
  hipLaunchKernelGGL(k_syrk, dim3(grid), dim3(512), 0, s, L, n, T, ld, Sigma, lds, nb);
  return (int)hipGetLastError();
}

#define SYMV_SLOT_SWITCH(slots, CALL)            \
  switch (slots) {                               \
    case 1: CALL(1); break;                      \
    case 2: CALL(2); break;                      \
    case 4: CALL(4); break;                      \
    case 8: CALL(8); break;                      \
    case 12: CALL(12); break;                    \
    case 16: CALL(16); break;                    \
    case 22: CALL(22); break;                    \
    case 28: CALL(28); break;                    \
    case 32: CALL(32); break;                    \
    default: return (int)hipErrorInvalidValue;   \
  }

int launch_symv(const SolveArgs &a, const float *Sigma, int64_t lds, int slots, hipStream_t s) {
#define CALL(E) hipLaunchKernelGGL(k_symv<E>, dim3(a.sweep_grid), dim3(256), 0, s, a, Sigma, lds)
  SYMV_SLOT_SWITCH(slots, CALL)
#undef CALL
  return (int)hipGetLastError();
}

int launch_symv_tail(const SolveArgs &a, const float *Sigma, int64_t lds, int slots, hipStream_t s) {
  if (launch_symv(a, Sigma, lds, slots, s)) return (int)hipErrorLaunchFailure;
  return launch_tail(a, slots, 1, s);
}

}  // namespace npga
