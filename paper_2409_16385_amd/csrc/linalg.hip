// Dense FP64 Cholesky factorization and solves for the reduced Newton system
// of one implicit step (used by the adjoint of a converged step).
//
// A is row-major with leading dimension lda; only its lower triangle is read
// and the factor L (A = L L^T) overwrites it.  Two-level blocked
// right-looking algorithm without scratch memory:
//   * inner steps of NB = 64 columns: the rows below the factored diagonal
//     tile are solved against it (k_chol_panel), then the tiles of the rest
//     of the outer block are updated with these 64 columns;
//   * outer blocks of OB = 256 columns: the trailing matrix is read and
//     written once per 256 columns, not once per 64 (at 64 that traffic
//     alone, 19 GB at n = 7644, costs 4 ms at the rate of a copy).
// Both updates run on the FP64 matrix cores (k_chol_update), and the
// workgroup that updates the next diagonal tile factors it at once, so an
// inner step is two launches.
#include <algorithm>
#include <cmath>

#include "common.h"

namespace eipc {

constexpr int NB = 64;        // inner block (columns per panel)
constexpr int NBP = NB + 1;   // LDS row padding
constexpr int OB = 256;       // outer block

typedef double v4d __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double lane_value(double v, int lane) {
  const uint64_t b = __double_as_longlong(v);
  const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)b, lane);
  const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), lane);
  return __longlong_as_double(((uint64_t)hi << 32) | lo);
}

// Factors the 64x64 tile s (lower triangle; LDS) in place, by the first four
// wavefronts of a workgroup.  Wavefront w holds columns 16 w .. 16 w + 15, lane = row:
// in step p wavefront p factors its 16 columns for all rows, passing column
// entries between lanes by readlane, and the later wavefronts apply them.
// Bound by the serial chain of 64 pivots.  k0 + 64 may pass n: the caller
// pads with the unit matrix.
__device__ __forceinline__ void chol_tile(double (*s)[NBP], int64_t n, int64_t k0, int64_t *info) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  double a[16] = {};
  if (w < 4) {
#pragma unroll
    for (int j = 0; j < 16; ++j) a[j] = s[lane][16 * w + j];
  }
  for (int p = 0; p < 4; ++p) {
    if (w == p) {
      int bad = NB;
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int c = 16 * p + j;
        double d = lane_value(a[j], c);
        // no branch on the pivots' chain: a bad one is replaced by 1 (the
        // factor stays finite) and reported after the panel
        const bool ok = d > 0.0 && d < INFINITY;
        bad = ok || bad < NB ? bad : c;
        d = ok ? d : 1.0;
        // 1 / sqrt(d): the hardware estimate (2^-24 or better) and one
        // third-order step
        double ri = __builtin_amdgcn_rsq(d);
        const double e = fma(-(d * ri), ri, 1.0);
        ri = fma(ri * e, fma(e, 0.375, 0.5), ri);
        a[j] = (lane == c ? d : a[j]) * ri;
#pragma unroll
        for (int l = j + 1; l < 16; ++l) a[l] -= a[j] * lane_value(a[j], 16 * p + l);
      }
      if (bad < NB && lane == 0 && k0 + bad < n)
        atomicCAS((unsigned long long *)info, 0ull, (unsigned long long)(k0 + bad + 1));
#pragma unroll
      for (int j = 0; j < 16; ++j) s[lane][16 * p + j] = a[j];
    }
    __syncthreads();
    if (w > p && w < 4) {
      double x[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) x[j] = s[lane][16 * p + j];
#pragma unroll
      for (int l = 0; l < 16; ++l)
#pragma unroll
        for (int j = 0; j < 16; ++j) a[l] -= x[j] * s[16 * w + l][16 * p + j];
    }
  }
}

// the diagonal tile at k0, loaded into s (unit matrix past n)
__device__ __forceinline__ void load_diag(double (*s)[NBP], const double *A, int64_t n, int64_t lda, int64_t k0) {
  // all loads first (a loop of load and store waits for each in turn: 1 us a
  // round), addresses clamped into the lower triangle's rows
  double v[16];
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int e = u * 256 + (int)threadIdx.x, r = e / NB, c = e % NB;
    const int64_t rr = k0 + r < n ? k0 + r : n - 1;
    v[u] = A[rr * lda + k0 + (k0 + c <= rr ? c : 0)];
  }
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int e = u * 256 + (int)threadIdx.x, r = e / NB, c = e % NB;
    s[r][c] = (k0 + r < n && c <= r) ? v[u] : (r == c ? 1.0 : 0.0);
  }
}
__device__ __forceinline__ void store_diag(const double (*s)[NBP], double *A, int64_t n, int64_t lda, int64_t k0) {
  for (int e = threadIdx.x; e < NB * NB; e += blockDim.x) {
    const int r = e / NB, c = e % NB;
    if (c <= r && k0 + r < n) A[(k0 + r) * lda + k0 + c] = s[r][c];
  }
}

__global__ __launch_bounds__(256) void k_chol_diag(double *A, int64_t n, int64_t lda, int64_t k0, int64_t *info) {
  __shared__ double s[NB][NBP];
  load_diag(s, A, n, lda, k0);
  __syncthreads();
  chol_tile(s, n, k0, info);
  __syncthreads();
  store_diag(s, A, n, lda, k0);
}

// Rows below the diagonal tile: X L_kk^T = A_ik, 64 rows per workgroup, 16
// per wavefront, as the transposed system L_kk Y = A_ik^T in blocks of 16:
// Y_p = inv(L_pp) (C_p - sum_{q < p} L_pq Y_q) on the matrix cores.  The
// product's result layout (row 4 e + lane / 16, column lane % 16) is the
// layout its right operand takes, so Y stays in registers.  The four 16x16
// inverses are formed in LDS, one column per lane of the first wavefront.
// Y_p is corrected once by its residual, Y_p += inv(L_pp) (D_p - L_pp Y_p):
// with the inverse alone the error grows with the condition of L_pp, and on
// matrices of stiff contacts (1e13) the factor's, relative to the diagonal,
// was 4.5e-15 at n = 1100 and 1.8e-14 at n = 200, where substitution has
// 5e-16 and 6e-16.
// (One row per lane and 2,016 FMA with L broadcast from LDS took 17 us more.)
__global__ __launch_bounds__(256) void k_chol_panel(double *A, int64_t n, int64_t lda, int64_t k0) {
  __shared__ double Ls[NB][NBP + 1];
  __shared__ double Iv[NB][17];  // row 16 p + i, column j: inv(L_pp)[i][j]
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  const int64_t r = k0 + NB * (1 + (int64_t)blockIdx.x) + 16 * w + lr;
  double *row = A + (r < n ? r : n - 1) * lda + k0;  // rows past n: clamped, not stored
  double vl[16];
  v4d c[4];
#pragma unroll
  for (int u = 0; u < 16; ++u) vl[u] = A[(k0 + u * 4 + w) * lda + k0 + lane];
#pragma unroll
  for (int p = 0; p < 4; ++p)
#pragma unroll
    for (int e = 0; e < 4; ++e) c[p][e] = row[16 * p + 4 * e + lk];
#pragma unroll
  for (int u = 0; u < 16; ++u) Ls[u * 4 + w][lane] = vl[u];
  __syncthreads();
  if (w == 0) {
    const double rd = 1.0 / Ls[lane][lane];
    double z[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) z[i] = i == lr ? 1.0 : 0.0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      z[i] *= __shfl(rd, 16 * lk + i, 64);
#pragma unroll
      for (int l = i + 1; l < 16; ++l) z[l] -= Ls[16 * lk + l][16 * lk + i] * z[i];
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) Iv[16 * lk + i][lr] = z[i];
  }
  __syncthreads();
  v4d y[4];
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    v4d sum = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < p; ++q)
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
        sum = __builtin_amdgcn_mfma_f64_16x16x4f64(Ls[16 * p + lr][16 * q + 4 * kk + lk], y[q][kk], sum, 0, 0, 0);
    const v4d d = c[p] - sum;
    y[p] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
      y[p] = __builtin_amdgcn_mfma_f64_16x16x4f64(Iv[16 * p + lr][4 * kk + lk], d[kk], y[p], 0, 0, 0);
    v4d ly = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const double l = Ls[16 * p + lr][16 * p + 4 * kk + lk];
      ly = __builtin_amdgcn_mfma_f64_16x16x4f64(4 * kk + lk <= lr ? l : 0.0, y[p][kk], ly, 0, 0, 0);
    }
    const v4d res = d - ly;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
      y[p] = __builtin_amdgcn_mfma_f64_16x16x4f64(Iv[16 * p + lr][4 * kk + lk], res[kk], y[p], 0, 0, 0);
  }
  if (r < n) {
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
      for (int e = 0; e < 4; ++e) row[16 * p + 4 * e + lk] = y[p][e];
  }
}

// Update A_ij -= P_i P_j^T of the lower tiles with columns in [r0, c_end),
// P the K finished columns from kc (K a multiple of NB, kc + K <= r0).  Tile
// TM x TM over 2 x 2 wavefronts (TM = 64) or 2 x 4 (TM = 128), each its part
// of it as products of v_mfma_f64_16x16x4; the operands go through LDS 16
// columns at a time, the next 16 loaded into registers meanwhile.  TM = 128
// halves the operand traffic of 64 and serves the trailing matrix; TM = 64
// serves the outer block's few columns and short remainders, where 128 leaves
// most of the 256 CUs without a tile.
// A run of products sums 64 columns and is then added to the tile's sum: one
// run over all 256 doubled the factor's error (dense matrix of condition
// 1e6, n = 1100: |A - L L^T| / |A| 4.2e-16; 2.2e-16 like this, as with 64
// columns at a time).  The second set of sums takes the registers of four
// wavefronts at TM = 128, hence eight (7,644 unknowns 9.95 and 9.60 ms).
// The first workgroup's tile holds the next diagonal tile, which it factors
// at once.  tri: the grid is the packed lower triangle of tiles, else (row
// tile, column tile).
constexpr int upd_threads(int tm) { return tm == 128 ? 512 : 256; }

template <int TM>
__global__ __launch_bounds__(upd_threads(TM)) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_chol_update(
    double *A, int64_t n, int64_t lda, int64_t kc, int K, int64_t r0, int64_t c_end, int tri, int64_t *info) {
  constexpr int KB = 16, KP = KB + 2;        // stride of 36 banks: 16 rows x 2 columns without conflict
  constexpr int TH = upd_threads(TM), WC = TH / 128;  // wavefronts: 2 x WC
  constexpr int NLD = TM * KB / TH;          // loads per thread and operand
  constexpr int MT = TM / 32, MC = TM / WC / 16;  // 16x16 products per wavefront: rows, columns
  __shared__ union {
    struct {
      double a[TM][KP], b[TM][KP];
    } op;
    double s[NB][NBP];
  } sh;
  int64_t i, j;
  if (tri) {
    const int64_t b = blockIdx.x;
    i = (int64_t)((sqrt(8.0 * (double)b + 1.0) - 1.0) * 0.5);
    while ((i + 1) * (i + 2) / 2 <= b) ++i;
    while (i * (i + 1) / 2 > b) --i;
    j = b - i * (i + 1) / 2;
  } else {
    i = blockIdx.x;
    j = blockIdx.y;
    if (j > i) return;
  }
  const int64_t ri = r0 + TM * i, rj = r0 + TM * j;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int wr = (w / WC) * (TM / 2), wc = (w % WC) * (TM / WC);
  const int lr = lane & 15, lk = lane >> 4;
  v4d sum[MT][MC];
#pragma unroll
  for (int u = 0; u < MT; ++u)
#pragma unroll
    for (int v = 0; v < MC; ++v) sum[u][v] = v4d{0.0, 0.0, 0.0, 0.0};
  double pa[NLD], pb[NLD];
  auto load = [&](int64_t k) {
#pragma unroll
    for (int u = 0; u < NLD; ++u) {
      const int e = u * TH + t, r = e / KB, c = e % KB;
      // rows past n clamped: their products are not stored
      pa[u] = A[(ri + r < n ? ri + r : n - 1) * lda + k + c];
      pb[u] = A[(rj + r < n ? rj + r : n - 1) * lda + k + c];
    }
  };
  load(kc);
  for (int k0 = 0; k0 < K; k0 += NB) {
    v4d acc[MT][MC];
#pragma unroll
    for (int u = 0; u < MT; ++u)
#pragma unroll
      for (int v = 0; v < MC; ++v) acc[u][v] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
    for (int k = k0; k < k0 + NB; k += KB) {
      __syncthreads();  // the previous chunk is consumed
#pragma unroll
      for (int u = 0; u < NLD; ++u) {
        const int e = u * TH + t, r = e / KB, c = e % KB;
        sh.op.a[r][c] = pa[u];
        sh.op.b[r][c] = pb[u];
      }
      __syncthreads();
      load(kc + (k + KB < K ? k + KB : k));  // unconditional: a branch here moves the sums between register files
#pragma unroll
      for (int kk = 0; kk < KB; kk += 4) {
        double fa[MT], fb[MC];
#pragma unroll
        for (int u = 0; u < MT; ++u) fa[u] = sh.op.a[wr + 16 * u + lr][kk + lk];
#pragma unroll
        for (int v = 0; v < MC; ++v) fb[v] = sh.op.b[wc + 16 * v + lr][kk + lk];
#pragma unroll
        for (int u = 0; u < MT; ++u)
#pragma unroll
          for (int v = 0; v < MC; ++v)
            acc[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[u], fb[v], acc[u][v], 0, 0, 0);
      }
    }
#pragma unroll
    for (int u = 0; u < MT; ++u)
#pragma unroll
      for (int v = 0; v < MC; ++v) sum[u][v] += acc[u][v];
  }
  const bool first = i == 0 && j == 0;
  if (first) {
    __syncthreads();  // operands consumed: their space takes the diagonal tile
    for (int e = t; e < NB * NB; e += TH) {
      const int r = e / NB, c = e % NB;
      sh.s[r][c] = r == c ? 1.0 : 0.0;
    }
    __syncthreads();
  }
  // a row of products at a time: its loads together (clamped into the row),
  // then its stores
#pragma unroll
  for (int u = 0; u < MT; ++u) {
    double x[MC][4];
#pragma unroll
    for (int v = 0; v < MC; ++v)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        int64_t r = ri + wr + 16 * u + 4 * e + lk;
        r = r < n ? r : n - 1;
        const int64_t c = rj + wc + 16 * v + lr;
        x[v][e] = A[r * lda + (c <= r ? c : r)];
      }
#pragma unroll
    for (int v = 0; v < MC; ++v)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int tr = wr + 16 * u + 4 * e + lk, tc = wc + 16 * v + lr;
        const int64_t r = ri + tr, c = rj + tc;
        if (r < n && c <= r && c < c_end) {
          const double y = x[v][e] - sum[u][v][e];
          if (first && tr < NB && tc < NB)
            sh.s[tr][tc] = y;
          else
            A[r * lda + c] = y;
        }
      }
  }
  if (first) {
    __syncthreads();
    chol_tile(sh.s, n, r0, info);
    __syncthreads();
    store_diag(sh.s, A, n, lda, r0);
  }
}

// ---------------------------------------------------------------------------
// Triangular solves, in place and without scratch: one launch per block of
// TB unknowns.  Launch k subtracts the solved block k from every remaining
// block (one workgroup each), and the workgroup of the next block then
// solves it, so a launch needs only what earlier launches finished.  Bound
// by the chain of n / TB launches, 15 us each.  The TB x TB diagonal block
// waits in LDS meanwhile; one wavefront solves it with two rows per lane, the
// solved unknown passed by readlane.
// ---------------------------------------------------------------------------
constexpr int TB = 128;
constexpr int TBH = TB / 2;

struct TrsvTile {
  double d00[TBH][TBH + 1], d10[TBH][TBH + 1], d11[TBH][TBH + 1];
  double part[4][TB];
};

__device__ __forceinline__ void load_tri(TrsvTile &s, const double *L, int64_t n, int64_t lda, int64_t r0) {
  // all loads in flight together; rows past n and columns past the diagonal
  // are clamped and replaced
  const bool two = r0 + TBH < n;  // a second half
  double v[3][16];
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int r = u * 4 + (int)(threadIdx.x >> 6), c = threadIdx.x & 63;
    const int64_t a = r0 + r < n ? r0 + r : n - 1;
    v[0][u] = L[a * lda + (r0 + c <= a ? r0 + c : a)];
  }
  if (two) {
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int r = u * 4 + (int)(threadIdx.x >> 6), c = threadIdx.x & 63;
      const int64_t b = r0 + TBH + r < n ? r0 + TBH + r : n - 1;
      v[1][u] = L[b * lda + (r0 + c <= b ? r0 + c : b)];
      v[2][u] = L[b * lda + (r0 + TBH + c <= b ? r0 + TBH + c : b)];
    }
  }
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int r = u * 4 + (int)(threadIdx.x >> 6), c = threadIdx.x & 63;
    s.d00[r][c] = r0 + r < n && c <= r ? v[0][u] : (r == c ? 1.0 : 0.0);
  }
  if (two) {
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int r = u * 4 + (int)(threadIdx.x >> 6), c = threadIdx.x & 63;
      const bool b = r0 + TBH + r < n;
      s.d10[r][c] = b ? v[1][u] : 0.0;
      s.d11[r][c] = b && c <= r ? v[2][u] : (r == c ? 1.0 : 0.0);
    }
  }
}

// The solves of one block's unknowns by one wavefront, rows lane and 64 +
// lane, the solved unknown passed by readlane: na unknowns of the first half
// and, with TWO, 64 of the second.  A last block of 64 rows or fewer takes na
// steps and no second half.
template <bool TWO, class N>
__device__ __forceinline__ void solve_lower(const TrsvTile &s, int lane, N na, double &ta, double &tb) {
  const double ia = 1.0 / s.d00[lane][lane];
#pragma unroll 8
  for (int j = 0; j < na; ++j) {
    const double y = lane_value(ta * ia, j);
    ta = lane > j ? ta - s.d00[lane][j] * y : ta;  // not the zeros above the diagonal: y may be infinite
    if (TWO) tb -= s.d10[lane][j] * y;
  }
  ta *= ia;
  if (TWO) {
    const double ib = 1.0 / s.d11[lane][lane];
#pragma unroll 8
    for (int j = 0; j < TBH; ++j) {
      const double y = lane_value(tb * ib, j);
      tb = lane > j ? tb - s.d11[lane][j] * y : tb;
    }
    tb *= ib;
  }
}
template <bool TWO, class N>
__device__ __forceinline__ void solve_upper(const TrsvTile &s, int lane, N na, double &ta, double &tb) {
  if (TWO) {
    const double ib = 1.0 / s.d11[lane][lane];
#pragma unroll 8
    for (int j = TBH - 1; j >= 0; --j) {
      const double x = lane_value(tb * ib, j);
      tb = lane < j ? tb - s.d11[j][lane] * x : tb;
      ta -= s.d10[j][lane] * x;
    }
    tb *= ib;
  }
  const double ia = 1.0 / s.d00[lane][lane];
#pragma unroll 8
  for (int j = na - 1; j >= 0; --j) {
    const double x = lane_value(ta * ia, j);
    ta = lane < j ? ta - s.d00[j][lane] * x : ta;
  }
  ta *= ia;
}

// Systems of up to 64 unknowns: one launch for both directions, four
// right-hand sides to a workgroup, a wavefront each.  (In the blocked form
// each right-hand side is a workgroup that fills 100 KiB of LDS, one to a CU:
// 3 and 30 unknowns with 8,192 right-hand sides 127 and 248 us, 9 and 20 like
// this; with one 12 and 10, and 8.)
constexpr int TS_RHS = 4;

__global__ __launch_bounds__(64 * TS_RHS) void k_trsv_small(const double *__restrict__ L, int n, int64_t lda, double *B,
                                                            int64_t nrhs) {
  __shared__ double d[TBH][TBH + 1];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  double v[TBH / TS_RHS];
#pragma unroll
  for (int u = 0; u < TBH / TS_RHS; ++u) {
    const int r = u * TS_RHS + w < n ? u * TS_RHS + w : n - 1;
    v[u] = L[r * lda + (lane <= r ? lane : r)];
  }
#pragma unroll
  for (int u = 0; u < TBH / TS_RHS; ++u) {
    const int r = u * TS_RHS + w;
    d[r][lane] = r < n && lane <= r ? v[u] : (r == lane ? 1.0 : 0.0);
  }
  __syncthreads();
  const int64_t rhs = (int64_t)blockIdx.x * TS_RHS + w;
  if (rhs >= nrhs) return;
  const double inv = 1.0 / d[lane][lane];
  double t = lane < n ? B[lane * nrhs + rhs] : 0.0;
#pragma unroll 8
  for (int j = 0; j < n; ++j) {
    const double y = lane_value(t * inv, j);
    t = lane > j ? t - d[lane][j] * y : t;
  }
  t *= inv;
#pragma unroll 8
  for (int j = n - 1; j >= 0; --j) {
    const double x = lane_value(t * inv, j);
    t = lane < j ? t - d[j][lane] * x : t;
  }
  if (lane < n) B[lane * nrhs + rhs] = t * inv;
}

// forward: block kb is solved (kb < 0: none yet); workgroup x updates block
// kb + 1 + x, and the first one solves its block
__global__ __launch_bounds__(256) void k_trsv_lower(const double *__restrict__ L, int64_t n, int64_t lda, double *B,
                                                    int64_t nrhs, int64_t kb) {
  __shared__ TrsvTile s;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int64_t rhs = blockIdx.y;
  const int64_t r0 = TB * (kb + 1 + (int64_t)blockIdx.x);
  const bool solve = blockIdx.x == 0;
  if (solve) load_tri(s, L, n, lda, r0);
  if (kb >= 0) {
    const int64_t c0 = TB * kb;  // a full block: kb is not the last
    const double y0 = B[(c0 + lane) * nrhs + rhs], y1 = B[(c0 + TBH + lane) * nrhs + rhs];
    // wavefront w: 32 rows, lane = column
    double v[32];
#pragma unroll
    for (int u = 0; u < 32; ++u) {
      const int64_t r = r0 + 32 * w + u;
      const double *p = L + (r < n ? r : n - 1) * lda + c0;
      v[u] = p[lane] * y0 + p[TBH + lane] * y1;
    }
    // sums over the lanes: each halving leaves half the rows to each half
#pragma unroll
    for (int h = 32; h > 1; h >>= 1)
#pragma unroll
      for (int u = 0; u < h / 2; ++u) {
        const bool up = (lane & (h / 2)) != 0;
        const double keep = up ? v[u + h / 2] : v[u], give = up ? v[u] : v[u + h / 2];
        v[u] = keep + __shfl_xor(give, h / 2, 64);
      }
    const double sum = v[0] + __shfl_xor(v[0], 32, 64);  // row = the lane's low five bits
    if (lane < 32) s.part[0][32 * w + lane] = sum;
  }
  __syncthreads();
  if (!solve) {
    const int64_t r = r0 + t;
    if (t < TB && r < n) B[r * nrhs + rhs] -= s.part[0][t];
    return;
  }
  if (w != 0) return;
  const int64_t ra = r0 + lane, rb = r0 + TBH + lane;
  double ta = ra < n ? B[ra * nrhs + rhs] : 0.0, tb = rb < n ? B[rb * nrhs + rhs] : 0.0;
  if (kb >= 0) {
    ta -= s.part[0][lane];
    tb -= s.part[0][TBH + lane];
  }
  if (r0 + TBH < n)
    solve_lower<true>(s, lane, std::integral_constant<int, TBH>{}, ta, tb);
  else
    solve_lower<false>(s, lane, (int)(n - r0), ta, tb);
  if (ra < n) B[ra * nrhs + rhs] = ta;
  if (rb < n) B[rb * nrhs + rhs] = tb;
}

// backward, L^T x = y: block kb is solved (kb = number of blocks: none yet);
// workgroup x updates block kb - 1 - x, and the first one solves its block
__global__ __launch_bounds__(256) void k_trsv_upper(const double *__restrict__ L, int64_t n, int64_t lda, double *B,
                                                    int64_t nrhs, int64_t kb) {
  __shared__ TrsvTile s;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int64_t rhs = blockIdx.y;
  const int64_t r0 = TB * (kb - 1 - (int64_t)blockIdx.x);
  const int64_t k0 = TB * kb;
  const bool solve = blockIdx.x == 0;
  const bool any = k0 < n;
  if (solve) load_tri(s, L, n, lda, r0);
  if (any) {
    // wavefront w: 32 rows of the solved block, lane = two columns of ours
    double a0 = 0.0, a1 = 0.0;
#pragma unroll
    for (int u = 0; u < 32; ++u) {
      const int64_t r = k0 + 32 * w + u;
      const bool in = r < n;
      const double x = in ? B[r * nrhs + rhs] : 0.0;
      const double *p = L + (in ? r : n - 1) * lda + r0;
      a0 += p[lane] * x;
      a1 += p[TBH + lane] * x;
    }
    s.part[w][lane] = a0;
    s.part[w][TBH + lane] = a1;
  }
  __syncthreads();
  auto part = [&](int k) { return any ? (s.part[0][k] + s.part[1][k]) + (s.part[2][k] + s.part[3][k]) : 0.0; };
  if (!solve) {
    if (t < TB) B[(r0 + t) * nrhs + rhs] -= part(t);  // not the last block: full
    return;
  }
  if (w != 0) return;
  const int64_t ra = r0 + lane, rb = r0 + TBH + lane;
  double ta = ra < n ? B[ra * nrhs + rhs] - part(lane) : 0.0;
  double tb = rb < n ? B[rb * nrhs + rhs] - part(TBH + lane) : 0.0;
  if (r0 + TBH < n)
    solve_upper<true>(s, lane, std::integral_constant<int, TBH>{}, ta, tb);
  else
    solve_upper<false>(s, lane, (int)(n - r0), ta, tb);
  if (ra < n) B[ra * nrhs + rhs] = ta;
  if (rb < n) B[rb * nrhs + rhs] = tb;
}

}  // namespace eipc

using namespace eipc;

extern "C" {

eipc_status eipc_cholesky(eipc_ctx *c, double *A, int64_t n, int64_t lda, int64_t *info, eipc_stream stream) {
  if (!c || n < 0 || lda < n || (n > 0 && !A) || !info) return c ? set_err(c, EIPC_ERR_ARG, "bad Cholesky arguments")
                                                                  : EIPC_ERR_ARG;
  EIPC_HIP(c, hipSetDevice(c->device));
  hipStream_t s = (hipStream_t)stream;
  int64_t *d_info = c->counters + 12;
  EIPC_TRY(launch_zero(c, d_info, 8, s));
  if (n > 0) {
    k_chol_diag<<<1, 256, 0, s>>>(A, n, lda, 0, d_info);
    EIPC_HIP(c, hipGetLastError());
  }
  for (int64_t k0 = 0; k0 + NB < n; k0 += NB) {
    const int64_t r0 = k0 + NB, o0 = k0 / OB * OB, oend = std::min<int64_t>(o0 + OB, n);
    const int64_t rem = (n - r0 + NB - 1) / NB;
    k_chol_panel<<<(unsigned)rem, 256, 0, s>>>(A, n, lda, k0);
    EIPC_HIP(c, hipGetLastError());
    if (r0 < oend) {
      // inside the outer block: its remaining columns, with these 64
      const unsigned nc = (unsigned)((oend - r0 + NB - 1) / NB);
      k_chol_update<64><<<dim3((unsigned)rem, nc), 256, 0, s>>>(A, n, lda, k0, NB, r0, oend, 0, d_info);
    } else {
      // the outer block is finished: the whole trailing matrix; 64-tiles
      // while 128-tiles would be fewer than two per CU
      const int64_t nt = (n - r0 + 127) / 128, nblk = nt * (nt + 1) / 2;
      if (nblk >= 2 * (int64_t)c->num_cu)
        k_chol_update<128><<<(unsigned)nblk, upd_threads(128), 0, s>>>(A, n, lda, o0, OB, r0, n, 1, d_info);
      else
        k_chol_update<64><<<(unsigned)(rem * (rem + 1) / 2), 256, 0, s>>>(A, n, lda, o0, OB, r0, n, 1, d_info);
    }
    EIPC_HIP(c, hipGetLastError());
  }
  EIPC_HIP(c, hipMemcpyAsync(info, d_info, 8, hipMemcpyDeviceToHost, s));
  EIPC_HIP(c, hipStreamSynchronize(s));
  return EIPC_OK;
}

eipc_status eipc_cholesky_solve(eipc_ctx *c, const double *L, int64_t n, int64_t lda, double *B, int64_t nrhs,
                                eipc_stream stream) {
  if (!c || n < 0 || lda < n || nrhs < 1 || (n > 0 && (!L || !B)))
    return c ? set_err(c, EIPC_ERR_ARG, "bad solve arguments") : EIPC_ERR_ARG;
  EIPC_HIP(c, hipSetDevice(c->device));
  hipStream_t s = (hipStream_t)stream;
  if (n > 0 && n <= TBH) {
    k_trsv_small<<<(unsigned)((nrhs + TS_RHS - 1) / TS_RHS), 64 * TS_RHS, 0, s>>>(L, (int)n, lda, B, nrhs);
    EIPC_HIP(c, hipGetLastError());
    return EIPC_OK;
  }
  const int64_t nt = (n + TB - 1) / TB;
  // right-hand sides go to the grid's second axis, in runs it can hold
  for (int64_t j0 = 0; j0 < nrhs; j0 += 65535) {
    const unsigned nj = (unsigned)std::min<int64_t>(nrhs - j0, 65535);
    for (int64_t k = -1; k < nt - 1; ++k) {
      k_trsv_lower<<<dim3(k < 0 ? 1u : (unsigned)(nt - 1 - k), nj), 256, 0, s>>>(L, n, lda, B + j0, nrhs, k);
      EIPC_HIP(c, hipGetLastError());
    }
    for (int64_t k = nt; k > 0; --k) {
      k_trsv_upper<<<dim3(k == nt ? 1u : (unsigned)k, nj), 256, 0, s>>>(L, n, lda, B + j0, nrhs, k);
      EIPC_HIP(c, hipGetLastError());
    }
  }
  return EIPC_OK;
}

}  // extern "C"
