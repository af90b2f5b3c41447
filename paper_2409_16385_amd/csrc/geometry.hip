// Embedding, scans, the spatial-hash broad phase and the narrow phase.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "common.h"
#include "pair_math.h"

namespace eipc {

// ---------------------------------------------------------------------------
// embedding x = W q + off (Eq. 14): CSR order from 0.0, one rounded multiply
// and one rounded add per term, off added last.  Output SoA (and AoS).
// ---------------------------------------------------------------------------
__global__ void k_embed(int n, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ col,
                        const double *__restrict__ val, const double *__restrict__ q,
                        const double *__restrict__ off, double *__restrict__ xs, double *__restrict__ x_aos,
                        const int32_t *__restrict__ vscene, int n_scene, uint32_t *status) {
#pragma clang fp contract(off)
  const int v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= n) return;
  double a0 = 0.0, a1 = 0.0, a2 = 0.0;
  const int k0 = rowptr[v], k1 = rowptr[v + 1];
  if (k1 - k0 > 4 || k1 < k0) atomicOr(status, ST_BAD_W);
  if (vscene && (unsigned)vscene[v] >= (unsigned)n_scene) atomicOr(status, ST_BAD_SCENE);
  for (int k = k0; k < k1; ++k) {
    const double w = val[k];
    const int64_t c = 3 * (int64_t)col[k];
    a0 = a0 + w * q[c];
    a1 = a1 + w * q[c + 1];
    a2 = a2 + w * q[c + 2];
  }
  if (off) {
    a0 = a0 + off[3 * (int64_t)v];
    a1 = a1 + off[3 * (int64_t)v + 1];
    a2 = a2 + off[3 * (int64_t)v + 2];
  }
  if (xs) {
    double2 *r = reinterpret_cast<double2 *>(xs + (int64_t)PSTRIDE * v);
    r[0] = double2{a0, a1};
    r[1] = double2{a2, 0.0};
  }
  if (x_aos) {
    x_aos[3 * (int64_t)v] = a0;
    x_aos[3 * (int64_t)v + 1] = a1;
    x_aos[3 * (int64_t)v + 2] = a2;
  }
  if (!(isfinite(a0) && isfinite(a1) && isfinite(a2))) atomicOr(status, ST_NONFINITE);
}

eipc_status launch_embed(eipc_ctx *c, const eipc_scene *sc, const double *q, const double *off, double *xs,
                         double *x_aos, hipStream_t s) {
  if (sc->n_vert == 0) return EIPC_OK;
  ProfScope ps(c, K_EMBED, s);
  k_embed<<<grid_for(sc->n_vert, 256), 256, 0, s>>>(sc->n_vert, sc->W_rowptr, sc->W_col, sc->W_val, q, off, xs,
                                                     x_aos, vscene_of(sc), n_scene_of(sc), c->status);
  EIPC_HIP(c, hipGetLastError());
  return EIPC_OK;
}

// x = W q + off, p = W dq + dx_off and the end positions x1 = x + p (one
// rounded add) in one pass over the rows of W (three launches and two reads
// of W otherwise); the sums are k_embed's.
__global__ void k_embed_swept(int n, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ col,
                              const double *__restrict__ val, const double *__restrict__ q,
                              const double *__restrict__ off, const double *__restrict__ dq,
                              const double *__restrict__ dx_off, double *__restrict__ xs, double *__restrict__ ps,
                              double *__restrict__ x1s, const int32_t *__restrict__ vscene, int n_scene,
                              uint32_t *status) {
#pragma clang fp contract(off)
  const int v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= n) return;
  double a[3] = {0.0, 0.0, 0.0}, b[3] = {0.0, 0.0, 0.0};
  const int k0 = rowptr[v], k1 = rowptr[v + 1];
  if (k1 - k0 > 4 || k1 < k0) atomicOr(status, ST_BAD_W);
  if (vscene && (unsigned)vscene[v] >= (unsigned)n_scene) atomicOr(status, ST_BAD_SCENE);
  for (int k = k0; k < k1; ++k) {
    const double w = val[k];
    const int64_t c = 3 * (int64_t)col[k];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      a[i] = a[i] + w * q[c + i];
      b[i] = b[i] + w * dq[c + i];
    }
  }
  bool fin = true;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    if (off) a[i] = a[i] + off[3 * (int64_t)v + i];
    if (dx_off) b[i] = b[i] + dx_off[3 * (int64_t)v + i];
    fin = fin && isfinite(a[i]) && isfinite(b[i]);
  }
  double2 *r = reinterpret_cast<double2 *>(xs + (int64_t)PSTRIDE * v);
  r[0] = double2{a[0], a[1]};
  r[1] = double2{a[2], 0.0};
  r = reinterpret_cast<double2 *>(ps + (int64_t)PSTRIDE * v);
  r[0] = double2{b[0], b[1]};
  r[1] = double2{b[2], 0.0};
  if (x1s) {
    r = reinterpret_cast<double2 *>(x1s + (int64_t)PSTRIDE * v);
    r[0] = double2{a[0] + b[0], a[1] + b[1]};
    r[1] = double2{a[2] + b[2], 0.0};
  }
  if (!fin) atomicOr(status, ST_NONFINITE);
}

eipc_status launch_embed_swept(eipc_ctx *c, const eipc_scene *sc, const double *q, const double *dq,
                               const double *dx_off, double *xs, double *ps, double *x1s, hipStream_t s) {
  if (sc->n_vert == 0) return EIPC_OK;
  ProfScope prof(c, K_EMBED, s);
  k_embed_swept<<<grid_for(sc->n_vert, 256), 256, 0, s>>>(sc->n_vert, sc->W_rowptr, sc->W_col, sc->W_val, q,
                                                           sc->x_off, dq, dx_off, xs, ps, x1s, vscene_of(sc),
                                                           n_scene_of(sc), c->status);
  EIPC_HIP(c, hipGetLastError());
  return EIPC_OK;
}

__global__ void k_zero(uint64_t *p, int64_t n64) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (; i < n64; i += (int64_t)gridDim.x * blockDim.x) p[i] = 0;
}
__global__ void k_zero_bytes(uint8_t *p, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

// Fill kernel (used instead of hipMemsetAsync so the sequence can be
// captured into a graph).
eipc_status launch_zero(eipc_ctx *c, void *p, size_t bytes, hipStream_t s) {
  if (bytes == 0) return EIPC_OK;
  int64_t n64 = (int64_t)(bytes / 8);
  if (((uintptr_t)p & 7) == 0 && n64 > 0) {
    int g = (int)std::min<int64_t>(grid_for(n64, 256), 4096);
    k_zero<<<g, 256, 0, s>>>((uint64_t *)p, n64);
    EIPC_HIP(c, hipGetLastError());
    size_t rem = bytes - (size_t)n64 * 8;
    if (rem) {
      k_zero_bytes<<<1, 64, 0, s>>>((uint8_t *)p + n64 * 8, (int64_t)rem);
      EIPC_HIP(c, hipGetLastError());
    }
  } else {
    k_zero_bytes<<<grid_for((int64_t)bytes, 256), 256, 0, s>>>((uint8_t *)p, (int64_t)bytes);
    EIPC_HIP(c, hipGetLastError());
  }
  return EIPC_OK;
}

// Every buffer that a call clears, in one launch: a launch of its own each
// costs about 4 us, which small scenes feel.
constexpr int FILL_WORDS = 2048;  // 8-byte words per workgroup and round
__global__ __launch_bounds__(256) void k_fill_list(FillList l) {
  int b = blockIdx.x, k = 0;
  while (k + 1 < l.n && b >= l.seg[k].blocks) b -= l.seg[k++].blocks;
  const FillSeg g = l.seg[k];
  for (int64_t base = (int64_t)b * FILL_WORDS; base < g.n; base += (int64_t)g.blocks * FILL_WORDS)
#pragma unroll
    for (int u = 0; u < FILL_WORDS / 256; ++u) {
      const int64_t i = base + u * 256 + threadIdx.x;
      if (i < g.n) g.p[i] = g.v;
    }
}

eipc_status launch_fill(eipc_ctx *c, FillList &l, hipStream_t s) {
  if (l.bad) return set_err(c, EIPC_ERR_ARG, "a buffer to clear is not whole words");
  if (l.n == 0) return EIPC_OK;
  int64_t blocks = 0;
  for (int k = 0; k < l.n; ++k) {
    l.seg[k].blocks = (int)std::min<int64_t>((l.seg[k].n + FILL_WORDS - 1) / FILL_WORDS, 2048);
    blocks += l.seg[k].blocks;
  }
  k_fill_list<<<(unsigned)blocks, 256, 0, s>>>(l);
  EIPC_HIP(c, hipGetLastError());
  l.n = 0;
  return EIPC_OK;
}

// ---------------------------------------------------------------------------
// exclusive scan: int32 counts[n] -> int64 offsets[n+1] (offsets[n] = total)
// tiles of 2048 elements (256 threads x 8), block sums scanned by one block
// ---------------------------------------------------------------------------
constexpr int SCAN_T = 256, SCAN_E = 8, SCAN_TILE = SCAN_T * SCAN_E;

__device__ __forceinline__ int64_t block_excl_scan(int64_t v, int64_t *smem, int64_t *total) {
  // inclusive wave scan
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  int64_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    int64_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) smem[wid] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t acc = 0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) {
      int64_t t = smem[w];
      smem[w] = acc;
      acc += t;
    }
    smem[16] = acc;
  }
  __syncthreads();
  int64_t r = x - v + smem[wid];
  *total = smem[16];
  __syncthreads();
  return r;
}

// Up to two scans side by side (grid y).  Arrays of up to SCAN_ONE entries:
// one launch, one workgroup each.  Larger ones: two launches over at most
// SCAN_BLOCKS ranges; the second sums the ranges before its own itself (at
// most four loads a thread), so no launch between them scans the sums.  One workgroup
// takes 5 us for one pass of 8,192 entries and 34 for four of them, the two
// launches 9.5 us for 32,768.
constexpr int64_t SCAN_ONE = 8192;
constexpr int SCAN_BLOCKS = 1024;
struct ScanArgs {
  const int32_t *in[2];
  int64_t n[2];
  int64_t *out[2];
  int64_t *bsum[2];
};

__global__ __launch_bounds__(1024) void k_scan_one(ScanArgs a) {
  __shared__ int64_t sm[17];
  const int32_t *in = a.in[blockIdx.y];
  const int64_t n = a.n[blockIdx.y];
  int64_t *out = a.out[blockIdx.y];
  int64_t carry = 0;
  for (int64_t b0 = 0; b0 < n; b0 += 1024 * SCAN_E) {
    const int64_t base = b0 + threadIdx.x * SCAN_E;
    int32_t v[SCAN_E];
    int64_t acc = 0, tot;
#pragma unroll
    for (int e = 0; e < SCAN_E; ++e) {
      v[e] = base + e < n ? in[base + e] : 0;
      acc += v[e];
    }
    int64_t ex = carry + block_excl_scan(acc, sm, &tot);
#pragma unroll
    for (int e = 0; e < SCAN_E; ++e) {
      if (base + e < n) out[base + e] = ex;
      ex += v[e];
    }
    carry += tot;
  }
  if (threadIdx.x == 0) out[n] = carry;
}

// tiles of a workgroup's range: consecutive, the same number for each
__device__ __forceinline__ int64_t scan_range(int64_t n, int64_t nb) {
  return ((n + SCAN_TILE - 1) / SCAN_TILE + nb - 1) / nb * SCAN_TILE;
}

__global__ __launch_bounds__(SCAN_T) void k_scan_partial(ScanArgs a) {
  __shared__ int64_t sm[17];
  const int32_t *in = a.in[blockIdx.y];
  const int64_t n = a.n[blockIdx.y], per = scan_range(n, gridDim.x);
  const int64_t r0 = blockIdx.x * per, r1 = r0 + per < n ? r0 + per : n;
  int64_t acc = 0;
  for (int64_t i = r0 + threadIdx.x; i < r1; i += SCAN_T) acc += in[i];
  int64_t tot;
  block_excl_scan(acc, sm, &tot);
  if (threadIdx.x == 0) a.bsum[blockIdx.y][blockIdx.x] = tot;
}

__global__ __launch_bounds__(SCAN_T) void k_scan_final(ScanArgs a) {
  __shared__ int64_t sm[17];
  const int32_t *in = a.in[blockIdx.y];
  int64_t *out = a.out[blockIdx.y];
  const int64_t *bsum = a.bsum[blockIdx.y];
  const int64_t n = a.n[blockIdx.y], per = scan_range(n, gridDim.x);
  const int64_t r0 = blockIdx.x * per, r1 = r0 + per < n ? r0 + per : n;
  int64_t before = 0, carry, tot;
  for (int64_t k = threadIdx.x; k < (int64_t)blockIdx.x; k += SCAN_T) before += bsum[k];
  block_excl_scan(before, sm, &carry);
  for (int64_t b0 = r0; b0 < r1; b0 += SCAN_TILE) {
    const int64_t base = b0 + threadIdx.x * SCAN_E;
    int32_t v[SCAN_E];
    int64_t acc = 0;
#pragma unroll
    for (int e = 0; e < SCAN_E; ++e) {
      v[e] = base + e < n ? in[base + e] : 0;
      acc += v[e];
    }
    int64_t ex = carry + block_excl_scan(acc, sm, &tot);
#pragma unroll
    for (int e = 0; e < SCAN_E; ++e) {
      if (base + e < n) out[base + e] = ex;
      ex += v[e];
    }
    carry += tot;
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) out[n] = carry;
}

eipc_status exclusive_scan2(eipc_ctx *c, const int32_t *in0, int64_t n0, int64_t *out0, const int32_t *in1,
                            int64_t n1, int64_t *out1, hipStream_t s) {
  const int ny = in1 ? 2 : 1;
  ScanArgs a{{in0, in1}, {n0, n1}, {out0, out1}, {nullptr, nullptr}};
  const int64_t n = std::max(n0, in1 ? n1 : 0);
  if (n <= SCAN_ONE) {
    k_scan_one<<<dim3(1, ny), 1024, 0, s>>>(a);
    EIPC_HIP(c, hipGetLastError());
    return EIPC_OK;
  }
  const int64_t nb = std::min<int64_t>((n + SCAN_TILE - 1) / SCAN_TILE, SCAN_BLOCKS);
  int64_t *bsum;
  EIPC_TRY(ensure_t(c, s == c->side ? B_SCANTMP_SIDE : B_SCANTMP, (size_t)(ny * nb), &bsum));
  a.bsum[0] = bsum;
  a.bsum[1] = bsum + nb;
  k_scan_partial<<<dim3((unsigned)nb, ny), SCAN_T, 0, s>>>(a);
  EIPC_HIP(c, hipGetLastError());
  k_scan_final<<<dim3((unsigned)nb, ny), SCAN_T, 0, s>>>(a);
  EIPC_HIP(c, hipGetLastError());
  return EIPC_OK;
}

eipc_status exclusive_scan(eipc_ctx *c, const int32_t *in, int64_t n, int64_t *out, hipStream_t s) {
  return exclusive_scan2(c, in, n, out, nullptr, 0, nullptr, s);
}

// ---------------------------------------------------------------------------
// Broad phase.  Boxes: per primitive, lo = min over its vertices (start and
// end positions when swept) - dhat/2, hi = max + dhat/2.  Items (faces for
// PT, edges for EE) are stored as 64-byte records; the uniform grid is a
// hash from (scene, cell) to the items whose boxes touch the cell.  Grid
// parameters are computed on the device, so the sequence can run without
// host synchronization once capacities are known.
// ---------------------------------------------------------------------------
struct ItemRec {
  double lo[3], hi[3];
  int32_t v[3];
  int32_t tag;  // bit 0: some vertex has a DoF; bits 1..: scene id
};

__device__ __forceinline__ bool has_dof(const int32_t *rowptr, int v) { return rowptr[v + 1] > rowptr[v]; }
__device__ __forceinline__ int scene_of(const int32_t *vscene, int v) { return vscene ? vscene[v] : 0; }

template <int NV>
__device__ __forceinline__ void prim_box(const int *vid, const double *xs, const double *x1s, int n_vert, double h,
                                         double *lo, double *hi) {
#pragma clang fp contract(off)
#pragma unroll
  for (int cax = 0; cax < 3; ++cax) {
    double mn = xs[(int64_t)PSTRIDE * vid[0] + cax], mx = mn;
#pragma unroll
    for (int a = 0; a < NV; ++a) {
      double v = xs[(int64_t)PSTRIDE * vid[a] + cax];
      mn = fmin(mn, v);
      mx = fmax(mx, v);
      if (x1s) {
        double w = x1s[(int64_t)PSTRIDE * vid[a] + cax];
        mn = fmin(mn, w);
        mx = fmax(mx, w);
      }
    }
    lo[cax] = mn - h;
    hi[cax] = mx + h;
  }
}

__device__ __forceinline__ uint64_t ord_key(double v) {
  uint64_t b = __double_as_longlong(v);
  return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}
__device__ __forceinline__ double ord_dec(uint64_t k) {
  uint64_t b = (k >> 63) ? (k & 0x7fffffffffffffffull) : ~k;
  return __longlong_as_double(b);
}

// Box records of the items (KIND 0: faces, 1: edges) and, for KIND 0, of the
// vertices (kept when vrec is given), with the statistics of the grid in the
// same pass: the first gi workgroups take the items, the others the
// vertices.  Statistics, STAT_COPIES copies of nine words, all starting from
// zero: [0..2] max of the complemented order key of lo (its min), [3..5] max
// of the key of hi, [6..8] sum of the item extents.  Workgroups end with nine
// atomics; their number is bounded and the copies keep the queue on a word
// to a few hundred (the statistics alone took 25 us of a config 2 chain when
// they read the records back in a launch of their own).
constexpr int STAT_T = 256, STAT_COPIES = 4, STAT_BLOCKS = 1024;
template <int KIND>
__global__ __launch_bounds__(STAT_T) void k_items(int n, const int32_t *__restrict__ idx, int n_vert,
                                                  const double *__restrict__ xs, const double *__restrict__ x1s,
                                                  double h, const int32_t *__restrict__ rowptr,
                                                  const int32_t *__restrict__ vscene, ItemRec *__restrict__ rec,
                                                  ItemRec *__restrict__ vrec, int gi, uint64_t *st) {
  constexpr int NV = KIND == 0 ? 3 : 2;
  __shared__ double s_red[STAT_T / 64][9];
  double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY}, ex[3] = {0, 0, 0};
  if ((int)blockIdx.x < gi) {
    for (int i = blockIdx.x * STAT_T + threadIdx.x; i < n; i += gi * STAT_T) {
      int vid[NV];
#pragma unroll
      for (int a = 0; a < NV; ++a) vid[a] = idx[(int64_t)NV * i + a];
      ItemRec r;
      prim_box<NV>(vid, xs, x1s, n_vert, h, r.lo, r.hi);
      int dof = 0;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        r.v[a] = a < NV ? vid[a < NV ? a : 0] : -1;
        if (a < NV) dof |= has_dof(rowptr, vid[a < NV ? a : 0]);
      }
      r.tag = dof | (scene_of(vscene, vid[0]) << 1);
      rec[i] = r;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        lo[a] = fmin(lo[a], r.lo[a]);
        hi[a] = fmax(hi[a], r.hi[a]);
        ex[a] += r.hi[a] - r.lo[a];
      }
    }
  } else {
    const int gv = gridDim.x - gi;
    for (int i = ((int)blockIdx.x - gi) * STAT_T + threadIdx.x; i < n_vert; i += gv * STAT_T) {
      ItemRec r;
      prim_box<1>(&i, xs, x1s, n_vert, h, r.lo, r.hi);
      if (vrec) {
        r.v[0] = i;
        r.v[1] = -1;
        r.v[2] = -1;
        r.tag = (int)has_dof(rowptr, i) | (scene_of(vscene, i) << 1);
        vrec[i] = r;
      }
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        lo[a] = fmin(lo[a], r.lo[a]);
        hi[a] = fmax(hi[a], r.hi[a]);
      }
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      lo[a] = fmin(lo[a], __shfl_xor(lo[a], o, 64));
      hi[a] = fmax(hi[a], __shfl_xor(hi[a], o, 64));
      ex[a] += __shfl_xor(ex[a], o, 64);
    }
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      s_red[w][a] = lo[a];
      s_red[w][3 + a] = hi[a];
      s_red[w][6 + a] = ex[a];
    }
  }
  __syncthreads();
  if (threadIdx.x < 9) {
    // one lane per statistic
    const int t = threadIdx.x;
    double v = s_red[0][t];
    for (int k = 1; k < STAT_T / 64; ++k) v = t < 3 ? fmin(v, s_red[k][t]) : (t < 6 ? fmax(v, s_red[k][t]) : v + s_red[k][t]);
    uint64_t *p = st + 9 * (blockIdx.x % STAT_COPIES) + t;
    if (t < 3)
      atomicMax((unsigned long long *)p, (unsigned long long)~ord_key(v));
    else if (t < 6)
      atomicMax((unsigned long long *)p, (unsigned long long)ord_key(v));
    else if (v != 0.0)
      atomicAdd((double *)p, v);
  }
}

struct GridDev {
  double o[3];
  double inv_h;
  int dim[3];
  int bad;  // non-finite boxes
};

constexpr int MAX_ITEM_CELLS = 64;
constexpr int BIG_CELLS = 4096;
constexpr int GRID_AXIS_MAX = 1 << 16;

// cell edge: cell_scale times the mean item box extent (largest axis of the
// mean), at least 1e-6 of the scene span, grown until every axis has at
// most 2^16 cells
// (from the statistics, by every workgroup that needs them first: nine lanes
// fold the copies, one forms the grid)
__device__ __forceinline__ void grid_params(const uint64_t *st, int n_items, double cell_scale, GridDev *g,
                                            double *s_stat) {
  if (threadIdx.x < 9) {
    const int t = threadIdx.x;
    uint64_t w[STAT_COPIES];
#pragma unroll
    for (int k = 0; k < STAT_COPIES; ++k) w[k] = st[9 * k + t];
    if (t < 6) {
      uint64_t m = w[0];
#pragma unroll
      for (int k = 1; k < STAT_COPIES; ++k) m = m > w[k] ? m : w[k];
      s_stat[t] = ord_dec(t < 3 ? ~m : m);
    } else {
      double e = 0.0;
#pragma unroll
      for (int k = 0; k < STAT_COPIES; ++k) e += __longlong_as_double(w[k]);
      s_stat[t] = e;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double lo[3], hi[3], ext[3];
    bool ok = true;
    for (int a = 0; a < 3; ++a) {
      lo[a] = s_stat[a];
      hi[a] = s_stat[3 + a];
      ext[a] = s_stat[6 + a];
      ok = ok && isfinite(lo[a]) && isfinite(hi[a]);
    }
    GridDev r;
    r.bad = ok ? 0 : 1;
    if (!ok)
      for (int a = 0; a < 3; ++a) {
        lo[a] = 0.0;
        hi[a] = 0.0;
      }
    double cell = cell_scale * fmax(ext[0], fmax(ext[1], ext[2])) / (double)(n_items > 0 ? n_items : 1);
    double span = fmax(hi[0] - lo[0], fmax(hi[1] - lo[1], hi[2] - lo[2]));
    cell = fmax(cell, span * 1e-6);
    if (!(cell > 0.0) || !isfinite(cell)) cell = 1.0;
    for (int it = 0; it < 64; ++it) {
      bool fits = true;
      for (int a = 0; a < 3; ++a)
        if (floor((hi[a] - lo[a]) / cell) + 1.0 > (double)GRID_AXIS_MAX) fits = false;
      if (fits) break;
      cell *= 2.0;
    }
    for (int a = 0; a < 3; ++a) {
      r.o[a] = lo[a];
      double d = floor((hi[a] - lo[a]) / cell) + 1.0;
      r.dim[a] = (int)fmin(d, (double)GRID_AXIS_MAX);
    }
    r.inv_h = 1.0 / cell;
    *g = r;
  }
  __syncthreads();
}

__device__ __forceinline__ int cell_of(double v, double o, double inv_h, int dim) {
#pragma clang fp contract(off)
  double t = floor((v - o) * inv_h);
  int c = t < 0.0 ? 0 : (t > (double)(dim - 1) ? dim - 1 : (int)t);
  return c;
}
__device__ __forceinline__ uint64_t cell_key(int x, int y, int z, int scene) {
  return (uint64_t)x | ((uint64_t)y << 16) | ((uint64_t)z << 32) | ((uint64_t)scene << 48);
}
__device__ __forceinline__ uint32_t cell_hash(int x, int y, int z, int scene) {
  return ((uint32_t)x * 73856093u) ^ ((uint32_t)y * 19349663u) ^ ((uint32_t)z * 83492791u) ^
         ((uint32_t)scene * 2654435761u);
}
__device__ __forceinline__ void cell_range(const GridDev &g, const double *lo, const double *hi, int *c0, int *c1) {
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    c0[a] = cell_of(lo[a], g.o[a], g.inv_h, g.dim[a]);
    c1[a] = cell_of(hi[a], g.o[a], g.inv_h, g.dim[a]);
  }
}

// the cells of a big item, one lane per cell
__device__ __forceinline__ void big_cell(const int *c0, const int *c1, int c, int &x, int &y, int &z) {
  const int sx = c1[0] - c0[0] + 1, sy = c1[1] - c0[1] + 1;
  x = c0[0] + c % sx;
  y = c0[1] + (c / sx) % sy;
  z = c0[2] + c / (sx * sy);
}

// Workgroup-local bucket table: the items of a workgroup are neighbours
// in mesh order, so their (item, cell) entries fall into few buckets.  Each
// distinct bucket takes one LDS slot (linear probing on the bucket id), the
// entries are counted there, and one global atomic per slot carries the
// count (histogram) or reserves the bucket's range (fill).  An entry whose
// probe finds neither its bucket nor a free slot within LT_PROBE steps goes
// to the global counters directly; its bucket then never enters the table.

// parts, at most, of a large box in a short list: its cells in turn
constexpr int LQ_PARTS = 32;

// Threads to an item (Q), which take its cells in turn, and items to a
// workgroup.  Short lists leave the chip idle with one thread to an item,
// its cells one chain of table lookups: with four, the fill of the sphere 54
// and 20 us, of a sheet 76 and 29 (both launches), of the grasp (825
// workgroups of 256 items) 157 and 104, its candidates 733 and 632 us as a
// whole.  Where the chip is full they only add divisions: the batch (above
// 4,000 workgroups) 271 and 409 us.  The line, 1,024 workgroups, lies well
// below that: single grasps gain little from there on (candidates with one
// thread and with four: 725 workgroups 485 and 447 us, 1,084 791 and 720,
// 2,115 1,889 and 1,782, 4,822 8,880 and 8,743), the batch loses much.
constexpr int lt_items(int q) { return q == 1 ? 256 : 128; }
constexpr int lt_threads(int q) { return q * lt_items(q); }
constexpr int LT_FEW = 4;       // four threads to an item below this many workgroups of 256 items per CU

// the cells of [c0, c1] that thread sub of Q takes
template <int Q, class F>
__device__ __forceinline__ void each_cell(const int *c0, const int *c1, int nc, int sub, F &&f) {
  if constexpr (Q == 1) {
    for (int z = c0[2]; z <= c1[2]; ++z)
      for (int y = c0[1]; y <= c1[1]; ++y)
        for (int x = c0[0]; x <= c1[0]; ++x) f(x, y, z);
  } else {
    for (int c = sub; c < nc; c += Q) {
      int x, y, z;
      big_cell(c0, c1, c, x, y, z);
      f(x, y, z);
    }
  }
}

constexpr int LT_SLOTS = 2048;  // LDS table slots
constexpr int LT_PROBE = 32;

__device__ __forceinline__ int lt_insert(uint32_t *key, uint32_t b) {
  uint32_t h = (b * 2654435761u) >> 21;  // 11 bits
  for (int p = 0; p < LT_PROBE; ++p) {
    const uint32_t old = atomicCAS(&key[h], 0u, b + 1u);
    if (old == 0u || old == b + 1u) return (int)h;
    h = (h + 1) & (LT_SLOTS - 1);
  }
  return -1;
}
__device__ __forceinline__ int lt_find(const uint32_t *key, uint32_t b) {
  uint32_t h = (b * 2654435761u) >> 21;
  for (int p = 0; p < LT_PROBE; ++p) {
    const uint32_t k = key[h];
    if (k == b + 1u) return (int)h;
    if (k == 0u) return -1;
    h = (h + 1) & (LT_SLOTS - 1);
  }
  return -1;
}

// One side of a hash: the items, or the query vertices over the same grid.
struct HSide {
  int n;
  const ItemRec *rec;
  int32_t *cnt;      // cells per record, 0: not hashed one thread per record
  int32_t *large;    // records tested against everything
  int64_t *n_large;
  int32_t *big;      // records hashed one wavefront each
  int64_t *n_big;    // {records, cells}
  int32_t *bcnt;     // entries per bucket; counted down again by the fill
  int64_t *bstart;
  struct Entry *ent;
  int64_t ent_cap;
};
struct HSides {
  HSide s[2];
  int blocks0;  // workgroups of the first side (the rest: the second)
};

// Items covering up to MAX_ITEM_CELLS cells are hashed one thread per
// item; larger ones with at most 64 cells per axis (the reach of the 6-bit
// offsets of an entry) and at most BIG_CELLS cells are hashed one wavefront
// per item (the big list, n_big = {items, cells}); the rest (the large
// list) are tested against every query instead.
// A first launch counts the cells and lists big and large records (count)
// and counts the entries per bucket (hist): one pass, or two where the
// number of buckets has to follow the number of entries.
template <int Q>
__global__ __launch_bounds__(lt_threads(Q)) void k_cells(HSides hs, const uint64_t *st, int n_items, double cell_scale,
                                                GridDev *gp, uint32_t bmask, bool count, bool hist, int64_t *n_ent,
                                                uint32_t *status) {
  __shared__ uint32_t s_key[LT_SLOTS];
  __shared__ int32_t s_cnt[LT_SLOTS];
  __shared__ GridDev s_g;
  __shared__ double s_stat[9];
  __shared__ int s_big[lt_items(Q)];
  __shared__ int s_nbig, s_ent;
  const bool second = (int)blockIdx.x >= hs.blocks0;
  const HSide &h = hs.s[second ? 1 : 0];
  if (hist)
    for (int k = threadIdx.x; k < LT_SLOTS; k += lt_threads(Q)) {
      s_key[k] = 0u;
      s_cnt[k] = 0;
    }
  if (threadIdx.x == 0) {
    s_nbig = 0;
    s_ent = 0;
  }
  if (count) {
    grid_params(st, n_items, cell_scale, &s_g, s_stat);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      *gp = s_g;
      if (s_g.bad) atomicOr(status, ST_NONFINITE);
    }
  } else if (threadIdx.x == 0) {
    s_g = *gp;
  }
  __syncthreads();
  const GridDev g = s_g;
  const int i = (blockIdx.x - (second ? hs.blocks0 : 0)) * lt_items(Q) + threadIdx.x / Q, sub = threadIdx.x % Q;
  if (i < h.n) {
    int c0[3], c1[3];
    cell_range(g, h.rec[i].lo, h.rec[i].hi, c0, c1);
    const int sx = c1[0] - c0[0] + 1, sy = c1[1] - c0[1] + 1, sz = c1[2] - c0[2] + 1;
    const int64_t nc = (int64_t)sx * sy * sz;
    // non-finite boxes: nothing is hashed (the error is reported)
    const bool small = nc <= MAX_ITEM_CELLS && !g.bad;
    const bool big = !small && sx <= 64 && sy <= 64 && sz <= 64 && nc <= BIG_CELLS && !g.bad;
    if (count && sub == 0) {
      h.cnt[i] = small ? (int32_t)nc : 0;
      if (big) {
        const int slot = (int)atomicAdd((unsigned long long *)&h.n_big[0], 1ull);
        h.big[slot] = i;
        atomicAdd((unsigned long long *)&h.n_big[1], (unsigned long long)nc);
      } else if (!small && !g.bad) {
        h.large[(int)atomicAdd((unsigned long long *)h.n_large, 1ull)] = i;
      }
      if (n_ent && small) atomicAdd(&s_ent, (int)nc);
    }
    if (hist && big && sub == 0) s_big[atomicAdd(&s_nbig, 1)] = i;
    if (hist && small) {
      const int sc = h.rec[i].tag >> 1;
      each_cell<Q>(c0, c1, (int)nc, sub, [&](int x, int y, int z) {
        const uint32_t b = cell_hash(x, y, z, sc) & bmask;
        const int t = lt_insert(s_key, b);
        if (t >= 0)
          atomicAdd(&s_cnt[t], 1);
        else
          atomicAdd(&h.bcnt[b], 1);
      });
    }
  }
  __syncthreads();
  if (n_ent && threadIdx.x == 0 && s_ent)
    atomicAdd((unsigned long long *)&n_ent[second ? 1 : 0], (unsigned long long)s_ent);
  if (!hist) return;
  for (int k = threadIdx.x; k < LT_SLOTS; k += lt_threads(Q))
    if (s_key[k] != 0u) atomicAdd(&h.bcnt[s_key[k] - 1u], s_cnt[k]);
  // the workgroup's big records: a wavefront each, adds that return nothing
  const int lane = threadIdx.x & 63;
  for (int w = threadIdx.x >> 6; w < s_nbig; w += lt_threads(Q) / 64) {
    const int ib = s_big[w];
    const int sc = h.rec[ib].tag >> 1;
    int c0[3], c1[3];
    cell_range(g, h.rec[ib].lo, h.rec[ib].hi, c0, c1);
    const int nc = (c1[0] - c0[0] + 1) * (c1[1] - c0[1] + 1) * (c1[2] - c0[2] + 1);
    for (int c = lane; c < nc; c += 64) {
      int x, y, z;
      big_cell(c0, c1, c, x, y, z);
      atomicAdd(&h.bcnt[cell_hash(x, y, z, sc) & bmask], 1);
    }
  }
}

// Hash entry: one (item, cell) pair.  The offset of the cell from the
// item's lower cell decides the lower-corner rule without the item's record.
struct Entry {
  uint64_t cell;
  int32_t item;
  int32_t dlo;  // cell minus the item's lower cell, 6 bits per axis
};

// Places the entries: a bucket's count is taken down from its end, so the
// counters need no second array and end at zero.
template <int Q>
__global__ __launch_bounds__(lt_threads(Q)) void k_item_fill(HSides hs, const GridDev *__restrict__ gp, uint32_t bmask,
                                                    uint32_t *status) {
  __shared__ uint32_t s_key[LT_SLOTS];
  __shared__ int32_t s_cnt[LT_SLOTS];
  __shared__ int32_t s_base[LT_SLOTS];
  const bool second = (int)blockIdx.x >= hs.blocks0;
  const HSide &h = hs.s[second ? 1 : 0];
  for (int k = threadIdx.x; k < LT_SLOTS; k += lt_threads(Q)) {
    s_key[k] = 0u;
    s_cnt[k] = 0;
  }
  __syncthreads();
  const int i = (blockIdx.x - (second ? hs.blocks0 : 0)) * lt_items(Q) + threadIdx.x / Q, sub = threadIdx.x % Q;
  const bool live = i < h.n && h.cnt[i] != 0;
  GridDev g;
  int sc = 0, nc = 0, c0[3] = {0, 0, 0}, c1[3] = {-1, -1, -1};
  if (live) {
    g = *gp;
    sc = h.rec[i].tag >> 1;
    cell_range(g, h.rec[i].lo, h.rec[i].hi, c0, c1);
    nc = (c1[0] - c0[0] + 1) * (c1[1] - c0[1] + 1) * (c1[2] - c0[2] + 1);
  }
  auto put = [&](int64_t slot, int x, int y, int z) {
    if (slot < h.ent_cap) {
      Entry en;
      en.cell = cell_key(x, y, z, sc);
      en.item = i;
      en.dlo = (x - c0[0]) | ((y - c0[1]) << 6) | ((z - c0[2]) << 12);
      h.ent[slot] = en;
    } else {
      atomicOr(status, ST_PLAN_OVERFLOW);
    }
  };
  // count per bucket in LDS (entries that find no slot take their global
  // slot now)
  each_cell<Q>(c0, c1, nc, sub, [&](int x, int y, int z) {
    const uint32_t b = cell_hash(x, y, z, sc) & bmask;
    const int t = lt_insert(s_key, b);
    if (t >= 0)
      atomicAdd(&s_cnt[t], 1);
    else
      put(h.bstart[b] + atomicSub(&h.bcnt[b], 1) - 1, x, y, z);
  });
  __syncthreads();
  // reserve each bucket's range once
  for (int k = threadIdx.x; k < LT_SLOTS; k += lt_threads(Q))
    if (s_key[k] != 0u) s_base[k] = atomicSub(&h.bcnt[s_key[k] - 1u], s_cnt[k]) - s_cnt[k];
  __syncthreads();
  // place: rank within the workgroup's range from the LDS count
  each_cell<Q>(c0, c1, nc, sub, [&](int x, int y, int z) {
    const uint32_t b = cell_hash(x, y, z, sc) & bmask;
    const int t = lt_find(s_key, b);
    if (t >= 0) put(h.bstart[b] + s_base[t] + atomicSub(&s_cnt[t], 1) - 1, x, y, z);
  });
}

// big records, cut into up to LQ_PARTS parts, a wavefront each (grid y: the
// side): the two ground triangles of the sphere took a wavefront each 14 us,
// one group of 64 returning adds after the other, and 4 like this.
__global__ void k_big_fill(HSides hs, const GridDev *__restrict__ gp, uint32_t bmask, uint32_t *status) {
  const HSide &h = hs.s[blockIdx.y];
  const int lane = threadIdx.x & 63;
  const int64_t nbig = h.n_big[0];
  const int64_t nw = ((int64_t)gridDim.x * blockDim.x) >> 6;
  int parts = 1;
  while (parts < LQ_PARTS && nbig * (2 * parts) <= nw) parts *= 2;
  for (int64_t w = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6; w < nbig * parts; w += nw) {
    const int i = h.big[w / parts], part = (int)(w % parts);
    const GridDev g = *gp;
    const int sc = h.rec[i].tag >> 1;
    int c0[3], c1[3];
    cell_range(g, h.rec[i].lo, h.rec[i].hi, c0, c1);
    const int nc = (c1[0] - c0[0] + 1) * (c1[1] - c0[1] + 1) * (c1[2] - c0[2] + 1);
    for (int c = 64 * part + lane; c < nc; c += 64 * parts) {
      int x, y, z;
      big_cell(c0, c1, c, x, y, z);
      const uint32_t b = cell_hash(x, y, z, sc) & bmask;
      const int64_t slot = h.bstart[b] + atomicSub(&h.bcnt[b], 1) - 1;
      if (slot < h.ent_cap) {
        Entry en;
        en.cell = cell_key(x, y, z, sc);
        en.item = i;
        en.dlo = (x - c0[0]) | ((y - c0[1]) << 6) | ((z - c0[2]) << 12);
        h.ent[slot] = en;
      } else {
        atomicOr(status, ST_PLAN_OVERFLOW);
      }
    }
  }
}

constexpr int BIG_BLOCKS = 256;

__device__ __forceinline__ bool overlap(const double *qlo, const double *qhi, const ItemRec &r) {
#pragma unroll
  for (int a = 0; a < 3; ++a)
    if (!(qlo[a] <= r.hi[a] && r.lo[a] <= qhi[a])) return false;
  return true;
}

template <int KIND>
__device__ __forceinline__ bool pair_ok(int q, int qa, int qb, bool qdof, int it, const ItemRec &r) {
  if (KIND == 1 && it <= q) return false;
  if (KIND == 0) {
    if (qa == r.v[0] || qa == r.v[1] || qa == r.v[2]) return false;
  } else {
    if (qa == r.v[0] || qa == r.v[1] || qb == r.v[0] || qb == r.v[1]) return false;
  }
  return qdof || (r.tag & 1);
}

// Scan the hash entries [e0, e1) of one bucket for the query's cell
// (x, y, z) (key), with the query's lower cell (qx, qy, qz): entries are
// read four at a time (independent loads), filtered on their own fields
// (cell, EE order, lower-corner rule), then the surviving items' records
// are read together and tested exactly; emit(item) for each candidate.
template <int KIND, class Emit>
__device__ __forceinline__ void scan_bucket(const Entry *__restrict__ ent, const ItemRec *__restrict__ items,
                                            int64_t e0, int64_t e1, uint64_t key, int x, int y, int z, int qx,
                                            int qy, int qz, int q, int qa, int qb, bool qdof, const double *qlo,
                                            const double *qhi, Emit emit) {
  for (int64_t e = e0; e < e1; e += 4) {
    Entry en[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (e + u < e1) {
        en[u] = ent[e + u];
      } else {
        en[u].cell = ~0ull;
        en[u].item = 0;
        en[u].dlo = 0;
      }
    }
    bool pass[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int it = en[u].item;
      const int ix = x - (en[u].dlo & 63), iy = y - ((en[u].dlo >> 6) & 63), iz = z - ((en[u].dlo >> 12) & 63);
      // & rather than &&: no branches between the fields' tests
      pass[u] = (en[u].cell == key) & (KIND == 0 || it > q) & ((ix > qx ? ix : qx) == x) &
                ((iy > qy ? iy : qy) == y) & ((iz > qz ? iz : qz) == z);
    }
    ItemRec r[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (pass[u]) r[u] = items[en[u].item];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (pass[u] && (pair_ok<KIND>(q, qa, qb, qdof, en[u].item, r[u]) & overlap(qlo, qhi, r[u]))) emit(en[u].item);
  }
}

constexpr int QT = 128;         // query threads per block
constexpr int XCD_CHUNK = 16;   // consecutive query workgroups kept on one XCD
constexpr int APPEND_BUF = 16;  // per-thread LDS staging for append mode

// append mode: stage a candidate in the thread's LDS slots; flush a full
// buffer with one atomic
__device__ __forceinline__ void stage_pair(int2 *buf, int &nb, int q, int it, unsigned long long *total,
                                           int32_t *out, int64_t cap) {
  buf[nb] = make_int2(q, it);
  if (++nb == APPEND_BUF) {
    const int64_t p = (int64_t)atomicAdd(total, (unsigned long long)APPEND_BUF);
    for (int j = 0; j < APPEND_BUF; ++j)
      if (p + j < cap) {
        out[2 * (p + j)] = buf[j].x;
        out[2 * (p + j) + 1] = buf[j].y;
      }
    nb = 0;
  }
}

// Flush every lane's staged pairs with one atomic for the wavefront (all
// lanes of the wavefront must call).
__device__ __forceinline__ void wave_flush(int2 *buf, int &nbuf, unsigned long long *total, int32_t *out,
                                           int64_t cap) {
  const int lane = threadIdx.x & 63;
  int64_t ex = nbuf;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int64_t yv = __shfl_up(ex, o, 64);
    if (lane >= o) ex += yv;
  }
  const int64_t wsum = __shfl(ex, 63, 64);
  int64_t p0 = 0;
  if (lane == 63 && wsum) p0 = (int64_t)atomicAdd(total, (unsigned long long)wsum);
  p0 = __shfl(p0, 63, 64);
  const int64_t p = p0 + ex - nbuf;
  for (int j = 0; j < nbuf; ++j)
    if (p + j < cap) {
      out[2 * (p + j)] = buf[j].x;
      out[2 * (p + j) + 1] = buf[j].y;
    }
  nbuf = 0;
}

struct QueryArgs {
  const GridDev *g;
  uint32_t bmask;
  const int64_t *bstart;
  const Entry *ent;
  int64_t ent_cap;
  const int32_t *large;
  const int64_t *n_large;
  const ItemRec *items;
  const int32_t *rowptr;
  const int32_t *vscene;
  const int32_t *qlist;    // when set: the queries to run, *n_qlist of them
  const int64_t *n_qlist;
  int32_t *defer;          // when set: queries spanning more than LQ_CELLS cells are
  int64_t *n_defer;        // listed here and skipped (k_query_lq runs them)
  int n_items;             // items in the hash (k_query_lq: a query of more cells tests them all)
};

// Queries whose boxes span more than this many cells run one wavefront
// each (k_query_lq) instead of one thread each.
constexpr int LQ_CELLS = 64;

__device__ __forceinline__ int64_t n_cells(const int *c0, const int *c1) {
  return (int64_t)(c1[0] - c0[0] + 1) * (c1[1] - c0[1] + 1) * (c1[2] - c0[2] + 1);
}

// box, vertices, DoF flag and scene of query q (a vertex for PT, an edge
// record for EE)
template <int KIND>
__device__ __forceinline__ void query_data(int q, const double *xs, const double *x1s, int n_vert, double h,
                                           const QueryArgs &qa_, double *qlo, double *qhi, int &qa, int &qb,
                                           bool &qdof, int &qsc) {
  if (KIND == 0) {
    qa = q;
    qb = -1;
    prim_box<1>(&qa, xs, x1s, n_vert, h, qlo, qhi);
    qdof = has_dof(qa_.rowptr, qa);
    qsc = scene_of(qa_.vscene, qa);
  } else {
    const ItemRec r = qa_.items[q];
    qa = r.v[0];
    qb = r.v[1];
    qdof = r.tag & 1;
    qsc = r.tag >> 1;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      qlo[a] = r.lo[a];
      qhi[a] = r.hi[a];
    }
  }
}

// modes: 0 count, 1 write (offset per query, sorted per query, capacity
// guarded)
template <int KIND, int MODE>
__global__ __launch_bounds__(QT) void k_query(int nq, const double *__restrict__ xs, const double *__restrict__ x1s,
                                              int n_vert, double h, QueryArgs qa_, int32_t *__restrict__ cnt,
                                              const int64_t *__restrict__ off, int32_t *__restrict__ out, int64_t cap,
                                              unsigned long long *total, uint32_t *status) {
  const GridDev g = *qa_.g;
  const ItemRec *items = qa_.items;
  const int nl = (int)*qa_.n_large;  // read before any store: a later load would wait for the stores
  // workgroups of consecutive queries in runs on one XCD (its L2 then holds
  // their hash entries)
  const int t = xcd_block(XCD_CHUNK) * blockDim.x + threadIdx.x;
  const int q = qa_.qlist ? (t < *qa_.n_qlist ? qa_.qlist[t] : -1) : t;
  const bool live = q >= 0 && q < nq;
  int qa = 0, qb = -1, qsc = 0;
  bool qdof = false;
  double qlo[3] = {0, 0, 0}, qhi[3] = {0, 0, 0};
  if (live) query_data<KIND>(q, xs, x1s, n_vert, h, qa_, qlo, qhi, qa, qb, qdof, qsc);
  int c0[3] = {0, 0, 0}, c1[3] = {-1, -1, -1};
  if (live) cell_range(g, qlo, qhi, c0, c1);
  if (live && qa_.defer && n_cells(c0, c1) > LQ_CELLS) {
    // a wavefront counts and writes this query (k_query_lq)
    if (MODE == 0) qa_.defer[atomicAdd((unsigned long long *)qa_.n_defer, 1ull)] = q;
    return;
  }
  const int64_t base = (MODE == 1 && live) ? off[q] : 0;
  int64_t k = 0;
  for (int z = c0[2]; z <= c1[2]; ++z)
    for (int y = c0[1]; y <= c1[1]; ++y)
      for (int x = c0[0]; x <= c1[0]; ++x) {
        const uint64_t key = cell_key(x, y, z, qsc);
        const uint32_t b = cell_hash(x, y, z, qsc) & qa_.bmask;
        const int64_t e1 = qa_.bstart[b + 1] < qa_.ent_cap ? qa_.bstart[b + 1] : qa_.ent_cap;
        // report only in the cell holding the lower corner of the overlap:
        // max(query low cell, item low cell) == this cell on every axis
        scan_bucket<KIND>(qa_.ent, items, qa_.bstart[b], e1, key, x, y, z, c0[0], c0[1], c0[2], q, qa, qb, qdof,
                          qlo, qhi, [&](int it) {
                            if (MODE == 1 && base + k < cap) {
                              out[2 * (base + k)] = q;
                              out[2 * (base + k) + 1] = it;
                            }
                            ++k;
                          });
      }
  if (live) {
    for (int j = 0; j < nl; ++j) {
      const int it = qa_.large[j];
      const ItemRec r = items[it];
      if ((r.tag >> 1) != qsc) continue;
      if (!pair_ok<KIND>(q, qa, qb, qdof, it, r)) continue;
      if (!overlap(qlo, qhi, r)) continue;
      if (MODE == 1 && base + k < cap) {
        out[2 * (base + k)] = q;
        out[2 * (base + k) + 1] = it;
      }
      ++k;
    }
  }
  if (MODE == 0 && live) cnt[q] = (int32_t)k;
  if (MODE == 1 && live) {
    if (base + k > cap) {
      atomicOr(status, ST_PLAN_OVERFLOW);
    } else if (k > 1) {
      int32_t *seg = out + 2 * base;
      for (int64_t i = 1; i < k; ++i) {
        int32_t v = seg[2 * i + 1];
        int64_t j = i - 1;
        while (j >= 0 && seg[2 * j + 1] > v) {
          seg[2 * (j + 1) + 1] = seg[2 * j + 1];
          --j;
        }
        seg[2 * (j + 1) + 1] = v;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Queries whose boxes span more than LQ_CELLS cells (listed by the
// per-query kernels, or too large to bin or hash): one wavefront per query,
// its cells and the items too large to hash spread over the 64 lanes, so
// that one huge box does not keep a single thread scanning thousands of
// cells.  MODE 0 counts each query's candidates into cnt[q]; MODE 1 writes
// them, unsorted, to tmp at the query's offset (k_seg_rank then puts them
// in order into out); MODE 2 appends them to out (staged per lane), with a
// short list's queries in up to LQ_PARTS parts, a wavefront each: one
// wavefront to each of the 10 large edges of a sheet took 62 us, most of it
// waits for one group of loads after the other; 9 us in 32 parts each.
// ---------------------------------------------------------------------------
template <int KIND, int MODE>
__global__ __launch_bounds__(QT) void k_query_lq(const int32_t *__restrict__ qlist, const int64_t *__restrict__ n_qlist,
                                                 const double *__restrict__ xs, const double *__restrict__ x1s,
                                                 int n_vert, double h, QueryArgs qa_, int32_t *__restrict__ cnt,
                                                 const int64_t *__restrict__ off, int32_t *__restrict__ tmp,
                                                 int32_t *__restrict__ out, int64_t cap, unsigned long long *total) {
  __shared__ int2 s_buf[QT * APPEND_BUF];
  int2 *buf = s_buf + threadIdx.x * APPEND_BUF;
  int nbuf = 0;
  const int lane = threadIdx.x & 63;
  const ItemRec *items = qa_.items;
  const GridDev g = *qa_.g;
  const int n_large = (int)*qa_.n_large;
  const int64_t nl = *n_qlist;
  const int64_t nw = ((int64_t)gridDim.x * QT) >> 6;
  int parts = 1;
  while (MODE == 2 && parts < LQ_PARTS && nl * (2 * parts) <= nw) parts *= 2;
  for (int64_t w = ((int64_t)blockIdx.x * QT + threadIdx.x) >> 6; w < nl * parts; w += nw) {
    const int q = qlist[w / parts], part = (int)(w % parts);
    double qlo[3], qhi[3];
    int qa, qb, qsc;
    bool qdof;
    query_data<KIND>(q, xs, x1s, n_vert, h, qa_, qlo, qhi, qa, qb, qdof, qsc);
    int c0[3], c1[3];
    cell_range(g, qlo, qhi, c0, c1);
    const int64_t nx = c1[0] - c0[0] + 1, ny = c1[1] - c0[1] + 1;
    const int64_t nc = n_cells(c0, c1);
    // a query whose cells outnumber the items by a sixteenth tests every
    // item instead, four independent record loads per lane at a time (the
    // same set: the cell scan reports each overlapping item once, the
    // unhashed ones from their list; a cell costs a chain of dependent
    // loads, an item one coalesced load)
    const bool all_items = qa_.n_items > 0 && 16 * nc > (int64_t)qa_.n_items;
    // this lane's share: cells lane, lane + 64, ..., then large items alike
    auto each = [&](auto emit) {
      if (all_items) {
        for (int i0 = 256 * part; i0 < qa_.n_items; i0 += 256 * parts) {
          ItemRec r[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int it = i0 + 64 * u + lane;
            r[u] = items[it < qa_.n_items ? it : 0];
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int it = i0 + 64 * u + lane;
            // & rather than &&: every record was read, so nothing needs a branch
            if ((it < qa_.n_items) & ((r[u].tag >> 1) == qsc) & pair_ok<KIND>(q, qa, qb, qdof, it, r[u]) &
                overlap(qlo, qhi, r[u]))
              emit(it);
          }
        }
        return;
      }
      for (int64_t ci = 64 * part + lane; ci < nc; ci += 64 * parts) {
        const int x = c0[0] + (int)(ci % nx), y = c0[1] + (int)((ci / nx) % ny), z = c0[2] + (int)(ci / (nx * ny));
        const uint64_t key = cell_key(x, y, z, qsc);
        const uint32_t b = cell_hash(x, y, z, qsc) & qa_.bmask;
        const int64_t e1 = qa_.bstart[b + 1] < qa_.ent_cap ? qa_.bstart[b + 1] : qa_.ent_cap;
        scan_bucket<KIND>(qa_.ent, items, qa_.bstart[b], e1, key, x, y, z, c0[0], c0[1], c0[2], q, qa, qb, qdof,
                          qlo, qhi, emit);
      }
      for (int j = 64 * part + lane; j < n_large; j += 64 * parts) {
        const int it = qa_.large[j];
        const ItemRec r = items[it];
        if ((r.tag >> 1) == qsc && pair_ok<KIND>(q, qa, qb, qdof, it, r) && overlap(qlo, qhi, r)) emit(it);
      }
    };
    if constexpr (MODE == 2) {
      each([&](int it) { stage_pair(buf, nbuf, q, it, total, out, cap); });
      wave_flush(buf, nbuf, total, out, cap);
    } else {
      int64_t k = 0;
      each([&](int) { ++k; });
      int64_t ex = k;  // inclusive scan over the lanes
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int64_t yv = __shfl_up(ex, o, 64);
        if (lane >= o) ex += yv;
      }
      if constexpr (MODE == 0) {
        if (lane == 63) cnt[q] = (int32_t)ex;
      } else {
        int64_t p = off[q] + ex - k;
        each([&](int it) {
          if (p < cap) tmp[p] = it;
          ++p;
        });
      }
    }
  }
}

// Sorts the candidates of each listed query (tmp, unsorted, at off[q]) into
// out by rank: the items of one query are distinct, so an item's position
// is the number of smaller items, counted against the query's list staged
// through LDS in tiles.  One workgroup per query.
constexpr int RANK_T = 256, RANK_TILE = 2048;
__global__ __launch_bounds__(RANK_T) void k_seg_rank(const int32_t *__restrict__ qlist,
                                                     const int64_t *__restrict__ n_qlist,
                                                     const int32_t *__restrict__ cnt, const int64_t *__restrict__ off,
                                                     const int32_t *__restrict__ tmp, int32_t *__restrict__ out,
                                                     int64_t cap) {
  __shared__ int32_t tile[RANK_TILE];
  const int64_t nl = *n_qlist;
  for (int64_t w = blockIdx.x; w < nl; w += gridDim.x) {
    const int q = qlist[w];
    const int64_t o = off[q], L = cnt[q];
    if (o + L > cap) continue;  // the host checked the total against the capacity
    for (int64_t c0 = 0; c0 < L; c0 += RANK_T) {
      const int64_t i = c0 + threadIdx.x;
      const int32_t v = i < L ? tmp[o + i] : 0x7fffffff;
      int64_t rank = 0;
      for (int64_t t0 = 0; t0 < L; t0 += RANK_TILE) {
        const int tn = (int)(L - t0 < RANK_TILE ? L - t0 : RANK_TILE);
        __syncthreads();
        for (int j = threadIdx.x; j < tn; j += RANK_T) tile[j] = tmp[o + t0 + j];
        __syncthreads();
        for (int j = 0; j < tn; ++j) rank += tile[j] < v;
      }
      if (i < L) {
        out[2 * (o + rank)] = q;
        out[2 * (o + rank) + 1] = v;
      }
    }
  }
}

template <int KIND, int MODE>
static void launch_query(int nq, const double *xs, const double *x1s, int n_vert, double h, const QueryArgs &qa,
                         int32_t *cnt, const int64_t *off, int32_t *out, int64_t cap, unsigned long long *total,
                         uint32_t *status, hipStream_t s) {
  k_query<KIND, MODE><<<grid_for(nq, QT), QT, 0, s>>>(nq, xs, x1s, n_vert, h, qa, cnt, off, out, cap, total,
                                                       status);
}

// ---------------------------------------------------------------------------
// Cell-parallel query (append mode): one thread per (query, cell of its
// box), listed in query order so that neighbouring threads share the query
// and its neighbourhood (mesh order is spatially coherent).  Queries
// covering more than MAX_ITEM_CELLS cells run per query (k_query on a
// list).
// ---------------------------------------------------------------------------
struct QEntry {
  uint64_t cell;
  int32_t q;
  int32_t dlo;  // cell minus the query's lower cell, 6 bits per axis
};

template <int KIND>
__global__ void k_qcells(int nq, const double *__restrict__ xs, const double *__restrict__ x1s, int n_vert, double h,
                         QueryArgs qa_, int32_t *qcnt, int32_t *qlarge, int64_t *n_qlarge) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= nq) return;
  const GridDev g = *qa_.g;
  double qlo[3], qhi[3];
  int qa, qb, qsc;
  bool qdof;
  query_data<KIND>(q, xs, x1s, n_vert, h, qa_, qlo, qhi, qa, qb, qdof, qsc);
  int c0[3], c1[3];
  cell_range(g, qlo, qhi, c0, c1);
  const int64_t nc = (int64_t)(c1[0] - c0[0] + 1) * (c1[1] - c0[1] + 1) * (c1[2] - c0[2] + 1);
  if (nc > MAX_ITEM_CELLS) {
    const int slot = (int)atomicAdd((unsigned long long *)n_qlarge, 1ull);
    qlarge[slot] = q;
    qcnt[q] = 0;
  } else {
    qcnt[q] = (int32_t)nc;
  }
}

template <int KIND>
__global__ void k_qlist(int nq, const double *__restrict__ xs, const double *__restrict__ x1s, int n_vert, double h,
                        QueryArgs qa_, const int32_t *qcnt, const int64_t *qoff, QEntry *qent, int64_t qent_cap,
                        uint32_t *status) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= nq || qcnt[q] == 0) return;
  const GridDev g = *qa_.g;
  double qlo[3], qhi[3];
  int qa, qb, qsc;
  bool qdof;
  query_data<KIND>(q, xs, x1s, n_vert, h, qa_, qlo, qhi, qa, qb, qdof, qsc);
  int c0[3], c1[3];
  cell_range(g, qlo, qhi, c0, c1);
  int64_t slot = qoff[q];
  for (int z = c0[2]; z <= c1[2]; ++z)
    for (int y = c0[1]; y <= c1[1]; ++y)
      for (int x = c0[0]; x <= c1[0]; ++x, ++slot) {
        if (slot < qent_cap)
          qent[slot] = QEntry{cell_key(x, y, z, qsc), q, (x - c0[0]) | ((y - c0[1]) << 6) | ((z - c0[2]) << 12)};
        else
          atomicOr(status, ST_PLAN_OVERFLOW);
      }
}

template <int KIND>
__global__ __launch_bounds__(QT) void k_query_ent(const int64_t *__restrict__ n_qent, int64_t qent_cap,
                                                  const QEntry *__restrict__ qent, const double *__restrict__ xs,
                                                  const double *__restrict__ x1s, int n_vert, double h, QueryArgs qa_,
                                                  int32_t *__restrict__ out, int64_t cap, unsigned long long *total) {
  __shared__ int2 s_buf[QT * APPEND_BUF];
  int2 *buf = s_buf + threadIdx.x * APPEND_BUF;
  int nbuf = 0;
  const ItemRec *items = qa_.items;
  const int nl = (int)*qa_.n_large;  // read before any store: a later load would wait for the stores
  const int64_t n = *n_qent < qent_cap ? *n_qent : qent_cap;
  for (int64_t base = (int64_t)blockIdx.x * QT; base < n; base += (int64_t)gridDim.x * QT) {
    const int64_t t = base + threadIdx.x;
    if (t < n) {
      const QEntry qe = qent[t];
      const int q = qe.q;
      double qlo[3], qhi[3];
      int qa, qb, qsc;
      bool qdof;
      query_data<KIND>(q, xs, x1s, n_vert, h, qa_, qlo, qhi, qa, qb, qdof, qsc);
      const int x = (int)(qe.cell & 0xffff), y = (int)((qe.cell >> 16) & 0xffff), z = (int)((qe.cell >> 32) & 0xffff);
      const int qx = x - (qe.dlo & 63), qy = y - ((qe.dlo >> 6) & 63), qz = z - ((qe.dlo >> 12) & 63);
      const uint32_t b = cell_hash(x, y, z, qsc) & qa_.bmask;
      const int64_t e1 = qa_.bstart[b + 1] < qa_.ent_cap ? qa_.bstart[b + 1] : qa_.ent_cap;
      scan_bucket<KIND>(qa_.ent, items, qa_.bstart[b], e1, qe.cell, x, y, z, qx, qy, qz, q, qa, qb, qdof, qlo, qhi,
                        [&](int it) { stage_pair(buf, nbuf, q, it, total, out, cap); });
      if (qe.dlo == 0) {
        // the query's lower cell also runs the items too large to hash
        for (int j = 0; j < nl; ++j) {
          const int it = qa_.large[j];
          const ItemRec r = items[it];
          if ((r.tag >> 1) != qsc) continue;
          if (!pair_ok<KIND>(q, qa, qb, qdof, it, r)) continue;
          if (!overlap(qlo, qhi, r)) continue;
          stage_pair(buf, nbuf, q, it, total, out, cap);
        }
      }
    }
    if (__any(nbuf >= APPEND_BUF / 2)) wave_flush(buf, nbuf, total, out, cap);
  }
  wave_flush(buf, nbuf, total, out, cap);
}

// Wavefront per (query, cell): the 64 lanes read 64 consecutive entries of
// the cell's bucket at once (coalesced), filter them in parallel and test
// the survivors exactly; the query's data is the same for every lane.
// Candidates are staged per lane in LDS as in k_query.  Query cells are
// taken in query order, one per wavefront at a time.
template <int KIND>
__global__ __launch_bounds__(QT) void k_query_wave(const int64_t *__restrict__ n_qent, int64_t qent_cap,
                                                   const QEntry *__restrict__ qent, const double *__restrict__ xs,
                                                   const double *__restrict__ x1s, int n_vert, double h,
                                                   QueryArgs qa_, int32_t *__restrict__ out, int64_t cap,
                                                   unsigned long long *total) {
  __shared__ int2 s_buf[QT * APPEND_BUF];
  int2 *buf = s_buf + threadIdx.x * APPEND_BUF;
  int nbuf = 0;
  const ItemRec *items = qa_.items;
  const int lane = threadIdx.x & 63;
  const int nl = (int)*qa_.n_large;  // read before any store: a later load would wait for the stores
  const int64_t n = *n_qent < qent_cap ? *n_qent : qent_cap;
  const int64_t wave = ((int64_t)blockIdx.x * QT + threadIdx.x) >> 6;
  const int64_t n_waves = ((int64_t)gridDim.x * QT) >> 6;
  for (int64_t t = wave; t < n; t += n_waves) {
    const QEntry qe = qent[t];
    const int q = qe.q;
    double qlo[3], qhi[3];
    int qa, qb, qsc;
    bool qdof;
    query_data<KIND>(q, xs, x1s, n_vert, h, qa_, qlo, qhi, qa, qb, qdof, qsc);
    const int x = (int)(qe.cell & 0xffff), y = (int)((qe.cell >> 16) & 0xffff), z = (int)((qe.cell >> 32) & 0xffff);
    const int qx = x - (qe.dlo & 63), qy = y - ((qe.dlo >> 6) & 63), qz = z - ((qe.dlo >> 12) & 63);
    const uint32_t b = cell_hash(x, y, z, qsc) & qa_.bmask;
    const int64_t e0 = qa_.bstart[b];
    const int64_t e1 = qa_.bstart[b + 1] < qa_.ent_cap ? qa_.bstart[b + 1] : qa_.ent_cap;
    for (int64_t base = e0; base < e1; base += 64) {
      const int64_t e = base + lane;
      if (e < e1) {
        const Entry en = qa_.ent[e];
        const int it = en.item;
        // report only in the cell holding the lower corner of the overlap
        const int ix = x - (en.dlo & 63), iy = y - ((en.dlo >> 6) & 63), iz = z - ((en.dlo >> 12) & 63);
        if (en.cell == qe.cell && (KIND == 0 || it > q) && (ix > qx ? ix : qx) == x && (iy > qy ? iy : qy) == y &&
            (iz > qz ? iz : qz) == z) {
          const ItemRec r = items[it];
          if (pair_ok<KIND>(q, qa, qb, qdof, it, r) && overlap(qlo, qhi, r)) buf[nbuf++] = make_int2(q, it);
        }
      }
      if (__any(nbuf >= APPEND_BUF - 1)) wave_flush(buf, nbuf, total, out, cap);
    }
    if (qe.dlo == 0) {
      // the query's lower cell also runs the items too large to hash
      for (int jb = 0; jb < nl; jb += 64) {
        const int j = jb + lane;
        if (j < nl) {
          const int it = qa_.large[j];
          const ItemRec r = items[it];
          if ((r.tag >> 1) == qsc && pair_ok<KIND>(q, qa, qb, qdof, it, r) && overlap(qlo, qhi, r))
            buf[nbuf++] = make_int2(q, it);
        }
        if (__any(nbuf >= APPEND_BUF - 1)) wave_flush(buf, nbuf, total, out, cap);
      }
    }
  }
  wave_flush(buf, nbuf, total, out, cap);
}

// Wavefront-level candidate staging: every lane of the wavefront calls
// push (ok false where it has nothing); positions come from the ballot, so
// the count stays the same on every lane and needs no atomics.  A flush
// reserves the whole staged run with one global atomic and writes it with
// consecutive lanes on consecutive pairs.
__device__ __forceinline__ void wave_push(bool ok, int2 pr, int2 *wout, int &wcnt) {
  const unsigned long long m = __ballot(ok);
  const int lane = threadIdx.x & 63;
  if (ok) wout[wcnt + __popcll(m & ((1ull << lane) - 1ull))] = pr;
  wcnt += __popcll(m);
}
__device__ __forceinline__ void wave_out_flush(int2 *wout, int &wcnt, unsigned long long *total,
                                               int32_t *out, int64_t cap) {
  if (wcnt == 0) return;
  __builtin_amdgcn_wave_barrier();
  const int lane = threadIdx.x & 63;
  int64_t p0 = 0;
  if (lane == 0) p0 = (int64_t)atomicAdd(total, (unsigned long long)wcnt);
  p0 = __shfl(p0, 0, 64);
  int2 *o2 = reinterpret_cast<int2 *>(out);
  for (int k = lane; k < wcnt; k += 64)
    if (p0 + k < cap) o2[p0 + k] = wout[k];
  __builtin_amdgcn_wave_barrier();
  wcnt = 0;
}

// Per-query append (work split 0) as rounds: in each round every lane
// advances its own query by one group of up to four hash entries (or four
// large items), so wavefront-uniform points come often enough to flush
// all lanes' staged pairs with one atomic per wavefront.  Visits the same
// cells, entries and large items in the same order as k_query.
template <int KIND>
__global__ __launch_bounds__(QT) void k_query_sm(int nq, const double *__restrict__ xs,
                                                 const double *__restrict__ x1s, int n_vert, double h, QueryArgs qa_,
                                                 int32_t *__restrict__ out, int64_t cap, unsigned long long *total) {
  __shared__ int2 s_buf[QT * APPEND_BUF];
  int2 *buf = s_buf + threadIdx.x * APPEND_BUF;
  int nbuf = 0;
  const ItemRec *items = qa_.items;
  const int t = xcd_block(XCD_CHUNK) * blockDim.x + threadIdx.x;
  const int q = qa_.qlist ? (t < *qa_.n_qlist ? qa_.qlist[t] : -1) : t;
  const bool live = q >= 0 && q < nq;
  int qa = 0, qb = -1, qsc = 0;
  bool qdof = false;
  double qlo[3] = {0, 0, 0}, qhi[3] = {0, 0, 0};
  int c0[3] = {0, 0, 0}, c1[3] = {0, 0, 0};
  bool deferred = false;
  if (live) {
    query_data<KIND>(q, xs, x1s, n_vert, h, qa_, qlo, qhi, qa, qb, qdof, qsc);
    cell_range(*qa_.g, qlo, qhi, c0, c1);
    if (qa_.defer && n_cells(c0, c1) > LQ_CELLS) {
      qa_.defer[atomicAdd((unsigned long long *)qa_.n_defer, 1ull)] = q;  // run by k_query_lq
      deferred = true;
    }
  }
  const int nl = (int)*qa_.n_large;
  int x = c0[0], y = c0[1], z = c0[2];
  int64_t e = 0, e1 = 0;
  uint64_t key = 0;
  int lj = 0;
  int phase = live && !deferred ? 0 : 3;  // 0 open cell, 1 scan its bucket, 2 large items, 3 done
  auto emit = [&](int it) { buf[nbuf++] = make_int2(q, it); };
  while (__any(phase != 3)) {
    if (phase == 0) {
      key = cell_key(x, y, z, qsc);
      const uint32_t b = cell_hash(x, y, z, qsc) & qa_.bmask;
      e = qa_.bstart[b];
      e1 = qa_.bstart[b + 1] < qa_.ent_cap ? qa_.bstart[b + 1] : qa_.ent_cap;
      phase = 1;
    }
    if (phase == 1) {
      if (e < e1) {
        const int64_t eg = e + 4 < e1 ? e + 4 : e1;
        scan_bucket<KIND>(qa_.ent, items, e, eg, key, x, y, z, c0[0], c0[1], c0[2], q, qa, qb, qdof, qlo, qhi, emit);
        e = eg;
      }
      if (e >= e1) {
        if (++x > c1[0]) {
          x = c0[0];
          if (++y > c1[1]) {
            y = c0[1];
            if (++z > c1[2]) phase = 2;
          }
        }
        if (phase == 1) phase = 0;
      }
    } else if (phase == 2) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int j = lj + u;
        if (j < nl) {
          const int it = qa_.large[j];
          const ItemRec r = items[it];
          if ((r.tag >> 1) == qsc && pair_ok<KIND>(q, qa, qb, qdof, it, r) && overlap(qlo, qhi, r)) emit(it);
        }
      }
      lj += 4;
      if (lj >= nl) phase = 3;
    }
    if (__any(nbuf > APPEND_BUF - 4)) wave_flush(buf, nbuf, total, out, cap);
  }
  wave_flush(buf, nbuf, total, out, cap);
}

// ---------------------------------------------------------------------------
// Bucket join (work split 3).  The queries are hashed like the items (PT:
// vertex records in a second hash over the same grid and buckets; EE: the
// edge hash itself), so every (query, item) pair that shares a cell lies in
// one bucket of both hashes.  A workgroup takes tiles of consecutive query
// entries (rows, in bucket order); the item entries of the buckets those
// rows touch form one contiguous window of the item hash, staged in LDS in
// chunks of JWIN entries together with their records.  Each row then tests
// the items of its own bucket from LDS: same cell, lower-corner rule
// (min of the two offsets from the lower cells is zero on every axis),
// adjacency and DoF rule, exact box overlap.  EE joins the edge hash with
// itself: each row pairs with about half of its bucket (the entries after
// it, wrapping to the bucket's start), so that every unordered pair of the
// bucket is tested once, and reports (min, max).  The row that is a query's lower cell also runs the
// items too large to hash, as in the per-query splits; queries too large
// to hash run per query (k_query_lq).
// ---------------------------------------------------------------------------
constexpr int JT = 128;     // threads of a workgroup
constexpr int JWIN = 192;   // item entries staged in LDS per chunk (five workgroups per CU)
constexpr int JOUT = 1024;  // candidates staged per wavefront
// Lanes to a row (log2; PT, EE): a row's partners are taken in turn by 4 or
// 2 lanes, and by up to 2^JSPLIT in a list so short that its rows would not
// fill the chip (below JSWG workgroups per CU).  A wavefront goes on for its
// longest row, and with few rows to it the rows of one bucket, of one
// length, are together: grasp (19.0 and 44.9 million tests) PT 148 us with
// one lane to a row, 104 with two, 92 with four, 131 with eight; EE 244 and
// 194 with one and two; the sphere's 5,072 PT rows 93 us and, with eight, 18;
// plate PT 100 and 68, but EE 107 and 121 (21 partners a row on average).
// The lines (a list takes 8 lanes up to 40,960 PT or 20,480 EE rows, an EE
// list 4 up to 40,960), with both sides in us:
//   PT, 4 and 8 lanes: 747 rows 11.5 and 9.6, 5,105 17.3 and 13.9, 15,411
//   21.1 and 21.4, 27,989 24.8 and 34.2, 52,868 44.6 and 54.7;
//   EE, 2, 4 and 8 lanes: the sphere's 23,493 rows, whose ground edges share
//   buckets with everything, 22.0, 18.6 and 26.3; grasps of 5,338 rows 11.3,
//   9.9 and 11.2, 18,945 14.6, 15.3 and 21.1, 34,254 16.0, 21.7 and 31.7.
// So short lists of long buckets set them; they cost even lists up to 10 us.
constexpr int JLANES[2] = {2, 1};
constexpr int JSPLIT = 3;
constexpr int JSWG[2] = {10, 5};
// A workgroup takes every gridDim-th tile, at most JWG workgroups per CU,
// and adds to the counter once at its end: with a workgroup to a tile and an
// add for each wavefront, the adds to that one address (7.5 ns each) took
// half of the batch's 959 us (62,072 wavefronts; now 569).  More workgroups
// add more often, fewer leave uneven tiles: 10, 20 and 40 to a CU, edges:
// candidates of the grasp 118, 117 and 165 us, its step 212, 199 and 195,
// plate 97, 108 and 123, batch 623, 569 and 558.
constexpr int JWG = 20;

struct JoinArgs {
  const Entry *rows;        // query entries in bucket order
  const int64_t *n_rows;    // number written (device), clamped to row_cap
  int64_t row_cap;
  const ItemRec *qrec;      // query records (PT: vertex records; EE: items)
  const int64_t *pbstart;   // item-hash bucket offsets (nb + 1)
  const Entry *pent;        // item entries
  int64_t pent_cap;
  const ItemRec *items;
  const int32_t *large;
  const int64_t *n_large;
  uint32_t bmask;
};

__device__ __forceinline__ uint32_t key_bucket(uint64_t key, uint32_t bmask) {
  return cell_hash((int)(key & 0xffff), (int)((key >> 16) & 0xffff), (int)((key >> 32) & 0xffff), (int)(key >> 48)) &
         bmask;
}

// lower-corner rule from the two offsets (cell minus lower cell, 6 bits per
// axis): on every axis one of the two offsets is zero.  With the row's
// nonzero fields as a mask (all ones in each such field) it is one AND per
// partner: (partner offsets & mask) == 0
__device__ __forceinline__ int nonzero_fields(int d) {
  return ((d & 63) != 0 ? 63 : 0) | ((d & (63 << 6)) != 0 ? 63 << 6 : 0) | ((d & (63 << 12)) != 0 ? 63 << 12 : 0);
}

// adjacency, DoF rule and exact box overlap of a (query, item) pair, with
// bitwise logic so that no part of it branches
template <int KIND>
__device__ __forceinline__ bool join_test(const ItemRec &r, int qa, int qb, bool qdof, const double *qlo,
                                          const double *qhi) {
  bool ok = (qa != r.v[0]) & (qa != r.v[1]);
  if (KIND == 0)
    ok &= qa != r.v[2];
  else
    ok &= (qb != r.v[0]) & (qb != r.v[1]);
  ok &= qdof | ((r.tag & 1) != 0);
  ok &= (qlo[0] <= r.hi[0]) & (r.lo[0] <= qhi[0]) & (qlo[1] <= r.hi[1]) & (r.lo[1] <= qhi[1]) &
        (qlo[2] <= r.hi[2]) & (r.lo[2] <= qhi[2]);
  return ok;
}

template <int KIND>
__global__ __launch_bounds__(JT) void k_join(JoinArgs ja, int64_t split_rows, int32_t *__restrict__ out, int64_t cap,
                                             unsigned long long *total) {
  __shared__ Entry s_ent[JWIN];
  __shared__ ItemRec s_rec[JWIN];
  __shared__ int2 s_out[JT / 64][JOUT];
  __shared__ int64_t s_win[2];
  __shared__ int s_left[JT / 64];
  int2 *wout = s_out[threadIdx.x >> 6];
  int wcnt = 0;
  const int64_t nr0 = *ja.n_rows;
  // read here, not after the scan: a late load of it waited for all of the
  // wavefront's stores, which kept finished wavefronts resident
  const int nl = (int)*ja.n_large;
  const int64_t n_rows = nr0 < ja.row_cap ? nr0 : ja.row_cap;
  int sp = JLANES[KIND];
  while (sp < JSPLIT && n_rows << (sp + 1) <= split_rows) ++sp;
  const int rt = JT >> sp, sub = threadIdx.x & ((1 << sp) - 1), step = 1 << sp;
  for (int64_t r0 = (int64_t)blockIdx.x * rt; r0 < n_rows; r0 += (int64_t)gridDim.x * rt) {  // uniform
    const int64_t r1 = r0 + rt < n_rows ? r0 + rt : n_rows;
    const int64_t i = r0 + (threadIdx.x >> sp);
    const bool live = i < r1;
    // the row: its entry, bucket, record and partner range
    Entry re{0, 0, 0};
    // partners: the entries [pa0, pa1) and then [pb0, pb1) of the row's
    // bucket [bs, be).  PT: the whole bucket.  EE: the next h entries after
    // the row, cyclically (wrapping to the bucket's start), with h = (n - 1)
    // / 2 for a bucket of n entries, plus one for the first half of an even
    // bucket (its partner n / 2 ahead): every unordered pair of the bucket
    // once, and every row about half the bucket, where scanning all later
    // entries left the first rows of a bucket with all of it.
    int64_t pa0 = 0, pa1 = 0, pb0 = 0, pb1 = 0, bs = 0, be = 0;
    double qlo[3] = {0, 0, 0}, qhi[3] = {0, 0, 0};
    int qa = 0, qb = -1, qsc = 0;
    bool qdof = false;
    if (live) {
      re = ja.rows[i];
      const uint32_t b = key_bucket(re.cell, ja.bmask);
      const int64_t e0 = ja.pbstart[b], e1 = ja.pbstart[b + 1];
      be = e1 < ja.pent_cap ? e1 : ja.pent_cap;
      bs = e0 < be ? e0 : be;
      if (KIND == 0) {
        pa0 = bs;
        pa1 = be;
      } else {
        const int64_t n = be - bs, pos = i - bs;
        const int64_t h = (n - 1) / 2 + ((n % 2 == 0 && pos < n / 2) ? 1 : 0);
        pa0 = i + 1;
        pa1 = i + 1 + h < be ? i + 1 + h : be;
        pb0 = bs;
        pb1 = bs + (i + 1 + h - be > 0 ? i + 1 + h - be : 0);
      }
      const ItemRec qr = ja.qrec[re.item];
      qa = qr.v[0];
      qb = qr.v[1];
      qdof = qr.tag & 1;
      qsc = qr.tag >> 1;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        qlo[a] = qr.lo[a];
        qhi[a] = qr.hi[a];
      }
    }
    // window of item entries for the whole tile: first row's bucket start to
    // last row's bucket end (rows are in bucket order)
    const int rmask = nonzero_fields(re.dlo);
    __syncthreads();  // the previous tile's window is read
    if (threadIdx.x == 0) s_win[0] = bs;
    if (i == r1 - 1) s_win[1] = be;
    __syncthreads();
    const int64_t w0 = s_win[0], w1 = s_win[1];
    for (int64_t c0 = w0; c0 < w1; c0 += JWIN) {
      const int nw = (int)(w1 - c0 < JWIN ? w1 - c0 : JWIN);
      __syncthreads();  // previous chunk consumed
      {
        constexpr int U = (JWIN + JT - 1) / JT;
        Entry e[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int k = u * JT + threadIdx.x;
          if (k < nw) e[u] = ja.pent[c0 + k];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int k = u * JT + threadIdx.x;
          if (k < nw) {
            s_ent[k] = e[u];
            s_rec[k] = ja.items[e[u].item];
          }
        }
      }
      __syncthreads();
      // this chunk's part of the two partner ranges, taken as one list
      const int64_t cend = c0 + nw;
      const int64_t a0 = pa0 > c0 ? pa0 : c0, a1 = pa1 < cend ? pa1 : cend;
      const int64_t b0 = pb0 > c0 ? pb0 : c0, b1 = pb1 < cend ? pb1 : cend;
      // chunk-relative: the list's entry tu is ra + tu below na, else rb + tu
      const int na = a1 > a0 ? (int)(a1 - a0) : 0;
      const int ntot = na + (b1 > b0 ? (int)(b1 - b0) : 0);
      const int ra = (int)(a0 - c0), rb = (int)(b0 - c0) - na;
      int t = sub;
      while (__any(t < ntot)) {
        // four partners per lane (the lanes of a row take them in turn): their entries and records read from LDS
        // without conditions (a conditional read kept the previous records
        // live in registers: ~45 copies per step and 200 VGPRs), then the
        // same-cell and lower-corner rule and the pair test
        Entry pe[4];
        bool pass[4];
        int idx[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int tu = t + u * step;
          idx[u] = tu < ntot ? (tu < na ? ra : rb) + tu : 0;
          pe[u] = s_ent[idx[u]];
        }
        ItemRec r[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) r[u] = s_rec[idx[u]];
#pragma unroll
        for (int u = 0; u < 4; ++u)
          pass[u] = (t + u * step < ntot) & (pe[u].cell == re.cell) & ((pe[u].dlo & rmask) == 0);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          // & rather than &&: the test is branch-free, a short circuit would branch
          const bool ok = pass[u] & join_test<KIND>(r[u], qa, qb, qdof, qlo, qhi);
          const int it = pe[u].item;
          const int2 pr = (KIND == 0 || re.item < it) ? make_int2(re.item, it) : make_int2(it, re.item);
          wave_push(ok, pr, wout, wcnt);
        }
        t += 4 * step;
        if (wcnt > JOUT - 4 * 64) wave_out_flush(wout, wcnt, total, out, cap);
      }
    }
    // the query's lower-cell row also runs the items too large to hash
    if (nl > 0) {
      const bool lower = live && re.dlo == 0;
      const int q = re.item;
      for (int jb = sub; __any(lower && jb < nl); jb += 4 * step) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int jj = jb + u * step;
          bool ok = false;
          int it = 0;
          if (lower && jj < nl) {
            it = ja.large[jj];
            const ItemRec r = ja.items[it];
            ok = ((r.tag >> 1) == qsc) & pair_ok<KIND>(q, qa, qb, qdof, it, r) & overlap(qlo, qhi, r);
          }
          wave_push(ok, make_int2(q, it), wout, wcnt);
        }
        if (wcnt > JOUT - 4 * 64) wave_out_flush(wout, wcnt, total, out, cap);
      }
    }
  }
  // what is left, with one atomic for the workgroup
  if ((threadIdx.x & 63) == 0) s_left[threadIdx.x >> 6] = wcnt;
  __syncthreads();
  int before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < JT / 64; ++w) {
    before += w < (int)(threadIdx.x >> 6) ? s_left[w] : 0;
    all += s_left[w];
  }
  if (all == 0) return;
  if (threadIdx.x == 0) s_win[0] = (int64_t)atomicAdd(total, (unsigned long long)all);
  __syncthreads();
  const int64_t p0 = s_win[0] + before;
  int2 *o2 = reinterpret_cast<int2 *>(out);
  for (int k = threadIdx.x & 63; k < wcnt; k += 64)
    if (p0 + k < cap) o2[p0 + k] = wout[k];
}

static BPRun bp_run(const eipc_scene *sc, int kind, const double *xs, const double *x1s, double dhat, bool join) {
  BPRun r{};
  r.sc = sc;
  r.kind = kind;
  r.slot = kind + 2 * (x1s != nullptr);
  r.nq = kind == 0 ? sc->n_vert : sc->n_edge;
  r.ni = kind == 0 ? sc->n_face : sc->n_edge;
  r.xs = xs;
  r.x1s = x1s;
  r.h = 0.5 * dhat;
  r.nb = 1024;
  r.ent_cap = 1;
  r.qent_cap = 1;
  r.vhash = kind == 0 && join;
  return r;
}

static eipc_status bp_scratch(eipc_ctx *c, BPRun &r) {
  const int base = B_BP0 + r.slot * BP_NBUF;
  const size_t nq = (size_t)r.nq, ni = (size_t)r.ni;
  BPScratch &b = r.b;
  EIPC_TRY(ensure_t(c, (BufId)(base + 0), ni, &b.items));
  EIPC_TRY(ensure_t(c, (BufId)(base + 1), ni, &b.cnt));
  EIPC_TRY(ensure_t(c, (BufId)(base + 2), ni, &b.large));
  EIPC_TRY(ensure_t(c, (BufId)(base + 4), (size_t)r.nb, &b.bcnt));
  EIPC_TRY(ensure_t(c, (BufId)(base + 5), r.vhash ? (size_t)r.nb : 1, &b.vbcnt));
  EIPC_TRY(ensure_t(c, (BufId)(base + 6), (size_t)r.nb + 1, &b.bstart));
  EIPC_TRY(ensure_t(c, (BufId)(base + 7), (size_t)std::max<int64_t>(r.ent_cap, 1), &b.ent));
  EIPC_TRY(ensure_t(c, (BufId)(base + 8), nq, &b.qcnt));
  EIPC_TRY(ensure_t(c, (BufId)(base + 9), nq + 1, &b.qoff));
  char *small;
  EIPC_TRY(ensure_t(c, (BufId)(base + 10), 512, &small));
  b.g = (GridDev *)small;
  b.n_large = (int64_t *)(small + 64);
  b.total = (unsigned long long *)(small + 72);
  b.n_qlarge = (int64_t *)(small + 80);
  b.n_big = (int64_t *)(small + 88);
  b.n_qbig = (int64_t *)(small + 104);
  b.n_ent = (int64_t *)(small + 120);
  b.flag = (uint32_t *)(small + 136);
  b.st = (uint64_t *)(small + 160);
  static_assert(sizeof(GridDev) <= 64 && 160 + 9 * 8 * STAT_COPIES <= 512, "small scratch");
  EIPC_TRY(ensure_t(c, (BufId)(base + 11), nq, &b.qlarge));
  EIPC_TRY(ensure_t(c, (BufId)(base + 12), (size_t)std::max<int64_t>(r.qent_cap, 1), &b.qent));
  EIPC_TRY(ensure_t(c, (BufId)(base + 13), r.vhash ? nq : 1, &b.vrec));
  EIPC_TRY(ensure_t(c, (BufId)(base + 14), r.vhash ? (size_t)r.nb + 1 : 1, &b.vbstart));
  EIPC_TRY(ensure_t(c, (BufId)(base + 15), ni, &b.big));
  EIPC_TRY(ensure_t(c, (BufId)(base + 16), r.vhash ? nq : 1, &b.qbig));
  return EIPC_OK;
}

static void bp_clear(const BPRun &r, FillList &fl, bool small, bool buckets) {
  if (small) fl.add(r.b.g, 512, 0);
  if (buckets) {
    fl.add(r.b.bcnt, fill_bytes(sizeof(int32_t) * (size_t)r.nb), 0);
    if (r.vhash) fl.add(r.b.vbcnt, fill_bytes(sizeof(int32_t) * (size_t)r.nb), 0);
  }
}

// threads to an item in the launches over items and records
static int bp_side_threads(const eipc_ctx *c, const BPRun &r) {
  return grid_for((int64_t)r.ni + (r.vhash ? r.nq : 0), 256) < LT_FEW * c->num_cu ? 4 : 1;
}

static HSides bp_sides(const BPRun &r, int q) {
  const BPScratch &b = r.b;
  HSides h{};
  h.s[0] = HSide{r.ni, b.items, b.cnt, b.large, b.n_large, b.big, b.n_big, b.bcnt, b.bstart, b.ent, r.ent_cap};
  h.s[1] = HSide{r.vhash ? r.nq : 0, b.vrec,  b.qcnt,    b.qlarge, b.n_qlarge, b.qbig,
                 b.n_qbig,           b.vbcnt, b.vbstart, reinterpret_cast<Entry *>(b.qent), r.qent_cap};
  h.blocks0 = grid_for(r.ni, lt_items(q));
  return h;
}
static unsigned bp_side_blocks(const BPRun &r, int q) {
  return (unsigned)(grid_for(r.ni, lt_items(q)) + (r.vhash ? grid_for(r.nq, lt_items(q)) : 0));
}

static eipc_status bp_items(eipc_ctx *c, const BPRun &r, hipStream_t s) {
  const eipc_scene *sc = r.sc;
  const int gi = std::min(grid_for(r.ni, STAT_T), STAT_BLOCKS);
  const int gv = r.kind == 0 ? std::min(grid_for(r.nq, STAT_T), STAT_BLOCKS) : 0;
  if (r.kind == 0)
    k_items<0><<<gi + gv, STAT_T, 0, s>>>(r.ni, sc->faces, sc->n_vert, r.xs, r.x1s, r.h, sc->W_rowptr, r.vscene(),
                                          r.b.items, r.vhash ? r.b.vrec : nullptr, gi, r.b.st);
  else
    k_items<1><<<gi, STAT_T, 0, s>>>(r.ni, sc->edges, sc->n_vert, r.xs, r.x1s, r.h, sc->W_rowptr, r.vscene(),
                                     r.b.items, nullptr, gi, r.b.st);
  EIPC_HIP(c, hipGetLastError());
  return EIPC_OK;
}

static eipc_status bp_cells(eipc_ctx *c, const BPRun &r, bool count, bool hist, int64_t *n_ent, uint32_t *status,
                            hipStream_t s) {
  const int q = bp_side_threads(c, r);
  const HSides h = bp_sides(r, q);
  if (q == 4)
    k_cells<4><<<bp_side_blocks(r, 4), lt_threads(4), 0, s>>>(h, r.b.st, r.ni, c->cell_scale, r.b.g, r.nb - 1, count,
                                                              hist, n_ent, status);
  else
    k_cells<1><<<bp_side_blocks(r, 1), lt_threads(1), 0, s>>>(h, r.b.st, r.ni, c->cell_scale, r.b.g, r.nb - 1, count,
                                                              hist, n_ent, status);
  EIPC_HIP(c, hipGetLastError());
  return EIPC_OK;
}

// bucket offsets and entries from the counts
static eipc_status bp_entries(eipc_ctx *c, const BPRun &r, uint32_t *status, hipStream_t s) {
  const BPScratch &b = r.b;
  EIPC_TRY(exclusive_scan2(c, b.bcnt, r.nb, b.bstart, r.vhash ? b.vbcnt : nullptr, r.nb, b.vbstart, s));
  const int q = bp_side_threads(c, r);
  const HSides h = bp_sides(r, q);
  if (q == 4)
    k_item_fill<4><<<bp_side_blocks(r, 4), lt_threads(4), 0, s>>>(h, b.g, r.nb - 1, status);
  else
    k_item_fill<1><<<bp_side_blocks(r, 1), lt_threads(1), 0, s>>>(h, b.g, r.nb - 1, status);
  EIPC_HIP(c, hipGetLastError());
  k_big_fill<<<dim3(BIG_BLOCKS, r.vhash ? 2 : 1), 256, 0, s>>>(h, b.g, r.nb - 1, status);
  EIPC_HIP(c, hipGetLastError());
  return EIPC_OK;
}

static QueryArgs bp_query_args(const BPRun &r) {
  return QueryArgs{r.b.g,      r.nb - 1,      r.b.bstart, r.b.ent, r.ent_cap, r.b.large, r.b.n_large, r.b.items,
                   r.sc->W_rowptr, r.vscene(), nullptr,   nullptr, nullptr,   nullptr,   r.ni};
}

// queries too large to bin or hash, one wavefront each, appended
static eipc_status bp_large(eipc_ctx *c, const BPRun &r, const int32_t *list, const int64_t *n_list, int32_t *out,
                            int64_t cap, unsigned long long *total, hipStream_t s) {
  const QueryArgs qa = bp_query_args(r);
  const int g = 2 * c->num_cu, nv = r.sc->n_vert;
  if (r.kind == 0)
    k_query_lq<0, 2><<<g, QT, 0, s>>>(list, n_list, r.xs, r.x1s, nv, r.h, qa, nullptr, nullptr, nullptr, out, cap, total);
  else
    k_query_lq<1, 2><<<g, QT, 0, s>>>(list, n_list, r.xs, r.x1s, nv, r.h, qa, nullptr, nullptr, nullptr, out, cap, total);
  EIPC_HIP(c, hipGetLastError());
  return EIPC_OK;
}

// workgroups of a join over at most row_cap rows
static int join_grid(eipc_ctx *c, int64_t row_cap) {
  return (int)std::min<int64_t>(grid_for(row_cap << JSPLIT, JT), (int64_t)JWG * c->num_cu);
}

// the bucket join of a built hash, appended to out (*total counts past cap)
static eipc_status bp_join(eipc_ctx *c, const BPRun &r, int32_t *out, int64_t cap, unsigned long long *total,
                           hipStream_t s) {
  const BPScratch &b = r.b;
  ProfScope ps(c, r.kind == 0 ? K_QUERY_WRITE_PT : K_QUERY_WRITE_EE, s);
  if (r.kind == 0) {
    const JoinArgs ja{reinterpret_cast<const Entry *>(b.qent), b.vbstart + r.nb, r.qent_cap, b.vrec, b.bstart, b.ent,
                      r.ent_cap, b.items, b.large, b.n_large, r.nb - 1};
    k_join<0><<<join_grid(c, r.qent_cap), JT, 0, s>>>(ja, (int64_t)JSWG[r.kind] * c->num_cu * JT, out, cap, total);
    EIPC_HIP(c, hipGetLastError());
    return bp_large(c, r, b.qlarge, b.n_qlarge, out, cap, total, s);
  }
  const JoinArgs ja{b.ent, b.bstart + r.nb, r.ent_cap, b.items, b.bstart, b.ent, r.ent_cap, b.items, b.large,
                    b.n_large, r.nb - 1};
  k_join<1><<<join_grid(c, r.ent_cap), JT, 0, s>>>(ja, (int64_t)JSWG[r.kind] * c->num_cu * JT, out, cap, total);
  EIPC_HIP(c, hipGetLastError());
  return bp_large(c, r, b.large, b.n_large, out, cap, total, s);
}

// the other work splits (tuning): per query, per (query, cell) thread or
// wavefront.  exact: the query entries are counted and sized first
// (synchronizes), else qent_cap is the plan's.
static eipc_status bp_append_split(eipc_ctx *c, BPRun &r, bool exact, int32_t *out, int64_t cap,
                                   unsigned long long *total, uint32_t *status, hipStream_t s) {
  const int qmode = c->query_mode[r.kind], nv = r.sc->n_vert, nq = r.nq;
  const QueryArgs qa = bp_query_args(r);
  ProfScope ps(c, r.kind == 0 ? K_QUERY_WRITE_PT : K_QUERY_WRITE_EE, s);
  if (qmode == 0) {
    QueryArgs qdef = qa;  // hands queries of many cells to k_query_lq
    qdef.defer = r.b.qlarge;
    qdef.n_defer = r.b.n_qlarge;
    EIPC_TRY(launch_zero(c, r.b.n_qlarge, 8, s));  // the list is rebuilt by every attempt
    if (r.kind == 0)
      k_query_sm<0><<<grid_for(nq, QT), QT, 0, s>>>(nq, r.xs, r.x1s, nv, r.h, qdef, out, cap, total);
    else
      k_query_sm<1><<<grid_for(nq, QT), QT, 0, s>>>(nq, r.xs, r.x1s, nv, r.h, qdef, out, cap, total);
    EIPC_HIP(c, hipGetLastError());
    return bp_large(c, r, r.b.qlarge, r.b.n_qlarge, out, cap, total, s);
  }
  const int gq = grid_for(nq, 256);
  EIPC_TRY(launch_zero(c, r.b.n_qlarge, 8, s));
  if (r.kind == 0)
    k_qcells<0><<<gq, 256, 0, s>>>(nq, r.xs, r.x1s, nv, r.h, qa, r.b.qcnt, r.b.qlarge, r.b.n_qlarge);
  else
    k_qcells<1><<<gq, 256, 0, s>>>(nq, r.xs, r.x1s, nv, r.h, qa, r.b.qcnt, r.b.qlarge, r.b.n_qlarge);
  EIPC_HIP(c, hipGetLastError());
  EIPC_TRY(exclusive_scan(c, r.b.qcnt, nq, r.b.qoff, s));
  if (exact) {
    int64_t tq = 0;
    EIPC_HIP(c, hipMemcpyAsync(&tq, r.b.qoff + nq, 8, hipMemcpyDeviceToHost, s));
    EIPC_HIP(c, hipStreamSynchronize(s));
    r.qent_cap = std::max<int64_t>(tq, 1);
    EIPC_TRY(bp_scratch(c, r));
  }
  if (r.kind == 0)
    k_qlist<0><<<gq, 256, 0, s>>>(nq, r.xs, r.x1s, nv, r.h, qa, r.b.qcnt, r.b.qoff, r.b.qent, r.qent_cap, status);
  else
    k_qlist<1><<<gq, 256, 0, s>>>(nq, r.xs, r.x1s, nv, r.h, qa, r.b.qcnt, r.b.qoff, r.b.qent, r.qent_cap, status);
  EIPC_HIP(c, hipGetLastError());
  if (qmode == 2) {
    const int gw = (int)std::min<int64_t>(grid_for(r.qent_cap * 64, QT), 32 * (int64_t)c->num_cu);
    if (r.kind == 0)
      k_query_wave<0><<<gw, QT, 0, s>>>(r.b.qoff + nq, r.qent_cap, r.b.qent, r.xs, r.x1s, nv, r.h, qa, out, cap, total);
    else
      k_query_wave<1><<<gw, QT, 0, s>>>(r.b.qoff + nq, r.qent_cap, r.b.qent, r.xs, r.x1s, nv, r.h, qa, out, cap, total);
  } else {
    const int ge = (int)std::min<int64_t>(grid_for(r.qent_cap, QT), 64 * (int64_t)c->num_cu);
    if (r.kind == 0)
      k_query_ent<0><<<ge, QT, 0, s>>>(r.b.qoff + nq, r.qent_cap, r.b.qent, r.xs, r.x1s, nv, r.h, qa, out, cap, total);
    else
      k_query_ent<1><<<ge, QT, 0, s>>>(r.b.qoff + nq, r.qent_cap, r.b.qent, r.xs, r.x1s, nv, r.h, qa, out, cap, total);
  }
  EIPC_HIP(c, hipGetLastError());
  return bp_large(c, r, r.b.qlarge, r.b.n_qlarge, out, cap, total, s);
}

// ---- planned (capacities known, nothing read by the host) ----

eipc_status bp_planned_begin(eipc_ctx *c, const eipc_scene *sc, int kind, const double *xs, const double *x1s,
                             double dhat, const BPPlan &plan, BPRun &r, FillList &fl) {
  r = bp_run(sc, kind, xs, x1s, dhat, c->query_mode[kind] == 3);
  if (r.nq == 0 || r.ni == 0) return EIPC_OK;
  r.nb = plan.nb;
  r.ent_cap = plan.ent_cap;
  r.qent_cap = plan.qent_cap;
  EIPC_TRY(bp_scratch(c, r));
  bp_clear(r, fl, true, true);
  return EIPC_OK;
}

eipc_status bp_planned_run(eipc_ctx *c, BPRun &r, int32_t *out, int64_t cap, int64_t *d_total, hipStream_t s) {
  if (r.nq == 0 || r.ni == 0) return EIPC_OK;  // *d_total was cleared by the caller
  EIPC_TRY(bp_items(c, r, s));
  EIPC_TRY(bp_cells(c, r, true, true, nullptr, c->status, s));
  EIPC_TRY(bp_entries(c, r, c->status, s));
  if (c->query_mode[r.kind] == 3) return bp_join(c, r, out, cap, (unsigned long long *)d_total, s);
  return bp_append_split(c, r, false, out, cap, (unsigned long long *)d_total, c->status, s);
}

// ---- sorted lists from an appended one ----
// The join's pairs are put in order by counting: each pair takes a slot of
// its first index (k_sort_slot), the slots' items are gathered per first
// index (k_sort_gather), and each pair's place is the number of smaller
// items of its first index (the items of one are distinct).  About 10 items
// per index on the benchmark scenes, read from cache.  The two passes of the
// per-query kernels (count, then write and insertion-sort) that this
// replaces took 3.9 ms for config 2's lists.
__global__ __launch_bounds__(256) void k_sort_slot(const int2 *__restrict__ list, const unsigned long long *total,
                                                   int64_t cap, int32_t *cnt, int32_t *__restrict__ slot) {
  const int64_t n = (int64_t)*total;
  if (n > cap) return;  // the list is cut: run again with a larger one
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
    slot[i] = atomicAdd(&cnt[list[i].x], 1);
}
__global__ __launch_bounds__(256) void k_sort_gather(const int2 *__restrict__ list, const unsigned long long *total,
                                                     int64_t cap, const int64_t *__restrict__ off,
                                                     const int32_t *__restrict__ slot, int32_t *__restrict__ tmp) {
  const int64_t n = (int64_t)*total;
  if (n > cap) return;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const int2 p = list[i];
    tmp[off[p.x] + slot[i]] = p.y;
  }
}
// nothing is written when the output is too small, nor from a pass that ran
// out of hash entries (cut): its list is a part, and run again
__global__ __launch_bounds__(256) void k_sort_rank(const int2 *__restrict__ list, const unsigned long long *total,
                                                   int64_t cap, const int64_t *__restrict__ off,
                                                   const int32_t *__restrict__ tmp, const uint32_t *cut,
                                                   int2 *__restrict__ out, int64_t out_cap) {
  const int64_t n = (int64_t)*total;
  if (n > cap || n > out_cap || *cut) return;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const int2 p = list[i];
    const int64_t o0 = off[p.x], o1 = off[p.x + 1];
    int64_t rank = 0;
    int64_t j = o0;
    for (; j + 4 <= o1; j += 4)
      rank += (int)(tmp[j] < p.y) + (int)(tmp[j + 1] < p.y) + (int)(tmp[j + 2] < p.y) + (int)(tmp[j + 3] < p.y);
    for (; j < o1; ++j) rank += tmp[j] < p.y;
    out[o0 + rank] = p;
  }
}

// ---- unplanned ----

// Sized step by step with the host reading the counts: no buffer is larger
// than its content (arena mode, where a caller's reservation was made for
// that, and the tuning work splits).  Sorted lists by two per-query passes.
static eipc_status bp_exact(eipc_ctx *c, const eipc_scene *sc, int kind, const double *xs, const double *x1s,
                            double dhat, BPReq &q, hipStream_t s) {
  const bool join = !q.sort && c->query_mode[kind] == 3;
  BPRun r = bp_run(sc, kind, xs, x1s, dhat, join);
  q.n = 0;
  if (r.nq == 0 || r.ni == 0) {
    c->last_plan[r.slot] = BPPlan{1024, 1, 0, 1};
    return EIPC_OK;
  }
  BPPlan &seen = c->last_plan[r.slot];
  FillList fl;
  EIPC_TRY(bp_scratch(c, r));
  bp_clear(r, fl, true, false);
  EIPC_TRY(launch_fill(c, fl, s));
  EIPC_TRY(bp_items(c, r, s));
  EIPC_TRY(bp_cells(c, r, true, false, r.b.n_ent, r.b.flag, s));
  // the scratch header: grid, counters and entry counts
  struct alignas(8) Head {
    char b[160];
  } hd;
  EIPC_HIP(c, hipMemcpyAsync(&hd, r.b.g, sizeof(Head), hipMemcpyDeviceToHost, s));
  EIPC_HIP(c, hipStreamSynchronize(s));
  auto word = [&](const void *d) {
    int64_t v;
    std::memcpy(&v, hd.b + ((const char *)d - (const char *)r.b.g), 8);
    return v;
  };
  GridDev gh;
  std::memcpy((void *)&gh, hd.b, sizeof(gh));
  if (gh.bad) {
    EIPC_TRY(launch_zero(c, c->status, 4, s));  // reported here instead
    return set_err(c, EIPC_ERR_NONFINITE, "non-finite primitive boxes");
  }
  const int64_t n_ent = word(r.b.n_ent) + word(r.b.n_big + 1);
  r.ent_cap = std::max<int64_t>(n_ent, 1);
  r.nb = (uint32_t)hash_buckets(n_ent);
  if (r.vhash) r.qent_cap = std::max<int64_t>(word(r.b.n_ent + 1) + word(r.b.n_qbig + 1), 1);
  EIPC_TRY(bp_scratch(c, r));
  seen.nb = r.nb;
  seen.ent_cap = r.ent_cap;
  bp_clear(r, fl, false, true);
  EIPC_TRY(launch_fill(c, fl, s));
  EIPC_TRY(bp_cells(c, r, false, true, nullptr, r.b.flag, s));
  EIPC_TRY(bp_entries(c, r, r.b.flag, s));
  int64_t total = 0;
  if (!q.sort) {
    int64_t cap = q.cap;
    int32_t *out = q.out;
    if (q.grow_id >= 0) {
      cap = (int64_t)(c->buf[q.grow_id].bytes / 8);
      if (cap > 64) cap -= 16;
      EIPC_TRY(ensure_t(c, (BufId)q.grow_id, (size_t)std::max<int64_t>(2 * cap, 2), &out));
    }
    for (int attempt = 0; attempt < 2; ++attempt) {
      EIPC_TRY(launch_zero(c, r.b.total, 8, s));
      if (join)
        EIPC_TRY(bp_join(c, r, out, cap, r.b.total, s));
      else
        EIPC_TRY(bp_append_split(c, r, true, out, cap, r.b.total, r.b.flag, s));
      EIPC_HIP(c, hipMemcpyAsync(&total, r.b.total, 8, hipMemcpyDeviceToHost, s));
      EIPC_HIP(c, hipStreamSynchronize(s));
      seen.qent_cap = r.qent_cap;
      q.n = total;
      if (total <= cap) {
        if (q.grow_id >= 0) q.out = out;
        seen.cand_cap = total;
        return EIPC_OK;
      }
      if (q.grow_id < 0) return EIPC_ERR_CAPACITY;
      cap = total + total / 4 + 1024;
      EIPC_TRY(ensure_t(c, (BufId)q.grow_id, (size_t)2 * cap, &out));
    }
    return set_err(c, EIPC_ERR_CAPACITY, "candidate append did not converge");
  }
  const QueryArgs qa = bp_query_args(r);
  QueryArgs qdef = qa;  // per-query kernels hand queries of many cells to k_query_lq
  qdef.defer = r.b.qlarge;
  qdef.n_defer = r.b.n_qlarge;
  const int glq = 2 * c->num_cu, nv = sc->n_vert, nq = r.nq;
  const double h = r.h;
  const BPScratch &b = r.b;
  {
    ProfScope ps(c, kind == 0 ? K_QUERY_COUNT_PT : K_QUERY_COUNT_EE, s);
    if (kind == 0) {
      launch_query<0, 0>(nq, xs, x1s, nv, h, qdef, b.qcnt, nullptr, nullptr, 0, nullptr, c->status, s);
      k_query_lq<0, 0><<<glq, QT, 0, s>>>(b.qlarge, b.n_qlarge, xs, x1s, nv, h, qa, b.qcnt, nullptr, nullptr, nullptr,
                                          0, nullptr);
    } else {
      launch_query<1, 0>(nq, xs, x1s, nv, h, qdef, b.qcnt, nullptr, nullptr, 0, nullptr, c->status, s);
      k_query_lq<1, 0><<<glq, QT, 0, s>>>(b.qlarge, b.n_qlarge, xs, x1s, nv, h, qa, b.qcnt, nullptr, nullptr, nullptr,
                                          0, nullptr);
    }
  }
  EIPC_HIP(c, hipGetLastError());
  EIPC_TRY(exclusive_scan(c, b.qcnt, nq, b.qoff, s));
  EIPC_HIP(c, hipMemcpyAsync(&total, b.qoff + nq, 8, hipMemcpyDeviceToHost, s));
  EIPC_HIP(c, hipStreamSynchronize(s));
  q.n = total;
  seen.cand_cap = total;
  if (total > q.cap) return EIPC_ERR_CAPACITY;
  if (total == 0 || q.out == nullptr) return EIPC_OK;
  {
    int32_t *tmp;
    EIPC_TRY(ensure_t(c, B_LQTMP, (size_t)std::max<int64_t>(q.cap, 1), &tmp));
    ProfScope ps(c, kind == 0 ? K_QUERY_WRITE_PT : K_QUERY_WRITE_EE, s);
    if (kind == 0) {
      launch_query<0, 1>(nq, xs, x1s, nv, h, qdef, b.qcnt, b.qoff, q.out, q.cap, nullptr, c->status, s);
      k_query_lq<0, 1><<<glq, QT, 0, s>>>(b.qlarge, b.n_qlarge, xs, x1s, nv, h, qa, nullptr, b.qoff, tmp, nullptr,
                                          q.cap, nullptr);
    } else {
      launch_query<1, 1>(nq, xs, x1s, nv, h, qdef, b.qcnt, b.qoff, q.out, q.cap, nullptr, c->status, s);
      k_query_lq<1, 1><<<glq, QT, 0, s>>>(b.qlarge, b.n_qlarge, xs, x1s, nv, h, qa, nullptr, b.qoff, tmp, nullptr,
                                          q.cap, nullptr);
    }
    k_seg_rank<<<glq, RANK_T, 0, s>>>(b.qlarge, b.n_qlarge, b.qcnt, b.qoff, tmp, q.out, q.cap);
  }
  EIPC_HIP(c, hipGetLastError());
  return EIPC_OK;
}

// Both kinds with one synchronization: every buffer is sized from the last
// pass on this context (or the scene's size on the first), the kernels keep
// within it and count what they need, and a pass that needed more is run
// again.  Results do not depend on the sizes.  `after` enqueues what follows
// (the lists and their device counts), so that it is read back together.
eipc_status broad_phase(eipc_ctx *c, const eipc_scene *sc, const double *xs, const double *x1s, double dhat,
                        BPReq req[2], hipStream_t s, const BPAfter &after) {
  const bool exact = c->arena || (!req[0].sort && c->query_mode[0] != 3) || (!req[1].sort && c->query_mode[1] != 3);
  if (exact) {
    eipc_status out = EIPC_OK;
    for (int kind = 0; kind < 2; ++kind) {
      const eipc_status st = bp_exact(c, sc, kind, xs, x1s, dhat, req[kind], s);
      if ((st != EIPC_OK && st != EIPC_ERR_CAPACITY) || c->scratch_short) return st;
      if (st != EIPC_OK) out = st;
    }
    if (out != EIPC_OK || !after) return out;
    const int32_t *lists[2] = {req[0].out, req[1].out};
    const int64_t caps[2] = {req[0].n, req[1].n};
    const int64_t *none[2] = {nullptr, nullptr};
    Collect col;
    c->collect_base = 0;
    EIPC_TRY(after(lists, caps, none, col));
    EIPC_TRY(launch_collect(c, col, s));
    EIPC_HIP(c, hipStreamSynchronize(s));
    return EIPC_OK;
  }
  for (int attempt = 0; attempt < 8; ++attempt) {
    BPRun run[2];
    FillList fl;
    int32_t *list[2] = {nullptr, nullptr}, *slot[2] = {nullptr, nullptr}, *tmp[2] = {nullptr, nullptr},
            *cnt[2] = {nullptr, nullptr};
    int64_t cap[2] = {0, 0};
    for (int kind = 0; kind < 2; ++kind) {
      BPReq &q = req[kind];
      BPRun &r = run[kind];
      r = bp_run(sc, kind, xs, x1s, dhat, true);
      if (r.nq == 0 || r.ni == 0) continue;
      BPPlan &g = c->bp_guess[r.slot];
      // about 4 to 8 cells per item at the default cell size
      r.ent_cap = std::max<int64_t>(g.ent_cap, 8 * (int64_t)r.ni + 1024);
      r.qent_cap = r.vhash ? std::max<int64_t>(g.qent_cap, 4 * (int64_t)r.nq + 1024) : 1;
      r.nb = (uint32_t)hash_buckets(8 * (int64_t)r.ni);
      cap[kind] = std::max<int64_t>(g.cand_cap, 4 * (int64_t)r.nq + 4096);
      EIPC_TRY(bp_scratch(c, r));
      bp_clear(r, fl, true, true);
      if (q.sort) {
        EIPC_TRY(ensure_t(c, B_SORT_LIST, (size_t)2 * cap[kind], &list[kind]));
        EIPC_TRY(ensure_t(c, B_SORT_SLOT, (size_t)cap[kind], &slot[kind]));
        EIPC_TRY(ensure_t(c, B_LQTMP, (size_t)cap[kind], &tmp[kind]));
        EIPC_TRY(ensure_t(c, kind == 0 ? B_SORT_CNT_PT : B_SORT_CNT_EE, (size_t)r.nq, &cnt[kind]));
        fl.add(cnt[kind], fill_bytes(sizeof(int32_t) * (size_t)r.nq), 0);
      } else {
        EIPC_TRY(ensure_t(c, (BufId)q.grow_id, (size_t)2 * cap[kind], &list[kind]));
      }
    }
    EIPC_TRY(launch_fill(c, fl, s));
    Collect col;
    for (int kind = 0; kind < 2; ++kind) {
      BPReq &q = req[kind];
      BPRun &r = run[kind];
      if (r.nq == 0 || r.ni == 0) continue;
      const BPScratch &b = r.b;
      EIPC_TRY(bp_items(c, r, s));
      EIPC_TRY(bp_cells(c, r, true, true, nullptr, b.flag, s));
      EIPC_TRY(bp_entries(c, r, b.flag, s));
      EIPC_TRY(bp_join(c, r, list[kind], cap[kind], b.total, s));
      if (q.sort) {
        ProfScope ps(c, kind == 0 ? K_QUERY_COUNT_PT : K_QUERY_COUNT_EE, s);
        const int g = (int)std::min<int64_t>(grid_for(cap[kind], 256), 16 * (int64_t)c->num_cu);
        const int2 *l2 = (const int2 *)list[kind];
        k_sort_slot<<<g, 256, 0, s>>>(l2, b.total, cap[kind], cnt[kind], slot[kind]);
        EIPC_HIP(c, hipGetLastError());
        EIPC_TRY(exclusive_scan(c, cnt[kind], r.nq, b.qoff, s));
        k_sort_gather<<<g, 256, 0, s>>>(l2, b.total, cap[kind], b.qoff, slot[kind], tmp[kind]);
        EIPC_HIP(c, hipGetLastError());
        k_sort_rank<<<g, 256, 0, s>>>(l2, b.total, cap[kind], b.qoff, tmp[kind], b.flag, (int2 *)q.out,
                                      q.out ? q.cap : 0);
        EIPC_HIP(c, hipGetLastError());
      }
      col.add(&b.g->bad, 4);
      col.add(b.total, 8);
      col.add(b.bstart + r.nb, 8);
      col.add(r.vhash ? b.vbstart + r.nb : b.bstart, 8);
    }
    const int head = col.n;
    if (after) {
      const int32_t *lists[2] = {list[0], list[1]};
      const int64_t *d_n[2] = {(const int64_t *)run[0].b.total, (const int64_t *)run[1].b.total};
      EIPC_TRY(after(lists, cap, d_n, col));
    }
    EIPC_TRY(launch_collect(c, col, s));
    EIPC_HIP(c, hipStreamSynchronize(s));
    bool again = false, full = false;
    int at = 0;
    for (int kind = 0; kind < 2; ++kind) {
      BPReq &q = req[kind];
      BPRun &r = run[kind];
      q.n = 0;
      if (r.nq == 0 || r.ni == 0) {
        c->last_plan[r.slot] = BPPlan{1024, 1, 0, 1};
        continue;
      }
      const int64_t *w = c->host_res + at;
      at += 4;
      if (w[0]) {
        EIPC_TRY(launch_zero(c, c->status, 4, s));  // reported here instead
        return set_err(c, EIPC_ERR_NONFINITE, "non-finite primitive boxes");
      }
      const int64_t total = w[1], ent = std::max<int64_t>(w[2], 1), qent = r.vhash ? std::max<int64_t>(w[3], 1) : 1;
      BPPlan &g = c->bp_guess[r.slot];
      const bool cut = ent > r.ent_cap || qent > r.qent_cap;
      if (ent > r.ent_cap) g.ent_cap = ent + ent / 4 + 1024;
      if (qent > r.qent_cap) g.qent_cap = qent + qent / 4 + 1024;
      if (total > cap[kind]) g.cand_cap = total + total / 4 + 1024;
      again = again || cut || total > cap[kind];
      q.n = total;
      c->last_plan[r.slot] = BPPlan{(uint32_t)hash_buckets(ent), ent, total, qent};
      if (!q.sort)
        q.out = list[kind];
      else if (total > q.cap)
        full = true;
    }
    if (again) continue;
    c->collect_base = head;
    return full ? EIPC_ERR_CAPACITY : EIPC_OK;
  }
  return set_err(c, EIPC_ERR_CAPACITY, "candidate append did not converge");
}

// ---------------------------------------------------------------------------
// narrow phase: distance type and d^2 per candidate; active (0 < d < dhat)
// pairs compacted by wavefront ballots into a workgroup stage in LDS and
// appended with one atomic per stage flush.
// ---------------------------------------------------------------------------
template <int KIND>
__device__ __forceinline__ void pair_vids(const int32_t *pairs, int64_t k, const int32_t *faces,
                                          const int32_t *edges, int *vid) {
  const int a = pairs[2 * k], b = pairs[2 * k + 1];
  if (KIND == 0) {
    vid[0] = a;
    vid[1] = faces[3 * (int64_t)b];
    vid[2] = faces[3 * (int64_t)b + 1];
    vid[3] = faces[3 * (int64_t)b + 2];
  } else {
    vid[0] = edges[2 * (int64_t)a];
    vid[1] = edges[2 * (int64_t)a + 1];
    vid[2] = edges[2 * (int64_t)b];
    vid[3] = edges[2 * (int64_t)b + 1];
  }
}

constexpr int NARROW_BUF = 1024;  // staged active pairs per workgroup (256 threads)

template <int KIND, bool FILTER>
__global__ void k_narrow(int64_t cap, const int64_t *d_n, const int32_t *__restrict__ pairs,
                         const int32_t *__restrict__ faces, const int32_t *__restrict__ edges,
                         const double *__restrict__ xs, int n_vert, double dhat2, double h,
                         int32_t *__restrict__ act, int32_t *__restrict__ typ, int64_t act_cap, int64_t *count,
                         int64_t *cand_count, uint32_t *status) {
  // active pairs staged in LDS and appended with one atomic per workgroup
  // flush (one atomic per wavefront on the shared counter serialises)
  __shared__ int2 s_act[NARROW_BUF];
  __shared__ int s_nact;
  __shared__ int64_t s_abase;
  const int64_t n = d_n ? (*d_n < cap ? *d_n : cap) : cap;
  // a planned list that was cut
  if (d_n && *d_n > cap && blockIdx.x == 0 && threadIdx.x == 0) atomicOr(status, ST_PLAN_OVERFLOW);
  const int lane = threadIdx.x & 63;
  int64_t n_cand = 0;
  if (threadIdx.x == 0) s_nact = 0;
  __syncthreads();
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t base = (int64_t)blockIdx.x * blockDim.x; base < n; base += stride) {
    const int64_t i = base + threadIdx.x;
    bool active = false;
    int ty = 0;
    if (i < n) {
      int vid[4];
      pair_vids<KIND>(pairs, i, faces, edges, vid);
      V3 x[4];
#pragma unroll
      for (int a = 0; a < 4; ++a) ld_pos(xs, vid[a], x[a].x, x[a].y, x[a].z);
      const bool cand = !FILTER || static_boxes_overlap<KIND>(x, h);
      if (cand) {
        ++n_cand;
        double s2 = pair_dist2<KIND>(x, &ty);
        if (!isfinite(s2)) {
          atomicOr(status, ST_NONFINITE);
        } else if (s2 < dhat2) {
          if (s2 <= 0.0)
            atomicOr(status, ST_INTERSECTING);
          else
            active = true;
        }
      }
    }
    const uint64_t mask = __ballot(active);
    int p0 = 0;
    if (lane == 0 && mask) p0 = atomicAdd(&s_nact, (int)__popcll(mask));
    p0 = __shfl(p0, 0, 64);
    if (active) s_act[p0 + __popcll(mask & ((1ull << lane) - 1ull))] = make_int2((int)i, ty);
    __syncthreads();
    const int na = s_nact;
    __syncthreads();  // every thread has read the count before it changes
    // flush when another round could overfill the stage, and at the end
    if (na > NARROW_BUF - (int)blockDim.x || base + stride >= n) {
      if (threadIdx.x == 0) s_abase = na ? (int64_t)atomicAdd((unsigned long long *)count, (unsigned long long)na) : 0;
      __syncthreads();
      const int64_t ab = s_abase;
      for (int k = threadIdx.x; k < na; k += blockDim.x) {
        const int64_t pos = ab + k;
        if (pos < act_cap) {
          act[pos] = s_act[k].x;
          typ[pos] = s_act[k].y;
        } else {
          atomicOr(status, ST_PLAN_OVERFLOW);
        }
      }
      __syncthreads();
      if (threadIdx.x == 0) s_nact = 0;
      __syncthreads();
    }
  }
  if (FILTER) {
    // the candidate count: one atomic per workgroup
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) n_cand += __shfl_xor(n_cand, o, 64);
    __shared__ int64_t s_cand[4];
    if (lane == 0) s_cand[threadIdx.x >> 6] = n_cand;
    __syncthreads();
    if (threadIdx.x == 0) {
      const int64_t tot = s_cand[0] + s_cand[1] + s_cand[2] + s_cand[3];
      if (tot) atomicAdd((unsigned long long *)cand_count, (unsigned long long)tot);
    }
  }
}

eipc_status launch_narrow(eipc_ctx *c, const eipc_scene *sc, int kind, const double *xs, const int32_t *pairs,
                          int64_t n, double dhat, int32_t *act, int32_t *typ, int64_t *d_count, hipStream_t s,
                          const int64_t *d_n, int64_t act_cap, int64_t *cand_count) {
  // a planned list without room is looked at too: its count may have passed it
  if (n == 0 && !d_n) return EIPC_OK;
  const double d2 = dhat * dhat;
  const double h = 0.5 * dhat;
  if (act_cap < 0) act_cap = n;
  const int blocks = (int)std::min<int64_t>(grid_for(n, 256), (int64_t)c->wg_per_cu[2] * c->num_cu);
  ProfScope ps(c, kind == 0 ? K_NARROW_PT : K_NARROW_EE, s);
  if (cand_count) {
    if (kind == 0)
      k_narrow<0, true><<<blocks, 256, 0, s>>>(n, d_n, pairs, sc->faces, sc->edges, xs, sc->n_vert, d2, h, act, typ,
                                               act_cap, d_count, cand_count, c->status);
    else
      k_narrow<1, true><<<blocks, 256, 0, s>>>(n, d_n, pairs, sc->faces, sc->edges, xs, sc->n_vert, d2, h, act, typ,
                                               act_cap, d_count, cand_count, c->status);
  } else {
    if (kind == 0)
      k_narrow<0, false><<<blocks, 256, 0, s>>>(n, d_n, pairs, sc->faces, sc->edges, xs, sc->n_vert, d2, h, act,
                                                typ, act_cap, d_count, nullptr, c->status);
    else
      k_narrow<1, false><<<blocks, 256, 0, s>>>(n, d_n, pairs, sc->faces, sc->edges, xs, sc->n_vert, d2, h, act,
                                                typ, act_cap, d_count, nullptr, c->status);
  }
  EIPC_HIP(c, hipGetLastError());
  return EIPC_OK;
}

}  // namespace eipc
