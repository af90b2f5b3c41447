// Per-pair barrier energy, gradient and (projected) Hessian, reduced through
// the embedding (Eq. 17) with LDS-staged accumulation; Hessian-vector
// products; BSR compaction of the reduced Hessian.
#include <algorithm>

#include "common.h"
#include "pair_math.h"

namespace eipc {

typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int BR_THREADS = 256;
constexpr int LGT = 512;    // LDS node-vector table entries (14 KiB)
constexpr int MAX_PROBE = 32;       // LDS tables (a miss falls back to the global table)
constexpr int GLOBAL_PROBE = 4096;  // global block table (at most half full; a miss is reported)

__device__ __forceinline__ uint32_t mix32(uint32_t k) {
  k ^= k >> 16;
  k *= 0x7feb352dU;
  k ^= k >> 15;
  k *= 0x846ca68bU;
  k ^= k >> 16;
  return k;
}

__device__ __forceinline__ uint32_t mix64(uint64_t k) {
  k ^= k >> 33;
  k *= 0xff51afd7ed558ccdULL;
  k ^= k >> 33;
  return (uint32_t)k;
}

// find-or-insert in an open-addressing table of 64-bit keys (-1 = empty)
__device__ __forceinline__ int64_t table_slot64(long long *keys, uint64_t mask, long long key, int max_probe) {
  uint64_t h = mix64((uint64_t)key) & mask;
  for (int p = 0; p < max_probe; ++p) {
    long long k = __hip_atomic_load(&keys[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (k == key) return (int64_t)h;
    if (k == -1) {
      long long old = (long long)atomicCAS((unsigned long long *)&keys[h], (unsigned long long)-1ll,
                                           (unsigned long long)key);
      if (old == -1 || old == key) return (int64_t)h;
    }
    h = (h + 1) & mask;
  }
  return -1;
}

// find-or-insert of key in an LDS open-addressing table of `size` entries
// (all bits set = empty): linear probing from a multiplicative range
// reduction of the key's hash.  All lanes of the wavefront call, `valid`
// marking the lanes that look up; a lane that finds no slot within
// MAX_PROBE probes gets -1.  fresh: this lane inserted the key.
template <typename K>
__device__ __forceinline__ int lds_slot(K *keys, int size, K key, bool valid, bool &fresh) {
  const uint32_t hv = sizeof(K) == 8 ? mix64((uint64_t)key) : mix32((uint32_t)key);
  int h = (int)(((uint64_t)hv * (uint32_t)size) >> 32);
  int slot = -1;
  fresh = false;
  bool pending = valid;
  for (int p = 0; p < MAX_PROBE; ++p) {
    if (!__any(pending)) break;
    if (pending) {
      K k = __hip_atomic_load(&keys[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (k == (K)~(K)0) {
        k = atomicCAS(&keys[h], (K)~(K)0, key);
        if (k == (K)~(K)0) {
          fresh = true;
          k = key;
        }
      }
      if (k == key) {
        slot = h;
        pending = false;
      } else {
        h = h + 1 == size ? 0 : h + 1;
      }
    }
  }
  return slot;
}

template <int KIND>
__device__ __forceinline__ void pair_vertices(const int32_t *pairs, int64_t k, const int32_t *faces,
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

__device__ __forceinline__ V3 load3(const double *xs, int n, int v) {
  V3 r;
  ld_pos(xs, v, r.x, r.y, r.z);
  return r;
}

// A workgroup's LDS table of node 3-vectors keyed by node.
struct LdsTables {
  uint32_t *gkey;
  double *gval;
};

// ---------------------------------------------------------------------------
// A pair's merged node set in one lane (the Hessian-vector product).  The
// 16 (node, weight) slots of a pair (4 vertices x up to 4 weights) are
// taken to the Q basis, z_s = w_s Q[a(s)] (3 numbers), sorted by node with
// a bitonic network, equal nodes merged, and sorted again to compact.
// ---------------------------------------------------------------------------
constexpr int NO_NODE = 0x7fffffff;

struct NodeSet {
  int node[16];
  double z[16][3];
};

__device__ __forceinline__ void cswap(NodeSet &S, int a, int b, bool up) {
  const bool sw = up ? (S.node[a] > S.node[b]) : (S.node[a] < S.node[b]);
  const int na = S.node[a], nb = S.node[b];
  S.node[a] = sw ? nb : na;
  S.node[b] = sw ? na : nb;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const double za = S.z[a][c], zb = S.z[b][c];
    S.z[a][c] = sw ? zb : za;
    S.z[b][c] = sw ? za : zb;
  }
}

__device__ __forceinline__ void sort16(NodeSet &S) {
#pragma unroll
  for (int k = 2; k <= 16; k <<= 1)
#pragma unroll
    for (int j = k >> 1; j > 0; j >>= 1)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int l = i ^ j;
        if (l > i) cswap(S, i, l, (i & k) == 0);
      }
}

// Rows hold at most 4 weights (checked when positions are embedded).
template <int KIND>
__device__ __forceinline__ bool gather_nodes(const int *vid, const int32_t *rowptr, const int32_t *col,
                                             const double *val, NodeSet &S, int &m) {
  bool ok = true;
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const int k0 = rowptr[vid[a]];
    const int cnt = rowptr[vid[a] + 1] - k0;
    ok = ok && cnt <= 4;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const bool v = k < cnt;
      const double w = v ? val[k0 + k] : 0.0;
      S.node[4 * a + k] = v ? col[k0 + k] : NO_NODE;
#pragma unroll
      for (int al = 0; al < 3; ++al) S.z[4 * a + k][al] = 0.5 * kS[a][al] * w;
    }
  }
  sort16(S);
#pragma unroll
  for (int s = 0; s < 15; ++s) {
    if (S.node[s] == S.node[s + 1] && S.node[s] != NO_NODE) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        S.z[s + 1][c] += S.z[s][c];
        S.z[s][c] = 0.0;
      }
      S.node[s] = NO_NODE;
    }
  }
  sort16(S);
  m = 0;
#pragma unroll
  for (int s = 0; s < 16; ++s) m += S.node[s] != NO_NODE;
  return ok;
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

struct Acc {
  LdsTables T;
  HessOut h;
  int n_node;
  double *grad;
  uint32_t *status;
};

// Add a lane's node 3-vector into the LDS node table (all lanes of the
// wavefront call): summed across the wavefront first when every valid lane
// holds the same node; a table miss goes to the output directly.
__device__ __forceinline__ void agg_vec(const Acc &A, bool valid, int node, double g0, double g1, double g2) {
  const uint64_t vm = __ballot(valid);
  if (vm == 0) return;
  const int first = __ffsll((unsigned long long)vm) - 1;
  const int k0 = __shfl(node, first, 64);
  bool ins = valid;
  if (__ballot(valid && node != k0) == 0) {
    g0 = wave_sum(valid ? g0 : 0.0);
    g1 = wave_sum(valid ? g1 : 0.0);
    g2 = wave_sum(valid ? g2 : 0.0);
    ins = (int)(threadIdx.x & 63) == first;
  }
  bool fresh;
  const int slot = lds_slot<uint32_t>(A.T.gkey, LGT, (uint32_t)node, ins, fresh);
  if (!ins) return;
  if (slot < 0) {
    atomicAdd(&A.grad[3 * (int64_t)node], g0);
    atomicAdd(&A.grad[3 * (int64_t)node + 1], g1);
    atomicAdd(&A.grad[3 * (int64_t)node + 2], g2);
    return;
  }
  atomicAdd(&A.T.gval[3 * slot], g0);
  atomicAdd(&A.T.gval[3 * slot + 1], g1);
  atomicAdd(&A.T.gval[3 * slot + 2], g2);
}

// Add a per-lane value into out[scene] (all lanes of the wavefront call):
// one atomic per wavefront when the contributing lanes share a scene.
__device__ __forceinline__ void agg_scene_add(double *out, bool valid, int scene, int n_scene, double v,
                                              uint32_t *status) {
  const bool ok = valid && (unsigned)scene < (unsigned)n_scene;
  if (valid && !ok) atomicOr(status, ST_BAD_SCENE);
  const uint64_t vm = __ballot(ok);
  if (vm == 0) return;
  const int first = __ffsll((unsigned long long)vm) - 1;
  const int s0 = __shfl(scene, first, 64);
  if (__ballot(ok && scene != s0) == 0) {
    const double t = wave_sum(ok ? v : 0.0);
    if ((int)(threadIdx.x & 63) == first && t != 0.0) atomicAdd(&out[s0], t);
  } else if (ok && v != 0.0) {
    atomicAdd(&out[scene], v);
  }
}

// ---------------------------------------------------------------------------
// Reduction through W (Eq. 17) of per-pair term records (gamma, X in the Q
// basis; TERM_REC doubles per pair).
//
// A contraction on the FP64 matrix cores.  With z_I = sum_{slots of node I}
// w Q[a] (3 numbers per node and pair) a pair adds
//   B(I, J)[r][c] += sum_{alpha, beta} z_I[alpha] X[3 alpha + r][3 beta + c] z_J[beta]
// to the 3x3 block of its nodes I and J.  Pairs come in locality order: a run
// of tens of them touches 16 nodes or fewer (on the grasp 19 point-triangle
// or 35 edge pairs, on average, before a table is put out).
// A wavefront keeps a table of up to 16 nodes and, for each of the six (r, c)
// with r <= c, the 16 x 16 matrix over (I, J) in four registers per lane;
// four pairs are one product with K = (pair, alpha) = 12:
//   C_rc += Z^T T_rc,  T_rc[(pair, alpha)][J] = sum_beta X z_J[beta],
// three v_mfma_f64_16x16x4 for each (r, c) and three for the gradient.  Only
// when a pair's nodes no longer fit the table do its blocks leave the
// registers, for the workgroup's LDS accumulator.
// The accumulator: nodes, not blocks, are looked up; a node's local index is
// its slot in a small open-addressing table of LN slots (installed by
// compare-and-swap), and the blocks of local nodes a <= b live in a dense
// packed upper triangle of LN x LN 3x3 FP64 blocks addressed arithmetically,
// the gradient in LN 3-vectors.  A node that finds no slot (the table is
// full) goes straight to the outputs.  Between steps the accumulator is
// flushed into the outputs once it holds more than LN / 2 nodes (each
// touched block once).
// What bounds it, 352,809 edge pairs of the grasp (276 us; the shares were
// counted in a build that took 310: 92,789 products, 10,101 tables put out;
// 2,048 wavefronts at a time): 35% of a wavefront's time in the products (21
// instructions of 64 cycles each, shared by two wavefronts), 20% in waits for
// records and rows of W, 15% at the barriers of unequal runs, 8% in finding
// slots, 6% in putting tables out.  The
// earlier form, one block per lane and 9 LDS atomics per block and pair (41
// blocks a pair), was bound by those atomics at 37 cycles per wavefront
// instruction: 405 us.
// ---------------------------------------------------------------------------
constexpr int EX_T = 512;                // eight wavefronts, two per SIMD
constexpr int EX_W = EX_T / 64;
constexpr int EX_PB = 4;                 // pairs per product
constexpr int EX_STEP = EX_W * 128;      // pairs per step
constexpr int EX_NS = 16;                // nodes of a wavefront's table
constexpr int LN = 56;                   // local node slots
constexpr int LNB = LN * (LN + 1) / 2;   // their upper 3x3 blocks (112 KiB)
constexpr int LN_PROBE = 16;
// Records and weights below these go into the products: x w w and its sums
// over a product's 16 x 12 terms then stay in range.  A pair with a larger
// one, or one that is not finite, is taken alone: in a product its infinite
// or undefined sums would reach nodes that it does not have (0 x Inf).
constexpr double EX_MAX_REC = 1e150, EX_MAX_W = 1e75;

struct LocalAcc {
  int *nkey;               // LN: node of the slot, -1 = empty
  double *bval;            // LNB * 9 (rows of the lower slot)
  unsigned char *touched;  // LNB
  double *gval;            // LN * 3
  int *count;              // nodes installed
};

__device__ __forceinline__ int ltri(int a, int b) { return a * LN - (a * (a - 1)) / 2 + (b - a); }  // a <= b

// local slot of node (all lanes of the wavefront call; valid marks the
// lookups); -1 when none is found within LN_PROBE probes
__device__ __forceinline__ int local_index(const LocalAcc &L, int node, bool valid) {
  int h = (int)(((uint64_t)mix32((uint32_t)node) * (uint32_t)LN) >> 32);
  int li = -1;
  bool pending = valid;
  for (int p = 0; p < LN_PROBE; ++p) {
    if (!__any(pending)) break;
    if (pending) {
      int k = __hip_atomic_load(&L.nkey[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (k == -1) {
        k = atomicCAS(&L.nkey[h], -1, node);
        if (k == -1) {
          atomicAdd(L.count, 1);
          k = node;
        }
      }
      if (k == node) {
        li = h;
        pending = false;
      } else {
        h = h + 1 == LN ? 0 : h + 1;
      }
    }
  }
  return li;
}

template <bool HESS>
__device__ __forceinline__ void local_init(const LocalAcc &L) {
  for (int t = threadIdx.x; t < LN; t += blockDim.x) L.nkey[t] = -1;
  if (HESS) {
    for (int t = threadIdx.x; t < LNB * 9; t += blockDim.x) L.bval[t] = 0.0;
    for (int t = threadIdx.x; t < LNB; t += blockDim.x) L.touched[t] = 0;
  }
  for (int t = threadIdx.x; t < LN * 3; t += blockDim.x) L.gval[t] = 0.0;
  if (threadIdx.x == 0) *L.count = 0;
}

// What a flush keeps in LDS meanwhile (in the wavefronts' staging, free
// between barriers): the touched blocks and where they go.
struct FlushList {
  int64_t dst[LNB];   // kind 2: table slot; kind 1: I * n_node + J
  uint16_t blk[LNB];  // local block | 0x8000: stored transposed to its rows
  int n;
};

// All threads of the workgroup call (between barriers).  First the touched
// blocks' global slots (table reads; a read issued after adds would wait for
// all of them), then the adds with consecutive lanes on consecutive entries
// of a block: the memory takes a wavefront's adds by the line, so that a
// block's nine adds are two requests and not nine.
__device__ __forceinline__ void flush_blocks(const LocalAcc &L, const HessOut &h, int n_node, uint32_t *status,
                                             FlushList &F) {
  if (threadIdx.x == 0) F.n = 0;
  __syncthreads();
  for (int idx = threadIdx.x; idx < LNB; idx += blockDim.x) {
    if (!L.touched[idx]) continue;
    // row a of the packed triangle: start(a) = a (2 LN - a + 1) / 2 <= idx
    int a = (int)((2.0 * LN + 1.0 - sqrt((2.0 * LN + 1.0) * (2.0 * LN + 1.0) - 8.0 * idx)) * 0.5);
    if (a < 0) a = 0;
    while (a + 1 < LN && ltri(a + 1, a + 1) <= idx) ++a;
    while (a > 0 && ltri(a, a) > idx) --a;
    const int b = a + (idx - ltri(a, a));
    const int na = L.nkey[a], nb = L.nkey[b];
    const bool tr = na > nb;
    const int64_t I = tr ? nb : na, J = tr ? na : nb;
    int64_t dst = -1;
    if (h.kind == 1) {
      dst = I * n_node + J;
    } else if (h.kind == 2) {
      dst = table_slot64((long long *)h.hkey, h.hmask, (long long)(I * n_node + J), GLOBAL_PROBE);
      if (dst < 0) atomicOr(status, ST_HASH_OVERFLOW);
    }
    L.touched[idx] = 0;
    if (dst < 0) {
#pragma unroll
      for (int t = 0; t < 9; ++t) L.bval[9 * idx + t] = 0.0;
      continue;
    }
    const int k = atomicAdd(&F.n, 1);
    F.dst[k] = dst;
    F.blk[k] = (uint16_t)(idx | (tr ? 0x8000 : 0));
  }
  __syncthreads();
  const int ne = 9 * F.n;
  for (int i = threadIdx.x; i < ne; i += blockDim.x) {
    const int k = i / 9, e = i - 9 * k;
    const int blk = F.blk[k], idx = blk & 0x7fff;
    const int r = e / 3, c = e - 3 * r;
    const int64_t dst = F.dst[k];
    double *v = &L.bval[9 * idx + ((blk & 0x8000) ? 3 * c + r : e)];
    if (h.kind == 1) {
      const int64_t n3 = 3 * (int64_t)n_node, I = dst / n_node, J = dst % n_node;
      atomicAdd(&h.dense[(3 * I + r) * n3 + 3 * J + c], *v);
    } else {
      atomicAdd(&h.hval[9 * dst + e], *v);
    }
    *v = 0.0;
  }
}

// the gradient, and the accumulator empty again
__device__ __forceinline__ void flush_nodes(const LocalAcc &L, double *grad) {
  for (int i = threadIdx.x; i < 3 * LN; i += blockDim.x) {
    const int node = L.nkey[i / 3];
    if (node >= 0 && grad) atomicAdd(&grad[3 * (int64_t)node + i % 3], L.gval[i]);
    L.gval[i] = 0.0;
  }
  __syncthreads();  // nkey is read above and reset below
  for (int li = threadIdx.x; li < LN; li += blockDim.x) L.nkey[li] = -1;
  if (threadIdx.x == 0) *L.count = 0;
}

// A wavefront's staging of one product's pairs.
struct ExStage {
  double x[EX_PB][54];          // [alpha][(r, c)][beta]
  double g[EX_PB][9];           // gamma
  double w[EX_PB][EX_NS][4];    // weight of (table slot, vertex)
};

// (r, c) of the six products, r <= c
__device__ __forceinline__ constexpr int ex_r(int k) { return k < 3 ? 0 : (k < 5 ? 1 : 2); }
__device__ __forceinline__ constexpr int ex_c(int k) { return k < 3 ? k : (k < 5 ? k - 2 : 2); }

// The wavefront's products into the workgroup's accumulator.  Lane (I = 4 e
// + lane / 16, J = lane % 16) holds B(I, J)[r][c] for r <= c, which is also
// B(J, I)[c][r]: of a stored block the lane whose row comes first adds the
// six entries r <= c and the other the three below the diagonal.
template <bool HESS>
__device__ __forceinline__ void expand_out(const LocalAcc &L, const HessOut &h, int n_node, double *grad,
                                           uint32_t *status, int tab, int cnt, uint32_t touched, const v4d *acc,
                                           v4d accg, bool want_g) {
  const int lane = threadIdx.x & 63, J = lane & 15;
  const int li = local_index(L, tab, lane < cnt);  // lanes 0 .. 15
  const int nJ = __shfl(tab, J, 64), lJ = __shfl(li, J, 64);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int I = 4 * e + (lane >> 4);
    const int nI = __shfl(tab, I, 64), lI = __shfl(li, I, 64);
    const uint32_t tI = (uint32_t)__shfl((int)touched, I, 64);
    if (want_g && I < cnt && J < 3) {
      if (lI >= 0)
        atomicAdd(&L.gval[3 * lI + J], accg[e]);
      else
        atomicAdd(&grad[3 * (int64_t)nI + J], accg[e]);
    }
    if (!HESS || !((tI >> J) & 1u)) continue;
    const bool both = lI >= 0 && lJ >= 0;
    const bool up = both ? lI <= lJ : nI <= nJ, low = both ? lI >= lJ : nI >= nJ;  // both on the diagonal
    if (both) {
      const int slot = lI <= lJ ? ltri(lI, lJ) : ltri(lJ, lI);
      double *B = L.bval + 9 * slot;
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        const int r = ex_r(k), c = ex_c(k);
        if (up) atomicAdd(&B[3 * r + c], acc[k][e]);
        if (low && r < c) atomicAdd(&B[3 * c + r], acc[k][e]);
      }
      L.touched[slot] = 1;
    } else {
      const int64_t R = up ? nI : nJ, C = up ? nJ : nI;
      double *B;
      int64_t ld = 3;
      if (h.kind == 1) {
        ld = 3 * (int64_t)n_node;
        B = h.dense + 3 * R * ld + 3 * C;
      } else {
        const int64_t slot = table_slot64((long long *)h.hkey, h.hmask, (long long)(R * n_node + C), GLOBAL_PROBE);
        if (slot < 0) {
          atomicOr(status, ST_HASH_OVERFLOW);
          continue;
        }
        B = h.hval + 9 * slot;
      }
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        const int r = ex_r(k), c = ex_c(k);
        if (up) atomicAdd(&B[r * ld + c], acc[k][e]);
        if (low && r < c) atomicAdd(&B[c * ld + r], acc[k][e]);
      }
    }
  }
}

// A pair that does not go into a product, straight to the outputs and entry
// by entry.  The pair's 16 entries of W are nd and wv of 16 lanes from l0.
template <bool HESS>
__device__ __forceinline__ void expand_alone(const double *R, int nd, double wv, int l0, const HessOut &h, int n_node,
                                             double *grad, uint32_t *status, bool want_g) {
  const int lane = threadIdx.x & 63;
  // Q = S / 2 with the Hadamard signs
  auto Q = [](int a, int k) { return ((k != 1 && a >= 2) != (k != 0 && (a & 1))) ? -0.5 : 0.5; };
  if (want_g && lane >= l0 && lane < l0 + 16 && nd >= 0) {
    const int a = (lane & 15) >> 2;
#pragma unroll 1
    for (int r = 0; r < 3; ++r)
      atomicAdd(&grad[3 * (int64_t)nd + r], wv * (Q(a, 0) * R[r] + Q(a, 1) * R[3 + r] + Q(a, 2) * R[6 + r]));
  }
  if (!HESS) return;
#pragma unroll 1
  for (int t = lane; t < 256; t += 64) {
    const int p = t >> 4, q = t & 15;
    const int64_t I = __shfl(nd, l0 + p, 64), J = __shfl(nd, l0 + q, 64);
    const double wp = __shfl(wv, l0 + p, 64), wq = __shfl(wv, l0 + q, 64);
    if (I < 0 || J < 0 || I > J) continue;
    double *B;
    int64_t ld = 3;
    if (h.kind == 1) {
      ld = 3 * (int64_t)n_node;
      B = h.dense + 3 * I * ld + 3 * J;
    } else {
      const int64_t slot = table_slot64((long long *)h.hkey, h.hmask, (long long)(I * n_node + J), GLOBAL_PROBE);
      if (slot < 0) {
        atomicOr(status, ST_HASH_OVERFLOW);
        continue;
      }
      B = h.hval + 9 * slot;
    }
#pragma unroll 1
    for (int e = 0; e < 9; ++e) {
      const int r = e / 3, c = e % 3;
      double v = 0.0;
#pragma unroll 1
      for (int k = 0; k < 9; ++k) v += Q(p >> 2, k / 3) * R[9 + pidx(3 * (k / 3) + r, 3 * (k % 3) + c)] * Q(q >> 2, k % 3);
      atomicAdd(&B[r * ld + c], wp * v * wq);
    }
  }
}

// Instantiated per pair kind (the code is the same) so that the two launches
// of a step carry their own names in kernel traces, and without the Hessian:
// then the workgroup's blocks (112 KiB of LDS, one workgroup per CU) are not
// there, and four fit (39,379 edge pairs: 56 and 33 us).
template <int KIND, bool HESS>
__global__ __launch_bounds__(EX_T) __attribute__((amdgpu_waves_per_eu(HESS ? 2 : 4, HESS ? 2 : 5))) void k_expand(
    const int4 *__restrict__ vid4, const int64_t *__restrict__ d_count, const int32_t *__restrict__ rowptr,
    const int32_t *__restrict__ col, const double *__restrict__ val, int n_node, const double *__restrict__ rec,
    int64_t cap, bool want_g, double *grad, HessOut h, uint32_t *status) {
  __shared__ int s_nkey[LN];
  __shared__ double s_bval[HESS ? LNB * 9 : 1];
  __shared__ double s_gval[LN * 3];
  __shared__ unsigned char s_touched[HESS ? LNB : 1];
  __shared__ int s_count;
  __shared__ union __align__(16) {
    ExStage stage[EX_W];
    std::conditional_t<HESS, FlushList, char> flush;
  } s_u;
  // consecutive ranges on one XCD (workgroups are dealt to the 8 XCDs in turn)
  int rid = blockIdx.x;
  if ((gridDim.x & 7) == 0) rid = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  const int64_t n = *d_count < cap ? *d_count : cap;
  const int64_t per = ((n + gridDim.x - 1) / gridDim.x + 63) / 64 * 64;
  const int64_t r0 = (int64_t)rid * per;
  const int64_t r1 = r0 + per < n ? r0 + per : n;
  if (r0 >= n) return;  // before the accumulator is cleared: most of a short list's time
  LocalAcc L{s_nkey, s_bval, s_touched, s_gval, &s_count};
  local_init<HESS>(L);
  __syncthreads();
  // the wavefront's number as a scalar: its ranges and loops are then uniform
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  ExStage &S = s_u.stage[wave];
  const int es = lane & 15, ea = es >> 2, ek = es & 3;  // this lane's (vertex, weight) of a pair
  const int lk = lane >> 4;
  // what this lane loads of a product's records: 216 entries of X in the
  // staged order and 36 of gamma, by the pair and the place in its record
  uint32_t xpr[4], xat[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int idx = lane + 64 * i < 54 * EX_PB ? lane + 64 * i : 0;
    const int e = idx % 54, al = e / 18, k = (e % 18) / 3, be = e % 3;
    const int u = 3 * al + (k < 3 ? 0 : (k < 5 ? 1 : 2)), v = 3 * be + (k < 3 ? k : (k < 5 ? k - 2 : 2));
    xpr[i] = idx / 54;
    xat[i] = 9 + pidx(u, v);
  }
  const uint32_t gpr = lane < 9 * EX_PB ? lane / 9 : 0, gat = lane % 9;
  int tab = -1, cnt = 0;     // the table: lane l holds slot l % 16; nodes in it
  uint32_t touched = 0;      // slots that share a pair with this lane's
  v4d acc[6], accg;
  auto clear = [&]() {
    tab = -1;
    cnt = 0;
    touched = 0;
#pragma unroll
    for (int k = 0; k < 6; ++k) acc[k] = v4d{0.0, 0.0, 0.0, 0.0};
    accg = v4d{0.0, 0.0, 0.0, 0.0};
  };
  clear();
  auto fence = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  for (int64_t base = r0; base < r1; base += EX_STEP) {
    // the step's pairs in equal runs over the wavefronts
    const int left = (int)(r1 - base < EX_STEP ? r1 - base : EX_STEP);
    const int run = (left + EX_W - 1) / EX_W;
    const int p0 = run * wave < left ? run * wave : left;
    const int p1 = p0 + run < left ? p0 + run : left;
    const bool last_step = base + EX_STEP >= r1;
    const int32_t *vids = reinterpret_cast<const int32_t *>(vid4 + base);
    const double *recs = rec + base * TERM_REC;
    // The vertex, its row of W and the row's entry are three dependent loads,
    // each issued one product ahead of the next.  Every load is issued by
    // every lane, at a place that is always there (a load under a condition
    // ends the block, and with it the loads in flight).
    // None of their results is touched before its product.
    int vid = 0, rk = 0, rn = 0, node = 0;
    bool has = false;
    double wt = 0.0, xr[4] = {0.0, 0.0, 0.0, 0.0}, gr = 0.0;
    auto load_vid = [&](int i) { vid = vids[4 * (uint32_t)(i + lk < p1 ? i + lk : p1 - 1) + ea]; };
    auto load_row = [&]() {
      rk = rowptr[vid];
      rn = rowptr[vid + 1];
    };
    auto load_entry = [&](int i) {
      has = i + lk < p1 && rk + ek < rn;
      const int32_t *cp = has ? col + (rk + ek) : vids;
      const double *vp = has ? val + (rk + ek) : recs;
      node = *cp;
      wt = *vp;
    };
    auto load_rec = [&](int i) {
      const uint32_t most = (uint32_t)(p1 - 1 - i);  // pairs past the run: its last one, not used
      const double *R = recs + (uint32_t)(TERM_REC * i);
      if (HESS) {
#pragma unroll
        for (int k = 0; k < 4; ++k) xr[k] = R[TERM_REC * (xpr[k] < most ? xpr[k] : most) + xat[k]];
      }
      gr = R[TERM_REC * (gpr < most ? gpr : most) + gat];
    };
    if (p0 < p1) {
      load_vid(p0);
      load_row();
      load_vid(p0 + EX_PB);
      load_entry(p0);
      load_row();
      load_vid(p0 + 2 * EX_PB);
      load_rec(p0);
    }
    int i0 = p0;           // the next product's first pair
    uint32_t pending = 0;  // its pairs that are not taken yet
    int nd = -1, slot = -1;
    double wv = 0.0;
    // one loop with one place where the table leaves the registers (code of
    // that size more than once does not fit the instruction cache)
    for (;;) {
      if (pending == 0 && i0 < p1) {
        const int np = p1 - i0 < EX_PB ? p1 - i0 : EX_PB;
        uint32_t bad = 0;  // pairs to be taken alone
        gr = want_g ? gr : 0.0;  // not written by the terms otherwise
        {
          uint32_t nf = fabs(gr) < EX_MAX_REC ? 0u : 1u << gpr;
          nf |= !has || fabs(wt) < EX_MAX_W ? 0u : 1u << lk;
          if (HESS) {
#pragma unroll
            for (int k = 0; k < 4; ++k) nf |= fabs(xr[k]) < EX_MAX_REC ? 0u : 1u << xpr[k];
          }
          if (__any(nf != 0)) {
#pragma unroll 1
            for (int j = 0; j < EX_PB; ++j) bad |= __any((nf >> j) & 1u) ? 1u << j : 0u;
            if (HESS) {
#pragma unroll
              for (int k = 0; k < 4; ++k) xr[k] = (bad >> xpr[k]) & 1u ? 0.0 : xr[k];
            }
            gr = (bad >> gpr) & 1u ? 0.0 : gr;
          }
        }
        fence();  // the previous product has read its stage
        if (HESS) {
#pragma unroll
          for (int k = 0; k < 4; ++k)
            if (lane + 64 * k < 54 * EX_PB) (&S.x[0][0])[lane + 64 * k] = xr[k];
        }
        if (lane < 9 * EX_PB) (&S.g[0][0])[lane] = gr;
        nd = has ? node : -1;
        wv = has ? wt : 0.0;
        // in registers of their own before the next loads: copied after
        // them, they would wait for them
        asm volatile("" : "+v"(nd), "+v"(wv));
        i0 += EX_PB;
        load_entry(i0);
        load_row();
        load_vid(i0 + 2 * EX_PB);
        load_rec(i0 < p1 ? i0 : p1 - 1);
        pending = (1u << np) - 1u;
        if (bad != 0) {
#pragma unroll 1
          for (uint32_t b = bad & pending; b != 0; b &= b - 1) {
            const int j = __ffs(b) - 1;
            expand_alone<HESS>(recs + (int64_t)TERM_REC * (i0 - EX_PB + j), nd, wv, 16 * j, h, n_node, grad, status,
                               want_g);
          }
          if ((bad >> lk) & 1u) nd = -1;
          pending &= ~bad;
          if (pending == 0) continue;
        }
        slot = -1;
#pragma unroll
        for (int j = 0; j < EX_NS; ++j) slot = nd == __builtin_amdgcn_readlane(tab, j) ? j : slot;
        if (nd < 0) slot = -1;
      }
      // pairs in order, as long as their nodes fit the table
      uint32_t take = pending;
      int pj = -1, c_before = 0;
      for (uint64_t mm; (mm = __ballot(nd >= 0 && slot < 0)) != 0;) {
        const int l = __builtin_ctzll(mm);
        if ((l >> 4) != pj) {
          pj = l >> 4;
          c_before = cnt;
        }
        if (cnt == EX_NS) {  // give back what this pair took
          if (es >= c_before) tab = -1;
          if (slot >= c_before) slot = -1;
          cnt = c_before;
          take &= (1u << pj) - 1u;
          break;
        }
        const int nn = __builtin_amdgcn_readlane(nd, l);
        if (es == cnt) tab = nn;
        if (nd == nn) slot = cnt;
        ++cnt;
      }
      if (take == 0) {
        // the table is full (an empty one holds any pair's 16 nodes), or the
        // run is done
        if (pending == 0 && !last_step) break;  // the next step goes on with this table
        expand_out<HESS>(L, h, n_node, grad, status, tab, cnt, touched, acc, accg, want_g);
        clear();
        slot = -1;
        if (pending == 0) break;
        continue;
      }
      pending &= ~take;
      const bool mine = nd >= 0 && ((take >> lk) & 1u);
      fence();
      {
        double2 *w2 = reinterpret_cast<double2 *>(&S.w[0][0][0]);
        w2[lane] = double2{0.0, 0.0};
        w2[lane + 64] = double2{0.0, 0.0};
      }
      fence();
      if (mine) atomicAdd(&S.w[lk][slot][ea], wv);
      fence();
      // nodes that share a pair: the pair's slots, over its 16 lanes
      int m = mine ? 1 << slot : 0;
      m |= __builtin_amdgcn_update_dpp(0, m, 0x128, 0xf, 0xf, false);  // row_ror:8
      m |= __builtin_amdgcn_update_dpp(0, m, 0x124, 0xf, 0xf, false);  // row_ror:4
      m |= __builtin_amdgcn_update_dpp(0, m, 0x122, 0xf, 0xf, false);  // row_ror:2
      m |= __builtin_amdgcn_update_dpp(0, m, 0x121, 0xf, 0xf, false);  // row_ror:1
#pragma unroll
      for (int j = 0; j < EX_PB; ++j) {
        const uint32_t mj = (uint32_t)__builtin_amdgcn_readlane(m, 16 * j);
        touched |= (mj >> es) & 1u ? mj : 0u;
      }
      if (mine) nd = -1;
#pragma unroll
      for (int st = 0; st < 3; ++st) {
        const int ka = 4 * st + lk, pr = ka / 3, al = ka - 3 * pr;
        const double *w = S.w[pr][es];
        const double w0 = w[0], w1 = w[1], w2 = w[2], w3 = w[3];
        // Q = S / 2 with the Hadamard signs
        const double z0 = 0.5 * ((w0 + w1) - (w2 + w3)), z1 = 0.5 * ((w0 - w1) + (w2 - w3)),
                     z2 = 0.5 * ((w0 - w1) - (w2 - w3));
        const double za = al == 0 ? z0 : (al == 1 ? z1 : z2);
        if (HESS) {
          const double *x = S.x[pr] + 18 * al;
          double t[6];
#pragma unroll
          for (int k = 0; k < 6; ++k) t[k] = x[3 * k] * z0 + x[3 * k + 1] * z1 + x[3 * k + 2] * z2;
#pragma unroll
          for (int k = 0; k < 6; ++k) acc[k] = __builtin_amdgcn_mfma_f64_16x16x4f64(za, t[k], acc[k], 0, 0, 0);
        }
        const double t = es < 3 ? S.g[pr][3 * al + es] : 0.0;
        accg = __builtin_amdgcn_mfma_f64_16x16x4f64(za, t, accg, 0, 0, 0);
      }
    }
    __syncthreads();
    if (last_step || s_count > LN / 2) {
      if constexpr (HESS) flush_blocks(L, h, n_node, status, s_u.flush);
      flush_nodes(L, want_g ? grad : nullptr);
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Locality order of the active pairs: a counting sort by the first coarse
// node of the pair's first vertex with a DoF, so that a workgroup's range
// of pairs touches few distinct node blocks (its LDS tables then absorb
// most of the accumulation).
// ---------------------------------------------------------------------------
// Per-lane offsets from counters ctr[key], one atomic per distinct key in
// the wavefront (lanes with equal keys are served together).  All lanes
// of the wavefront must call.
__device__ __forceinline__ int wave_key_add(int *ctr, int key, bool valid) {
  const int lane = threadIdx.x & 63;
  const uint64_t lt = (1ull << lane) - 1ull;
  // group the lanes first, then one atomic instruction for all groups (an
  // atomic inside the loop waits once per distinct key)
  int leader_of = lane, rank = 0, count = 0;
  uint64_t pending = __ballot(valid);
  while (pending) {
    const int leader = __ffsll((unsigned long long)pending) - 1;
    const int lk = __builtin_amdgcn_readlane(key, __builtin_amdgcn_readfirstlane(leader));
    const uint64_t m = __ballot(valid && key == lk) & pending;
    if ((m >> lane) & 1ull) {
      leader_of = leader;
      rank = __popcll(m & lt);
    }
    if (lane == leader) count = __popcll(m);
    pending &= ~m;
  }
  const int base = count > 0 ? atomicAdd(&ctr[key], count) : 0;
  const int res = __shfl(base, leader_of, 64) + rank;
  return res;
}

template <int KIND>
__global__ void k_pair_keys(const int32_t *__restrict__ pairs, const int32_t *__restrict__ act,
                            const int64_t *__restrict__ d_count, int64_t cap, const int32_t *__restrict__ faces,
                            const int32_t *__restrict__ edges, const int32_t *__restrict__ rowptr,
                            const int32_t *__restrict__ col, int n_node, int32_t *__restrict__ key, int32_t *hist,
                            int4 *__restrict__ vidu) {
  const int64_t n = *d_count < cap ? *d_count : cap;
  for (int64_t base = (int64_t)blockIdx.x * blockDim.x; base < n; base += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = base + threadIdx.x;
    const bool live = i < n;
    int k = 0;
    if (live) {
      int vid[4];
      pair_vertices<KIND>(pairs, act[i], faces, edges, vid);
      k = -1;
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const int r0 = rowptr[vid[a]];
        if (k < 0 && rowptr[vid[a] + 1] > r0) k = col[r0];
      }
      if ((unsigned)k >= (unsigned)n_node) k = 0;
      key[i] = k;
      vidu[i] = make_int4(vid[0], vid[1], vid[2], vid[3]);
    }
    wave_key_add(hist, k, live);
  }
}

__global__ void k_pair_scatter(const int32_t *__restrict__ act, const int32_t *__restrict__ typ,
                               const int64_t *__restrict__ d_count, int64_t cap, const int32_t *__restrict__ key,
                               const int64_t *__restrict__ start, int32_t *fill, int32_t *__restrict__ act2,
                               int32_t *__restrict__ typ2, const int4 *__restrict__ vidu, int4 *__restrict__ vid2) {
  const int64_t n = *d_count < cap ? *d_count : cap;
  for (int64_t base = (int64_t)blockIdx.x * blockDim.x; base < n; base += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = base + threadIdx.x;
    const bool live = i < n;
    const int k = live ? key[i] : 0;
    const int off = wave_key_add(fill, k, live);
    if (live) {
      const int64_t pos = start[k] + off;
      act2[pos] = act[i];
      typ2[pos] = typ[i];
      vid2[pos] = vidu[i];
    }
  }
}

// the counters of sort_active, to be cleared before it runs
eipc_status sort_clear(eipc_ctx *c, const eipc_scene *sc, int kind, FillList &fl) {
  const int nn = std::max(sc->n_node, 1);
  const size_t bytes = fill_bytes(sizeof(int32_t) * ((size_t)nn + 1));
  int32_t *hist, *fill;
  EIPC_TRY(ensure_t(c, kind ? B_SHIST_EE : B_SHIST, (size_t)nn + 1, &hist));
  EIPC_TRY(ensure_t(c, kind ? B_SFILL_EE : B_SFILL, (size_t)nn + 1, &fill));
  fl.add(hist, bytes, 0);
  fl.add(fill, bytes, 0);
  return EIPC_OK;
}

static eipc_status sort_active(eipc_ctx *c, const eipc_scene *sc, int kind, const int32_t *pairs, const int32_t *act,
                               const int32_t *typ, const int64_t *d_count, int64_t cap, const int32_t **act2,
                               const int32_t **typ2, const int4 **vid2, hipStream_t s) {
  const int nn = std::max(sc->n_node, 1);
  int32_t *key, *hist, *fill, *a2, *t2;
  int4 *vu, *v2;
  int64_t *start;
  // per kind, so that the two kinds can be sorted concurrently
  const bool e = kind != 0;
  EIPC_TRY(ensure_t(c, e ? B_SKEY_EE : B_SKEY, (size_t)cap, &key));
  EIPC_TRY(ensure_t(c, e ? B_SHIST_EE : B_SHIST, (size_t)nn + 1, &hist));
  EIPC_TRY(ensure_t(c, e ? B_SFILL_EE : B_SFILL, (size_t)nn + 1, &fill));
  EIPC_TRY(ensure_t(c, e ? B_SSTART_EE : B_SSTART, (size_t)nn + 1, &start));
  EIPC_TRY(ensure_t(c, e ? B_SACT_EE : B_SACT, (size_t)cap, &a2));
  EIPC_TRY(ensure_t(c, e ? B_STYP_EE : B_STYP, (size_t)cap, &t2));
  EIPC_TRY(ensure_t(c, e ? B_SVIDU_EE : B_SVIDU, (size_t)cap, &vu));
  EIPC_TRY(ensure_t(c, e ? B_SVID_EE : B_SVID, (size_t)cap, &v2));
  const int blocks = (int)std::min<int64_t>(grid_for(cap, 256), 8 * (int64_t)c->num_cu);
  if (kind == 0)
    k_pair_keys<0><<<blocks, 256, 0, s>>>(pairs, act, d_count, cap, sc->faces, sc->edges, sc->W_rowptr, sc->W_col,
                                          nn, key, hist, vu);
  else
    k_pair_keys<1><<<blocks, 256, 0, s>>>(pairs, act, d_count, cap, sc->faces, sc->edges, sc->W_rowptr, sc->W_col,
                                          nn, key, hist, vu);
  EIPC_HIP(c, hipGetLastError());
  EIPC_TRY(exclusive_scan(c, hist, nn, start, s));
  k_pair_scatter<<<blocks, 256, 0, s>>>(act, typ, d_count, cap, key, start, fill, a2, t2, vu, v2);
  EIPC_HIP(c, hipGetLastError());
  *act2 = a2;
  *typ2 = t2;
  if (vid2) *vid2 = v2;
  return EIPC_OK;
}

// ---------------------------------------------------------------------------
// Per active pair: the energy (Eq. 7, summed per scene), its Q-basis
// gradient and (projected) Hessian, stored as a term record in the pair's
// (locality-order) position for k_expand.
//
// A workgroup takes a contiguous range of the active pairs in tiles of up
// to TERMS_TILE pairs.  Each tile is put in order of pair class (point-point,
// point-line, interior, mollified) by a counting sort in LDS, so that the
// lanes of a wavefront nearly always share one derivative path; each
// wavefront then takes 64 pairs of the tile at a time, one per lane.
// ---------------------------------------------------------------------------
constexpr int TERMS_T = 256;      // four wavefronts, one per SIMD (the 9x9 projection's registers)
constexpr int TERMS_TILE = 2048;  // pairs per class-sorted tile

// GEN: pairs may be mollified (general 9x9 path) or take the reduced-block
// projection; without it the registers fit two wavefronts per SIMD.
template <int KIND, bool REDUCED, bool GEN>
__global__ __launch_bounds__(TERMS_T) __attribute__((amdgpu_waves_per_eu(GEN ? 1 : 2))) void k_pair_terms(
    const int32_t *__restrict__ pairs, const int32_t *__restrict__ act, const int32_t *__restrict__ typ,
    const int4 *__restrict__ vid4, const int64_t *__restrict__ d_count, int64_t cap,
    const int32_t *__restrict__ faces, const int32_t *__restrict__ edges, const double *__restrict__ xs,
    const double *__restrict__ x_rest, int n_vert, double dhat, double kappa, uint32_t flags, bool want_g,
    bool want_h, double *energy, double *__restrict__ rec, const int32_t *__restrict__ vscene, int n_scene,
    uint32_t *status, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ col,
    const double *__restrict__ val) {
  __shared__ int s_tile[TERMS_TILE];
  __shared__ int s_cnt[4];
  __shared__ double s_e[TERMS_T / 64];
  const bool expand = want_g || want_h;
  // the reduced-block projection takes the true X and projects after the transform
  const bool reduced = REDUCED && want_h;
  const bool project = (flags & EIPC_PROJECT) && !reduced;
  const bool sq = flags & EIPC_SQDIST;
  const bool moll = GEN && (KIND == 1) && (flags & EIPC_MOLLIFY) && x_rest;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  constexpr int NW = TERMS_T / 64;
  const int64_t n = *d_count < cap ? *d_count : cap;
  const int64_t per = ((n + gridDim.x - 1) / gridDim.x + 63) / 64 * 64;
  const int64_t r0 = (int64_t)blockIdx.x * per;
  const int64_t r1 = r0 + per < n ? r0 + per : n;
  double e_acc = 0.0;
  for (int64_t tb = r0; tb < r1; tb += TERMS_TILE) {
    const int tn = (int)(r1 - tb < TERMS_TILE ? r1 - tb : TERMS_TILE);
    if (threadIdx.x < 4) s_cnt[threadIdx.x] = 0;
    __syncthreads();
    // class of each pair of the tile and its rank within the class
    constexpr int PER_T = TERMS_TILE / TERMS_T;
    int cls_of[PER_T], rank_of[PER_T];
#pragma unroll
    for (int u = 0; u < PER_T; ++u) {
      const int li = u * TERMS_T + threadIdx.x;
      const bool v = li < tn;
      int cls = 0;
      if (v && expand) {
        const int64_t i = tb + li;
        const int ty = typ[i];
        if (moll) {
          int vid[4];
          if (vid4) {
            const int4 v4 = vid4[i];
            vid[0] = v4.x;
            vid[1] = v4.y;
            vid[2] = v4.z;
            vid[3] = v4.w;
          } else {
            pair_vertices<KIND>(pairs, act[i], faces, edges, vid);
          }
          V3 x[4], r[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            x[q] = load3(xs, n_vert, vid[q]);
            r[q] = V3{x_rest[3 * (int64_t)vid[q]], x_rest[3 * (int64_t)vid[q] + 1], x_rest[3 * (int64_t)vid[q] + 2]};
          }
          cls = pair_class<KIND>(ty, x, mollifier_eps(r));
        } else {
          cls = type_fn<KIND>(ty);
        }
      }
      cls_of[u] = cls;
      rank_of[u] = wave_key_add(s_cnt, cls, v);
    }
    __syncthreads();
    {
      const int c0 = s_cnt[0], c1 = s_cnt[1], c2 = s_cnt[2];
#pragma unroll
      for (int u = 0; u < PER_T; ++u) {
        const int li = u * TERMS_T + threadIdx.x;
        if (li < tn) {
          const int cls = cls_of[u];
          const int base = cls == 0 ? 0 : (cls == 1 ? c0 : (cls == 2 ? c0 + c1 : c0 + c1 + c2));
          s_tile[base + rank_of[u]] = li | (cls << 16);
        }
      }
    }
    __syncthreads();
    const int nc = (tn + 63) / 64;
    for (int ch = wave; ch < nc; ch += NW) {
      const int pos = ch * 64 + lane;
      const bool live = pos < tn;
      double e_pair = 0.0;
      int scene = 0;
      if (live) {
        const int code = s_tile[pos];
        const int64_t i = tb + (code & 0xffff);
        const int cls = code >> 16;
        const int ty = typ[i];
        int vid[4];
        if (vid4) {
          const int4 v4 = vid4[i];
          vid[0] = v4.x;
          vid[1] = v4.y;
          vid[2] = v4.z;
          vid[3] = v4.w;
        } else {
          pair_vertices<KIND>(pairs, act[i], faces, edges, vid);
        }
        if (vscene) scene = vscene[vid[0]];
        V3 x[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) x[q] = load3(xs, n_vert, vid[q]);
        double eps = 0.0;
        if (moll && (cls == CLS_GEN || !expand)) {
          V3 r[4];
#pragma unroll
          for (int q = 0; q < 4; ++q)
            r[q] = V3{x_rest[3 * (int64_t)vid[q]], x_rest[3 * (int64_t)vid[q] + 1], x_rest[3 * (int64_t)vid[q] + 2]};
          eps = mollifier_eps(r);
        }
        if (expand && !GEN) {
          // straight into the record (held in registers as a whole it takes
          // 108 of them beside the projection's)
          double *r = (double *)__builtin_assume_aligned(rec + i * TERM_REC, 16);
          e_pair = pair_qterms<KIND, GEN>(cls, ty, x, eps, dhat, kappa, want_g, want_h, project, sq, r, r + 9);
        } else if (expand) {
          double tv[54];
          e_pair = pair_qterms<KIND, GEN>(cls, ty, x, eps, dhat, kappa, want_g, want_h, project, sq, tv, tv + 9);
          if (reduced) {
            // dot products of the four vertices' rows of W
            int cc[4][4];
            double ww[4][4];
#pragma unroll
            for (int a = 0; a < 4; ++a) {
              const int k0 = rowptr[vid[a]];
              const int n = rowptr[vid[a] + 1] - k0;
#pragma unroll
              for (int k = 0; k < 4; ++k) {
                const bool v = k < n;
                cc[a][k] = v ? col[k0 + k] : -1 - (4 * a + k);
                ww[a][k] = v ? val[k0 + k] : 0.0;
              }
            }
            double M4[16];
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
              for (int b = a; b < 4; ++b) {
                double acc = 0.0;
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                  for (int l = 0; l < 4; ++l) acc += cc[a][k] == cc[b][l] ? ww[a][k] * ww[b][l] : 0.0;
                M4[a * 4 + b] = acc;
                M4[b * 4 + a] = acc;
              }
            reduced_block_projection(M4, tv + 9);
          }
          double2 *r2 = (double2 *)(rec + i * TERM_REC);
          const int nst = want_h ? 27 : 5;
#pragma unroll
          for (int q = 0; q < 27; ++q)
            if (q < nst) r2[q] = make_double2(tv[2 * q], tv[2 * q + 1]);
        } else {
          e_pair = pair_energy<KIND>(ty, x, eps, dhat, kappa, sq);
        }
      }
      if (energy && vscene) agg_scene_add(energy, live, scene, n_scene, e_pair, status);
      e_acc += e_pair;
    }
  }
  if (energy && !vscene) {
    e_acc = wave_sum(e_acc);
    if (lane == 0) s_e[wave] = e_acc;
    __syncthreads();
    if (threadIdx.x == 0) {
      double t = 0.0;
      for (int w = 0; w < NW; ++w) t += s_e[w];
      if (t != 0.0) atomicAdd(energy, t);
    }
  }
}

eipc_status launch_barrier(eipc_ctx *c, const eipc_scene *sc, int kind, const double *xs, const int32_t *pairs,
                           const int32_t *act, const int32_t *typ, const int64_t *d_count, int64_t max_count,
                           double dhat, double kappa, uint32_t flags, double *energy, double *grad,
                           const HessOut &h, hipStream_t s) {
  if (max_count == 0) return EIPC_OK;
  // the interface's limit (a reduction that packed node ids with four bits
  // set it); larger systems stay refused
  if (sc->n_node >= (1 << 27)) return set_err(c, EIPC_ERR_ARG, "n_node must be below 2^27");
  const bool want_g = (flags & EIPC_GRAD) && grad;
  const bool want_h = (flags & EIPC_HESS) && h.kind != 0;
  const int64_t cap = max_count;
  const int4 *vid4 = nullptr;  // vertex ids of the sorted pairs
  double *rec = nullptr;
  if (want_g || want_h) {
    EIPC_TRY(sort_active(c, sc, kind, pairs, act, typ, d_count, cap, &act, &typ, &vid4, s));
    EIPC_TRY(ensure_t(c, kind == 0 ? B_PX_PT : B_PX_EE, (size_t)TERM_REC * cap, &rec));
  }
  const int blocks =
      (int)std::max<int64_t>(1, std::min<int64_t>(grid_for(max_count, 64), (int64_t)c->wg_per_cu[0] * c->num_cu));
  const int32_t *vsc = vscene_of(sc);
  const int nsc = n_scene_of(sc);
  {
    ProfScope ps(c, kind == 0 ? K_BARRIER_PT : K_BARRIER_EE, s);
#define EIPC_TERMS_LAUNCH(K, R, G)                                                                                 \
  k_pair_terms<K, R, G><<<blocks, TERMS_T, 0, s>>>(pairs, act, typ, vid4, d_count, cap, sc->faces, sc->edges, xs,        \
                                                sc->x_rest, sc->n_vert, dhat, kappa, flags, want_g, want_h, energy, \
                                                rec, vsc, nsc, c->status, sc->W_rowptr, sc->W_col, sc->W_val)
    const bool reduced = want_h && (flags & EIPC_PROJECT_REDUCED);
    const bool moll = (flags & EIPC_MOLLIFY) && sc->x_rest;
    if (kind == 0) {
      if (reduced)
        EIPC_TERMS_LAUNCH(0, true, true);
      else
        EIPC_TERMS_LAUNCH(0, false, false);
    } else {
      if (reduced)
        EIPC_TERMS_LAUNCH(1, true, true);
      else if (moll)
        EIPC_TERMS_LAUNCH(1, false, true);
      else
        EIPC_TERMS_LAUNCH(1, false, false);
    }
#undef EIPC_TERMS_LAUNCH
    EIPC_HIP(c, hipGetLastError());
  }
  if (!want_g && !want_h) return EIPC_OK;
  return launch_expand(c, sc, kind, vid4, d_count, cap, rec, want_g, want_h, want_g ? grad : nullptr,
                       want_h ? h : HessOut{}, s);
}

eipc_status launch_expand(eipc_ctx *c, const eipc_scene *sc, int kind, const int4 *vid4, const int64_t *d_count,
                          int64_t cap, const double *rec, bool want_g, bool want_h, double *grad, const HessOut &h,
                          hipStream_t s) {
  if (sc->n_node >= (1 << 27)) return set_err(c, EIPC_ERR_ARG, "n_node must be below 2^27");
  const int blocks =
      (int)std::max<int64_t>(1, std::min<int64_t>(grid_for(cap, 64), (int64_t)c->wg_per_cu[1] * c->num_cu));
  ProfScope ps(c, kind == 0 ? K_EXPAND_PT : K_EXPAND_EE, s);
#define EX_CALL(KIND, H)                                                                                              \
  k_expand<KIND, H><<<blocks, EX_T, 0, s>>>(vid4, d_count, sc->W_rowptr, sc->W_col, sc->W_val, sc->n_node, rec, cap, \
                                            want_g, grad, h, c->status)
  if (kind == 0) {
    if (want_h)
      EX_CALL(0, true);
    else
      EX_CALL(0, false);
  } else {
    if (want_h)
      EX_CALL(1, true);
    else
      EX_CALL(1, false);
  }
#undef EX_CALL
  EIPC_HIP(c, hipGetLastError());
  return EIPC_OK;
}

// lower 3x3 blocks of the dense reduced Hessian from the upper ones
__global__ void k_dense_mirror(int n_node, double *d) {
  const int64_t n3 = 3 * (int64_t)n_node;
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n3 * n3) return;
  const int64_t r = idx / n3, cc = idx % n3;
  if (r / 3 > cc / 3) d[idx] = d[cc * n3 + r];
}

eipc_status launch_dense_mirror(eipc_ctx *c, int n_node, double *dense, hipStream_t s) {
  int64_t n3 = 3 * (int64_t)n_node;
  if (n3 == 0) return EIPC_OK;
  k_dense_mirror<<<grid_for(n3 * n3, 256), 256, 0, s>>>(n_node, dense);
  EIPC_HIP(c, hipGetLastError());
  return EIPC_OK;
}

// ---------------------------------------------------------------------------
// BSR from the global hash of upper blocks: count per row (both
// triangles), scan, fill, sort each row by column, gather values.
// ---------------------------------------------------------------------------
__global__ void k_hash_rowcount(int64_t cap, const int64_t *hkey, int n_node, int32_t *rowcnt) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= cap) return;
  const int64_t key = hkey[t];
  if (key < 0) return;
  const int I = (int)(key / n_node), J = (int)(key % n_node);
  atomicAdd(&rowcnt[I], 1);
  if (I != J) atomicAdd(&rowcnt[J], 1);
}

__global__ void k_hash_rowfill(int64_t cap, const int64_t *hkey, int n_node, const int64_t *rowptr,
                               int32_t *rowfill, int32_t *bcol, int64_t *bsrc, int64_t nnzb_cap) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= cap) return;
  const int64_t key = hkey[t];
  if (key < 0) return;
  const int I = (int)(key / n_node), J = (int)(key % n_node);
  int64_t p = rowptr[I] + atomicAdd(&rowfill[I], 1);
  if (p < nnzb_cap) {
    bcol[p] = J;
    bsrc[p] = 2 * t;  // even: as stored
  }
  if (I != J) {
    p = rowptr[J] + atomicAdd(&rowfill[J], 1);
    if (p < nnzb_cap) {
      bcol[p] = I;
      bsrc[p] = 2 * t + 1;  // odd: transposed
    }
  }
}

// Sort each BSR row by column, out of place (bcol, bsrc -> bcol2, bsrc2):
// one wavefront per row.  Columns of a row are distinct, so an entry's
// position is its rank, the number of entries of the row with a smaller
// column.  Rows of up to 64 entries rank by shuffles; longer rows are
// taken 64 entries at a time, each ranked against the whole row by
// wavefront-uniform reads (any length; time grows as len^2 / 64).
// A capacity that is too small raises the overflow and cuts the list: rows
// past it are empty, and what lies within it of the row that crosses it is
// marked as having no source (column 0, a zero block).
__global__ void k_row_sort(int n_node, const int64_t *rowptr, const int32_t *bcol, const int64_t *bsrc,
                           int32_t *bcol2, int64_t *bsrc2, int32_t *rowptr32, int64_t nnzb_cap, uint32_t *status) {
  const int lane = threadIdx.x & 63;
  const int r = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  if (r > n_node) return;
  if (r == n_node) {
    if (lane == 0) {
      const int64_t tot = rowptr[r];
      rowptr32[r] = (int32_t)(tot < nnzb_cap ? tot : nnzb_cap);
      if (tot > nnzb_cap) atomicOr(status, ST_PLAN_OVERFLOW);
    }
    return;
  }
  const int64_t b = rowptr[r], e = rowptr[r + 1];
  if (lane == 0) rowptr32[r] = (int32_t)(b < nnzb_cap ? b : nnzb_cap);
  if (e > nnzb_cap) {
    for (int64_t p = b + lane; p < nnzb_cap; p += 64) {
      bcol2[p] = 0;
      bsrc2[p] = -1;
    }
    return;
  }
  const int64_t len = e - b;
  if (len <= 64) {
    const bool v = lane < len;
    const int32_t cv = v ? bcol[b + lane] : 0x7fffffff;
    int rank = 0;
    for (int j = 0; j < len; ++j) rank += __shfl(cv, j, 64) < cv;
    if (v) {
      bcol2[b + rank] = cv;
      bsrc2[b + rank] = bsrc[b + lane];
    }
    return;
  }
  for (int64_t c0 = 0; c0 < len; c0 += 64) {
    const int64_t idx = c0 + lane;
    const bool v = idx < len;
    const int32_t cv = v ? bcol[b + idx] : 0x7fffffff;
    int64_t rank = 0;
    for (int64_t j = 0; j < len; ++j) rank += bcol[b + j] < cv;
    if (v) {
      bcol2[b + rank] = cv;
      bsrc2[b + rank] = bsrc[b + idx];
    }
  }
}

// blocks in BSR order; the count is read from the device (capped)
__global__ void k_bsr_gather(int64_t cap, const int32_t *rowptr32, int n_node, const int64_t *bsrc,
                             const double *hval, double *blocks) {
  const int64_t nnzb = rowptr32[n_node];
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < nnzb && p < cap;
       p += (int64_t)gridDim.x * blockDim.x) {
    const int64_t src = bsrc[p];
    if (src < 0) {  // in the row that the capacity cuts
#pragma unroll
      for (int t = 0; t < 9; ++t) blocks[9 * p + t] = 0.0;
      continue;
    }
    const double *v = hval + 9 * (src >> 1);
    if ((src & 1) == 0) {
#pragma unroll
      for (int t = 0; t < 9; ++t) blocks[9 * p + t] = v[t];
    } else {
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) blocks[9 * p + 3 * i + j] = v[3 * j + i];
    }
  }
}

// the row counters of bsr_compact, to be cleared before it runs
eipc_status bsr_clear(eipc_ctx *c, int n_node, FillList &fl) {
  const size_t bytes = fill_bytes(sizeof(int32_t) * ((size_t)n_node + 1));
  int32_t *rowcnt, *rowfill;
  EIPC_TRY(ensure_t(c, B_ROWCNT, (size_t)n_node + 1, &rowcnt));
  EIPC_TRY(ensure_t(c, B_ROWFILL, (size_t)n_node + 1, &rowfill));
  fl.add(rowcnt, bytes, 0);
  fl.add(rowfill, bytes, 0);
  return EIPC_OK;
}

eipc_status bsr_compact(eipc_ctx *c, int n_node, const HessOut &h, eipc_bsr *out, hipStream_t s, int64_t nnzb_cap,
                        uint32_t *status) {
  const int64_t cap = (int64_t)h.hmask + 1;
  int32_t *rowcnt, *rowfill, *bcol, *rowptr32;
  int64_t *rowptr, *bsrc;
  double *blocks;
  EIPC_TRY(ensure_t(c, B_ROWCNT, (size_t)n_node + 1, &rowcnt));
  EIPC_TRY(ensure_t(c, B_ROWFILL, (size_t)n_node + 1, &rowfill));
  EIPC_TRY(ensure_t(c, B_ROWPTR, (size_t)n_node + 1, &rowptr));
  k_hash_rowcount<<<grid_for(cap, 256), 256, 0, s>>>(cap, h.hkey, n_node, rowcnt);
  EIPC_HIP(c, hipGetLastError());
  EIPC_TRY(exclusive_scan(c, rowcnt, n_node, rowptr, s));
  const bool planned = nnzb_cap >= 0;
  int64_t nnzb = 0;
  if (!planned) {
    EIPC_HIP(c, hipMemcpyAsync(&nnzb, rowptr + n_node, 8, hipMemcpyDeviceToHost, s));
    EIPC_HIP(c, hipStreamSynchronize(s));
    nnzb_cap = nnzb;
  }
  EIPC_TRY(ensure_t(c, B_BCOL, (size_t)std::max<int64_t>(nnzb_cap, 1), &bcol));
  EIPC_TRY(ensure_t(c, B_BSRC, (size_t)std::max<int64_t>(nnzb_cap, 1), &bsrc));
  EIPC_TRY(ensure_t(c, B_BBLK, (size_t)std::max<int64_t>(nnzb_cap, 1) * 9, &blocks));
  int32_t *bcol2;
  int64_t *bsrc2;
  EIPC_TRY(ensure_t(c, B_BCOL2, (size_t)std::max<int64_t>(nnzb_cap, 1), &bcol2));
  EIPC_TRY(ensure_t(c, B_BSRC2, (size_t)std::max<int64_t>(nnzb_cap, 1), &bsrc2));
  rowptr32 = rowcnt;  // counts are no longer needed once scanned
  k_hash_rowfill<<<grid_for(cap, 256), 256, 0, s>>>(cap, h.hkey, n_node, rowptr, rowfill, bcol, bsrc, nnzb_cap);
  EIPC_HIP(c, hipGetLastError());
  k_row_sort<<<grid_for((int64_t)(n_node + 1) * 64, 256), 256, 0, s>>>(n_node, rowptr, bcol, bsrc, bcol2, bsrc2,
                                                                        rowptr32, nnzb_cap, status);
  EIPC_HIP(c, hipGetLastError());
  if (nnzb_cap > 0) {
    k_bsr_gather<<<std::min(grid_for(nnzb_cap, 256), 16 * c->num_cu), 256, 0, s>>>(nnzb_cap, rowptr32, n_node, bsrc2,
                                                                                   h.hval, blocks);
    EIPC_HIP(c, hipGetLastError());
  }
  out->n_rows = n_node;
  out->nnzb = planned ? -1 : nnzb;
  out->rowptr = rowptr32;
  out->col = bcol2;
  out->blocks = blocks;
  return EIPC_OK;
}

// ---------------------------------------------------------------------------
// Hessian-vector product: y = H_x z per pair, z = (W v + v_off) on the
// pair's vertices, scattered through W^T (and unreduced into out_off).
// H_x = Q X Q^T:  zeta = Q^T z, eta = X zeta, y = Q eta.
// ---------------------------------------------------------------------------
template <int KIND, bool GEN>
__global__ __launch_bounds__(BR_THREADS) __attribute__((amdgpu_waves_per_eu(GEN ? 1 : 2))) void k_hvp(
    const int32_t *__restrict__ pairs, const int32_t *__restrict__ act, const int32_t *__restrict__ typ,
    const int64_t *__restrict__ d_count, const int32_t *__restrict__ faces, const int32_t *__restrict__ edges,
    const int32_t *__restrict__ rowptr, const int32_t *__restrict__ col, const double *__restrict__ val,
    const double *__restrict__ xs, const double *__restrict__ xvs, const double *__restrict__ x_rest, int n_vert,
    int n_node, double dhat, double kappa, uint32_t flags, double *out, double *out_off, uint32_t *status) {
  __shared__ uint32_t s_gkey[LGT];
  __shared__ double s_gval[LGT * 3];
  __shared__ int s_used;
  LdsTables T{s_gkey, s_gval};
  HessOut none{0, nullptr, nullptr, nullptr, 0};
  Acc A{T, none, n_node, out, status};
  const bool moll = GEN && (KIND == 1) && (flags & EIPC_MOLLIFY) && x_rest;
  for (int t = threadIdx.x; t < LGT; t += BR_THREADS) s_gkey[t] = 0xffffffffu;
  for (int t = threadIdx.x; t < LGT * 3; t += BR_THREADS) s_gval[t] = 0.0;
  __syncthreads();
  const int64_t n = *d_count;
  const int64_t per = ((n + gridDim.x - 1) / gridDim.x + BR_THREADS - 1) / BR_THREADS * BR_THREADS;
  const int64_t r0 = (int64_t)blockIdx.x * per;
  const int64_t r1 = r0 + per < n ? r0 + per : n;
  for (int64_t base = r0; base < r1; base += BR_THREADS) {
    const int64_t i = base + threadIdx.x;
    const bool active = i < r1;
    double eta[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    int vid[4] = {0, 0, 0, 0};
    if (active) {
      const int64_t k = act[i];
      const int ty = typ[i];
      pair_vertices<KIND>(pairs, k, faces, edges, vid);
      V3 x[4], z[4];
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        x[a] = load3(xs, n_vert, vid[a]);
        z[a] = load3(xvs, n_vert, vid[a]);
      }
      double eps = 0.0;
      if (moll) {
        V3 r[4];
#pragma unroll
        for (int a = 0; a < 4; ++a)
          r[a] = V3{x_rest[3 * (int64_t)vid[a]], x_rest[3 * (int64_t)vid[a] + 1], x_rest[3 * (int64_t)vid[a] + 2]};
        eps = mollifier_eps(r);
      }
      // the Hessian of the barrier stage's per-class path
      double gam[9], M[45];
      pair_qterms<KIND, GEN>(pair_class<KIND>(ty, x, eps), ty, x, eps, dhat, kappa, false, true,
                        (flags & EIPC_PROJECT) != 0, (flags & EIPC_SQDIST) != 0, gam, M);
      // zeta = Q^T z, eta = X zeta
      double zeta[9];
#pragma unroll
      for (int al = 0; al < 3; ++al) {
        double zx = 0, zy = 0, zz = 0;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          const double sg = 0.5 * kS[a][al];
          zx += sg * z[a].x;
          zy += sg * z[a].y;
          zz += sg * z[a].z;
        }
        zeta[3 * al] = zx;
        zeta[3 * al + 1] = zy;
        zeta[3 * al + 2] = zz;
      }
#pragma unroll
      for (int r = 0; r < 9; ++r) {
        double acc = 0.0;
#pragma unroll
        for (int cc = 0; cc < 9; ++cc) acc += M[pidx(r, cc)] * zeta[cc];
        eta[r] = acc;
      }
      if (out_off) {
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          double y0 = 0, y1 = 0, y2 = 0;
#pragma unroll
          for (int al = 0; al < 3; ++al) {
            const double sg = 0.5 * kS[a][al];
            y0 += sg * eta[3 * al];
            y1 += sg * eta[3 * al + 1];
            y2 += sg * eta[3 * al + 2];
          }
          atomicAdd(&out_off[3 * (int64_t)vid[a]], y0);
          atomicAdd(&out_off[3 * (int64_t)vid[a] + 1], y1);
          atomicAdd(&out_off[3 * (int64_t)vid[a] + 2], y2);
        }
      }
    }
    // reduced product through the merged node set: out[I] += z_I^T eta
    NodeSet S;
    int m = 0;
    if (active) gather_nodes<KIND>(vid, rowptr, col, val, S, m);
#pragma unroll
    for (int sl = 0; sl < 16; ++sl) {
      const bool v = active && sl < m;
      if (__any(v)) {
        double g[3];
#pragma unroll
        for (int c = 0; c < 3; ++c)
          g[c] = S.z[sl][0] * eta[c] + S.z[sl][1] * eta[3 + c] + S.z[sl][2] * eta[6 + c];
        agg_vec(A, v, v ? S.node[sl] : -1, g[0], g[1], g[2]);
      }
    }
    __syncthreads();
    const bool last = base + BR_THREADS >= r1;
    if (!last) {
      if (threadIdx.x == 0) s_used = 0;
      __syncthreads();
      int cnt = 0;
      for (int t = threadIdx.x; t < LGT; t += BR_THREADS) cnt += s_gkey[t] != 0xffffffffu;
      if (cnt) atomicAdd(&s_used, cnt);
      __syncthreads();
    }
    if (last || s_used > LGT / 2) {
      for (int t = threadIdx.x; t < LGT; t += BR_THREADS) {
        const int key = (int)s_gkey[t];
        if (key != -1) {
          atomicAdd(&out[3 * (int64_t)key], s_gval[3 * t]);
          atomicAdd(&out[3 * (int64_t)key + 1], s_gval[3 * t + 1]);
          atomicAdd(&out[3 * (int64_t)key + 2], s_gval[3 * t + 2]);
          s_gkey[t] = 0xffffffffu;
          s_gval[3 * t] = s_gval[3 * t + 1] = s_gval[3 * t + 2] = 0.0;
        }
      }
    }
    __syncthreads();
  }
}

eipc_status launch_hvp(eipc_ctx *c, const eipc_scene *sc, int kind, const double *xs, const double *xvs,
                       const int32_t *pairs, const int32_t *act, const int32_t *typ, const int64_t *d_count,
                       int64_t max_count, double dhat, double kappa, uint32_t flags, double *out,
                       double *out_off, hipStream_t s, bool locality_sort) {
  if (max_count == 0) return EIPC_OK;
  // the locality order only cuts the flushes of the LDS tables
  if (locality_sort) EIPC_TRY(sort_active(c, sc, kind, pairs, act, typ, d_count, max_count, &act, &typ, nullptr, s));
  int blocks = (int)std::min<int64_t>(grid_for(max_count, BR_THREADS), 4 * (int64_t)c->num_cu);
  ProfScope ps(c, kind == 0 ? K_HVP_PT : K_HVP_EE, s);
  if (kind == 0)
    k_hvp<0, false><<<blocks, BR_THREADS, 0, s>>>(pairs, act, typ, d_count, sc->faces, sc->edges, sc->W_rowptr, sc->W_col,
                                            sc->W_val, xs, xvs, sc->x_rest, sc->n_vert, sc->n_node, dhat, kappa,
                                            flags, out, out_off, c->status);
  else if ((flags & EIPC_MOLLIFY) && sc->x_rest)
    k_hvp<1, true><<<blocks, BR_THREADS, 0, s>>>(pairs, act, typ, d_count, sc->faces, sc->edges, sc->W_rowptr, sc->W_col,
                                            sc->W_val, xs, xvs, sc->x_rest, sc->n_vert, sc->n_node, dhat, kappa,
                                            flags, out, out_off, c->status);
  else
    k_hvp<1, false><<<blocks, BR_THREADS, 0, s>>>(pairs, act, typ, d_count, sc->faces, sc->edges, sc->W_rowptr, sc->W_col,
                                            sc->W_val, xs, xvs, sc->x_rest, sc->n_vert, sc->n_node, dhat, kappa,
                                            flags, out, out_off, c->status);
  EIPC_HIP(c, hipGetLastError());
  return EIPC_OK;
}

// ---------------------------------------------------------------------------
// per-pair inspection: type, s, e, g (12), H (12x12)
// ---------------------------------------------------------------------------
template <int KIND>
__global__ __launch_bounds__(64) void k_pair_eval(int64_t n, const int32_t *__restrict__ pairs, const int32_t *__restrict__ faces,
                            const int32_t *__restrict__ edges, const double *__restrict__ xs,
                            const double *__restrict__ x_rest, int n_vert, double dhat, double kappa,
                            uint32_t flags, int32_t *type, double *sq, double *e, double *g, double *H) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int vid[4];
  pair_vertices<KIND>(pairs, i, faces, edges, vid);
  V3 x[4];
#pragma unroll
  for (int a = 0; a < 4; ++a) x[a] = load3(xs, n_vert, vid[a]);
  int ty;
  const double s2 = pair_dist2<KIND>(x, &ty);
  if (type) type[i] = ty;
  if (sq) sq[i] = s2;
  const bool active = s2 > 0.0 && s2 < dhat * dhat;
  double eps = 0.0;
  if (KIND == 1 && (flags & EIPC_MOLLIFY) && x_rest) {
    V3 r[4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
      r[a] = V3{x_rest[3 * (int64_t)vid[a]], x_rest[3 * (int64_t)vid[a] + 1], x_rest[3 * (int64_t)vid[a] + 2]};
    eps = mollifier_eps(r);
  }
  // the barrier stage's own per-class path; x-space gradient g_x = Q gamma
  double gam[9], M[45];
  double ev = 0.0;
  if (active) {
    const int cls = pair_class<KIND>(ty, x, eps);
    ev = pair_qterms<KIND, true>(cls, ty, x, eps, dhat, kappa, true, true, (flags & EIPC_PROJECT) != 0,
                           (flags & EIPC_SQDIST) != 0, gam, M);
  }
  if (e) e[i] = ev;
  if (g) {
    for (int a = 0; a < 4; ++a)
      for (int c = 0; c < 3; ++c) {
        double acc = 0.0;
        if (active)
          for (int al = 0; al < 3; ++al) acc += (0.5 * kS[a][al]) * gam[3 * al + c];
        g[12 * i + 3 * a + c] = acc;
      }
  }
  if (H) {
    for (int a = 0; a < 4; ++a)
      for (int b = 0; b < 4; ++b) {
        double B[9];
        if (active)
          x_block(M, a, b, B);
        else
          for (int t = 0; t < 9; ++t) B[t] = 0.0;
        for (int ii = 0; ii < 3; ++ii)
          for (int jj = 0; jj < 3; ++jj) H[144 * i + (3 * a + ii) * 12 + 3 * b + jj] = B[3 * ii + jj];
      }
  }
}

eipc_status launch_pair_eval(eipc_ctx *c, const eipc_scene *sc, int kind, const double *xs, const int32_t *pairs,
                             int64_t n, double dhat, double kappa, uint32_t flags, int32_t *type, double *sq,
                             double *e, double *g, double *H, hipStream_t s) {
  if (n == 0) return EIPC_OK;
  if (kind == 0)
    k_pair_eval<0><<<grid_for(n, 64), 64, 0, s>>>(n, pairs, sc->faces, sc->edges, xs, sc->x_rest, sc->n_vert, dhat,
                                                   kappa, flags, type, sq, e, g, H);
  else
    k_pair_eval<1><<<grid_for(n, 64), 64, 0, s>>>(n, pairs, sc->faces, sc->edges, xs, sc->x_rest, sc->n_vert, dhat,
                                                   kappa, flags, type, sq, e, g, H);
  EIPC_HIP(c, hipGetLastError());
  return EIPC_OK;
}

}  // namespace eipc
