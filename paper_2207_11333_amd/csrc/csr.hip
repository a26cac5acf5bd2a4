// Step S0: batch validation and the destination-sorted CSR.  Small batches take
// one launch (k_csr_small), larger ones a chain of seven.
//
// Edges of a batch of molecular graphs (Table 1 layout: edge_index (2, E),
// row 0 source, row 1 destination) are grouped by destination and, within a
// destination, ordered by (source id, edge id).  The by-source transpose
// lists, for every node, the CSR positions of its out-edges in ascending
// order; the aggregation adjoint uses it to sum per-edge gradients by source
// without atomics.  Atomic counters only place edges into their segment; a
// per-segment sort then fixes the order, so every integer output is
// deterministic and independent of the COO edge order.
#include "common.hpp"

#include <algorithm>

namespace hgnn {

namespace {

__global__ void __launch_bounds__(kErrWords)
k_set_dims(Dims *d, int B, int N, int E, int *__restrict__ err) {
  if (threadIdx.x == 0 && d) *d = Dims{B, N, E, 0};
  err[threadIdx.x] = 0;
}

// node -> graph id by binary search over graph_ptr (staged in LDS when it
// fits, so the search costs no dependent global loads); zero the counters;
// check graph_ptr; the first layer's input zero-padded from F to Fp columns.
// Thread t covers node t and the four padded-input columns 4 (t % (Fp/4)) ..
// of row t / (Fp/4), so the grid spreads the copy over many CUs.
constexpr int kInitThreads = 256;
constexpr int kGraphPtrLds = 4096;

__global__ void __launch_bounds__(kInitThreads)
k_csr_init(const Dims *__restrict__ dims, const int *__restrict__ graph_ptr,
           int *__restrict__ node_graph, int *__restrict__ cnt_in, int *__restrict__ cnt_out,
           int *__restrict__ err, const float *__restrict__ x, int F,
           float *__restrict__ xpad, int Fp) {
  __shared__ int s_gp[kGraphPtrLds];
  const int B = dims->B, N = dims->N;
  const int i = blockIdx.x * kInitThreads + threadIdx.x;
  // only workgroups holding nodes search (the condition is uniform per block)
  const bool staged = B + 1 <= kGraphPtrLds && (int)blockIdx.x * kInitThreads < N;
  if (staged)
    for (int k = threadIdx.x; k <= B; k += kInitThreads) s_gp[k] = graph_ptr[k];
  __syncthreads();
  if (i < B) {
    if (graph_ptr[i + 1] <= graph_ptr[i]) atomicOr(err, ERR_GRAPH_PTR);
  }
  if (i == 0) {
    if (graph_ptr[0] != 0 || graph_ptr[B] != N) atomicOr(err, ERR_GRAPH_PTR);
  }
  if (i < N) {
    // last b with graph_ptr[b] <= i (two loops, so that each reads its own
    // address space: LDS reads rather than generic ones)
    int lo = 0, hi = B;
    if (staged) {
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (s_gp[mid] <= i) lo = mid; else hi = mid;
      }
    } else {
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (graph_ptr[mid] <= i) lo = mid; else hi = mid;
      }
    }
    node_graph[i] = lo;
    cnt_in[i] = 0;
    cnt_out[i] = 0;
  }
  const int q = Fp >> 2; // 16-byte groups per padded row
  if (x && i < N * q) {
    const int r = i / q, c0 = (i - r * q) * 4;
    const float *xr = x + (size_t)r * F;
    f4 v;
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = c0 + k < F ? xr[c0 + k] : 0.f;
    if (!(isfinite(v[0]) && isfinite(v[1]) && isfinite(v[2]) && isfinite(v[3])))
      atomicOr(err, ERR_NONFINITE);
    *reinterpret_cast<f4 *>(xpad + (size_t)r * Fp + c0) = v;
  }
}

__device__ __forceinline__ bool edge_ok(int s, int d, int N,
                                        const int *__restrict__ node_graph) {
  return s >= 0 && s < N && d >= 0 && d < N && node_graph[s] == node_graph[d];
}

__global__ void k_csr_count(const Dims *__restrict__ dims,
                            const int *__restrict__ ei,
                            const int *__restrict__ node_graph,
                            int *__restrict__ cnt_in, int *__restrict__ cnt_out,
                            int *__restrict__ err) {
  const int N = dims->N, E = dims->E;
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= E) return;
  const int s = ei[k], d = ei[E + k];
  if (s < 0 || s >= N || d < 0 || d >= N) {
    atomicOr(err, ERR_EDGE_RANGE);
    return;
  }
  if (node_graph[s] != node_graph[d]) {
    atomicOr(err, ERR_EDGE_CROSS);
    return;
  }
  atomicAdd(&cnt_in[d], 1);
  atomicAdd(&cnt_out[s], 1);
}

// Exclusive scans of both degree counters (rowptr, srcptr) over all nodes in
// three passes, no workgroup waiting on another: per block of kScanNodes
// nodes (one per thread) the counter sums and the node count of every degree
// bucket (k_scan_count); one workgroup, a wave per column, turns those into
// block offsets and bucket offsets (k_scan_top); every block then scans its
// own nodes again, adds its offsets and writes rowptr, srcptr, degrees,
// scalers and, with degree buckets, each node's place in the (degree, node
// id) order (k_scan_apply).
constexpr int kScanTop = 1024;
static_assert(kScanNodes == 256, "one node per thread of a 256-thread block");

__device__ __forceinline__ int wave_incl_scan(int v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(v, o, 64);
    if (lane >= o) v += t;
  }
  return v;
}

__device__ __forceinline__ int bucket_of(int d, int max_degree) {
  return d < max_degree ? d : max_degree; // clamped: a bad degree is flagged elsewhere
}

__global__ void __launch_bounds__(kScanNodes)
k_scan_count(const Dims *__restrict__ dims, const int *__restrict__ cnt_in,
             const int *__restrict__ cnt_out, int max_degree, int nb,
             int *__restrict__ scan) {
  __shared__ int s_w[2 + kMaxBuckets][kScanNodes / 64];
  const int N = dims->N;
  const int base = blockIdx.x * kScanNodes;
  if (base >= N) return;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int i = base + tid;
  const int vi = i < N ? cnt_in[i] : 0, vo = i < N ? cnt_out[i] : 0;
  const int bq = i < N ? bucket_of(vi, max_degree) : -1;
  const int si = wave_incl_scan(vi), so = wave_incl_scan(vo);
  if (lane == 63) {
    s_w[0][wid] = si;
    s_w[1][wid] = so;
  }
  for (int q = 0; q < nb; ++q) {
    const unsigned long long m = __ballot(bq == q);
    if (lane == 0) s_w[2 + q][wid] = __popcll(m);
  }
  __syncthreads();
  int *rec = scan + (size_t)blockIdx.x * kScanRec;
  if (tid < 2 + nb) rec[tid] = s_w[tid][0] + s_w[tid][1] + s_w[tid][2] + s_w[tid][3];
}

// One workgroup; wave c scans column c of the block records (c < 2 + nb)
// over the blocks, 64 at a time with a carry.  The column totals give
// rowptr[N], srcptr[N] and the first row of every degree bucket (brow[q] =
// nodes of lower degree), which k_scan_apply adds to the bucket columns.
__global__ void __launch_bounds__(kScanTop)
k_scan_top(const Dims *__restrict__ dims, int nb, int *__restrict__ scan,
           int *__restrict__ brow, int *__restrict__ rowptr, int *__restrict__ srcptr) {
  __shared__ int tot[kScanRec];
  const int N = dims->N;
  const int nblk = (N + kScanNodes - 1) / kScanNodes;
  const int ncol = 2 + nb;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  for (int c = wid; c < ncol; c += kScanTop / 64) {
    int carry = 0;
    for (int b0 = 0; b0 < nblk; b0 += 64) {
      const int k = b0 + lane;
      int *cell = scan + (size_t)k * kScanRec + c;
      const int v = k < nblk ? *cell : 0;
      const int inc = wave_incl_scan(v);
      if (k < nblk) *cell = carry + inc - v;
      carry += __shfl(inc, 63, 64);
    }
    if (lane == 0) tot[c] = carry;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    rowptr[N] = tot[0];
    srcptr[N] = tot[1];
    if (nb) {
      int a = 0;
      for (int q = 0; q < nb; ++q) {
        brow[q] = a;
        a += tot[2 + q];
      }
      brow[nb] = a;
    }
  }
}

// Per block: its own exclusive scans plus the block offsets.  A node's place
// among the nodes of its degree bucket counts the block's earlier nodes of
// that bucket (earlier waves, then earlier lanes of its wave), so the
// permutation is stable in node id.
//
// fused (at most kScanFuse blocks): k_scan_top is not run; each block sums
// the raw block records itself (a wave per column: the records of earlier
// blocks and of all blocks), and block 0 writes rowptr[N], srcptr[N] and the
// bucket bounds.  One dependent launch fewer on the step's critical path.
constexpr int kScanFuse = 256;

__global__ void __launch_bounds__(kScanNodes)
k_scan_apply(const Dims *__restrict__ dims, int *__restrict__ cnt_in,
             int *__restrict__ cnt_out, const int *__restrict__ scan,
             const float *__restrict__ table, int max_degree, int nb,
             int *__restrict__ rowptr, int *__restrict__ srcptr, int *__restrict__ deg,
             float *__restrict__ sp, float *__restrict__ sm, int *__restrict__ perm,
             int *__restrict__ brow, int *__restrict__ err, int fused) {
  __shared__ int s_w[2][kScanNodes / 64];
  __shared__ int s_bw[kScanNodes / 64][kMaxBuckets];
  __shared__ int s_off[kScanRec], s_tot[kScanRec];
  const int N = dims->N;
  const int base = blockIdx.x * kScanNodes;
  if (base >= N) return;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int *rec = scan + (size_t)blockIdx.x * kScanRec;
  if (fused) {
    const int nblk = (N + kScanNodes - 1) / kScanNodes;
    for (int c = wid; c < 2 + nb; c += kScanNodes / 64) {
      int before = 0, total = 0;
      for (int k = lane; k < nblk; k += 64) {
        const int v = scan[(size_t)k * kScanRec + c];
        total += v;
        before += k < (int)blockIdx.x ? v : 0;
      }
      for (int o = 32; o > 0; o >>= 1) {
        before += __shfl_xor(before, o, 64);
        total += __shfl_xor(total, o, 64);
      }
      if (lane == 0) {
        s_off[c] = before;
        s_tot[c] = total;
      }
    }
  }
  const int i = base + tid;
  const int vi = i < N ? cnt_in[i] : 0, vo = i < N ? cnt_out[i] : 0;
  const int bq = i < N ? bucket_of(vi, max_degree) : -1;
  const int ii = wave_incl_scan(vi), io = wave_incl_scan(vo);
  if (lane == 63) {
    s_w[0][wid] = ii;
    s_w[1][wid] = io;
  }
  // rank among the wave's earlier lanes of the same bucket
  const unsigned long long below = (1ull << lane) - 1ull;
  int pos = 0;
  for (int q = 0; q < nb; ++q) {
    const unsigned long long m = __ballot(bq == q);
    if (lane == 0) s_bw[wid][q] = __popcll(m);
    if (bq == q) pos = __popcll(m & below);
  }
  __syncthreads();
  if (fused && blockIdx.x == 0 && tid == 0) {
    rowptr[N] = s_tot[0];
    srcptr[N] = s_tot[1];
    if (nb) {
      int a = 0;
      for (int q = 0; q < nb; ++q) {
        brow[q] = a;
        a += s_tot[2 + q];
      }
      brow[nb] = a;
    }
  }
  if (i >= N) return;
  const int r0 = fused ? s_off[0] : rec[0], r1 = fused ? s_off[1] : rec[1];
  int ei_ = r0 + ii - vi, eo_ = r1 + io - vo;
  for (int w = 0; w < wid; ++w) {
    ei_ += s_w[0][w];
    eo_ += s_w[1][w];
  }
  rowptr[i] = ei_;
  srcptr[i] = eo_;
  deg[i] = vi;
  sp[i] = table[2 * bq];
  sm[i] = table[2 * bq + 1];
  cnt_in[i] = 0;
  cnt_out[i] = 0;
  if (nb) {
    int p = pos;
    if (fused) {
      p += s_off[2 + bq];
      for (int q = 0; q < bq; ++q) p += s_tot[2 + q]; // the bucket's first row
    } else {
      p += brow[bq] + rec[2 + bq];
    }
    for (int w = 0; w < wid; ++w) p += s_bw[w][bq];
    perm[p] = i;
  }
  if (vi > max_degree || vo > max_degree) atomicOr(err, ERR_DEGREE);
}

__global__ void k_csr_fill(const Dims *__restrict__ dims,
                           const int *__restrict__ ei,
                           const int *__restrict__ node_graph,
                           const int *__restrict__ rowptr,
                           const int *__restrict__ srcptr,
                           int *__restrict__ cnt_in, int *__restrict__ cnt_out,
                           int *__restrict__ csr_eid, int *__restrict__ tmp_out) {
  const int N = dims->N, E = dims->E;
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= E) return;
  const int s = ei[k], d = ei[E + k];
  if (!edge_ok(s, d, N, node_graph)) return;
  csr_eid[rowptr[d] + atomicAdd(&cnt_in[d], 1)] = k;
  tmp_out[srcptr[s] + atomicAdd(&cnt_out[s], 1)] = k;
}

// Segments of at most kRegSort entries (every molecular graph's) are
// sorted in registers: their entries are loaded at once and put in order by
// a fixed network of compare-exchanges, so a segment costs a few rounds of
// independent loads.  Longer segments take an insertion sort in place.
constexpr int kRegSort = 8;

template <typename K> __device__ __forceinline__ void cswap(K &a, K &b) {
  const K lo = a < b ? a : b, hi = a < b ? b : a;
  a = lo;
  b = hi;
}

// odd-even transposition sort of kRegSort keys (ascending)
template <typename K> __device__ __forceinline__ void sort_regs(K (&v)[kRegSort]) {
#pragma unroll
  for (int pass = 0; pass < kRegSort; ++pass)
#pragma unroll
    for (int a = pass & 1; a + 1 < kRegSort; a += 2) cswap(v[a], v[a + 1]);
}

// Per destination: order the segment by (source, edge id); write csr_src,
// the inverse map and the edge attributes in CSR order.
__global__ void k_csr_sort_in(const Dims *__restrict__ dims,
                              const int *__restrict__ ei,
                              const int *__restrict__ rowptr,
                              int *__restrict__ csr_eid, int *__restrict__ csr_src,
                              int *__restrict__ csr_dst, int *__restrict__ csr_pos,
                              const float *__restrict__ edge_attr, int Fe,
                              float *__restrict__ csr_e, int max_degree,
                              int *__restrict__ err) {
  const int N = dims->N;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  const int lo = rowptr[i], hi = rowptr[i + 1], n = hi - lo;
  if (n <= kRegSort) {
    // key = source << 32 | edge id; empty slots sort last
    unsigned long long key[kRegSort];
    int k[kRegSort];
#pragma unroll
    for (int a = 0; a < kRegSort; ++a) k[a] = a < n ? csr_eid[lo + a] : 0;
#pragma unroll
    for (int a = 0; a < kRegSort; ++a)
      key[a] = a < n ? ((unsigned long long)(unsigned)ei[k[a]] << 32) | (unsigned)k[a]
                     : ~0ull;
    sort_regs(key);
    bool finite = true;
#pragma unroll
    for (int a = 0; a < kRegSort; ++a)
      if (a < n) {
        const int ka = (int)(unsigned)(key[a] & 0xffffffffu);
        csr_eid[lo + a] = ka;
        csr_src[lo + a] = (int)(key[a] >> 32);
        csr_dst[lo + a] = i;
        csr_pos[ka] = lo + a;
        for (int f = 0; f < Fe; ++f) {
          const float v = edge_attr[(size_t)ka * Fe + f];
          finite = finite && isfinite(v);
          csr_e[(size_t)(lo + a) * Fe + f] = v;
        }
      }
    if (!finite) atomicOr(err, ERR_NONFINITE);
    return;
  }
  if (n <= max_degree) {
    for (int a = lo + 1; a < hi; ++a) { // insertion sort by (src, eid)
      const int ka = csr_eid[a];
      const int sa = ei[ka];
      int b = a - 1;
      while (b >= lo) {
        const int kb = csr_eid[b];
        const int sb = ei[kb];
        if (sb < sa || (sb == sa && kb < ka)) break;
        csr_eid[b + 1] = kb;
        --b;
      }
      csr_eid[b + 1] = ka;
    }
  }
  for (int q = lo; q < hi; ++q) {
    const int k = csr_eid[q];
    csr_src[q] = ei[k];
    csr_dst[q] = i;
    csr_pos[k] = q;
  }
  bool finite = true;
  for (int q = lo; q < hi; ++q) {
    const int k = csr_eid[q];
    for (int f = 0; f < Fe; ++f) {
      const float v = edge_attr[(size_t)k * Fe + f];
      finite = finite && isfinite(v);
      csr_e[(size_t)q * Fe + f] = v;
    }
  }
  if (!finite) atomicOr(err, ERR_NONFINITE);
}

// Per source: CSR positions of its out-edges, ascending.
__global__ void k_csr_sort_out(const Dims *__restrict__ dims,
                               const int *__restrict__ srcptr,
                               const int *__restrict__ tmp_out,
                               const int *__restrict__ csr_pos,
                               int *__restrict__ t2csr, int max_degree) {
  const int N = dims->N;
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= N) return;
  const int lo = srcptr[j], hi = srcptr[j + 1], n = hi - lo;
  if (n <= kRegSort) {
    int k[kRegSort];
    unsigned v[kRegSort];
#pragma unroll
    for (int a = 0; a < kRegSort; ++a) k[a] = a < n ? tmp_out[lo + a] : 0;
#pragma unroll
    for (int a = 0; a < kRegSort; ++a) v[a] = a < n ? (unsigned)csr_pos[k[a]] : ~0u;
    sort_regs(v);
#pragma unroll
    for (int a = 0; a < kRegSort; ++a)
      if (a < n) t2csr[lo + a] = (int)v[a];
    return;
  }
  for (int p = lo; p < hi; ++p) t2csr[p] = csr_pos[tmp_out[p]];
  if (n > max_degree) return;
  for (int a = lo + 1; a < hi; ++a) {
    const int va = t2csr[a];
    int b = a - 1;
    while (b >= lo && t2csr[b] > va) {
      t2csr[b + 1] = t2csr[b];
      --b;
    }
    t2csr[b + 1] = va;
  }
}

__global__ void k_pad_copy(const Dims *__restrict__ dims, const float *__restrict__ x,
                           int F, float *__restrict__ xp, int Fp) {
  const int N = dims->N;
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const int i = (int)(t / Fp), c = (int)(t % Fp);
  if (i >= N) return;
  xp[t] = c < F ? x[(size_t)i * F + c] : 0.0f;
}

// The whole build in one launch, for batches whose nodes and edges fit a
// workgroup's LDS and 16 bits.  The chain of kernels above costs its launches
// (2 to 5 us each, every one waiting for the last) and not its work: with the
// launch that clears the error words 20 us for one molecule (25 nodes), 26 at
// 1.1k nodes and 2.3k edges, 31 at 4.5k and 9.3k; this kernel 6, 10 and 16.
//
// Every workgroup reads all edges and counts all in-degrees (the offsets and
// degree buckets of its nodes need them), then writes the CSR of its own nodes:
// a run of whole graphs, so that no edge of another workgroup touches them.
// What is repeated is bound by one CU's loads and LDS (10 of the 16 us); one
// workgroup alone takes 41 us at 4.5k nodes, most of it in the scattered
// stores.  The code runs once per launch, so it is fetched rather than bound
// by its instructions: loops are kept rolled (unrolled over 12 edges a thread
// in registers it took 5 us longer).
//
// LDS counters, the in-degree in the low and the out-degree in the high half
// of a word, become both prefix sums in one scan of the packed words, and then
// cursors that place the own edges.  An edge's place in its segment is the
// number of smaller keys there ((source, edge id) by destination; CSR position
// by source): the order of the chain's per-segment sorts.
//
// Workgroups past the first `parts` only copy the padded input.  Every
// workgroup stores an error word of its own and the first one clears the rest,
// so that no launch has to come before.
struct CsrSmall {
  Dims *dims;
  int set, B, N, E; // set: B, N, E hold and are written to dims; else read there
  int parts, step;  // workgroups that build, and about the nodes each has
  const int *graph_ptr, *ei;
  const float *edge_attr;
  int Fe, max_degree;
  const float *table;
  CsrBufs c;
  const float *x;
  int F;
  float *xpad;
  int Fp;
};

typedef int i4 __attribute__((ext_vector_type(4)));

// padded input, four lanes to a row, from row t0 / 4 on: whether all are finite
__device__ __forceinline__ bool pad_rows(const CsrSmall &a, int N, int t0, int nt) {
  bool finite = true;
#pragma unroll 1
  for (int r = t0 >> 2; r < N; r += nt >> 2) {
    const float *xr = a.x + (size_t)r * a.F;
#pragma unroll 1
    for (int c0 = 4 * (t0 & 3); c0 < a.Fp; c0 += 16) {
      f4 v;
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = c0 + k < a.F ? xr[c0 + k] : 0.f;
      finite = finite && isfinite(v[0]) && isfinite(v[1]) && isfinite(v[2]) && isfinite(v[3]);
      *reinterpret_cast<f4 *>(a.xpad + (size_t)r * a.Fp + c0) = v;
    }
  }
  return finite;
}

// Inclusive scans over a wave by DPP (row shifts, then the last lane of a row
// into the rows above it): no LDS traffic, which bounds this kernel.
template <int CTRL, int ROWS> __device__ __forceinline__ unsigned dpp0(unsigned v) {
  return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ unsigned wave_add_scan(unsigned v) {
  v += dpp0<0x111, 0xf>(v);
  v += dpp0<0x112, 0xf>(v);
  v += dpp0<0x114, 0xf>(v);
  v += dpp0<0x118, 0xf>(v);
  v += dpp0<0x142, 0xa>(v); // lane 15 of rows 0 and 2 into rows 1 and 3
  v += dpp0<0x143, 0xc>(v); // lane 31 into rows 2 and 3
  return v;
}

template <int T, int CAPN, int CAPE>
__global__ void __launch_bounds__(T) k_csr_small(const CsrSmall a) {
  constexpr int W = T / 64, U = 2;
  __shared__ unsigned s_ptr[CAPN + 1];     // packed degrees, then packed rowptr | srcptr << 16
  __shared__ unsigned short s_graph[CAPN]; // node -> graph
  // 10 bytes an edge: first the endpoints as loaded and graph_ptr, later
  __shared__ __attribute__((aligned(16))) unsigned s_edge[CAPE * 5 / 2];
  unsigned *s_key = s_edge; // source << 16 | edge id, by CSR position
  // by CSR position, unordered in a segment: its destination; by source,
  // unordered: CSR positions, and the source of each
  unsigned short *s_dst = reinterpret_cast<unsigned short *>(s_edge + CAPE);
  unsigned short *s_out = s_dst + CAPE, *s_src = s_out + CAPE;
  int *s_es = reinterpret_cast<int *>(s_edge), *s_gp = s_es + 2 * CAPE;
  __shared__ unsigned s_w[W];
  __shared__ int s_bw[W][kMaxBuckets], s_tot[kMaxBuckets], s_bef[kMaxBuckets];
  __shared__ int s_err, s_lo, s_hi, s_base, s_total;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int N = a.set ? a.N : a.dims->N;
  const bool alone = gridDim.x == 1;
  const int part = blockIdx.x;
  if (part >= a.parts) {
    const bool fin = pad_rows(a, N, (part - a.parts) * T + tid, ((int)gridDim.x - a.parts) * T);
    const int bits = __syncthreads_or(!fin) ? ERR_NONFINITE : 0;
    if (tid == 0) a.c.err[blockIdx.x] = bits;
    return;
  }
  const int B = a.set ? a.B : a.dims->B, E = a.set ? a.E : a.dims->E;
  const int nb = a.c.nb;
  const int *s_ed = s_es + E;
  // both rows of the edge list, as one run of 2 E words
  constexpr int V = CAPE / (2 * T);
  i4 ev[V];
#pragma unroll
  for (int u = 0; u < V; ++u) {
    const int k = 4 * (tid + u * T);
    if (k + 4 <= 2 * E) ev[u] = *reinterpret_cast<const i4 *>(a.ei + k);
  }
  if (tid < (2 * E & 3)) s_es[(2 * E & ~3) + tid] = a.ei[(2 * E & ~3) + tid];
#pragma unroll 1
  for (int k = tid; k <= B; k += T) s_gp[k] = a.graph_ptr[k];
#pragma unroll 1
  for (int i = tid; i < N; i += T) {
    s_ptr[i] = 0;
    s_graph[i] = 0;
  }
  if (tid < kMaxBuckets) s_tot[tid] = s_bef[tid] = 0;
  if (tid == 0) {
    s_err = s_base = s_total = 0;
    s_lo = part ? N : 0;
    s_hi = N;
    if (a.set && part == 0) *a.dims = Dims{B, N, E, 0};
  }
  int bad = 0;
  if (alone && a.x && !pad_rows(a, N, tid, T)) bad |= ERR_NONFINITE;
#pragma unroll
  for (int u = 0; u < V; ++u) {
    const int k = 4 * (tid + u * T);
    if (k + 4 <= 2 * E) *reinterpret_cast<i4 *>(s_es + k) = ev[u];
  }
  __syncthreads();

  // own nodes: from the first graph that begins at or after part step to the
  // next part's; node -> graph, eight lanes to a graph
#pragma unroll 1
  for (int b = tid; b <= B; b += T) {
    const int g = s_gp[b], g1 = b ? s_gp[b - 1] : -1;
    if (g1 >= g || (b == 0 && g != 0) || (b == B && g != N)) bad |= ERR_GRAPH_PTR;
    const int t_lo = part * a.step, t_hi = t_lo + a.step;
    if (part && g1 < t_lo && g >= t_lo) s_lo = g;
    if (g1 < t_hi && g >= t_hi) s_hi = g;
  }
#pragma unroll 1
  for (int b = tid >> 3; b < B; b += T / 8) {
    const int i0 = max(s_gp[b], 0), i1 = min(s_gp[b + 1], N);
#pragma unroll 1
    for (int i = i0 + (tid & 7); i < i1; i += 8) s_graph[i] = (unsigned short)b;
  }
  // with a malformed graph_ptr no edge counts (and one workgroup owns all)
  const bool ok = !__syncthreads_or(bad & ERR_GRAPH_PTR);
  const int lo = ok ? s_lo : (part ? N : 0), hi = ok ? s_hi : N;

  // degrees: everyone's in-degree, own nodes' out-degree
  int total = 0, base = 0;
#pragma unroll 1
  for (int k = tid; k - tid < E; k += T) {
    const int s = s_es[k], d = s_ed[k];
    const bool in = s >= 0 && s < N && d >= 0 && d < N;
    bool live = k < E;
    if (live && !in) bad |= ERR_EDGE_RANGE;
    live = live && in && ok;
    if (live && s_graph[s] != s_graph[d]) {
      bad |= ERR_EDGE_CROSS;
      live = false;
    }
    if (live) {
      const bool own = d >= lo && d < hi;
      atomicAdd(&s_ptr[d], own && s == d ? 0x10001u : 1u);
      if (own && s != d) atomicAdd(&s_ptr[s], 1u << 16);
    }
    total += __popcll(__ballot(live));
    base += __popcll(__ballot(live && d < lo));
  }
  if (lane == 0) {
    atomicAdd(&s_total, total);
    atomicAdd(&s_base, base);
  }
  __syncthreads();

  // nodes of every degree, and those before the own ones (lane q: bucket q)
  if (nb) {
    // a lane's nodes of bucket q in bits 4 q of h, those before in hb (at most
    // CAPN / T = 6 a lane)
    static_assert(CAPN / T < 16, "four bits a bucket");
    unsigned long long h = 0, hb = 0;
#pragma unroll 1
    for (int i = tid; i < N; i += T) {
      const unsigned long long one =
          1ull << (4 * bucket_of((int)(s_ptr[i] & 0xffffu), a.max_degree));
      h += one;
      hb += i < lo ? one : 0ull;
    }
#pragma unroll 1
    for (int q = 0; q < nb; ++q) {
      const unsigned both = wave_add_scan((unsigned)(h & 15u) | (unsigned)(hb & 15u) << 16);
      if (lane == 63) {
        atomicAdd(&s_tot[q], (int)(both & 0xffffu));
        atomicAdd(&s_bef[q], (int)(both >> 16));
      }
      h >>= 4;
      hb >>= 4;
    }
    __syncthreads();
  }
  // lane q: the first row of bucket q
  const int bt = lane < nb ? s_tot[lane] : 0;
  const int brow = (int)wave_add_scan((unsigned)bt) - bt;
  if (part == 0) {
    if (wid == 0 && nb && lane <= nb) a.c.brow[lane] = brow;
    if (tid == 0) a.c.rowptr[N] = a.c.srcptr[N] = s_total;
  }

  // own nodes' offsets
  unsigned carry = (unsigned)s_base * 0x10001u;
#pragma unroll 1
  for (int i0 = lo; i0 < hi; i0 += T) {
    const int i = i0 + tid;
    const unsigned deg = i < hi ? s_ptr[i] : 0u;
    const unsigned inc = wave_add_scan(deg);
    const int vi = (int)(deg & 0xffffu), vo = (int)(deg >> 16);
    const int bq = i < hi ? bucket_of(vi, a.max_degree) : -1;
    int rank = 0, count = 0;
#pragma unroll 1
    for (int q = 0; q < nb; ++q) {
      const unsigned long long m = __ballot(bq == q);
      if (lane == q) count = __popcll(m);
      if (bq == q) rank = __popcll(m & ((1ull << lane) - 1ull));
    }
    if (lane < nb) s_bw[wid][lane] = count;
    if (lane == 63) s_w[wid] = inc;
    __syncthreads();
    const unsigned tot = lane < W ? s_w[lane] : 0u; // lane w: wave w's sum
    const unsigned upto = wave_add_scan(tot);
    const unsigned before = (unsigned)__builtin_amdgcn_readlane((int)(upto - tot), wid);
    const unsigned all = (unsigned)__builtin_amdgcn_readlane((int)upto, 63);
    if (i < hi) {
      const unsigned ptr = carry + before + inc - deg;
      s_ptr[i] = ptr;
      a.c.node_graph[i] = s_graph[i];
      a.c.rowptr[i] = (int)(ptr & 0xffffu);
      a.c.srcptr[i] = (int)(ptr >> 16);
      a.c.deg[i] = vi;
      a.c.sp[i] = a.table[2 * bq];
      a.c.sm[i] = a.table[2 * bq + 1];
      if (vi > a.max_degree || vo > a.max_degree) bad |= ERR_DEGREE;
    }
    if (nb) {
      int p = __shfl(brow, bq < 0 ? 0 : bq, 64) + rank;
      if (i < hi) {
        p += s_bef[bq];
#pragma unroll 1
        for (int w = 0; w < wid; ++w) p += s_bw[w][bq];
        a.c.perm[p] = i;
      }
    }
    carry += all;
    __syncthreads();
    if (nb && i0 + T < hi) { // the next nodes' bucket places
      if (tid < nb)
#pragma unroll 1
        for (int w = 0; w < W; ++w) s_bef[tid] += s_bw[w][tid];
      __syncthreads();
    }
  }
  if (tid == 0) s_ptr[hi] = carry; // past the own nodes: degrees no longer needed
  __syncthreads();
  const int p_lo = s_base, p_hi = (int)(s_ptr[hi] & 0xffffu);

  // place the own edges: the low half of s_ptr counts up to the segment's end
  if (p_hi > p_lo) {
#pragma unroll 1
    for (int k0 = tid; k0 - tid < E; k0 += U * T) {
      int s[U], d[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = min(k0 + u * T, E - 1);
        s[u] = a.ei[k];
        d[u] = a.ei[E + k];
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (k0 + u * T < E && d[u] >= lo && d[u] < hi && s[u] >= lo && s[u] < hi &&
            s_graph[s[u]] == s_graph[d[u]]) {
          const unsigned p = atomicAdd(&s_ptr[d[u]], 1u) & 0xffffu;
          s_key[p] = (unsigned)s[u] << 16 | (unsigned)(k0 + u * T);
          s_dst[p] = (unsigned short)d[u];
        }
    }
  }
  __syncthreads();
  // order the segments; s_ptr[d] now holds a segment's end, and the one before
  // it its begin.  Longer ones than max_degree (an error) stay unordered.
#pragma unroll 1
  for (int p = p_lo + tid; p < p_hi; p += T) {
    const unsigned key = s_key[p];
    const int d = s_dst[p], k = (int)(key & 0xffffu), s = (int)(key >> 16);
    const int p0 = d > lo ? (int)(s_ptr[d - 1] & 0xffffu) : p_lo;
    const int n = (int)(s_ptr[d] & 0xffffu) - p0;
    int pos = p;
    if (n <= a.max_degree) {
      pos = p0;
#pragma unroll 1
      for (int j = 0; j < n; ++j) pos += s_key[p0 + j] < key;
    }
    a.c.csr_eid[pos] = k;
    a.c.csr_src[pos] = s;
    a.c.csr_dst[pos] = d;
#pragma unroll 1
    for (int f = 0; f < a.Fe; ++f) {
      const float v = a.edge_attr[(size_t)k * a.Fe + f];
      if (!isfinite(v)) bad |= ERR_NONFINITE;
      a.c.csr_e[(size_t)pos * a.Fe + f] = v;
    }
    const unsigned q = atomicAdd(&s_ptr[s], 1u << 16) >> 16;
    s_out[q] = (unsigned short)pos;
    s_src[q] = (unsigned short)s;
  }
  __syncthreads();
#pragma unroll 1
  for (int q = p_lo + tid; q < p_hi; q += T) {
    const int pos = s_out[q], s = s_src[q];
    const int q0 = s > lo ? (int)(s_ptr[s - 1] >> 16) : p_lo;
    const int n = (int)(s_ptr[s] >> 16) - q0;
    int r = q;
    if (n <= a.max_degree) {
      r = q0;
#pragma unroll 1
      for (int j = 0; j < n; ++j) r += (int)s_out[q0 + j] < pos;
    }
    a.c.t2csr[r] = pos;
  }
  if (bad) atomicOr(&s_err, bad);
  __syncthreads();
  if (tid == 0) a.c.err[blockIdx.x] = s_err;
  if (part == 0 && tid < kErrWords && tid >= (int)gridDim.x) a.c.err[tid] = 0;
}

// Batches the one-launch build takes, by capacity: 0 none, 1 with 256 threads
// (16-wave barriers and their launch cost a molecule 3 us more), 2 with 1024.
inline int small_class(int B, int N, int E) {
  if (N <= 256 && E <= 512 && B < 256) return 1;
  if (N <= 6144 && E <= 12288 && B < 6144) return 2;
  return 0;
}

inline int cdiv(long long a, int b) { return (int)((a + b - 1) / b); }

} // namespace

hipError_t launch_csr_build(Dims *dims, bool set, int capB, int capN, int capE,
                            const int *graph_ptr, const int *edge_index,
                            const float *edge_attr, int Fe, int max_degree,
                            const float *table, const CsrBufs &c,
                            const float *x, int F, float *xpad, int Fp, hipStream_t s) {
  // Fp is a multiple of 16 (whole 16-byte groups per padded row)
  if (x && Fp % 16) return hipErrorInvalidValue;
  const long long pad = x ? (long long)capN * (Fp / 4) : 0;
  const bool al16 = ((uintptr_t)edge_index & 15) == 0; // its rows are read 16 bytes at a time
  if (const int cls = al16 ? small_class(capB, capN, capE) : 0) {
    // up to 1024 edges one workgroup (nothing to split: 6 to 8 us), which also
    // pads a small input; above, one per 512 edges (per 256 and per 1024 within
    // 1.2 us of it from 2.3k to 9.6k edges)
    const int T = cls == 1 ? 256 : 1024;
    const int parts = capE <= 1024 ? 1 : cdiv(capE, 512);
    const bool alone = parts == 1 && pad <= 4 * T;
    const CsrSmall a{dims, set, capB, capN, capE, parts, cdiv(capN, parts), graph_ptr, edge_index, edge_attr, Fe,
                     max_degree, table, c, x, F, xpad, Fp};
    const dim3 grid(alone ? 1 : std::min<int>(kErrWords, parts + cdiv(pad, T)));
    if (cls == 1) k_csr_small<256, 256, 512><<<grid, 256, 0, s>>>(a);
    else k_csr_small<1024, 6144, 12288><<<grid, 1024, 0, s>>>(a);
    return hipGetLastError();
  }
  k_set_dims<<<1, kErrWords, 0, s>>>(set ? dims : nullptr, capB, capN, capE, c.err);
  long long nt = capN > capB ? capN : capB;
  if (x && (long long)capN * (Fp / 4) > nt) nt = (long long)capN * (Fp / 4);
  k_csr_init<<<cdiv(nt > 0 ? nt : 1, kInitThreads), kInitThreads, 0, s>>>(
      dims, graph_ptr, c.node_graph, c.cnt_in, c.cnt_out, c.err, x, F, xpad, Fp);
  if (capE > 0)
    k_csr_count<<<cdiv(capE, 256), 256, 0, s>>>(dims, edge_index, c.node_graph,
                                                c.cnt_in, c.cnt_out, c.err);
  {
    const int nsb = cdiv(capN > 0 ? capN : 1, kScanNodes);
    const int fused = nsb <= kScanFuse;
    k_scan_count<<<nsb, 256, 0, s>>>(dims, c.cnt_in, c.cnt_out, max_degree, c.nb, c.scan);
    if (!fused)
      k_scan_top<<<1, kScanTop, 0, s>>>(dims, c.nb, c.scan, c.brow, c.rowptr, c.srcptr);
    k_scan_apply<<<nsb, 256, 0, s>>>(dims, c.cnt_in, c.cnt_out, c.scan, table, max_degree,
                                     c.nb, c.rowptr, c.srcptr, c.deg, c.sp, c.sm, c.perm,
                                     c.brow, c.err, fused);
  }
  if (capE > 0)
    k_csr_fill<<<cdiv(capE, 256), 256, 0, s>>>(dims, edge_index, c.node_graph, c.rowptr,
                                               c.srcptr, c.cnt_in, c.cnt_out, c.csr_eid,
                                               c.tmp_out);
  if (capN > 0) {
    k_csr_sort_in<<<cdiv(capN, 128), 128, 0, s>>>(dims, edge_index, c.rowptr, c.csr_eid,
                                                  c.csr_src, c.csr_dst, c.csr_pos, edge_attr, Fe,
                                                  c.csr_e, max_degree, c.err);
    k_csr_sort_out<<<cdiv(capN, 128), 128, 0, s>>>(dims, c.srcptr, c.tmp_out, c.csr_pos,
                                                   c.t2csr, max_degree);
  }
  return hipGetLastError();
}

hipError_t launch_pad_copy(const Dims *dims, int capN, const float *x, int F,
                           float *xp, int Fp, hipStream_t s) {
  if (capN <= 0) return hipSuccess;
  k_pad_copy<<<cdiv((long long)capN * Fp, 256), 256, 0, s>>>(dims, x, F, xp, Fp);
  return hipGetLastError();
}

} // namespace hgnn
