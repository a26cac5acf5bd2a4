// Steps S4 and S5: global mean pooling over each graph's nodes (Section 3.1),
// the fully connected head Linear(H,H)-ReLU-Linear(H,1), the MSE loss
// (Section 3.2) and their adjoint; generalised to several graph-level heads
// and to node-level heads (HydraGNN's multi-headed outputs) with a weighted
// sum of the heads' losses.  One workgroup per graph; every reduction
// runs in a fixed order, so results are deterministic and a graph's
// prediction does not depend on the other graphs of the batch.
#include "common.hpp"

namespace hgnn {

namespace {

inline int cdiv(long long a, int b) { return (int)((a + b - 1) / b); }
constexpr int kHeadThreads = 256;
// the graph part of the head adjoint: one workgroup per graph, whose time is
// the latency of its dg = W1^T dq sums (split into P = threads / H ordered
// partial ranges) and of its nodes' stores; 512 threads halve the ranges
// (C1 step 184.5k -> 185.9k graphs/s)
constexpr int kHeadBwdThreads = 512;
constexpr int kMaxGraphHeads = 8;

// Node range of graph b, clamped to [0, N] so that an unvalidated malformed
// graph_ptr (reported through the error word) never leads out of bounds.
__device__ __forceinline__ void graph_range(const int *gptr, int b, int N, int &lo, int &hi) {
  lo = min(max(gptr[b], 0), N);
  hi = min(max(gptr[b + 1], lo), N);
}

// Fixed-shape tree reduction over a workgroup of NT threads (deterministic).
template <int NT = kHeadThreads>
__device__ float block_sum(float v, float *red) {
  const int tid = threadIdx.x;
  red[tid] = v;
  __syncthreads();
  for (int s = NT / 2; s > 0; s >>= 1) {
    if (tid < s) red[tid] += red[tid + s];
    __syncthreads();
  }
  const float r = red[0];
  __syncthreads();
  return r;
}

// Graph head t of Tg (blockIdx.y): head weights at wh + t (H^2 + 2H + 1) as
// W1 [H, H], b1 [H], w2 [H], b2 [1]; q of head t at q + (t B + b) H; the
// prediction goes to pred[b Tg + t].  W1T (nullable): the staged transposes
// [Tg][H][H] of the W1s, read along the threads' outputs (coalesced); the
// sums run over k in the same order either way.
// 512 threads: thread (p, c) takes feature c and the p-th of P = 512 / H
// ranges of the graph's nodes (pooling) and of k (the W1 product); the P
// partial sums are added in order through LDS.  One thread per feature left
// half of a 256-thread workgroup idle at H = 128 and walked all H rows of W1
// in one chain.
// G graphs a workgroup (1, 2 or 4) share each W1 value read: at 1024 graphs and
// H = 256 one graph a workgroup reads 268 MB of W1 from L2 (23 us, 44 with
// untransposed rows), four a quarter of it (16.6).  All G are pooled at once, 16
// bytes a lane.
constexpr int kHeadFwdThreads = 512;

// four values at p, 16-byte aligned if vec
__device__ __forceinline__ f4 load4(const float *p, bool vec) {
  if (vec) return *reinterpret_cast<const f4 *>(p);
  return f4{p[0], p[1], p[2], p[3]};
}

template <int G>
__global__ void __launch_bounds__(kHeadFwdThreads)
k_head_forward(const Dims *__restrict__ dims, int H, int Tg, const int *__restrict__ gptr,
               const float *__restrict__ h, int vec, const float *__restrict__ wh,
               const float *__restrict__ W1T, float *__restrict__ g, float *__restrict__ q,
               float *__restrict__ pred, float *__restrict__ pred2) {
  constexpr int NT = kHeadFwdThreads;
  __shared__ __attribute__((aligned(16))) float gs[512][G];
  __shared__ __attribute__((aligned(16))) float red[G * NT];
  __shared__ float inv_n[G];
  const int b0 = blockIdx.x * G, t = blockIdx.y;
  const int B = dims->B;
  if (b0 >= B) return;
  const float *W1 = wh + (size_t)t * (H * H + 2 * H + 1);
  const float *b1 = W1 + H * H, *w2 = b1 + H, *b2 = w2 + H;
  const int P = NT / H; // H <= 512
  const int tid = threadIdx.x, c = tid % H, p = tid / H;
  const bool act = p < P;
  // pooling.  One graph: range p, feature c; several: range pp of graph j,
  // features 4 cq .. (the divisions that find them cost one graph 1 us)
  if constexpr (G == 1) {
    int lo, hi;
    graph_range(gptr, b0, dims->N, lo, hi);
    const int R = (hi - lo + P - 1) / P;
    const int i0 = min(lo + p * R, hi), i1 = min(i0 + R, hi);
    float s = 0.f;
    if (act) {
#pragma unroll 8
      for (int i = i0; i < i1; ++i) s += h[(size_t)i * H + c];
    }
    red[tid] = s;
    if (tid == 0) inv_n[0] = 1.0f / (float)(hi - lo);
  } else {
    const int nq = H / 4, cq = tid % nq, j = tid / nq / P, pp = tid / nq % P;
    if (j < G) {
      f4 s = {0.f, 0.f, 0.f, 0.f};
      int lo = 0, hi = 0;
      if (b0 + j < B) graph_range(gptr, b0 + j, dims->N, lo, hi);
      const int R = (hi - lo + P - 1) / P;
      const int i0 = min(lo + pp * R, hi), i1 = min(i0 + R, hi);
#pragma unroll 8
      for (int i = i0; i < i1; ++i) s += load4(h + (size_t)i * H + 4 * cq, vec);
      *reinterpret_cast<f4 *>(red + (j * P + pp) * H + 4 * cq) = s;
      if (cq == 0 && pp == 0) inv_n[j] = 1.0f / (float)(hi - lo);
    }
  }
  __syncthreads();
  for (int e = tid; e < G * H; e += NT) {
    const int j = G == 1 ? 0 : e / H, cc = G == 1 ? c : e % H; // G = 1: e = tid < H
    float s = red[j * P * H + cc];
    for (int k = 1; k < P; ++k) s += red[(j * P + k) * H + cc];
    const float gv = s * inv_n[j];
    gs[cc][j] = gv;
    if (t == 0 && b0 + j < B) g[(size_t)(b0 + j) * H + cc] = gv;
  }
  __syncthreads();
  // the W1 product over k = p RK ..
  {
    const int RK = (H + P - 1) / P;
    const int k0 = min(p * RK, H), k1 = min(k0 + RK, H);
    float s[G] = {};
    if (G > 1 && !W1T) {
      // W1 as stored, 16 columns of every range at a time through LDS: its rows
      // read by the threads' outputs took 44 us, this 26 (transposed rows, where the
      // context holds them, 17)
      constexpr int KC = 16, U = KC;
      __shared__ float tile[G > 1 ? NT : 1][KC + 1];
      int at[U]; // element u of a chunk: row (range, feature) r, column kk
      const int kk = tid & (KC - 1);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int r = (tid >> 4) + u * (NT / KC), rp = r / H;
        at[u] = rp < P ? (r - rp * H) * H + min(rp * RK, H) + kk : -1;
      }
      for (int d = 0; d < RK; d += KC) {
        float v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = W1[min(max(at[u], 0) + d, H * H - 1)];
        __syncthreads(); // the last chunk is read
#pragma unroll
        for (int u = 0; u < U; ++u) tile[(tid >> 4) + u * (NT / KC)][kk] = v[u];
        __syncthreads();
        if (act)
          for (int k = 0; k < KC && k0 + d + k < k1; ++k) {
            const float wv = tile[p * H + c][k];
#pragma unroll
            for (int j = 0; j < G; ++j) s[j] += wv * gs[k0 + d + k][j];
          }
      }
    } else if (act && W1T) {
      const float *w = W1T + (size_t)t * H * H + c;
#pragma unroll 8
      for (int k = k0; k < k1; ++k) {
        const float wv = w[(size_t)k * H];
#pragma unroll
        for (int j = 0; j < G; ++j) s[j] += wv * gs[k][j];
      }
    } else if (act) { // one graph: a row of W1 as stored, consecutive loads (16 bytes
      // each; one loop for both strides loads 4: H = 400, 21 graphs, 42 -> 92 us
      // forward and backward)
      const float *w = W1 + (size_t)c * H;
#pragma unroll 8
      for (int k = k0; k < k1; ++k) s[0] += w[k] * gs[k][0];
    }
#pragma unroll
    for (int j = 0; j < G; ++j) red[j * NT + tid] = s[j]; // the last reads were before a barrier
  }
  __syncthreads();
  float part[G];
#pragma unroll
  for (int j = 0; j < G; ++j) {
    part[j] = 0.f;
    if (p == 0) {
      float s = b1[c];
      for (int k = 0; k < P; ++k) s += red[j * NT + k * H + c];
      const float qv = s > 0.f ? s : 0.f;
      if (b0 + j < B) q[((size_t)t * B + b0 + j) * H + c] = qv;
      part[j] = w2[c] * qv;
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < G; ++j) red[j * NT + tid] = part[j];
  __syncthreads();
  // block_sum's tree, of the G graphs together
  for (int lg = 8; lg >= 0; --lg) {
    static_assert(NT == 2 << 8, "the tree's first level");
    for (int e = tid; e < G << lg; e += NT) {
      const int at = (e >> lg) * NT + (e & ((1 << lg) - 1));
      red[at] += red[at + (1 << lg)];
    }
    __syncthreads();
  }
  if (tid < G && b0 + tid < B) {
    const float y = red[tid * NT] + b2[0];
    pred[(size_t)(b0 + tid) * Tg + t] = y;
    if (pred2) pred2[(size_t)(b0 + tid) * Tg + t] = y;
  }
}

// loss = sum_t gw_t mean_b (pred - y)^2 + sum_s nw_s mean_i (z - z_target)^2,
// each mean a fixed-order workgroup sum (weights default to 1).
__global__ void __launch_bounds__(kHeadThreads)
k_loss(const Dims *__restrict__ dims, int Tg, const float *__restrict__ pred,
       const float *__restrict__ t, const float *__restrict__ gw, int Tn,
       const float *__restrict__ z, const float *__restrict__ zt,
       const float *__restrict__ nw, float *__restrict__ loss) {
  __shared__ float red[kHeadThreads];
  const int B = dims->B, N = dims->N;
  float acc = 0.f;
  for (int k = 0; k < Tg; ++k) {
    float s = 0.f;
    for (int b = threadIdx.x; b < B; b += kHeadThreads) {
      const float d = pred[(size_t)b * Tg + k] - t[(size_t)b * Tg + k];
      s += d * d;
    }
    acc += (gw ? gw[k] : 1.0f) * (block_sum(s, red) / (float)B);
  }
  for (int k = 0; k < Tn; ++k) {
    float s = 0.f;
#pragma unroll 8
    for (int i = threadIdx.x; i < N; i += kHeadThreads) {
      const float d = z[(size_t)i * Tn + k] - zt[(size_t)i * Tn + k];
      s += d * d;
    }
    acc += (nw ? nw[k] : 1.0f) * (block_sum(s, red) / (float)N);
  }
  if (threadIdx.x == 0) *loss = acc;
}

// Per graph, for every graph head t: dy, dq_t = dy w2_t * [q_t > 0]; then
// dg = sum_t W1_t^T dq_t and dh_i = dg / n_b (+ add_i, the node heads' share),
// masked by relu_of > 0 when given.  The sums over c are split into P
// contiguous ranges (P = 512 / H threads per output) whose
// partials are added in range order.
// G graphs a workgroup (more than one with a single head) share each W1 value
// (1024 graphs, H = 256, 40k nodes: 27 -> 18 us, of which 8 store dh).
template <int G>
__global__ void __launch_bounds__(kHeadBwdThreads)
k_head_bwd_graph(const Dims *__restrict__ dims, int H, int Tg, const int *__restrict__ gptr,
                 const float *__restrict__ wh, const float *__restrict__ q,
                 const float *__restrict__ pred, const float *__restrict__ target,
                 const float *__restrict__ dpred, const float *__restrict__ gw,
                 float *__restrict__ dy, float *__restrict__ dq, float *__restrict__ dh,
                 const float *__restrict__ relu_of, const float *__restrict__ add, int vec) {
  constexpr int NT = kHeadBwdThreads;
  // [head][feature][graph]
  __shared__ __attribute__((aligned(16))) float dqs[(G == 1 ? kMaxGraphHeads : 1) * 512][G];
  __shared__ float red[G * NT];
  __shared__ __attribute__((aligned(16))) float dgs[G][512];
  const int b0 = blockIdx.x * G, tid = threadIdx.x;
  const int B = dims->B;
  if (b0 >= B) return;
  const size_t HS = (size_t)H * H + 2 * H + 1;
  for (int t = 0; t < Tg; ++t) {
    for (int e = tid; e < G * H; e += NT) {
      const int j = G == 1 ? 0 : e / H, c = G == 1 ? e : e % H, b = b0 + j;
      float v = 0.f;
      if (b < B) {
        const size_t o = (size_t)b * Tg + t;
        const float dyb = dpred ? dpred[o]
                                : (2.0f * (pred[o] - target[o]) / (float)B) * (gw ? gw[t] : 1.0f);
        if (c == 0) dy[o] = dyb;
        const size_t at = ((size_t)t * B + b) * H + c;
        v = q[at] > 0.f ? dyb * wh[t * HS + H * H + H + c] : 0.f;
        dq[at] = v;
      }
      dqs[t * H + c][j] = v;
    }
  }
  __syncthreads();
  const int P = NT / H; // H <= 512
  const int k = tid % H, p = tid / H;
  if (p < P) {
    const int c0 = (p * H) / P, c1 = ((p + 1) * H) / P;
    float s[G] = {};
    for (int t = 0; t < Tg; ++t) {
      const float *W1 = wh + t * HS;
      auto add = [&](float wv, int c) {
#pragma unroll
        for (int j = 0; j < G; ++j) s[j] += wv * dqs[t * H + c][j];
      };
      int c = c0;
      for (; c + 16 <= c1; c += 16) { // 16 loads in flight
        float wv[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) wv[u] = W1[(size_t)(c + u) * H + k];
#pragma unroll
        for (int u = 0; u < 16; ++u) add(wv[u], c + u);
      }
#pragma unroll 8
      for (; c < c1; ++c) add(W1[(size_t)c * H + k], c);
    }
#pragma unroll
    for (int j = 0; j < G; ++j) red[j * NT + tid] = s[j];
  }
  __syncthreads();
  for (int e = tid; e < G * H; e += NT) {
    const int j = G == 1 ? 0 : e / H, kk = G == 1 ? e : e % H;
    float s = red[j * NT + kk];
    for (int u = 1; u < P; ++u) s += red[j * NT + u * H + kk];
    dgs[j][kk] = s;
  }
  __syncthreads();
  // dh of the nodes, 16 bytes a lane
  const int nq = H / 4, kq = tid % nq, row = tid / nq, rows = NT / nq;
#pragma unroll
  for (int j = 0; j < G; ++j) {
    if (b0 + j >= B) break;
    int lo, hi;
    graph_range(gptr, b0 + j, dims->N, lo, hi);
    const float inv_n = 1.0f / (float)(hi - lo);
    if (row >= rows) continue;
    const f4 dg = *reinterpret_cast<const f4 *>(&dgs[j][4 * kq]);
#pragma unroll 4
    for (int i = lo + row; i < hi; i += rows) {
      const size_t at = (size_t)i * H + 4 * kq;
      f4 o = dg * inv_n;
      if (add) o += load4(add + at, vec);
      // fold in the ReLU adjoint of the layer that produced h
      if (relu_of) {
        const f4 r = load4(relu_of + at, vec);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (!(r[e] > 0.f)) o[e] = 0.f;
      }
      if (vec) {
        *reinterpret_cast<f4 *>(dh + at) = o;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) dh[at + e] = o[e];
      }
    }
  }
}

// Head weight gradients, each a fixed-order sum over the graphs.
// Output layout (packed): dW1 [H, H], db1 [H], dw2 [H], db2 [1].  A
// workgroup owns 32 outputs; its 8 thread groups sum interleaved graphs and
// the 8 partial sums are added in a fixed order.
constexpr int kHeadOut = 32, kHeadParts = 8;

__global__ void __launch_bounds__(256)
k_head_bwd_weights(const Dims *__restrict__ dims, int H, int Tg, const float *__restrict__ g,
                   const float *__restrict__ qall, const float *__restrict__ dyall,
                   const float *__restrict__ dqall, float *__restrict__ outall) {
  __shared__ float red[kHeadParts][kHeadOut];
  const int o = threadIdx.x % kHeadOut, p = threadIdx.x / kHeadOut;
  const int t = blockIdx.x * kHeadOut + o;
  const int B = dims->B;
  const int n1 = H * H, total = n1 + 2 * H + 1;
  // graph head blockIdx.y: its q, dq, dy column and output block
  const int hd = blockIdx.y;
  const float *q = qall + (size_t)hd * B * H, *dq = dqall + (size_t)hd * B * H;
  float *out = outall + (size_t)hd * total;
  struct Col {
    const float *p;
    int s;
    __device__ float operator[](int b) const { return p[(size_t)b * s]; }
  } dy{dyall + hd, Tg};
  float s = 0.f;
  if (t < n1) {
    const int c = t / H, k = t % H;
    for (int b = p; b < B; b += kHeadParts) s += dq[(size_t)b * H + c] * g[(size_t)b * H + k];
  } else if (t < n1 + H) {
    const int c = t - n1;
    for (int b = p; b < B; b += kHeadParts) s += dq[(size_t)b * H + c];
  } else if (t < n1 + 2 * H) {
    const int c = t - n1 - H;
    for (int b = p; b < B; b += kHeadParts) s += dy[b] * q[(size_t)b * H + c];
  } else if (t < total) {
    for (int b = p; b < B; b += kHeadParts) s += dy[b];
  }
  red[p][o] = s;
  __syncthreads();
  if (p == 0 && t < total) {
    float acc = red[0][o];
    for (int j = 1; j < kHeadParts; ++j) acc += red[j][o];
    out[t] = acc;
  }
}

// The same gradients for large batches, in two launches.  The graphs are
// split into Z chunks of R = ceil(B / Z); k_head_w_part writes every
// output's sum over each chunk (P [Tg][Z][n], n = H^2 + 2H + 1) and
// k_head_w_sum adds the chunks in order.  dW1: a workgroup takes a 16 x 64
// block of (c, k) and walks its chunk 64 graphs at a time, the rows of dq
// and g staged in LDS (thread: one c, four k); db1, dw2 and db2 take one more
// workgroup per chunk (thread: one c, the chunk's graphs in order,
// eight loads in flight: one at a time they were the launch's 21 us, now 10).  The
// one-pass kernel above reads each g and dq value once per output.
constexpr int kHeadChunks = 16, kHeadTC = 16, kHeadTK = 64, kHeadRows = 64;
constexpr int kHeadChunkedMinB = 512;

__global__ void __launch_bounds__(256)
k_head_w_part(const Dims *__restrict__ dims, int H, int Tg, int Z, const float *__restrict__ g,
              const float *__restrict__ qall, const float *__restrict__ dyall,
              const float *__restrict__ dqall, float *__restrict__ Pall) {
  __shared__ float sdq[kHeadRows][kHeadTC];
  __shared__ f4 sg[kHeadRows][kHeadTK / 4];
  const int B = dims->B, n1 = H * H, n = n1 + 2 * H + 1;
  const int hd = blockIdx.z, z = blockIdx.y;
  const float *q = qall + (size_t)hd * B * H, *dq = dqall + (size_t)hd * B * H;
  float *P = Pall + ((size_t)hd * Z + z) * n;
  const int R = (B + Z - 1) / Z, b_lo = min(z * R, B), b_hi = min(b_lo + R, B);
  const int ntk = (H + kHeadTK - 1) / kHeadTK, tiles = (H / kHeadTC) * ntk;
  const int t = threadIdx.x;
  if ((int)blockIdx.x == tiles) { // db1, dw2, db2 over this chunk
    for (int c = t; c < H; c += 256) {
      float s1 = 0.f, s2 = 0.f;
#pragma unroll 8
      for (int b = b_lo; b < b_hi; ++b) {
        s1 += dq[(size_t)b * H + c];
        s2 += dyall[(size_t)b * Tg + hd] * q[(size_t)b * H + c];
      }
      P[n1 + c] = s1;
      P[n1 + H + c] = s2;
    }
    if (t == 0) {
      float s3 = 0.f;
#pragma unroll 8
      for (int b = b_lo; b < b_hi; ++b) s3 += dyall[(size_t)b * Tg + hd];
      P[n1 + 2 * H] = s3;
    }
    return;
  }
  const int c0 = (blockIdx.x / ntk) * kHeadTC, k0 = (blockIdx.x % ntk) * kHeadTK;
  const int ci = t / (kHeadTK / 4), kq = t % (kHeadTK / 4);
  const int kk = k0 + 4 * kq; // first k of this thread (H is a multiple of 16)
  f4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int r0 = b_lo; r0 < b_hi; r0 += kHeadRows) {
    const int nr = min(kHeadRows, b_hi - r0);
    __syncthreads();
    // stage rows r0 .. r0 + nr - 1: dq[., c0 .. c0 + 15], g[., k0 .. k0 + 63]
    for (int e = t; e < kHeadRows * kHeadTC; e += 256) {
      const int r = e / kHeadTC, cc = e % kHeadTC;
      sdq[r][cc] = r < nr ? dq[(size_t)(r0 + r) * H + c0 + cc] : 0.f;
    }
    for (int e = t; e < kHeadRows * (kHeadTK / 4); e += 256) {
      const int r = e / (kHeadTK / 4), kc = e % (kHeadTK / 4), k = k0 + 4 * kc;
      sg[r][kc] = (r < nr && k < H) ? *reinterpret_cast<const f4 *>(g + (size_t)(r0 + r) * H + k)
                                    : f4{0.f, 0.f, 0.f, 0.f};
    }
    __syncthreads();
    for (int r = 0; r < nr; ++r) acc += sdq[r][ci] * sg[r][kq];
  }
  if (kk < H) *reinterpret_cast<f4 *>(P + (size_t)(c0 + ci) * H + kk) = acc;
}

__global__ void __launch_bounds__(256)
k_head_w_sum(int H, int Z, const float *__restrict__ Pall, float *__restrict__ outall) {
  const int n = H * H + 2 * H + 1, hd = blockIdx.y;
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t >= n) return;
  const float *P = Pall + (size_t)hd * Z * n + t;
  float s = 0.f;
  for (int z = 0; z < Z; ++z) s += P[(size_t)z * n];
  outall[(size_t)hd * n + t] = s;
}

// ---- node-level heads (Tn of them; head s at wn + s (H^2 + 2H + 1)) ------
// Their hidden layer Q_s = ReLU(h W1_s^T + b1_s) [N, H] comes from the NT
// GEMM (Q_s at Qn + s capN H); these kernels do the rest.

// 16-byte-aligned copies of W1_s for the GEMMs: W1n [Tn][H][H] as stored and
// W1nT [H][Tn H] with W1nT[n][s H + c] = W1_s[c][n].
__global__ void __launch_bounds__(256)
k_stage_node_heads(int H, int Tn, const float *__restrict__ wn, float *__restrict__ W1n,
                   float *__restrict__ W1nT) {
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long n = (long long)Tn * H * H;
  if (t >= n) return;
  const int sh = (int)(t / ((long long)H * H)), r = (int)((t / H) % H), k = (int)(t % H);
  const float v = wn[(size_t)sh * (H * H + 2 * H + 1) + (size_t)r * H + k];
  W1n[t] = v;
  W1nT[(size_t)k * Tn * H + (size_t)sh * H + r] = v;
}

// z[i, s] = w2_s . Q_s[i] + b2_s (one thread per node and head).
__global__ void __launch_bounds__(256)
k_node_head_out(const Dims *__restrict__ dims, int H, int Tn, size_t capN,
                const float *__restrict__ Qn, const float *__restrict__ wn,
                float *__restrict__ z, float *__restrict__ z2) {
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const int N = dims->N;
  if (t >= (long long)N * Tn) return;
  const int i = (int)(t / Tn), sh = (int)(t % Tn);
  const float *w2 = wn + (size_t)sh * (H * H + 2 * H + 1) + H * H + H;
  const float *q = Qn + (size_t)sh * capN * H + (size_t)i * H;
  float acc = w2[H];
#pragma unroll 8
  for (int c = 0; c < H; c += 4) { // H is a multiple of 16
    const f4 v = *reinterpret_cast<const f4 *>(q + c);
#pragma unroll
    for (int e = 0; e < 4; ++e) acc += w2[c + e] * v[e];
  }
  z[t] = acc;
  if (z2) z2[t] = acc;
}

// e[i, s] = 2 nw_s (z - z_target) / N and dQ_s[i, c] = e w2_s[c] [Q_s[i, c] > 0].
__global__ void __launch_bounds__(256)
k_node_head_err(const Dims *__restrict__ dims, int H, int Tn, size_t capN,
                const float *__restrict__ Qn, const float *__restrict__ wn,
                const float *__restrict__ z, const float *__restrict__ zt,
                const float *__restrict__ nw, float *__restrict__ e, float *__restrict__ dQ) {
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const int N = dims->N;
  if (t >= (long long)N * Tn * H) return;
  const int c = (int)(t % H);
  const long long is = t / H;
  const int i = (int)(is / Tn), sh = (int)(is % Tn);
  const float ev = (2.0f * (z[is] - zt[is]) / (float)N) * (nw ? nw[sh] : 1.0f);
  if (c == 0) e[is] = ev;
  const size_t o = (size_t)sh * capN * H + (size_t)i * H + c;
  const float w2 = wn[(size_t)sh * (H * H + 2 * H + 1) + H * H + H + c];
  dQ[o] = Qn[o] > 0.f ? ev * w2 : 0.f;
}

// dw2_s[c] = sum_i e[i, s] Q_s[i, c] and db2_s = sum_i e[i, s] (column c = H),
// in a fixed order: the nodes are cut into kNodeChunks contiguous chunks
// (blockIdx.x), each chunk's sum goes to part[s][chunk][c], and
// k_node_head_small_sum adds the chunks in order.  Both are chains of loads:
// 12 and 32 in flight (4.5k nodes, two heads: 10.3 -> 5.9 us and 5.6 -> 3.1; the
// node heads' part of k_loss with 8, 14.7 -> 8.5 for the launch).
constexpr int kNodeChunks = 128;

__global__ void __launch_bounds__(256)
k_node_head_small(const Dims *__restrict__ dims, int H, int Tn, size_t capN,
                  const float *__restrict__ Qn, const float *__restrict__ e,
                  float *__restrict__ part) {
  const int r = blockIdx.x, sh = blockIdx.y;
  const int N = dims->N;
  const int rows = (N + kNodeChunks - 1) / kNodeChunks;
  const int i0 = min(r * rows, N), i1 = min(i0 + rows, N);
  const float *Q = Qn + (size_t)sh * capN * H;
  float *out = part + ((size_t)sh * kNodeChunks + r) * (H + 1);
  for (int c = threadIdx.x; c <= H; c += 256) {
    float s = 0.f;
    if (c < H)
#pragma unroll 12
      for (int i = i0; i < i1; ++i) s += e[(size_t)i * Tn + sh] * Q[(size_t)i * H + c];
    else
#pragma unroll 12
      for (int i = i0; i < i1; ++i) s += e[(size_t)i * Tn + sh];
    out[c] = s;
  }
}

__global__ void __launch_bounds__(256)
k_node_head_small_sum(int H, const float *__restrict__ part, float *__restrict__ gwn) {
  const int sh = blockIdx.x;
  const float *p = part + (size_t)sh * kNodeChunks * (H + 1);
  float *dw2 = gwn + (size_t)sh * (H * H + 2 * H + 1) + H * H + H;
  for (int c = threadIdx.x; c <= H; c += 256) {
    float s = 0.f;
#pragma unroll 32
    for (int r = 0; r < kNodeChunks; ++r) s += p[(size_t)r * (H + 1) + c];
    dw2[c] = s;
  }
}

} // namespace

hipError_t launch_stage_node_heads(int H, int Tn, const float *wn, float *W1n, float *W1nT,
                                   hipStream_t s) {
  const long long n = (long long)Tn * H * H;
  if (n <= 0) return hipSuccess;
  k_stage_node_heads<<<cdiv(n, 256), 256, 0, s>>>(H, Tn, wn, W1n, W1nT);
  return hipGetLastError();
}

hipError_t launch_node_head_out(const Dims *dims, int capN, int H, int Tn, const float *Qn,
                                const float *wn, float *z, float *z2, hipStream_t s) {
  if (capN <= 0 || Tn <= 0) return hipSuccess;
  k_node_head_out<<<cdiv((long long)capN * Tn, 256), 256, 0, s>>>(dims, H, Tn, (size_t)capN,
                                                                  Qn, wn, z, z2);
  return hipGetLastError();
}

hipError_t launch_node_head_err(const Dims *dims, int capN, int H, int Tn, const float *Qn,
                                const float *wn, const float *z, const float *zt,
                                const float *nw, float *e, float *dQ, hipStream_t s) {
  if (capN <= 0 || Tn <= 0) return hipSuccess;
  k_node_head_err<<<cdiv((long long)capN * Tn * H, 256), 256, 0, s>>>(
      dims, H, Tn, (size_t)capN, Qn, wn, z, zt, nw, e, dQ);
  return hipGetLastError();
}

size_t node_head_small_floats(int H, int Tn) { return (size_t)Tn * kNodeChunks * (H + 1); }

hipError_t launch_node_head_small(const Dims *dims, int capN, int H, int Tn, const float *Qn,
                                  const float *e, float *part, float *gwn, hipStream_t s) {
  if (Tn <= 0) return hipSuccess;
  k_node_head_small<<<dim3(kNodeChunks, Tn), 256, 0, s>>>(dims, H, Tn, (size_t)capN, Qn, e,
                                                          part);
  k_node_head_small_sum<<<Tn, 256, 0, s>>>(H, part, gwn);
  return hipGetLastError();
}

// Graphs a workgroup of the head takes: as many as leave every CU a workgroup.
static int graphs_per_group(int capB) { return capB >= 1024 ? 4 : capB >= 512 ? 2 : 1; }

hipError_t launch_head_forward(const Dims *dims, int capB, int H, int Tg, const int *graph_ptr,
                               const float *h, const float *wh, const float *W1T, float *g,
                               float *q, float *pred, float *pred2, hipStream_t s) {
  if (capB <= 0) return hipSuccess;
  if (Tg < 1 || Tg > kMaxGraphHeads || H < 4 || H > 512 || H % 4) return hipErrorInvalidValue;
  const int vec = ((uintptr_t)h & 15) == 0;
  const int G = graphs_per_group(capB);
#define HGNN_HEAD(GG)                                                                          \
  k_head_forward<GG><<<dim3(cdiv(capB, GG), Tg), kHeadFwdThreads, 0, s>>>(                     \
      dims, H, Tg, graph_ptr, h, vec, wh, W1T, g, q, pred, pred2)
  if (G == 4) HGNN_HEAD(4);
  else if (G == 2) HGNN_HEAD(2);
  else HGNN_HEAD(1);
#undef HGNN_HEAD
  return hipGetLastError();
}

// W1T[t][k][c] = W1_t[c][k] for the Tg graph heads, through 32 x 32 LDS tiles.
__global__ void __launch_bounds__(256)
k_stage_head_t(const float *__restrict__ wh, int H, float *__restrict__ W1T) {
  __shared__ float tl[32][33];
  const int t = blockIdx.z;
  const float *W1 = wh + (size_t)t * (H * H + 2 * H + 1);
  float *out = W1T + (size_t)t * H * H;
  const int c0 = blockIdx.y * 32, k0 = blockIdx.x * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int r = ty; r < 32; r += 8) {
    const int c = c0 + r, k = k0 + tx;
    tl[r][tx] = (c < H && k < H) ? W1[(size_t)c * H + k] : 0.f;
  }
  __syncthreads();
  for (int r = ty; r < 32; r += 8) {
    const int k = k0 + r, c = c0 + tx;
    if (k < H && c < H) out[(size_t)k * H + c] = tl[tx][r];
  }
}

hipError_t launch_stage_head_t(const float *wh, int H, int Tg, float *W1T, hipStream_t s) {
  const dim3 grid(cdiv(H, 32), cdiv(H, 32), Tg);
  k_stage_head_t<<<grid, 256, 0, s>>>(wh, H, W1T);
  return hipGetLastError();
}

hipError_t launch_loss(const Dims *dims, int Tg, const float *pred, const float *t,
                       const float *gw, int Tn, const float *z, const float *zt,
                       const float *nw, float *loss, hipStream_t s) {
  k_loss<<<1, kHeadThreads, 0, s>>>(dims, Tg, pred, t, gw, Tn, z, zt, nw, loss);
  return hipGetLastError();
}

hipError_t launch_head_backward(const Dims *dims, int capB, int H, int Tg, const int *graph_ptr,
                                const float *wh, const float *g, const float *q,
                                const float *pred, const float *target, const float *dpred,
                                const float *gw, float *dy, float *dq, float *dh,
                                float *dw_head, const float *relu_of, const float *add,
                                float *part, hipStream_t s) {
  if (capB <= 0) return hipSuccess;
  if (Tg < 1 || Tg > kMaxGraphHeads || H < 4 || H > 512 || H % 4) return hipErrorInvalidValue;
  const int vec = (((uintptr_t)dh | (uintptr_t)relu_of | (uintptr_t)add) & 15) == 0;
  const int G = Tg == 1 ? graphs_per_group(capB) : 1;
#define HGNN_HEAD(GG)                                                                          \
  k_head_bwd_graph<GG><<<cdiv(capB, GG), kHeadBwdThreads, 0, s>>>(                             \
      dims, H, Tg, graph_ptr, wh, q, pred, target, dpred, gw, dy, dq, dh, relu_of, add, vec)
  if (G == 4) HGNN_HEAD(4);
  else if (G == 2) HGNN_HEAD(2);
  else HGNN_HEAD(1);
#undef HGNN_HEAD
  const int n = H * H + 2 * H + 1;
  if (part && capB >= kHeadChunkedMinB && H % 16 == 0) {
    const int Z = std::min(kHeadChunks, cdiv(capB, kHeadRows));
    const int tiles = (H / kHeadTC) * cdiv(H, kHeadTK);
    k_head_w_part<<<dim3(tiles + 1, Z, Tg), 256, 0, s>>>(dims, H, Tg, Z, g, q, dy, dq, part);
    k_head_w_sum<<<dim3(cdiv(n, 256), Tg), 256, 0, s>>>(H, Z, part, dw_head);
  } else {
    k_head_bwd_weights<<<dim3(cdiv(n, kHeadOut), Tg), 256, 0, s>>>(dims, H, Tg, g, q, dy, dq,
                                                                   dw_head);
  }
  return hipGetLastError();
}

size_t head_partial_floats(int H, int Tg) {
  return (size_t)Tg * kHeadChunks * ((size_t)H * H + 2 * H + 1);
}

} // namespace hgnn
