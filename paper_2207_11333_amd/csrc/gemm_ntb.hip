// NT-form MFMA GEMM with its operand tiles copied from HBM straight into LDS
// (steps S1, S3 and the layer-input gradient of S6 + S8).
//
// Every A segment is in the product's own precision in HBM: FP32 as it lies,
// or for BF16 a copy its producer wrote (RNE-rounded, the rounding the
// register-staged kernel applies while staging); BF16 products of small grids
// without a copy take FP32 and round it in registers.  A K tile goes from HBM to LDS by gfx950's LDS-DMA loads
// (global_load_lds_dwordx4: 16 bytes per lane, written to LDS in lane order),
// never through registers, which are left to the products.
//
// LDS rows are 128 bytes: one K tile holds 32 FP32 or 64 BF16 of k.  Chunk c
// (16 bytes) of row r is stored at 16 (c ^ (r & 7)), so the eight rows read by
// eight adjacent lanes of a fragment load fall in distinct banks (the LDS
// bank-conflict counter reads 0).  A DMA instruction fills 8 rows: lane L
// writes row L / 8, position L % 8, so it loads logical chunk (L % 8) ^ (L / 8)
// of that row.  The loads of a tile (A rows, weight rows, BF16 weight low
// halves) are dealt to the waves in turn, the same number to each.
//
// Pipeline: a ring of NST LDS stages; tiles t + 1 .. t + NST - 1 are in flight
// while tile t computes.  Each wave counts its own DMA loads (vmcnt) and one
// plain s_barrier per tile (the fence of __syncthreads would wait for every
// load in flight) makes every wave's loads visible and frees the stage read
// by the previous tile.  The barrier sits before the tile's last products,
// which cover the next tile's fragment reads.
//
// What bounds it: a workgroup's K loop is a chain of short steps (64 x 64
// tiles: 128 to 512 matrix-core cycles a wave and step), so whatever a step
// does beside its products lengthens every workgroup.  The loads themselves
// are not the limit (a streaming test: eight waves with two loads each in
// flight copy 54 bytes a cycle and CU from L2, four waves with four loads as
// much).  Each lane therefore keeps its load addresses and moves them on by a
// constant; looking up the segment and forming row addresses for every tile
// (scalar loads, waits and 64-bit products) cost about as long as the
// products: with addresses kept, FP32 at 4.5k rows and H = 128 the update
// linear 22.3 -> 17.7 us, message 10.5 -> 9.5, layer-input gradient
// 16.5 -> 12.9; BF16 update 10.7 -> 8.9 us; one molecule (29 rows, a single
// row tile) BF16 update 9.1 -> 7.8 us.  128 x 128 tiles, whose products
// are longer, gained nothing (105 us BF16 update at 40k rows).
//
// Three tile shapes: 128 x 128 (waves of 64 x 32) for grids that fill the GPU,
// 64 x 64 (32 x 16) and 32 x 32 (16 x 16, four waves) for smaller ones, whose
// time is set by how many tiles run at once (tile_side).  FP32's matrix
// instructions bound a small grid: a 64 x 64 tile of the update linear (K = 640)
// is 9 us of them on its CU, whatever the other CUs do.  Three stages: 144 KB for
// 128 x 128 in BF16, 24 to 96 KB for the others, so that several workgroups share
// a CU.  Five for 64 x 64 in BF16 (120 KB, one workgroup): 28k nodes, H = 64,
// message linear 9.6 -> 12.6 us, a training step 1161 -> 1210; four to ten for
// 32 x 32: BF16 update linear at 4.5k nodes 9.2 -> 9.5 to 17 us.
//
// Products and their order per output are those of the register-staged
// kernel when it runs unsplit (FP32: per 16 k, four k-slots of
// v_mfma_f32_16x16x4_f32; BF16: per 64 k, weight hi over k 0-31 and 32-63,
// then lo over the same), so outputs are bitwise equal to its unsplit form; with
// chunks above one (FP32) the sums are those of its split-K form and its reduction.
#include "mfma_tile.hpp"

namespace hgnn {

namespace {

typedef __attribute__((address_space(3))) void lds_t;

constexpr int kQRow = 128; // bytes per LDS row (one K tile)
constexpr int kQWGM = 2; // waves of a workgroup: kQWGM x waves_n
constexpr int waves_n(int tile) { return tile == 32 ? 2 : 4; }
constexpr int kStages = 3; // LDS stages

// PREC 0: FP32 operands and weights; 1: BF16 operands, weights as hi + lo; 2: as
// 1 with FP32 operands, rounded when a tile's fragments are used.
// BM x BN tile, WGM x WGN waves, NST LDS stages.
// SHORT: for a short first segment (GemmNTB::short0); instances of their own, as
// its address selects cost the others 5 to 10 %.
template <int PREC, int BM, int BN, int WGM, int WGN, int NST, int TAG, bool SHORT>
__global__ void __launch_bounds__(64 * WGM * WGN, 1)
k_gemm_ntb(const Dims *__restrict__ dims, const GemmNTB g, int ntiles_n) {
  constexpr bool SPLIT = PREC != 0, A32 = PREC == 2;
  constexpr bool FOLD = PREC == 0 && BM < 128; // chunked sums: small FP32 grids only
  constexpr int ESZ = SPLIT ? 2 : 4, ESA = PREC == 1 ? 2 : 4; // bytes of a weight, of an A element
  constexpr int NAH = A32 ? 2 : 1; // A: rows of 128 bytes per K tile and row
  constexpr int BKE = kQRow / ESZ; // k per K tile
  constexpr int NW = WGM * WGN, WM = BM / WGM, WN = BN / WGN, TM = WM / 16, TN = WN / 16;
  constexpr int IA = BM / 8, IB = BN / 8; // DMA loads (8 rows each) of A and of one B half
  static_assert(IA % NW == 0 && IB % NW == 0 && TM >= 1 && TN >= 1, "tile shape");
  constexpr int UA = IA / NW, UB = IB / NW; // per wave
  constexpr int DMA = UA * NAH + UB * (SPLIT ? 2 : 1);
  constexpr int SH = BM * kQRow, SA = SH * NAH, SB = BN * kQRow, STAGE = SA + SB * (SPLIT ? 2 : 1);
  __shared__ __attribute__((aligned(1024))) char smem[NST * STAGE];

  const int M = g.M_fixed >= 0 ? g.M_fixed : dims->N;
  int mtiles = (M + BM - 1) / BM;
  int mt, n0, m0, m_hi = M, bq = 0;
  if (g.perm) {
    const BucketWalk bw(g.brow, g.nb, BM);
    mtiles = bw.total();
    if ((int)blockIdx.x >= mtiles * ntiles_n) return;
    const int tile = xcd_tile(blockIdx.x, mtiles * ntiles_n);
    mt = tile / ntiles_n;
    n0 = (tile % ntiles_n) * BN;
    bw.find(mt, bq, m0, m_hi);
  } else {
    if ((int)blockIdx.x >= mtiles * ntiles_n) return;
    const int tile = xcd_tile(blockIdx.x, mtiles * ntiles_n);
    mt = tile / ntiles_n;
    n0 = (tile % ntiles_n) * BN;
    m0 = mt * BM;
  }
  const int tid = threadIdx.x, L = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = (w / WGN) * WM, wn0 = (w % WGN) * WN;

  int KT = 0;
  for (int q = 0; q < g.nseg; ++q) KT += (g.seg[q].k + BKE - 1) / BKE;
  // A short first segment ends in a tile of kv columns, tile t_short: lanes past
  // the segment or the weight row load the row's first bytes instead, and both
  // operands there are zeroed when the tile is used.
  const int kv = SHORT ? g.seg[0].k % BKE : 0;
  const int t_short = kv ? g.seg[0].k / BKE : -1;

  // This wave's DMA loads of a K tile: UA of A rows, UB of weight rows and
  // (BF16) UB of weight low halves, 8 rows each; load u of a kind covers rows
  // 8 (w + NW u) .. of the tile.  Each lane keeps the 64-bit address of its
  // 16 bytes and moves it on by one K tile per issue, so a tile's loads cost
  // two additions each; the segment's fields are read only where a segment
  // begins (the weights' columns run on through the segments).  Rows and
  // columns past the matrix read clamped (valid) rows, whose products land
  // only in outputs that are never stored.
  const int dr = L >> 3;
  const int db = 16 * ((L & 7) ^ dr); // first byte of the chunk this lane loads
  const char *pa[UA], *pb[UB], *pl[SPLIT ? UB : 1];
  int rowa[UA];
#pragma unroll
  for (int u = 0; u < UB; ++u) {
    const int r = min(n0 + 8 * (w + NW * u) + dr, g.Ncols - 1);
    const size_t off = (size_t)ESZ * ((size_t)bq * g.bstride + (size_t)r * g.ldb) + db;
    pb[u] = static_cast<const char *>(g.B) + off;
    if constexpr (SPLIT) pl[u] = static_cast<const char *>(g.B_lo) + off;
  }
#pragma unroll
  for (int u = 0; u < UA; ++u) {
    const int m = min(m0 + 8 * (w + NW * u) + dr, m_hi - 1);
    rowa[u] = g.perm ? g.perm[m] : m;
  }
  int q = 0, left = 0; // next segment, K tiles left in the current one
  auto dma = [](const char *src, char *dst) {
    // the builtin takes a non-const pointer: without the cast the host pass
    // drops the kernel templates (their launch handles stay undefined)
    __builtin_amdgcn_global_load_lds((void *)src, (lds_t *)dst, 16, 0, 0);
  };
  // the next K tile's loads into the stage at byte offset st
  auto issue = [&](int st) {
    if (left == 0) {
      const char *ap = static_cast<const char *>(g.seg[q].ptr) + db;
      const int lda = g.seg[q].ld;
      left = (g.seg[q].k + BKE - 1) / BKE;
      ++q;
#pragma unroll
      for (int u = 0; u < UA; ++u) pa[u] = ap + (size_t)rowa[u] * lda * ESA;
    }
    --left;
    char *d = smem + st + 8 * kQRow * w;
    // Byte offsets from the kept addresses, and the weights' step: selected, on one
    // path for short tiles and others.  With a branch for the short tile that
    // returned early the compiler moved the kept addresses' additions so that one
    // of the copies of this code loaded from an address never written.
    const bool sh = SHORT && kv && q == 1 && left == 0;
    int oa[NAH], ob = 0;
    const int bstep = sh ? kv * ESZ : kQRow;
#pragma unroll
    for (int h = 0; h < NAH; ++h) oa[h] = sh && h * kQRow + db >= kv * ESA ? -db : h * kQRow;
    if constexpr (SHORT) ob = sh && t_short * kQRow + db >= g.ldb * ESZ ? -db : 0;
#pragma unroll
    for (int u = 0; u < UA; ++u) {
#pragma unroll
      for (int h = 0; h < NAH; ++h) dma(pa[u] + oa[h], d + h * SH + 8 * kQRow * NW * u);
      pa[u] += kQRow * NAH;
    }
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      dma(pb[u] + ob, d + SA + 8 * kQRow * NW * u);
      pb[u] += bstep;
      if constexpr (SPLIT) {
        dma(pl[u] + ob, d + SA + SB + 8 * kQRow * NW * u);
        pl[u] += bstep;
      }
    }
  };

  // fragment reads: lane (r = L % 16, group L / 16) takes row r of each
  // 16-row block and logical chunk 4 c + L / 16 of the tile's two halves c
  // (BF16: 8 k per lane of a 32-deep MFMA; FP32: 4 k, the k-slots of four
  // 4-deep MFMAs)
  // FP32 A of a BF16 product: half c is its own 128-byte row, a lane's 8 k are
  // logical chunks 2 (L / 16) and the next, rounded (RNE) when the tile begins
  using V = typename Frag<SPLIT>::V;
  const int fr = L & 15;
  const int p0 = (L >> 4) ^ (fr & 7);
  const int offA0 = (wm0 + fr) * kQRow + 16 * p0, offA1 = (wm0 + fr) * kQRow + 16 * (p0 ^ 4);
  const int offB0 = SA + (wn0 + fr) * kQRow + 16 * p0;
  const int offB1 = SA + (wn0 + fr) * kQRow + 16 * (p0 ^ 4);
  const int q0 = 16 * ((2 * (L >> 4)) ^ (fr & 7)); // A32: the first chunk; the other is 16 bytes off
  V fa[A32 ? 1 : 2][2][TM], fb[2][2][TN], fl[2][2][SPLIT ? TN : 1]; // [set][half][block]
  f4 raw[A32 ? 2 : 1][A32 ? TM : 1][2];
  auto read = [&](auto set, int st) {
    constexpr int S = decltype(set)::value;
    const char *base = smem + st;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      if constexpr (A32) {
        const char *row = base + (wm0 + fr + 16 * i) * kQRow;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          raw[h][i][0] = *reinterpret_cast<const f4 *>(row + h * SH + q0);
          raw[h][i][1] = *reinterpret_cast<const f4 *>(row + h * SH + (q0 ^ 16));
        }
      } else {
        fa[S][0][i] = *reinterpret_cast<const V *>(base + offA0 + 16 * i * kQRow);
        fa[S][1][i] = *reinterpret_cast<const V *>(base + offA1 + 16 * i * kQRow);
      }
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      fb[S][0][j] = *reinterpret_cast<const V *>(base + offB0 + 16 * j * kQRow);
      fb[S][1][j] = *reinterpret_cast<const V *>(base + offB1 + 16 * j * kQRow);
    }
    if constexpr (SPLIT) {
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        fl[S][0][j] = *reinterpret_cast<const V *>(base + SB + offB0 + 16 * j * kQRow);
        fl[S][1][j] = *reinterpret_cast<const V *>(base + SB + offB1 + 16 * j * kQRow);
      }
    }
  };

  f4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
  // chunked sums (g.chunks > 1): chunk z holds K tiles [KT z / chunks ..) in
  // pairs; tot adds the finished ones, with more than four as two halves
  f4 tot[FOLD ? 2 : 1][TM][TN];
  int z = 0, z_end = KT, z_half = 0;
  const int adj = KT & 1, KT64 = (KT + adj) / 2; // a short segment of one tile is a 64-deep piece
  if constexpr (FOLD) {
    if (g.chunks > 1) {
      z_end = 2 * (KT64 / g.chunks) - adj;
      z_half = g.chunks > 4 ? (g.chunks + 1) / 2 : g.chunks;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) tot[0][i][j] = tot[1][i][j] = f4{0.f, 0.f, 0.f, 0.f};
    }
  }
  auto fold = [&]() {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        if (z < z_half) tot[0][i][j] += acc[i][j];
        else tot[FOLD][i][j] += acc[i][j];
      }
  };
  auto mm = [&](const V (&a)[TM], const V (&b)[TN]) { mma_frags<SPLIT, TM, TN>(a, b, acc); };
  auto next = [](int st) { return st == (NST - 1) * STAGE ? 0 : st + STAGE; };

  // tile t (register set S, LDS stage st): its first products; then, if a
  // tile follows, wait for it, refill this stage with tile t + NST and read
  // tile t + 1's fragments; then the last products
  auto step = [&](auto set, int t, int st) {
    constexpr int S = decltype(set)::value;
    if constexpr (FOLD) {
      if (t == z_end) { // a chunk is complete
        fold();
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
        ++z;
        z_end = 2 * (KT64 * (z + 1) / g.chunks) - adj;
      }
    }
    constexpr int SF = A32 ? 0 : S;
    if constexpr (A32) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int e = 0; e < 8; ++e) fa[0][h][i][e] = (__bf16)raw[h][i][e >> 2][e & 3];
    }
    if constexpr (SHORT) {
      if (t == t_short) {
        // both operands: the weights there may be infinite
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const bool past = (BKE / 2) * h + (BKE / 8) * (L >> 4) >= kv;
#pragma unroll
          for (int i = 0; i < TM; ++i) fa[SF][h][i] = past ? V{} : fa[SF][h][i];
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            fb[S][h][j] = past ? V{} : fb[S][h][j];
            if constexpr (SPLIT) fl[S][h][j] = past ? V{} : fl[S][h][j];
          }
        }
      }
    }
    mm(fa[SF][0], fb[S][0]);
    if constexpr (SPLIT) {
      mm(fa[SF][1], fb[S][1]);
      mm(fa[SF][0], fl[S][0]);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (t + 1 < KT) {
      wait_groups<DMA, NST - 2>(KT - 2 - t);
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      if (t + NST < KT) issue(st);
      read(IC<1 - S>{}, next(st));
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (SPLIT) mm(fa[SF][1], fl[S][1]);
    else mm(fa[SF][1], fb[S][1]);
  };

  for (int t = 0, st = 0; t < NST && t < KT; ++t, st += STAGE) issue(st);
  wait_groups<DMA, NST - 1>(KT - 1);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  read(IC<0>{}, 0);
  int st = 0;
  for (int t = 0; t < KT; t += 2) {
    step(IC<0>{}, t, st);
    st = next(st);
    if (t + 1 >= KT) break;
    step(IC<1>{}, t + 1, st);
    st = next(st);
  }

  if constexpr (FOLD) {
    if (g.chunks > 1) {
      fold();
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = g.chunks > 4 ? tot[0][i][j] + tot[1][i][j] : tot[0][i][j];
    }
  }

  // Epilogue (as the register-staged kernel's): lane (cr = 4 (L / 16),
  // cc = L % 16) holds rows wm0 + 16 i + cr + v, columns wn0 + 16 j + cc; the
  // rows' nodes are fetched once, from clamped indices, without a branch.
  const int cr = 4 * (L >> 4), cc = L & 15;
  int node[TM][4];
  bool rok[TM][4];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = m0 + wm0 + i * 16 + cr + v;
      rok[i][v] = r < m_hi;
      const int rr = min(r, m_hi - 1);
      node[i][v] = g.perm ? g.perm[rr] : rr;
    }
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int n = n0 + wn0 + j * 16 + cc;
    const bool nok = n < g.Ncols;
    const int nc = min(n, g.Ncols - 1);
    const float bias = g.bias ? g.bias[nc] : 0.f;
    float o[TM][4];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) o[i][v] = acc[i][j][v] + bias;
    if (g.addend) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) o[i][v] += g.addend[(size_t)node[i][v] * g.ld_add + nc];
    }
    if (g.relu) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) o[i][v] = o[i][v] > 0.f ? o[i][v] : 0.f;
    }
    if (g.mask) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (!(g.mask[(size_t)node[i][v] * g.ldc + nc] > 0.f)) o[i][v] = 0.f;
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (nok && rok[i][v]) {
          if (g.C) g.C[(size_t)node[i][v] * g.ldc + n] = o[i][v];
          if (g.Cb) g.Cb[(size_t)node[i][v] * g.ldcb + n] = (__bf16)o[i][v];
        }
  }
}

inline bool al16(const void *p) { return ((uintptr_t)p & 15) == 0; }

// Tile side by the grid it gives: 128 when that fills every CU at least once and its
// rounds over the 256 CUs are at least 0.8 full; 64 when its own rounds are; else 32.
// Each is a quarter of the work of the one before (and more of them share a CU), at
// twice the operand traffic.  128 against 64, four layers, FP32 inference of SAGE
// H = 256: 17.9k nodes (280: a second round for 24) 323 and 259 us, 23.9k (374) 341
// and 298, 40.4k (632: three rounds, 0.82 full) 488 and 488; H = 128 at 50.3k (393,
// 0.77 full) 252 and 242.  Update linear of H = 128, FP32, 64 against 32: 1.1k nodes (23 of 256
// CUs busy) 11.3 -> 6.8 us, 4.5k (150) 17.9 -> 15.1, 8.9k (290: a second round
// for 34) 28.9 -> 23.3, but 15.7k (502) 31.5 -> 35.1.  BF16's products are a quarter
// as long or less, so that a second round costs less than that traffic: inference of
// four layers, 64 against 32, H = 384 at 2.5k nodes (264) 169 and 190 us, H = 448 at
// 4.5k (525) 331 and 369, H = 256 at 6.3k (416) 200 and 209.  Not where the operands
// are FP32, twice the traffic again (training of H = 256 at 4.5k, whose layer-input
// gradient has 304 tiles, 583 and 575).
int tile_side(int capM, const GemmNTB &g, int precision) {
  auto grid = [&](int B) {
    return (long long)(cdiv(capM, B) + (g.perm ? g.nb : 0)) * cdiv(g.Ncols, B);
  };
  auto full = [](long long n, long long rounds) { return 10 * n >= 8 * 256 * rounds; };
  const long long l = grid(128), n = grid(64);
  if (l >= 256 && full(l, (l + 255) / 256) && g.chunks <= 1 && !g.short0) return 128;
  return full(n, precision == 1 ? 1 : (n + 255) / 256) ? 64 : 32;
}

} // namespace

bool gemm_ntb_ok(const GemmNTB &g, int precision) {
  const int bke = precision ? 64 : 32, esz = precision ? 2 : 4, esa = precision == 1 ? 2 : 4;
  if (g.nseg < 1 || g.nseg > kMaxSeg || !g.B || !(g.C || g.Cb) || g.Ncols <= 0)
    return false;
  if ((precision != 0) != (g.B_lo != nullptr) || (precision == 0 && g.Cb)) return false;
  if ((g.ldb * esz) % 16 || !al16(g.B) || (g.B_lo && !al16(g.B_lo))) return false;
  if (g.perm && (!g.brow || g.nb < 1 || (g.bstride * esz) % 16)) return false;
  int boff = 0, pieces = 0; // the segments' weight columns follow one another from 0
  if (g.short0 && precision == 1) return false;
  for (int q = 0; q < g.nseg; ++q) {
    const SegB &s = g.seg[q];
    if (!s.ptr || !al16(s.ptr) || s.k <= 0 || (s.ld * esa) % 16 || s.boff != boff) return false;
    if (g.short0 && q == 0) {
      if (s.k % 16 || s.k > 64) return false;
    } else if (s.k % bke || (g.chunks > 1 && s.k % 64)) {
      return false;
    }
    boff += s.k;
    pieces += (s.k + 63) / 64;
  }
  if (g.chunks > 1 && (precision || g.chunks > 8 || pieces < g.chunks)) return false;
  return true;
}

hipError_t launch_gemm_ntb(const Dims *dims, int capM, const GemmNTB &g, int precision,
                           hipStream_t s, int tag, hipEvent_t ev0, hipEvent_t ev1) {
  if (capM <= 0) return hipSuccess;
  if (!gemm_ntb_ok(g, precision)) return hipErrorInvalidValue;
  const int B = tile_side(capM, g, precision);
  const int nt = cdiv(g.Ncols, B);
  // bucketed rows: each bucket's last tile may be partial
  const dim3 grid((cdiv(capM, B) + (g.perm ? g.nb : 0)) * nt), block(64 * kQWGM * waves_n(B));
  const int key = precision * 10000 + B * 10 + tag + (g.short0 ? 5 : 0);
  switch (key) {
#define HGNN_NTB(P, BB, T, SH)                                                                 \
  case P * 10000 + BB * 10 + T + (SH ? 5 : 0):                                                 \
    hipExtLaunchKernelGGL(                                                                     \
        (k_gemm_ntb<P, BB, BB, kQWGM, waves_n(BB), kStages, T, SH>), grid, block, 0, s, \
        ev0, ev1, 0, dims, g, nt);                                                             \
    break;
#define HGNN_NTB_TAGS(P, BB)                                                                   \
  HGNN_NTB(P, BB, 0, false) HGNN_NTB(P, BB, 1, false) HGNN_NTB(P, BB, 2, false)                \
  HGNN_NTB(P, BB, 4, false)
#define HGNN_NTB_SHORT(P, BB)                                                                  \
  HGNN_NTB(P, BB, 0, true) HGNN_NTB(P, BB, 1, true) HGNN_NTB(P, BB, 2, true) HGNN_NTB(P, BB, 4, true)
    HGNN_NTB_TAGS(0, 32)
    HGNN_NTB_TAGS(1, 32)
    HGNN_NTB_TAGS(0, 64)
    HGNN_NTB_TAGS(0, 128)
    HGNN_NTB_TAGS(1, 64)
    HGNN_NTB_TAGS(1, 128)
    HGNN_NTB_TAGS(2, 32)
    HGNN_NTB_TAGS(2, 64)
    HGNN_NTB_SHORT(0, 32)
    HGNN_NTB_SHORT(0, 64)
    HGNN_NTB_SHORT(2, 32)
    HGNN_NTB_SHORT(2, 64)
#undef HGNN_NTB_SHORT
#undef HGNN_NTB_TAGS
#undef HGNN_NTB
  default:
    return hipErrorInvalidValue; // a tag without an instance
  }
  return hipGetLastError();
}

} // namespace hgnn
