// Weight gradients (S6, S8): P[z] = X^T [Y | 1] over a fixed chunk z of the
// node rows; reduce.hip adds the chunks in order and scatters the result into
// the packed gradient.  One launch takes a list of such products (a layer's,
// or every layer's of a backward pass).
//
// A workgroup (4 wave64 in a 2 x 2 grid) owns one output tile of one chunk.
// Both operand tiles go from HBM to LDS by LDS-DMA loads as they lie in
// memory, node row after node row ([k][columns], FP32), 16 rows a step in FP32
// lists and pairs, 32 in FP32 products by themselves and in BF16.  Rows past the
// chunk repeat its last one; the last step zeroes them in LDS, so no product is
// masked.
//
// MFMA operands: a wave's tile is 16 TW x 16 TW (TW = 4 or 2 blocks a side).
// The 16 rows of block i are the tile's columns TW r + i, r = 0..15, so one
// LDS read of TW consecutive floats gives a lane its operand of all TW blocks
// for one k: FP32 needs two LDS reads per TW^2 matrix instructions, against
// one read per block and operand when a block's rows are adjacent, and the
// reads of a 16-lane group are 16 TW consecutive floats (no bank conflict).
// The outputs of a lane are TW consecutive columns (16- or 8-byte stores).
// BF16 reads 8 k (rows 8 g .. 8 g + 7 of lane group g) and rounds them (RNE)
// in registers: no BF16 copy is written and no transposing read is needed.
//
// Measured, six PNA layers of H = 128 at 4.5k nodes (81 MB of partials): FP32
// 84 us in one launch, against 190 us for the twelve launches of the 64 x 64
// kernel it replaces (operands staged through registers, one LDS read per block
// and k); BF16 37 us against 132.  What is left in FP32: the products alone take
// 77 us (the matrix cores reach 140 TFLOP/s in a loop of this instruction: 47
// us), the loads alone 42.
//
// The sum column (bias gradients; the edge-feature columns of the message
// weights, which need no product at all) is X^T times a constant-one operand
// that is never loaded: TW extra matrix instructions per k in the waves of
// the first column tile.  Tiles of rows from sum_from on do only that.
#include "mfma_tile.hpp"

namespace hgnn {

namespace {

typedef __attribute__((address_space(3))) void lds_t;
typedef float f2 __attribute__((ext_vector_type(2)));
// pointers that come out of memory: constant and global, not generic
typedef const __attribute__((address_space(4))) int cint_t;
typedef __attribute__((address_space(1))) float gfloat_t;
template <int TW> struct VecOf;
template <> struct VecOf<4> { using T = f4; };
template <> struct VecOf<2> { using T = f2; };

// Node rows per step (R) and LDS stages.  FP32 lists: 16 rows, 24 KB a workgroup;
// BF16, whose instruction takes 32 rows, 48 KB (TW = 2) or 64 KB (TW = 4: two
// workgroups a CU; a third stage would leave one).  FP32 products launched alone,
// beside the adjoint on the other stream, keep 32 rows a step in flight (48 KB):
// at 24k nodes and H = 256 their launches take 231 us in place of 258 (a list at
// 4.5k nodes 557 us a training step in place of 549).
template <int TW> constexpr int wg_stages() { return TW == 4 ? 2 : 3; }
constexpr int kWgChunk = 32; // chunks are multiples of this many rows

// tile counts of a job: full column tiles of the rows before sum_from, one
// (sum only) of the rest
struct WgTiles {
  int mfull, nt, tpc;
  int rows; // rows of nt tiles that hold them (by_row)
};
__host__ __device__ inline WgTiles wg_tiles(const WgJob &j, int B) {
  WgTiles t;
  const int mt = (j.M + B - 1) / B;
  t.mfull = j.sum_from < j.M ? (j.sum_from + B - 1) / B : mt;
  t.nt = (j.N + B - 1) / B;
  t.tpc = t.mfull * t.nt + (mt - t.mfull);
  t.rows = (t.tpc + t.nt - 1) / t.nt;
  return t;
}

// A workgroup's place in a job: chunk z, its rows [i_lo, i_hi) of the (maybe
// permuted) row order, and the output tile at (m0, n0).
struct WgPlace {
  int z, i_lo, i_hi, m0, n0;
};

// FULL: the product and, in the first column tile, the sum column; else the
// sum column alone.  PERM: rows through j.perm.
template <int PREC, int TW, int R, bool FULL, bool PERM>
__device__ __forceinline__ void wgrad_body(const WgJob &j, const WgPlace &pl, char *smem) {
  using V = typename VecOf<TW>::T;
  constexpr int B = 32 * TW;               // output tile
  constexpr int ROWB = B * 4;              // bytes per LDS row
  constexpr int RPI = 1024 / ROWB;         // rows per DMA load
  constexpr int U = R / RPI / 4;     // DMA loads per wave, operand and step
  constexpr int NST = wg_stages<TW>(), OPB = R * ROWB, STAGE = 2 * OPB;
  constexpr int DMA = FULL ? 2 * U : U;
  const int z = pl.z, i_lo = pl.i_lo, i_hi = pl.i_hi, m0 = pl.m0, n0 = pl.n0;
  const int KT = i_hi > i_lo ? (i_hi - i_lo + R - 1) / R : 0;
  const int tid = threadIdx.x, L = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = (w >> 1) * 16 * TW, wn0 = (w & 1) * 16 * TW;

  // DMA: load u of wave w covers tile rows RPI (U w + u) ..; this lane takes
  // row lr of them and 16 bytes of columns (columns past the matrix read the
  // last ones, whose products are not stored)
  constexpr int LPR = 64 / RPI; // lanes per row
  const int lr = L / LPR, lc = 4 * (L % LPR);
  const float *xb = j.X + min(m0 + lc, j.M - 4);
  int n = min(n0 + lc, j.N - 4);
  const bool s1 = j.nseg > 1 && n >= j.seg[0].ncols;
  const float *yb = s1 ? j.seg[1].ptr + (n - j.seg[0].ncols) : j.seg[0].ptr + n;
  const int ldx = j.ldx, ldy = s1 ? j.seg[1].ld : j.seg[0].ld;
  // Row of this lane in load u of tile t.  A load's rows are the same for the
  // whole wave but for the lane's place lr among them: permuted row ids come
  // by scalar loads (they count apart from the vector loads in flight).
  cint_t *perm = (cint_t *)j.perm;
  auto row_of = [&](int t, int u) {
    const int i = i_lo + t * R + RPI * (U * w + u);
    if constexpr (!PERM) return min(i + lr, i_hi - 1);
    int r = perm[min(i, i_hi - 1)];
#pragma unroll
    for (int k = 1; k < RPI; ++k) {
      const int rk = perm[min(i + k, i_hi - 1)];
      r = lr == k ? rk : r;
    }
    return r;
  };
  auto dma = [](const void *src, char *dst) {
    __builtin_amdgcn_global_load_lds((void *)src, (lds_t *)dst, 16, 0, 0);
  };
  auto issue = [&](int t, int st) {
    char *d = smem + st + 1024 * U * w;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = row_of(t, u);
      dma(xb + (size_t)r * ldx, d + 1024 * u);
      if constexpr (FULL) dma(yb + (size_t)r * ldy, d + OPB + 1024 * u);
    }
  };

  f4 acc[TW][TW], acc1[TW];
#pragma unroll
  for (int i = 0; i < TW; ++i) {
    acc1[i] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < TW; ++k) acc[i][k] = f4{0.f, 0.f, 0.f, 0.f};
  }
  const int r = L & 15, g = L >> 4;
  const bool ones = n0 == 0 && wn0 == 0;
  const int offA = wm0 + TW * r, offB = wn0 + TW * r;

  auto compute = [&](int st) {
    const float *As = reinterpret_cast<const float *>(smem + st);
    const float *Bs = reinterpret_cast<const float *>(smem + st + OPB);
    if constexpr (PREC == 0) {
      // instruction kk: lane group g takes row 16 (kk / 4) + 4 g + kk % 4
      if constexpr (FULL) {
#pragma unroll
        for (int kk = 0; kk < R / 4; ++kk) {
          const V a = *reinterpret_cast<const V *>(As + (16 * (kk / 4) + 4 * g + kk % 4) * B + offA);
          const V b = *reinterpret_cast<const V *>(Bs + (16 * (kk / 4) + 4 * g + kk % 4) * B + offB);
#pragma unroll
          for (int i = 0; i < TW; ++i)
#pragma unroll
            for (int k = 0; k < TW; ++k)
              acc[i][k] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[k], acc[i][k], 0, 0, 0);
        }
      }
      if (ones) {
#pragma unroll
        for (int kk = 0; kk < R / 4; ++kk) {
          const V a = *reinterpret_cast<const V *>(As + (16 * (kk / 4) + 4 * g + kk % 4) * B + offA);
#pragma unroll
          for (int i = 0; i < TW; ++i)
            acc1[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], 1.0f, acc1[i], 0, 0, 0);
        }
      }
    } else {
      // lane group g takes rows 8 g .. 8 g + 7
      bf16x8 a[TW], b[TW];
      auto frag = [&](const float *base, int off, bf16x8 (&f)[TW]) {
        V v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e)
          v[e] = *reinterpret_cast<const V *>(base + (8 * g + e) * B + off);
#pragma unroll
        for (int i = 0; i < TW; ++i)
#pragma unroll
          for (int e = 0; e < 8; ++e) f[i][e] = (__bf16)v[e][i];
      };
      frag(As, offA, a);
      if constexpr (FULL) {
        frag(Bs, offB, b);
#pragma unroll
        for (int i = 0; i < TW; ++i)
#pragma unroll
          for (int k = 0; k < TW; ++k)
            acc[i][k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[k], acc[i][k], 0, 0, 0);
      }
      if (ones) {
        bf16x8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = (__bf16)1.0f;
#pragma unroll
        for (int i = 0; i < TW; ++i)
          acc1[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], o, acc1[i], 0, 0, 0);
      }
    }
  };

  // The first NST tiles are loaded in any case (tiles past the chunk repeat its
  // last row and are not used).
  if (KT > 0) {
#pragma unroll
    for (int t = 0; t < NST; ++t) issue(t, t * STAGE);
  }
  int st = 0;
  for (int t = 0; t < KT; ++t) {
    wait_groups<DMA, NST - 1>(max(KT, NST) - 1 - t); // tile t has landed
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    const int valid = i_hi - i_lo - t * R; // rows of the chunk from this tile on
    if (valid < R) { // its last, partial tile
      for (int c = valid * (ROWB / 16) + tid; c < R * (ROWB / 16); c += 256) {
        reinterpret_cast<f4 *>(smem + st)[c] = f4{0.f, 0.f, 0.f, 0.f};
        if constexpr (FULL) reinterpret_cast<f4 *>(smem + st + OPB)[c] = f4{0.f, 0.f, 0.f, 0.f};
      }
      __builtin_amdgcn_s_waitcnt(0xc07f); // lgkmcnt(0)
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
    }
    compute(st);
    __builtin_amdgcn_sched_barrier(0);
    if (t + NST < KT) {
      // refill the stage once every wave has read tile t
      __builtin_amdgcn_s_waitcnt(0xc07f); // lgkmcnt(0)
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      issue(t + NST, st);
    }
    st = st == (NST - 1) * STAGE ? 0 : st + STAGE;
  }
  // loads of unused tiles end before the workgroup does (they write LDS)
  __builtin_amdgcn_s_waitcnt(0x0f70); // vmcnt(0)

  // lane (group g, r) holds rows TW (4 g + v) + i and columns TW r .. of the
  // wave's tile
  typedef __attribute__((address_space(1))) V gV;
  typedef __attribute__((address_space(1))) f4 g4;
  const int ldp = j.N + 4;
  gfloat_t *Pz = (gfloat_t *)j.P + (size_t)z * j.M * ldp;
#pragma unroll
  for (int i = 0; i < TW; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int m = m0 + wm0 + TW * (4 * g + v) + i, nn = n0 + wn0 + TW * r;
      if (m >= j.M) continue;
      gfloat_t *row = Pz + (size_t)m * ldp;
      if (FULL && nn < j.N) {
        V o;
#pragma unroll
        for (int k = 0; k < TW; ++k) o[k] = acc[i][k][v];
        *(gV *)(row + nn) = o;
      }
      if (ones && r == 0) *(g4 *)(row + j.N) = f4{acc1[i][v], 0.f, 0.f, 0.f};
    }
}

template <int PREC, int TW, int R>
__device__ __forceinline__ void wgrad_tile(const Dims *__restrict__ dims, const WgJob &j, int blk) {
  constexpr int B = 32 * TW, STAGE = 2 * R * B * 4;
  __shared__ __attribute__((aligned(1024))) char smem[wg_stages<TW>() * STAGE];
  // chunk z and output tile: a chunk's tiles read the same rows and stay on
  // one XCD (the block index's remainder by 8), whose L2 serves the re-reads
  const WgTiles tl = wg_tiles(j, B);
  const int Z = j.splits + (j.perm ? j.nb : 0);
  // (by_row: a row of them; see wg_by_row)
  const int l = blk >> 3, x = (blk - j.rot) & 7;
  int z, jt;
  if (j.by_row) {
    const int g = (l / tl.nt) * 8 + x;
    z = g / tl.rows;
    jt = (g % tl.rows) * tl.nt + l % tl.nt;
  } else {
    z = (l / tl.tpc) * 8 + x;
    jt = l % tl.tpc;
  }
  if (z >= Z || jt >= tl.tpc) return;
  const bool full = jt < tl.mfull * tl.nt;
  const int mt = full ? jt / tl.nt : tl.mfull + (jt - tl.mfull * tl.nt);
  const int m0 = mt * B, n0 = full ? (jt % tl.nt) * B : 0;
  const int rows = dims->N;
  int chunk = (rows + j.splits - 1) / j.splits;
  chunk = (chunk + kWgChunk - 1) / kWgChunk * kWgChunk;
  if (j.perm) {
    // bucket-pure chunks over the permuted rows: bucket q holds
    // ceil(n_q / chunk) chunks, in bucket order; the chunks past the last
    // are empty and write zero partials
    int bq, r0, r1;
    BucketWalk(j.brow, j.nb, chunk).find(z, bq, r0, r1);
    if (jt == 0 && threadIdx.x == 0) {
      j.zscale[2 * z] = bq >= 0 ? j.table[2 * bq] : 0.f;
      j.zscale[2 * z + 1] = bq >= 0 ? j.table[2 * bq + 1] : 0.f;
    }
    const WgPlace pl{z, bq >= 0 ? r0 : 0, bq >= 0 ? min(r1, r0 + chunk) : 0, m0, n0};
    wgrad_body<PREC, TW, R, true, true>(j, pl, smem);
    return;
  }
  const int i_lo = min(z * chunk, rows);
  const WgPlace pl{z, i_lo, min(rows, i_lo + chunk), m0, n0};
  if (full) wgrad_body<PREC, TW, R, true, false>(j, pl, smem);
  else wgrad_body<PREC, TW, R, false, false>(j, pl, smem);
}

// one FP32 product, on the tile of wg_tile_all
__global__ void __launch_bounds__(256, 2) k_wgrad(const Dims *__restrict__ dims, const WgJob j) {
  wgrad_tile<0, 2, 32>(dims, j, blockIdx.x);
}

// a layer's two products
template <int PREC, int TW>
__global__ void __launch_bounds__(256, 2)
k_wgrad_pair(const Dims *__restrict__ dims, const WgJob j0, const WgJob j1, int n0) {
  const bool first = (int)blockIdx.x < n0;
  wgrad_tile<PREC, TW, PREC ? 32 : 16>(dims, first ? j0 : j1, first ? blockIdx.x : blockIdx.x - n0);
}

// blockIdx.y: the job, in device memory; blocks past a job's have nothing to do
template <int PREC, int TW>
__global__ void __launch_bounds__(256, 2)
k_wgrad_all(const Dims *__restrict__ dims, const WgJob *__restrict__ tab) {
  wgrad_tile<PREC, TW, PREC ? 32 : 16>(dims, tab[blockIdx.y], blockIdx.x);
}

inline bool al16(const void *p) { return ((uintptr_t)p & 15) == 0; }

} // namespace

bool wg_job_ok(const WgJob &j) {
  if (!j.X || !j.P || j.M < 4 || j.M % 4 || j.N < 4 || j.N % 4 || j.splits < 1) return false;
  if (j.ldx % 4 || !al16(j.X) || !al16(j.P) || j.nseg < 1 || j.nseg > 2) return false;
  if (j.perm && (!j.brow || j.nb < 1 || !j.table || !j.zscale || j.sum_from < j.M)) return false;
  int n = 0;
  for (int q = 0; q < j.nseg; ++q) {
    if (!j.seg[q].ptr || !al16(j.seg[q].ptr) || j.seg[q].ld % 4 || j.seg[q].ncols % 4) return false;
    n += j.seg[q].ncols;
  }
  return n == j.N;
}

// Output tile side of a list of products that has `blocks128` workgroups of
// 128 x 128.  FP32: 64 (a step's matrix instructions take four times BF16's, and
// the smaller tiles deal them to the CUs more evenly: six layers of H = 128 at
// 4.5k nodes 84 us against 89, at 16k nodes 252 against 269).  BF16: 128, whose
// operands are read half as often, where that gives every CU two workgroups.
int wg_tile_all(int blocks128, int precision) { return precision && blocks128 >= 512 ? 128 : 64; }

int wg_groups(const WgJob &j, int tile) {
  const int Z = j.splits + (j.perm ? j.nb : 0);
  return j.by_row ? Z * wg_tiles(j, tile).rows : Z;
}

int wg_blocks(const WgJob &j, int tile) {
  const WgTiles t = wg_tiles(j, tile);
  return 8 * ((wg_groups(j, tile) + 7) / 8) * (j.by_row ? t.nt : t.tpc);
}

// Which FP32 products deal rows of tiles to the XCDs.  Whole chunks keep a chunk's
// rows in one L2, but few chunks leave XCDs idle, the more so where they are unequal
// (bucketed ones).  In a list, by chunks and by rows (a training step): H = 512,
// with 7 and 3 chunks a layer, one layer at 14k nodes 1920 and 1402 us, two 3847 and
// 3124; one CGCNN layer 2275 and 1323; H = 256, with 12 and 9, one layer 562 and
// 511, four 2090 and 1961; H = 192, with 16 and 15, six layers 1938 and 1897 but one
// 365 and 370; H = 128, with 29 each, single layers at 1k to 5k nodes up to 3 % slower
// by rows.  BF16 products too: GraphSAGE and CGCNN of H = 256 at 14k nodes 4 and 2 %.
// Launched alone (24k nodes): three layers of H = 384, 8 chunks, 5770 and 4869 us; of
// H = 192 1692 and 1645; and rows where the chunks do not deal evenly: 12 of H = 256,
// four layers, 3521 and 3382.
bool wg_by_row(const WgJob &j, bool alone) {
  const int Z = j.splits + (j.perm ? j.nb : 0);
  return Z < 14 || (alone && (Z <= 16 || Z % 8));
}

hipError_t launch_wgrad(const Dims *dims, const WgJob &j, hipStream_t s, hipEvent_t ev0,
                        hipEvent_t ev1) {
  if (!wg_job_ok(j)) return hipErrorInvalidValue;
  WgJob k = j;
  k.by_row = wg_by_row(j, true);
  hipExtLaunchKernelGGL(k_wgrad, dim3(wg_blocks(k, 64)), dim3(256), 0, s, ev0, ev1, 0, dims, k);
  return hipGetLastError();
}

hipError_t launch_wgrad_pair(const Dims *dims, const WgJob &j0, const WgJob &j1, int precision,
                             hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  if (!wg_job_ok(j0) || !wg_job_ok(j1)) return hipErrorInvalidValue;
  const int tile = wg_tile_all(wg_blocks(j0, 128) + wg_blocks(j1, 128), precision);
  WgJob k0 = j0, k1 = j1;
  k0.by_row = !precision && wg_by_row(j0, false);
  k1.by_row = !precision && wg_by_row(j1, false);
  k1.rot = wg_groups(k0, tile) % 8;
  const int n0 = wg_blocks(k0, tile);
  const dim3 grid(n0 + wg_blocks(k1, tile));
#define HGNN_WG(P, W)                                                                          \
  hipExtLaunchKernelGGL((k_wgrad_pair<P, W>), grid, dim3(256), 0, s, ev0, ev1, 0, dims, k0, k1, n0)
  if (!precision) HGNN_WG(0, 2);
  else if (tile == 128) HGNN_WG(1, 4);
  else HGNN_WG(1, 2);
#undef HGNN_WG
  return hipGetLastError();
}

hipError_t launch_wgrad_all(const Dims *dims, const WgJob *tab, int n, int most, int precision,
                            int tile, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  if (n <= 0 || most <= 0) return hipSuccess;
  if (most % 8 || (tile != 128 && tile != 64)) return hipErrorInvalidValue;
  const dim3 grid(most, n);
#define HGNN_WG(P, W)                                                                          \
  hipExtLaunchKernelGGL((k_wgrad_all<P, W>), grid, dim3(256), 0, s, ev0, ev1, 0, dims, tab)
  if (precision) {
    if (tile == 128) HGNN_WG(1, 4);
    else HGNN_WG(1, 2);
  } else {
    if (tile != 64) return hipErrorInvalidValue; // see wg_tile_all
    HGNN_WG(0, 2);
  }
#undef HGNN_WG
  return hipGetLastError();
}

} // namespace hgnn
