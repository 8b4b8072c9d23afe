// Strip solver of vgpr_fit_predict: every FP64 solve of more than 16 points.
//
// The voxel's points are taken in strips of 16 and K + S is factored as L L^T
// strip by strip; nothing but 16 x 16 tiles on the FP64 matrix cores, with the
// rows being solved held in registers from the kernel entries to the result.
// Sixteen columns at a time (data rows of L, or queries) a wavefront carries
//     acc(i) = K(i, cols) - sum_{j done} L(i, j) Z(j),        i = strips left,
// one 16 x 16 tile per strip in the accumulator layout of the 16 x 16 x 4
// product (lane l, register k: row l / 16 + 4 k, column l % 16). Step j takes
//     Z(j) = L(j, j)^-1 acc(j)
// and subtracts L(i, j) Z(j) from the tiles below. In that layout register k
// of Z is at once the right operand of the k-th 16 x 16 x 4 product of the
// updates, and, for data columns, the left operand that a later use of the
// finished tile L(cols, j) wants (lane l: row l % 16, column 4 k + l / 16): no
// value ever moves between lanes, a tile is stored and fetched as it lies in
// registers, and the triangular solve has no barrier.
//
// A workgroup of WV wavefronts owns one voxel. Data strips are taken WV at a
// time (wavefront w: strip r = WV S + w); the strips before them are
// eliminated by each wavefront alone, the WV x WV diagonal corner together.
// Queries go 16 to a wavefront, independently.
//
// What bounds it: FP64 arithmetic. The matrix and the vector unit share one
// FP64 pipe here (4 matrix products and 32 vector FMAs take 184 ns together,
// 117 and 67 apart), so the kernel entries count beside the products.
#pragma once

typedef double dbl2 __attribute__((ext_vector_type(2)));

constexpr int kStrip = 16;
constexpr int kTileDbl = kStrip * kStrip;  // doubles of one tile
constexpr int strip_tiles(int ns) { return ns * (ns + 1) / 2; }

// Voxels of up to 128 points keep their tiles in LDS; above that the workgroup owns a scratch area
// (256 points: 272 KB of tiles, against 160 KB of LDS).
constexpr bool strip_lds(int ns) { return ns <= 8; }
// One wavefront a voxel as long as its tiles leave room for several a CU (64 points: 20 KB), four above: 20,000
// voxels, 8 x 8 / 16 x 16 grid, four wavefronts against one: 64 points 553 / 922 us against 505 / 1,042 (400 voxels
// 75 / 90 against 85 / 120), 96 points 1,225 / 1,922 against 1,604 / 3,395, 128 points 1,895 / 3,339 against
// 3,407 / 7,963.
constexpr int strip_waves(int ns) { return ns <= 4 ? 1 : 4; }
constexpr size_t strip_scratch_doubles(int ns) { return strip_lds(ns) ? 0 : (size_t)strip_tiles(ns) * kTileDbl; }

// 2^t for t <= 0: t split into an integer and |f| <= 1/2 (exactly), 2^f by its Chebyshev
// interpolant of degree 11 (within 2.0e-17 with the coefficients as rounded here), scaled by the exponent. Far below the smallest
// exponent the result is 0, which is what the padded points rely on. (So it is for a NaN, which the caller keeps out.)
__device__ __forceinline__ double exp2_neg(double t) {
  t = fmax(t, -2000.0);  // (also keeps a product in the argument from being contracted into the subtraction)
  const double n = __builtin_rint(t);
  const double f = t - n;
  double p = 4.4558179083360645e-10;
  p = fma(p, f, 7.074194297288521e-09);
  p = fma(p, f, 1.0178057087733941e-07);
  p = fma(p, f, 1.3215432535912375e-06);
  p = fma(p, f, 1.5252733841556773e-05);
  p = fma(p, f, 0.00015403530463724353);
  p = fma(p, f, 0.001333355814640647);
  p = fma(p, f, 0.009618129107587256);
  p = fma(p, f, 0.055504108664821625);
  p = fma(p, f, 0.24022650695910158);
  p = fma(p, f, 0.6931471805599453);
  p = fma(p, f, 1.0);
  return __builtin_ldexp(p, (int)n);
}

// 1 / sqrt(d): the hardware estimate (2^-24) and one third-order step; zero, negative or NaN d gives a
// NaN or infinity that the caller's pivot test catches.
__device__ __forceinline__ double rsqrt_step(double d) {
  const double r = __builtin_amdgcn_rsq(d);
  const double e = fma(-(d * r), r, 1.0);
  return fma(r * e, fma(e, 0.375, 0.5), r);
}

// Sum over the 16 lanes of a row (lanes with the same l / 16), in every lane.
__device__ __forceinline__ double row_sum16(double v) {
#define VGPR_ROR_ADD(n)                                                                       \
  {                                                                                           \
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x120 + n, 0xf, 0xf, false); \
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x120 + n, 0xf, 0xf, false); \
    v += __hiloint2double(hi, lo);                                                            \
  }
  VGPR_ROR_ADD(8)
  VGPR_ROR_ADD(4)
  VGPR_ROR_ADD(2)
  VGPR_ROR_ADD(1)
#undef VGPR_ROR_ADD
  return v;
}

// One tile as it lies in registers: lane l's four values as two 16-byte halves, 1 KB apart. Tiles are
// addressed by address space (LDS or global), a uniform base and the lane's byte offset 16 l.
struct Tile {
  dbl2 h[2];
  __device__ __forceinline__ double operator[](int k) const { return h[k >> 1][k & 1]; }
};
template <int AS>
using TilePtr = __attribute__((address_space(AS))) char*;
constexpr int kAsGlobal = 1, kAsLds = 3;
constexpr int kTileBytes = kTileDbl * 8;

// A base address kept in scalar registers: the tile's offset is added there and the lane's offset in the
// access, so that no vector register holds an address (136 of them would be computed ahead of the voxel loop).
template <int AS>
__device__ __forceinline__ TilePtr<AS> tile_at(TilePtr<AS> T, int index) {
  if constexpr (AS == kAsGlobal) index = __builtin_amdgcn_readfirstlane(index);
  TilePtr<AS> p = T + (size_t)(uint32_t)index * kTileBytes;
  if constexpr (AS == kAsGlobal) asm volatile("" : "+s"(p));
  return p;
}
template <int AS>
__device__ __forceinline__ Tile tile_load(TilePtr<AS> T, int index, uint32_t off) {
  typedef const __attribute__((address_space(AS))) dbl2* Half;
  const TilePtr<AS> p = tile_at<AS>(T, index);
  Tile t;
  t.h[0] = *(Half)(p + off);
  t.h[1] = *(Half)(p + kTileBytes / 2 + off);
  return t;
}
template <int AS>
__device__ __forceinline__ void tile_store(TilePtr<AS> T, int index, uint32_t off, dbl4 v) {
  typedef __attribute__((address_space(AS))) dbl2* Half;
  const TilePtr<AS> p = tile_at<AS>(T, index);
  *(Half)(p + off) = dbl2{v[0], v[1]};
  *(Half)(p + kTileBytes / 2 + off) = dbl2{v[2], v[3]};
}

// A value the compiler takes as new at every use: what is computed from it is computed where it is used,
// instead of being kept in a register from before the voxel loop.
__device__ __forceinline__ int fresh(int v) {
  asm volatile("" : "+v"(v));
  return v;
}
__device__ __forceinline__ int fresh_uniform(int v) {
  asm volatile("" : "+s"(v));
  return v;
}
// A value that is the same in every lane, in scalar registers.
__device__ __forceinline__ double uniform(double v) {
  return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                          __builtin_amdgcn_readfirstlane(__double2loint(v)));
}
// The value of the lane whose number differs in the bits of `mask`.
__device__ __forceinline__ double from_lane_xor(double v, int mask, int lane) {
  const int at = (fresh(lane) ^ mask) << 2;
  return __hiloint2double(__builtin_amdgcn_ds_bpermute(at, __double2hiint(v)),
                          __builtin_amdgcn_ds_bpermute(at, __double2loint(v)));
}

// Keeps the fetches issued before it before it: the compiler would sink a fetch into the branch that uses its
// value, to wait there for all of its latency.
__device__ __forceinline__ void issued() { asm volatile("" ::: "memory"); }

// First tile (the diagonal one) of column j: tiles (j .. NS - 1, j) follow one another.
template <int NS>
__device__ __forceinline__ constexpr int tile_col(int j) {
  return j * NS - (j * (j - 1)) / 2;
}

// The elimination, written as nested conditions so that every register is named at compile time and a tile on
// its way is only ever defined on the one path that uses it (in loops, the compiler joined the strips past
// `rows` with the others through register copies that waited for the fetches, and spilled).
template <int D>
struct Ahead {
  Tile t[D];
};

// acc(i) += -L(i, J) Z(J) for i = J + 1 + K, J + 2 + K, ... below `rows`; q holds the next D tiles.
template <int NS, int D, int J, int K, int AS, typename I>
__device__ __forceinline__ void update_column(dbl4 (&acc)[NS], TilePtr<AS> T, int rows, uint32_t off, const dbl4& z,
                                              Ahead<D> q, I&& init) {
  constexpr int i = J + 1 + K;
  if constexpr (i < NS) {
    if (i < rows) {
      const Tile t = q.t[0];
      Ahead<D> n;
#pragma unroll
      for (int e = 0; e + 1 < D; ++e) n.t[e] = q.t[e + 1];
      // past the column's end the last tile again: a fetch of anything else would be waited for in its turn
      if constexpr (i + D < NS) n.t[D - 1] = tile_load<AS>(T, tile_col<NS>(J) + min(1 + K + D, rows - 1 - J), off);
      issued();
      if constexpr (J == 0) acc[i] = init(i);
#pragma unroll
      for (int s = 0; s < 4; ++s) acc[i] = mfma_f64(t[s], z[s], acc[i]);
      update_column<NS, D, J, K + 1, AS>(acc, T, rows, off, z, n, init);
    }
  }
}

// Tiles FROM .. TO - 1 of column J's window (column J has rows - J tiles, its diagonal one among them).
template <int NS, int FROM, int TO, int J, int AS, int D>
__device__ __forceinline__ void column_head(TilePtr<AS> T, int rows, uint32_t off, Ahead<D>& n) {
#pragma unroll
  for (int e = FROM; e < TO; ++e)
    if (J + 1 + e < NS) n.t[e] = tile_load<AS>(T, tile_col<NS>(J) + max(min(1 + e, rows - 1 - J), 0), off);
}

template <int NS, int D, int H, int J, int AS, typename I, typename F>
__device__ __forceinline__ void eliminate_from(dbl4 (&acc)[NS], TilePtr<AS> T, int rows_, uint32_t off, Tile w, Ahead<D> q,
                                               I&& init, F&& step) {
  if constexpr (J < NS) {
    const int rows = fresh_uniform(rows_);
    if (J < rows) {
      column_head<NS, H, D, J, AS>(T, rows, off, q);
      issued();
      dbl4 z = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int s = 0; s < 4; ++s) z = mfma_f64(w[s], acc[J][s], z);
      Tile wn{};
      Ahead<D> n;
      if constexpr (J + 1 < NS) wn = tile_load<AS>(T, J + 1 < rows ? tile_col<NS>(J + 1) : tile_col<NS>(J), off);
      column_head<NS, 0, H, J + 1, AS>(T, rows, off, n);
      issued();
      step(J, z);
      update_column<NS, D, J, 0, AS>(acc, T, rows, off, z, q, init);
      eliminate_from<NS, D, H, J + 1, AS>(acc, T, rows_, off, wn, n, init, step);
    }
  }
}

// Eliminate `rows` strips (at least one) of sixteen columns whose kernel tiles are init(i), taken when column 0
// reaches them: Z(j) goes to step(j, Z). Tiles are stored negated, so that an update adds; they are fetched D
// ahead: the inverse of the next diagonal tile and a column's first H tiles while the column before runs, the
// rest of its first D while its Z is formed.
template <int NS, int D, int H, int AS, typename I, typename F>
__device__ __forceinline__ void eliminate(TilePtr<AS> T, int rows, uint32_t off, I&& init, F&& step) {
  dbl4 acc[NS];
  Ahead<D> q;
  const Tile w = tile_load<AS>(T, 0, off);
  column_head<NS, 0, H, 0, AS>(T, rows, off, q);
  acc[0] = init(0);
  eliminate_from<NS, D, H, 0, AS>(acc, T, rows, off, w, q, init, step);
}

// cor[t] -= L(i0 + t, j) L(r, j)^T for t < C over the eliminated strips j < i0: the tiles are stored negated,
// the product of two of them is negated again.
template <int NS, int C, int AS, int M>
__device__ __forceinline__ void corner_update(dbl4 (&cor)[M], TilePtr<AS> T, int i0, int r, uint32_t off) {
  Tile bn = tile_load<AS>(T, r, off), an[C];
#pragma unroll
  for (int t = 0; t < C; ++t) an[t] = tile_load<AS>(T, i0 + t, off);
#pragma unroll 1
  for (int j = 0; j < i0; ++j) {
    const Tile b = bn;
    Tile a[C];
#pragma unroll
    for (int t = 0; t < C; ++t) a[t] = an[t];
    const int jn = min(j + 1, i0 - 1);
    const int col = tile_col<NS>(jn) - jn;
    bn = tile_load<AS>(T, col + r, off);
#pragma unroll
    for (int t = 0; t < C; ++t) an[t] = tile_load<AS>(T, col + i0 + t, off);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
#pragma unroll
      for (int t = 0; t < C; ++t) cor[t] = mfma_f64(a[t][s], -b[s], cor[t]);
    }
  }
}

// Cholesky factor and its inverse of one symmetric 16 x 16 tile D (accumulator layout), four columns at a
// time: every lane takes row r = l % 16 of the panel, factors the panel's 4 x 4 block and solves its row; the
// update of the tile is one 16 x 16 x 4 product. Identity rows ride along (F = their transpose) and end as
// L^-T, so W = L^-1 comes out: register b of lane l is W(4 b + l / 16, l % 16). Returns false on a pivot that
// is not positive. (One wavefront; about 1.2 us: the chain of 16 reciprocal square roots.)
__device__ __forceinline__ bool factor16(dbl4 D, int lane_, double (&W)[4]) {
  const int lane = fresh(lane_);
  const int l16 = lane & 15, l4 = lane >> 4;
  dbl4 F;
#pragma unroll
  for (int k = 0; k < 4; ++k) F[k] = l4 + 4 * k == l16 ? 1.0 : 0.0;
  bool ok = true;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    double p[4], f[4];  // entries 4 b + c of row l16 of the tile and of F, on their way while the pivots are found
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int at = (c * 16 + l16) << 2;
      p[c] = __hiloint2double(__builtin_amdgcn_ds_bpermute(at, __double2hiint(D[b])),
                              __builtin_amdgcn_ds_bpermute(at, __double2loint(D[b])));
      f[c] = __hiloint2double(__builtin_amdgcn_ds_bpermute(at, __double2hiint(F[b])),
                              __builtin_amdgcn_ds_bpermute(at, __double2loint(F[b])));
    }
    issued();
    auto d = [&](int r, int c) { return bcast(D[b], r * 16 + 4 * b + c); };
    const double d0 = d(0, 0), r0 = rsqrt_step(d0);
    const double l10 = d(1, 0) * r0, l20 = d(2, 0) * r0, l30 = d(3, 0) * r0;
    const double d1 = fma(-l10, l10, d(1, 1)), r1 = rsqrt_step(d1);
    const double l21 = fma(-l20, l10, d(2, 1)) * r1, l31 = fma(-l30, l10, d(3, 1)) * r1;
    const double d2 = fma(-l21, l21, fma(-l20, l20, d(2, 2))), r2 = rsqrt_step(d2);
    const double l32 = fma(-l31, l21, fma(-l30, l20, d(3, 2))) * r2;
    const double d3 = fma(-l32, l32, fma(-l31, l31, fma(-l30, l30, d(3, 3)))), r3 = rsqrt_step(d3);
    ok = ok && d0 > 0.0 && d1 > 0.0 && d2 > 0.0 && d3 > 0.0;
    // both rows together; all four entries on every lane (the chain must not be split into branches by l / 16)
    double x0 = p[0] * r0, y0 = f[0] * r0;
    double x1 = fma(-x0, l10, p[1]) * r1, y1 = fma(-y0, l10, f[1]) * r1;
    double x2 = fma(-x1, l21, fma(-x0, l20, p[2])) * r2, y2 = fma(-y1, l21, fma(-y0, l20, f[2])) * r2;
    double x3 = fma(-x2, l32, fma(-x1, l31, fma(-x0, l30, p[3]))) * r3;
    double y3 = fma(-y2, l32, fma(-y1, l31, fma(-y0, l30, f[3]))) * r3;
    asm volatile("" : "+v"(x0), "+v"(x1), "+v"(x2), "+v"(x3), "+v"(y0), "+v"(y1), "+v"(y2), "+v"(y3));
    const double ylo = l4 & 1 ? y1 : y0, yhi = l4 & 1 ? y3 : y2, y = l4 & 2 ? yhi : ylo;
    W[b] = y;
    if (b < 3) {
      const double xlo = l4 & 1 ? x1 : x0, xhi = l4 & 1 ? x3 : x2;
      // rows above the panel's diagonal are finished (their entries are rounding residue)
      const double x = l16 >= 4 * b + l4 ? (l4 & 2 ? xhi : xlo) : 0.0;
      D = mfma_f64(x, -x, D);
      F = mfma_f64(x, -y, F);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  return ok;
}

// Workgroup barrier that orders LDS only: global stores may still be on their way.
__device__ __forceinline__ void sync_lds() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Workgroups a CU to build for: what LDS and the accumulators allow. 256 points, 4,000 voxels (8 x 8 / 16 x 16 grid):
// two 1,058 / 1,715 us, one 1,449 / 2,299; 96 and 128 points as two or one are within 6%; up to 64 points three
// leave 168 registers (built for two, 64 points: 505 / 1,042 -> 483 / 969); the 512-point shape fills a CU's LDS.
template <int NS>
__global__ void __launch_bounds__(64 * strip_waves(NS), NS <= 4 ? 3 : (NS <= 16 ? 2 : 1))
    fit_strip_kernel(FitParams P, FitArgs io, const SlotRec* __restrict__ recs, const RotRec* __restrict__ rots,
                     const float4* __restrict__ staged, const int32_t* __restrict__ slots,
                     const uint32_t* __restrict__ count, uint32_t* __restrict__ fetch, double* __restrict__ scratch) {
  constexpr int WV = strip_waves(NS);
  constexpr int NT = 64 * WV;
  constexpr int N = NS * kStrip;
  constexpr bool kLds = strip_lds(NS);
  constexpr bool kTab = !kLds;              // separable query tables in LDS
  // Tiles in flight, and those of the next column among them. Tiles in scratch need them: 512 points, 1,500 voxels
  // (8 x 8 / 16 x 16 grid), D = 4 2,033 / 2,989 us, 2 2,101 / 3,174; 256 points with more than two spill, and one
  // costs 7% / 9%. From LDS one to four are within 2%. H = 0 to 4 are within 1% at 512 points.
  constexpr int D = NS >= 32 ? 4 : (NS == 2 ? 1 : 2);
  constexpr int H = NS >= 32 ? 4 : 0;
  // Rounds of queries written together, so that all lanes write: 20,000 voxels, 16 x 16 grid, four 458 and 1,042 us
  // (32 and 64 points), one 472 and 1,067. Within the spread above 64 points.
  constexpr int kBatch = NS <= 8 ? 4 : 1;
  // Voxels of up to 32 points are taken at a fixed stride: they are solved faster than the one counter gives
  // out numbers (~9 ns each; 20,000 voxels on an 8 x 8 grid 308 us, so 230). Larger ones are not, and differ
  // more (20,000 of 64 points: counter 595 us, stride 860).
  constexpr bool kStride = NS == 2;
  constexpr int TS = N + 4;                 // row stride of the query tables (16 rows 4 apart: no bank conflict)
  constexpr int kPub = kTab ? 4 * kTileDbl : 2;
  constexpr int kBig = kLds ? strip_tiles(NS) * kTileDbl : (2 * kMaxGridSide * TS > kPub ? 2 * kMaxGridSide * TS : kPub);
  __shared__ __attribute__((aligned(16))) double s_big[kBig];  // the tiles, or the query tables (data phase: pub)
  __shared__ double pu[N], pw[N], pf[N], sy[N];
  __shared__ float pn[N];
  __shared__ double s_frac[kMaxGridSide], gridu[kMaxGridSide], gridw[kMaxGridSide];
  __shared__ int s_item, s_fail;
  __shared__ unsigned s_maxvar;

  const int tid = threadIdx.x;
  const int lane = lane_id();
  const int w = WV == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int AS = kLds ? kAsLds : kAsGlobal;
  const uint32_t off = 16u * (uint32_t)lane;
  TilePtr<AS> T;
  if constexpr (kLds)
    T = (TilePtr<AS>)s_big;
  else
    T = (TilePtr<AS>)(scratch + (size_t)blockIdx.x * strip_scratch_doubles(NS));
  // kTab: the corner's tiles of the current column, so that they need not come back from memory
  const TilePtr<kAsLds> pub = (TilePtr<kAsLds>)s_big;
  const int items = (int)*count;
  const double sf2 = uniform((double)P.sf2);
  auto sync = [] {
    if constexpr (WV == 1)
      wave_sync();
    else
      __syncthreads();
  };

  if (tid < P.nq) s_frac[tid] = grid_frac(P, tid);
  if (tid == 0) {  // for the first voxel; the end of each clears them for the next
    s_fail = 0;
    s_maxvar = 0u;
  }
  sync();
  int item = (int)blockIdx.x;
  while (item < items) {
    const int slot = slots ? slots[item] : item;
    const SlotRec rec = recs[slot];
    const FrameRec& fr = rec.fr;
    const RotRec* rot = rots ? rots + slot : nullptr;
    const int n = fr.n;
    const int nb = (n + kStrip - 1) / kStrip;
    // coordinates scaled so that kappa = s_f^2 2^-(du^2 + dw^2); the padding points lie so far from the
    // data, the queries and each other that their kernel entries are zero
    const double lam2 = fr.lam * 1.4426950408889634;
    const double sc = uniform(lam2 * rsqrt_step(lam2));
    if (const int i = fresh(tid); i < P.nq) {
      float gu, gw;
      coords_from_frac(P, fr, s_frac[i], s_frac[i], &gu, &gw);
      gridu[i] = ((double)gu - fr.anc_u) * sc;
      gridw[i] = ((double)gw - fr.anc_w) * sc;
    }
    for (int i = fresh(tid); i < nb * kStrip; i += NT) {
      double xu = 1e30 * (i + 1), xw = 0.0, fv = 0.0;
      float nz = 0.f;
      if (i < n) {
        const float4 pt = staged[rec.off + i];
        local_point(P, fr, rot, pt, &xu, &xw, &fv);
        xu *= sc;
        xw *= sc;
        nz = pt.w;
        // a point that is not finite fails its voxel here: exp2_neg would make 0 of a NaN distance, and an
        // infinite pivot in the last place is positive and followed by none
        if (!(isfinite(xu) && isfinite(xw) && isfinite(fv) && isfinite(nz))) s_fail = 1;
      }
      pu[i] = xu;
      pw[i] = xw;
      pf[i] = fv;
      pn[i] = nz;
    }
    sync();

    auto entry = [&](int row, double xu, double xw) {
      const double du = pu[row] - xu, dw = pw[row] - xw;
      return sf2 * exp2_neg(-fma(du, du, dw * dw));
    };
    // the 16 x 16 tile of kernel entries of strip i against the points (xu, xw) of this lane's column
    auto kernel_tile = [&](int i, double xu, double xw) {
      dbl4 v;
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = entry(i * kStrip + (lane >> 4) + 4 * k, xu, xw);
      __builtin_amdgcn_sched_barrier(0);  // a few entries at a time: registers
      return v;
    };
    const int njobs = (nb + WV - 1) / WV;                     // rounds of WV data strips
    const int nqueries = (P.m + WV * kStrip - 1) / (WV * kStrip);  // rounds of WV x 16 queries
    float maxvar = 0.f;
    double qzz = 0.0, qzy = 0.0;  // up to four rounds' sums of this lane's query
    uint32_t ahead = 0;
#pragma unroll 1
    for (int job = 0; job < njobs + nqueries; ++job) {
      const bool data = job < njobs;
      if (job == njobs) {
        // the next voxel's number is fetched while the queries run: by now the workgroups are apart (all of
        // them asking as they start waited up to 40 us on the one counter)
        if (!kStride && tid == 0) ahead = items > (int)gridDim.x ? gridDim.x + atomicAdd(fetch, 1u) : (uint32_t)items;
        sync();  // the factor is complete
        if constexpr (kTab) {
          // kappa factors over the grid's rows and columns: two tables of n_q x n entries
          double* tu = s_big;
          double* tw = s_big + kMaxGridSide * TS;
          for (int i = 0; i < P.nq; ++i) {
            const double qu = gridu[i], qw = gridw[i];
            for (int c = fresh(tid); c < nb * kStrip; c += NT) {
              const double du = qu - pu[c], dw = qw - pw[c];
              tu[i * TS + c] = sf2 * exp2_neg(-(du * du));
              tw[i * TS + c] = exp2_neg(-(dw * dw));
            }
          }
          sync();
        }
      }
      const int i0 = job * WV;             // data: first strip of the round
      const int r = i0 + w;                // data: this wavefront's strip
      const int rows = data ? i0 : nb;     // strips to eliminate
      const int q0 = ((job - njobs) * WV + w) * kStrip;  // queries: the wavefront's first
      const bool active = data ? r < nb : q0 < P.m;
      dbl4 own = {0.0, 0.0, 0.0, 0.0};     // data: K + S of the strip with itself, minus the eliminated strips
      dbl4 cor[WV > 1 ? WV - 1 : 1];       // data: ... and of the round's earlier strips with it
      double zy = 0.0, zz = 0.0;           // sums of Z y and Z^2 over this lane's rows
      if (active) {
        const int l16 = fresh(lane) & 15;
        double xu, xw;
        const double* tu = nullptr;
        const double* tw = nullptr;
        if (data) {
          xu = pu[r * kStrip + l16];
          xw = pw[r * kStrip + l16];
          const double nz = (double)pn[r * kStrip + l16];
          const int l4 = fresh(lane) >> 4;
          own = kernel_tile(r, xu, xw);
#pragma unroll
          for (int k = 0; k < 4; ++k)
            if (l4 + 4 * k == l16) own[k] += nz;
          if constexpr (kTab) {
            // the kernel tiles wait where the tiles of L that replace them go
#pragma unroll 1
            for (int i = 0; i < rows; ++i) tile_store<AS>(T, tile_col<NS>(i) + r - i, off, kernel_tile(i, xu, xw));
          }
        } else {
          const int q = q0 + l16 < P.m ? q0 + l16 : P.m - 1;
          const int qi = q / P.nq, qj = q - qi * P.nq;
          xu = gridu[qi];
          xw = gridw[qj];
          if constexpr (kTab) {
            tu = s_big + qi * TS + (fresh(lane) >> 4);
            tw = s_big + (kMaxGridSide + qj) * TS + (fresh(lane) >> 4);
          }
        }
        if (rows > 0) {
          const double* ys = sy + (fresh(lane) >> 4);
          eliminate<NS, D, H, AS>(
              T, rows, off,
              [&](int i) {
                if constexpr (kTab) {
                  dbl4 v;
                  if (data) {
                    const Tile t = tile_load<AS>(T, tile_col<NS>(i) + r - i, off);
#pragma unroll
                    for (int k = 0; k < 4; ++k) v[k] = t[k];
                  } else {
#pragma unroll
                    for (int k = 0; k < 4; ++k) v[k] = tu[i * kStrip + 4 * k] * tw[i * kStrip + 4 * k];
                  }
                  return v;
                } else {
                  return kernel_tile(i, xu, xw);
                }
              },
              [&](int j, dbl4 z) {
#pragma unroll
                for (int k = 0; k < 4; ++k) zy = fma(z[k], ys[j * kStrip + 4 * k], zy);
                if (data) {
                  const dbl4 m = -z;
                  tile_store<AS>(T, tile_col<NS>(j) + r - j, off, m);
#pragma unroll
                  for (int k = 0; k < 4; ++k) own = mfma_f64(z[k], m[k], own);
                } else {
#pragma unroll
                  for (int k = 0; k < 4; ++k) zz = fma(z[k], z[k], zz);
                }
              });
        }
        if constexpr (WV > 1) {
          if (data) {
            const int at = r * kStrip + (fresh(lane) & 15);  // read again: two values less to hold until here
            xu = pu[at];
            xw = pw[at];
#pragma unroll
            for (int t = 0; t < WV - 1; ++t)
              if (t < w) cor[t] = kernel_tile(i0 + t, xu, xw);
          }
        }
      }
      if (!data) {
        // the round's 16 queries: their sums over the rows go to the lanes with l / 16 = round % kBatch, so that
        // kBatch rounds are written together, one query a lane
        const int round = job - njobs;
        zz += from_lane_xor(zz, 16, lane);
        zy += from_lane_xor(zy, 16, lane);
        zz += from_lane_xor(zz, 32, lane);
        zy += from_lane_xor(zy, 32, lane);
        const int l4 = fresh(lane) >> 4, at = round & (kBatch - 1);
        if (kBatch == 1 || l4 == at) {
          qzz = zz;
          qzy = zy;
        }
        if (at == kBatch - 1 || round + 1 == nqueries) {
          const int q = ((round - at + l4) * WV + w) * kStrip + (fresh(lane) & 15);
          if (l4 <= at && q < P.m) {
            const int qi = q / P.nq, qj = q - qi * P.nq;
            float gu, gw;
            coords_from_frac(P, fr, s_frac[qi], s_frac[qj], &gu, &gw);
            const bool failed = s_fail != 0;
            const double var = sf2 - qzz;
            const float vv = failed ? __int_as_float(0x7fc00000) : (float)(var > 0.0 ? var : 0.0);
            const double fh = failed ? (double)__int_as_float(0x7fc00000) : fr.mu + qzy;
            reinterpret_cast<float4*>(io.out)[(size_t)rec.v * P.m + q] = make_row(P, fr, rot, fh, gu, gw, vv);
            maxvar = fmaxf(maxvar, failed ? 0.f : vv);
          }
        }
        continue;
      }
      if constexpr (WV > 1) {
        if (i0 > 0) {
          sync();  // every strip's tiles are stored
          if (active) {
            if (w == 1) corner_update<NS, 1, AS>(cor, T, i0, r, off);
            if (w == 2) corner_update<NS, 2, AS>(cor, T, i0, r, off);
            if (w == 3) corner_update<NS, 3, AS>(cor, T, i0, r, off);
          }
        }
      }
      // the corner: strip by strip, the strip's own wavefront factors its diagonal tile, the later strips
      // take their tile of that column
#pragma unroll
      for (int t = 0; t < WV; ++t) {
        const int it = i0 + t;
        if (w == t && active) {
          double W[4];
          const bool ok = factor16(own, lane, W);
          if (!ok) s_fail = 1;
          const int l16 = fresh(lane) & 15, l4 = fresh(lane) >> 4;
          // the right-hand side's rows, then y = W rhs
          zy += from_lane_xor(zy, 16, lane);
          zy += from_lane_xor(zy, 32, lane);
          const double g = pf[it * kStrip + l16] - zy;
          // element (4 b + l / 16, l % 16) of W goes where a left operand's lanes read it
          const int at = (l16 >> 3) * 128 + ((l16 & 3) * 16 + l4) * 2 + ((l16 >> 2) & 1);
          typedef __attribute__((address_space(AS))) double* Elem;
          const Elem Wt = (Elem)(T + (size_t)tile_col<NS>(it) * kTileBytes) + at;
#pragma unroll
          for (int b = 0; b < 4; ++b) {
            const double y = row_sum16(W[b] * g);
            if (l16 == 0) sy[it * kStrip + 4 * b + l4] = y;
            Wt[8 * b] = W[b];
            if constexpr (kTab) s_big[at + 8 * b] = W[b];
          }
        }
        if constexpr (WV > 1) {
          if (it + 1 >= nb) break;  // no later strip (the same for every wavefront)
          if (t + 1 == WV) {
            sync();  // the next round reads this one's tiles
          } else {
            sync_lds();
            dbl4 z = {0.0, 0.0, 0.0, 0.0};
            if (w > t && active) {
              const Tile wt = kTab ? tile_load<kAsLds>(pub, 0, off) : tile_load<AS>(T, tile_col<NS>(it), off);
#pragma unroll
              for (int s = 0; s < 4; ++s) z = mfma_f64(wt[s], cor[t][s], z);
              const dbl4 m = -z;
              tile_store<AS>(T, tile_col<NS>(it) + r - it, off, m);
              if constexpr (kTab) {
                if (w < WV - 1) tile_store<kAsLds>(pub, w, off, m);
              }
              const int l4 = fresh(lane) >> 4;
#pragma unroll
              for (int k = 0; k < 4; ++k) {
                zy = fma(z[k], sy[it * kStrip + l4 + 4 * k], zy);
                own = mfma_f64(z[k], m[k], own);
              }
            }
            sync_lds();
            if (active) {
#pragma unroll
              for (int t2 = t + 1; t2 < WV - 1; ++t2)
                if (t2 < w) {
                  const Tile a =
                      kTab ? tile_load<kAsLds>(pub, t2, off) : tile_load<AS>(T, tile_col<NS>(it) + t2 - t, off);
#pragma unroll
                  for (int s = 0; s < 4; ++s) cor[t2] = mfma_f64(a[s], z[s], cor[t2]);
                }
            }
          }
        }
      }
      if constexpr (WV == 1) sync();
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) maxvar = fmaxf(maxvar, __shfl_xor(maxvar, d, 64));
    if (lane == 0) atomicMax(&s_maxvar, __float_as_uint(maxvar));
    if (!kStride && tid == 0) s_item = (int)ahead;
    sync();
    if (tid == 0) {
      finish_voxel(P, io, rec.v, slot, rec.cnt, fr.axes, s_fail != 0, false, __uint_as_float(s_maxvar), nullptr, nullptr);
      s_fail = 0;
      s_maxvar = 0u;
    }
    item = kStride ? item + (int)gridDim.x : __builtin_amdgcn_readfirstlane(s_item);
    sync();
  }
}
