// Block (s-step) form of the modified Arnoldi process of Section 5.2, step
// (iv), for FP64 Krylov columns.
//
// One block takes the composite basis Q = (S_m v_1 .. v_k) from p = m + k + 1
// to p + s columns.  q_{p-1} = v_{k+1} is the newest column, not yet
// multiplied by A:
//   * Krylov directions from the Chebyshev recurrence on [-e, e] (e a bound
//     of A's spectral radius, so the directions stay well conditioned):
//       W_0 = q_{p-1},  W_1 = A W_0 / e,  W_{i+1} = 2 A W_i / e - W_{i-1},
//     that is A W_{0..s-1} = W_{0..s} Th with Th the (s+1) x s tridiagonal
//     matrix of the recurrence (Th[1][0] = e, Th[j-1][j] = Th[j+1][j] = e/2);
//   * block classical Gram-Schmidt against Q with one full second pass:
//       C1 = Q^dag W, W -= Q C1;  C2 = Q^dag W, G = W^dag W, W -= Q C2;
//     R = chol(G - C2^dag C2) (upper), new columns q_p .. q_{p+s-1} = W R^-1;
//   * the Hessenberg columns p-1 .. p+s-2 from the change of basis: with
//       Rc = [e_{p-1} | (C1 + C2; R)]   ((p + s) x (s + 1), W_{0..s} = Q Rc)
//     A Q Rc' = Q Rc Th (Rc' its first s columns), and A's action on the
//     first p - 1 columns is the known H_{p x (p-1)}, so
//       H(:, p-1 .. p+s-2) = (Rc Th - [H_{p x (p-1)} Rc'_top; 0]) Rb^-1,
//     Rb = rows p-1 .. p+s-2 of Rc' (upper triangular, diagonal 1, R_ii).
// In exact arithmetic this is the Krylov space, basis and Hessenberg matrix
// of the one-vector process (A Q_k = Q_{k+1} Hbar_k, Eq. eq:modArnoldi): the
// Schur columns enter through A S = S T, which the T block of H records.  It
// reads Q four times per block of s steps instead of twice per step.
//
// The two block products are tall and skinny (Q^dag W: p x N times N x s;
// Q C: N x p times p x s), so they run on the FP64 matrix cores
// (v_mfma_f64_16x16x4f64) with the real and imaginary parts of 8 block
// vectors side by side in the 16-wide dimension (s <= 16: two halves): two
// real products per 16 x 4 fragment of Q and half give the complex result
// without cross-lane sums.
// Every sum has a fixed order, so results do not depend on the launch.
//
// A launch carries one or several right-hand sides of one field at the same
// basis size (the batched applies advance in lockstep): the Schur columns S
// are shared, each source has its own Krylov columns V_r, block vectors,
// coefficients, factors and Hessenberg matrix at fixed strides, and the
// launch position z (fastest in the workgroup numbering, so that the
// workgroups reading the same rows of S run together) selects slot act[z].
// Per slot the arithmetic does not depend on the other slots.
#include "internal.h"
#include "context.h"
#include "rowchunks.h"

typedef double v4d __attribute__((ext_vector_type(4)));

// A complex zero in device memory for lanes outside the block (their loads
// read it, so every load is issued unconditionally; see zgemm.hip)
__device__ double2 sgn_block_zero_entry;

namespace {

__device__ inline v4d mfma(double a, double b, v4d c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }

// Loads through pointers known to address device (global) memory: global
// rather than flat instructions, which would also wait on the LDS counter.
typedef double d2v __attribute__((ext_vector_type(2)));
typedef const d2v __attribute__((address_space(1)))* gptr;
__device__ inline gptr to_global(const double2* p) { return (gptr)p; }
__device__ inline double2 gload(gptr p) {
  const d2v v = *p;
  return make_double2(v.x, v.y);
}

// k-steps whose loads a lane issues together in the block products
constexpr int kUnroll = 8;
// tiles of 16 columns per wavefront of the packed dot pass (sharing the
// block-vector loads)
constexpr int kDotTiles = 2;
// tiles per wavefront of the three-multiplication dot pass in a launch of
// kWideFrom or more slots (the block-vector loads shared by four tiles);
// launches of fewer slots take two, or one where two would leave CUs idle
constexpr int kDot3Tiles = 4;
// workgroups that fill the chip
constexpr int kFullChip = 512;
// slots from which a launch takes the wide tiles
constexpr int kWideFrom = 4;
// The three-multiplication update pass takes whole rows per wavefront (else a
// quarter of the columns) in launches of kWholeRows rows over all slots, which
// fill the chip so and whose short bases leave a quarter few products, and from
// kWholeEntries entries of basis over all slots on: past the 256 MB of the
// Infinity Cache, where reading 2048 adjacent bytes of a column per workgroup
// instead of 256 counts; there a wavefront has kRowBlocks blocks of 16 rows,
// below one.  us by events, split / whole: 6^4 x 8 slots, 116 columns, 14.5 M
// entries 50 / 55, 196 columns, 24.5 M 91 / 86, 340 columns 152 / 139; x 4, 340
// columns, 21.2 M 73 / 71; x 3, 15.9 M 48 / 55.  All updates of a short apply,
// split / one / two blocks of rows (the former kernel): 12^4 x 4, 32 columns 703 /
// 598 / 615 us (587), x 1, 48 columns 272 / 250 / 257 (234); 1680 sites x 8, 161280
// rows, 48 columns 214 / 204 / - (198); 8^4 x 3, 147456 rows, 48 columns 172 / 166 /
// 176 (167), 300 columns 3.33 / 3.33 / - ms (3.44); 6^4 x 8, 124416 rows, 160 columns
// 890 / 912 / - us (870); 6^4 x 7 780 / 822 / - (800).
constexpr int kRowBlocks = 2;
constexpr double kWholeEntries = 20e6, kWholeRows = 1.5e5;

// the composite basis of one launch: column c < m is S[c], column c >= m of
// slot r is V_r[c - m] (V_r = V + r vstride), all with leading dimension ldq
struct BlockGeo {
  const double2* S;
  const double2* V;
  size_t vstride;
  size_t ldq;
  int m, p, s, N;
  int nb;
  int act[kMaxBatch];
};

// Workgroup i runs on XCD i % 8 (round-robin dispatch).  Map i to (tile b,
// launch position z, index k) so that the workgroups of one tile and position
// run on one XCD, whose L2 then serves what they share (the slot's block
// vectors for every column group, and the rows of the Schur columns for every
// slot where all positions have the same tile there): with j = z + nb k,
// i = 8 (j + nb nk q) + x -> b = 8 q + x.  With few tiles some XCDs would have
// one more than others, so where the shares would differ by more than an eighth
// position z counts its tiles on from z ntiles (elsewhere the slots share the
// Schur rows: 6^4 x 8 slots, 31 chunks, HBM traffic of the dot pass 1.02 of the
// algorithmic bytes, 1.11 if they counted on).  The update passes take the
// tiles downwards, so that what the dot pass read last is still in the caches
// (and what they read last, for the next dot pass).  A grid of 8 nb nk
// ceil(ntiles / 8) workgroups covers every (b, z, k) once; false for the
// padding (b >= ntiles).
__device__ inline bool uneven(int ntiles) { return 8 * ((ntiles + 7) >> 3) > ntiles + (ntiles >> 3); }
template <bool DOWN>
__device__ inline bool xcd_tile(int i, int nb, int nk, int ntiles, int& b, int& z, int& k) {
  const int x = i & 7, l = i >> 3, up = l / (nb * nk), j = l - up * nb * nk;
  const int q = DOWN ? ((ntiles - 1) >> 3) - up : up;
  k = j / nb;
  z = j - k * nb;
  b = 8 * q + (uneven(ntiles) ? (x - z * ntiles) & 7 : x);
  return b < ntiles;
}
inline unsigned xcd_grid(int per, int ntiles) { return 8u * (unsigned)per * (unsigned)((ntiles + 7) / 8); }

__device__ inline const double2* qcol(const double2* S, const double2* Vr, int m, size_t ldq, int c) {
  return c < m ? S + (size_t)c * ldq : Vr + (size_t)(c - m) * ldq;
}

__device__ inline double2 wsum2(double2 v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    v.x += __shfl_xor(v.x, off, 64);
    v.y += __shfl_xor(v.y, off, 64);
  }
  return v;
}

// v_1 = u * inv per slot: the first Krylov column
__global__ void bstart_kernel(BlockGeo g, const double2* __restrict__ u, size_t ustride,
                              const double* __restrict__ inv, int istride) {
  const int z = blockIdx.y, r = g.act[z];
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= g.N) return;
  double2* v = const_cast<double2*>(g.V) + (size_t)r * g.vstride;
  v[i] = cscale(u[(size_t)r * ustride + i], inv[(size_t)r * istride]);
}

// ---------------------------------------------------------------------------
// The s <= 16 block vectors fill the matrix instruction's 16-wide dimension
// in halves of 8: half h holds vectors 8 h .. 8 h + 7, real parts in rows
// (or columns) 0..7 and imaginary parts in 8..15.  kHalves halves cover
// kBlockMax vectors; a launch uses nh = ceil(s / 8) of them.
constexpr int kHalves = kBlockMax / 8;

// dot pass: partial sums of conj(col_c) . W_v over row chunks.  Columns c < p
// are the basis; with ncol = p + s, columns p + u are W_u (the Gram matrix).
// Wavefront: 32 columns (two tiles of 16 sharing the A fragments) x rpw
// rows; lane (li, lk) = (lane % 16, lane / 16) holds, per k-step of four
// rows, row lk of column li of each tile (B fragment) and, per half, of
// block vector 8 h + li % 8, real part for li < 8, imaginary for li >= 8 (A
// fragment).  D1 = A Re(Q), D2 = A Im(Q) give
//   Re C[j][v] = D1[v][j] + D2[v+8][j],  Im C[j][v] = D1[v+8][j] - D2[v][j].
// Workgroup: four wavefronts on consecutive row ranges, summed in order.
struct BDot {
  const double2* W;  // slot block vectors, ld ldq
  size_t wstride;
  int ncol;
  int rpw;  // rows per wavefront, a multiple of 4
  int ncg;  // column groups
  int nch;  // row chunks
  double2* part;  // per slot [chunk][ncol][kBlockMax]
  size_t pstride;
};

__global__ void __launch_bounds__(256) bdot_kernel(BlockGeo g, BDot a) {
  // tile = row chunk: all slots and column groups of a chunk on one XCD
  int chunk, z, cg;
  if (!xcd_tile<false>(blockIdx.x, g.nb, a.ncg, a.nch, chunk, z, cg)) return;
  const int r = g.act[z];
  const double2* Vr = g.V + (size_t)r * g.vstride;
  const double2* Wr = a.W + (size_t)r * a.wstride;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const int v = li & 7;
  const bool imag = li >= 8;
  const int nh = (g.s + 7) >> 3;  // halves in use (uniform)
  const int r0 = (chunk * 4 + wave) * a.rpw;
  const int r1 = min(r0 + a.rpw, g.N);
  const int nit = r1 > r0 ? (r1 - r0) >> 2 : 0;
  // a column past ncol reads column ncol - 1 (its sums are not written)
  const double2* qp[kDotTiles];
#pragma unroll
  for (int t = 0; t < kDotTiles; ++t) {
    const int cc = min((cg * kDotTiles + t) * 16 + li, a.ncol - 1);
    qp[t] = (cc < g.p ? qcol(g.S, Vr, g.m, g.ldq, cc) : Wr + (size_t)(cc - g.p) * g.ldq) + r0 + lk;
  }
  // the A fragments: the lane's real or imaginary part, loaded as one double
  const double* wp[kHalves];
  int dw[kHalves];
#pragma unroll
  for (int h = 0; h < kHalves; ++h) {
    const bool vok = 8 * h + v < g.s;
    wp[h] = vok ? reinterpret_cast<const double*>(Wr + (size_t)(8 * h + v) * g.ldq + r0 + lk) + (imag ? 1 : 0)
                : reinterpret_cast<const double*>(&sgn_block_zero_entry);
    dw[h] = vok ? 8 : 0;  // four rows, in doubles
  }
  v4d d1[kHalves][kDotTiles], d2[kHalves][kDotTiles];
#pragma unroll
  for (int h = 0; h < kHalves; ++h)
#pragma unroll
    for (int t = 0; t < kDotTiles; ++t) {
      d1[h][t] = v4d{0.0, 0.0, 0.0, 0.0};
      d2[h][t] = v4d{0.0, 0.0, 0.0, 0.0};
    }
  constexpr int U = kUnroll / 2;
  int it = 0;
  for (; it + U <= nit; it += U) {
    double2 qv[U][kDotTiles];
    double wv[U][kHalves];
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int t = 0; t < kDotTiles; ++t) qv[u][t] = qp[t][4 * u];
#pragma unroll
      for (int h = 0; h < kHalves; ++h) wv[u][h] = wp[h][dw[h] * u];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int h = 0; h < kHalves; ++h)
        if (h < nh)
#pragma unroll
          for (int t = 0; t < kDotTiles; ++t) {
            d1[h][t] = mfma(wv[u][h], qv[u][t].x, d1[h][t]);
            d2[h][t] = mfma(wv[u][h], qv[u][t].y, d2[h][t]);
          }
#pragma unroll
    for (int t = 0; t < kDotTiles; ++t) qp[t] += 4 * U;
#pragma unroll
    for (int h = 0; h < kHalves; ++h) wp[h] += U * dw[h];
  }
  for (; it < nit; ++it) {
    double wv[kHalves];
#pragma unroll
    for (int h = 0; h < kHalves; ++h) wv[h] = *wp[h];
#pragma unroll
    for (int t = 0; t < kDotTiles; ++t) {
      const double2 qv = *qp[t];
#pragma unroll
      for (int h = 0; h < kHalves; ++h)
        if (h < nh) {
          d1[h][t] = mfma(wv[h], qv.x, d1[h][t]);
          d2[h][t] = mfma(wv[h], qv.y, d2[h][t]);
        }
      qp[t] += 4;
    }
#pragma unroll
    for (int h = 0; h < kHalves; ++h) wp[h] += dw[h];
  }
  // lane (j = li, lk): items of half h's D hold rows lk + 4 t: vectors
  // 8 h + lk and 8 h + lk + 4
  __shared__ double2 red[4][64][2 * kDotTiles * kHalves];
  double2 cs[kDotTiles][kHalves][2];
#pragma unroll
  for (int t = 0; t < kDotTiles; ++t)
#pragma unroll
    for (int h = 0; h < kHalves; ++h) {
      cs[t][h][0] = make_double2(d1[h][t][0] + d2[h][t][2], d1[h][t][2] - d2[h][t][0]);
      cs[t][h][1] = make_double2(d1[h][t][1] + d2[h][t][3], d1[h][t][3] - d2[h][t][1]);
      red[wave][lane][(t * kHalves + h) * 2] = cs[t][h][0];
      red[wave][lane][(t * kHalves + h) * 2 + 1] = cs[t][h][1];
    }
  __syncthreads();
  if (wave != 0) return;
#pragma unroll
  for (int t = 0; t < kDotTiles; ++t) {
    const int c = (cg * kDotTiles + t) * 16 + li;
    if (c >= a.ncol) continue;
    double2* o = a.part + (size_t)r * a.pstride + ((size_t)chunk * a.ncol + c) * kBlockMax;
#pragma unroll
    for (int h = 0; h < kHalves; ++h) {
      double2 c0 = cs[t][h][0], c1 = cs[t][h][1];
#pragma unroll
      for (int w = 1; w < 4; ++w) {
        c0 = cadd(c0, red[w][lane][(t * kHalves + h) * 2]);
        c1 = cadd(c1, red[w][lane][(t * kHalves + h) * 2 + 1]);
      }
      // vectors past s have zero fragments, so their sums are zero
      o[8 * h + lk] = c0;
      o[8 * h + lk + 4] = c1;
    }
  }
}

// The dot pass for s > 8 with three real products per fragment (the
// Gauss form of the complex product): lane (li, lk) holds row lk of block
// vector li (A fragment, both parts) and of column li of each tile (B
// fragment);
//   T1 = Wr^T Re(Q),  T2 = Wi^T Im(Q),  T3 = (Wr + Wi)^T (Re(Q) - Im(Q)),
//   Re C = T1 + T2,  Im C = T3 - T1 + T2,
// a quarter fewer matrix-core instructions than two halves of 8.
template <int T>
__global__ void __launch_bounds__(256) bdot3_kernel(BlockGeo g, BDot a) {
  int chunk, z, cg;
  if (!xcd_tile<false>(blockIdx.x, g.nb, a.ncg, a.nch, chunk, z, cg)) return;
  const int r = g.act[z];
  const double2* Vr = g.V + (size_t)r * g.vstride;
  const double2* Wr = a.W + (size_t)r * a.wstride;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const int r0 = (chunk * 4 + wave) * a.rpw;
  const int r1 = min(r0 + a.rpw, g.N);
  const int nit = r1 > r0 ? (r1 - r0) >> 2 : 0;
  gptr qp[T];
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int cc = min((cg * T + t) * 16 + li, a.ncol - 1);
    qp[t] = to_global((cc < g.p ? qcol(g.S, Vr, g.m, g.ldq, cc) : Wr + (size_t)(cc - g.p) * g.ldq) + r0 + lk);
  }
  const bool vok = li < g.s;
  gptr wp = to_global(vok ? Wr + (size_t)li * g.ldq + r0 + lk : &sgn_block_zero_entry);
  const int dw = vok ? 4 : 0;
  v4d t1[T], t2[T], t3[T];
#pragma unroll
  for (int t = 0; t < T; ++t) {
    t1[t] = v4d{0.0, 0.0, 0.0, 0.0};
    t2[t] = v4d{0.0, 0.0, 0.0, 0.0};
    t3[t] = v4d{0.0, 0.0, 0.0, 0.0};
  }
  // groups of U k-steps, the loads of the next group issued before the
  // products of the current one (two register sets)
  constexpr int U = T == 1 ? kUnroll / 2 : kUnroll / 4;
  auto load = [&](double2 (&qv)[U][T], double2 (&wv)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int t = 0; t < T; ++t) qv[u][t] = gload(qp[t] + 4 * u);
      wv[u] = gload(wp + dw * u);
    }
#pragma unroll
    for (int t = 0; t < T; ++t) qp[t] += 4 * U;
    wp += U * dw;
  };
  auto mul = [&](const double2 (&qv)[U][T], const double2 (&wv)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const double ws = wv[u].x + wv[u].y;
#pragma unroll
      for (int t = 0; t < T; ++t) {
        t1[t] = mfma(wv[u].x, qv[u][t].x, t1[t]);
        t2[t] = mfma(wv[u].y, qv[u][t].y, t2[t]);
        t3[t] = mfma(ws, qv[u][t].x - qv[u][t].y, t3[t]);
      }
    }
  };
  int it = 0;
  {
    double2 qa[U][T], wa[U], qb[U][T], wb[U];
    if (nit >= U) load(qa, wa);
    for (; it + 2 * U <= nit; it += 2 * U) {
      load(qb, wb);
      mul(qa, wa);
      if (it + 3 * U <= nit) load(qa, wa);
      mul(qb, wb);
    }
    if (it + U <= nit) {
      mul(qa, wa);
      it += U;
    }
  }
  for (; it < nit; ++it) {
    const double2 wv = gload(wp);
    const double ws = wv.x + wv.y;
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const double2 qv = gload(qp[t]);
      t1[t] = mfma(wv.x, qv.x, t1[t]);
      t2[t] = mfma(wv.y, qv.y, t2[t]);
      t3[t] = mfma(ws, qv.x - qv.y, t3[t]);
      qp[t] += 4;
    }
    wp += dw;
  }
  // lane (j = li, lk): item q holds vector lk + 4 q of column j
  __shared__ double2 red[4][64][4 * T];
  double2 cs[T][4];
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      cs[t][q] = make_double2(t1[t][q] + t2[t][q], t3[t][q] - t1[t][q] + t2[t][q]);
      red[wave][lane][4 * t + q] = cs[t][q];
    }
  __syncthreads();
  if (wave != 0) return;
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int c = (cg * T + t) * 16 + li;
    if (c >= a.ncol) continue;
    double2* o = a.part + (size_t)r * a.pstride + ((size_t)chunk * a.ncol + c) * kBlockMax;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      double2 acc = cs[t][q];
#pragma unroll
      for (int w = 1; w < 4; ++w) acc = cadd(acc, red[w][lane][4 * t + q]);
      o[lk + 4 * q] = acc;  // zero for vectors past s
    }
  }
}

// sum of the dot partials over chunks in a fixed order: 32 entries per
// workgroup, 8 threads per entry (every 8th chunk), then the 8 in order.
// Entry e = c * kBlockMax + v; c < p goes to C[c][v] (and C1[c][v] + C[c][v]
// to Ct[c][v] if Ct), c >= p to G[c - p][v].
struct BRed {
  const double2* part;
  size_t pstride;
  int nchunk, nent, nblk;
  double2* C;
  const double2* C1;
  double2* Ct;
  size_t cstride;
  double2* G;
  size_t gstride;
};

__global__ void __launch_bounds__(256) bred_kernel(BlockGeo g, BRed a) {
  const int z = blockIdx.x % g.nb, blk = blockIdx.x / g.nb;
  const int r = g.act[z];
  const double2* __restrict__ part = a.part + (size_t)r * a.pstride;
  const int el = threadIdx.x & 31, q = threadIdx.x >> 5;
  const int e = blk * 32 + el;
  const int nchunk = a.nchunk, nent = a.nent;
  double2 acc = make_double2(0.0, 0.0);
  if (e < nent)
    for (int t0 = q; t0 < nchunk; t0 += 64) {
      double2 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int t = t0 + 8 * u;
        const double2 x = part[(size_t)min(t, nchunk - 1) * nent + e];
        v[u] = make_double2(t < nchunk ? x.x : 0.0, t < nchunk ? x.y : 0.0);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) acc = cadd(acc, v[u]);
    }
  __shared__ double2 rs[8][33];
  rs[q][el] = acc;
  __syncthreads();
  if (q == 0 && e < nent) {
    double2 t = rs[0][el];
    for (int w = 1; w < 8; ++w) t = cadd(t, rs[w][el]);
    const int c = e / kBlockMax;
    const size_t co = (size_t)r * a.cstride;
    if (c < g.p) {
      a.C[co + e] = t;
      if (a.Ct) a.Ct[co + e] = cadd(a.C1[co + e], t);
    } else {
      a.G[(size_t)r * a.gstride + e - g.p * kBlockMax] = t;
    }
  }
}

// ---------------------------------------------------------------------------
// Q C on the matrix cores: 16 rows of the composite basis (S, Vr; ld ldq)
// times the coefficients C[c][v] of columns c < ncol, for the k-steps (four
// columns) k0, k0 + dk, ... .  Lane (li, lk) holds row li of column
// 4 ks + lk (A fragment) and that column's coefficient for block vector
// 8 h + li % 8 of each half h (B fragments), so that
//   D[h] += Re(Q) [Re C | Im C] + Im(Q) [-Im C | Re C]
// is [Re | Im] of (Q C) for the 16 rows and half h's 8 vectors (rows lk + 4 t
// in item t, vector 8 h + li % 8, real part for li < 8).  Columns past ncol
// read the zero entry; halves h >= nh are skipped.
__device__ inline void qc_steps(const double2* __restrict__ S, const double2* __restrict__ Vr, int m, size_t ldq,
                                int row, int ncol, const double2* __restrict__ C, int v, bool imag, int s, int lk,
                                int k0, int dk, v4d (&d)[kHalves]) {
  const double2* zero = &sgn_block_zero_entry;
  const int nk = (ncol + 3) >> 2;
  const int nh = (s + 7) >> 3;
  bool vok[kHalves];
#pragma unroll
  for (int h = 0; h < kHalves; ++h) vok[h] = 8 * h + v < s;
  int ks = k0;
  constexpr int U = kUnroll / kHalves;
  for (; ks + (U - 1) * dk < nk; ks += U * dk) {
    double2 qv[U], cv[U][kHalves];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int col = 4 * (ks + u * dk) + lk;
      const bool ok = col < ncol;
      qv[u] = *(ok ? qcol(S, Vr, m, ldq, col) + row : zero);
#pragma unroll
      for (int h = 0; h < kHalves; ++h)
        cv[u][h] = *((ok & vok[h]) ? C + (size_t)col * kBlockMax + 8 * h + v : zero);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int h = 0; h < kHalves; ++h)
        if (h < nh) {
          const double b1 = imag ? cv[u][h].y : cv[u][h].x;
          const double b2 = imag ? cv[u][h].x : -cv[u][h].y;
          d[h] = mfma(qv[u].x, b1, d[h]);
          d[h] = mfma(qv[u].y, b2, d[h]);
        }
  }
  for (; ks < nk; ks += dk) {
    const int col = 4 * ks + lk;
    const bool ok = col < ncol;
    const double2 qv = *(ok ? qcol(S, Vr, m, ldq, col) + row : zero);
#pragma unroll
    for (int h = 0; h < kHalves; ++h)
      if (h < nh) {
        const double2 cv = *((ok & vok[h]) ? C + (size_t)col * kBlockMax + 8 * h + v : zero);
        const double b1 = imag ? cv.y : cv.x;
        const double b2 = imag ? cv.x : -cv.y;
        d[h] = mfma(qv.x, b1, d[h]);
        d[h] = mfma(qv.y, b2, d[h]);
      }
  }
}

// Q C for s > 8 with three real products per fragment (the Gauss form):
// lane (li, lk) holds row li of column 4 ks + lk (A fragment) and that
// column's coefficient for block vector li (B fragment);
//   T1 = Re(Q) Re(C),  T2 = Im(Q) Im(C),  T3 = (Re Q + Im Q)(Re C + Im C),
//   Re(Q C) = T1 - T2,  Im(Q C) = T3 - T1 - T2
// for the 16 rows (rows lk + 4 t in item t) and vector li.  RB blocks of 16
// rows (rows[b]: this lane's row of block b) share each coefficient load.
template <int RB, int U>
__device__ inline void qc_steps3(const double2* __restrict__ S, const double2* __restrict__ Vr, int m, size_t ldq,
                                 const int (&rows)[RB], int ncol, const double2* __restrict__ C, int s, int li,
                                 int lk, int k0, int dk, int nk, v4d (&t1)[RB], v4d (&t2)[RB], v4d (&t3)[RB]) {
  const gptr zero = to_global(&sgn_block_zero_entry);
  const bool vok = li < s;
  int ks = k0;
  for (; ks + (U - 1) * dk < nk; ks += U * dk) {
    double2 qv[U][RB], cv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int col = 4 * (ks + u * dk) + lk;
      const bool ok = col < ncol;
      const double2* qc = qcol(S, Vr, m, ldq, col);
#pragma unroll
      for (int b = 0; b < RB; ++b) qv[u][b] = gload(ok ? to_global(qc + rows[b]) : zero);
      cv[u] = gload((ok & vok) ? to_global(C + (size_t)col * kBlockMax + li) : zero);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const double cs = cv[u].x + cv[u].y;
#pragma unroll
      for (int b = 0; b < RB; ++b) {
        t1[b] = mfma(qv[u][b].x, cv[u].x, t1[b]);
        t2[b] = mfma(qv[u][b].y, cv[u].y, t2[b]);
        t3[b] = mfma(qv[u][b].x + qv[u][b].y, cs, t3[b]);
      }
    }
  }
  for (; ks < nk; ks += dk) {
    const int col = 4 * ks + lk;
    const bool ok = col < ncol;
    const double2* qc = qcol(S, Vr, m, ldq, col);
    const double2 cv = gload((ok & vok) ? to_global(C + (size_t)col * kBlockMax + li) : zero);
#pragma unroll
    for (int b = 0; b < RB; ++b) {
      const double2 qv = gload(ok ? to_global(qc + rows[b]) : zero);
      t1[b] = mfma(qv.x, cv.x, t1[b]);
      t2[b] = mfma(qv.y, cv.y, t2[b]);
      t3[b] = mfma(qv.x + qv.y, cv.x + cv.y, t3[b]);
    }
  }
}

// complex entries (Re in lane li < 8, Im from lane li + 8) of a Q C tile
__device__ inline void qc_pairs(const v4d& d, double2 (&res)[4]) {
#pragma unroll
  for (int t = 0; t < 4; ++t) res[t] = make_double2(d[t], __shfl_xor(d[t], 8, 64));
}

// The block's Hessenberg columns p-1 .. p+s-2, one thread per (row r, column
// j): M[i] = (Rc Th)[r][i] - P[r][i-1] for i <= j (P = H_{p x (p-1)} Ct, zero
// for rows r >= p), H[r][p-1+j] = sum_{i <= j} M[i] Rbi[i][j]; zero below the
// subdiagonal.  Rc(r, 0) = [r == p-1]; Rc(r, i) = Ct[r][i-1] (r < p) or
// R[r-p][i-1] (r >= p, upper triangular).  Per slot: Ct, P at cstride (P
// laid out [v][r] with ld ldp), R and Rbi at rstride, H at hstride.
struct BHess {
  double e;
  const double2* Ct;
  const double2* P;
  size_t cstride;
  int ldp;
  const double2* R;
  const double2* Rbi;
  size_t rstride;
  double2* H;
  size_t hstride;
  int ldh;
};

__device__ void hess_entry(const BlockGeo& g, const BHess& h, int r_slot, int idx) {
  const int r = idx / kBlockMax, j = idx % kBlockMax;
  const int p = g.p;
  if (r >= p + g.s || j >= g.s) return;
  const double2* Ct = h.Ct + (size_t)r_slot * h.cstride;
  const double2* P = h.P + (size_t)r_slot * h.cstride;
  const double2* R = h.R + (size_t)r_slot * h.rstride;
  const double2* Rbi = h.Rbi + (size_t)r_slot * h.rstride;
  auto rc = [&](int i) -> double2 {
    if (i == 0) return make_double2(r == p - 1 ? 1.0 : 0.0, 0.0);
    if (r < p) return Ct[(size_t)r * kBlockMax + i - 1];
    const int rr = r - p;
    return rr <= i - 1 ? R[rr * kBlockMax + i - 1] : make_double2(0.0, 0.0);
  };
  double2 acc = make_double2(0.0, 0.0);
  for (int i = 0; i <= j; ++i) {
    double2 mi;
    if (i == 0) {
      mi = cscale(rc(1), h.e);
    } else {
      mi = cscale(cadd(rc(i - 1), rc(i + 1)), 0.5 * h.e);
      if (r < p) mi = csub(mi, P[(size_t)(i - 1) * h.ldp + r]);
    }
    acc = cfma(mi, Rbi[i * kBlockMax + j], acc);
  }
  // column p-1+j has its subdiagonal in row p+j; below it H is zero
  h.H[(size_t)r_slot * h.hstride + (size_t)(p - 1 + j) * h.ldh + r] = (r <= p + j) ? acc : make_double2(0.0, 0.0);
}

// ---------------------------------------------------------------------------
// update pass: Wout = (Win - Q C) [Rinv].  With Rinv (the second pass) the
// first workgroups (padded to whole rounds of the XCDs) write the block's
// Hessenberg columns (hess).  The others take the rows by chunks: with s > 8 the
// dot pass's row chunks, a chunk on the XCD that read it there (on small
// lattices the columns are then still in that XCD's L2).
struct BUpd {
  const double2* C;
  size_t cstride;
  const double2* Win;
  size_t winstride;
  double2* Wout;
  size_t woutstride;
  const double2* Rinv;  // per slot [kBlockMax][kBlockMax] upper triangular at rstride, or null
  size_t rstride;
  int nch, crows;  // row chunks and rows of one (a multiple of 64)
  int nhess;       // workgroups on the Hessenberg columns (with Rinv), a multiple of 8
  BHess hess;
};

// workgroup -> slot position z and first row; false: no rows (padding, or a
// Hessenberg workgroup, done here)
__device__ inline bool upd_rows(const BlockGeo& g, const BUpd& a, int rows, int& z, int& r0) {
  int i = blockIdx.x;
  if (i < a.nhess) {
    const int t = i / g.nb;
    hess_entry(g, a.hess, g.act[i - t * g.nb], t * 256 + threadIdx.x);
    return false;
  }
  const int subs = a.crows / rows;
  int chunk, sub;
  if (!xcd_tile<true>(i - a.nhess, g.nb, subs, a.nch, chunk, z, sub)) return false;
  r0 = chunk * a.crows + sub * rows;
  return r0 < g.N;
}

// s <= 8, the packed form.  Wavefront: 16 rows x all p columns.
__global__ void __launch_bounds__(256) bupdate_kernel(BlockGeo g, BUpd a) {
  int z, wg0;
  if (!upd_rows(g, a, 64, z, wg0)) return;
  const int rs = g.act[z];
  const double2* Vr = g.V + (size_t)rs * g.vstride;
  const double2* Cr = a.C + (size_t)rs * a.cstride;
  const double2* Win = a.Win + (size_t)rs * a.winstride;
  double2* Wout = a.Wout + (size_t)rs * a.woutstride;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const int r0 = wg0 + wave * 16;
  const bool active = r0 < g.N;  // wavefront-uniform
  const int v = li & 7;
  const int row = min(r0 + li, g.N - 1);
  v4d d[kHalves];
#pragma unroll
  for (int h = 0; h < kHalves; ++h) d[h] = v4d{0.0, 0.0, 0.0, 0.0};
  if (active) qc_steps(g.S, Vr, g.m, g.ldq, row, g.p, Cr, v, li >= 8, g.s, lk, 0, 1, d);
  // res[h][t]: (Q C)[row r0 + lk + 4 t][vector vec(h)] in the lanes that own one
  double2 res[kHalves][4];
  bool own[kHalves];
  int vec[kHalves];
#pragma unroll
  for (int h = 0; h < kHalves; ++h) {
    qc_pairs(d[h], res[h]);
    vec[h] = 8 * h + v;
    own[h] = li < 8 && vec[h] < g.s;
  }
  if (!a.Rinv) {
    if (active)
#pragma unroll
      for (int h = 0; h < kHalves; ++h) {
        if (!own[h]) continue;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int rr = r0 + lk + 4 * t;
          if (rr < g.N) {
            const size_t o = (size_t)vec[h] * g.ldq + rr;
            Wout[o] = csub(Win[o], res[h][t]);
          }
        }
      }
    return;
  }
  // second pass: W'' = Win - Q C, then W'' Rinv per row (through LDS; the
  // workgroup's slot is the same for all four wavefronts)
  __shared__ double2 tile[4][16][kBlockMax];
  __shared__ double2 ri[kBlockMax * kBlockMax];
  {
    const double2* Ri = a.Rinv + (size_t)rs * a.rstride;
    for (int e = threadIdx.x; e < kBlockMax * kBlockMax; e += 256) ri[e] = Ri[e];
  }
  // every (row, vector) of the tile: vectors past s and rows past N as zero
#pragma unroll
  for (int h = 0; h < kHalves; ++h) {
    if (li >= 8) continue;
    const int vv = 8 * h + v;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int rl = lk + 4 * t, rr = r0 + rl;
      double2 val = make_double2(0.0, 0.0);
      if (active && own[h] && rr < g.N) val = csub(Win[(size_t)vv * g.ldq + rr], res[h][t]);
      tile[wave][rl][vv] = val;
    }
  }
  __syncthreads();
  if (!active) return;
  constexpr int kOut = 16 * kBlockMax / 64;  // outputs per lane
  // (not unrolled: this epilogue would otherwise set the kernel's register
  // count, and with it the occupancy of the sweep above)
#pragma unroll 1
  for (int q = 0; q < kOut; ++q) {
    const int idx = lane + 64 * q;
    const int rl = idx / kBlockMax, vv = idx % kBlockMax;
    double2 acc = make_double2(0.0, 0.0);
#pragma unroll 4
    for (int u = 0; u < kBlockMax; ++u) acc = cfma(tile[wave][rl][u], ri[u * kBlockMax + vv], acc);
    const int rr = r0 + rl;
    if (vv < g.s && rr < g.N) Wout[(size_t)vv * g.ldq + rr] = acc;
  }
}

// s > 8, the three-multiplication form.  A row's sums run over the k-steps of
// four quarters of the columns, one chain of products each, which are then
// added in order; the two kernels below differ in who runs the chains.
__device__ inline int quarter(int p) { return (((p + 3) >> 2) + 3) >> 2; }  // k-steps of a quarter

// Small launches: a workgroup takes 16 rows and each of its wavefronts a
// quarter, whose sums meet in LDS.  The chain of waits is a quarter of the
// other form's and the launch has four times the wavefronts: 4x4x4x6, 268
// columns, 1 slot: 13 us (events), 28 us with whole rows per wavefront; 6^4,
// 176 columns: 16 against 24 us.
__global__ void __launch_bounds__(256) bupdate3_split_kernel(BlockGeo g, BUpd a) {
  int z, r0;
  if (!upd_rows(g, a, 16, z, r0)) return;
  const int rs = g.act[z];
  const double2* Vr = g.V + (size_t)rs * g.vstride;
  const double2* Cr = a.C + (size_t)rs * a.cstride;
  const double2* Win = a.Win + (size_t)rs * a.winstride;
  double2* Wout = a.Wout + (size_t)rs * a.woutstride;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lk = lane >> 4;
  // this thread's output: row r0 + rl of vector v
  const int rl = threadIdx.x & 15, v = threadIdx.x >> 4;
  const bool own = v < g.s && r0 + rl < g.N;
  const size_t o = (size_t)min(v, g.s - 1) * g.ldq + min(r0 + rl, g.N - 1);
  double2 w = Win[o];
  v4d t1[1] = {v4d{0.0, 0.0, 0.0, 0.0}}, t2[1] = {t1[0]}, t3[1] = {t1[0]};
  const int rows[1] = {min(r0 + li, g.N - 1)};
  const int qk = quarter(g.p), nk = (g.p + 3) >> 2;
  qc_steps3<1, 4>(g.S, Vr, g.m, g.ldq, rows, g.p, Cr, g.s, li, lk, wave * qk, 1, min((wave + 1) * qk, nk), t1, t2,
                  t3);
  // rows padded to 17 entries, so that a column of them spreads over the banks
  __shared__ double2 part[4][16][kBlockMax + 1];
  __shared__ double2 ri[kBlockMax * kBlockMax];
#pragma unroll
  for (int t = 0; t < 4; ++t)
    part[wave][lk + 4 * t][li] = make_double2(t1[0][t] - t2[0][t], t3[0][t] - t1[0][t] - t2[0][t]);
  if (a.Rinv) ri[threadIdx.x] = a.Rinv[(size_t)rs * a.rstride + threadIdx.x];
  static_assert(kBlockMax * kBlockMax == 256, "one output and one entry of Rinv per thread");
  __syncthreads();
  double2 sum = part[0][rl][v];
#pragma unroll
  for (int q = 1; q < 4; ++q) sum = cadd(sum, part[q][rl][v]);
  w = csub(w, sum);
  if (!a.Rinv) {
    if (own) Wout[o] = w;
    return;
  }
  // second pass: W'' Rinv per row, W'' in place of the first quarter's sums
  // (each thread replaces the entry that it alone has read)
  part[0][rl][v] = w;
  __syncthreads();
  if (!own) return;
  double2 acc = make_double2(0.0, 0.0);
  for (int u = 0; u <= v; ++u) acc = cfma(part[0][rl][u], ri[u * kBlockMax + v], acc);
  Wout[o] = acc;
}

// Large launches: a wavefront owns RB blocks of 16 rows and runs the four
// chains itself, RB blocks sharing each coefficient load, and keeps the sum of
// the finished quarters in LDS.  Bound by memory: 6^4 x 8 slots, 340 columns,
// 650 MB: 139 us (events), 4.7 TB/s.
template <int RB>
__global__ void __launch_bounds__(256) bupdate3_kernel(BlockGeo g, BUpd a) {
  constexpr int kRows = 16 * RB;
  int z, wg0;
  if (!upd_rows(g, a, 4 * kRows, z, wg0)) return;
  const int rs = g.act[z];
  const double2* Vr = g.V + (size_t)rs * g.vstride;
  const double2* Cr = a.C + (size_t)rs * a.cstride;
  const double2* Win = a.Win + (size_t)rs * a.winstride;
  double2* Wout = a.Wout + (size_t)rs * a.woutstride;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const int r0 = wg0 + wave * kRows;
  const bool active = r0 < g.N;  // wavefront-uniform
  __shared__ double2 tile[4][kRows][kBlockMax];
  __shared__ double2 ri[kBlockMax * kBlockMax];
  if (a.Rinv) ri[threadIdx.x] = a.Rinv[(size_t)rs * a.rstride + threadIdx.x];
  static_assert(kBlockMax * kBlockMax == 256, "one entry of Rinv per thread");
  int rows[RB];
#pragma unroll
  for (int b = 0; b < RB; ++b) rows[b] = min(r0 + 16 * b + li, g.N - 1);
  const int qk = quarter(g.p), nk = (g.p + 3) >> 2;
  if (active)
    for (int q = 0; q < 4; ++q) {
      v4d t1[RB], t2[RB], t3[RB];
#pragma unroll
      for (int b = 0; b < RB; ++b) {
        t1[b] = v4d{0.0, 0.0, 0.0, 0.0};
        t2[b] = t1[b];
        t3[b] = t1[b];
      }
      qc_steps3<RB, kUnroll / (2 * RB)>(g.S, Vr, g.m, g.ldq, rows, g.p, Cr, g.s, li, lk, q * qk, 1,
                                        min((q + 1) * qk, nk), t1, t2, t3);
      // each lane owns its entries of the tile
#pragma unroll
      for (int b = 0; b < RB; ++b)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const double2 x = make_double2(t1[b][t] - t2[b][t], t3[b][t] - t1[b][t] - t2[b][t]);
          double2& e = tile[wave][16 * b + lk + 4 * t][li];
          e = q ? cadd(e, x) : x;
        }
    }
  const bool own = li < g.s;
#pragma unroll
  for (int b = 0; b < RB; ++b)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int rl = 16 * b + lk + 4 * t, rr = r0 + rl;
      const size_t o = (size_t)li * g.ldq + rr;
      double2 val = make_double2(0.0, 0.0);
      if (active && own && rr < g.N) {
        val = csub(Win[o], tile[wave][rl][li]);
        if (!a.Rinv) Wout[o] = val;
      }
      if (a.Rinv) tile[wave][rl][li] = val;  // every entry: vectors past s and rows past N as zero
    }
  if (!a.Rinv) return;
  // second pass: W'' Rinv per row
  __syncthreads();
  if (!active) return;
  constexpr int kOut = kRows * kBlockMax / 64;  // outputs per lane
  // (not unrolled: this epilogue would otherwise set the kernel's register
  // count, and with it the occupancy of the sweep above)
#pragma unroll 1
  for (int q = 0; q < kOut; ++q) {
    const int idx = lane + 64 * q;
    const int rl = idx / kBlockMax, vv = idx % kBlockMax;
    double2 acc = make_double2(0.0, 0.0);
#pragma unroll 4
    for (int u = 0; u < kBlockMax; ++u) acc = cfma(tile[wave][rl][u], ri[u * kBlockMax + vv], acc);
    const int rr = r0 + rl;
    if (vv < g.s && rr < g.N) Wout[(size_t)vv * g.ldq + rr] = acc;
  }
}

// ---------------------------------------------------------------------------
// Between the two passes' reductions and the second update: per slot, one
// workgroup factors the block, G'' = G - C2^dag C2 = R^dag R (R upper), and
// forms R^-1 and Rb^-1 (Rb = [1, Ct[p-1][0 .. s-2]; 0, R[0 .. s-2][0 .. s-2]]);
// it raises the slot's flag when the block is not numerically of full rank
// (a pivot below 1e-12 of the block's size, or below 1e-7 of the largest
// pivot) or not finite.  C2^dag C2 and the diagonal of Ct^dag Ct (the block
// vectors' size before projection) run on the matrix cores, the four
// wavefronts taking every fourth k-step.  The other workgroups form
// P = H_{p x (p-1)} Ct for 16 rows each (the four wavefronts take every
// fourth k-step, summed in order), from the first column where a row of the
// tile can be nonzero (H is upper Hessenberg below the T block, T upper
// triangular).  Workgroup id = z + nb t: t = 0 factors, t >= 1 is row tile
// t - 1.
struct BSmall {
  const double2* C2;
  const double2* Ct;
  size_t cstride;
  const double2* G;
  size_t gstride;
  const double2* H;
  size_t hstride;
  int ldh;
  double2* P;  // [v][r], ld ldp
  int ldp;
  double2* R;  // per slot: R, R^-1, Rb^-1 (kBlockMax^2 each) at rstride
  size_t rstride;
  int* flag;
};

__device__ void block_factor(const BlockGeo& gg, const BSmall& a, int rs) {
  constexpr int B = kBlockMax;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int s = gg.s, p = gg.p;
  const double2* C2 = a.C2 + (size_t)rs * a.cstride;
  const double2* Ct = a.Ct + (size_t)rs * a.cstride;
  const double2* G = a.G + (size_t)rs * a.gstride;
  double2* Rout = a.R + (size_t)rs * a.rstride;
  __shared__ v4d red[4][2][64];
  __shared__ double redn[4][64];
  static_assert(B * B == 256, "one entry per thread");
  __shared__ double2 g[B][B], Ri[B][B], X[B][B], cl[B];
  __shared__ double ref_s;
  // C2^dag C2 (16 x 16 complex) on the matrix cores: A = C2^dag (row u, k = c),
  // B = C2 (k = c, column v); lane (li, lk) loads C2[c][li] for c = 4 ks + lk.
  // Re += Re A Re B + Im A Im B... with A = conj(C2)^T:
  //   Re(conj(a) b) = ar br + ai bi,  Im(conj(a) b) = ar bi - ai br
  {
    const int li = lane & 15, lk = lane >> 4;
    v4d dre = {0.0, 0.0, 0.0, 0.0}, dim = {0.0, 0.0, 0.0, 0.0};
    double nn = 0.0;
    const double2* zero = &sgn_block_zero_entry;
    const int nk = (p + 3) >> 2;
    // the loads of kUnroll k-steps first (one wait per group, not per step)
    int ks = wave;
    for (; ks + 4 * (kUnroll - 1) < nk; ks += 4 * kUnroll) {
      double2 x[kUnroll], y[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const int c = 4 * (ks + 4 * u) + lk;
        const bool ok = c < p && li < s;
        x[u] = *(ok ? C2 + (size_t)c * B + li : zero);
        y[u] = *(ok ? Ct + (size_t)c * B + li : zero);
      }
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        dre = mfma(x[u].x, x[u].x, dre);
        dre = mfma(x[u].y, x[u].y, dre);
        dim = mfma(x[u].x, x[u].y, dim);
        dim = mfma(-x[u].y, x[u].x, dim);
        nn += cabs2(y[u]);
      }
    }
    for (; ks < nk; ks += 4) {
      const int c = 4 * ks + lk;
      const bool ok = c < p && li < s;
      const double2 x = *(ok ? C2 + (size_t)c * B + li : zero);
      const double2 y = *(ok ? Ct + (size_t)c * B + li : zero);
      dre = mfma(x.x, x.x, dre);
      dre = mfma(x.y, x.y, dre);
      dim = mfma(x.x, x.y, dim);
      dim = mfma(-x.y, x.x, dim);
      nn += cabs2(y);
    }
    red[wave][0][lane] = dre;
    red[wave][1][lane] = dim;
    redn[wave][lane] = nn;
  }
  const int u0 = tid / B, v0 = tid % B;  // this thread's entry of the 16 x 16 matrices
  __syncthreads();
  double2 gv = make_double2(0.0, 0.0);  // G - C2^dag C2, then the trailing block
  if (u0 < s && v0 < s) {
    // D[u][v] sits in lane v + 16 (u % 4), item u / 4
    const int l = v0 + 16 * (u0 & 3), it = u0 >> 2;
    double sre = red[0][0][l][it], sim = red[0][1][l][it];
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      sre += red[w][0][l][it];
      sim += red[w][1][l][it];
    }
    gv = csub(G[tid], make_double2(sre, sim));
  }
  if (tid < 64) {
    // the block vectors' size before projection, G[v][v] + |Ct[:, v]|^2
    // (redn: over the lanes holding v, li = v, and the wavefronts), its largest
    double rf = 0.0;
    if (tid < s) {
      rf = 0.0;
      for (int w = 0; w < 4; ++w)
        for (int q = 0; q < 4; ++q) rf += redn[w][tid + 16 * q];
      rf += G[tid * B + tid].x;
    }
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) {
      const double o = __shfl_xor(rf, off, 64);
      rf = (o > rf || !(o == o)) ? o : rf;  // a NaN stays
    }
    if (tid == 0) ref_s = rf;
  }
  // Right-looking Cholesky of G = R^dag R with the identity beside it: step j
  // forms row j of R and of E = R^-dag and updates the rows below, each thread
  // its entry of both (one barrier per step: row j of both goes through LDS
  // and step j leaves it alone).
  double2 ev = make_double2(u0 == v0 ? 1.0 : 0.0, 0.0), rv = make_double2(0.0, 0.0);
  double dmin = HUGE_VAL, dmax = 0.0;
  bool bad = false;
  g[u0][v0] = gv;
  Ri[u0][v0] = ev;  // E while it forms
  __syncthreads();
  for (int j = 0; j < s; ++j) {
    double dj = g[j][j].x;
    const bool okp = dj > 0.0 && isfinite(dj);
    if (!okp) dj = 1.0;
    const double ip = rsqrt(dj), pj = dj * ip;
    bad = bad || !okp;
    dmin = fmin(dmin, pj);
    dmax = fmax(dmax, pj);
    if (u0 == j) {
      // row j of R and of E, each thread its entry
      if (v0 >= j && v0 < s) rv = v0 == j ? make_double2(pj, 0.0) : cscale(g[j][v0], ip);
      ev = cscale(Ri[j][v0], ip);
    } else if (u0 > j && u0 < s) {
      const double2 f = cscale(g[j][u0], ip);  // R[j][u0]
      if (v0 > j && v0 < s) {
        gv = csub(gv, cmulc(f, cscale(g[j][v0], ip)));
        g[u0][v0] = gv;
      }
      if (v0 <= j) {
        ev = csub(ev, cmulc(f, cscale(Ri[j][v0], ip)));
        Ri[u0][v0] = ev;
      }
    }
    __syncthreads();
  }
  // R^-1 = E^dag (upper); Rb^-1 = [1, -c R'^-1; 0, R'^-1] with R' the leading
  // (s - 1) x (s - 1) block of R and c the last basis column's coefficients
  const bool in = u0 < s && v0 < s;
  X[v0][u0] = (in && v0 <= u0) ? make_double2(ev.x, -ev.y) : make_double2(0.0, 0.0);
  if (tid < B) cl[tid] = tid + 1 < s ? Ct[(size_t)(p - 1) * B + tid] : make_double2(0.0, 0.0);
  __syncthreads();
  double2 rb = make_double2(0.0, 0.0);
  if (in) {
    if (u0 > 0) {
      if (v0 >= u0) rb = X[u0 - 1][v0 - 1];
    } else if (v0 == 0) {
      rb = make_double2(1.0, 0.0);
    } else {
      for (int l = 0; l < v0; ++l) rb = csub(rb, cmul(cl[l], X[l][v0 - 1]));
    }
  }
  Rout[tid] = in ? rv : make_double2(0.0, 0.0);
  Rout[B * B + tid] = X[u0][v0];
  Rout[2 * B * B + tid] = rb;
  if (tid == 0) {
    const double rf = ref_s;
    if (bad || !(rf > 0.0) || !isfinite(rf) || dmin * dmin < 1e-24 * rf || dmin < 1e-7 * dmax) a.flag[rs] = 1;
  }
}

template <bool G>
__global__ void __launch_bounds__(256) bsmall_kernel(BlockGeo g, BSmall a) {
  const int z = blockIdx.x % g.nb, t = blockIdx.x / g.nb;
  const int rs = g.act[z];
  if (t == 0) {
    block_factor(g, a, rs);
    return;
  }
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const int p = g.p;
  const int r0 = (t - 1) * 16;
  const int row = min(r0 + li, p - 1);
  const int v = li & 7;
  const int c0 = r0 < g.m ? r0 : max(g.m, r0 - 1);  // columns below c0 are zero in these rows
  const double2* H = a.H + (size_t)rs * a.hstride;
  const double2* Ct = a.Ct + (size_t)rs * a.cstride;
  double2* P = a.P + (size_t)rs * a.cstride;
  // only the columns 0 .. s-2 of Ct enter P
  if constexpr (G) {
    v4d t1[1] = {v4d{0.0, 0.0, 0.0, 0.0}}, t2[1] = {t1[0]}, t3[1] = {t1[0]};
    const int rows[1] = {row};
    qc_steps3<1, kUnroll / 2>(H, H, 0, (size_t)a.ldh, rows, p - 1, Ct, g.s - 1, li, lk, (c0 >> 2) + wave, 4, (p + 2) >> 2, t1, t2, t3);
    __shared__ v4d red3[4][3][64];
    red3[wave][0][lane] = t1[0];
    red3[wave][1][lane] = t2[0];
    red3[wave][2][lane] = t3[0];
    __syncthreads();
    if (wave != 0) return;
    v4d u1 = t1[0], u2 = t2[0], u3 = t3[0];
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      u1 += red3[w][0][lane];
      u2 += red3[w][1][lane];
      u3 += red3[w][2][lane];
    }
    if (li < g.s - 1)
#pragma unroll
      for (int tt = 0; tt < 4; ++tt) {
        const int rr = r0 + lk + 4 * tt;
        if (rr < p) P[(size_t)li * a.ldp + rr] = make_double2(u1[tt] - u2[tt], u3[tt] - u1[tt] - u2[tt]);
      }
  } else {
    v4d d[kHalves];
#pragma unroll
    for (int h = 0; h < kHalves; ++h) d[h] = v4d{0.0, 0.0, 0.0, 0.0};
    qc_steps(H, H, 0, (size_t)a.ldh, row, p - 1, Ct, v, li >= 8, g.s - 1, lk, (c0 >> 2) + wave, 4, d);
    __shared__ v4d red[4][kHalves][64];
#pragma unroll
    for (int h = 0; h < kHalves; ++h) red[wave][h][lane] = d[h];
    __syncthreads();
    if (wave != 0) return;
#pragma unroll
    for (int h = 0; h < kHalves; ++h) {
      v4d dh = red[0][h][lane];
#pragma unroll
      for (int w = 1; w < 4; ++w) dh += red[w][h][lane];
      double2 res[4];
      qc_pairs(dh, res);
      if (li < 8 && 8 * h + v < g.s - 1)
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
          const int rr = r0 + lk + 4 * tt;
          if (rr < p) P[(size_t)(8 * h + v) * a.ldp + rr] = res[tt];
        }
    }
  }
}

BlockGeo make_geo(const BlockSpan& sp) {
  BlockGeo g;
  g.S = sp.S;
  g.V = sp.V;
  g.vstride = sp.vstride;
  g.ldq = sp.ldq;
  g.m = sp.m;
  g.p = 0;
  g.s = 0;
  g.N = sp.N;
  g.nb = sp.nb;
  for (int z = 0; z < sp.nb; ++z) g.act[z] = sp.act[z];
  return g;
}

}  // namespace

void block_alloc(BlockWork& b, int N, size_t ldq, int ncap, int nslots) {
  block_free(b);
  int rpw = 0;
  const int nch = row_chunks(N, rpw);
  const size_t S = (size_t)nslots;
  b.nslots = nslots;
  b.wstride = ldq * kBlockMax;
  b.pstride = (size_t)nch * (ncap + kBlockMax) * kBlockMax;
  b.cstride = (size_t)ncap * kBlockMax;
  b.gstride = kBlockMax * kBlockMax;
  b.rstride = 3 * kBlockMax * kBlockMax;
  SGN_HIP(hipMalloc(&b.W, sizeof(double2) * b.wstride * S));
  SGN_HIP(hipMalloc(&b.part, sizeof(double2) * b.pstride * S));
  SGN_HIP(hipMalloc(&b.C1, sizeof(double2) * b.cstride * S));
  SGN_HIP(hipMalloc(&b.C2, sizeof(double2) * b.cstride * S));
  SGN_HIP(hipMalloc(&b.Ct, sizeof(double2) * b.cstride * S));
  SGN_HIP(hipMalloc(&b.P, sizeof(double2) * b.cstride * S));
  SGN_HIP(hipMalloc(&b.G, sizeof(double2) * b.gstride * S));
  SGN_HIP(hipMalloc(&b.R, sizeof(double2) * b.rstride * S));
  SGN_HIP(hipMalloc(&b.flag, sizeof(int) * S));
  b.ncap = ncap;
}

void block_free(BlockWork& b) {
  for (double2** p : {&b.W, &b.part, &b.C1, &b.C2, &b.Ct, &b.P, &b.G, &b.R})
    if (*p) {
      (void)hipFree(*p);
      *p = nullptr;
    }
  if (b.flag) (void)hipFree(b.flag);
  b.flag = nullptr;
  b.ncap = 0;
  b.nslots = 0;
}

void block_first(const BlockSpan& sp, const double2* u, size_t ustride, const double* inv, int istride,
                 hipStream_t s) {
  BlockGeo g = make_geo(sp);
  hipLaunchKernelGGL(bstart_kernel, dim3((sp.N + 255) / 256, sp.nb), dim3(256), 0, s, g, u, ustride, inv, istride);
  SGN_HIP(hipGetLastError());
}

void block_step(const BlockSpan& sp, BlockWork& b, const Lattice& lat, const double2* links, int k, int sb, double e,
                hipStream_t s, Profiler* prof) {
  const int m = sp.m, N = sp.N, p = m + 1 + k, nb = sp.nb;
  const size_t ldq = sp.ldq;
  SGN_REQUIRE(sb >= 1 && sb <= kBlockMax && p + sb <= sp.ncap && b.ncap >= sp.ncap && nb >= 1 && nb <= kMaxBatch &&
                  nb <= b.nslots,
              SGN_EINVAL, "block step exceeds the workspace");
  BlockGeo g = make_geo(sp);
  g.p = p;
  g.s = sb;
  // the newest basis column q_{p-1} = V_r[p-1-m]
  const double2* w0 = sp.V + (size_t)(p - 1 - m) * ldq;
  // Krylov directions: W_1 = A W_0 / e, W_{i+1} = 2 A W_i / e - W_{i-1}
  SlotMap map;
  map.n = nb;
  for (int z = 0; z < nb; ++z) map.slot[z] = sp.act[z];
  struct Dir {
    double2* p;
    size_t stride;
  };
  auto dir = [&](int i) {  // W_i
    return i == 0 ? Dir{const_cast<double2*>(w0), sp.vstride} : Dir{b.W + (size_t)(i - 1) * ldq, b.wstride};
  };
  const bool pairs = wilson_pairs(lat, nb);
  for (int i = 1; i <= sb; ++i) {
    const Dir in = dir(i - 1), out = dir(i), pv = i > 1 ? dir(i - 2) : Dir{nullptr, 0};
    const double ca = (i == 1 ? 1.0 : 2.0) / e, cb = i == 1 ? 0.0 : -1.0;
    if (pairs && i < sb) {
      const Dir next = dir(++i);
      wilson_apply_cheb_pair(lat, links, in.p, in.stride, out.p, out.stride, next.p, next.stride, pv.p, pv.stride, ca,
                             cb, 2.0 / e, -1.0, map, s, prof);
    } else {
      wilson_apply_cheb_slots(lat, links, in.p, in.stride, out.p, out.stride, pv.p, pv.stride, ca, cb, map, s, prof);
    }
  }
  int rpw = 0;
  const int nch = row_chunks(N, rpw);
  // more than 8 block vectors: the products in their three-multiplication form
  const bool gauss = sb > 8;
  // launches of several slots: four column tiles per dot wavefront and two
  // blocks of 16 rows per update wavefront (three-multiplication form); the
  // arithmetic of every entry is the same either way
  const bool wide = gauss && nb >= kWideFrom;
  auto tiles_for = [&](int ncol) {
    if (!gauss) return kDotTiles;
    if (wide) return kDot3Tiles;
    return nb * nch * ((ncol + 31) / 32) >= kFullChip ? 2 : 1;
  };
  // rows per workgroup of the update pass: whole rows per wavefront, or in
  // small launches the columns split over the wavefronts
  const bool large = (double)N * nb * p >= kWholeEntries;
  const bool whole = !gauss || large || (double)N * nb >= kWholeRows;
  const int upd_rows_wg = !whole ? 16 : gauss && large ? 64 * kRowBlocks : 64;
  void (*upd_kernel)(BlockGeo, BUpd) = !gauss  ? bupdate_kernel
                                       : large ? bupdate3_kernel<kRowBlocks>
                                       : whole ? bupdate3_kernel<1>
                                               : bupdate3_split_kernel;
  auto dot = [&](double2* C, int ncol, const double2* C1, double2* Ct) {
    const int tiles = tiles_for(ncol);
    void (*dot_kernel)(BlockGeo, BDot) = !gauss       ? bdot_kernel
                                         : tiles == 4 ? bdot3_kernel<4>
                                         : tiles == 2 ? bdot3_kernel<2>
                                                      : bdot3_kernel<1>;
    static_assert(kDot3Tiles == 4, "the instances above");
    const int ncg = (ncol + 16 * tiles - 1) / (16 * tiles);
    BDot d{b.W, b.wstride, ncol, rpw, ncg, nch, b.part, b.pstride};
    // the basis read once (S once for the launch, the slots' own columns and
    // W as columns per slot), W once per slot, partials written
    const double bytes =
        16.0 * N * ((double)m + (double)nb * (ncol - m + sb)) + 16.0 * nch * ncol * kBlockMax * (double)nb;
    prof_launch(prof, K_BDOT, bytes, 8.0 * N * ncol * sb * nb, dot_kernel, dim3(xcd_grid(nb * ncg, nch)), dim3(256),
                0, s, g, d);
    const int nent = ncol * kBlockMax, nblk = (nent + 31) / 32;
    BRed rd{b.part, b.pstride, nch, nent, nblk, C, C1, Ct, b.cstride, b.G, b.gstride};
    prof_launch(prof, K_BRED, (16.0 * (double)nch * nent + 16.0 * nent) * nb, 2.0 * nch * nent * nb, bred_kernel,
                dim3(nblk * nb), dim3(256), 0, s, g, rd);
  };
  // rows that a launch keeps on one XCD: the dot pass's chunks (on lattices where
  // their columns may still be in the L2; else chunks of about that size, whole
  // workgroups of 128 rows), or (packed form) the workgroup's own 64 rows, whose
  // shares are even on small lattices too.  us
  // of a whole apply's updates, chunks / own rows (the former kernels): 4^4 x 16
  // slots, s = 2, 200 columns 5340 / 4580 (4520); 12^4 x 4, s = 4, 240 columns 56.6
  // / 55.5 ms (56.4)
  const int crows = gauss ? update_chunk(rpw) : upd_rows_wg, uch = (N + crows - 1) / crows;
  SGN_REQUIRE(crows % upd_rows_wg == 0, SGN_EINVAL, "block step: update rows do not tile the chunk");
  const unsigned ugrid = xcd_grid(nb * (crows / upd_rows_wg), uch);
  // the basis (S once for the launch), W read and written, the coefficients
  const double upd_bytes = 16.0 * N * ((double)m + (double)nb * (p - m + 2.0 * sb)) + 16.0 * p * sb * (double)nb;
  // pass 1
  dot(b.C1, p, nullptr, nullptr);
  {
    BUpd u{b.C1, b.cstride, b.W, b.wstride, b.W, b.wstride, nullptr, 0, uch, crows, 0, BHess{}};
    prof_launch(prof, K_BUPDATE, upd_bytes, 8.0 * N * p * sb * nb, upd_kernel, dim3(ugrid), dim3(256), 0, s, g, u);
  }
  // pass 2 with the Gram matrix of the projected block
  dot(b.C2, p + sb, b.C1, b.Ct);
  {
    BSmall sm{b.C2, b.Ct, b.cstride, b.G, b.gstride, sp.H, sp.hstride, sp.ldh, b.P, sp.ncap, b.R, b.rstride, b.flag};
    const double hb = 16.0 * ((double)p * p / 2 + 3.0 * p * sb) * nb;
    prof_launch(prof, K_BSMALL, hb, 8.0 * p * p * sb / 2 * nb, sb - 1 > 8 ? bsmall_kernel<true> : bsmall_kernel<false>,
                dim3((1 + (p + 15) / 16) * nb), dim3(256), 0, s, g, sm);
  }
  {
    BHess h{e, b.Ct, b.P, b.cstride, sp.ncap, b.R, b.R + 2 * kBlockMax * kBlockMax, b.rstride, sp.H, sp.hstride,
            sp.ldh};
    const int nh = (((p + sb) * kBlockMax + 255) / 256 * nb + 7) / 8 * 8;
    BUpd u{b.C2, b.cstride, b.W, b.wstride, const_cast<double2*>(sp.V) + (size_t)(p - m) * ldq, sp.vstride,
           b.R + kBlockMax * kBlockMax, b.rstride, uch, crows, nh, h};
    prof_launch(prof, K_BUPDATE, upd_bytes, 8.0 * N * p * sb * nb, upd_kernel, dim3(nh + ugrid), dim3(256), 0, s, g,
                u);
  }
}
