// One-reduction modified Arnoldi step with delayed re-orthogonalisation
// (Section 5.2, step (iv), Eq. eq:modArnoldi), for FP64 or FP32 Krylov-vector
// storage and for a batch of right-hand sides advancing in lock step.
//
// State before step j (J = m + j finished columns of Q = (S_m v_1 .. v_j)):
// u, the candidate for column J, orthogonalised once against Q_J but neither
// re-orthogonalised nor normalised.  With z = A u (the stencil, outside):
//   dot:    a = Q_J^dag u, b = Q_J^dag z, c = u^dag u, d = u^dag z   (1 sweep)
//           rho = sqrt(c - |a|^2),  gam = (d - a^dag b) / rho
//   update: v_J = (u - Q_J a) / rho                                    (1 sweep)
//           u'  = (z - (gam/rho) u - Q_J (b - (gam/rho) a)) / rho
//               = (1 - Q_{J+1} Q_{J+1}^dag) A v_J
//           column J-1 of H += a, H[J][J-1] = rho  (re-orthogonalisation)
//           column J of H = ([b; gam] - Hbar_J a) / rho
// Hbar_J is the (J+1) x J leading block of the composite H with the corrected
// column J-1, so that A Q_J = Q_{J+1} Hbar_J.  At j = 0 the correction goes to
// c0 = S^dag x and rho is beta = |x_perp|.  This is classical Gram-Schmidt
// with one full re-orthogonalisation, rescheduled so that each step needs a
// single global reduction and two sweeps over the basis.
//
// Precision: S, u, H, all dot products and all coefficients are FP64; the
// Krylov columns v_j and the stencil operand/result (z) are stored as VT
// (double2, or float2 in mixed precision).
//
// Batching: each workgroup serves one right-hand side; per-RHS buffers are
// laid out at fixed strides.  The dot and update passes number their
// workgroups with the right-hand side varying fastest, so the workgroups of
// all right-hand sides that read the same rows of the shared Schur block S run
// together and S comes from cache after the first of them.  Every reduction
// has a fixed order, so results are bitwise independent of the batch.
#include "internal.h"
#include "krylov.h"
#include "tilemap.h"

namespace {

constexpr int kRpl = 8;                 // dot: rows per lane
constexpr int kDRows = 64 * kRpl;       // dot: rows per tile (4 wavefronts of CPW columns each)
static_assert(kDRows == kTileRows, "the tile map's rows");
constexpr int kUWaves = 8;              // combine (and the default update): wavefronts per 64-row workgroup
constexpr int kUThreads = 64 * kUWaves;
constexpr int kCBatch = 8;              // combine: column loads issued together per lane

__device__ inline double2 ld2(const double2* p, size_t i) { return p[i]; }
__device__ inline double2 ld2(const float2* p, size_t i) {
  const float2 v = p[i];
  return make_double2((double)v.x, (double)v.y);
}
__device__ inline void st2(double2* p, size_t i, double2 v) { p[i] = v; }
__device__ inline void st2(float2* p, size_t i, double2 v) { p[i] = make_float2((float)v.x, (float)v.y); }

// Rows per lane group of the dot and update passes: 1 with FP64 Krylov
// columns, 2 with FP32 columns, whose lanes then take adjacent row pairs so
// that a column load is 16 bytes per lane
template <typename VT>
constexpr int rows_per_lane() { return sizeof(VT) == 8 ? 2 : 1; }

// v of lane l ^ 8, 4, 2 or 1, by data-parallel moves within 16 lanes
template <int CTRL>
__device__ inline double dpp_move(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
__device__ inline double lane_xor8(double v) { return dpp_move<0x128>(v); }                   // row_ror:8
__device__ inline double lane_xor4(double v) { return dpp_move<0x1B>(dpp_move<0x141>(v)); }  // half mirror, quad reversal
__device__ inline double lane_xor2(double v) { return dpp_move<0x4E>(v); }                    // quad_perm 2 3 0 1
__device__ inline double lane_xor1(double v) { return dpp_move<0xB1>(v); }                    // quad_perm 1 0 3 2

// a of lanes with the bit clear beside b of its partners, and the other way
// round: after the swap x + y is, in a lane with the bit clear, a + (a of
// lane ^ bit), and with the bit set the same of b
template <int BIT>
__device__ inline double swap_add(double a, double b) {
  static_assert(BIT == 32 || BIT == 16, "half-wavefront or row swaps");
  const unsigned al = (unsigned)__double2loint(a), ah = (unsigned)__double2hiint(a);
  const unsigned bl = (unsigned)__double2loint(b), bh = (unsigned)__double2hiint(b);
  if constexpr (BIT == 32) {
    const auto l = __builtin_amdgcn_permlane32_swap(al, bl, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(ah, bh, false, false);
    return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
  } else {
    const auto l = __builtin_amdgcn_permlane16_swap(al, bl, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(ah, bh, false, false);
    return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
  }
}
__device__ inline double pick_add8(double a, double b, bool set) {
  const double keep = set ? b : a, send = set ? a : b;
  return keep + lane_xor8(send);
}

// the sum over the 64 lanes, in every lane: an xor butterfly with offsets 32,
// 16, 8, 4, 2, 1 without LDS
__device__ inline double wsum1(double v) {
  v = swap_add<32>(v, v);
  v = swap_add<16>(v, v);
  v += lane_xor8(v);
  v += lane_xor4(v);
  v += lane_xor2(v);
  v += lane_xor1(v);
  return v;
}
__device__ inline double2 wsum2(double2 v) { return make_double2(wsum1(v.x), wsum1(v.y)); }

// Sums of NV values over the 64 lanes, each in the order of an xor butterfly
// with offsets 32, 16, 8, 4, 2, 1.  The first log2(NV) steps also halve the
// number of values a lane holds (a lane keeps the half its bit names), so the
// 8 values of two columns take 10 exchanges instead of 48.  On return a lane
// holds the sum of value (its top log2(NV) bits).
template <int NV>
__device__ inline double wave_sums(double (&v)[NV], int lane) {
  static_assert(NV == 4 || NV == 8, "one or two columns");
#pragma unroll
  for (int i = 0; i < NV / 2; ++i) v[i] = swap_add<32>(v[i], v[i + NV / 2]);
#pragma unroll
  for (int i = 0; i < NV / 4; ++i) v[i] = swap_add<16>(v[i], v[i + NV / 4]);
  if constexpr (NV >= 8) {
    v[0] = pick_add8(v[0], v[1], lane & 8);
  } else {
    v[0] += lane_xor8(v[0]);
  }
  v[0] += lane_xor4(v[0]);
  v[0] += lane_xor2(v[0]);
  v[0] += lane_xor1(v[0]);
  return v[0];
}

// wavefront index as a scalar (uniform) value
__device__ inline int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// launch position z (an index into the batch) -> buffer slot and step
__device__ inline int slot_of(const KrylovArgs& A, int z) { return A.act[z]; }
__device__ inline int step_of(const KrylovArgs& A, int z) { return A.jdev ? *A.jdev + A.joff : A.jv[z]; }

// ---------------------------------------------------------------------------
// dot pass: sums of Q^dag u and Q^dag z over row tiles, plus |u|^2, u^dag z,
// |z|^2 per tile.  Rows past N carry zero weights (uv = zv = 0 there) and load
// a valid row instead: unconditional loads, all in flight together.
// Row of a lane's slot t in a tile: R = 1, row0 + 64 t + lane; R = 2 (FP32
// columns), the pair row0 + 128 (t / 2) + 2 lane + {0, 1}
template <int R>
__device__ inline int dot_row(int row0, int t, int lane) {
  return R == 1 ? row0 + t * 64 + lane : row0 + (t >> 1) * 128 + 2 * lane + (t & 1);
}

// 16 bytes of a basis column: cached, or (NT) streamed past the caches
typedef float f4v __attribute__((ext_vector_type(4)));
typedef double d2v __attribute__((ext_vector_type(2)));
template <bool NT>
__device__ inline float4 col_load(const float4* p) {
  if constexpr (NT) {
    const f4v v = __builtin_nontemporal_load(reinterpret_cast<const f4v*>(p));
    return make_float4(v.x, v.y, v.z, v.w);
  }
  return *p;
}
template <bool NT>
__device__ inline double2 col_load(const double2* p) {
  if constexpr (NT) {
    const d2v v = __builtin_nontemporal_load(reinterpret_cast<const d2v*>(p));
    return make_double2(v.x, v.y);
  }
  return *p;
}

// a lane's kRpl rows of one column, as loaded: FP64 entries, or FP32 pairs
template <typename QT>
struct ColBuf {
  double2 q[kRpl];
  template <int R, bool NT>
  __device__ inline void load(const double2* __restrict__ p, int row0, int lane, int N) {
#pragma unroll
    for (int t = 0; t < kRpl; t += R) {
      const int i = min(dot_row<R>(row0, t, lane), N - R);
#pragma unroll
      for (int k = 0; k < R; ++k) q[t + k] = col_load<NT>(p + i + k);
    }
  }
  __device__ inline double2 at(int t) const { return q[t]; }
};
template <>
struct ColBuf<float2> {
  float4 q[kRpl / 2];
  template <int R, bool NT>
  __device__ inline void load(const float2* __restrict__ p, int row0, int lane, int N) {
    static_assert(R == 2, "FP32 columns come in row pairs");
    // N is even, so a pair lies wholly below N or wholly at or above it
#pragma unroll
    for (int t = 0; t < kRpl; t += 2)
      q[t / 2] = col_load<NT>(reinterpret_cast<const float4*>(p + min(dot_row<2>(row0, t, lane), N - 2)));
  }
  __device__ inline double2 at(int t) const {
    const float4 v = q[t / 2];
    return t & 1 ? make_double2((double)v.z, (double)v.w) : make_double2((double)v.x, (double)v.y);
  }
};

// the tile's weights u and z in a lane, and its raw sums |u|^2, u^dag z, |z|^2
template <typename VT, int R>
struct Weights {
  double2 u[kRpl], z[kRpl];
  __device__ inline void load(const KrylovArgs& A, int r, int row0, int lane, bool with_z) {
    const double2* __restrict__ up = A.u + (size_t)r * A.ustride;
    const VT* __restrict__ zp = static_cast<const VT*>(A.z) + (size_t)r * A.zstride;
    const bool whole = row0 + kDRows <= A.N;  // uniform; else rows past N carry zeros
#pragma unroll
    for (int t = 0; t < kRpl; ++t) {
      const int i = dot_row<R>(row0, t, lane);
      u[t] = up[min(i, A.N - 1)];
      z[t] = with_z ? ld2(zp, min(i, A.N - 1)) : make_double2(0.0, 0.0);
    }
    if (whole) return;
#pragma unroll
    for (int t = 0; t < kRpl; ++t)
      if (dot_row<R>(row0, t, lane) >= A.N) u[t] = z[t] = make_double2(0.0, 0.0);
  }
  __device__ inline void raw_sums(double* __restrict__ out, int lane) const {
    double cs = 0.0, zs = 0.0;
    double2 ds = make_double2(0.0, 0.0);
#pragma unroll
    for (int t = 0; t < kRpl; ++t) {
      cs += cabs2(u[t]);
      zs += cabs2(z[t]);
      ds = cfmac(u[t], z[t], ds);
    }
    double v[4] = {cs, ds.x, ds.y, zs};
    const double sum = wave_sums<4>(v, lane);
    if ((lane & 15) == 0) out[lane >> 4] = sum;
  }
  // the sums of C columns: value 4 cc + {0, 1, 2, 3} is Re a, Im a, Re b, Im b
  // of column cc; on return lane l holds value l / (16 / C)
  template <typename QT, int C>
  __device__ inline double dot(const ColBuf<QT> (&q)[C], int lane) const {
    double v[4 * C];
#pragma unroll
    for (int cc = 0; cc < C; ++cc) {
      double2 aa = make_double2(0.0, 0.0), bb = make_double2(0.0, 0.0);
#pragma unroll
      for (int t = 0; t < kRpl; ++t) {
        const double2 qv = q[cc].at(t);
        aa = cfmac(qv, u[t], aa);
        bb = cfmac(qv, z[t], bb);
      }
      v[4 * cc] = aa.x;
      v[4 * cc + 1] = aa.y;
      v[4 * cc + 2] = bb.x;
      v[4 * cc + 3] = bb.y;
    }
    return wave_sums<4 * C>(v, lane);
  }
};

// C columns from c0 on of the Schur (S) or Krylov part; columns past cend
// reload the last one (their sums are not used)
template <typename QT, int C, int R, bool NT = false>
__device__ inline void load_cols(ColBuf<QT> (&q)[C], const QT* __restrict__ base, size_t ldq, int c0, int cend,
                                 int row0, int lane, int N) {
#pragma unroll
  for (int cc = 0; cc < C; ++cc) q[cc].template load<R, NT>(base + (size_t)min(c0 + cc, cend - 1) * ldq, row0, lane, N);
}

// Columns [c0, c0 + C ng) of one base against the tile's weights, C at a time,
// the next C loaded before the sums of the current ones; put(c, k, sum) takes
// value k of column c (counted from the base)
template <typename QT, int C, int R, bool NT, typename W, typename Put>
__device__ inline void dot_walk(const W& w, const QT* __restrict__ base, size_t ldq, int c0, int ng, int cend,
                                int row0, int lane, int N, Put put) {
  auto out = [&](int cb, double sum) {
    constexpr int kLanes = 16 / C;  // lanes that hold the same value
    const int k = lane / kLanes;
    if (lane % kLanes == 0 && cb + k / 4 < cend) put(cb + k / 4, k % 4, sum);
  };
  ColBuf<QT> qa[C], qb[C];
  load_cols<QT, C, R, NT>(qa, base, ldq, c0, cend, row0, lane, N);
  for (int g = 0; g < ng; g += 2) {
    const int cb = c0 + g * C;
    if (cb >= cend) return;
    const bool second = g + 1 < ng && cb + C < cend;
    if (second) load_cols<QT, C, R, NT>(qb, base, ldq, cb + C, cend, row0, lane, N);
    out(cb, w.template dot<QT, C>(qa, lane));
    if (!second) return;
    if (g + 2 < ng && cb + 2 * C < cend) load_cols<QT, C, R, NT>(qa, base, ldq, cb + 2 * C, cend, row0, lane, N);
    out(cb + C, w.template dot<QT, C>(qb, lane));
  }
}

// Column groups of a launch: gs groups of `width` Schur columns, then the
// Krylov columns' groups (a group never mixes the two)
struct ColGroups {
  int gs, width;
};

// Many row tiles: a workgroup's four wavefronts take ng batches of C columns
// each of one tile; the partial sums of every tile go to memory and
// kred_kernel adds them in a fixed order.  Bound by memory: 12^4 x 32 slots,
// 40 Schur and 130 FP32 columns, 8.4 GB: 1.88 ms with the reduction, 4.5 TB/s
// (2.45 ms with one column's loads in flight and six shuffles for each of its
// four sums); without Schur columns 4.9 TB/s, of the 6.1 that a plain read of
// this size reaches.
template <typename VT, int C>
__global__ void __launch_bounds__(256) kdot_kernel(KrylovArgs A, int with_z, ColGroups G, int ng, int ngroups,
                                                   int keep) {
  constexpr int R = rows_per_lane<VT>();
  int rt, zb, cg;
  if (!tile_of<false, false>(blockIdx.x, A.nb * ngroups, A.nb, A.nrt_dot, A.N, rt, zb, cg)) return;
  const int r = slot_of(A, zb);
  const int lane = threadIdx.x & 63, wave = wave_id();
  const int N = A.N, kcols = step_of(A, zb), J = A.m + kcols;
  const int row0 = rt * kDRows;
  const bool schur = cg < G.gs;
  const int c0 = (schur ? cg : cg - G.gs) * G.width + wave * ng * C, cend = schur ? A.m : kcols;
  const bool raw = cg == 0 && wave == 0;
  if (c0 >= cend && !raw) return;
  Weights<VT, R> w;
  w.load(A, r, row0, lane, with_z);
  if (raw) w.raw_sums(A.Pcd + (size_t)r * A.cdstride + 4 * rt, lane);
  if (c0 >= cend) return;
  double* pa = reinterpret_cast<double*>(A.Pa + (size_t)r * A.pstride + (size_t)rt * A.ldp);
  double* pb = reinterpret_cast<double*>(A.Pb + (size_t)r * A.pstride + (size_t)rt * A.ldp);
  const int off = schur ? 0 : A.m;
  auto put = [&](int c, int k, double sum) { (k < 2 ? pa : pb)[2 * (off + c) + (k & 1)] = sum; };
  // FP64 Schur columns beside FP32 Krylov columns: half the batch for the same bytes
  constexpr int CS = R == 2 && C > 1 ? C / 2 : C;
  const VT* V = static_cast<const VT*>(A.V) + (size_t)r * A.vstride;
  if (schur)
    dot_walk<double2, CS, R, false>(w, A.S, A.ldq, c0, ng * (C / CS), cend, row0, lane, N, put);
  else if (rt < A.nrt_dot - keep)
    dot_walk<VT, C, R, true>(w, V, A.ldq, c0, ng, cend, row0, lane, N, put);
  else
    dot_walk<VT, C, R, false>(w, V, A.ldq, c0, ng, cend, row0, lane, N, put);
}

// lane's part of raw scalar q (0..3) over the row tiles: tiles lane, lane + 64, ...
__device__ inline double raw_part(const double* __restrict__ Pcd, int q, int nrt, int lane) {
  double acc = 0.0;
  for (int t0 = lane; t0 < nrt; t0 += 64 * 8) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = (t0 + 64 * u < nrt) ? Pcd[4 * (t0 + 64 * u) + q] : 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) acc += v[u];
  }
  return acc;
}

// Few row tiles (kPartTiles or fewer): a workgroup takes C ng columns and the
// tiles p, p + 8, ... of part p = 0..7, a wavefront per tile, and adds their
// sums in order; the update pass adds the eight parts in order itself.  The
// sums are those of kdot_kernel and kred_kernel, without the reduction's
// launch (3.6 us of a step).  A wavefront's weights are as many bytes as one or
// two columns, so one slot's wavefronts keep them for ng columns (C = 1): dot
// and update of a step, two columns a workgroup / this, 2400 sites FP64, 150
// columns 32.8 / 28.0 us, 300 columns 54.4 / 49; 2430 sites FP32, 150 columns
// 26.4 / 22.1, 300 columns 43.4 / 35.9; 6^4, 150 columns 20.2 / 19.8.
constexpr int kParts = 8;
constexpr int kPartTiles = 64;
constexpr int kPartWidth = 16;  // most columns of a workgroup: a thread of its first wavefront per sum
template <typename VT, int C>
__global__ void __launch_bounds__(64 * kPartTiles / kParts) kdot_parts_kernel(KrylovArgs A, int with_z, ColGroups G,
                                                                      int ng) {
  constexpr int R = rows_per_lane<VT>();
  static_assert(kParts == kXcds, "the tiles of a part run on one XCD");
  const unsigned l = blockIdx.x / kParts;
  const int cg = (int)(l / A.nb), zb = (int)(l - (unsigned)cg * A.nb);
  const int part = rotate_tile(blockIdx.x % kParts, zb, A.nrt_dot);
  const int r = slot_of(A, zb);
  const int lane = threadIdx.x & 63, wave = wave_id();
  const int kcols = step_of(A, zb);
  const bool schur = cg < G.gs;
  const int c0 = (schur ? cg : cg - G.gs) * G.width, cend = min(c0 + G.width, schur ? A.m : kcols);
  const bool raw = cg == 0;
  const int ntiles = part < A.nrt_dot ? (A.nrt_dot - part + kParts - 1) / kParts : 0;
  __shared__ double sums[kPartTiles / kParts][4 * kPartWidth];
  const int nw = blockDim.x >> 6;
  auto walk = [&](const auto* base, auto tag) {
    using QT = decltype(tag);
    for (int tl = wave; tl < ntiles; tl += nw) {
      const int rt = part + kParts * tl, row0 = rt * kDRows;
      if constexpr (C == 1) {
        Weights<VT, R> w;
        w.load(A, r, row0, lane, with_z);
        if (c0 < cend)
          dot_walk<QT, 1, R, false>(w, base, A.ldq, c0, ng, cend, row0, lane, A.N,
                                    [&](int c, int k, double sum) { sums[tl][4 * (c - c0) + k] = sum; });
        if (raw) w.raw_sums(A.Pcd + (size_t)r * A.cdstride + 4 * rt, lane);
      } else {
        ColBuf<QT> q[C];
        if (c0 < cend) load_cols<QT, C, R>(q, base, A.ldq, c0, cend, row0, lane, A.N);
        Weights<VT, R> w;
        w.load(A, r, row0, lane, with_z);
        if (c0 < cend) {
          const double sum = w.template dot<QT, C>(q, lane);
          if (lane % (16 / C) == 0) sums[tl][lane / (16 / C)] = sum;
        }
        if (raw) w.raw_sums(A.Pcd + (size_t)r * A.cdstride + 4 * rt, lane);
      }
    }
  };
  if (c0 < cend || raw) {
    if (schur)
      walk(A.S, double2{});
    else
      walk(static_cast<const VT*>(A.V) + (size_t)r * A.vstride, VT{});
  }
  __syncthreads();
  const int k = threadIdx.x;
  if (k < 4 * (cend - c0)) {
    double acc = 0.0;
    for (int tl = 0; tl < ntiles; ++tl) acc += sums[tl][k];
    double2* P = (k & 2 ? A.Pb : A.Pa) + (size_t)r * A.pstride + (size_t)part * A.ldp;
    reinterpret_cast<double*>(P + (schur ? 0 : A.m) + c0 + k / 4)[k & 1] = acc;
  }
}

// The fewest row tiles (kParts or fewer: one per part): a workgroup takes C
// columns over all rows, a wavefront per tile, and adds the tiles' sums from
// LDS in order, so that a, b and the raw scalars are complete.
template <typename VT, int C>
__global__ void __launch_bounds__(64 * kParts) kdot_whole_kernel(KrylovArgs A, int with_z, ColGroups G) {
  constexpr int R = rows_per_lane<VT>();
  const int cg = blockIdx.x / A.nb, zb = blockIdx.x - cg * A.nb;
  const int r = slot_of(A, zb);
  const int lane = threadIdx.x & 63, wave = wave_id();
  const int kcols = step_of(A, zb);
  const bool schur = cg < G.gs;
  const int c0 = (schur ? cg : cg - G.gs) * C, cend = schur ? A.m : kcols;
  const bool raw = cg == 0;
  if (c0 >= cend && !raw) return;
  const int nrt = A.nrt_dot, nw = blockDim.x >> 6;
  __shared__ double sums[kParts][4 * C];
  __shared__ double rsum[4 * kParts];
  auto walk = [&](const auto* base, auto tag) {
    using QT = decltype(tag);
    for (int rt = wave; rt < nrt; rt += nw) {
      const int row0 = rt * kDRows;
      ColBuf<QT> q[C];
      if (c0 < cend) load_cols<QT, C, R>(q, base, A.ldq, c0, cend, row0, lane, A.N);
      Weights<VT, R> w;
      w.load(A, r, row0, lane, with_z);
      if (c0 < cend) {
        const double sum = w.template dot<QT, C>(q, lane);
        if (lane % (16 / C) == 0) sums[rt][lane / (16 / C)] = sum;
      }
      if (raw) w.raw_sums(rsum + 4 * rt, lane);
    }
  };
  if (schur)
    walk(A.S, double2{});
  else
    walk(static_cast<const VT*>(A.V) + (size_t)r * A.vstride, VT{});
  __syncthreads();
  const int k = threadIdx.x;
  if (k < 4 * C && c0 + k / 4 < cend) {
    double acc = 0.0;
    for (int rt = 0; rt < nrt; ++rt) acc += sums[rt][k];
    double2* out = (k & 2 ? A.b : A.a) + (size_t)r * A.abstride;
    reinterpret_cast<double*>(out + (schur ? 0 : A.m) + c0 + k / 4)[k & 1] = acc;
  }
  if (raw)  // scalar q of wavefronts q, q + nw, ...
    for (int q = wave; q < 4; q += nw) {
      const double acc = wsum1(raw_part(rsum, q, nrt, lane));
      if (lane == 0) A.sc[(size_t)r * kScStride + kScRawC + q] = acc;
    }
}

// Column c of a (or b) from the eight parts P, in order
__device__ inline double2 sum_parts(const double2* __restrict__ P, int ldp, int c) {
  double2 v[kParts];
#pragma unroll
  for (int p = 0; p < kParts; ++p) v[p] = P[(size_t)p * ldp + c];
  double2 sum = v[0];
#pragma unroll
  for (int p = 1; p < kParts; ++p) sum = cadd(sum, v[p]);
  return sum;
}

// reduce the dot partials over row tiles in a fixed order: 32 columns per
// workgroup, 8 threads per column (each sums every 8th row tile), then a
// fixed-order combine; workgroup 0 also sums the scalars c, d, |z|^2.
// parts: the partials are those of kdot_parts_kernel (eight per column)
__global__ void __launch_bounds__(256) kred_kernel(KrylovArgs A, int parts) {
  const int r = slot_of(A, blockIdx.z);
  const int J = A.m + step_of(A, blockIdx.z), nrt = parts ? kParts : A.nrt_dot;
  const double2* Pa = A.Pa + (size_t)r * A.pstride;
  const double2* Pb = A.Pb + (size_t)r * A.pstride;
  const double* Pcd = A.Pcd + (size_t)r * A.cdstride;
  const int cl = threadIdx.x & 31, part = threadIdx.x >> 5;
  const int c = blockIdx.x * 32 + cl;
  const double2 zero = make_double2(0.0, 0.0);
  double2 sa = zero, sb = zero;
  // tiles t = part, part + 8, ... in that order, eight loads in flight
  if (c < J)
    for (int t0 = part; t0 < nrt; t0 += 64) {
      double2 va[8], vb[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int t = t0 + 8 * u;
        va[u] = t < nrt ? Pa[(size_t)t * A.ldp + c] : zero;
        vb[u] = t < nrt ? Pb[(size_t)t * A.ldp + c] : zero;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        sa = cadd(sa, va[u]);
        sb = cadd(sb, vb[u]);
      }
    }
  __shared__ double2 ra[8][33], rb[8][33];
  ra[part][cl] = sa;
  rb[part][cl] = sb;
  __syncthreads();
  if (part == 0 && c < J) {
    double2 ta = ra[0][cl], tb = rb[0][cl];
    for (int q = 1; q < 8; ++q) {
      ta = cadd(ta, ra[q][cl]);
      tb = cadd(tb, rb[q][cl]);
    }
    A.a[(size_t)r * A.abstride + c] = ta;
    A.b[(size_t)r * A.abstride + c] = tb;
  }
  if (blockIdx.x == 0) {
    // wavefront q sums scalar q over the row tiles: lane partials, then a
    // fixed butterfly
    const int q = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const double acc = wsum1(raw_part(Pcd, q, A.nrt_dot, lane));
    if (lane == 0) A.sc[(size_t)r * kScStride + kScRawC + q] = acc;
  }
}

// Step scalars from a, b and the raw sums.  Each thread brings its partial
// sums over the columns c = tid, tid + NT, ... (|a_c|^2 and conj(a_c) b_c);
// they are combined by wavefront butterflies and then over the wavefronts in
// a fixed order, so every workgroup computes them identically.
struct StepScalars {
  double rho, inv;
  double2 gam, gr;
  bool brk, finite;
  double scale;
};

template <int NW>
__device__ StepScalars step_scalars(const KrylovArgs& A, int r, double ref, double s0, double2 s12,
                                    double* red /* LDS [3][NW] */, const double* raw /* the raw sums */) {
  const int lane = threadIdx.x & 63, wave = wave_id();
  s0 = wsum1(s0);
  s12 = wsum2(s12);
  if (lane == 0) {
    red[wave] = s0;
    red[NW + wave] = s12.x;
    red[2 * NW + wave] = s12.y;
  }
  __syncthreads();
  double aa = red[0];
  double2 ab = make_double2(red[NW], red[2 * NW]);
  for (int w = 1; w < NW; ++w) {
    aa += red[w];
    ab.x += red[NW + w];
    ab.y += red[2 * NW + w];
  }
  StepScalars st;
  const double c = raw[0];
  const double2 d = make_double2(raw[1], raw[2]);
  const double zz = raw[3];
  const double rho2 = c - aa;
  const double rho = rho2 > 0.0 ? sqrt(rho2) : 0.0;
  st.finite = isfinite(c) && isfinite(d.x) && isfinite(d.y) && isfinite(zz);
  st.brk = !(rho > A.brk_tol * ref) || !st.finite;
  st.inv = st.brk ? 0.0 : 1.0 / rho;
  st.rho = st.brk ? 0.0 : rho;
  st.gam = cscale(csub(d, ab), st.inv);
  st.gr = cscale(st.gam, st.inv);
  st.scale = sqrt(zz) * st.inv;
  return st;
}

// Coefficients a, b of up to kCoefCap columns of a step in LDS, as every
// wavefront of the update pass reads them; longer steps take them in spans.
// kCoefPad zeros follow, the coefficients of a last batch's missing columns.
constexpr int kCoefCap = 1024;
constexpr int kCoefPad = 64;
struct Coefs {
  const double2 *a, *b;  // LDS, column c at c - c0
  int c0;
};

// a, b of columns [c0, c0 + n) into LDS from the eight parts of the dot pass
__device__ inline void fetch_coefs(const KrylovArgs& A, int r, int c0, int n, double2* la, double2* lb) {
  const int tid = threadIdx.x, nt = blockDim.x;
  const double2* Pa = A.Pa + (size_t)r * A.pstride;
  const double2* Pb = A.Pb + (size_t)r * A.pstride;
  for (int i = tid; i < 2 * n; i += nt) {
    const bool second = i >= n;
    const int c = second ? i - n : i;
    (second ? lb : la)[c] = sum_parts(second ? Pb : Pa, A.ldp, c0 + c);
  }
  for (int i = tid; i < kCoefPad; i += nt) la[n + i] = lb[n + i] = make_double2(0.0, 0.0);
}

// the raw sums u^dag u, u^dag z (re, im), |z|^2 into LDS: wavefront q < 4 sums
// scalar q over the row tiles
__device__ inline void fetch_raw(const KrylovArgs& A, int r, double* raw) {
  const int lane = threadIdx.x & 63, wave = wave_id();
  if (wave >= 4) return;
  const double acc = wsum1(raw_part(A.Pcd + (size_t)r * A.cdstride, wave, A.nrt_dot, lane));
  if (lane == 0) raw[wave] = acc;
}

// this thread's partial sums over the columns c = tid, tid + NT, ... of a span
// (spans are multiples of NT): |a_c|^2 and conj(a_c) b_c
template <int NT>
__device__ inline void scalar_partials(const double2* la, const double2* lb, int n, double& s0, double2& s12) {
  for (int i = threadIdx.x; i < n; i += NT) {
    const double2 x1 = la[i], x2 = lb[i];
    s0 += cabs2(x1);
    s12 = cadd(s12, cmulc(x1, x2));
  }
}

// Hessenberg column J and the re-orthogonalisation of column J-1, one row per
// wavefront (the lanes split the sum over columns); at j = 0 the correction
// goes to c0 instead.
__device__ void hcol_row_wave(const KrylovArgs& A, int r, int j, int row, int lane, const StepScalars& st) {
  const int J = A.m + j;
  const double2* a = A.a + (size_t)r * A.abstride;
  const double2* b = A.b + (size_t)r * A.abstride;
  double2* H = A.H + (size_t)r * A.hstride;
  const int ldh = A.ldh;
  const int lim = (j > 0) ? J - 1 : J;
  double2 ha = make_double2(0.0, 0.0);
  if (row < J)  // row J of columns < J-1 is below the subdiagonal (zero)
    // columns l = lane, lane + 64, ... in order, 4 loads of each operand in
    // flight per lane (deeper batches raise the kernel's register count, and
    // with it lower the occupancy of the sweep workgroups)
    for (int l0 = 0; l0 < lim; l0 += 4 * 64) {
      double2 hv[4], xv[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int l = l0 + t * 64 + lane;
        if (l < lim) {
          hv[t] = H[(size_t)l * ldh + row];
          xv[t] = a[l];
        }
      }
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (l0 + t * 64 + lane < lim) ha = cfma(hv[t], xv[t], ha);
    }
  ha = wsum2(ha);
  if (lane != 0) return;
  const double rho = st.rho, inv = st.inv;
  const double2 g = (row < J) ? b[row] : st.gam;
  if (j > 0) {
    const double2 hl = (row < J) ? cadd(H[(size_t)(J - 1) * ldh + row], a[row]) : make_double2(rho, 0.0);
    ha = cfma(hl, a[J - 1], ha);
    H[(size_t)(J - 1) * ldh + row] = hl;
  } else if (row < A.m) {
    double2* c0 = A.c0 + (size_t)r * A.c0stride;
    c0[row] = cadd(c0[row], a[row]);
  }
  H[(size_t)J * ldh + row] = cscale(csub(g, ha), inv);
}

// The same row with the coefficients in LDS; the gather of its first 4 x 64
// entries and its entry of column J-1 are under way before they are (start).
struct HRow {
  double2 hv[4], hl, ha, c0;
  __device__ inline void load(const double2* H, int ldh, int row, int lane, int l0, int end) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int l = l0 + t * 64 + lane;
      if (l < end) hv[t] = H[(size_t)l * ldh + row];
    }
  }
  __device__ inline void start(const KrylovArgs& A, int r, int j, int row, int lane, int lim) {
    const int J = A.m + j;
    ha = make_double2(0.0, 0.0);
    if (row >= J) return;
    const double2* H = A.H + (size_t)r * A.hstride;
    load(H, A.ldh, row, lane, 0, lim);
    if (j > 0)
      hl = H[(size_t)(J - 1) * A.ldh + row];
    else if (row < A.m)
      c0 = A.c0[(size_t)r * A.c0stride + row];
  }
  // columns l = lane, lane + 64, ... of [c0, c0 + n) below lim, in order, 4
  // loads in flight per lane
  __device__ inline void sum(const KrylovArgs& A, int r, int row, int lane, int c0, int n, int lim,
                             const double2* la) {
    const double2* H = A.H + (size_t)r * A.hstride;
    const int end = min(c0 + n, lim);
    for (int l0 = c0; l0 < end; l0 += 4 * 64) {
      if (l0 > 0) load(H, A.ldh, row, lane, l0, end);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int l = l0 + t * 64 + lane;
        if (l < end) ha = cfma(hv[t], la[l - c0], ha);
      }
    }
  }
  __device__ inline void store(const KrylovArgs& A, int r, int j, int row, int lane, double2 b_row, double2 a_row,
                               double2 a_last, const StepScalars& st) {
    const int J = A.m + j;
    double2* H = A.H + (size_t)r * A.hstride;
    ha = wsum2(ha);
    if (lane != 0) return;
    const double2 g = (row < J) ? b_row : st.gam;
    if (j > 0) {
      const double2 h1 = (row < J) ? cadd(hl, a_row) : make_double2(st.rho, 0.0);
      ha = cfma(h1, a_last, ha);
      H[(size_t)(J - 1) * A.ldh + row] = h1;
    } else if (row < A.m) {
      A.c0[(size_t)r * A.c0stride + row] = cadd(c0, a_row);
    }
    H[(size_t)J * A.ldh + row] = cscale(csub(g, ha), st.inv);
  }
};

// sa += sum_c q_c[i] coef_c over the columns c = c0, c0 + NW, ... < cend, in
// that order; column c sits at base + (c - cofs) ldq.  Each batch of KB column
// loads (and their coefficients) is issued before its arithmetic, the last,
// partial batch too: a slot past cend reloads column cend - 1 (a cache hit)
// and adds it with coefficient zero, which leaves the sums unchanged since
// basis vectors are finite.
// (rows past N load row N-1 and are never written: unconditional loads; c
// is wavefront-uniform, so the coefficients come through scalar loads)
template <typename QT, int KB, int NW>
__device__ inline void combine_cols(const QT* __restrict__ base, int cofs, size_t ldq, int c, int cend, int i,
                                    const double2* __restrict__ cf, double2& sa) {
  const double2 zero = make_double2(0.0, 0.0);
  for (; c < cend; c += KB * NW) {
    double2 qv[KB], ca[KB];
#pragma unroll
    for (int t = 0; t < KB; ++t) {
      const int cc = c + t * NW, cl = min(cc, cend - 1);
      qv[t] = ld2(base + (size_t)(cl - cofs) * ldq, i);
      ca[t] = cf[cl];
      if (cc >= cend) ca[t] = zero;
    }
#pragma unroll
    for (int t = 0; t < KB; ++t) sa = cfma(qv[t], ca[t], sa);
  }
}

// KB column entries of a lane's R rows, as loaded
template <typename QT, int KB, int R>
struct SweepBuf {
  double2 q[KB][R];
  template <bool NT>
  __device__ inline void load(const QT* __restrict__ p, int t, int i) {
#pragma unroll
    for (int k = 0; k < R; ++k) q[t][k] = col_load<NT>(p + i + k);
  }
  __device__ inline double2 at(int t, int k) const { return q[t][k]; }
};
template <int KB>
struct SweepBuf<float2, KB, 2> {
  float4 q[KB];
  template <bool NT>
  __device__ inline void load(const float2* __restrict__ p, int t, int i) {
    q[t] = col_load<NT>(reinterpret_cast<const float4*>(p + i));
  }
  __device__ inline double2 at(int t, int k) const {
    return k ? make_double2((double)q[t].z, (double)q[t].w) : make_double2((double)q[t].x, (double)q[t].y);
  }
};

// sa += sum_c q_c a_c, sb += sum_c q_c b_c for a lane's R rows over the
// columns c, c + NW, ... < cend of one base (column c at base + (c - cofs)
// ldq), in that order, KB columns at a time with the next batch's loads issued
// before the current batch's sums (two register sets).  start() issues the
// first batch, before the coefficients are needed.  A slot past cend reloads
// column cend - 1 (a cache hit) and adds it with coefficient zero, which
// leaves the sums unchanged since basis vectors are finite.
template <typename QT, int KB, int NW, int R>
struct Sweep {
  SweepBuf<QT, KB, R> x, y;
  const QT* base;
  size_t ldq;
  int cofs, c, cend, i;
  __device__ inline void fill(SweepBuf<QT, KB, R>& b, int cb) {
#pragma unroll
    for (int t = 0; t < KB; ++t) b.template load<false>(base + (size_t)(min(cb + t * NW, cend - 1) - cofs) * ldq, t, i);
  }
  __device__ inline void start() {
    if (c < cend) fill(x, c);
  }
  // the columns of one batch; LAST (the Schur part, which other columns'
  // coefficients follow): those past cend weigh nothing
  template <bool LAST>
  __device__ inline void add(const SweepBuf<QT, KB, R>& b, int cb, const Coefs& cf, double2 (&sa)[R],
                             double2 (&sb)[R]) {
    const double2 zero = make_double2(0.0, 0.0);
    const double2 *pa = cf.a + (cb - cf.c0), *pb = cf.b + (cb - cf.c0);
#pragma unroll
    for (int t = 0; t < KB; ++t) {
      double2 ca = pa[t * NW], cb2 = pb[t * NW];
      if (LAST && cb + t * NW >= cend) ca = cb2 = zero;
#pragma unroll
      for (int k = 0; k < R; ++k) {
        sa[k] = cfma(b.at(t, k), ca, sa[k]);
        sb[k] = cfma(b.at(t, k), cb2, sb[k]);
      }
    }
  }
  // one register set (the Schur columns, a batch or two per wavefront)
  __device__ inline void run_single(const Coefs& cf, double2 (&sa)[R], double2 (&sb)[R]) {
    while (c < cend) {
      add<true>(x, c, cf, sa, sb);
      c += KB * NW;
      if (c < cend) fill(x, c);
    }
  }
  __device__ inline void run(const Coefs& cf, double2 (&sa)[R], double2 (&sb)[R]) {
    for (; c < cend; c += 2 * KB * NW) {
      const int c1 = c + KB * NW, c2 = c + 2 * KB * NW;
      if (c1 < cend) fill(y, c1);
      add<false>(x, c, cf, sa, sb);
      if (c1 >= cend) return;
      if (c2 < cend) fill(x, c2);
      add<false>(y, c1, cf, sa, sb);
    }
  }
};

// sa += sum_c q_c a_c, sb += sum_c q_c b_c as Sweep forms them, with the
// reduced coefficients read from memory (c is wavefront-uniform, so they come
// through scalar loads): one batch of KB column loads and their coefficients
// at a time, the last, partial batch too
template <typename QT, int KB, int NW, int R, bool NT>
__device__ inline void sweep_mem(const QT* __restrict__ base, int cofs, size_t ldq, int c, int cend, int i,
                                 const double2* __restrict__ av, const double2* __restrict__ bv, double2 (&sa)[R],
                                 double2 (&sb)[R]) {
  const double2 zero = make_double2(0.0, 0.0);
  for (; c < cend; c += KB * NW) {
    SweepBuf<QT, KB, R> q;
    double2 ca[KB], cb[KB];
#pragma unroll
    for (int t = 0; t < KB; ++t) {
      const int cc = c + t * NW, cl = min(cc, cend - 1);
      q.template load<NT>(base + (size_t)(cl - cofs) * ldq, t, i);
      ca[t] = av[cl];
      cb[t] = bv[cl];
      if (cc >= cend) ca[t] = cb[t] = zero;
    }
#pragma unroll
    for (int t = 0; t < KB; ++t)
#pragma unroll
      for (int k = 0; k < R; ++k) {
        sa[k] = cfma(q.at(t, k), ca[t], sa[k]);
        sb[k] = cfma(q.at(t, k), cb[t], sb[k]);
      }
  }
}

// first column >= m that wavefront w of NW takes (c = w mod NW)
template <int NW>
__device__ inline int first_col(int m, int w) { return m + ((w - m % NW) + NW) % NW; }

// update pass.  The first workgroups (nh per slot, padded to whole rounds of
// the XCDs) compute the Hessenberg column J (one row per wavefront), the
// others each own 64 R rows and all J columns: their NW wavefronts take
// interleaved columns, combined in LDS in a fixed order.  R = 1 for FP64
// columns; R = 2 for FP32 columns, whose lanes then take two adjacent rows
// each, so that a column load is 16 bytes per lane (every row's sums are the
// same as with R = 1).  Both kinds compute the step scalars; the Hessenberg
// rows, a strided gather, run beside the sweeps.  Every operand that does not
// depend on the coefficients is loaded first.  Small launches are bound by the
// chain of waits (4^4, 20 columns: 4.8 us, of them 2.45 an empty launch), large
// ones by memory (8^4 x 6 slots, 30 + 150 columns, 732 MB: 140 us, 5.2 TB/s;
// 148 us before the rows of a tile stayed on one XCD).
// PARTS (small launches): every workgroup adds the dot pass's eight parts
// itself and keeps the step's coefficients in LDS (steps of more than
// kCoefCap columns in spans of that many); two register sets of KB columns.
// Else the coefficients are reduced in memory (kred_kernel).
template <typename VT, int KB, int NW, bool PARTS>
__global__ void __launch_bounds__(64 * NW, 4) kupdate_kernel(KrylovArgs A, int nh, unsigned nhess, int keep) {
  constexpr int NT = 64 * NW;
  constexpr int R = rows_per_lane<VT>();
  constexpr int kSub = kDRows / (64 * R);  // workgroups per row tile
  static_assert(kCoefCap % NT == 0, "spans hold whole rounds of the threads");
  const bool hess = blockIdx.x < nhess;
  int zb, bb, rt = 0;
  if (hess) {
    bb = blockIdx.x / A.nb;
    zb = blockIdx.x - bb * A.nb;
    if (bb >= nh) return;
  } else {
    int sub;
    if (!tile_of<true, PARTS>(blockIdx.x - nhess, A.nb * kSub, A.nb, A.nrt_dot, A.N, rt, zb, sub)) return;
    bb = rt * kSub + sub;
    if (bb * 64 * R >= A.N) return;
  }
  const int r = slot_of(A, zb);
  const int tid = threadIdx.x, lane = tid & 63, wave = wave_id();
  const int N = A.N, j = step_of(A, zb), J = A.m + j;
  const double2 zero = make_double2(0.0, 0.0);
  const double ref = A.sc[(size_t)r * kScStride + kScRef + (j & 1)];
  const double2* av = A.a + (size_t)r * A.abstride;
  const double2* bv = A.b + (size_t)r * A.abstride;
  __shared__ double red[3 * NW];
  __shared__ double raw_lds[4];
  const double* raw = PARTS ? raw_lds : A.sc + (size_t)r * kScStride + kScRawC;
  __shared__ double2 ps[2][NW][64 * R];
  extern __shared__ double2 coef_lds[];  // PARTS: a, then b, of a span
  static_assert(!PARTS || NW * KB <= kCoefPad, "the padding covers a batch");
  double2* la = coef_lds;
  double2* lb = coef_lds + min(J, kCoefCap) + kCoefPad;
  double s0 = 0.0;
  double2 s12 = zero;
  if (hess) {
    const int row = bb * NW + wave, lim = (j > 0) ? J - 1 : J;
    if constexpr (PARTS) {
      HRow h;
      h.start(A, r, j, row, lane, lim);
      fetch_raw(A, r, raw_lds);
      double2 a_row = zero, b_row = zero, a_last = zero;
      for (int c0 = 0; c0 < J; c0 += kCoefCap) {
        const int n = min(J - c0, kCoefCap);
        if (c0) __syncthreads();
        fetch_coefs(A, r, c0, n, la, lb);
        __syncthreads();
        scalar_partials<NT>(la, lb, n, s0, s12);
        if (row < J) {  // row J of columns < J-1 is below the subdiagonal (zero)
          h.sum(A, r, row, lane, c0, n, lim, la);
          if (row >= c0 && row < c0 + n) {
            a_row = la[row - c0];
            b_row = lb[row - c0];
          }
        }
        if (J - 1 < c0 + n) a_last = la[J - 1 - c0];
      }
      __syncthreads();  // raw, where J = 0
      const StepScalars st = step_scalars<NW>(A, r, ref, s0, s12, red, raw);
      if (row <= J) h.store(A, r, j, row, lane, b_row, a_row, a_last, st);
    } else {
      scalar_partials<NT>(av, bv, J, s0, s12);
      const StepScalars st = step_scalars<NW>(A, r, ref, s0, s12, red, raw);
      if (row <= J) hcol_row_wave(A, r, j, row, lane, st);
    }
    return;
  }
  const int blk = bb;
  const int i = blk * 64 * R + R * lane;  // this lane's first row
  const bool ok = i < N;                  // N is even: with R = 2, row i + 1 < N too
  const int il = ok ? i : N - R;
  // u may be updated in place (unext == u): each lane reads its u[i] before
  // writing u'[i], and no other thread of the step touches row i of u
  const double2* u = A.u + (size_t)r * A.ustride;
  const VT* __restrict__ z = static_cast<const VT*>(A.z) + (size_t)r * A.zstride;
  double2 ui[R], zi[R];
#pragma unroll
  for (int k = 0; k < R; ++k) {
    ui[k] = u[il + k];
    zi[k] = ld2(z, il + k);
  }
  // sweep: sa = Q a, sb = Q b (the step scalars enter only afterwards:
  // Q (b - gr a) = sb - gr sa).  FP64 Schur columns of a row pair take two
  // loads per lane: half the batch keeps the bytes in flight (the batch size
  // does not change any sum)
  double2 sa[R], sb[R];
#pragma unroll
  for (int k = 0; k < R; ++k) sa[k] = sb[k] = zero;
  constexpr int KS = R == 1 || KB == 2 ? KB : KB / 2;
  const VT* V = static_cast<const VT*>(A.V) + (size_t)r * A.vstride;
  if constexpr (PARTS) {
    for (int c0 = 0; c0 < J || c0 == 0; c0 += kCoefCap) {
      const int n = min(J - c0, kCoefCap), ce = c0 + n;
      if (c0) __syncthreads();
      fetch_coefs(A, r, c0, n, la, lb);
      // this wavefront's columns of the span: c = wave mod NW (c0 is a multiple of NW)
      Sweep<double2, KS, NW, R> ws{{}, {}, A.S, A.ldq, 0, c0 + wave, min(ce, A.m), il};
      Sweep<VT, KB, NW, R> wv{{}, {}, V, A.ldq, A.m, max(c0 + wave, first_col<NW>(A.m, wave)), ce, il};
      ws.start();
      wv.start();
      if (c0 == 0) fetch_raw(A, r, raw_lds);
      __syncthreads();
      const Coefs cf{la, lb, c0};
      ws.run_single(cf, sa, sb);
      wv.run(cf, sa, sb);
      scalar_partials<NT>(la, lb, n, s0, s12);
    }
  } else {
    sweep_mem<double2, KS, NW, R, false>(A.S, 0, A.ldq, wave, min(J, A.m), il, av, bv, sa, sb);
    const int cv = first_col<NW>(A.m, wave);
    if (rt >= keep)
      sweep_mem<VT, KB, NW, R, true>(V, A.m, A.ldq, cv, J, il, av, bv, sa, sb);
    else
      sweep_mem<VT, KB, NW, R, false>(V, A.m, A.ldq, cv, J, il, av, bv, sa, sb);
    scalar_partials<NT>(av, bv, J, s0, s12);
  }
#pragma unroll
  for (int k = 0; k < R; ++k) {
    ps[0][wave][R * lane + k] = sa[k];
    ps[1][wave][R * lane + k] = sb[k];
  }
  const StepScalars st = step_scalars<NW>(A, r, ref, s0, s12, red, raw);  // contains __syncthreads
  if (blk == 0 && tid == 0) {
    double* sc = A.sc + (size_t)r * kScStride;
    sc[kScRho] = st.rho;
    sc[kScInv] = st.inv;
    sc[kScGamRe] = st.gam.x;
    sc[kScGamIm] = st.gam.y;
    sc[kScGrRe] = st.gr.x;
    sc[kScGrIm] = st.gr.y;
    sc[kScScale] = st.scale;
    // reference size for the next step's breakdown test (the other parity
    // slot: this step's slot is still being read by other workgroups)
    sc[kScRef + ((j + 1) & 1)] = st.scale;
    if (j == 0 && A.beta) A.beta[r] = st.rho;
    if (A.flag) {
      int* f = A.flag + r;
      if (!st.finite)
        *f = -1;
      else if (st.brk && *f == 0)
        *f = j + 1;
    }
  }
  // combine the wavefronts (fixed order) and write v_J and u'
  if (wave == 0 && ok) {
    VT* vout = static_cast<VT*>(A.V) + (size_t)r * A.vstride + (size_t)(J - A.m) * A.ldq;
    double2 vo[R], nx[R];
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int row = R * lane + q;
      double2 ta = ps[0][0][row], tb = ps[1][0][row];
#pragma unroll
      for (int w = 1; w < NW; ++w) {
        ta = cadd(ta, ps[0][w][row]);
        tb = cadd(tb, ps[1][w][row]);
      }
      const double2 te = csub(tb, cmul(st.gr, ta));
      vo[q] = cscale(csub(ui[q], ta), st.inv);
      nx[q] = cscale(csub(csub(zi[q], cmul(st.gr, ui[q])), te), st.inv);
    }
#pragma unroll
    for (int q = 0; q < R; ++q) {
      st2(vout, i + q, vo[q]);
      A.unext[(size_t)r * A.ustride + i + q] = nx[q];
      if (A.ulonext) st2(static_cast<VT*>(A.ulonext) + (size_t)r * A.zstride, i + q, nx[q]);
    }
  }
}

// y = S c_S + V c_V for slot r (coefficients c[0..ncol)): 64 rows per
// workgroup, wavefront w sums the columns c = w mod kUWaves, fixed-order combine
template <typename VT>
__global__ void __launch_bounds__(kUThreads) kcombine_kernel(KrylovArgs A, const double2* __restrict__ coef,
                                                             int cstride, double2* __restrict__ y, size_t ystride,
                                                             int ncol) {
  const int r = slot_of(A, blockIdx.z);
  const int lane = threadIdx.x & 63, wave = wave_id();
  const int i = blockIdx.x * 64 + lane;
  const bool ok = i < A.N;
  const double2* cf = coef + (size_t)r * cstride;
  double2 acc = make_double2(0.0, 0.0);
  const int il = ok ? i : A.N - 1;
  combine_cols<double2, kCBatch, kUWaves>(A.S, 0, A.ldq, wave, min(ncol, A.m), il, cf, acc);
  combine_cols<VT, kCBatch, kUWaves>(static_cast<const VT*>(A.V) + (size_t)r * A.vstride, A.m, A.ldq,
                                     first_col<kUWaves>(A.m, wave), ncol, il, cf, acc);
  __shared__ double2 ps[kUWaves][64];
  ps[wave][lane] = acc;
  __syncthreads();
  if (wave == 0 && ok) {
    double2 t = ps[0][lane];
#pragma unroll
    for (int w = 1; w < kUWaves; ++w) t = cadd(t, ps[w][lane]);
    y[(size_t)r * ystride + i] = t;
  }
}

__global__ void set_index_kernel(int* p, int v, int add) {
  if (threadIdx.x == 0) *p = add ? *p + v : v;
}

// dst = H[:n,:n] with column n-1 += a (slot r), dst dense n x n per slot
__global__ void kpatch_kernel(KrylovArgs A, int n, double2* __restrict__ dst, size_t dstride, int with_a) {
  const int r = slot_of(A, blockIdx.z);
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (size_t)n * n) return;
  const int c = (int)(e / n), row = (int)(e - (size_t)c * n);
  const double2* H = A.H + (size_t)r * A.hstride;
  double2 v = H[(size_t)c * A.ldh + row];
  if (with_a && c == n - 1) v = cadd(v, A.a[(size_t)r * A.abstride + row]);
  dst[(size_t)blockIdx.z * dstride + e] = v;
}

}  // namespace

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
void krylov_alloc(KrylovWork& w, int N, size_t ldq, int ncol_cap, int nslots) {
  krylov_free(w);
  (void)ldq;
  w.nrt_dot = (N + kDRows - 1) / kDRows;
  w.ncol_cap = ncol_cap;
  w.nslots = nslots;
  w.ldp = ncol_cap;
  static_assert(kDRows == 512 && kParts == 8, "krylov_part_tiles");
  w.pstride = krylov_part_tiles(N) * ncol_cap;
  w.cdstride = (size_t)4 * w.nrt_dot;
  w.abstride = (size_t)ncol_cap;
  const size_t S = (size_t)nslots;
  SGN_HIP(hipMalloc(&w.Pa, sizeof(double2) * w.pstride * S));
  SGN_HIP(hipMalloc(&w.Pb, sizeof(double2) * w.pstride * S));
  SGN_HIP(hipMalloc(&w.Pcd, sizeof(double) * w.cdstride * S));
  SGN_HIP(hipMalloc(&w.a, sizeof(double2) * w.abstride * S));
  SGN_HIP(hipMalloc(&w.b, sizeof(double2) * w.abstride * S));
  SGN_HIP(hipMalloc(&w.sc, sizeof(double) * kScStride * S));
  SGN_HIP(hipMemset(w.sc, 0, sizeof(double) * kScStride * S));
  SGN_HIP(hipDeviceSynchronize());
}

void krylov_free(KrylovWork& w) {
  for (void* p : {(void*)w.Pa, (void*)w.Pb, (void*)w.Pcd, (void*)w.a, (void*)w.b, (void*)w.sc})
    if (p) (void)hipFree(p);
  w = KrylovWork{};
}

void krylov_bind(const KrylovWork& w, KrylovArgs& A) {
  A.Pa = w.Pa;
  A.Pb = w.Pb;
  A.Pcd = w.Pcd;
  A.ldp = w.ldp;
  A.pstride = w.pstride;
  A.cdstride = w.cdstride;
  A.a = w.a;
  A.b = w.b;
  A.abstride = w.abstride;
  A.sc = w.sc;
  A.nrt_dot = w.nrt_dot;
}

static void check_args(const KrylovWork& w, const KrylovArgs& A) {
  SGN_REQUIRE(A.nb >= 1 && A.nb <= w.nslots && A.nb <= kMaxBatch, SGN_EINVAL, "krylov: batch exceeds workspace");
  // a device step index is shared by every launch slot (all at the same step)
  SGN_REQUIRE(!A.jdev || A.joff >= 0, SGN_EINVAL, "krylov: negative step offset");
  for (int z = 0; z < A.nb; ++z) {
    SGN_REQUIRE(A.act[z] >= 0 && A.act[z] < w.nslots, SGN_EINVAL, "krylov: slot out of range");
    SGN_REQUIRE(A.jv[z] >= 0 && A.m + A.jv[z] <= w.ncol_cap, SGN_EINVAL, "krylov: J exceeds workspace");
  }
}

// columns a launch reads, for the algorithmic byte counts: the FP64 Schur
// part, shared by the slots (once), and the sum of the slots' Krylov parts
static void col_sums(const KrylovArgs& A, double& sum_m, double& sum_k) {
  sum_m = A.m;
  sum_k = 0.0;
  for (int z = 0; z < A.nb; ++z) sum_k += A.jv[z];
}

bool krylov_tune_valid(const KrylovTune& t) {
  return (t.ub == 4 || t.ub == 8 || t.ub == 16) && (t.cpw == 1 || t.cpw == 2 || t.cpw == 4) &&
         (t.uw == 8 || t.uw == 16);
}

template <typename VT, int NW, bool PARTS>
static auto update_kernel_nw(int ub) {
  // ub column loads in flight per lane (PARTS: two register sets of half as
  // many, at most four columns each: 128 registers keep two workgroups per CU)
  switch (ub) {
    case 4: return kupdate_kernel<VT, (PARTS ? 2 : 4), NW, PARTS>;
    case 16: return kupdate_kernel<VT, (PARTS ? 4 : 16), NW, PARTS>;
    default: return kupdate_kernel<VT, (PARTS ? 4 : 8), NW, PARTS>;
  }
}

template <typename VT, bool PARTS>
static auto update_kernel_for(const KrylovTune& t) {
  return t.uw == 16 ? update_kernel_nw<VT, 16, PARTS>(t.ub) : update_kernel_nw<VT, 8, PARTS>(t.ub);
}

// Row tiles whose Krylov columns a pass leaves in the caches for the next pass,
// which walks the other way: the last ones of its walk, as far as they fit
// beside the Schur columns; the others are streamed past the caches.  us for
// dot and update of a step, all cached / all streamed / by this rule: 8^4 x 6
// slots, FP64, 70 columns 126 / 140 / 123, 100 columns 171 / 178 / 166, 200
// columns 334 / 320 / 316; 12^4, 80 columns 146 / 140 / 133, 300 columns 437 /
// 391 / 388; 12^4 x 16, FP32, 130 columns 1628 / 1522 / 1515 (the dot pass
// alone 5.1 -> 5.6 TB/s).  128 or 256 MB instead of 200: within 2 per cent.
constexpr double kKeepBytes = 200e6;
template <typename VT>
static int kept_tiles(const KrylovWork& w, const KrylovArgs& A) {
  double sm, sk;
  col_sums(A, sm, sk);
  const double tile = (double)kDRows * sizeof(VT) * std::max(sk, 1.0);
  return (int)std::min((double)w.nrt_dot, std::max(0.0, kKeepBytes - 16.0 * A.N * sm) / tile);
}

// wavefronts that one slot's dot pass by parts is left with (512 and 1024: up to
// 3 us slower at 1920 sites and 150 columns, 24.3 us), and those from which
// several slots take two columns a workgroup
constexpr size_t kDotWaves = 768, kDotWavesBatch = 2048;

// How a launch forms the dot pass's sums (the same sums in the same order).
// Dot and update of one step back to back, by form (us; the general one with
// its reduction): 4^4, 60 / 280 columns: Whole 9.1 / 13.6, Parts 11.5 / 15.9,
// the former kernels 15.1 / 19.1.  6^4, 80 / 320 columns: Parts 13.2 / 34.8,
// Whole 21.2 / 43.0, former 18.4 / 38.0.  Three slots of 1350 sites, 150
// columns: Parts 43.5, Tiles 47.4, former 46.9.  8^4, 160 columns, FP64:
// Tiles 52.7, Parts 52.4, former 55.7; FP32: Tiles 36.7, Parts 38.2 (56.7
// against 47.5 at 260 columns), former 36.7.  8^4 x 6 slots, 180 columns:
// Tiles 283.5, former 301.7.
// Every workgroup of the update adds the parts for itself, J times 256 bytes, and
// every column of Whole reads u and z again: what that costs grows with tiles x
// slots x columns, and past a bound it is more than the reduction's launch.
// Parts / Tiles (former kernels): two slots of 900 sites, 60 columns 15.0 / 17.7
// (20.4), 1440 sites, 300 columns 73.5 / 60.6 (62.6), FP32 60.3 / 43.7 (46.8);
// four of 450 sites, 60 columns 19.1 / 19.3, 1260 sites, FP32, 420 columns 109 /
// 79 (82); one of 1260 sites, 120 / 420 / 580 columns 17.3 / 18.1, 43.6 / 43.0,
// 59.7 / 55.9, of 2640 sites, 60 / 120 / 580 columns 19.4 / 20.0, 29.5 / 28.0,
// 124 / 101 (108).  In applies of one source the line lies higher, and higher for
// FP64: 400 columns, lines at 10000 / 18000: 2352 sites 16.36 / 16.19 ms, FP32 12.81 /
// 12.85, 1440 sites FP32 10.45 / 10.76.  Whole / Tiles, FP32: 8 slots of 256 sites, 60 / 120 / 420
// columns 15.2 / 17.4, 22.5 / 20.6, 57.5 / 49.2; FP64: 12 of 200 sites, 60 / 300 /
// 580 columns 22.3 / 23.4, 65.3 / 61.8, 139 / 124.
constexpr int kPartSlots = 4;
constexpr long long kPartWork = 5000, kPartWorkOne = 18000, kPartWorkOne32 = 10000;
constexpr long long kWholeWork = 20000, kWholeWork32 = 5000;
enum class DotForm { Whole, Parts, Tiles };
template <typename VT>
static DotForm dot_form(const KrylovWork& w, const KrylovArgs& A) {
  constexpr bool kF32 = sizeof(VT) == 8;
  const long long work = (long long)w.nrt_dot * A.nb, cols = work * (A.m + A.jmax());
  if (w.nrt_dot <= kParts)
    return work <= kPartTiles && cols <= (kF32 ? kWholeWork32 : kWholeWork) ? DotForm::Whole : DotForm::Tiles;
  const long long most = A.nb > 1 ? kPartWork : kF32 ? kPartWorkOne32 : kPartWorkOne;
  if (w.nrt_dot <= kPartTiles && A.nb <= kPartSlots && work <= 2 * kPartTiles && cols <= most) return DotForm::Parts;
  return DotForm::Tiles;
}

// 16-byte loads of row pairs of the FP32 columns (dot and update passes)
template <typename VT>
static void check_pairs(const KrylovArgs& A) {
  static_assert(kRpl % 2 == 0, "dot tiles hold whole row pairs");
  if (rows_per_lane<VT>() == 2) {
    SGN_REQUIRE(A.N % 2 == 0 && A.ldq % 2 == 0 && A.vstride % 2 == 0 && (reinterpret_cast<uintptr_t>(A.V) & 15) == 0,
                SGN_EINVAL, "krylov: FP32 basis needs an even row count and strides and a 16-byte aligned base");
  }
}

template <typename VT>
void krylov_dot(const KrylovWork& w, const KrylovArgs& Ain, bool with_z, bool reduce, hipStream_t s, Profiler* prof) {
  KrylovArgs A = Ain;
  krylov_bind(w, A);
  check_args(w, A);
  check_pairs<VT>(A);
  SGN_REQUIRE(krylov_tune_valid(A.tune), SGN_EINVAL, "krylov: invalid launch shape");
  const int kmax = A.jmax(), Jmax = A.m + kmax;
  const double vb = (double)sizeof(VT);
  double sm, sk;
  col_sums(A, sm, sk);
  const double qbytes = (double)A.N * (16.0 * sm + vb * sk);
  // per-slot work counts S for every slot
  const double cols = A.nb * (double)A.m + sk;
  // algorithmic bytes: Q, u, z read once; a, b written
  const double bytes = qbytes + A.nb * A.N * (16.0 + (with_z ? vb : 0.0)) + 32.0 * cols;
  const double flops = 16.0 * (double)A.N * cols;
  const DotForm form = dot_form<VT>(w, A);
  auto groups = [&](int width, int& ng) {
    ColGroups G{(A.m + width - 1) / width, width};
    ng = std::max(1, G.gs + (kmax + width - 1) / width);
    return G;
  };
  int ngroups = 0;
  if (form == DotForm::Whole) {
    const ColGroups G = groups(1, ngroups);
    const size_t nwg = (size_t)A.nb * ngroups;
    SGN_REQUIRE(nwg * 64 * w.nrt_dot < (size_t(1) << 32), SGN_EINVAL, "krylov: dot grid too large");
    prof_launch(prof, K_KDOT, bytes, flops, kdot_whole_kernel<VT, 1>, dim3((unsigned)nwg), dim3(64 * w.nrt_dot), 0, s,
                A, with_z ? 1 : 0, G);
    return;
  }
  const bool parts = form == DotForm::Parts;
  if (parts) {
    // several slots: two columns per workgroup, or one where two would leave the
    // chip short of wavefronts (1350 sites x 3, 150 columns: 45.4 us a step, 49.7
    // with columns one after another).  One slot: as many columns one after
    // another as leave it kDotWaves
    int C = 1, ng = 1;
    if (A.nb > 1) {
      if (A.tune.cpw > 1 && (size_t)w.nrt_dot * A.nb * ((Jmax + 1) / 2) >= kDotWavesBatch) C = 2;
    } else {
      while (2 * ng <= kPartWidth && (size_t)w.nrt_dot * (Jmax / (2 * ng)) >= kDotWaves) ng *= 2;
    }
    const ColGroups G = groups(C * ng, ngroups);
    const size_t nwg = (size_t)kParts * A.nb * ngroups;
    const int nw = (w.nrt_dot + kParts - 1) / kParts;
    SGN_REQUIRE(nwg * 64 * nw < (size_t(1) << 32), SGN_EINVAL, "krylov: dot grid too large");
    prof_launch(prof, K_KDOT, bytes, flops,
                C == 1 ? kdot_parts_kernel<VT, 1> : kdot_parts_kernel<VT, 2>,
                dim3((unsigned)nwg), dim3(64 * nw), 0, s, A, with_z ? 1 : 0, G, ng);
  } else {
    // columns whose loads a wavefront issues together, and batches of them per
    // wavefront.  8^4, 130 FP32 columns: 21.3 us with the reduction for two
    // columns by four batches, 22.5 for four by one, 26.4 for one by one (and
    // four by four as two by four); 8^4 x 6 slots, 130 FP64 columns: 123.8 for
    // two by two, 128.7 for two by four, 133.6 for one by one
    const int C = std::min(A.tune.cpw, 2), batches = sizeof(VT) == 16 ? 2 : 4;
    const ColGroups G = groups(4 * C * batches, ngroups);
    const size_t nwg = tile_grid((size_t)A.nb * ngroups, w.nrt_dot, A.N, false);
    SGN_REQUIRE(nwg * 256 < (size_t(1) << 32), SGN_EINVAL, "krylov: dot grid too large");
    prof_launch(prof, K_KDOT, bytes, flops, C == 1 ? kdot_kernel<VT, 1> : kdot_kernel<VT, 2>, dim3((unsigned)nwg),
                dim3(256), 0, s, A, with_z ? 1 : 0, G, batches, ngroups, kept_tiles<VT>(w, A));
  }
  if (parts && !reduce) return;
  // partial sums read, a, b written
  const double np = parts ? kParts : w.nrt_dot;
  prof_launch(prof, K_KRED, 32.0 * cols * (np + 1.0) + 32.0 * A.nb * w.nrt_dot, 4.0 * cols * np, kred_kernel,
              dim3(std::max(1, (Jmax + 31) / 32), 1, A.nb), dim3(256), 0, s, A, parts ? 1 : 0);
}

template <typename VT>
void krylov_update(const KrylovWork& w, const KrylovArgs& Ain, hipStream_t s, Profiler* prof) {
  KrylovArgs A = Ain;
  krylov_bind(w, A);
  check_args(w, A);
  SGN_REQUIRE(A.m + A.jmax() + 1 <= A.ldh, SGN_EINVAL, "krylov: H too small");
  SGN_REQUIRE(krylov_tune_valid(A.tune), SGN_EINVAL, "krylov: invalid launch shape");
  // Hessenberg-row workgroups for rows 0..m+jmax of every slot, then the
  // blocks of 64 R rows by row tile
  const int Jmax = A.m + A.jmax();
  const int nh = (Jmax + 1 + A.tune.uw - 1) / A.tune.uw;
  check_pairs<VT>(A);
  const unsigned nhess = ((unsigned)nh * A.nb + kXcds - 1) / kXcds * kXcds;
  const bool parts = dot_form<VT>(w, A) == DotForm::Parts;
  const size_t nwg = nhess + tile_grid((size_t)A.nb * (kDRows / (64 * rows_per_lane<VT>())), w.nrt_dot, A.N, parts);
  const int nthr = 64 * A.tune.uw;
  SGN_REQUIRE(nwg * nthr < (size_t(1) << 32), SGN_EINVAL, "krylov: update grid too large");
  const double vb = (double)sizeof(VT);
  double sm, sk;
  col_sums(A, sm, sk);
  const double qbytes = (double)A.N * (16.0 * sm + vb * sk);
  // read Q, u, z; write v_J, u' (+ its low-precision copy)
  const double vec = A.N * (16.0 + vb + vb + 16.0 + (A.ulonext ? vb : 0.0));
  const double cols = A.nb * (double)A.m + sk;  // per-slot work counts S for every slot
  const uint32_t lds = parts ? (uint32_t)(2 * sizeof(double2)) * (uint32_t)(std::min(Jmax, kCoefCap) + kCoefPad) : 0;
  prof_launch(prof, K_KUPDATE, qbytes + A.nb * vec + 32.0 * cols, 16.0 * (double)A.N * cols,
              parts ? update_kernel_for<VT, true>(A.tune) : update_kernel_for<VT, false>(A.tune), dim3((unsigned)nwg),
              dim3(nthr), lds, s, A, nh, nhess, kept_tiles<VT>(w, A));
}

template <typename VT>
void krylov_combine(const KrylovWork& w, const KrylovArgs& Ain, const double2* coef, int cstride, double2* y,
                    size_t ystride, int ncol, hipStream_t s, Profiler* prof) {
  KrylovArgs A = Ain;
  krylov_bind(w, A);
  check_args(w, A);
  SGN_REQUIRE(ncol >= 0 && ncol <= w.ncol_cap, SGN_EINVAL, "krylov: ncol exceeds workspace");
  const double vb = (double)sizeof(VT);
  const int nm = std::min(ncol, A.m);
  prof_launch(prof, K_KCOMBINE, (double)A.N * (16.0 * nm + A.nb * (vb * (ncol - nm) + 16.0)),
              A.nb * 8.0 * (double)A.N * ncol, kcombine_kernel<VT>, dim3((A.N + 63) / 64, 1, A.nb), dim3(kUThreads),
              0, s, A, coef, cstride, y, ystride, ncol);
}

void krylov_set_index(int* p, int v, bool add, hipStream_t s) {
  hipLaunchKernelGGL(set_index_kernel, dim3(1), dim3(64), 0, s, p, v, add ? 1 : 0);
  SGN_HIP(hipGetLastError());
}

void krylov_patch(const KrylovWork& w, const KrylovArgs& Ain, int n, double2* dst, size_t dstride, bool with_a,
                  hipStream_t s) {
  KrylovArgs A = Ain;
  krylov_bind(w, A);
  check_args(w, A);
  const size_t tot = (size_t)n * n;
  if (tot == 0) return;
  hipLaunchKernelGGL(kpatch_kernel, dim3((unsigned)((tot + 255) / 256), 1, A.nb), dim3(256), 0, s, A, n, dst,
                     dstride, with_a ? 1 : 0);
  SGN_HIP(hipGetLastError());
}

template void krylov_dot<double2>(const KrylovWork&, const KrylovArgs&, bool, bool, hipStream_t, Profiler*);
template void krylov_dot<float2>(const KrylovWork&, const KrylovArgs&, bool, bool, hipStream_t, Profiler*);
template void krylov_update<double2>(const KrylovWork&, const KrylovArgs&, hipStream_t, Profiler*);
template void krylov_update<float2>(const KrylovWork&, const KrylovArgs&, hipStream_t, Profiler*);
template void krylov_combine<double2>(const KrylovWork&, const KrylovArgs&, const double2*, int, double2*, size_t,
                                      int, hipStream_t, Profiler*);
template void krylov_combine<float2>(const KrylovWork&, const KrylovArgs&, const double2*, int, double2*, size_t, int,
                                     hipStream_t, Profiler*);
