// Wilson-Dirac stencil H_w(mu) = gamma5 D_w(mu) (Eq. Dw, Section 2) for gfx950.
//
// Internal layout (structure of arrays, one coalesced stream per component):
//   spinor  v[c * V + n],        c = 3 spin + colour, n = site index
//   links   U[(nu * 6 + 3 row + col) * V + n],  rows 0 and 1 only
// so that the 64 lanes of a wavefront, which own 64 consecutive sites, read
// every component with one fully coalesced 1 KiB load.  Neighbour spinors
// (8 per site) are re-read through L2 / MALL; each link is used by two sites.
// A link is an SU(3) matrix, so its third row is the complex conjugate of
// the cross product of the first two (unitarity and det U = 1; sgn_create
// checks both): the stencil stores 12 of the 18 reals and rebuilds the third
// row in registers, 24 instead of 36 link entries per site (the stencil's
// bytes fall from 60 to 48 complex numbers per site).  The antiperiodic time
// boundary is then a sign on the hops that cross it (folded into the link it
// would change the determinant); kappa and e^{+-mu} stay scalars.
//
// Spin structure (chiral basis): (1 +- gamma_nu) has rank 2, so each hop
// projects the 4-spinor onto a 2-spinor ("half spinor"), multiplies the two
// colour vectors by the link, and reconstructs the lower two spin components
// from the upper two.  In the chiral basis, with psi = (p0,p1,p2,p3):
//   (1 + g1): h = (p0 - i p3, p1 - i p2),   lower = ( i h1,  i h0)
//   (1 + g2): h = (p0 - p3,   p1 + p2),     lower = ( h1,   -h0)
//   (1 + g3): h = (p0 - i p2, p1 + i p3),   lower = ( i h0, -i h1)
//   (1 + g4): h = (p0 + p2,   p1 + p3),     lower = ( h0,    h1)
// and (1 - g_nu) flips the sign of every gamma term (lower = -(same map)).
#include <initializer_list>

#include "internal.h"

namespace {

// complex helpers generic over double2 / float2
template <typename C> struct Real;
template <> struct Real<double2> { using type = double; };
template <> struct Real<float2> { using type = float; };
template <typename C>
__device__ inline C mk(typename Real<C>::type x, typename Real<C>::type y) {
  C c;
  c.x = x;
  c.y = y;
  return c;
}
template <typename C> __device__ inline C tadd(C a, C b) { return mk<C>(a.x + b.x, a.y + b.y); }
template <typename C> __device__ inline C tsub(C a, C b) { return mk<C>(a.x - b.x, a.y - b.y); }
template <typename C> __device__ inline C tscale(C a, typename Real<C>::type s) { return mk<C>(a.x * s, a.y * s); }
template <typename C> __device__ inline C tmul(C a, C b) { return mk<C>(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); }
template <typename C> __device__ inline C tfma(C a, C b, C acc) {
  return mk<C>(acc.x + a.x * b.x - a.y * b.y, acc.y + a.x * b.y + a.y * b.x);
}
// Spin projection of (1 + gamma_nu) in the chiral basis, one colour vector
// su = 0, 1 of the half spinor at a time:
//   h_su = p_su + a p[partner],  lower component 2 + li = b chi_su  (chi = U h),
// with a, b in {+-1, +-i} as (re, im) pairs; (1 - gamma_nu) negates a and b.
// Computed rather than looked up: a switch over nu or a table in memory would
// put branches or another wait before the first loads.
struct SpinProj {
  int partner, li, ar, ai, br, bi;
};

__device__ inline SpinProj spin_proj(int nu, int su) {
  const bool odd = nu & 1;
  SpinProj P;
  P.partner = nu < 2 ? 3 - su : 2 + su;
  P.li = nu < 2 ? 1 - su : su;
  const int re_a = su == 0 && nu == 1 ? -1 : 1, im_a = su == 1 && nu == 2 ? 1 : -1;
  const int re_b = P.li == 1 && nu == 1 ? -1 : 1, im_b = P.li == 1 && nu == 2 ? -1 : 1;
  P.ar = odd ? re_a : 0;
  P.ai = odd ? 0 : im_a;
  P.br = odd ? re_b : 0;
  P.bi = odd ? 0 : im_b;
  return P;
}

constexpr int kLinkRows = 2;               // rows of an SU(3) link held in memory
constexpr int kLinkEntries = 3 * kLinkRows;  // complex entries per link and site

// the link of site ls in direction nu: rows 0 and 1 from memory, row 2 =
// conj(row 0 x row 1)
template <typename C>
__device__ inline void load_link(const C* __restrict__ links, int V, int nu, int ls, C u[9]) {
  const C* __restrict__ lp = links + (size_t)nu * kLinkEntries * V;
#pragma unroll
  for (int e = 0; e < kLinkEntries; ++e) u[e] = lp[(size_t)e * V + ls];
  // cross product of the first two rows, conjugated
  const C c0 = tsub(tmul(u[1], u[5]), tmul(u[2], u[4]));
  const C c1 = tsub(tmul(u[2], u[3]), tmul(u[0], u[5]));
  const C c2 = tsub(tmul(u[0], u[4]), tmul(u[1], u[3]));
  u[6] = mk<C>(c0.x, -c0.y);
  u[7] = mk<C>(c1.x, -c1.y);
  u[8] = mk<C>(c2.x, -c2.y);
}

// Quotient by a divisor fixed per launch: q = n / d for 0 <= n < 2^31 as one
// high multiplication, M = ceil(2^(31 + s) / d) with 2^(s-1) < d <= 2^s (the
// error n (M d - 2^(31+s)) / (d 2^(31+s)) stays below 1 / d).  The compiler's
// division by a runtime value is a chain of about 25 instructions, and the
// site's coordinates take three of them before the first load can issue.
struct FastDiv {
  unsigned m = 0, s = 0;  // s = 0: d = 1
  __host__ static FastDiv make(int d) {
    FastDiv f;
    while ((1ll << f.s) < d) ++f.s;
    f.m = (unsigned)(((1ull << (31 + f.s)) + (unsigned long long)d - 1) / (unsigned long long)d);
    return f;
  }
  __device__ inline int div(int n) const {
    const unsigned h = __umulhi((unsigned)n, m);
    return s ? (int)(h >> (s - 1)) : n;
  }
};

// Workgroup b runs on XCD b mod 8, each XCD with its own L2.  Renumber the
// blocks so that XCD x works through one contiguous range of sites (about
// 1/8 of the lattice): the neighbour spinors and backward-hop links a block
// reads were then mostly fetched into the same L2 by the blocks just before
// it.  A bijection on [0, nblk).
constexpr int kXcds = 8;
constexpr int kSiteGroup = 32;  // the walk blocks are segments of this many sites
__device__ inline int xcd_block(unsigned b, unsigned nblk) {
  const int x = b % kXcds, i = b / kXcds, q = nblk / kXcds, r = nblk % kXcds;
  return x * q + min(x, r) + i;
}

// Order in which the workgroups (lexicographically consecutive sites each)
// visit the lattice.  Lexicographic order puts the t-neighbours of a site a
// whole time slice of work away, beyond L2 on large lattices.  The blocked
// order walks 4D blocks of Lx x By x Bz x Bt sites (inside a block: segments
// of By rows, then z, then t; the blocks with t fastest), so every neighbour
// of a site is touched within about Lx By Bz sites of work.
// on = 0: lexicographic (lattices the blocks do not tile, or too small to care).
struct SiteOrder {
  int on = 0;
  int By = 1, Bz = 1, Bt = 1;
  int wpb = 1;  // workgroups per block
  FastDiv dwpb, dseg, dsegz, dntb, dnyz;  // by wpb, segw, segw Bz, Lt / Bt, (Lt / Bt)(Lz / Bz)
  int segw = 1, ntb = 1, nzb = 1;         // workgroups per segment, blocks in t and z
};

// first site of logical workgroup w
__device__ inline int order_site(int w, const SiteOrder& o, int Lx, int Ly, int Lz, int sites_per_wg) {
  if (!o.on) return w * sites_per_wg;
  const int blk = o.dwpb.div(w), in = w - blk * o.wpb;
  const int i1 = o.dseg.div(in), ti = o.dsegz.div(in);
  const int seg = in - i1 * o.segw, zi = i1 - ti * o.Bz;
  const int b1 = o.dntb.div(blk), yb = o.dnyz.div(blk);
  const int tb = blk - b1 * o.ntb, zb = b1 - yb * o.nzb;
  const int t = tb * o.Bt + ti, z = zb * o.Bz + zi, y0 = yb * o.By;
  return ((t * Lz + z) * Ly + y0) * Lx + seg * sites_per_wg;
}

// lattice extents and strides with the quotients the site coordinates need
// (indexed by the direction; nblk: workgroups per right-hand side)
struct Geom {
  int L[4], stride[4];
  FastDiv div[4];  // by stride[nu]
  int V, nblk;
  double kappa, emu, emmu;
};

// value of lane l % 32 (lo: the forward hop) and of lane 32 + l % 32 (hi: the
// backward hop) in every lane l
template <typename R>
struct Halves {
  R lo, hi;
};
__device__ inline Halves<float> halves(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return {__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ inline Halves<double> halves(double v) {
  const unsigned l = (unsigned)__double2loint(v), h = (unsigned)__double2hiint(v);
  const auto rl = __builtin_amdgcn_permlane32_swap(l, l, false, false);
  const auto rh = __builtin_amdgcn_permlane32_swap(h, h, false, false);
  return {__hiloint2double((int)rh[0], (int)rl[0]), __hiloint2double((int)rh[1], (int)rl[1])};
}

// Out_r = H_w(mu) In_r.  A workgroup holds S sites and four wavefronts,
// wavefront nu taking direction nu for all S sites: lanes 0..31 the forward
// hop, lanes 32..63 the backward hop.  With S = 32 a lane forms both colour
// vectors of its hop's half spinor; with S = 16 lanes l and l + 16 of a half
// form one each (12 instead of 18 operand loads per lane and twice the
// workgroups).  The direction, its link array, spin projector and phase are
// uniform over the wavefront; the backward lanes turn U_{m,nu} into
// U_{m,nu}^dag with selects, so both halves run one instruction stream.  A
// lane-half swap gives every lane both hops: the first half writes the upper
// spin components fwd + bwd, the second the lower ones, b_nu (fwd - bwd); the
// four directions meet in LDS and are summed in direction order.  Every
// component's arithmetic is the same for either S.  The site's own spinor
// entries for the second phase are loaded with the hop operands, so a
// workgroup waits on memory once.
// blockIdx.y = right-hand side (slot map).  Optional: scale = *inv_beta on
// input and output, copy_out = In * scale; with TERMS 1, Out_r = ca H_w In_r +
// cb Prev_r (Prev_r = prev + slot pstride; prev null: cb ignored), a step of
// a three-term recurrence in H_w; with TERMS 2, Out_r = ca (H_w In_r + cb
// Prev_r) + cc Prev2_r (prev2 null: cc ignored), one in H_w^2 with In = H_w
// Prev.  The terms come with the stencil's own operands, so a step of the
// recurrence in H_w^2 takes two launches (6^4: 3.8 and 3.9 us; a third one that
// adds the terms took 2.4, and the deflation setup of m = 20 121 instead of 101
// ms).
// ABI: in and out are in the interface layout (component 12 n + c).  A
// site's 12 entries are then contiguous, so the wavefront reads its neighbour
// sites' entries in that order and turns them through LDS.
//
// Small lattices are bound by the chain of dependent steps (an empty kernel
// takes 2.45 us back to back): 6^4 takes 3.4 us with S = 16, 3.9 with S = 32
// (5.1 with divisions, a switch over nu and both hops' twelve components
// through the shuffles).  Large ones are bound by memory: 32^4, 0.81 GB of
// operands, by events in applies 235 us = 3.4 TB/s with S = 32, 280 us with S =
// 16 (241 us before), and in sgn_matvec 264 us in the interface layout with S =
// 16 (287 us with S = 32, whose 53 KB of LDS leave two wavefronts per SIMD
// less); packing, applying (251 us) and unpacking took 415 us.
// the terms that a launch adds to ca H_w In
template <typename C>
struct Terms {
  const C *prev = nullptr, *prev2 = nullptr;
  size_t pstride = 0;  // slot stride of both
  double ca = 1.0, cb = 0.0, cc = 0.0;
};

template <typename C, int S, int TERMS, bool ABI>
__global__ void __launch_bounds__(256)
wilson_hw_dir_kernel(const C* __restrict__ links, const C* __restrict__ in, size_t istride, C* __restrict__ out,
                     size_t ostride, const double* __restrict__ inv_beta, C* __restrict__ copy_out, Geom g,
                     SlotMap map, SiteOrder order, Terms<C> terms) {
  using R = typename Real<C>::type;
  static_assert(S == 32 || S == 16, "sites per workgroup");
  constexpr int kThreads = 256, kOut = 12 * S;
  constexpr int kRounds = (kOut + kThreads - 1) / kThreads;
  constexpr int NH = S / 16;  // colour vectors per lane
  constexpr int kPad = ABI ? 13 : S;  // LDS row: one site's components (ABI), else one component's sites
  const int V = g.V;
  const int lane = threadIdx.x & 63;
  const int nu = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int sl = lane & (S - 1);
  const int hs = (lane >> 4) & 1;  // S = 16: this lane's colour vector
  const bool fwd = lane < 32;
  const int slot = map.slot[blockIdx.y];
  const int n0 = order_site(xcd_block(blockIdx.x, g.nblk), order, g.L[0], g.L[1], g.L[2], S);
  const int n = n0 + sl;
  const int nc = n < V ? n : V - 1;  // lanes past the lattice work on a valid site, never written out
  const C* __restrict__ v = in + (size_t)slot * istride;
  // the coordinate along nu: n / stride_nu mod L_nu, from the next direction's quotient
  const int Lnu = g.L[nu], stride = g.stride[nu];
  const int q0 = g.div[nu].div(nc), q1 = nu == 3 ? 0 : g.div[(nu + 1) & 3].div(nc);
  const int coord = q0 - q1 * Lnu;
  // neighbour along the hop, periodic wrap
  const bool wrap = coord == (fwd ? Lnu - 1 : 0);
  const int m = nc + (fwd ? stride : -stride) * (wrap ? 1 - Lnu : 1);
  const int ls = fwd ? nc : m;  // site that owns the link
  // spinor entries of the hop: colour vector su needs spins su and its partner
  C pu[NH][3], pl[NH][3];
  // the partial sums of direction k at smem[k kSlab]; before them (ABI) that
  // wavefront's neighbour entries in the same place
  constexpr int kSlab = ABI ? 2 * S * kPad : 12 * S;
  __shared__ C smem[4 * kSlab];
  if constexpr (ABI) {
    // entry e of the wavefront's 2 S neighbour sites: site e / 12, component e % 12
    C* const nbr = smem + nu * kSlab;
    constexpr int kEnt = 2 * S * 12 / 64;
    C ent[kEnt];
#pragma unroll
    for (int i = 0; i < kEnt; ++i) {
      const int e = i * 64 + lane, q = e / 12, comp = e - 12 * q;
      // sites 0..S-1: forward (lanes 0..S-1), S..2S-1: backward (lanes 32..)
      const int mq = __shfl(m, q < S ? q : 32 + q - S, 64);
      ent[i] = v[(size_t)mq * 12 + comp];
    }
#pragma unroll
    for (int i = 0; i < kEnt; ++i) {
      const int e = i * 64 + lane, q = e / 12, comp = e - 12 * q;
      nbr[q * kPad + comp] = ent[i];
    }
    __syncthreads();
    const C* row = nbr + ((fwd ? 0 : S) + sl) * kPad;
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      const int su = NH == 2 ? h : hs, lo = spin_proj(nu, su).partner;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        pu[h][c] = row[3 * su + c];
        pl[h][c] = row[3 * lo + c];
      }
    }
  } else {
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      const int su = NH == 2 ? h : hs, lo = spin_proj(nu, su).partner;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        pu[h][c] = v[(size_t)((3 * su + c) * V + m)];
        pl[h][c] = v[(size_t)((3 * lo + c) * V + m)];
      }
    }
  }
  C u[9];
  load_link<C>(links, V, nu, ls, u);
  // second-phase outputs of this thread: p = tid + q kThreads < kOut, i.e.
  // component p / S of site n0 + p % S (ABI: component p % 12 of site n0 + p / 12)
  C self[kRounds], pv[kRounds], pv2[kRounds];
  const C* __restrict__ pr = (TERMS > 0 && terms.prev) ? terms.prev + (size_t)slot * terms.pstride : nullptr;
  const C* __restrict__ pr2 = (TERMS > 1 && terms.prev2) ? terms.prev2 + (size_t)slot * terms.pstride : nullptr;
#pragma unroll
  for (int q = 0; q < kRounds; ++q) {
    const int p = threadIdx.x + q * kThreads, s2 = ABI ? p / 12 : p % S, nn = n0 + s2;
    const bool ok = p < kOut && nn < V;
    const size_t idx = ABI ? (size_t)n0 * 12 + p : (size_t)(p / S) * V + nn;
    self[q] = ok ? v[idx] : mk<C>(0, 0);
    // the recurrence's other terms, loaded with the operands (one wait)
    if constexpr (TERMS > 0) pv[q] = (ok && pr) ? pr[idx] : mk<C>(0, 0);
    if constexpr (TERMS > 1) pv2[q] = (ok && pr2) ? pr2[idx] : mk<C>(0, 0);
  }
  // the matrix applied to the half spinor: U (forward) or U^dag (backward)
  const R sg = fwd ? (R)1 : (R)-1;
  C w9[9];
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const C a = u[3 * r + c], b = u[3 * c + r];
      w9[3 * r + c] = fwd ? a : mk<C>(b.x, -b.y);
    }
  // e^{+-mu} on time hops, and the antiperiodic sign on the two hops across
  // the time boundary (forward from the last slice, backward from the first)
  const R phase = (nu == 3) ? (fwd ? (R)g.emu : (R)g.emmu) * (wrap ? (R)-1 : (R)1) : (R)1;
  C chi[NH][3];
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    // h = p_u + sg a p_l with a in {+-1, +-i}: the products are exact
    const SpinProj P = spin_proj(nu, NH == 2 ? h : hs);
    const R ar = sg * (R)P.ar, ai = sg * (R)P.ai;
    C hv[3];
#pragma unroll
    for (int c = 0; c < 3; ++c)
      hv[c] = mk<C>(fma(ar, pl[h][c].x, fma(-ai, pl[h][c].y, pu[h][c].x)),
                    fma(ar, pl[h][c].y, fma(ai, pl[h][c].x, pu[h][c].y)));
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      C s0 = mk<C>(0, 0);
#pragma unroll
      for (int c = 0; c < 3; ++c) s0 = tfma(w9[3 * r + c], hv[c], s0);
      chi[h][r] = tscale(s0, phase);
    }
  }
  // both hops in every lane: the first half of the lanes sums the upper
  // components, the second forms the lower ones: spin 2 + i is b_i chi[j_i]
  auto at = [&](int k, int comp, int site) -> C& {
    return smem[k * kSlab + (ABI ? site * kPad + comp : comp * S + site)];
  };
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    const int su = NH == 2 ? h : hs;
    const SpinProj P = spin_proj(nu, su);
    const R br = (R)P.br, bi = (R)P.bi;
    const int comp0 = 3 * (fwd ? su : 2 + P.li);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const auto hx = halves(chi[h][c].x), hy = halves(chi[h][c].y);
      const C f = mk<C>(hx.lo, hy.lo), b = mk<C>(hx.hi, hy.hi);
      const C d = tsub(f, b);
      const C up = tadd(f, b), low = mk<C>(br * d.x - bi * d.y, br * d.y + bi * d.x);
      // (a select of the parts: one of the structs would go through scratch)
      at(nu, comp0 + c, sl) = mk<C>(fwd ? up.x : low.x, fwd ? up.y : low.y);
    }
  }
  __syncthreads();
  const R kappa = (R)g.kappa;
  const R scale = inv_beta ? (R)(*inv_beta) : (R)1;
  C* __restrict__ w = out + (size_t)slot * ostride;
#pragma unroll
  for (int q = 0; q < kRounds; ++q) {
    const int p = threadIdx.x + q * kThreads;
    const int comp = ABI ? p % 12 : p / S, s2 = ABI ? p / 12 : p % S, nn = n0 + s2;
    if (p >= kOut || nn >= V) continue;
    C acc = mk<C>(0, 0);
#pragma unroll
    for (int k = 0; k < 4; ++k) acc = tadd(acc, at(k, comp, s2));
    const size_t idx = ABI ? (size_t)n0 * 12 + p : (size_t)comp * V + nn;
    // gamma5 (psi - kappa * hops), all times 1/beta
    const R g5 = comp < 6 ? (R)1 : (R)-1;
    C val = tscale(tsub(self[q], tscale(acc, kappa)), g5 * scale);
    if constexpr (TERMS == 1) {
      val = tscale(val, (R)terms.ca);
      if (pr) val = tadd(val, tscale(pv[q], (R)terms.cb));
    }
    if constexpr (TERMS == 2) {
      const R ca = (R)terms.ca, cb = (R)terms.cb, cc = (R)terms.cc;
      val = mk<C>(ca * fma(cb, pv[q].x, val.x), ca * fma(cb, pv[q].y, val.y));
      if (pr2) val = mk<C>(fma(cc, pv2[q].x, val.x), fma(cc, pv2[q].y, val.y));
    }
    w[idx] = val;
    if (copy_out) copy_out[idx] = tscale(self[q], scale);
  }
}

// Two applications in one launch, for lattices that leave most of the chip
// idle.  A launch of theirs is little more than the launch itself (2.45 us of
// the 3.7 that one application of 4^3 x 6 sites takes), so a workgroup owns
// four sites and nine wavefronts: wavefront 0 applies H_w at the sites
// themselves, wavefront 1 + 2 nu + d at their neighbours along +-nu (d = 0, 1),
// which makes the first application nine times over, and after one exchange
// through LDS wavefront 0 applies H_w again.  Lane = site (4) x direction (4) x
// hop (forward, backward) x colour vector of the half spinor (2).  Every sum
// has the operations and the order of wilson_hw_dir_kernel.
//   SQUARE: M = H_w In, Out = ca2 (H_w M + cb2 In) + cc Prev (M not written);
//   else:   Mid = ca1 H_w In + cb1 Prev, Out = ca2 H_w Mid + cb2 In;
// prev null: without its term.  One launch / two, us back to back: 4^4 4.6 /
// 6.4, 4^3 x 6 two slots 4.8 / 6.5.
template <bool SQUARE>
__global__ void __launch_bounds__(576)
wilson_pair_kernel(const double2* __restrict__ links, const double2* __restrict__ in, size_t istride,
                   double2* __restrict__ mid, size_t mstride, double2* __restrict__ out, size_t ostride,
                   const double2* __restrict__ prev, size_t pstride, Geom g, SlotMap map, double ca1, double cb1,
                   double ca2, double cb2, double cc) {
  using C = double2;
  __shared__ C chis[9][8][6][4];  // [wavefront][2 nu + hop][3 su + colour][site]
  __shared__ C mids[9][12][4];    // [wavefront][component][site]
  const int V = g.V;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int site = lane & 3, nu = (lane >> 2) & 3, hop = (lane >> 4) & 1, su = lane >> 5;
  const bool fwd = hop == 0;
  const int slot = map.slot[blockIdx.y];
  const int n0 = 4 * xcd_block(blockIdx.x, g.nblk) + site;
  const bool own = n0 < V;
  int n = own ? n0 : V - 1;  // lanes past the lattice work on a valid site, never written out
  int c0, c1, c2, c3;
  {
    const int q1 = g.div[1].div(n), q2 = g.div[2].div(n), q3 = g.div[3].div(n);
    c0 = n - q1 * g.L[0];
    c1 = q1 - q2 * g.L[1];
    c2 = q2 - q3 * g.L[2];
    c3 = q3;
  }
  // this wavefront's site: the own one, or its neighbour (periodic wrap)
  if (wave > 0) {
    const int d = (wave - 1) >> 1, step = (wave - 1) & 1 ? -1 : 1, L = g.L[d];
    const int c = d == 0 ? c0 : d == 1 ? c1 : d == 2 ? c2 : c3;
    const int cn = c + step < 0 ? L - 1 : c + step == L ? 0 : c + step;
    n += (cn - c) * g.stride[d];
    if (d == 0) c0 = cn;
    if (d == 1) c1 = cn;
    if (d == 2) c2 = cn;
    if (d == 3) c3 = cn;
  }
  const C* __restrict__ v = in + (size_t)slot * istride;
  const int coord = nu == 0 ? c0 : nu == 1 ? c1 : nu == 2 ? c2 : c3;
  const int L = nu == 0 ? g.L[0] : nu == 1 ? g.L[1] : nu == 2 ? g.L[2] : g.L[3];
  const int stride = nu == 0 ? 1 : nu == 1 ? g.stride[1] : nu == 2 ? g.stride[2] : g.stride[3];
  const bool wrap = coord == (fwd ? L - 1 : 0);
  const int m = n + (fwd ? stride : -stride) * (wrap ? 1 - L : 1);
  const SpinProj P = spin_proj(nu, su);
  C pu[3], pl[3], u[9];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    pu[c] = v[(size_t)(3 * su + c) * V + m];
    pl[c] = v[(size_t)(3 * P.partner + c) * V + m];
  }
  load_link<C>(links, V, nu, fwd ? n : m, u);
  // component lane / 4 of site lane % 4 (lanes below 48), for both sums
  const bool ok = lane < 48;
  const int comp = ok ? lane >> 2 : 0;
  const C self = v[(size_t)comp * V + n];
  C pv = mk<C>(0, 0);
  if (prev && (!SQUARE || wave == 0)) pv = prev[(size_t)slot * pstride + (size_t)comp * V + n];
  const double sg = fwd ? 1.0 : -1.0;
  C w9[9];
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const C a = u[3 * r + c], b = u[3 * c + r];
      w9[3 * r + c] = mk<C>(fwd ? a.x : b.x, fwd ? a.y : -b.y);
    }
  const double phase = nu == 3 ? (fwd ? g.emu : g.emmu) * (wrap ? -1.0 : 1.0) : 1.0;
  const double ar = sg * P.ar, ai = sg * P.ai;
  // this lane's colour vector of its hop into chis[w]
  auto hop_product = [&](const C (&x)[3], const C (&y)[3], int w) {
    C hv[3];
#pragma unroll
    for (int c = 0; c < 3; ++c)
      hv[c] = mk<C>(fma(ar, y[c].x, fma(-ai, y[c].y, x[c].x)), fma(ar, y[c].y, fma(ai, y[c].x, x[c].y)));
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      C s0 = mk<C>(0, 0);
#pragma unroll
      for (int c = 0; c < 3; ++c) s0 = tfma(w9[3 * r + c], hv[c], s0);
      chis[w][2 * nu + hop][3 * su + r][site] = tscale(s0, phase);
    }
  };
  // gamma5 (psi - kappa hops) of this lane's component
  auto apply = [&](C psi, int w) {
    const int i = comp / 3, c = comp - 3 * i;
    C acc = mk<C>(0, 0);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int s1 = i < 2 ? i : (k < 2 ? 3 - i : i - 2);  // the colour vector behind spin i
      const C f = chis[w][2 * k][3 * s1 + c][site], b = chis[w][2 * k + 1][3 * s1 + c][site];
      const SpinProj Q = spin_proj(k, s1);
      const double br = Q.br, bi = Q.bi;
      const C d = tsub(f, b), up = tadd(f, b), low = mk<C>(br * d.x - bi * d.y, br * d.y + bi * d.x);
      acc = tadd(acc, mk<C>(i < 2 ? up.x : low.x, i < 2 ? up.y : low.y));
    }
    return tscale(tsub(psi, tscale(acc, g.kappa)), comp < 6 ? 1.0 : -1.0);
  };
  hop_product(pu, pl, wave);
  __syncthreads();
  if (ok) {
    C val = apply(self, wave);
    if constexpr (!SQUARE) {
      val = tscale(val, ca1);
      if (prev) val = tadd(val, tscale(pv, cb1));
      if (wave == 0 && own) mid[(size_t)slot * mstride + (size_t)comp * V + n] = val;
    }
    mids[wave][comp][site] = val;
  }
  __syncthreads();
  if (wave == 0) {
    const int w = 1 + 2 * nu + hop;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      pu[c] = mids[w][3 * su + c][site];
      pl[c] = mids[w][3 * P.partner + c][site];
    }
    hop_product(pu, pl, 0);
  }
  __syncthreads();
  if (wave > 0 || !ok || !own) return;
  C val = apply(mids[0][comp][site], 0);
  if constexpr (SQUARE) {
    val = mk<C>(ca2 * fma(cb2, self.x, val.x), ca2 * fma(cb2, self.y, val.y));
    if (prev) val = mk<C>(fma(cc, pv.x, val.x), fma(cc, pv.y, val.y));
  } else {
    val = tadd(tscale(val, ca2), tscale(self, cb2));
  }
  out[(size_t)slot * ostride + (size_t)comp * V + n] = val;
}

__global__ void links_to_f32_kernel(const double2* __restrict__ a, float2* __restrict__ b, size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) b[i] = make_float2((float)a[i].x, (float)a[i].y);
}

// rows 0 and 1 of every link into the internal layout; bad = 1 if some link
// is not SU(3) to 1e-10 (|U U^dag - I|, |det U - 1|), since row 2 is rebuilt
__global__ void pack_links_kernel(const double2* __restrict__ g, double2* __restrict__ U, int V, int* bad) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= V) return;
  bool ok = true;
  for (int nu = 0; nu < 4; ++nu) {
    double2 a[9];
    for (int e = 0; e < 9; ++e) a[e] = g[((size_t)n * 4 + nu) * 9 + e];
    for (int e = 0; e < kLinkEntries; ++e) U[((size_t)nu * kLinkEntries + e) * V + n] = a[e];
    double dev = 0.0;
    for (int i = 0; i < 3; ++i)
      for (int j = 0; j < 3; ++j) {
        double2 acc = make_double2(0.0, 0.0);
        for (int k = 0; k < 3; ++k) acc = cfma(a[3 * i + k], make_double2(a[3 * j + k].x, -a[3 * j + k].y), acc);
        dev = fmax(dev, fabs(acc.x - (i == j ? 1.0 : 0.0)) + fabs(acc.y));
      }
    // det = row 2 . (row 0 x row 1)
    const double2 c0 = csub(cmul(a[1], a[5]), cmul(a[2], a[4]));
    const double2 c1 = csub(cmul(a[2], a[3]), cmul(a[0], a[5]));
    const double2 c2 = csub(cmul(a[0], a[4]), cmul(a[1], a[3]));
    const double2 det = cadd(cadd(cmul(a[6], c0), cmul(a[7], c1)), cmul(a[8], c2));
    dev = fmax(dev, fabs(det.x - 1.0) + fabs(det.y));
    if (!(dev <= 1e-10)) ok = false;
  }
  if (!ok) *bad = 1;
}

// threads run over the interface layout, so the reads are contiguous; the
// writes go to 12 streams (one per component), each contiguous across the
// lanes that share a component (as in unpack_kernel, the other way round)
__global__ void pack_kernel(const double2* __restrict__ x, double2* __restrict__ v, int V) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;  // ABI index 12 n + c
  if (i >= 12 * V) return;
  const int n = i / 12, c = i - 12 * n;
  v[(size_t)c * V + n] = x[i];
}

__global__ void unpack_kernel(const double2* __restrict__ v, double2* __restrict__ y, int V) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;  // ABI index 12 n + c
  if (i >= 12 * V) return;
  const int n = i / 12, c = i - 12 * n;
  y[i] = v[c * V + n];
}

}  // namespace

void wilson_pack_links(const Lattice& lat, const double2* gauge_abi, double2* links, int* bad, hipStream_t s) {
  const int V = lat.V;
  hipLaunchKernelGGL(pack_links_kernel, dim3((V + 255) / 256), dim3(256), 0, s, gauge_abi, links, V, bad);
  SGN_HIP(hipGetLastError());
}

size_t wilson_link_entries(int V) { return (size_t)4 * kLinkEntries * V; }

void wilson_pack(const Lattice& lat, const double2* x_abi, double2* v, hipStream_t s) {
  const int n = 12 * lat.V;
  hipLaunchKernelGGL(pack_kernel, dim3((n + 255) / 256), dim3(256), 0, s, x_abi, v, lat.V);
  SGN_HIP(hipGetLastError());
}

void wilson_unpack(const Lattice& lat, const double2* v, double2* y_abi, hipStream_t s) {
  const int n = 12 * lat.V;
  hipLaunchKernelGGL(unpack_kernel, dim3((n + 255) / 256), dim3(256), 0, s, v, y_abi, lat.V);
  SGN_HIP(hipGetLastError());
}

// y = x + gamma5 y in the interface layout (component 12 n + 3 spin + colour;
// gamma5 = diag(1, 1, -1, -1) in spin): the last step of D_ov(mu) x
__global__ void overlap_finish_kernel(const double2* __restrict__ x, double2* __restrict__ y, size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double2 xi = x[i], si = y[i];
  y[i] = (i % 12 < 6) ? make_double2(xi.x + si.x, xi.y + si.y) : make_double2(xi.x - si.x, xi.y - si.y);
}

void overlap_finish(const double2* x, double2* y, size_t n, hipStream_t s) {
  if (n == 0) return;
  hipLaunchKernelGGL(overlap_finish_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, x, y, n);
  SGN_HIP(hipGetLastError());
}

// the adjoint D_ov(mu)^dag x = x + sgn(H_w(mu))^dag gamma5 x, in the interface
// layout: y = gamma5 x before the sign, y = x + y after it
__global__ void gamma5_abi_kernel(const double2* __restrict__ x, double2* __restrict__ y, size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double2 xi = x[i];
  y[i] = (i % 12 < 6) ? xi : make_double2(-xi.x, -xi.y);
}

__global__ void add_abi_kernel(const double2* __restrict__ x, double2* __restrict__ y, size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double2 xi = x[i], si = y[i];
  y[i] = make_double2(xi.x + si.x, xi.y + si.y);
}

// y = a x + b g y, g = gamma5 (if g5) or 1, in the interface layout; x may be y
__global__ void axpby_abi_kernel(const double2* x, double2* y, double a, double b, int g5, size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double2 xi = x[i], yi = y[i];
  const double bb = (g5 && i % 12 >= 6) ? -b : b;
  y[i] = make_double2(a * xi.x + bb * yi.x, a * xi.y + bb * yi.y);
}

void axpby_abi(const double2* x, double2* y, double a, double b, bool g5, size_t n, hipStream_t s) {
  if (n == 0) return;
  hipLaunchKernelGGL(axpby_abi_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, x, y, a, b, g5 ? 1 : 0,
                     n);
  SGN_HIP(hipGetLastError());
}

void overlap_adjoint_start(const double2* x, double2* y, size_t n, hipStream_t s) {
  if (n == 0) return;
  hipLaunchKernelGGL(gamma5_abi_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, x, y, n);
  SGN_HIP(hipGetLastError());
}

void overlap_adjoint_finish(const double2* x, double2* y, size_t n, hipStream_t s) {
  if (n == 0) return;
  hipLaunchKernelGGL(add_abi_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, x, y, n);
  SGN_HIP(hipGetLastError());
}

// the blocked order when the lattice is large enough to leave L2 and its
// extents admit the blocks (Lx By a multiple of kSiteGroup); spw: sites per
// workgroup, a divisor of kSiteGroup
static SiteOrder site_order(const Lattice& lat, int spw) {
  SiteOrder o;
  const int Lx = lat.L[0], Ly = lat.L[1], Lz = lat.L[2], Lt = lat.L[3];
  if (lat.blk[0] < 0) return o;
  if (lat.blk[0] > 0) {  // set by sgn_set_stencil_blocks (validated there)
    o.By = lat.blk[0];
    o.Bz = lat.blk[1];
    o.Bt = lat.blk[2];
  } else {
    if (lat.V < 65536) return o;
    // preferred extents first (at 32^4, Lx x 4 x 16 x 4 walked 6 % faster than
    // Lx x 8 x 8 x 4 and 14 % faster than the natural order)
    auto pick = [](int L, std::initializer_list<int> pref, auto ok) {
      for (int b : pref)
        if (L % b == 0 && ok(b)) return b;
      return 0;
    };
    o.By = pick(Ly, {4, 8, 2, 16, 1}, [&](int b) { return (Lx * b) % kSiteGroup == 0; });
    o.Bz = pick(Lz, {16, 8, 4, 2, 1}, [](int) { return true; });
    o.Bt = pick(Lt, {4, 8, 2, 1}, [](int) { return true; });
    if (o.By == 0 || o.Bz == 0 || o.Bt == 0) return SiteOrder{};
  }
  o.segw = Lx * o.By / spw;
  o.wpb = o.segw * o.Bz * o.Bt;
  o.ntb = Lt / o.Bt;
  o.nzb = Lz / o.Bz;
  o.dwpb = FastDiv::make(o.wpb);
  o.dseg = FastDiv::make(o.segw);
  o.dsegz = FastDiv::make(o.segw * o.Bz);
  o.dntb = FastDiv::make(o.ntb);
  o.dnyz = FastDiv::make(o.ntb * o.nzb);
  o.on = 1;
  return o;
}

static Geom geom(const Lattice& lat, int nblk) {
  Geom g{};
  int st = 1;
  for (int nu = 0; nu < 4; ++nu) {
    g.L[nu] = lat.L[nu];
    g.stride[nu] = st;
    g.div[nu] = FastDiv::make(st);
    st *= lat.L[nu];
  }
  g.V = lat.V;
  g.nblk = nblk;
  g.kappa = lat.kappa;
  g.emu = lat.emu;
  g.emmu = lat.emmu;
  return g;
}

bool wilson_blocks_valid(const Lattice& lat, int By, int Bz, int Bt) {
  if (By == 0 && Bz == 0 && Bt == 0) return true;
  if (By < 0) return Bz <= 0 && Bt <= 0;
  return By >= 1 && Bz >= 1 && Bt >= 1 && lat.L[1] % By == 0 && lat.L[2] % Bz == 0 && lat.L[3] % Bt == 0 &&
         (lat.L[0] * By) % kSiteGroup == 0;
}

// One launch of the stencil for the slots of map.  The site split S by the
// number of 32-site workgroups: below two per CU the chip is short of
// workgroups and 16 sites are faster (6^4 x 8 slots, 328 of them: 5.7 against
// 6.1 us; 8^4 x 3, 384: 5.6 against 6.0), above it the link loads that the two
// lanes of a site repeat cost more (12^4, 648: 7.4 against 7.2 us; 8^4 x 8,
// 1024: 9.3 against 8.9).
constexpr long long kSplitBelow = 512;

template <typename C, int S, int TERMS, bool ABI>
static void hw_launch_as(const Lattice& lat, const C* links, const C* in, size_t istride, C* out, size_t ostride,
                         const double* inv_beta, C* copy_out, const SlotMap& map, const Terms<C>& terms, double bytes,
                         hipStream_t s, Profiler* prof) {
  const int nblk = (lat.V + S - 1) / S;
  prof_launch(prof, K_WILSON, bytes, 1392.0 * lat.V * map.n, wilson_hw_dir_kernel<C, S, TERMS, ABI>,
              dim3(nblk, map.n), dim3(256), 0, s, links, in, istride, out, ostride, inv_beta, copy_out,
              geom(lat, nblk), map, site_order(lat, S), terms);
}

template <typename C, int TERMS>
static void hw_launch(const Lattice& lat, const C* links, const C* in, size_t istride, C* out, size_t ostride,
                      const double* inv_beta, C* copy_out, const SlotMap& map, const Terms<C>& terms, double bytes,
                      hipStream_t s, Profiler* prof) {
  const bool fine = (long long)((lat.V + 31) / 32) * map.n < kSplitBelow;
  (fine ? hw_launch_as<C, 16, TERMS, false> : hw_launch_as<C, 32, TERMS, false>)(
      lat, links, in, istride, out, ostride, inv_beta, copy_out, map, terms, bytes, s, prof);
}

static SlotMap one_slot() {
  SlotMap m;
  m.n = 1;
  return m;
}

void wilson_apply(const Lattice& lat, const double2* links, const double2* in, double2* out,
                  const double* inv_beta, double2* copy_out, hipStream_t s, Profiler* prof) {
  // algorithmic bytes: read v (12), write w (12), 4 links of 6 stored entries
  // (24) per site; + copy (12)
  const double per_site = (48.0 + (copy_out ? 12.0 : 0.0)) * 16.0;
  hw_launch<double2, 0>(lat, links, in, 0, out, 0, inv_beta, copy_out, one_slot(), Terms<double2>{},
                        per_site * lat.V, s, prof);
}

void wilson_apply32(const Lattice& lat, const float2* links, const float2* in, float2* out, hipStream_t s,
                    Profiler* prof) {
  hw_launch<float2, 0>(lat, links, in, 0, out, 0, nullptr, nullptr, one_slot(), Terms<float2>{}, 48.0 * 8.0 * lat.V,
                       s, prof);
}

void wilson_apply_abi(const Lattice& lat, const double2* links, const double2* x, double2* y, hipStream_t s,
                      Profiler* prof) {
  hw_launch_as<double2, 16, 0, true>(lat, links, x, 0, y, 0, nullptr, nullptr, one_slot(), Terms<double2>{},
                                     48.0 * 16.0 * lat.V, s, prof);
}

// Lattices and slots whose pairs of applications take one launch: those with
// one of its workgroups (four sites) per CU or less.  A second one on a CU
// costs more than the launch saved: 4^4 x 4 slots, 256 workgroups, 4.9 us (two
// launches 6.5), 6^4, 324, 7.7 us (6.5).
constexpr long long kPairWgs = 256;
bool wilson_pairs(const Lattice& lat, int slots) { return (long long)((lat.V + 3) / 4) * slots <= kPairWgs; }

template <bool SQUARE>
static void pair_launch(const Lattice& lat, const double2* links, const double2* in, size_t istride, double2* mid,
                        size_t mstride, double2* out, size_t ostride, const double2* prev, size_t pstride,
                        const SlotMap& map, double ca1, double cb1, double ca2, double cb2, double cc, hipStream_t s,
                        Profiler* prof) {
  const int nblk = (lat.V + 3) / 4;
  // per site: the links once, per slot read the input and prev, write the results
  const double bytes = (24.0 + ((SQUARE ? 24.0 : 36.0) + (prev ? 12.0 : 0.0)) * map.n) * 16.0 * lat.V;
  prof_launch(prof, K_WILSON, bytes, 2.0 * 1392.0 * lat.V * map.n, wilson_pair_kernel<SQUARE>, dim3(nblk, map.n),
              dim3(576), 0, s, links, in, istride, mid, mstride, out, ostride, prev, pstride, geom(lat, nblk), map, ca1,
              cb1, ca2, cb2, cc);
}

void wilson_apply_cheb_pair(const Lattice& lat, const double2* links, const double2* in, size_t istride, double2* mid,
                            size_t mstride, double2* out, size_t ostride, const double2* prev, size_t pstride,
                            double ca1, double cb1, double ca2, double cb2, const SlotMap& map, hipStream_t s,
                            Profiler* prof) {
  SGN_REQUIRE(map.n >= 1 && map.n <= kMaxBatch, SGN_EINVAL, "wilson: slot map must hold 1..64 slots");
  pair_launch<false>(lat, links, in, istride, mid, mstride, out, ostride, prev, pstride, map, ca1, cb1, ca2, cb2, 0.0,
                     s, prof);
}

void wilson_apply_cheb_slots(const Lattice& lat, const double2* links, const double2* in, size_t istride,
                             double2* out, size_t ostride, const double2* prev, size_t pstride, double ca, double cb,
                             const SlotMap& map, hipStream_t s, Profiler* prof) {
  SGN_REQUIRE(map.n >= 1 && map.n <= kMaxBatch, SGN_EINVAL, "wilson: slot map must hold 1..64 slots");
  // per site: the links (24 stored entries) once, per slot read v and
  // prev, write w (12 each)
  const double bytes = (24.0 + (24.0 + (prev ? 12.0 : 0.0)) * map.n) * 16.0 * lat.V;
  Terms<double2> t;
  t.prev = prev;
  t.pstride = pstride;
  t.ca = ca;
  t.cb = cb;
  hw_launch<double2, 1>(lat, links, in, istride, out, ostride, nullptr, nullptr, map, t, bytes, s, prof);
}

void wilson_apply_square(const Lattice& lat, const double2* links, const double2* y, double2* tmp, double2* out,
                         double a, double c, double b, const double2* yp, hipStream_t s, Profiler* prof) {
  if (wilson_pairs(lat, 1)) {
    pair_launch<true>(lat, links, y, 0, nullptr, 0, out, 0, yp, 0, one_slot(), 1.0, 0.0, a, -c, -b, s, prof);
    return;
  }
  wilson_apply(lat, links, y, tmp, nullptr, nullptr, s, prof);
  Terms<double2> t;
  t.prev = y;
  t.prev2 = yp;
  t.ca = a;
  t.cb = -c;
  t.cc = -b;
  const double per_site = (60.0 + (yp ? 12.0 : 0.0)) * 16.0;
  hw_launch<double2, 2>(lat, links, tmp, 0, out, 0, nullptr, nullptr, one_slot(), t, per_site * lat.V, s, prof);
}

template <typename C>
void wilson_apply_slots(const Lattice& lat, const C* links, const C* in, size_t istride, C* out, size_t ostride,
                        const SlotMap& map, hipStream_t s, Profiler* prof) {
  SGN_REQUIRE(map.n >= 1 && map.n <= kMaxBatch, SGN_EINVAL, "wilson: slot map must hold 1..64 slots");
  // per site: the links (24 stored entries) once, per slot read v (12) and write w (12)
  const double b = (double)sizeof(C);
  hw_launch<C, 0>(lat, links, in, istride, out, ostride, nullptr, nullptr, map, Terms<C>{},
                  (24.0 + 24.0 * map.n) * b * lat.V, s, prof);
}
template void wilson_apply_slots<double2>(const Lattice&, const double2*, const double2*, size_t, double2*, size_t,
                                          const SlotMap&, hipStream_t, Profiler*);
template void wilson_apply_slots<float2>(const Lattice&, const float2*, const float2*, size_t, float2*, size_t,
                                         const SlotMap&, hipStream_t, Profiler*);

void wilson_links_f32(const double2* links, float2* links32, int V, hipStream_t s) {
  const size_t n = wilson_link_entries(V);
  hipLaunchKernelGGL(links_to_f32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, links, links32, n);
  SGN_HIP(hipGetLastError());
}
