// Small dense complex linear algebra on the host, used by the deflation setup
// (Section 5.2, step (i)) for the Rayleigh-Ritz problems of size <= a few
// hundred: Hessenberg reduction by Householder reflections, the implicit
// single-shift QR algorithm with Wilkinson shifts (complex Schur form
// A = Z T Z^H), eigenvectors of the triangular factor by back substitution,
// and a thin QR factorisation (modified Gram-Schmidt, applied twice).
//
// The inner loops run down columns (or over the adjacent entries of two rows)
// on four doubles at a time, and sums that are one chain of additions run four
// at a time, in code for AVX2 where the host has it.  Every entry sees the
// operations of the plain loops in their order, without contraction, so the
// results do not depend on the host.  The eigenproblem of 90 columns that a
// restart of the m = 20 setup solves: 9.2 ms with strided scalar loops,
// 5.4 ms so.
#include "hostla.h"

#include <algorithm>
#include <cmath>
#include <limits>

#pragma clang fp contract(off)

namespace hostla {

namespace {

#define SGN_HOST_INLINE inline __attribute__((always_inline))
// name(params) from name_body, compiled for any x86-64 and for AVX2
#define SGN_HOST_CLONES(ret, name, params, args)                                     \
  namespace {                                                                        \
  __attribute__((target("avx2"))) ret name##_avx2 params { return name##_body args; } \
  }                                                                                  \
  ret name params { return __builtin_cpu_supports("avx2") ? name##_avx2 args : name##_body args; }

typedef double v2 __attribute__((vector_size(16), aligned(8)));  // an entry
typedef double v4 __attribute__((vector_size(32), aligned(8)));  // two adjacent entries

SGN_HOST_INLINE v4 load2(const cplx* p) { return *reinterpret_cast<const v4*>(p); }
SGN_HOST_INLINE void store2(cplx* p, v4 v) { *reinterpret_cast<v4*>(p) = v; }
SGN_HOST_INLINE v4 swap2(v4 v) { return __builtin_shufflevector(v, v, 1, 0, 3, 2); }

// y += a x (SUB: y -= a x) over n entries
template <bool SUB>
SGN_HOST_INLINE void axpy(int n, cplx a, const cplx* x, cplx* y) {
  const double r = a.real(), m = a.imag();
  const v4 ar = {r, r, r, r}, ai = {-m, m, -m, m};
  int i = 0;
  for (; i + 2 <= n; i += 2) {
    const v4 xv = load2(x + i), p = ar * xv + ai * swap2(xv);
    store2(y + i, SUB ? load2(y + i) - p : load2(y + i) + p);
  }
  if (i < n) {
    if (SUB)
      y[i] -= a * x[i];
    else
      y[i] += a * x[i];
  }
}

// out[k] = sum_i conj(x_k[i]) y_k[i] for K pairs, each sum in the order of i
template <int K>
SGN_HOST_INLINE void dots(int n, const cplx* const* x, const cplx* const* y, cplx* out) {
  v2 s[K];
  for (int k = 0; k < K; ++k) s[k] = v2{0.0, 0.0};
  for (int i = 0; i < n; ++i)
    for (int k = 0; k < K; ++k) {
      const v2 a = *reinterpret_cast<const v2*>(x[k] + i), b = *reinterpret_cast<const v2*>(y[k] + i);
      const v2 re = {a[0], a[0]}, im = {a[1], -a[1]};
      s[k] += re * b + im * __builtin_shufflevector(b, b, 1, 0);
    }
  for (int k = 0; k < K; ++k) out[k] = cplx(s[k][0], s[k][1]);
}

// the sums conj(x_k)^T y for k = 0 .. n-1, four at a time: one of x and y is a
// column per k (x0 + k ldx, y0 + k ldy), put(k, sum)
template <typename Put>
SGN_HOST_INLINE void dot_cols(int len, int n, const cplx* x0, size_t ldx, const cplx* y0, size_t ldy, Put put) {
  int k = 0;
  cplx out[4];
  for (; k + 4 <= n; k += 4) {
    const cplx* x[4] = {x0 + k * ldx, x0 + (k + 1) * ldx, x0 + (k + 2) * ldx, x0 + (k + 3) * ldx};
    const cplx* y[4] = {y0 + k * ldy, y0 + (k + 1) * ldy, y0 + (k + 2) * ldy, y0 + (k + 3) * ldy};
    dots<4>(len, x, y, out);
    for (int t = 0; t < 4; ++t) put(k + t, out[t]);
  }
  for (; k < n; ++k) {
    const cplx *x = x0 + k * ldx, *y = y0 + k * ldy;
    dots<1>(len, &x, &y, out);
    put(k, out[0]);
  }
}

// (a, b) -> (c a + s b, -conj(s) a + c b) for the entry pairs (a, b) = x[0],
// x[1] of n columns `ld` apart: two adjacent rows
SGN_HOST_INLINE void rot_rows(int n, double c, cplx s, cplx* x, size_t ld) {
  const double r = s.real(), m = s.imag();
  const v4 cv = {c, c, c, c}, fr = {r, m, -r, m}, fi = {-m, r, -m, -r};
  for (int j = 0; j < n; ++j, x += ld) {
    const v4 v = load2(x);
    const v4 re = __builtin_shufflevector(v, v, 2, 2, 0, 0), im = __builtin_shufflevector(v, v, 3, 3, 1, 1);
    store2(x, cv * v + (fr * re + fi * im));
  }
}

// (a, b) -> (c a + conj(s) b, -s a + c b) over n rows of two columns
SGN_HOST_INLINE void rot_cols(int n, double c, cplx s, cplx* a, cplx* b) {
  const double r = s.real(), m = s.imag();
  const v4 cv = {c, c, c, c}, rv = {r, r, r, r}, mv = {m, -m, m, -m};
  int i = 0;
  for (; i + 2 <= n; i += 2) {
    const v4 av = load2(a + i), bv = load2(b + i);
    store2(a + i, cv * av + (rv * bv + mv * swap2(bv)));
    store2(b + i, (mv * swap2(av) - rv * av) + cv * bv);
  }
  if (i < n) {
    const cplx x = a[i], y = b[i];
    a[i] = c * x + std::conj(s) * y;
    b[i] = -s * x + c * y;
  }
}

inline double abs1(cplx z) { return std::abs(z.real()) + std::abs(z.imag()); }

// Givens rotation G = [[c, s], [-conj(s), c]] with G (x, y)^T = (r, 0)^T.
inline void givens(cplx x, cplx y, double& c, cplx& s) {
  const double ax = std::abs(x), ay = std::abs(y);
  if (ay == 0.0) {
    c = 1.0;
    s = 0.0;
    return;
  }
  if (ax == 0.0) {
    c = 0.0;
    s = std::conj(y) / ay;
    return;
  }
  const double nrm = std::hypot(ax, ay);
  c = ax / nrm;
  s = (x / ax) * std::conj(y) / nrm;
}

}  // namespace

// A (n x n, column-major) -> upper Hessenberg H = Q^H A Q (in place), Q accumulated.
static SGN_HOST_INLINE void hessenberg_body(int n, cplx* H, cplx* Q) {
  auto h = [&](int i, int j) -> cplx& { return H[(size_t)j * n + i]; };
  auto q = [&](int i, int j) -> cplx& { return Q[(size_t)j * n + i]; };
  for (int j = 0; j < n; ++j)
    for (int i = 0; i < n; ++i) q(i, j) = (i == j) ? 1.0 : 0.0;
  std::vector<cplx> v(n), tmp(n);
  for (int k = 0; k + 2 < n; ++k) {
    const int len = n - k - 1;
    double xn = 0.0;
    for (int i = 0; i < len; ++i) xn += std::norm(h(k + 1 + i, k));
    xn = std::sqrt(xn);
    if (xn == 0.0) continue;
    const cplx x0 = h(k + 1, k);
    const cplx ph = (std::abs(x0) > 0.0) ? x0 / std::abs(x0) : cplx(1.0, 0.0);
    const cplx alpha = -ph * xn;
    for (int i = 0; i < len; ++i) v[i] = h(k + 1 + i, k);
    v[0] -= alpha;
    double vn = 0.0;
    for (int i = 0; i < len; ++i) vn += std::norm(v[i]);
    if (vn == 0.0) continue;
    const double tau = 2.0 / vn;
    // left: H[k+1:, k:] -= tau v (v^H H[k+1:, k:])
    dot_cols(len, n - k, v.data(), 0, &h(k + 1, k), n,
             [&](int j, cplx sum) __attribute__((always_inline)) { axpy<true>(len, sum * tau, v.data(), &h(k + 1, k + j)); });
    // right: H[:, k+1:] -= tau (H[:, k+1:] v) v^H ; same for Q
    for (cplx* M : {H, Q}) {
      cplx* cols = M + (size_t)(k + 1) * n;
      std::fill(tmp.begin(), tmp.end(), cplx(0.0, 0.0));
      for (int l = 0; l < len; ++l) axpy<false>(n, v[l], cols + (size_t)l * n, tmp.data());
      for (int i = 0; i < n; ++i) tmp[i] *= tau;
      for (int l = 0; l < len; ++l) axpy<true>(n, std::conj(v[l]), tmp.data(), cols + (size_t)l * n);
    }
    for (int i = 2; i <= len; ++i) h(k + i, k) = 0.0;
  }
}
SGN_HOST_CLONES(void, hessenberg, (int n, cplx* H, cplx* Q), (n, H, Q))

// Hessenberg H -> Schur form T (in place), Z updated so that A = Z T Z^H.
static SGN_HOST_INLINE bool schur_from_hessenberg_body(int n, cplx* H, cplx* Z) {
  auto h = [&](int i, int j) -> cplx& { return H[(size_t)j * n + i]; };
  auto z = [&](int i, int j) -> cplx& { return Z[(size_t)j * n + i]; };
  const double eps = std::numeric_limits<double>::epsilon();
  int hi = n - 1;
  int iter = 0, total = 0;
  while (hi > 0) {
    int l = hi;
    for (; l > 0; --l) {
      const double s = abs1(h(l - 1, l - 1)) + abs1(h(l, l));
      if (abs1(h(l, l - 1)) <= eps * (s > 0 ? s : 1.0)) {
        h(l, l - 1) = 0.0;
        break;
      }
    }
    if (l == hi) {
      --hi;
      iter = 0;
      continue;
    }
    if (++total > 100 * n) return false;
    ++iter;
    // Wilkinson shift from the trailing 2x2 block
    cplx mu;
    if (iter % 11 == 10) {
      mu = h(hi, hi) + cplx(std::abs(h(hi, hi - 1).real()) + std::abs(h(hi, hi - 1).imag()), 0.0);
    } else {
      const cplx a = h(hi - 1, hi - 1), b = h(hi - 1, hi), c = h(hi, hi - 1), d = h(hi, hi);
      const cplx half = 0.5 * (a - d);
      const cplx disc = std::sqrt(half * half + b * c);
      const cplx m1 = 0.5 * (a + d) + disc, m2 = 0.5 * (a + d) - disc;
      mu = (std::abs(m1 - d) < std::abs(m2 - d)) ? m1 : m2;
    }
    // implicit QR sweep on the active block l..hi (bulge chase with Givens)
    cplx x = h(l, l) - mu, y = h(l + 1, l);
    for (int k = l; k < hi; ++k) {
      double c;
      cplx s;
      givens(x, y, c, s);
      const int jc = (k > l) ? k - 1 : l;
      rot_rows(n - jc, c, s, &h(k, jc), n);
      rot_cols(std::min(k + 2, hi) + 1, c, s, &h(0, k), &h(0, k + 1));
      rot_cols(n, c, s, &z(0, k), &z(0, k + 1));
      if (k > l) h(k + 1, k - 1) = 0.0;
      if (k + 1 < hi) {
        x = h(k + 1, k);
        y = h(k + 2, k);
      }
    }
  }
  // clean the strictly lower part
  for (int j = 0; j < n; ++j)
    for (int i = j + 1; i < n; ++i) h(i, j) = 0.0;
  return true;
}
SGN_HOST_CLONES(bool, schur_from_hessenberg, (int n, cplx* H, cplx* Z), (n, H, Z))

static SGN_HOST_INLINE bool eig_body(int n, const cplx* A, cplx* w, cplx* V) {
  std::vector<cplx> T(A, A + (size_t)n * n), Z((size_t)n * n);
  hessenberg(n, T.data(), Z.data());
  if (!schur_from_hessenberg(n, T.data(), Z.data())) return false;
  auto t = [&](int i, int j) -> cplx& { return T[(size_t)j * n + i]; };
  double tn = 0.0;
  for (auto& v : T) tn = std::max(tn, std::abs(v));
  const double small = std::numeric_limits<double>::epsilon() * (tn > 0 ? tn : 1.0);
  std::vector<cplx> x(n), Tt((size_t)n * n);  // Tt: T by rows
  for (int j = 0; j < n; ++j)
    for (int i = 0; i <= j; ++i) Tt[(size_t)i * n + j] = t(i, j);
  for (int i = 0; i < n; ++i) {
    w[i] = t(i, i);
    x[i] = 1.0;
    for (int j = i - 1; j >= 0; --j) {
      cplx s = 0.0;
      for (int l = j + 1; l <= i; ++l) s += Tt[(size_t)j * n + l] * x[l];
      cplx d = t(j, j) - t(i, i);
      if (std::abs(d) < small) d = small;
      x[j] = -s / d;
    }
    // column i of V = Z X, of unit length
    cplx* y = V + (size_t)i * n;
    std::fill(y, y + n, cplx(0.0, 0.0));
    for (int l = 0; l <= i; ++l) axpy<false>(n, x[l], &Z[(size_t)l * n], y);
    double nn = 0.0;
    for (int r = 0; r < n; ++r) nn += std::norm(y[r]);
    nn = std::sqrt(nn);
    for (int r = 0; r < n; ++r) y[r] /= nn;
  }
  return true;
}
SGN_HOST_CLONES(bool, eig, (int n, const cplx* A, cplx* w, cplx* V), (n, A, w, V))

static SGN_HOST_INLINE int thin_qr_body(int rows, int cols, cplx* A, double rank_tol) {
  auto a = [&](int i, int j) -> cplx& { return A[(size_t)j * rows + i]; };
  int rank = 0;
  std::vector<double> norm0(cols, 0.0);
  for (int j = 0; j < cols; ++j) {
    for (int i = 0; i < rows; ++i) norm0[j] += std::norm(a(i, j));
    norm0[j] = std::sqrt(norm0[j]);
  }
  for (int j = 0; j < cols; ++j) {
    const double n0 = norm0[j];
    // the first pass against columns 0 .. j-1 is done (below); the second
    for (int k = 0; k < j; ++k)
      dot_cols(rows, 1, &a(0, k), rows, &a(0, j), rows,
               [&](int, cplx sum) __attribute__((always_inline)) { axpy<true>(rows, sum, &a(0, k), &a(0, j)); });
    double nn = 0.0;
    for (int i = 0; i < rows; ++i) nn += std::norm(a(i, j));
    nn = std::sqrt(nn);
    if (nn <= rank_tol * (n0 > 0 ? n0 : 1.0)) {
      for (int i = 0; i < rows; ++i) a(i, j) = 0.0;
    } else {
      for (int i = 0; i < rows; ++i) a(i, j) /= nn;
      ++rank;
    }
    // first pass of the later columns against column j
    dot_cols(rows, cols - j - 1, &a(0, j), 0, &A[(size_t)(j + 1) * rows], rows,
             [&](int l, cplx sum) __attribute__((always_inline)) { axpy<true>(rows, sum, &a(0, j), &a(0, j + 1 + l)); });
  }
  return rank;
}
SGN_HOST_CLONES(int, thin_qr, (int rows, int cols, cplx* A, double rank_tol), (rows, cols, A, rank_tol))

static SGN_HOST_INLINE void project_body(int n, int k, const cplx* H, const cplx* Q, cplx* T, int ldt) {
  std::vector<cplx> hq(n);
  for (int j = 0; j < k; ++j) {
    std::fill(hq.begin(), hq.end(), cplx(0.0, 0.0));
    for (int l = 0; l < n; ++l) {
      const cplx y = Q[(size_t)j * n + l];
      if (y != cplx(0.0, 0.0)) axpy<false>(n, y, H + (size_t)l * n, hq.data());
    }
    dot_cols(n, k, Q, n, hq.data(), 0, [&](int i, cplx sum) __attribute__((always_inline)) { T[(size_t)j * ldt + i] = sum; });
  }
}
SGN_HOST_CLONES(void, project, (int n, int k, const cplx* H, const cplx* Q, cplx* T, int ldt), (n, k, H, Q, T, ldt))

}  // namespace hostla

extern "C" int sgn_host_eig(int n, const double* A, double* w, double* V) {
  if (n < 1 || !A || !w || !V) return -1;
  try {
    const auto* a = reinterpret_cast<const hostla::cplx*>(A);
    return hostla::eig(n, a, reinterpret_cast<hostla::cplx*>(w), reinterpret_cast<hostla::cplx*>(V)) ? 0 : -5;
  } catch (...) {
    return -2;
  }
}
