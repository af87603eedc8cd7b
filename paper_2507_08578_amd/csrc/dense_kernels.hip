// Small dense FP64 linear algebra of the subspace steps, plus element-wise
// helpers.  Section 5.1 (Rayleigh-Ritz: a dense Hermitian eigenproblem of
// the block size) and section 5.4 (full-band Cholesky orthogonalisation).
//
//  * chol      : S = U^H U (upper Cholesky), blocked: each 64-wide diagonal
//                block is factored and inverted in LDS by one workgroup; the
//                row panels and trailing updates are MFMA products.
//  * heev      : cyclic two-sided Jacobi with the round-robin (circle)
//                ordering: in each round all n/2 disjoint pairs rotate at
//                once, A <- G^H A G, V <- V G.  For n <= 64 the whole solve
//                runs in one workgroup with A and V in LDS; larger n run a
//                block Jacobi whose block pairs take one such sweep each in
//                LDS, applied to A and V as tiled products.
#include "pw_internal.h"

#include <algorithm>
#include <cfloat>
#include <cmath>

namespace {

__device__ __forceinline__ cplx cmul(cplx a, cplx b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ cplx cconj(cplx a) { return make_double2(a.x, -a.y); }
__device__ __forceinline__ cplx cadd(cplx a, cplx b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ cplx csub(cplx a, cplx b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ cplx cscale(cplx a, double s) { return make_double2(a.x * s, a.y * s); }
__device__ __forceinline__ double cabs2(cplx a) { return a.x * a.x + a.y * a.y; }

// ---------------------------------------------------------------------------
// element-wise helpers
// ---------------------------------------------------------------------------
struct KinArgs {
  double b[9];
  double k[3];
};

__global__ void k_kinetic(int64_t npw, const int* __restrict__ miller, KinArgs a,
                          double* __restrict__ kin) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= npw) return;
  const double u0 = miller[3 * g] + a.k[0], u1 = miller[3 * g + 1] + a.k[1],
               u2 = miller[3 * g + 2] + a.k[2];
  const double qx = u0 * a.b[0] + u1 * a.b[3] + u2 * a.b[6];
  const double qy = u0 * a.b[1] + u1 * a.b[4] + u2 * a.b[7];
  const double qz = u0 * a.b[2] + u1 * a.b[5] + u2 * a.b[8];
  kin[g] = 0.5 * (qx * qx + qy * qy + qz * qz);
}

__global__ void k_scale_copy(int64_t n, const double* __restrict__ src, double scale,
                             double* __restrict__ dst) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = scale * src[i];
}

__global__ void __launch_bounds__(1024) k_max_reduce(int64_t n, const double* __restrict__ x,
                                                     double* out) {
  __shared__ double red[1024];
  double m = -DBL_MAX;
  for (int64_t i = threadIdx.x; i < n; i += blockDim.x) m = fmax(m, x[i]);
  red[threadIdx.x] = m;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + s]);
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = red[0];
}

__global__ void k_check_finite(int64_t n, const double* __restrict__ x, int* flag) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n && !isfinite(x[i])) atomicOr(flag, 1);
}

// The Hermitian matrix from its upper triangle: A[j][i] = conj(A[i][j]) for
// i < j, real diagonal (the lower triangle is not read).
__device__ __forceinline__ void hermitize_body(int64_t n, cplx* a, int64_t lda, int bx_) {
  const int64_t idx = (int64_t)bx_ * blockDim.x + threadIdx.x;
  if (idx >= n * n) return;
  const int64_t j = idx / n, i = idx - j * n;
  if (i > j) return;
  if (i == j) {
    a[i + j * lda].y = 0.0;
    return;
  }
  a[j + i * lda] = cconj(a[i + j * lda]);
}

__global__ void 
k_hermitize(int64_t n, cplx* a, int64_t lda) {
  hermitize_body(n, a, lda, blockIdx.x);
}

__device__ __forceinline__ void copy_block_body(int64_t rows, int64_t cols, const cplx* __restrict__ src, int64_t lds,
                             cplx* __restrict__ dst, int64_t ldd, int bx_) {
  const int64_t idx = (int64_t)bx_ * blockDim.x + threadIdx.x;
  if (idx >= rows * cols) return;
  const int64_t j = idx / rows, i = idx - j * rows;
  dst[i + j * ldd] = src[i + j * lds];
}

__global__ void 
k_copy_block(int64_t rows, int64_t cols, const cplx* __restrict__ src, int64_t lds,
                             cplx* __restrict__ dst, int64_t ldd) {
  copy_block_body(rows, cols, src, lds, dst, ldd, blockIdx.x);
}

__global__ void k_scale_rows_cols(int64_t n, const double* __restrict__ d, cplx* a, int64_t lda) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n * n) return;
  const int64_t j = idx / n, i = idx - j * n;
  a[i + j * lda] = cscale(a[i + j * lda], d[i] * d[j]);
}

__device__ __forceinline__ void axpby_block_body(int64_t npw, int64_t nb, double a, const cplx* x, int64_t ldx,
                              double b, const cplx* y, int64_t ldy, cplx* out, int64_t ldo,
                              const double* __restrict__ coef, int bx_) {
  const int64_t idx = (int64_t)bx_ * blockDim.x + threadIdx.x;
  if (idx >= npw * nb) return;
  if (coef) {
    a = coef[0];
    b = coef[1];
  }
  const int64_t j = idx / npw, i = idx - j * npw;
  const cplx u = x[i + j * ldx], v = y[i + j * ldy];
  out[i + j * ldo] = make_double2(a * u.x + b * v.x, a * u.y + b * v.y);
}

__global__ void 
k_axpby_block(int64_t npw, int64_t nb, double a, const cplx* x, int64_t ldx,
                              double b, const cplx* y, int64_t ldy, cplx* out, int64_t ldo,
                              const double* __restrict__ coef) {
  axpby_block_body(npw, nb, a, x, ldx, b, y, ldy, out, ldo, coef, blockIdx.x);
}

__device__ __forceinline__ void residuals_body(int64_t npw, const cplx* __restrict__ W, int64_t ldw, const cplx* __restrict__ Y,
            int64_t ldy, const double* __restrict__ lam, double* __restrict__ resid, int bx_) {
  __shared__ double red[256];
  const int64_t b = bx_;
  const double l = lam[b];
  const cplx* w = W + b * ldw;
  const cplx* y = Y + b * ldy;
  double s = 0.0;
  for (int64_t g = threadIdx.x; g < npw; g += blockDim.x) {
    const cplx d = make_double2(w[g].x - l * y[g].x, w[g].y - l * y[g].y);
    s += cabs2(d);
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if ((int)threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) resid[b] = sqrt(red[0]);
}

__global__ void __launch_bounds__(256) 
k_residuals(int64_t npw, const cplx* __restrict__ W, int64_t ldw, const cplx* __restrict__ Y,
            int64_t ldy, const double* __restrict__ lam, double* __restrict__ resid) {
  residuals_body(npw, W, ldw, Y, ldy, lam, resid, blockIdx.x);
}

// ---------------------------------------------------------------------------
// Blocked Cholesky (S = U^H U) for large n: per diagonal block of kb <= 64
// one workgroup factors it in LDS and inverts the factor; the row panel and
// the trailing update are matrix products (k_gemm_cn) issued by the host.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void chol_init_body(int n, const cplx* __restrict__ A, int64_t lda,
                                                    double* tol, int* status) {
  __shared__ double red[1024];
  __shared__ int bad[1024];
  double m = 0.0;
  int b = n;   // first diagonal entry that is NaN or infinite (a non-finite column)
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    const double d = A[i + (int64_t)i * lda].x;
    m = fmax(m, d);
    if (!isfinite(d)) b = min(b, i);
  }
  red[threadIdx.x] = m;
  bad[threadIdx.x] = b;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + s]);
      bad[threadIdx.x] = min(bad[threadIdx.x], bad[threadIdx.x + s]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    tol[0] = (double)n * DBL_EPSILON * red[0];
    status[0] = bad[0] < n ? kCholNonFinite - bad[0] : -1;
  }
}

__global__ void __launch_bounds__(1024) 
k_chol_init(int n, const cplx* __restrict__ A, int64_t lda,
                                                    double* tol, int* status) {
  chol_init_body(n, A, lda, tol, status);
}

// Factor the kb x kb diagonal block at A(k0, k0) (upper triangle read),
// write U back (zeros below its diagonal) and U^{-1} to dinv (ld kb).  A
// pivot at or below tol records k0 + p in status unless an earlier block did.
// 1/sqrt(x) and 1/x for x > 0 (normal): the hardware estimate refined by two
// Newton steps (each doubles the correct bits), much shorter dependency
// chains than the correctly rounded sequences; about 1 ulp.
__device__ __forceinline__ double rsqrt_nr(double x) {
  double y = __builtin_amdgcn_rsq(x);
  const double hx = 0.5 * x;
  y = y * fma(-hx * y, y, 1.5);
  y = y * fma(-hx * y, y, 1.5);
  return y;
}
__device__ __forceinline__ double rcp_nr(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = y * fma(-x, y, 2.0);
  y = y * fma(-x, y, 2.0);
  return y;
}

// Upper Cholesky of the kb x kb diagonal block at (k0, k0) (kb <= 64; 256
// threads, as both launchers give) and the inverse of its factor into dinv (ld kb).  Right-looking
// with the pivot row left unscaled, a_ij -= conj(a_pi) a_pj / a_pp for
// p < i <= j (thread (ti, tj) of a 16 x 16 grid owns the entries i = ti + 16u,
// j = tj + 16v), one barrier per pivot; the rows are scaled by 1/sqrt(a_pp)
// at the end.  The inverse is formed column by column, each entry's sum
// split over four lanes and joined by shuffles.
__device__ __forceinline__ void chol_diag_body(int kb, int k0, cplx* __restrict__ A, int64_t lda, cplx* __restrict__ dinv,
            const double* __restrict__ tol, int* status) {
  extern __shared__ cplx sm[];
  const int trs = kb + 1;
  cplx* a = sm;
  cplx* x = sm + kb * trs;
  __shared__ double sq[kCholBlock], rs[kCholBlock];   // sqrt(a_pp), 1 / sqrt(a_pp)
  const int tid = threadIdx.x, nt = blockDim.x;
  cplx* Ab = A + k0 + (int64_t)k0 * lda;
  for (int idx = tid; idx < kb * kb; idx += nt) {
    const int j = idx / kb, i = idx - j * kb;
    a[i + j * trs] = (i <= j) ? Ab[i + (int64_t)j * lda] : make_double2(0.0, 0.0);
  }
  __syncthreads();
  const double t = tol[0];
  const int ti = tid & 15, tj = (tid >> 4) & 15;
  int fail = -1;
  for (int p = 0; p < kb; ++p) {
    const double d = a[p + p * trs].x;   // the same value in every thread
    if (!(d > t)) {
      fail = p;
      break;
    }
    const double rd = rcp_nr(d);
#pragma unroll
    for (int u = 0; u < kCholBlock / 16; ++u) {
      const int i = ti + 16 * u;
      if (i <= p || i >= kb) continue;
      const cplx c = cscale(cconj(a[p + i * trs]), rd);
#pragma unroll
      for (int v = 0; v < kCholBlock / 16; ++v) {
        const int j = tj + 16 * v;
        if (j < i || j >= kb) continue;
        a[i + j * trs] = csub(a[i + j * trs], cmul(c, a[p + j * trs]));
      }
    }
    __syncthreads();
  }
  if (fail >= 0) {
    if (tid == 0 && status[0] == -1) status[0] = k0 + fail;
    return;
  }
  for (int i = tid; i < kb; i += nt) {
    sq[i] = sqrt(a[i + i * trs].x);
    rs[i] = rsqrt_nr(a[i + i * trs].x);
  }
  __syncthreads();
  for (int idx = tid; idx < kb * kb; idx += nt) {
    const int j = idx / kb, i = idx - j * kb;
    cplx u = make_double2(0.0, 0.0);
    if (i == j) u = make_double2(sq[i], 0.0);
    else if (i < j) u = cscale(a[i + j * trs], rs[i]);
    a[i + j * trs] = u;
    Ab[i + (int64_t)j * lda] = u;
  }
  __syncthreads();
  // x = U^{-1}: x_jj = 1/u_jj, x_ij = -(sum_{i <= p < j} x_ip u_pj) / u_jj
  const int i = tid >> 2, q = tid & 3;
  for (int j = 0; j < kb; ++j) {
    double sr = 0.0, si = 0.0;
    if (i < j)
      for (int p = i + q; p < j; p += 4) {
        const cplx xv = x[i + p * trs], uv = a[p + j * trs];
        sr += xv.x * uv.x - xv.y * uv.y;
        si += xv.x * uv.y + xv.y * uv.x;
      }
    sr += __shfl_xor(sr, 1, 64);
    si += __shfl_xor(si, 1, 64);
    sr += __shfl_xor(sr, 2, 64);
    si += __shfl_xor(si, 2, 64);
    if (q == 0 && i < kb) {
      const double rinv = rs[j];
      x[i + j * trs] = i < j ? make_double2(-sr * rinv, -si * rinv)
                             : make_double2(i == j ? rinv : 0.0, 0.0);
    }
    __syncthreads();
  }
  for (int idx = tid; idx < kb * kb; idx += nt) {
    const int j = idx / kb, i = idx - j * kb;
    dinv[i + j * kb] = x[i + j * trs];
  }
}

__global__ void __launch_bounds__(256) 
k_chol_diag(int kb, int k0, cplx* __restrict__ A, int64_t lda, cplx* __restrict__ dinv,
            const double* __restrict__ tol, int* status) {
  chol_diag_body(kb, k0, A, lda, dinv, tol, status);
}

__global__ void k_zero_lower(int n, cplx* A, int64_t lda) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)n * n) return;
  const int64_t j = idx / n, i = idx - j * n;
  if (i > j) A[i + j * lda] = make_double2(0.0, 0.0);
}

__global__ void k_identity_ld(int n, cplx* A, int64_t lda) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)n * n) return;
  const int64_t j = idx / n, i = idx - j * n;
  A[i + j * lda] = make_double2(i == j ? 1.0 : 0.0, 0.0);
}

// ---------------------------------------------------------------------------
// Jacobi
// ---------------------------------------------------------------------------
struct Rot {
  double cs, sn, t;
  cplx ph;     // c / |c|
  bool on;
};

// Round r of the circle method over n2 (even) indices: pair k -> (p < q).
__device__ __forceinline__ void rr_pair(int r, int k, int n2, int* p, int* q) {
  const int m = n2 - 1;
  const int a = k == 0 ? m : (r + k) % m;
  const int b = k == 0 ? r : (r - k + m) % m;
  *p = min(a, b);
  *q = max(a, b);
}

// number of i's pair in round r of the circle method, m = n2 - 1
__device__ __forceinline__ int rr_slot(int r, int i, int m) {
  const int k = i < r ? i - r + m : i - r;
  return (i == m || i == r) ? 0 : min(k, m - k);
}

// Rotation J = [[cs, sn ph], [-sn conj(ph), cs]] with J^H [[a, c], [conj c, b]] J diagonal:
// tau = (b - a)/(2|c|), t = sign(tau)/(|tau| + sqrt(1 + tau^2)), cs = 1/sqrt(1+t^2), sn = t cs;
// new diagonal a - t|c|, b + t|c|.  |c| below 1e-150 (|c|^2 near the
// denormal range) counts as zero: no rotation.  (Matrix entries here are
// O(1) Hamiltonian elements.)
// *tan, *absc: t and |c| unselected, for a diagonal update in one rounding
__device__ __forceinline__ Rot make_rot(double a, double b, cplx c, double* tan = nullptr,
                                        double* absc = nullptr) {
  // branch-free (callers form several rotations side by side); a zero c
  // selects the identity at the end (the arithmetic before it may be inf/NaN)
  Rot R;
  const double m2 = c.x * c.x + c.y * c.y;
  R.on = m2 > 1e-300;
  const double rmag = rsqrt_nr(m2);
  const double mag = m2 * rmag;
  const double tau = 0.5 * (b - a) * rmag;
  const double at = fabs(tau);
  // for |tau| > 1e100, sqrt(1 + tau^2) = |tau| to working precision
  const double u = 1.0 + tau * tau;
  const double ru = u * rsqrt_nr(u);
  const double root = at > 1e100 ? at : ru;
  const double t = copysign(rcp_nr(at + root), tau);
  const double cs = rsqrt_nr(1.0 + t * t);
  R.cs = R.on ? cs : 1.0;
  R.sn = R.on ? t * cs : 0.0;
  R.t = R.on ? t * mag : 0.0;
  if (tan) *tan = t, *absc = mag;
  R.ph = R.on ? make_double2(c.x * rmag, c.y * rmag) : make_double2(1.0, 0.0);
  return R;
}

// The products of a rotation with their rounding written out: left to the
// compiler, which of two products is fused depends on the code around it, and
// the phases of nearly degenerate vectors follow the last bit.
__device__ __forceinline__ cplx rmul(cplx a, cplx b) {
  return make_double2(fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x));
}
__device__ __forceinline__ cplx rmac(cplx a, double c, cplx s) {   // a c + s
  return make_double2(fma(a.x, c, s.x), fma(a.y, c, s.y));
}

// 2x2 block update X <- Jp^H X Jq, X = [[x11, x12], [x21, x22]]
__device__ __forceinline__ void rot_block(const Rot& P, const Rot& Q, cplx* x11, cplx* x12,
                                          cplx* x21, cplx* x22) {
  // M = X Jq: Jq = [[cs, sn ph], [-sn conj(ph), cs]]
  const cplx q12 = cscale(Q.ph, Q.sn);              // sn ph
  const cplx q21 = cscale(cconj(Q.ph), -Q.sn);      // -sn conj(ph)
  const cplx m11 = rmac(*x11, Q.cs, rmul(*x12, q21));
  const cplx m12 = rmac(*x12, Q.cs, rmul(*x11, q12));
  const cplx m21 = rmac(*x21, Q.cs, rmul(*x22, q21));
  const cplx m22 = rmac(*x22, Q.cs, rmul(*x21, q12));
  // Jp^H = [[cs, -sn ph], [sn conj(ph), cs]]
  const cplx p12 = cscale(P.ph, -P.sn);
  const cplx p21 = cscale(cconj(P.ph), P.sn);
  *x11 = rmac(m11, P.cs, rmul(p12, m21));
  *x12 = rmac(m12, P.cs, rmul(p12, m22));
  *x21 = rmac(m21, P.cs, rmul(p21, m11));
  *x22 = rmac(m22, P.cs, rmul(p21, m12));
}

// row update [vp, vq] <- [vp, vq] Jq
__device__ __forceinline__ void rot_row(const Rot& Q, cplx* vp, cplx* vq) {
  const cplx q12 = cscale(Q.ph, Q.sn);
  const cplx q21 = cscale(cconj(Q.ph), -Q.sn);
  const cplx a = *vp, b = *vq;
  *vp = rmac(a, Q.cs, rmul(b, q21));
  *vq = rmac(b, Q.cs, rmul(a, q12));
}

constexpr int kJacSmallMax = 64;
constexpr int kJacThreads = 1024;
constexpr int kMaxSweeps = kHeevMaxSweeps;

__device__ __forceinline__ double jac_tol(int n) { return fmax(1e-15, 2.2e-16 * n); }

// Workgroup size of the one-workgroup solve: one thread per 2x2 block of a
// round (h^2, h = ceil(n/2)), a power of two in [64, 1024].
inline int jac_threads(int n) {
  const int h = (n + 1) / 2;
  int t = 64;
  while (t < h * h && t < kJacThreads) t *= 2;
  return t;
}

// Whole Jacobi solve in LDS for n <= kJacMidMax, cyclic by the circle method on
// n padded to even (n2 = 2 h) with a zero row and column, which never rotates.
//
// The matrix is kept by position, not by index: position (role, k) holds the
// index that pair k of the current round has in that role, so thread t < h^2
// always works on block (pair t / h, pair t % h) at fixed addresses, and
// writes it to where its indices stand in the next round, a fixed permutation:
//   (a,0) -> (a,0), (a,1) -> (b,0), (a,k) -> (a,k-1), (b,k) -> (b,k+1),
//   (b,h-1) -> (a,h-1);
// m = n2 - 1 rounds bring every index back.  A and V are double-buffered, so a
// round has one barrier and every thread forms the two rotations it needs.
//
// One wavefront issues an instruction about every five cycles here, so the
// instructions of a round are its time.  Against indices by the circle method
// in place, two barriers and the rotations formed by h threads (jacobi_64_body),
// random matrices: n = 16 146 -> 60 us, 24 286 -> 116, 32 400 -> 156, 45 about
// 1200 -> 513 (n odd costs that form twice as much).
constexpr int kJacMidMax = 46;   // two copies of A and V: 135 KiB of LDS
struct RotS {
  double cs, t;     // cosine; change of the diagonal (0 where no rotation)
  cplx s;           // sn ph
  bool on;          // false: identity (c zero, or NaN)
};
// y = 1/sqrt(x): one third-order step from the hardware's estimate, with the
// rounding of x y carried along (correct to about half a unit)
__device__ __forceinline__ double rsqrt_h(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double xy = x * y, lo = fma(x, y, -xy);
  const double e = fma(-lo, y, fma(-xy, y, 1.0));
  return fma(y * e, fma(0.375, e, 0.5), y);
}
// The rotation of make_rot in the shortest chain of dependent operations: with
// d = b - a, r = sqrt(d^2 + 4 |c|^2), p = |d| + r and y = 1/sqrt(p^2 + 4 |c|^2)
// (= 1/sqrt(2 r p)): cs = p y, sn ph = 2 c y sign(d), t |c| = 4 |c|^2 r y^2
// sign(d); cs^2 + |sn|^2 = 1 to the rounding of y alone.
__device__ __forceinline__ RotS make_rot_s(double a, double b, cplx c) {
  const double m2 = c.x * c.x + c.y * c.y, d = b - a;
  const bool on = m2 > 1e-300;
  const double m4 = 4.0 * m2, q = fma(d, d, m4);
  const double r = q * rsqrt_h(q), p = fabs(d) + r;
  const double y = rsqrt_h(fma(p, p, m4)), y2 = copysign(2.0 * y, d);
  RotS R;
  R.on = on;
  R.cs = on ? p * y : 1.0;
  R.t = on ? (0.5 * m4 * y2) * (r * y) : 0.0;   // no factor beyond |c|^2 in size
  R.s = on ? make_double2(c.x * y2, c.y * y2) : make_double2(0.0, 0.0);
  return R;
}
// LDS: four entry planes of A's blocks and two of V's pairs, twice each
inline size_t jac_mid_lds(int64_t n) {
  const size_t h = (size_t)(n + 1) / 2;
  return 2 * (4 * h * h + 2 * 2 * h * h) * sizeof(cplx);
}

__device__ __forceinline__ void jacobi_mid_body(int n, const cplx* __restrict__ Ain, int64_t lda,
                                                double* __restrict__ w, cplx* __restrict__ Q,
                                                int64_t ldq, int* sweeps_out) {
  extern __shared__ cplx sm[];
  __shared__ double red[2][kJacThreads / 64];
  __shared__ int rank_[kJacMidMax];
  const int h = (n + 1) / 2, n2 = 2 * h, m = n2 - 1, hh = h * h;
  const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wave = tid >> 6;
  // buffer u: A entry planes e = 2 (row role) + (column role) at e hh, V planes (column
  // role) at (4 + 2 role) hh, [row][pair]
  const int bufsz = 8 * hh;
  // position (role, k) -> index in round 0, and -> position 2 k + role of the next round
  auto index0 = [&](int role, int k) { return k == 0 ? (role ? 0 : m) : role ? m - k : k; };
  auto next = [&](int role, int k) {
    if (role) return k == h - 1 ? 2 * k : 2 * (k + 1) + 1;
    return k == 0 ? 0 : k == 1 ? 1 : 2 * (k - 1);
  };
  const bool own = tid < hh;
  const int P = own ? tid / h : 0, Qb = own ? tid - P * h : 0;
  if (own) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int i = index0(e >> 1, P), j = index0(e & 1, Qb);
      sm[e * hh + tid] = (i < n && j < n) ? Ain[i + (int64_t)j * lda] : make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int g = 0; g < 2; ++g)
        sm[(4 + 2 * c) * hh + (P + g * h) * h + Qb] =
            make_double2(P + g * h == index0(c, Qb) ? 1.0 : 0.0, 0.0);
  }
  // where this thread's results go
  int dst[4], vdst[2];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int i = h > 1 ? next(e >> 1, P) : e >> 1, j = h > 1 ? next(e & 1, Qb) : e & 1;
    dst[e] = (2 * (i & 1) + (j & 1)) * hh + (i >> 1) * h + (j >> 1);
  }
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int j = h > 1 ? next(c, Qb) : c;
    vdst[c] = (4 + 2 * (j & 1)) * hh + P * h + (j >> 1);
  }
  const int dP = P * (h + 1), dQ = Qb * (h + 1);   // the pairs' diagonal blocks
  __syncthreads();
  int sweeps = 0, cur = 0;
  bool done = false;
  for (; sweeps < kMaxSweeps; ++sweeps) {
    {
      const cplx* A = sm + cur * bufsz;
      double off = 0.0, tot = 0.0;
      if (own) {
        const double m11 = cabs2(A[tid]), m12 = cabs2(A[hh + tid]);
        const double m21 = cabs2(A[2 * hh + tid]), m22 = cabs2(A[3 * hh + tid]);
        off = m12 + m21;
        tot = off + m11 + m22;
        if (P != Qb) off = tot;
      }
#pragma unroll
      for (int s = 32; s > 0; s >>= 1) {
        off += __shfl_xor(off, s, 64);
        tot += __shfl_xor(tot, s, 64);
      }
      if (lane == 0) {
        red[0][wave] = off;
        red[1][wave] = tot;
      }
      __syncthreads();
      // the owners' wavefronts in order: independent of the workgroup's size
      off = tot = 0.0;
      for (int q = 0; q < (hh + 63) / 64; ++q) {
        off += red[0][q];
        tot += red[1][q];
      }
      const double tl = jac_tol(n);
      done = off <= tl * tl * tot;
    }
    if (done) break;
    for (int r = 0; r < m; ++r) {
      if (own) {
        const cplx* A = sm + cur * bufsz;
        cplx* B = sm + (bufsz - cur * bufsz);
        const double ap = A[dP].x, aq = A[3 * hh + dP].x, bp = A[dQ].x, bq = A[3 * hh + dQ].x;
        const cplx cp = A[hh + dP], cq = A[hh + dQ];
        cplx x11 = A[tid], x12 = A[hh + tid], x21 = A[2 * hh + tid], x22 = A[3 * hh + tid];
        const cplx* V = A + 4 * hh + tid;
        const cplx y1 = V[0], y2 = V[2 * hh], z1 = V[hh], z2 = V[3 * hh];
        const RotS RP = make_rot_s(ap, aq, cp), RQ = make_rot_s(bp, bq, cq);
        {
          // M = X Jq, then Jp^H M
          const cplx q21 = make_double2(-RQ.s.x, RQ.s.y);
          const cplx m11 = cadd(cscale(x11, RQ.cs), cmul(x12, q21));
          const cplx m12 = cadd(cmul(x11, RQ.s), cscale(x12, RQ.cs));
          const cplx m21 = cadd(cscale(x21, RQ.cs), cmul(x22, q21));
          const cplx m22 = cadd(cmul(x21, RQ.s), cscale(x22, RQ.cs));
          const cplx p12 = make_double2(-RP.s.x, -RP.s.y), p21 = cconj(RP.s);
          x11 = cadd(cscale(m11, RP.cs), cmul(p12, m21));
          x12 = cadd(cscale(m12, RP.cs), cmul(p12, m22));
          x21 = cadd(cmul(p21, m11), cscale(m21, RP.cs));
          x22 = cadd(cmul(p21, m12), cscale(m22, RP.cs));
          // an identity leaves the block as it is: a NaN stays, and the solve
          // then ends without convergence instead of losing it
          if (P == Qb && RQ.on) {
            x11 = make_double2(ap - RQ.t, 0.0);
            x22 = make_double2(aq + RQ.t, 0.0);
            x12 = x21 = make_double2(0.0, 0.0);
          }
          B[dst[0]] = x11;
          B[dst[1]] = x12;
          B[dst[2]] = x21;
          B[dst[3]] = x22;
          B[vdst[0]] = cadd(cscale(y1, RQ.cs), cmul(y2, q21));
          B[vdst[0] + hh] = cadd(cscale(z1, RQ.cs), cmul(z2, q21));
          B[vdst[1]] = cadd(cmul(y1, RQ.s), cscale(y2, RQ.cs));
          B[vdst[1] + hh] = cadd(cmul(z1, RQ.s), cscale(z2, RQ.cs));
        }
      }
      __syncthreads();
      cur ^= 1;
    }
  }
  // sort ascending (rank by value, ties by index) and write out
  const cplx* A = sm + cur * bufsz;
  // position of index i in round 0: diagonal entry and V column
  auto role0 = [&](int i) { return i == m || (i > 0 && i < h) ? 0 : 1; };
  auto pair0 = [&](int i) { return i == m || i == 0 ? 0 : i < h ? i : m - i; };
  auto diag = [&](int i) { return A[3 * hh * role0(i) + pair0(i) * (h + 1)].x; };
  for (int i = tid; i < n; i += nt) {
    const double di = diag(i);
    int rk = 0;
    for (int j = 0; j < n; ++j) {
      const double dj = diag(j);
      if (dj < di || (dj == di && j < i)) ++rk;
    }
    rank_[i] = rk;
    w[rk] = di;
  }
  __syncthreads();
  for (int idx = tid; idx < n * n; idx += nt) {
    const int j = idx / n, i = idx - j * n;
    Q[i + (int64_t)rank_[j] * ldq] = A[(4 + 2 * role0(j)) * hh + i * h + pair0(j)];
  }
  if (tid == 0) sweeps_out[0] = done ? sweeps : -1;
}

// Whole Jacobi solve in LDS for kJacMidMax < n <= 64 (two copies of A and V do
// not fit the LDS): in place, the rotations of a round formed by h threads.
__device__ __forceinline__ void jacobi_64_body(int n, const cplx* __restrict__ Ain, int64_t lda, double* __restrict__ w,
               cplx* __restrict__ Q, int64_t ldq, int* sweeps_out) {
  extern __shared__ cplx sm[];
  const int n2 = n + (n & 1);
  const int h = n2 / 2;
  // A with an odd leading dimension: the 2x2 blocks a round updates sit in
  // columns n + 1 entries apart, which spreads them over the LDS banks
  const int la = n + 1;
  cplx* a = sm;               // n x n, ld la
  cplx* v = sm + n * la;      // n x n, ld n
  __shared__ Rot rots[kJacSmallMax / 2];
  __shared__ int pp[kJacSmallMax / 2], pq[kJacSmallMax / 2];   // this round's pairs
  __shared__ double red[kJacThreads];
  __shared__ double red2[kJacThreads];
  __shared__ int done;
  __shared__ int rank_[kJacSmallMax];
  const int tid = threadIdx.x, nt = blockDim.x;
  for (int idx = tid; idx < n * n; idx += nt) {
    const int j = idx / n, i = idx - j * n;
    a[i + j * la] = Ain[i + (int64_t)j * lda];
    v[idx] = make_double2(i == j ? 1.0 : 0.0, 0.0);
  }
  if (tid == 0) done = 0;
  __syncthreads();
  int sweeps = 0;
  for (; sweeps < kMaxSweeps; ++sweeps) {
    // convergence test before the sweep: 64 fixed partial sums, so the
    // summation order does not depend on the workgroup size
    if (tid < 64) {
      double off = 0.0, tot = 0.0;
      for (int idx = tid; idx < n * n; idx += 64) {
        const int j = idx / n, i = idx - j * n;
        const double m2 = cabs2(a[i + j * la]);
        tot += m2;
        if (i != j) off += m2;
      }
      red[tid] = off;
      red2[tid] = tot;
    }
    __syncthreads();
    for (int s = 32; s > 0; s >>= 1) {
      if (tid < s) {
        red[tid] += red[tid + s];
        red2[tid] += red2[tid + s];
      }
      __syncthreads();
    }
    if (tid == 0) {
      const double tl = jac_tol(n);
      done = (red[0] <= tl * tl * red2[0]) ? 1 : 0;
    }
    __syncthreads();
    if (done) break;
    for (int r = 0; r < n2 - 1; ++r) {
      if (tid < h) {
        int p, q;
        rr_pair(r, tid, n2, &p, &q);
        pp[tid] = p;
        pq[tid] = q;
        if (q < n) rots[tid] = make_rot(a[p + p * la].x, a[q + q * la].x, a[p + q * la]);
        else rots[tid] = make_rot(0.0, 0.0, make_double2(0.0, 0.0));
      }
      __syncthreads();
      for (int idx = tid; idx < h * h; idx += nt) {
        const int P = idx / h, Qb = idx - P * h;
        const int p1 = pp[P], q1 = pq[P], p2 = pp[Qb], q2 = pq[Qb];
        const Rot& RP = rots[P];
        const Rot& RQ = rots[Qb];
        if (q1 >= n || q2 >= n) {
          // pairs holding the padding index rotate nothing; update the real rows/cols only
          if (q1 < n && RP.on) {   // Q pair is (p2, pad): column p2 only
            cplx x1 = a[p1 + p2 * la], x2 = a[q1 + p2 * la];
            cplx y1 = x1, y2 = x2;
            // Jp^H [x1; x2]
            const cplx p12 = cscale(RP.ph, -RP.sn), p21 = cscale(cconj(RP.ph), RP.sn);
            y1 = cadd(cscale(x1, RP.cs), cmul(p12, x2));
            y2 = cadd(cmul(p21, x1), cscale(x2, RP.cs));
            a[p1 + p2 * la] = y1;
            a[q1 + p2 * la] = y2;
          } else if (q2 < n && RQ.on) {   // P pair is (p1, pad): row p1 only
            cplx x1 = a[p1 + p2 * la], x2 = a[p1 + q2 * la];
            rot_row(RQ, &x1, &x2);
            a[p1 + p2 * la] = x1;
            a[p1 + q2 * la] = x2;
          }
          continue;
        }
        if (P == Qb) {
          if (RP.on) {
            const double ap = a[p1 + p1 * la].x, aq = a[q1 + q1 * la].x;
            a[p1 + p1 * la] = make_double2(ap - RP.t, 0.0);
            a[q1 + q1 * la] = make_double2(aq + RP.t, 0.0);
            a[p1 + q1 * la] = make_double2(0.0, 0.0);
            a[q1 + p1 * la] = make_double2(0.0, 0.0);
          }
          continue;
        }
        if (!RP.on && !RQ.on) continue;
        cplx x11 = a[p1 + p2 * la], x12 = a[p1 + q2 * la], x21 = a[q1 + p2 * la], x22 = a[q1 + q2 * la];
        rot_block(RP, RQ, &x11, &x12, &x21, &x22);
        a[p1 + p2 * la] = x11;
        a[p1 + q2 * la] = x12;
        a[q1 + p2 * la] = x21;
        a[q1 + q2 * la] = x22;
      }
      for (int idx = tid; idx < n * h; idx += nt) {
        const int Qb = idx / n, i = idx - Qb * n;
        const int p2 = pp[Qb], q2 = pq[Qb];
        if (q2 >= n || !rots[Qb].on) continue;
        cplx x1 = v[i + p2 * n], x2 = v[i + q2 * n];
        rot_row(rots[Qb], &x1, &x2);
        v[i + p2 * n] = x1;
        v[i + q2 * n] = x2;
      }
      __syncthreads();
    }
  }
  // sort ascending (rank by value, ties by index) and write out
  for (int i = tid; i < n; i += nt) {
    const double di = a[i + i * la].x;
    int rk = 0;
    for (int j = 0; j < n; ++j) {
      const double dj = a[j + j * la].x;
      if (dj < di || (dj == di && j < i)) ++rk;
    }
    rank_[i] = rk;
  }
  __syncthreads();
  for (int i = tid; i < n; i += nt) w[rank_[i]] = a[i + i * la].x;
  for (int idx = tid; idx < n * n; idx += nt) {
    const int j = idx / n, i = idx - j * n;
    Q[i + (int64_t)rank_[j] * ldq] = v[i + j * n];
  }
  if (tid == 0) sweeps_out[0] = done ? sweeps : -1;
}

__device__ __forceinline__ void jacobi_small_body(int n, const cplx* __restrict__ Ain, int64_t lda,
                                                  double* __restrict__ w, cplx* __restrict__ Q,
                                                  int64_t ldq, int* sweeps_out) {
  if (n <= kJacMidMax) jacobi_mid_body(n, Ain, lda, w, Q, ldq, sweeps_out);
  else jacobi_64_body(n, Ain, lda, w, Q, ldq, sweeps_out);
}
// dynamic LDS of solves of up to n
inline size_t jac_small_lds(int64_t n) {
  const size_t mid = jac_mid_lds(std::min<int64_t>(n, kJacMidMax));
  return n > kJacMidMax ? std::max(mid, (size_t)(n * (2 * n + 1)) * sizeof(cplx)) : mid;
}

__global__ void __launch_bounds__(kJacThreads)
k_jacobi_small(int n, const cplx* __restrict__ Ain, int64_t lda, double* __restrict__ w,
               cplx* __restrict__ Q, int64_t ldq, int* sweeps_out) {
  jacobi_small_body(n, Ain, lda, w, Q, ldq, sweeps_out);
}

// n > 64: block Jacobi.  The matrix (padded with zero rows and columns to
// n2p, a multiple of 2 kBJ) is cut into blocks of kBJ indices; an outer
// round pairs the blocks by the circle method and, for every pair (I, J) at
// once, runs one cyclic Jacobi sweep on the 2 kBJ x 2 kBJ sub-problem
// A[I u J, I u J] in LDS, accumulating its rotations in a unitary Q_k; then
// A <- G^H A G and V <- V G with G the block-diagonal product of the Q_k, as
// two tiled products.  Every index pair meets in each outer sweep (pairs
// inside a block in every round), so the outer sweeps converge like cyclic
// Jacobi.  Rounds 1 .. nblk - 2 of a sweep each take one launch that also
// applies the previous round's update (k_bj_step); round 0 and the last
// update have launches of their own.  Padding indices have zero rows and
// columns and never rotate.  The
// convergence test runs on the device before every outer sweep; once it
// passes, conv[0] is set and every later launch of the solve returns at
// once, so a fixed number of sweeps can be issued with no host read.
constexpr int kBJ = 16;           // block size
constexpr int kBJS = 2 * kBJ;     // sub-problem size
constexpr int kBJTile = 64;       // row tile of the V update (and the padding of n)

// global index of sub-problem index i of block pair (I, J)
__device__ __forceinline__ int bj_index(int i, int I, int J) {
  return i < kBJ ? I * kBJ + i : J * kBJ + (i - kBJ);
}

// One sweep on each block pair of outer round r (workgroup k: pair k);
// Qout[k] (kBJS x kBJS, column-major) receives the accumulated rotations.
//
// An inner round is a chain of dependent steps with one barrier, and a
// wavefront issues an instruction about every five cycles, so the instructions
// of the wavefronts on that chain are its time.  Wavefronts 0 .. 3 hold one 2x2
// block of A per thread: thread (P, Qb) has rows of pair P and columns of pair
// Qb.  A is kept by pair position, the lower index of pair k at 2 k and the
// higher at 2 k + 1, in four planes (row and column position even or odd), so
// every round reads the same addresses; where the results stand in the next
// round comes from a table.  Every thread forms the rotation of pair Qb and
// takes pair P's from lane P of its wavefront.  A is double-buffered.
// Wavefronts 4 .. 7 apply the previous round's rotations, which the first ones
// leave in LDS, to V (rows Qb and Qb + kBJ of pair P).  With V, and the circle
// method's index arithmetic, on the chain's own wavefronts a sweep of 31 rounds
// took 31.4 us (k_bj_inner) and a fused step 40.4 us at n = 160 and 45.5 us at
// n = 512; as it is, 24.2, 32.2 and 36.6 us.
constexpr int kBJHalf = kBJ * kBJ;               // threads of the A part
constexpr int kBJThreads = 2 * kBJHalf;
constexpr int kBJA = 4 * kBJHalf;                // entries of one copy of A
static_assert(2 * kBJHalf == kBJS * kBJ, "V (row, pair) items: two per thread");
static_assert(64 % kBJ == 0, "the lanes P < kBJ of every wavefront hold the pairs' rotations");
// offsets of a row and of a column position in the planes
__host__ __device__ constexpr int bj_rowpart(int pos) { return (pos & 1) * 2 * kBJHalf + (pos >> 1) * kBJ; }
__host__ __device__ constexpr int bj_colpart(int pos) { return (pos & 1) * kBJHalf + (pos >> 1); }
// Per round and pair: the pair's indices, and the row and column offsets of
// their positions in the next round.
struct BjTable {
  unsigned pq[kBJS - 1][kBJ], row[kBJS - 1][kBJ], col[kBJS - 1][kBJ];   // low half: lower index
};
constexpr BjTable bj_make_table() {
  BjTable t{};
  constexpr int m = kBJS - 1;
  int lo[kBJS][kBJ] = {}, hi[kBJS][kBJ] = {}, pos[kBJS][kBJS] = {};
  for (int r = 0; r <= m; ++r)
    for (int k = 0; k < kBJ; ++k) {
      const int a = k == 0 ? m : (r % m + k) % m, b = k == 0 ? r % m : (r % m - k + m) % m;
      lo[r][k] = a < b ? a : b;
      hi[r][k] = a < b ? b : a;
      pos[r][lo[r][k]] = 2 * k;
      pos[r][hi[r][k]] = 2 * k + 1;
    }
  for (int r = 0; r < m; ++r)
    for (int k = 0; k < kBJ; ++k) {
      const int p = pos[r + 1][lo[r][k]], q = pos[r + 1][hi[r][k]];
      t.pq[r][k] = lo[r][k] | hi[r][k] << 16;
      t.row[r][k] = bj_rowpart(p) | bj_rowpart(q) << 16;
      t.col[r][k] = bj_colpart(p) | bj_colpart(q) << 16;
    }
  return t;
}
__device__ const BjTable bj_table = bj_make_table();
// position of index i in round 0: pairs (k, 31 - k), and (0, 31) for k = 0
__device__ __forceinline__ int bj_pos0(int i) { return i < kBJ ? 2 * i : 2 * (kBJS - 1 - i) + 1; }
__device__ __forceinline__ int bj_place0(int i, int j) {
  return bj_rowpart(bj_pos0(i)) + bj_colpart(bj_pos0(j));
}

// LDS beside the two copies of A: V, two rounds of rotations, the table
struct BjSweepLds {
  cplx v[kBJS * kBJS];
  Rot rots[2][kBJ];
  BjTable tab;
};
// a0: the sub-problem on entry, entry (i, j) at bj_place0(i, j)
__device__ __forceinline__ void bj_inner_sweep(cplx* a0, cplx* a1, BjSweepLds* L,
                                               cplx* __restrict__ qo) {
  const int tid = threadIdx.x;
  cplx* v = L->v;
  for (int idx = tid; idx < kBJS * kBJS; idx += kBJThreads) {
    const int j = idx / kBJS, i = idx - j * kBJS;
    v[idx] = make_double2(i == j ? 1.0 : 0.0, 0.0);
  }
  for (int idx = tid; idx < (int)(sizeof(BjTable) / 4); idx += kBJThreads)
    reinterpret_cast<unsigned*>(&L->tab)[idx] = reinterpret_cast<const unsigned*>(&bj_table)[idx];
  __syncthreads();
  const bool apart = tid < kBJHalf;
  const int P = (tid % kBJHalf) / kBJ, Qb = tid % kBJ;
  // V of round rr: rows Qb, Qb + kBJ of pair P
  auto v_round = [&](int rr) {
    const Rot R = L->rots[rr & 1][P];
    const unsigned pq = L->tab.pq[rr][P];
    const int p = pq & 0xffff, q = pq >> 16;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int vi = Qb + h * kBJ;
      cplx x1 = v[vi + p * kBJS], x2 = v[vi + q * kBJS];
      rot_row(R, &x1, &x2);
      v[vi + p * kBJS] = x1;
      v[vi + q * kBJS] = x2;
    }
  };
  for (int rr = 0; rr < kBJS - 1; ++rr) {
    if (apart) {
      const cplx* ac = rr & 1 ? a1 : a0;
      cplx* an = rr & 1 ? a0 : a1;
      const int dg = Qb * (kBJ + 1);
      double tq, cq;
      const Rot RQ = make_rot(ac[dg].x, ac[3 * kBJHalf + dg].x, ac[kBJHalf + dg], &tq, &cq);
      Rot RP;
      RP.cs = __shfl(RQ.cs, P, 64);
      RP.sn = __shfl(RQ.sn, P, 64);
      RP.ph = make_double2(__shfl(RQ.ph.x, P, 64), __shfl(RQ.ph.y, P, 64));
      if (P == 0) L->rots[rr & 1][Qb] = RQ;
      cplx x11 = ac[tid], x12 = ac[kBJHalf + tid];
      cplx x21 = ac[2 * kBJHalf + tid], x22 = ac[3 * kBJHalf + tid];
      const unsigned row = L->tab.row[rr][P], col = L->tab.col[rr][Qb];
      // an identity rotation (pair off) leaves the values unchanged exactly
      if (P == Qb) {
        if (RQ.on) {
          x11 = make_double2(fma(-cq, tq, x11.x), 0.0);
          x22 = make_double2(fma(cq, tq, x22.x), 0.0);
          x12 = make_double2(0.0, 0.0);
          x21 = make_double2(0.0, 0.0);
        }
      } else {
        rot_block(RP, RQ, &x11, &x12, &x21, &x22);
      }
      const int r1 = row & 0xffff, r2 = row >> 16, c1 = col & 0xffff, c2 = col >> 16;
      an[r1 + c1] = x11;
      an[r1 + c2] = x12;
      an[r2 + c1] = x21;
      an[r2 + c2] = x22;
    } else if (rr > 0) {
      v_round(rr - 1);
    }
    __syncthreads();
  }
  if (!apart) v_round(kBJS - 2);
  __syncthreads();
  for (int idx = tid; idx < kBJS * kBJS; idx += kBJThreads) qo[idx] = v[idx];
}

// Round 0 of a sweep: the sub-problems read straight from A.
__global__ void __launch_bounds__(kBJThreads)
k_bj_inner(int n2p, int r, const cplx* __restrict__ A, cplx* __restrict__ Qout,
           const int* __restrict__ conv) {
  if (conv[0]) return;
  __shared__ cplx a[2][kBJA];
  __shared__ BjSweepLds lds;
  int I, J;
  rr_pair(r, blockIdx.x, n2p / kBJ, &I, &J);
  for (int idx = threadIdx.x; idx < kBJS * kBJS; idx += kBJThreads) {
    const int j = idx / kBJS, i = idx - j * kBJS;
    a[0][bj_place0(i, j)] = A[bj_index(i, I, J) + (int64_t)bj_index(j, I, J) * n2p];
  }
  bj_inner_sweep(a[0], a[1], &lds, Qout + (int64_t)blockIdx.x * kBJS * kBJS);
}

// Two-sided update of outer round r.  Workgroup w < npair^2 takes the
// sub-block of A on block pair p = w / npair (rows) and block pair q =
// w % npair (columns): Aout[idx_p, idx_q] <- Q_p^H Ain[idx_p, idx_q] Q_q,
// both products in LDS.  Workgroup npair^2 + t npair + q takes kBJTile rows
// of V from row t kBJTile: V[rows, idx_q] <- V[rows, idx_q] Q_q.  Each
// workgroup reads and writes only its own elements, so Ain may be Aout.
// sm: LDS of kBJUpdateSm entries.
constexpr int kBJUThreads = kBJThreads;
constexpr int kBJUSmA = (kBJS + 1) * kBJS + 2 * kBJS * kBJS, kBJUSmV = kBJTile * kBJS + kBJS * kBJS;
constexpr int kBJUpdateSm = kBJUSmA > kBJUSmV ? kBJUSmA : kBJUSmV;
__device__ __forceinline__ void bj_update_body(int n, int n2p, int r, const cplx* Ain, cplx* Aout,
                                               cplx* __restrict__ V, const cplx* __restrict__ Qk,
                                               int w, cplx* sm) {
  constexpr int LX = kBJS + 1;                         // odd row pitch of the A sub-block
  const int tid = threadIdx.x;
  const int nblk = n2p / kBJ, npair = nblk / 2;
  if (w < npair * npair) {
    const int p = w / npair, q = w - p * npair;
    int Ip, Jp, Iq, Jq;
    rr_pair(r, p, nblk, &Ip, &Jp);
    rr_pair(r, q, nblk, &Iq, &Jq);
    cplx* X = sm;                       // [i + j LX]
    cplx* Qp = sm + LX * kBJS;          // [i + m kBJS] = conj(Q_p(m, i)): the lanes of
    cplx* Qq = Qp + kBJS * kBJS;        //   a wavefront read consecutive i
    const cplx* gp = Qk + (int64_t)p * kBJS * kBJS;
    const cplx* gq = Qk + (int64_t)q * kBJS * kBJS;
    for (int idx = tid; idx < kBJS * kBJS; idx += kBJUThreads) {
      const int j = idx / kBJS, i = idx - j * kBJS;
      X[i + j * LX] = Ain[bj_index(i, Ip, Jp) + (int64_t)bj_index(j, Iq, Jq) * n2p];
      Qp[j + i * kBJS] = cconj(gp[idx]);
      Qq[idx] = gq[idx];
    }
    __syncthreads();
    constexpr int NJ = kBJS * kBJS / kBJUThreads;      // outputs per thread
    constexpr int G = kBJUThreads / kBJS;
    const int i = tid % kBJS, jg = tid / kBJS;
    cplx acc[NJ];
#pragma unroll
    for (int t = 0; t < NJ; ++t) acc[t] = make_double2(0.0, 0.0);
    // T = Q_p^H X
#pragma unroll 8
    for (int m = 0; m < kBJS; ++m) {
      const cplx qh = Qp[i + m * kBJS];
#pragma unroll
      for (int t = 0; t < NJ; ++t) {
        const cplx x = X[m + (jg + t * G) * LX];
        acc[t].x += qh.x * x.x - qh.y * x.y;
        acc[t].y += qh.x * x.y + qh.y * x.x;
      }
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < NJ; ++t) X[i + (jg + t * G) * LX] = acc[t];
    __syncthreads();
    // out = T Q_q
#pragma unroll
    for (int t = 0; t < NJ; ++t) acc[t] = make_double2(0.0, 0.0);
#pragma unroll 8
    for (int m = 0; m < kBJS; ++m) {
      const cplx x = X[i + m * LX];
#pragma unroll
      for (int t = 0; t < NJ; ++t) {
        const cplx qv = Qq[m + (jg + t * G) * kBJS];
        acc[t].x += x.x * qv.x - x.y * qv.y;
        acc[t].y += x.x * qv.y + x.y * qv.x;
      }
    }
    const int gi = bj_index(i, Ip, Jp);
#pragma unroll
    for (int t = 0; t < NJ; ++t)
      Aout[gi + (int64_t)bj_index(jg + t * G, Iq, Jq) * n2p] = acc[t];
    return;
  }
  const int vw = w - npair * npair;
  const int tile = vw / npair, q = vw - tile * npair;
  int Iq, Jq;
  rr_pair(r, q, nblk, &Iq, &Jq);
  const int r0 = tile * kBJTile;
  cplx* T = sm;                         // [i + m kBJTile]: V[r0 + i, idx_q[m]]
  cplx* Qq = sm + kBJTile * kBJS;       // [m + j kBJS]
  const cplx* gq = Qk + (int64_t)q * kBJS * kBJS;
  for (int idx = tid; idx < kBJTile * kBJS; idx += kBJUThreads) {
    const int m = idx / kBJTile, i = idx - m * kBJTile;
    T[idx] = (r0 + i < n) ? V[(r0 + i) + (int64_t)bj_index(m, Iq, Jq) * n] : make_double2(0.0, 0.0);
  }
  for (int idx = tid; idx < kBJS * kBJS; idx += kBJUThreads) Qq[idx] = gq[idx];
  __syncthreads();
  constexpr int G = kBJUThreads / kBJTile, NJ = kBJS / G;
  const int i = tid % kBJTile, jg = tid / kBJTile;
  cplx acc[NJ];
#pragma unroll
  for (int t = 0; t < NJ; ++t) acc[t] = make_double2(0.0, 0.0);
#pragma unroll 8
  for (int m = 0; m < kBJS; ++m) {
    const cplx x = T[i + m * kBJTile];
#pragma unroll
    for (int t = 0; t < NJ; ++t) {
      const cplx qv = Qq[m + (jg + t * G) * kBJS];
      acc[t].x += x.x * qv.x - x.y * qv.y;
      acc[t].y += x.x * qv.y + x.y * qv.x;
    }
  }
  if (r0 + i < n) {
#pragma unroll
    for (int t = 0; t < NJ; ++t)
      V[(r0 + i) + (int64_t)bj_index(jg + t * G, Iq, Jq) * n] = acc[t];
  }
}

// The update of the last round of a sweep, in place.
__global__ void __launch_bounds__(kBJUThreads)
k_bj_update(int n, int n2p, int r, cplx* __restrict__ A, cplx* __restrict__ V,
            const cplx* __restrict__ Qk, const int* __restrict__ conv) {
  if (conv[0]) return;
  __shared__ cplx sm[kBJUpdateSm];
  bj_update_body(n, n2p, r, A, A, V, Qk, blockIdx.x, sm);
}

// Sub-problem of round r's pair (I, J) of M_r = G^H M G, G the block-
// diagonal unitary of round r - 1 (Qin, its pairs), M = Min, formed by the
// workgroup itself: with block I in round-(r-1) pair p1 (offset o1 = 0 for
// its first block, kBJ for its second) and J in p2, entry (a, b) of the
// (I, I) block is sum conj(Q_p1(m, o1 + a)) M[idx_p1(m), idx_p1(n)]
// Q_p1(n, o1 + b), and so on for (I, J) and (J, J); (J, I) is the conjugate
// transpose of (I, J).  The products run in the order of bj_update_body
// (Q^H M first, then the right factor), the sums over m and n ascending.
// sm: kBJLookSm entries of scratch (disjoint from a0).
constexpr int kBJLookSm = (kBJS + 1) * kBJS + 4 * kBJS * kBJ + kBJ * (kBJS + 1);
__device__ __forceinline__ void bj_lookahead(int n2p, int r, int I, int J, const cplx* __restrict__ Min,
                                             const cplx* __restrict__ Qin, cplx* a0, cplx* sm) {
  constexpr int LX = kBJS + 1, LT = kBJ;
  const int tid = threadIdx.x;
  const int nblk = n2p / kBJ, npair = nblk / 2;
  // the round-(r-1) pairs of blocks I and J, and which of the pair they are
  const int m = nblk - 1;
  const int p1 = rr_slot(r - 1, I, m), p2 = rr_slot(r - 1, J, m);
  int I1, J1, I2, J2;
  rr_pair(r - 1, p1, nblk, &I1, &J1);
  rr_pair(r - 1, p2, nblk, &I2, &J2);
  const int o1 = I1 == I ? 0 : kBJ, o2 = I2 == J ? 0 : kBJ;
  cplx* X = sm;                         // [i + j LX]: a kBJS x kBJS block of Min
  cplx* L1 = X + LX * kBJS;             // [a + m kBJ] = conj(Q_p1(m, o1 + a))
  cplx* L2 = L1 + kBJS * kBJ;           // the same for p2
  cplx* R1 = L2 + kBJS * kBJ;           // [m + b kBJS] = Q_p1(m, o1 + b)
  cplx* R2 = R1 + kBJS * kBJ;
  cplx* T = R2 + kBJS * kBJ;            // [a + j LT]: (Q^H X)(a, j), kBJ x kBJS
  const cplx* q1 = Qin + (int64_t)p1 * kBJS * kBJS;
  const cplx* q2 = Qin + (int64_t)p2 * kBJS * kBJS;
  // three blocks: (I, I) from (p1, p1), (I, J) from (p1, p2), (J, J) from
  // (p2, p2); each block's entries are loaded into registers while the
  // previous block's products run
  constexpr int NX = kBJS * kBJS / kBJThreads;
  typedef double dv2 __attribute__((ext_vector_type(2)));   // native vector: stays in registers
  dv2 xr[NX];
  auto load_x = [&](int blk) {
    const int Ir = blk < 2 ? I1 : I2, Jr = blk < 2 ? J1 : J2;       // row pair of Min
    const int Ic = blk == 0 ? I1 : I2, Jc = blk == 0 ? J1 : J2;     // column pair
#pragma unroll
    for (int t = 0; t < NX; ++t) {
      const int idx = tid + t * kBJThreads;
      const int j = idx / kBJS, i = idx - j * kBJS;
      xr[t] = *reinterpret_cast<const dv2*>(Min + bj_index(i, Ir, Jr) + (int64_t)bj_index(j, Ic, Jc) * n2p);
    }
  };
  load_x(0);
  for (int idx = tid; idx < kBJS * kBJ; idx += kBJThreads) {
    const int b = idx / kBJS, m = idx - b * kBJS;
    const cplx v1 = q1[m + (o1 + b) * kBJS], v2 = q2[m + (o2 + b) * kBJS];
    R1[idx] = v1;
    R2[idx] = v2;
    L1[b + m * kBJ] = cconj(v1);
    L2[b + m * kBJ] = cconj(v2);
  }
  for (int blk = 0; blk < 3; ++blk) {
    const cplx* L = blk < 2 ? L1 : L2;
    const cplx* R = blk == 0 ? R1 : R2;
    const int da = blk < 2 ? 0 : kBJ, db = blk == 0 ? 0 : kBJ;      // place in the sub-problem
    __syncthreads();   // X and T free (previous block done; Q copies stored)
#pragma unroll
    for (int t = 0; t < NX; ++t) {
      const int idx = tid + t * kBJThreads;
      const int j = idx / kBJS, i = idx - j * kBJS;
      X[i + j * LX] = make_double2(xr[t].x, xr[t].y);
    }
    if (blk < 2) load_x(blk + 1);
    __syncthreads();
    {   // T = L X: kBJ x kBJS, one entry per thread
      const int a = tid % kBJ, j = tid / kBJ;
      cplx acc = make_double2(0.0, 0.0);
#pragma unroll 8
      for (int m = 0; m < kBJS; ++m) {
        const cplx qh = L[a + m * kBJ];
        const cplx x = X[m + j * LX];
        acc.x += qh.x * x.x - qh.y * x.y;
        acc.y += qh.x * x.y + qh.y * x.x;
      }
      T[a + j * LT] = acc;
    }
    __syncthreads();
    if (tid < kBJHalf) {   // S = T R: kBJ x kBJ, one entry per thread
      const int a = tid % kBJ, b = tid / kBJ;
      cplx acc = make_double2(0.0, 0.0);
#pragma unroll 8
      for (int m = 0; m < kBJS; ++m) {
        const cplx x = T[a + m * LT];
        const cplx qv = R[m + b * kBJS];
        acc.x += x.x * qv.x - x.y * qv.y;
        acc.y += x.x * qv.y + x.y * qv.x;
      }
      a0[bj_place0(da + a, db + b)] = acc;
      if (blk == 1) a0[bj_place0(db + b, da + a)] = cconj(acc);
    }
  }
  __syncthreads();
}

// Outer round r >= 1 of a sweep fused with the update of round r - 1.
// Workgroups [0, npair): the inner sweep of round r, each forming its
// sub-problem of the rotated matrix itself (bj_lookahead from Ain and Qin)
// and writing its rotations to Qout.  Workgroups [npair, npair + ugrid):
// the update of round r - 1 from Ain into Aout (and V) with Qin.  The two
// kinds read the same inputs and write disjoint outputs, so the update of
// one round runs beside the inner sweep of the next.
constexpr int kBJSweepSm = 2 * kBJA + (int)((sizeof(BjSweepLds) + sizeof(cplx) - 1) / sizeof(cplx));
constexpr int kBJInnerSm = kBJA + kBJLookSm > kBJSweepSm ? kBJA + kBJLookSm : kBJSweepSm;
constexpr int kBJStepSm = kBJUpdateSm > kBJInnerSm ? kBJUpdateSm : kBJInnerSm;
__global__ void __launch_bounds__(kBJUThreads)
k_bj_step(int n, int n2p, int r, const cplx* __restrict__ Ain, cplx* __restrict__ Aout,
          cplx* __restrict__ V, const cplx* __restrict__ Qin, cplx* __restrict__ Qout,
          const int* __restrict__ conv) {
  if (conv[0]) return;
  __shared__ cplx sm[kBJStepSm];
  const int npair = n2p / kBJ / 2;
  if ((int)blockIdx.x >= npair) {
    bj_update_body(n, n2p, r - 1, Ain, Aout, V, Qin, blockIdx.x - npair, sm);
    return;
  }
  int I, J;
  rr_pair(r, blockIdx.x, n2p / kBJ, &I, &J);
  cplx* a0 = sm;
  cplx* scr = sm + kBJA;
  bj_lookahead(n2p, r, I, J, Ain, Qin, a0, scr);   // ends with a barrier: scr is free
  bj_inner_sweep(a0, scr, reinterpret_cast<BjSweepLds*>(scr + kBJA),
                 Qout + (int64_t)blockIdx.x * kBJS * kBJS);
}

// A0 = [a 0; 0 0] (n2 x n2), V0 = [I 0] (n x n2)
__global__ void k_jacobi_init(int n, int n2, const cplx* __restrict__ a, int64_t lda,
                              cplx* __restrict__ A0, cplx* __restrict__ V0, int* __restrict__ conv) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx == 0) {
    conv[0] = 0;   // converged
    conv[1] = 0;   // sweeps when it converged
  }
  const int64_t na = (int64_t)n2 * n2;
  if (idx < na) {
    const int j = (int)(idx / n2), i = (int)(idx - (int64_t)j * n2);
    A0[idx] = (i < n && j < n) ? a[i + (int64_t)j * lda] : make_double2(0.0, 0.0);
    return;
  }
  const int64_t vi = idx - na;
  if (vi >= (int64_t)n * n2) return;
  const int j = (int)(vi / n), i = (int)(vi - (int64_t)j * n);
  V0[vi] = make_double2(i == j ? 1.0 : 0.0, 0.0);
}

// Rank of index p's eigenvalue among 0..n-1 (ties by index).
__global__ void k_jacobi_rank(int n, int ld, const cplx* __restrict__ A, int* __restrict__ rank,
                              const int* __restrict__ conv, int* __restrict__ sweeps_out) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p == 0) sweeps_out[0] = conv[0] ? conv[1] : -1;
  if (p >= n) return;
  const double dp = A[p + (int64_t)p * ld].x;
  int rk = 0;
  for (int q = 0; q < n; ++q) {
    const double dq = A[q + (int64_t)q * ld].x;
    if (dq < dp || (dq == dp && q < p)) ++rk;
  }
  rank[p] = rk;
}

__global__ void k_jacobi_scatter(int n, int ld, const cplx* __restrict__ A,
                                 const cplx* __restrict__ V, const int* __restrict__ rank,
                                 double* __restrict__ w, cplx* __restrict__ Q, int64_t ldq) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)n * n) return;
  const int p = (int)(idx / n), i = (int)(idx - (int64_t)p * n);
  const int rp = rank[p];
  Q[i + (int64_t)rp * ldq] = V[i + (int64_t)p * n];
  if (i == 0) w[rp] = A[p + (int64_t)p * ld].x;
}

// Squared off-diagonal and total Frobenius norms of A (n x n), in two fixed-
// order stages: kOffParts workgroups sum interleaved slices into part[2 w],
// part[2 w + 1]; one workgroup adds the parts.
constexpr int kOffParts = 256;
__global__ void __launch_bounds__(256) k_offnorm_part(int n, const cplx* __restrict__ A,
                                                      double* __restrict__ part,
                                                      const int* __restrict__ conv) {
  if (conv[0]) return;
  __shared__ double r1[256], r2[256];
  double off = 0.0, tot = 0.0;
  const int64_t nn = (int64_t)n * n;
  for (int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x; idx < nn;
       idx += (int64_t)kOffParts * 256) {
    const int64_t j = idx / n, i = idx - j * n;
    const double m2 = cabs2(A[idx]);
    tot += m2;
    if (i != j) off += m2;
  }
  r1[threadIdx.x] = off;
  r2[threadIdx.x] = tot;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      r1[threadIdx.x] += r1[threadIdx.x + s];
      r2[threadIdx.x] += r2[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = r1[0];
    part[2 * blockIdx.x + 1] = r2[0];
  }
}

// ... and sets conv = {1, sweep} when off <= tol2 * total (the test that
// precedes outer sweep `sweep`).
__global__ void __launch_bounds__(kOffParts) k_offnorm_final(const double* __restrict__ part,
                                                            double tol2, int sweep,
                                                            int* __restrict__ conv) {
  if (conv[0]) return;
  __shared__ double r1[kOffParts], r2[kOffParts];
  r1[threadIdx.x] = part[2 * threadIdx.x];
  r2[threadIdx.x] = part[2 * threadIdx.x + 1];
  __syncthreads();
  for (int s = kOffParts / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      r1[threadIdx.x] += r1[threadIdx.x + s];
      r2[threadIdx.x] += r2[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0 && r1[0] <= tol2 * r2[0]) {
    conv[1] = sweep;
    conv[0] = 1;
  }
}

// ---------------------------------------------------------------------------
// precision conversions for the low-precision filter path
// ---------------------------------------------------------------------------
__device__ __forceinline__ void block_to_f32_body(int64_t rows, int64_t cols, const cplx* __restrict__ x, int64_t ldx,
                               float2* __restrict__ y, int64_t ldy, int bx_) {
  const int64_t idx = (int64_t)bx_ * blockDim.x + threadIdx.x;
  if (idx >= rows * cols) return;
  const int64_t j = idx / rows, i = idx - j * rows;
  const cplx v = x[i + j * ldx];
  y[i + j * ldy] = make_float2((float)v.x, (float)v.y);
}

__global__ void 
k_block_to_f32(int64_t rows, int64_t cols, const cplx* __restrict__ x, int64_t ldx,
                               float2* __restrict__ y, int64_t ldy) {
  block_to_f32_body(rows, cols, x, ldx, y, ldy, blockIdx.x);
}

__device__ __forceinline__ void block_to_f64_body(int64_t rows, int64_t cols, const float2* __restrict__ x, int64_t ldx,
                               cplx* __restrict__ y, int64_t ldy, int bx_) {
  const int64_t idx = (int64_t)bx_ * blockDim.x + threadIdx.x;
  if (idx >= rows * cols) return;
  const int64_t j = idx / rows, i = idx - j * rows;
  const float2 v = x[i + j * ldx];
  y[i + j * ldy] = make_double2((double)v.x, (double)v.y);
}

__global__ void 
k_block_to_f64(int64_t rows, int64_t cols, const float2* __restrict__ x, int64_t ldx,
                               cplx* __restrict__ y, int64_t ldy) {
  block_to_f64_body(rows, cols, x, ldx, y, ldy, blockIdx.x);
}

// out = fp32(a x + b y), x and y FP64
__device__ __forceinline__ void axpby_to_f32_body(int64_t rows, int64_t cols, double a, const cplx* __restrict__ x,
                               int64_t ldx, double b, const cplx* __restrict__ y, int64_t ldy,
                               float2* __restrict__ out, int64_t ldo, const double* __restrict__ coef, int bx_) {
  const int64_t idx = (int64_t)bx_ * blockDim.x + threadIdx.x;
  if (idx >= rows * cols) return;
  if (coef) {
    a = coef[0];
    b = coef[1];
  }
  const int64_t j = idx / rows, i = idx - j * rows;
  const cplx u = x[i + j * ldx], v = y[i + j * ldy];
  out[i + j * ldo] = make_float2((float)(a * u.x + b * v.x), (float)(a * u.y + b * v.y));
}

__global__ void 
k_axpby_to_f32(int64_t rows, int64_t cols, double a, const cplx* __restrict__ x,
                               int64_t ldx, double b, const cplx* __restrict__ y, int64_t ldy,
                               float2* __restrict__ out, int64_t ldo, const double* __restrict__ coef) {
  axpby_to_f32_body(rows, cols, a, x, ldx, b, y, ldy, out, ldo, coef, blockIdx.x);
}

__global__ void k_real_to_f32(int64_t n, const double* __restrict__ src, double scale,
                              float* __restrict__ dst) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = (float)(scale * src[i]);
}

__global__ void k_tw_to_f32(int n, const cplx* __restrict__ src, float2* __restrict__ dst) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = make_float2((float)src[i].x, (float)src[i].y);
}

// Chebyshev filter coefficients on the device from the current Ritz values
// (a = largest, a0 = smallest) and the upper bound b: step i (0-based) of the
// scaled recurrence is out = alpha (H in) + beta in + gamma prev with
//   i = 0: alpha = s/e, beta = -s c/e, gamma = 0            (s = e/(a0 - c))
//   i > 0: s' = 1/(2/s_0 - s), alpha = 2 s'/e, beta = -alpha c, gamma = -s s'; s = s'
// If a0 < a < b fails, every step becomes the identity and flag[0] is set.
__device__ __forceinline__ void cheb_coef_body(const double* __restrict__ eig, int nb, const double* __restrict__ upper,
                            int degree, double* __restrict__ coef, int* flag) {
  if (threadIdx.x != 0) return;
  const double a = eig[nb - 1], a0 = eig[0], b = upper[0];
  if (!(a0 < a && a < b)) {
    for (int i = 0; i < degree; ++i) {
      coef[3 * i] = 0.0;
      coef[3 * i + 1] = 1.0;
      coef[3 * i + 2] = 0.0;
    }
    flag[0] = 1;
    return;
  }
  const double e = 0.5 * (b - a), c = 0.5 * (b + a);
  double sigma = e / (a0 - c);
  const double tau = 2.0 / sigma;
  coef[0] = sigma / e;
  coef[1] = -sigma * c / e;
  coef[2] = 0.0;
  for (int i = 1; i < degree; ++i) {
    const double sn = 1.0 / (tau - sigma);
    const double al = 2.0 * sn / e;
    coef[3 * i] = al;
    coef[3 * i + 1] = -al * c;
    coef[3 * i + 2] = -sigma * sn;
    sigma = sn;
  }
}

__global__ void 
k_cheb_coef(const double* __restrict__ eig, int nb, const double* __restrict__ upper,
                            int degree, double* __restrict__ coef, int* flag) {
  cheb_coef_body(eig, nb, upper, degree, coef, flag);
}

// Sticky per-item failure flags of a batched iteration:
// flags[0] = first failing Cholesky pivot + 1 (or -(column + 1) for a Gram
// diagonal entry that is not finite), flags[1] = eigensolver hit the
// sweep limit, flags[2] = bad filter interval (set by k_cheb_coef),
// flags[3] = largest sweep count seen.
__device__ __forceinline__ void batch_flags_body(const int* __restrict__ chol_status, const int* __restrict__ sweeps,
                              int* flags) {
  if (threadIdx.x != 0) return;
  if (chol_status && chol_status[0] != -1 && flags[0] == 0)
    flags[0] = chol_status[0] >= 0 ? chol_status[0] + 1 : chol_status[0] - kCholNonFinite - 1;
  const int sw = sweeps[0];
  if (sw < 0) flags[1] = 1;
  else if (sw > flags[3]) flags[3] = sw;
}

__global__ void 
k_batch_flags(const int* __restrict__ chol_status, const int* __restrict__ sweeps,
                              int* flags) {
  batch_flags_body(chol_status, sweeps, flags);
}

// ---- fused-batch steps: item = blockIdx.y for the element-wise steps (x covers
// the largest item), blockIdx.x for the one-workgroup steps
__global__ void kb_cheb_coef(const ItemDev* __restrict__ D, int degree) {
  const ItemDev& d = D[blockIdx.x];
  cheb_coef_body(d.eig, d.nb, d.upper, degree, d.coef, d.flags + 2);
}

// first filter step from W = H Y: FP64 blk, or FP32 b32[1]
__global__ void kb_filter_first(const ItemDev* __restrict__ D, int fp32) {
  const ItemDev& d = D[blockIdx.y];
  if (fp32)
    axpby_to_f32_body(d.npw, d.nb, 0.0, d.hy, d.npw, 0.0, d.y, d.npw, d.b32[1], d.npw, d.coef,
                      blockIdx.x);
  else
    axpby_block_body(d.npw, d.nb, 0.0, d.hy, d.npw, 0.0, d.y, d.npw, d.blk, d.npw, d.coef,
                     blockIdx.x);
}

__global__ void kb_to_f32(const ItemDev* __restrict__ D) {
  const ItemDev& d = D[blockIdx.y];
  block_to_f32_body(d.npw, d.nb, d.y, d.npw, d.b32[0], d.npw, blockIdx.x);
}

__global__ void kb_to_f64(const ItemDev* __restrict__ D, int sel) {
  const ItemDev& d = D[blockIdx.y];
  block_to_f64_body(d.npw, d.nb, item_blk32(d, sel), d.npw, d.y, d.npw, blockIdx.x);
}

__global__ void kb_copy(const ItemDev* __restrict__ D, int sel_src, int sel_dst) {
  const ItemDev& d = D[blockIdx.y];
  copy_block_body(d.npw, d.nb, item_blk64(d, sel_src), d.npw, item_blk64(d, sel_dst), d.npw,
                  blockIdx.x);
}

__global__ void kb_hermitize(const ItemDev* __restrict__ D) {
  const ItemDev& d = D[blockIdx.y];
  hermitize_body(d.nb, d.sub0, d.nb, blockIdx.x);
}

__global__ void __launch_bounds__(1024) kb_chol_init(const ItemDev* __restrict__ D) {
  const ItemDev& d = D[blockIdx.x];
  chol_init_body(d.nb, d.sub0, d.nb, d.dtol, d.status);
}

__global__ void __launch_bounds__(256) kb_chol_diag(const ItemDev* __restrict__ D) {
  const ItemDev& d = D[blockIdx.x];
  chol_diag_body(d.nb, 0, d.sub0, d.nb, d.dinv, d.dtol, d.status);
}

__global__ void __launch_bounds__(kJacThreads) kb_jacobi(const ItemDev* __restrict__ D) {
  const ItemDev& d = D[blockIdx.x];
  jacobi_small_body(d.nb, d.sub0, d.nb, d.eig, d.sub1, d.nb, d.sweeps);
}

__global__ void __launch_bounds__(256) kb_residuals(const ItemDev* __restrict__ D) {
  const ItemDev& d = D[blockIdx.y];
  if ((int)blockIdx.x >= d.nb) return;
  residuals_body(d.npw, d.hy, d.npw, d.y, d.npw, d.eig, d.resid, blockIdx.x);
}

__global__ void kb_flags(const ItemDev* __restrict__ D) {
  const ItemDev& d = D[blockIdx.x];
  batch_flags_body(d.status, d.sweeps, d.flags);
}

inline unsigned nblocks(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

}  // namespace

hipError_t launch_kinetic(int64_t npw, const int* miller, const double* recip9, const double* k3,
                          double* kin, hipStream_t s) {
  KinArgs a;
  for (int i = 0; i < 9; ++i) a.b[i] = recip9[i];
  for (int i = 0; i < 3; ++i) a.k[i] = k3[i];
  hipLaunchKernelGGL(k_kinetic, dim3(nblocks(npw, 256)), dim3(256), 0, s, npw, miller, a, kin);
  return hipGetLastError();
}

hipError_t launch_scale_copy(int64_t n, const double* src, double scale, double* dst, hipStream_t s) {
  hipLaunchKernelGGL(k_scale_copy, dim3(nblocks(n, 256)), dim3(256), 0, s, n, src, scale, dst);
  return hipGetLastError();
}

hipError_t launch_max_reduce(int64_t n, const double* x, double* out1, hipStream_t s) {
  hipLaunchKernelGGL(k_max_reduce, dim3(1), dim3(1024), 0, s, n, x, out1);
  return hipGetLastError();
}

hipError_t launch_check_finite(int64_t n, const double* x, int* flag, hipStream_t s) {
  hipLaunchKernelGGL(k_check_finite, dim3(nblocks(n, 256)), dim3(256), 0, s, n, x, flag);
  return hipGetLastError();
}

hipError_t launch_hermitize(int64_t n, cplx* a, int64_t lda, hipStream_t s) {
  hipLaunchKernelGGL(k_hermitize, dim3(nblocks(n * n, 256)), dim3(256), 0, s, n, a, lda);
  return hipGetLastError();
}

hipError_t launch_copy_block(int64_t rows, int64_t cols, const cplx* src, int64_t lds, cplx* dst,
                             int64_t ldd, hipStream_t s) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_copy_block, dim3(nblocks(rows * cols, 256)), dim3(256), 0, s, rows, cols, src,
                     lds, dst, ldd);
  return hipGetLastError();
}

hipError_t launch_scale_rows_cols(int64_t n, const double* d, cplx* a, int64_t lda, hipStream_t s) {
  hipLaunchKernelGGL(k_scale_rows_cols, dim3(nblocks(n * n, 256)), dim3(256), 0, s, n, d, a, lda);
  return hipGetLastError();
}

hipError_t launch_axpby_block(int64_t npw, int64_t nb, double a, const cplx* x, int64_t ldx, double b,
                              const cplx* y, int64_t ldy, cplx* out, int64_t ldo, hipStream_t s,
                              const double* coef) {
  hipLaunchKernelGGL(k_axpby_block, dim3(nblocks(npw * nb, 256)), dim3(256), 0, s, npw, nb, a, x,
                     ldx, b, y, ldy, out, ldo, coef);
  return hipGetLastError();
}

hipError_t launch_batch_flags(const int* chol_status, const int* sweeps, int* flags, hipStream_t s) {
  hipLaunchKernelGGL(k_batch_flags, dim3(1), dim3(64), 0, s, chol_status, sweeps, flags);
  return hipGetLastError();
}

hipError_t launch_cheb_coef(const double* eig, int nb, const double* upper, int degree, double* coef,
                            int* flag, hipStream_t s) {
  hipLaunchKernelGGL(k_cheb_coef, dim3(1), dim3(64), 0, s, eig, nb, upper, degree, coef, flag);
  return hipGetLastError();
}

hipError_t launch_block_to_f32(int64_t rows, int64_t cols, const cplx* x, int64_t ldx, float2* y,
                               int64_t ldy, hipStream_t s) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_block_to_f32, dim3(nblocks(rows * cols, 256)), dim3(256), 0, s, rows, cols, x,
                     ldx, y, ldy);
  return hipGetLastError();
}

hipError_t launch_block_to_f64(int64_t rows, int64_t cols, const float2* x, int64_t ldx, cplx* y,
                               int64_t ldy, hipStream_t s) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_block_to_f64, dim3(nblocks(rows * cols, 256)), dim3(256), 0, s, rows, cols, x,
                     ldx, y, ldy);
  return hipGetLastError();
}

hipError_t launch_axpby_to_f32(int64_t rows, int64_t cols, double a, const cplx* x, int64_t ldx,
                               double b, const cplx* y, int64_t ldy, float2* out, int64_t ldo,
                               hipStream_t s, const double* coef) {
  hipLaunchKernelGGL(k_axpby_to_f32, dim3(nblocks(rows * cols, 256)), dim3(256), 0, s, rows, cols, a,
                     x, ldx, b, y, ldy, out, ldo, coef);
  return hipGetLastError();
}

__global__ void k_block_to_b16(int64_t rows, int64_t cols, const cplx* __restrict__ x, int64_t ldx,
                               bf16c* __restrict__ y, int64_t ldy) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= rows * cols) return;
  const int64_t j = idx / rows, i = idx - j * rows;
  y[i + j * ldy] = st_c<bf16c>(x[i + j * ldx]);
}

__global__ void k_block_b16_to_f64(int64_t rows, int64_t cols, const bf16c* __restrict__ x,
                                   int64_t ldx, cplx* __restrict__ y, int64_t ldy) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= rows * cols) return;
  const int64_t j = idx / rows, i = idx - j * rows;
  const float2 v = ld_c(x[i + j * ldx]);
  y[i + j * ldy] = make_double2(v.x, v.y);
}

__global__ void k_axpby_to_b16(int64_t rows, int64_t cols, double a, const cplx* __restrict__ x,
                               int64_t ldx, double b, const cplx* __restrict__ y, int64_t ldy,
                               bf16c* __restrict__ out, int64_t ldo, const double* __restrict__ coef) {
  if (coef) {
    a = coef[0];
    b = coef[1];
  }
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= rows * cols) return;
  const int64_t j = idx / rows, i = idx - j * rows;
  const cplx u = x[i + j * ldx], v = y[i + j * ldy];
  out[i + j * ldo] = st_c<bf16c>(make_double2(a * u.x + b * v.x, a * u.y + b * v.y));
}

hipError_t launch_block_to_b16(int64_t rows, int64_t cols, const cplx* x, int64_t ldx, bf16c* y,
                               int64_t ldy, hipStream_t s) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_block_to_b16, dim3(nblocks(rows * cols, 256)), dim3(256), 0, s, rows, cols,
                     x, ldx, y, ldy);
  return hipGetLastError();
}

hipError_t launch_block_b16_to_f64(int64_t rows, int64_t cols, const bf16c* x, int64_t ldx, cplx* y,
                                   int64_t ldy, hipStream_t s) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_block_b16_to_f64, dim3(nblocks(rows * cols, 256)), dim3(256), 0, s, rows,
                     cols, x, ldx, y, ldy);
  return hipGetLastError();
}

hipError_t launch_axpby_to_b16(int64_t rows, int64_t cols, double a, const cplx* x, int64_t ldx,
                               double b, const cplx* y, int64_t ldy, bf16c* out, int64_t ldo,
                               hipStream_t s, const double* coef) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_axpby_to_b16, dim3(nblocks(rows * cols, 256)), dim3(256), 0, s, rows, cols,
                     a, x, ldx, b, y, ldy, out, ldo, coef);
  return hipGetLastError();
}

hipError_t launch_real_to_f32(int64_t n, const double* src, double scale, float* dst, hipStream_t s) {
  hipLaunchKernelGGL(k_real_to_f32, dim3(nblocks(n, 256)), dim3(256), 0, s, n, src, scale, dst);
  return hipGetLastError();
}

hipError_t launch_tw_to_f32(int n, const cplx* src, float2* dst, hipStream_t s) {
  hipLaunchKernelGGL(k_tw_to_f32, dim3(nblocks(n, 256)), dim3(256), 0, s, n, src, dst);
  return hipGetLastError();
}

hipError_t launch_residuals(int64_t npw, int64_t nb, const cplx* W, int64_t ldw, const cplx* Y,
                            int64_t ldy, const double* lam, double* resid, hipStream_t s) {
  hipLaunchKernelGGL(k_residuals, dim3((unsigned)nb), dim3(256), 0, s, npw, W, ldw, Y, ldy, lam,
                     resid);
  return hipGetLastError();
}

hipError_t launch_chol_init(int64_t n, const cplx* a, int64_t lda, double* tol, int* status,
                            hipStream_t s) {
  hipLaunchKernelGGL(k_chol_init, dim3(1), dim3(1024), 0, s, (int)n, a, lda, tol, status);
  return hipGetLastError();
}

hipError_t launch_chol_diag(int kb, int k0, cplx* a, int64_t lda, cplx* dinv, const double* tol,
                            int* status, hipStream_t s) {
  const size_t lds = (size_t)2 * kb * (kb + 1) * sizeof(cplx);
  hipLaunchKernelGGL(k_chol_diag, dim3(1), dim3(256), lds, s, kb, k0, a, lda, dinv, tol, status);
  return hipGetLastError();
}

hipError_t launch_zero_lower(int64_t n, cplx* a, int64_t lda, hipStream_t s) {
  hipLaunchKernelGGL(k_zero_lower, dim3(nblocks(n * n, 256)), dim3(256), 0, s, (int)n, a, lda);
  return hipGetLastError();
}

hipError_t launch_identity(int64_t n, cplx* a, int64_t lda, hipStream_t s) {
  hipLaunchKernelGGL(k_identity_ld, dim3(nblocks(n * n, 256)), dim3(256), 0, s, (int)n, a, lda);
  return hipGetLastError();
}

// padded size: a multiple of the update tiles (and so of 2 kBJ)
static int64_t bj_padded(int64_t n) { return (n + kBJTile - 1) / kBJTile * kBJTile; }

// Work layout for n > 64: A (n2p x n2p), V (n x n2p), the block pairs'
// unitaries (n2p / kBJS of kBJS x kBJS), n ints of ranks, then two 16-byte
// aligned doubles.
size_t heev_work_bytes(int64_t n) {
  const int64_t n2p = bj_padded(n);
  return (size_t)(2 * n2p * n2p + n * n2p + 2 * n2p * kBJS) * sizeof(cplx) +
         (size_t)(n + 8) * sizeof(int) + 64 + 2 * kOffParts * sizeof(double);
}

hipError_t heev_set_lds_limit(size_t bytes) {
  const void* fns[4] = {(const void*)k_jacobi_small, (const void*)k_chol_diag,
                        (const void*)kb_jacobi, (const void*)kb_chol_diag};
  for (const void* f : fns) {
    hipFuncAttributes at;
    hipError_t e = hipFuncGetAttributes(&at, f);
    if (e != hipSuccess) return e;
    const size_t dyn = bytes > at.sharedSizeBytes ? bytes - at.sharedSizeBytes : 0;
    e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_heev_small_async(int64_t n, const cplx* a, int64_t lda, double* w, cplx* q,
                                   int64_t ldq, int* sweeps_dev, hipStream_t s) {
  if (n > kJacSmallMax) return hipErrorInvalidValue;
  const size_t lds = jac_small_lds(n);
  hipLaunchKernelGGL(k_jacobi_small, dim3(1), dim3(jac_threads((int)n)), lds, s, (int)n, a, lda, w,
                     q, ldq, sweeps_dev);
  return hipGetLastError();
}

hipError_t launch_heev_async(int64_t n, const cplx* a, int64_t lda, double* w, cplx* q,
                             int64_t ldq, void* work, int* sweeps_dev, int max_sweeps,
                             hipStream_t s) {
  if (n <= kJacSmallMax) return launch_heev_small_async(n, a, lda, w, q, ldq, sweeps_dev, s);
  if (max_sweeps < 1 || max_sweeps > kMaxSweeps) return hipErrorInvalidValue;
  const int64_t n2p = bj_padded(n);
  char* base = static_cast<char*>(work);
  const size_t mat_bytes = (size_t)(2 * n2p * n2p + n * n2p + 2 * n2p * kBJS) * sizeof(cplx);
  int* rank = reinterpret_cast<int*>(base + mat_bytes);
  int* conv = rank + n;                  // {converged, sweeps}
  const size_t stat_off = (mat_bytes + (size_t)(n + 8) * sizeof(int) + 15) & ~(size_t)15;
  double* dpart = reinterpret_cast<double*>(base + stat_off) + 2;   // kOffParts pairs
  // A: the matrix at the start of every sweep; A1: the other copy of the
  // fused rounds (each reads one and writes the other, an even number per
  // sweep); Q0 / Q1: the unitaries of consecutive rounds
  cplx* A = reinterpret_cast<cplx*>(base);
  cplx* A1 = A + n2p * n2p;
  cplx* V = A1 + n2p * n2p;
  cplx* Q0 = V + n * n2p;
  cplx* Q1 = Q0 + n2p * kBJS;
  hipLaunchKernelGGL(k_jacobi_init, dim3(nblocks(n2p * n2p + n * n2p, 256)), dim3(256), 0, s,
                     (int)n, (int)n2p, a, lda, A, V, conv);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int nblk = (int)(n2p / kBJ), npair = nblk / 2;
  const int vtiles = (int)((n + kBJTile - 1) / kBJTile);
  const unsigned ugrid = (unsigned)(npair * npair + vtiles * npair);
  const double tl = std::max(1e-15, 2.2e-16 * (double)n);
  for (int sw = 0; sw <= max_sweeps; ++sw) {
    hipLaunchKernelGGL(k_offnorm_part, dim3(kOffParts), dim3(256), 0, s, (int)n2p, (const cplx*)A,
                       dpart, (const int*)conv);
    hipLaunchKernelGGL(k_offnorm_final, dim3(1), dim3(kOffParts), 0, s, (const double*)dpart,
                       tl * tl, sw, conv);
    if (sw == max_sweeps) break;
    // round 0 from A; rounds 1 .. nblk - 2 each beside the previous round's
    // update (A -> A1 -> A ...: nblk - 2 copies, even); the last update in place
    hipLaunchKernelGGL(k_bj_inner, dim3(npair), dim3(kBJThreads), 0, s, (int)n2p, 0,
                       (const cplx*)A, Q0, (const int*)conv);
    cplx* cur = A;
    cplx* nxt = A1;
    for (int r = 1; r < nblk - 1; ++r) {
      hipLaunchKernelGGL(k_bj_step, dim3((unsigned)npair + ugrid), dim3(kBJUThreads), 0, s, (int)n,
                         (int)n2p, r, (const cplx*)cur, nxt, V, (const cplx*)(r & 1 ? Q0 : Q1),
                         r & 1 ? Q1 : Q0, (const int*)conv);
      std::swap(cur, nxt);
    }
    hipLaunchKernelGGL(k_bj_update, dim3(ugrid), dim3(kBJUThreads), 0, s, (int)n, (int)n2p,
                       nblk - 2, cur, V, (const cplx*)((nblk - 2) & 1 ? Q1 : Q0), (const int*)conv);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_jacobi_rank, dim3(nblocks(n, 256)), dim3(256), 0, s, (int)n, (int)n2p,
                     (const cplx*)A, rank, (const int*)conv, sweeps_dev);
  hipLaunchKernelGGL(k_jacobi_scatter, dim3(nblocks(n * n, 256)), dim3(256), 0, s, (int)n, (int)n2p,
                     (const cplx*)A, (const cplx*)V, (const int*)rank, w, q, ldq);
  return hipGetLastError();
}

hipError_t launch_heev(int64_t n, const cplx* a, int64_t lda, double* w, cplx* q, int64_t ldq,
                       void* work, int* sweeps_dev, int* host_scratch, int* sweeps_done,
                       hipStream_t s) {
  hipError_t e = launch_heev_async(n, a, lda, w, q, ldq, work, sweeps_dev, kMaxSweeps, s);
  if (e == hipSuccess) e = hipMemcpyAsync(host_scratch, sweeps_dev, sizeof(int), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e == hipSuccess) *sweeps_done = host_scratch[0];
  return e;
}

// First failure since the last clear wins: rec = {status, op, info}.
__global__ void k_status_record(const int* __restrict__ chol_status, const int* __restrict__ sweeps,
                                int op, int* __restrict__ rec) {
  if (threadIdx.x != 0 || rec[0] != 0) return;
  if (chol_status && chol_status[0] >= 0) {
    rec[0] = 5;   // PW_ERR_NOT_POSDEF
    rec[1] = op;
    rec[2] = chol_status[0];
  } else if (chol_status && chol_status[0] <= kCholNonFinite) {
    rec[0] = 6;   // PW_ERR_NONFINITE
    rec[1] = op;
    rec[2] = kCholNonFinite - chol_status[0];
  } else if (sweeps && sweeps[0] < 0) {
    rec[0] = 7;   // PW_ERR_NO_CONVERGENCE
    rec[1] = op;
    rec[2] = 0;
  }
}

__global__ void k_fill_int(int n, int v, int* __restrict__ p) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

hipError_t launch_status_record(const int* chol_status, const int* sweeps, int op, int* rec,
                                hipStream_t s) {
  hipLaunchKernelGGL(k_status_record, dim3(1), dim3(64), 0, s, chol_status, sweeps, op, rec);
  return hipGetLastError();
}

hipError_t launch_fill_int(int n, int v, int* p, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_int, dim3((n + 255) / 256), dim3(256), 0, s, n, v, p);
  return hipGetLastError();
}

// ---- fused-batch step launchers (npw_nb_max = max over items of npw * nb)
hipError_t launch_fused_dense(FusedStep step, int nitems, int64_t npw_nb_max, int nb_max,
                              const ItemDev* D, int arg0, int arg1, hipStream_t s) {
  if (nitems <= 0) return hipSuccess;
  const dim3 ew(nblocks(npw_nb_max, 256), nitems);
  switch (step) {
    case FS_CHEB_COEF:
      hipLaunchKernelGGL(kb_cheb_coef, dim3(nitems), dim3(64), 0, s, D, arg0);
      break;
    case FS_FILTER_FIRST:
      hipLaunchKernelGGL(kb_filter_first, ew, dim3(256), 0, s, D, arg0);
      break;
    case FS_TO_F32:
      hipLaunchKernelGGL(kb_to_f32, ew, dim3(256), 0, s, D);
      break;
    case FS_TO_F64:
      hipLaunchKernelGGL(kb_to_f64, ew, dim3(256), 0, s, D, arg0);
      break;
    case FS_COPY:
      hipLaunchKernelGGL(kb_copy, ew, dim3(256), 0, s, D, arg0, arg1);
      break;
    case FS_HERMITIZE:
      hipLaunchKernelGGL(kb_hermitize, dim3(nblocks((int64_t)nb_max * nb_max, 256), nitems),
                         dim3(256), 0, s, D);
      break;
    case FS_CHOL_INIT:
      hipLaunchKernelGGL(kb_chol_init, dim3(nitems), dim3(1024), 0, s, D);
      break;
    case FS_CHOL_DIAG:
      hipLaunchKernelGGL(kb_chol_diag, dim3(nitems), dim3(256),
                         (size_t)2 * nb_max * (nb_max + 1) * sizeof(cplx), s, D);
      break;
    case FS_JACOBI:
      hipLaunchKernelGGL(kb_jacobi, dim3(nitems), dim3(jac_threads(nb_max)),
                         jac_small_lds(nb_max), s, D);
      break;
    case FS_RESIDUALS:
      hipLaunchKernelGGL(kb_residuals, dim3(nb_max, nitems), dim3(256), 0, s, D);
      break;
    case FS_FLAGS:
      hipLaunchKernelGGL(kb_flags, dim3(nitems), dim3(64), 0, s, D);
      break;
  }
  return hipGetLastError();
}
