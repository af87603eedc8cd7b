// Plane kernels (FP64 and FP32) for boxes whose N1 and N2 each split into two
// factors N = P Q of at most 16 and hold the density's sphere (4 |m| <= N on
// both axes, the usual choice of box), whatever the two lengths are.
//
// A transform of length N is spread over L = max(P, Q) lanes in two steps with
// one exchange through LDS:
//   step 1: lane b < Q holds x[Q a + b] (a < P): a P-point DFT in registers
//           over a, the twiddle w_N^(b k1), stored as row k1 of the group's buffer;
//   step 2: lane k1 < P reads row k1: a Q-point DFT, outputs X[k1 + P k2].
// The forward transform runs the same steps backwards and leaves the layout
// step 1 started from, so a row of the plane goes backward, x V/N_box, forward
// with two exchanges.  Lanes of a group sit in one wavefront, whose LDS
// operations execute in order, so an exchange needs no barrier.  P >= Q, and
// the inputs of step 1 known to be zero (a with no |m| <= N/4) are literal
// zeros that the P-point DFT folds away; on the way back only the other
// outputs are formed.
//
// E[e][m2] in LDS holds the plane's extent columns between the axes.  N1 and
// N2 are chosen by a switch inside the kernel (uniform over the launch), so
// the two lengths combine freely with every transform's indexing known at
// compile time; the kernels are built for four bounds of P (registers).
#include "fft_common.h"

#include <algorithm>
#include <type_traits>

using namespace pwfft;

namespace {

// the lengths built, with their larger factor at most 8, 10, 12, 16
#define PQ_SIZES8(X) X(16) X(18) X(20) X(24) X(25) X(30) X(32) X(36) X(40) X(48) X(64)
#define PQ_SIZES10(X) X(27) X(45) X(50) X(54) X(60) X(72) X(80) X(81) X(90) X(100)
#define PQ_SIZES12(X) X(96) X(108) X(120) X(144)
#define PQ_SIZES16(X) X(75) X(128) X(135) X(150) X(160)
#define PQ_SIZES(X) PQ_SIZES8(X) PQ_SIZES10(X) PQ_SIZES12(X) PQ_SIZES16(X)

// larger factor of the split: the smallest divisor of n that is >= sqrt(n) and <= 16
constexpr int pq_p(int n) {
  for (int p = 1; p <= 16; ++p)
    if (p * p >= n && n % p == 0) return p;
  return 0;
}
constexpr int pq_lanes(int n) { return pq_p(n); }
constexpr int pq_groups(int n) { return 64 / pq_lanes(n); }
// Exchange buffer of one group: P rows of Q entries, row k at k Q + k / s.
// One entry more every s-th row (s Q a multiple of the period of the LDS banks)
// keeps the rows that step 2 reads side by side on distinct banks; an odd
// length staggers the groups.
// SPLIT (FP64 from P = 12 on): the real and the imaginary parts pass through
// the same buffer one after the other.  Twice the LDS instructions for the
// same bytes (FP64 80 x 80, 12 wavefronts: 0.96 against 0.84 ms), but half the
// buffer, without which the extent array of a long N2 leaves room for few
// wavefronts (FP64 120 x 120: 9 instead of 4, 1.36 against 1.74 ms; 144 x 144:
// 3 instead of 1, 1.73 against 4.1).
template <class C, bool SPLIT>
struct PqEntry {
  using type = C;
};
template <class C>
struct PqEntry<C, true> {
  using type = real_t<C>;
};
template <class C, bool SPLIT>
using pq_entry = typename PqEntry<C, SPLIT>::type;
template <class C, int PMAX>
constexpr bool pq_split() { return sizeof(C) == sizeof(double2) && PMAX >= 12; }
// for entries of `size` bytes
constexpr int pq_skip(int n, int size) {
  return 256 / size / gcd_ce(n / pq_p(n), 256 / size);
}
constexpr int pq_buf(int n, int size) { return (n + (pq_p(n) - 1) / pq_skip(n, size)) | 1; }

__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <class C, int N, bool SPLIT>
struct Pq {
  static constexpr int P = pq_p(N), Q = N / P, GPW = pq_groups(N);
  static constexpr int SKIP = pq_skip(N, sizeof(pq_entry<C, SPLIT>));
  static constexpr int BUF = pq_buf(N, sizeof(pq_entry<C, SPLIT>));
  using B = pq_entry<C, SPLIT>;
  __device__ __forceinline__ static int off(int k) { return k * Q + k / SKIP; }
  // some position Q a + b (b < Q) has a centred index in [-N/4, N/4]
  static constexpr bool live(int a) { return 4 * Q * a <= N || 4 * (Q * a + Q - 1) >= 3 * N; }

  C w[P - 1];   // lane b: exp(-2 pi i b k / N), k = 1 .. P - 1

  __device__ __forceinline__ void load(int lb, const C* __restrict__ tw) {
    const int b = lb < Q ? lb : 0;
#pragma unroll
    for (int k = 1; k < P; ++k) w[k - 1] = tw[b * k];
  }
  // in: lane b < Q holds x[Q a + b] in v[a] for live a (the others are zero);
  // out: lane k1 holds X[k1 + P k2] in v[k2]
  // bwd1 leaves the exchange half done (real parts, or all, in the buffer)
  __device__ __forceinline__ void bwd1(C (&v)[P], B* buf, int lb) const {
    if (Q == P || lb < Q) {
#pragma unroll
      for (int a = 0; a < P; ++a)
        if (!live(a)) v[a] = czero<C>();
      dft_reg<P, +1>(v);
#pragma unroll
      for (int k = 1; k < P; ++k) v[k] = conj_mul(v[k], w[k - 1]);
#pragma unroll
      for (int k = 0; k < P; ++k) {
        if constexpr (SPLIT) buf[off(k) + lb] = v[k].x;
        else buf[off(k) + lb] = v[k];
      }
    }
    wave_lds_fence();
  }
  __device__ __forceinline__ void bwd2(C (&v)[P], B* buf, int lb) const {
    if constexpr (SPLIT) {
#pragma unroll
      for (int b = 0; b < Q; ++b) v[b].x = buf[off(lb) + b];
      wave_lds_fence();
      if (Q == P || lb < Q) {
#pragma unroll
        for (int k = 0; k < P; ++k) buf[off(k) + lb] = v[k].y;
      }
      wave_lds_fence();
#pragma unroll
      for (int b = 0; b < Q; ++b) v[b].y = buf[off(lb) + b];
    } else {
#pragma unroll
      for (int b = 0; b < Q; ++b) v[b] = buf[off(lb) + b];
    }
    dft_reg<Q, +1>(v);
  }
  // in: lane k1 holds Z[k1 + P k2] in v[k2]; out: lane b < Q holds X'[Q a + b]
  // in v[a] (live a are used)
  __device__ __forceinline__ void fwd(C (&v)[P], B* buf, int lb) const {
    dft_reg<Q, -1>(v);
    if constexpr (SPLIT) {
#pragma unroll
      for (int b = 0; b < Q; ++b) buf[off(lb) + b] = v[b].x;
      wave_lds_fence();
      if (Q == P || lb < Q) {
#pragma unroll
        for (int k = 0; k < P; ++k) v[k].x = buf[off(k) + lb];
      }
      wave_lds_fence();
#pragma unroll
      for (int b = 0; b < Q; ++b) buf[off(lb) + b] = v[b].y;
      wave_lds_fence();
    } else {
#pragma unroll
      for (int b = 0; b < Q; ++b) buf[off(lb) + b] = v[b];
      wave_lds_fence();
    }
    if (Q == P || lb < Q) {
#pragma unroll
      for (int k = 0; k < P; ++k) {
        if constexpr (SPLIT) v[k].y = buf[off(k) + lb];
        else v[k] = buf[off(k) + lb];
      }
#pragma unroll
      for (int k = 1; k < P; ++k) v[k] = cmul(v[k], w[k - 1]);
      dft_reg<P, -1>(v);
    }
    wave_lds_fence();
  }
};

struct PqArgs {        // one wavefront's view of the workgroup
  int wave, nw, lane;
};

// Keeps what a phase derives from its lane and its twiddles inside the phase:
// without it the compiler moves the index arithmetic and the twiddle loads of
// every length of the switch out of the plane loop, and spills them.
__device__ __forceinline__ int pq_here(int lane) {
  asm volatile("" : "+v"(lane));
  return lane;
}
template <class C>
__device__ __forceinline__ const C* pq_here(const C* tw) {
  asm volatile("" : "+s"(tw));
  return tw;
}

// N2 transforms of the xr extent columns of E (column pitch trs), direction S,
// one column per lane group: column t + ceil(xr / GPW) g for group g, task t.
template <class C, int N, bool SPLIT, int S>
__device__ __forceinline__ void pq_cols(C* E, int trs, int xr, pq_entry<C, SPLIT>* wbuf, const C* __restrict__ tw,
                                        const PqArgs& A) {
  using F = Pq<C, N, SPLIT>;
  const int lane = pq_here(A.lane), g = lane / F::P, lb = lane - g * F::P;
  if (g >= F::GPW) return;
  pq_entry<C, SPLIT>* buf = wbuf + g * F::BUF;
  F f;
  f.load(lb, pq_here(tw));
  const int stride = (xr + F::GPW - 1) / F::GPW;
  for (int t = A.wave; t < stride; t += A.nw) {
    const int e = t + stride * g;
    if (e >= xr) continue;
    C* col = E + e * trs;
    C v[F::P];
    if constexpr (S > 0) {
      if (F::Q == F::P || lb < F::Q) {
#pragma unroll
        for (int a = 0; a < F::P; ++a)
          if (F::live(a)) v[a] = col[F::Q * a + lb];
      }
      f.bwd1(v, buf, lb);
      f.bwd2(v, buf, lb);
#pragma unroll
      for (int k = 0; k < F::Q; ++k) col[lb + F::P * k] = v[k];
      wave_lds_fence();
    } else {
#pragma unroll
      for (int k = 0; k < F::Q; ++k) v[k] = col[lb + F::P * k];
      f.fwd(v, buf, lb);
      if (F::Q == F::P || lb < F::Q) {
#pragma unroll
        for (int a = 0; a < F::P; ++a)
          if (F::live(a)) col[F::Q * a + lb] = v[a];
      }
    }
  }
}

// Rows of the plane: backward along N1, x V/N_box, forward along N1.
template <class C, int N, bool SPLIT>
__device__ __forceinline__ void pq_rows(C* E, int trs, int rows, pq_entry<C, SPLIT>* wbuf, const int* slot,
                                        const C* __restrict__ tw,
                                        const real_t<C>* __restrict__ vp, const PqArgs& A) {
  using F = Pq<C, N, SPLIT>;
  const int lane = pq_here(A.lane), g = lane / F::P, lb = lane - g * F::P;
  if (g >= F::GPW) return;
  pq_entry<C, SPLIT>* buf = wbuf + g * F::BUF;
  F f;
  f.load(lb, pq_here(tw));
  int sl[F::P];   // E offset of position Q a + lb, -1 outside the extent
#pragma unroll
  for (int a = 0; a < F::P; ++a)
    if (F::live(a)) {
      const int s = lb < F::Q ? slot[F::Q * a + lb] : -1;
      sl[a] = s >= 0 ? s * trs : -1;
    }
  const int stride = (rows + F::GPW - 1) / F::GPW;
  for (int t = A.wave; t < stride; t += A.nw) {
    const int row = t + stride * g;
    if (row >= rows) continue;
    C v[F::P];
    const real_t<C>* vr = vp + (size_t)row * N + lb;
    real_t<C> vv[F::Q];
#pragma unroll
    for (int a = 0; a < F::P; ++a)
      if (F::live(a)) v[a] = sl[a] >= 0 ? E[sl[a] + row] : czero<C>();
    f.bwd1(v, buf, lb);
#pragma unroll
    for (int k = 0; k < F::Q; ++k) vv[k] = vr[F::P * k];
    f.bwd2(v, buf, lb);
#pragma unroll
    for (int k = 0; k < F::Q; ++k) v[k] = cscale(v[k], vv[k]);
    f.fwd(v, buf, lb);
#pragma unroll
    for (int a = 0; a < F::P; ++a)
      if (F::live(a) && sl[a] >= 0) E[sl[a] + row] = v[a];
  }
}

// Rows of the plane, backward along N1 only: part[row][j1] (+)= wb |.|^2.  The
// element of a lane and task is the same for every band, so the sums in part
// (the workgroup's own, in its L2) have one writer.
template <class C, int N, bool SPLIT>
__device__ __forceinline__ void pq_rows_density(const C* E, int trs, int rows,
                                                pq_entry<C, SPLIT>* wbuf, const int* slot,
                                                const C* __restrict__ tw, double wb, bool fresh,
                                                double* part, const PqArgs& A) {
  using F = Pq<C, N, SPLIT>;
  const int lane = pq_here(A.lane), g = lane / F::P, lb = lane - g * F::P;
  if (g >= F::GPW) return;
  pq_entry<C, SPLIT>* buf = wbuf + g * F::BUF;
  F f;
  f.load(lb, pq_here(tw));
  int sl[F::P];
#pragma unroll
  for (int a = 0; a < F::P; ++a)
    if (F::live(a)) {
      const int s = lb < F::Q ? slot[F::Q * a + lb] : -1;
      sl[a] = s >= 0 ? s * trs : -1;
    }
  const int stride = (rows + F::GPW - 1) / F::GPW;
  for (int t = A.wave; t < stride; t += A.nw) {
    const int row = t + stride * g;
    if (row >= rows) continue;
    double* d = part + (size_t)row * N + lb;
    double old[F::Q];
#pragma unroll
    for (int k = 0; k < F::Q; ++k) old[k] = fresh ? 0.0 : d[F::P * k];
    C v[F::P];
#pragma unroll
    for (int a = 0; a < F::P; ++a)
      if (F::live(a)) v[a] = sl[a] >= 0 ? E[sl[a] + row] : czero<C>();
    f.bwd1(v, buf, lb);
    f.bwd2(v, buf, lb);
    wave_lds_fence();
#pragma unroll
    for (int k = 0; k < F::Q; ++k)
      d[F::P * k] = old[k] + wb * (v[k].x * v[k].x + v[k].y * v[k].y);
  }
}

// Columns of the sphere per thread kept in registers from one plane to the
// next (the next plane's are loaded while the current one is transformed);
// plans with more columns load the rest directly.
template <class C>
constexpr int pq_pre() { return sizeof(C) == sizeof(float2) ? 4 : 2; }

#define PQ_SWITCH_CASE(N) \
  case N:                 \
    if constexpr (pq_p(N) <= PMAX) { PQ_CALL(N); } \
    break;
#define PQ_SWITCH(n) \
  switch (n) { PQ_SIZES(PQ_SWITCH_CASE) }

// Planes L0, L0 + step, ... < Lend of T (plane L: band L / n3, z-plane L % n3).
// LDS: E (xr x trs), the wavefronts' exchange buffers (wbuf entries each), slots.
template <class C, int PMAX>
__device__ __forceinline__ void plane_pq_body(const BoxPlan& Pl, const C* __restrict__ tw1,
                                              const C* __restrict__ tw2,
                                              const real_t<C>* __restrict__ vs, C* __restrict__ T,
                                              int L0, int Lend, int step, int wbuf) {
  extern __shared__ __align__(16) char lds_raw[];
  constexpr bool SPLIT = pq_split<C, PMAX>();
  const int n1 = Pl.n1, n2 = Pl.n2, xr = Pl.xr, ncols = Pl.ncols, trs = n2 | 1;
  const int tid = threadIdx.x, nt = blockDim.x;
  C* E = reinterpret_cast<C*>(lds_raw);
  pq_entry<C, SPLIT>* X = reinterpret_cast<pq_entry<C, SPLIT>*>(E + (size_t)xr * trs);
  int* slot = reinterpret_cast<int*>(X + (size_t)(nt >> 6) * wbuf);
  PqArgs A;
  A.wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  A.nw = nt >> 6;
  A.lane = tid & 63;
  X += (size_t)A.wave * wbuf;
  for (int i = tid; i < n1; i += nt) slot[i] = -1;
  __syncthreads();
  for (int e = tid; e < xr; e += nt) slot[Pl.ext_m1[e]] = e;
  constexpr int kPqPre = pq_pre<C>();
  int cpos[kPqPre];
#pragma unroll
  for (int k = 0; k < kPqPre; ++k) {
    const int c = tid + k * nt;
    cpos[k] = c < ncols ? Pl.col_e[c] * trs + Pl.col_m2[c] : 0;
  }
  real_t<C> prex[kPqPre], prey[kPqPre];   // scalars: an array of C would live in scratch memory
  auto fetch = [&](int L) {
    if (L < Lend) {
      const C* tq = T + (size_t)L * Pl.ldt;
#pragma unroll
      for (int k = 0; k < kPqPre; ++k)
        if (tid + k * nt < ncols) {
          const C x = tq[tid + k * nt];
          prex[k] = x.x;
          prey[k] = x.y;
        }
    }
  };
  fetch(L0);
  // positions m2 that step 1 of the N2 transforms may read: [0, zlo) and [zhi, n2)
  const int zlo = min(n2, n2 / 4 + 16), zhi = max(zlo, n2 - n2 / 4 - 16), zn = zlo + n2 - zhi;
  for (int L = L0; L < Lend; L += step) {
    const int j3 = L % Pl.n3;
    C* tp = T + (size_t)L * Pl.ldt;
    __syncthreads();   // the previous plane's columns have left E
    for (int i = tid; i < xr * zn; i += nt) {
      const int e = i / zn, j = i - e * zn;
      E[e * trs + (j < zlo ? j : j - zlo + zhi)] = czero<C>();
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPqPre; ++k)
      if (tid + k * nt < ncols) {
        C x;
        x.x = prex[k];
        x.y = prey[k];
        E[cpos[k]] = x;
      }
    for (int c = tid + kPqPre * nt; c < ncols; c += nt)
      E[Pl.col_e[c] * trs + Pl.col_m2[c]] = tp[c];
    __syncthreads();
    fetch(L + step);
#define PQ_CALL(N) pq_cols<C, N, SPLIT, +1>(E, trs, xr, X, tw2, A)
    PQ_SWITCH(n2)
#undef PQ_CALL
    __syncthreads();
    const real_t<C>* vp = vs + (size_t)j3 * n2 * n1;
#define PQ_CALL(N) pq_rows<C, N, SPLIT>(E, trs, n2, X, slot, tw1, vp, A)
    PQ_SWITCH(n1)
#undef PQ_CALL
    __syncthreads();
#define PQ_CALL(N) pq_cols<C, N, SPLIT, -1>(E, trs, xr, X, tw2, A)
    PQ_SWITCH(n2)
#undef PQ_CALL
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPqPre; ++k)
      if (tid + k * nt < ncols) tp[tid + k * nt] = E[cpos[k]];
    for (int c = tid + kPqPre * nt; c < ncols; c += nt)
      tp[c] = E[Pl.col_e[c] * trs + Pl.col_m2[c]];
  }
}

// wavefronts per SIMD that the kernel's registers allow, and per workgroup
template <class C, int PMAX>
constexpr int pq_simd_waves() {
  return sizeof(C) == sizeof(float2) ? (PMAX <= 8 ? 5 : 4)
                                     : (PMAX <= 8 ? 4 : PMAX <= 12 ? 3 : 2);
}
template <class C, int PMAX>
constexpr int pq_max_waves() {
  return PMAX <= 8 ? 8 : std::min(16, 4 * pq_simd_waves<C, PMAX>());
}
#define PQ_BOUNDS_D \
  __launch_bounds__((64 * pq_max_waves<double2, PMAX>()), (pq_simd_waves<double2, PMAX>()))
#define PQ_BOUNDS __launch_bounds__((64 * pq_max_waves<C, PMAX>()), (pq_simd_waves<C, PMAX>()))

template <class C, int PMAX>
__global__ void PQ_BOUNDS
k_plane_pq(BoxPlan Pl, const C* __restrict__ tw1, const C* __restrict__ tw2,
           const real_t<C>* __restrict__ vs, C* __restrict__ T, int nplanes, int wbuf) {
  plane_pq_body<C, PMAX>(Pl, tw1, tw2, vs, T, blockIdx.x, nplanes, gridDim.x, wbuf);
}

// Electron density of one z-plane and band group: bands b = g, g + ngroup, ...
// of the chunk, backward along N2 and N1, w_b |.|^2 added to the group's
// partial array part[g][j3][j2][j1] (add: it already holds earlier chunks).
// Bound like the H*psi planes; 108 x 80 x 72, 192 bands: 2.64 ms with the
// general kernel, 0.64 here.
template <int PMAX>
__global__ void PQ_BOUNDS_D
k_density_pq(BoxPlan Pl, const double2* __restrict__ tw1, const double2* __restrict__ tw2,
             const double2* __restrict__ T, int nbc, const double* __restrict__ w, int ngroup,
             double* __restrict__ part, int add, int wbuf) {
  using C = double2;
  extern __shared__ __align__(16) char lds_raw[];
  constexpr bool SPLIT = pq_split<C, PMAX>();
  const int n1 = Pl.n1, n2 = Pl.n2, xr = Pl.xr, ncols = Pl.ncols, trs = n2 | 1;
  const int tid = threadIdx.x, nt = blockDim.x, j3 = blockIdx.x, g = blockIdx.y;
  C* E = reinterpret_cast<C*>(lds_raw);
  pq_entry<C, SPLIT>* X = reinterpret_cast<pq_entry<C, SPLIT>*>(E + (size_t)xr * trs);
  int* slot = reinterpret_cast<int*>(X + (size_t)(nt >> 6) * wbuf);
  PqArgs A;
  A.wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  A.nw = nt >> 6;
  A.lane = tid & 63;
  X += (size_t)A.wave * wbuf;
  double* pp = part + ((size_t)g * Pl.n3 + j3) * n2 * n1;
  if (g >= nbc && !add)   // a group without bands in the first chunk starts from zero
    for (int i = tid; i < n2 * n1; i += nt) pp[i] = 0.0;
  for (int i = tid; i < n1; i += nt) slot[i] = -1;
  __syncthreads();
  for (int e = tid; e < xr; e += nt) slot[Pl.ext_m1[e]] = e;
  const int zlo = min(n2, n2 / 4 + 16), zhi = max(zlo, n2 - n2 / 4 - 16), zn = zlo + n2 - zhi;
  bool fresh = !add;
  for (int b = g; b < nbc; b += ngroup) {
    const C* tp = T + ((size_t)b * Pl.n3 + j3) * Pl.ldt;
    __syncthreads();   // the previous band's rows are done with E
    for (int i = tid; i < xr * zn; i += nt) {
      const int e = i / zn, j = i - e * zn;
      E[e * trs + (j < zlo ? j : j - zlo + zhi)] = czero<C>();
    }
    __syncthreads();
    for (int c = tid; c < ncols; c += nt) E[Pl.col_e[c] * trs + Pl.col_m2[c]] = tp[c];
    __syncthreads();
#define PQ_CALL(N) pq_cols<C, N, SPLIT, +1>(E, trs, xr, X, tw2, A)
    PQ_SWITCH(n2)
#undef PQ_CALL
    __syncthreads();
    const double wb = w[b];
#define PQ_CALL(N) pq_rows_density<C, N, SPLIT>(E, trs, n2, X, slot, tw1, wb, fresh, pp, A)
    PQ_SWITCH(n1)
#undef PQ_CALL
    fresh = false;
  }
}

// fused batch: one plane per workgroup, item = blockIdx.z, lengths and tables from its descriptor
template <class C, int PMAX>
__global__ void PQ_BOUNDS
kb_plane_pq(const ItemDev* __restrict__ D, int wbuf) {
  const ItemDev& d = D[blockIdx.z];
  if ((int)blockIdx.y >= d.nb || (int)blockIdx.x >= d.plan.n3) return;
  const int L = blockIdx.y * d.plan.n3 + blockIdx.x;
  if constexpr (sizeof(C) == sizeof(double2))
    plane_pq_body<C, PMAX>(d.plan, d.plan.ax1.tw, d.plan.ax2.tw, d.vs, d.T, L, L + 1, 1, wbuf);
  else
    plane_pq_body<C, PMAX>(d.plan, d.plan.ax1.tw32, d.plan.ax2.tw32, d.vs32, d.T32, L, L + 1, 1, wbuf);
}

size_t g_pq_lds_limit = 64 * 1024;
int g_pq_cus = 256;

int pq_axis_p(int n) {
#define CASE(N) if (n == N) return pq_p(N);
  PQ_SIZES(CASE)
#undef CASE
  return 0;
}

// f with the kernel bound PMAX for the larger factor p of a box as std::integral_constant
template <class F>
auto pq_dispatch(int p, const F& f) {
  if (p <= 8) return f(std::integral_constant<int, 8>{});
  if (p <= 10) return f(std::integral_constant<int, 10>{});
  if (p <= 12) return f(std::integral_constant<int, 12>{});
  return f(std::integral_constant<int, 16>{});
}
int pq_box_p(const BoxPlan& p) { return std::max(pq_axis_p(p.n1), pq_axis_p(p.n2)); }

// exchange buffers of one wavefront, in entries, for both axes and the kernel bound pmax
template <class C>
int pq_wave_buf(int n1, int n2, int pmax) {
  const int size = pq_dispatch(pmax, [](auto pm) {
    return (int)sizeof(pq_entry<C, pq_split<C, pm.value>()>);
  });
  int w = 0;
#define CASE(N) if (n1 == N || n2 == N) w = std::max(w, pq_groups(N) * pq_buf(N, size));
  PQ_SIZES(CASE)
#undef CASE
  return w;
}

template <class C>
size_t pq_lds_bytes(int extent_entries, int waves, int wbuf, int n1, int pmax) {
  const size_t size = pq_dispatch(pmax, [](auto pm) {
    return sizeof(pq_entry<C, pq_split<C, pm.value>()>);
  });
  return (size_t)extent_entries * sizeof(C) + (size_t)waves * wbuf * size + (size_t)n1 * sizeof(int);
}
template <class C>
size_t pq_lds(const BoxPlan& p, int waves) {
  const int pm = pq_box_p(p);
  return pq_lds_bytes<C>(p.xr * (p.n2 | 1), waves, pq_wave_buf<C>(p.n1, p.n2, pm), p.n1, pm);
}

// Wavefronts per workgroup and workgroups per CU.  The wavefronts of one
// workgroup pass the same phases (LDS bound, then arithmetic bound) together,
// so several workgroups overlap better than one large one; three or more
// take four wavefronts each or two, which loads the SIMDs evenly (two, what
// fits if the same SIMD takes both their odd wavefronts).  Of
// the shapes that the LDS (handed out in units of 1280 bytes) holds, the one
// with the most wavefronts x weight; the weights are fitted to sweeps of
// 22 boxes, in which the shape chosen stays within 8% of the best.  Examples,
// workgroups x wavefronts: FP32 96 x 96 3 x 4 0.63 ms, 2 x 8 0.64, 1 x 16 0.84;
// FP32 36 x 40 8 x 2 0.088, 4 x 4 0.109, 2 x 8 0.156; FP32 120 x 120 2 x 4 (half
// the wavefronts) 0.78, 1 x 16 0.76; FP32 108 x 64 3 x 4 0.45, 4 x 3 0.58.
constexpr int kPqMaxWg = 8;
constexpr double kPqWeight[kPqMaxWg + 1] = {0.0, 0.6, 1.0, 1.35, 1.4, 1.5, 1.6, 1.65, 1.7};

template <class C>
void pq_shape(const BoxPlan& p, size_t lds_limit, int* waves, int* per_cu) {
  const int gpw = 64 / pq_axis_p(p.n1), tasks = (p.n2 + gpw - 1) / gpw;
  const int cu = pq_dispatch(pq_box_p(p), [](auto pm) { return 4 * pq_simd_waves<C, pm.value>(); });
  const int wmax = pq_dispatch(pq_box_p(p), [](auto pm) { return pq_max_waves<C, pm.value>(); });
  double best = 0.0;
  *waves = *per_cu = 0;
  for (int wg = 1; wg <= kPqMaxWg; ++wg) {
    int nw = std::min({cu / wg, wmax, tasks});
    while (nw > 0 && wg * ((pq_lds<C>(p, nw) + 1279) / 1280 * 1280) > lds_limit) --nw;
    if (wg == 2)
      while (nw > 2 && wg * ((nw + 3) / 4) > cu / 4) --nw;
    else if (wg > 2)
      nw = nw >= 4 ? nw / 4 * 4 : nw & 2;
    if (wg * nw * kPqWeight[wg] > best) {
      best = wg * nw * kPqWeight[wg];
      *waves = nw;
      *per_cu = wg;
    }
  }
}

template <class C>
hipError_t plane_pq(const BoxPlan& p, int nb, const real_t<C>* vs, const C* tw1, const C* tw2, C* T,
                    hipStream_t s) {
  int waves, per_cu;
  pq_shape<C>(p, g_pq_lds_limit, &waves, &per_cu);
  if (waves < 1) return hipErrorInvalidValue;
  if (nb <= 0) return hipSuccess;
  const size_t lds = pq_lds<C>(p, waves);
  const int64_t nplanes = (int64_t)p.n3 * nb;
  const dim3 grid((unsigned)std::min<int64_t>(nplanes, (int64_t)g_pq_cus * per_cu));
  const int wbuf = pq_wave_buf<C>(p.n1, p.n2, pq_box_p(p));
  pq_dispatch(pq_box_p(p), [&](auto pm) {
    hipLaunchKernelGGL((k_plane_pq<C, pm.value>), grid, dim3(64 * waves), lds, s, p, tw1, tw2, vs, T,
                       (int)nplanes, wbuf);
  });
  return hipGetLastError();
}

}  // namespace

bool fft_plane_pq_supported(const BoxPlan& p, bool fp32, size_t lds_limit) {
  if (!p.holds12 || !pq_axis_p(p.n1) || !pq_axis_p(p.n2)) return false;
  int waves, per_cu;
  if (fp32) pq_shape<float2>(p, lds_limit, &waves, &per_cu);
  else pq_shape<double2>(p, lds_limit, &waves, &per_cu);
  return waves >= 1;
}

hipError_t launch_fft_plane_pq(const BoxPlan& p, int nb, const double* vscaled, cplx* T,
                               hipStream_t s) {
  return plane_pq<double2>(p, nb, vscaled, p.ax1.tw, p.ax2.tw, T, s);
}
hipError_t launch_fft_plane_pq32(const BoxPlan& p, int nb, const float* vscaled, float2* T,
                                 hipStream_t s) {
  return plane_pq<float2>(p, nb, vscaled, p.ax1.tw32, p.ax2.tw32, T, s);
}

// Square boxes that also have a lane-shuffle kernel (fft_reg.hip): whether the
// two-factor kernel is the faster one.  Measured over 24 .. 144 (1e8 to 2e8 box
// points x bands, two-factor against lane-shuffle): FP32 36 72 against 106 us,
// 48 170 / 211, 64 440 / 475, 72 620 / 870, 96 630 / 680, 120 750 / 1120, 144 640 /
// 730, but 24 44 / 37, 32 slower, 128 (16 x 8, half the lanes idle in one step)
// 890 / 790; FP64 36 128 / 164, 72 1190 / 1740, elsewhere the exchange through
// LDS costs what it saves in arithmetic: 48 320 / 320, 64 830 / 830, 96 1220 /
// 1060, 120 1470 / 1500, 144 1730 / 1400.
bool fft_plane_pq_wins(int n, bool fp32) {
  return fp32 ? n >= 36 && n != 128 && n != 160 : n == 36 || n == 72;
}

bool fft_plane_pq_large(const BoxPlan& p) { return (size_t)p.xr * (p.n2 | 1) * sizeof(double2) > 65536; }

void fused_pq_add(FusedFft* f, const BoxPlan& p) {
  int waves, per_cu;
  pq_shape<double2>(p, g_pq_lds_limit, &waves, &per_cu);
  if (waves == 0) pq_shape<float2>(p, g_pq_lds_limit, &waves, &per_cu);   // an FP32-only box
  f->pq_pmax = std::max(f->pq_pmax, pq_box_p(p));
  f->pq_waves = std::max(f->pq_waves, waves);
  for (int pm : {8, 16})   // 16-byte and 8-byte entries
    f->pq_wbuf = std::max(f->pq_wbuf, pq_wave_buf<double2>(p.n1, p.n2, pm));
  f->pq_e = std::max(f->pq_e, p.xr * (p.n2 | 1));
  f->pq_n1 = std::max(f->pq_n1, p.n1);
}

namespace {
template <class C>
hipError_t fused_plane_pq(const FusedFft& f, const ItemDev* D, hipStream_t s) {
  // the items' largest extent array, buffers and table together may exceed
  // what one of them needs: fewer wavefronts then (one always fits: an item
  // with a large extent array only shares its group with its own lengths)
  auto bytes = [&](int w) {
    return pq_lds_bytes<C>(f.pq_e, w, f.pq_wbuf, f.pq_n1, f.pq_pmax);
  };
  int waves = std::min(f.pq_waves, pq_dispatch(f.pq_pmax, [](auto pm) {
    return pq_max_waves<C, pm.value>();
  }));
  while (waves > 1 && bytes(waves) > g_pq_lds_limit) --waves;
  if (waves < 1 || bytes(waves) > g_pq_lds_limit) return hipErrorInvalidValue;
  const dim3 grid(f.n3_max, f.nb_max, f.nitems);
  pq_dispatch(f.pq_pmax, [&](auto pm) {
    hipLaunchKernelGGL((kb_plane_pq<C, pm.value>), grid, dim3(64 * waves), bytes(waves), s, D,
                       f.pq_wbuf);
  });
  return hipGetLastError();
}
}  // namespace

hipError_t launch_fused_plane_pq(const FusedFft& f, bool fp32, const ItemDev* D, hipStream_t s) {
  return fp32 ? fused_plane_pq<float2>(f, D, s) : fused_plane_pq<double2>(f, D, s);
}

// Square planes, against the register kernel of density.hip (same sizes as
// above): 36 97 against 221 us, 72 970 / 1060, 128 1270 / 1560; the others 24 45 /
// 43, 48 231 / 221, 64 653 / 518, 96 976 / 923, 120 1055 / 1067, 144 1253 / 1163.
bool density_pq_wins(int n) { return n == 36 || n == 72 || n == 128; }

int density_pq_groups(const BoxPlan& p, int cus, int most) {
  int waves, per_cu;
  pq_shape<double2>(p, g_pq_lds_limit, &waves, &per_cu);
  return std::max(1, std::min(most, 4 * cus * per_cu / p.n3));
}

hipError_t launch_density_planes_pq(const BoxPlan& p, int nbc, const cplx* T, const double* w,
                                    int ngroup, double* part, int add, hipStream_t s) {
  int waves, per_cu;
  pq_shape<double2>(p, g_pq_lds_limit, &waves, &per_cu);
  if (waves < 1) return hipErrorInvalidValue;
  const size_t lds = pq_lds<double2>(p, waves);
  const int wbuf = pq_wave_buf<double2>(p.n1, p.n2, pq_box_p(p));
  pq_dispatch(pq_box_p(p), [&](auto pm) {
    hipLaunchKernelGGL((k_density_pq<pm.value>), dim3(p.n3, ngroup), dim3(64 * waves), lds, s, p,
                       p.ax1.tw, p.ax2.tw, T, nbc, w, ngroup, part, add, wbuf);
  });
  return hipGetLastError();
}

hipError_t fft_pq_set_lds_limit(size_t bytes) {
  g_pq_lds_limit = bytes;
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) == hipSuccess &&
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && cus > 0)
    g_pq_cus = cus;
#define FN(C, PM) (const void*)k_plane_pq<C, PM>, (const void*)kb_plane_pq<C, PM>
  const void* fns[20] = {(const void*)k_density_pq<8>, (const void*)k_density_pq<10>,
                         (const void*)k_density_pq<12>, (const void*)k_density_pq<16>,
                         FN(double2, 8), FN(float2, 8), FN(double2, 10), FN(double2, 12), FN(double2, 16),
                         FN(float2, 10),  FN(float2, 12),  FN(float2, 16)};
#undef FN
  for (const void* f : fns) {
    hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}
