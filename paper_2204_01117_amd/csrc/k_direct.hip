// Direct solution of the pressure system A x = b (the 7-point negative
// Laplacian on a box, Neumann or zero-ghost outlet sides) for the multigrid
// configuration's solves: A is a sum of one-dimensional operators whose
// eigenvectors are sines and cosines known in closed form, so
//
//   1. z and y are transformed to their eigenvectors by dense products on
//      the matrix cores (k_ds_row over the z rows, k_ds_col over y),
//   2. every (y mode, z mode) is a tridiagonal system along x (k_ds_tri),
//   3. the products back give z = A^-1 r up to the rounding of the products,
//   4. k_ds_finish forms the residual r - A z, removes most of it (it is
//      grid-scale rounding noise) with one damped-Jacobi sweep e, adds z + e
//      to the iterate and sums the residual that is left.
//
// That is one iteration; the solve stops, as the CG does, on
// ||r|| <= tol ||b|| of the recursively updated residual.  Most FP32 steps
// need one; where a large grid's first leaves a few times the threshold, the
// next is two more sweeps instead of products (k_ds_finish, SMOOTH).  The products cost 4 (ny + nz) flops
// per cell and iteration (FP32 on the matrix cores: 157 TFLOP/s nominal),
// a CG iteration moves about 55 bytes per cell: see direct_use for where
// the line between the two lies.
//
// Layouts: the residual and z are padded cell arrays; between the products
// the values sit in W[y][x][z] (x, z contiguous, row stride ldw), so that
// the product over y is one (ny x ny) x (ny x nx nz) product whatever the
// sizes, and the tridiagonal solve reads rows of z.
#include <cmath>
#include <vector>

#include "pressure_common.h"

namespace uf {

constexpr int kDsThreads = 256;
constexpr double kDsOmega = 0.75;   // Jacobi weight of the closing sweep (0.7 to 0.85: within 10%)
// Weights of the two sweeps of a smoothing iteration, and the multiple of the
// threshold that it is trusted to remove: 5.3 to 5.8 of white noise, 3.3 to
// 4.7 measured on grids of 17x33x31 to 512x6x8 cells, whose noise is smoother;
// where it falls short a third iteration, of products, follows.
constexpr double kDsOmegaZ = 0.563, kDsOmegaE = 1.485, kDsReach = 4.5;

// Matrix-core tile of a type: MT x MT results, KT terms per instruction.
// Lane l supplies A[l % MT][l / MT] and B[l / MT][l % MT] and holds column
// l % MT of the result; row() is the row of its register q.
template <class T>
struct Mfma;
template <>
struct Mfma<float> {
  static constexpr int MT = 32, KT = 2, NR = 16, BK = 16, VEC = 4;
  typedef float Acc __attribute__((ext_vector_type(16)));
  typedef float Vec __attribute__((ext_vector_type(4)));
  __device__ static __forceinline__ Acc mul(float a, float b, Acc c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
  }
  __device__ static __forceinline__ int row(int q, int hi) { return 8 * (q >> 2) + 4 * hi + (q & 3); }
};
template <>
struct Mfma<double> {
  static constexpr int MT = 16, KT = 4, NR = 4, BK = 8, VEC = 2;
  typedef double Acc __attribute__((ext_vector_type(4)));
  typedef double Vec __attribute__((ext_vector_type(2)));
  __device__ static __forceinline__ Acc mul(double a, double b, Acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  __device__ static __forceinline__ int row(int q, int hi) { return 4 * q + hi; }
};

// A block of four wavefronts (2 x 2) computes a BM x BN tile, each wavefront
// WM x WN matrix-core tiles of it, from BK-deep slices staged in LDS twice
// (the next slice is loaded into registers while the current one is
// multiplied, and stored to the other buffer: one barrier per slice).
template <class T, int WM_, int WN_>
struct DsTile {
  static constexpr int WM = WM_, WN = WN_;
  static constexpr int BM = 2 * WM * Mfma<T>::MT, BN = 2 * WN * Mfma<T>::MT, BK = Mfma<T>::BK;
  // LDS row strides: the lanes of one fragment read 64 / MT rows at once,
  // which fall into different halves of the banks
  static constexpr int SN = BN + Mfma<T>::MT, SM = BM + Mfma<T>::MT;
};

template <class T, int WM, int WN>
__device__ __forceinline__ void ds_mul(const T* __restrict__ As, int sa, const T* __restrict__ Bs, int sb, int m0,
                                       int n0, typename Mfma<T>::Acc (&acc)[WM][WN]) {
  using X = Mfma<T>;
  const int l = threadIdx.x & 63, lo = l % X::MT, hi = l / X::MT;
#pragma unroll
  for (int k = 0; k < X::BK; k += X::KT) {
    T a[WM], b[WN];
#pragma unroll
    for (int p = 0; p < WM; ++p) a[p] = As[(k + hi) * sa + m0 + p * X::MT + lo];
#pragma unroll
    for (int q = 0; q < WN; ++q) b[q] = Bs[(k + hi) * sb + n0 + q * X::MT + lo];
#pragma unroll
    for (int p = 0; p < WM; ++p)
#pragma unroll
      for (int q = 0; q < WN; ++q) acc[p][q] = X::mul(a[p], b[q], acc[p][q]);
  }
}

// The forward product over y sums the cells in their order; its rounding,
// relative to the partial sums, is an error of every mode alike, which the
// division by the eigenvalues turns into an error of the smooth modes (1e-6
// of the FP32 pressure at 256x256x64).  In FP32 (SPLIT) it therefore sums
// kDsChain slices (64 terms) at a time and those sums among themselves:
// from about sqrt(K / 4) roundings to 4, and 3e-7 there.
constexpr int kDsChain = 4;

template <class T, int WM, int WN>
__device__ __forceinline__ void ds_fold(typename Mfma<T>::Acc (&acc)[WM][WN], typename Mfma<T>::Acc (&tot)[WM][WN]) {
#pragma unroll
  for (int p = 0; p < WM; ++p)
#pragma unroll
    for (int q = 0; q < WN; ++q) {
      tot[p][q] += acc[p][q];
      acc[p][q] = typename Mfma<T>::Acc{};
    }
}

// Is there nothing for the transforms of the iteration to do?
__device__ __forceinline__ bool ds_idle(const CgState* st) { return st->done || st->smooth; }

// C[m][n] = sum_k At[k][m] B[k][n], m < M, n < N, k < K: the transform over
// y.  At is padded with zeros to multiples of BK rows and 128 columns; B and
// C have row stride ldw (a multiple of the vector width).
template <class T, int WM, int WN, bool SPLIT>
__global__ __launch_bounds__(kDsThreads) void k_ds_col(const T* __restrict__ At, int lda, const T* __restrict__ B,
                                                       T* __restrict__ C, int M, int K, int N, long long ldw, int mt,
                                                       int nt, const CgState* __restrict__ st) {
  using X = Mfma<T>;
  using D = DsTile<T, WM, WN>;
  using Vec = typename X::Vec;
  __shared__ __align__(16) T As[2][D::BK * D::SM];
  __shared__ __align__(16) T Bs[2][D::BK * D::SN];
  if (ds_idle(st)) return;   // uniform over the grid
  int bm, bn;
  if (!xcd_block(mt, nt, bm, bn)) return;   // the tiles of one column of B run together
  const int tid = threadIdx.x, m0 = bm * D::BM, n0 = bn * D::BN;
  constexpr int RA = D::BM / X::VEC, RB = D::BN / X::VEC;   // vectors per slice row
  constexpr int VA = (D::BK * RA + kDsThreads - 1) / kDsThreads, VB = (D::BK * RB + kDsThreads - 1) / kDsThreads;
  Vec ra[VA], rb[VB];
  auto load = [&](int k0) {
#pragma unroll
    for (int v = 0; v < VA; ++v) {
      const int q = min(tid + v * kDsThreads, D::BK * RA - 1), k = q / RA, m = (q % RA) * X::VEC;
      ra[v] = *reinterpret_cast<const Vec*>(At + (long long)(k0 + k) * lda + m0 + m);
    }
#pragma unroll
    for (int v = 0; v < VB; ++v) {
      const int q = min(tid + v * kDsThreads, D::BK * RB - 1);
      const int k = min(k0 + q / RB, K - 1);   // rows past K meet zeros of At
      const long long n = min((long long)n0 + (q % RB) * X::VEC, ldw - X::VEC);
      rb[v] = *reinterpret_cast<const Vec*>(B + k * ldw + n);
    }
  };
  auto store = [&](int s) {
#pragma unroll
    for (int v = 0; v < VA; ++v) {
      const int q = tid + v * kDsThreads;
      if (q < D::BK * RA) *reinterpret_cast<Vec*>(&As[s][(q / RA) * D::SM + (q % RA) * X::VEC]) = ra[v];
    }
#pragma unroll
    for (int v = 0; v < VB; ++v) {
      const int q = tid + v * kDsThreads;
      if (q < D::BK * RB) *reinterpret_cast<Vec*>(&Bs[s][(q / RB) * D::SN + (q % RB) * X::VEC]) = rb[v];
    }
  };
  const int w = tid >> 6, wm = (w >> 1) * WM * X::MT, wn = (w & 1) * WN * X::MT;
  typename X::Acc acc[WM][WN] = {}, tot[SPLIT ? WM : 1][SPLIT ? WN : 1] = {};
  load(0);
  store(0);
  __syncthreads();
  int s = 0, c = 0;
  for (int k0 = 0; k0 < K; k0 += D::BK, s ^= 1) {
    const bool more = k0 + D::BK < K;
    if (more) load(k0 + D::BK);
    ds_mul<T, WM, WN>(As[s], D::SM, Bs[s], D::SN, wm, wn, acc);
    if constexpr (SPLIT) {
      if (++c == kDsChain || !more) {
        ds_fold<T, WM, WN>(acc, tot);
        c = 0;
      }
    }
    if (more) store(s ^ 1);
    __syncthreads();
  }
  const int l = tid & 63, lo = l % X::MT, hi = l / X::MT;
#pragma unroll
  for (int p = 0; p < WM; ++p)
#pragma unroll
    for (int q = 0; q < WN; ++q) {
      const int n = n0 + wn + q * X::MT + lo;
      if (n >= N) continue;
#pragma unroll
      for (int e = 0; e < X::NR; ++e) {
        const int m = m0 + wm + p * X::MT + X::row(e, hi);
        if (m < M) C[m * ldw + n] = SPLIT ? tot[SPLIT ? p : 0][SPLIT ? q : 0][e] : acc[p][q][e];
      }
    }
}

// The transform over z: row (i, j) of length nz times the nz x nz matrix E
// (E[k][n], padded with zeros to multiples of BK rows and 128 columns).
// FWD: from the padded array to W; otherwise back from W to the padded
// array.  Rows are numbered j fastest, as the padded array holds them.
// The loads of a row are scalar: padded rows have no common alignment.
template <class T, int WM, int WN, bool FWD>
__global__ __launch_bounds__(kDsThreads) void k_ds_row(Layout L, const T* __restrict__ in, T* __restrict__ out,
                                                       const T* __restrict__ E, int lde, long long ldw, int mt,
                                                       int nt, const CgState* __restrict__ st) {
  using X = Mfma<T>;
  using D = DsTile<T, WM, WN>;
  using Vec = typename X::Vec;
  constexpr int SA = D::BM + 36;   // transposing stores of 16 (k) x 4 (rows) lanes hit distinct banks
  __shared__ __align__(16) T As[2][D::BK * SA];
  __shared__ __align__(16) T Bs[2][D::BK * D::SN];
  if (ds_idle(st)) return;
  int bn, bm;
  if (!xcd_block(nt, mt, bn, bm)) return;
  const int nz = L.nz, M = L.nx * L.ny;
  const int tid = threadIdx.x, m0 = bm * D::BM, n0 = bn * D::BN;
  constexpr int RP = kDsThreads / D::BK, VA = D::BM / RP;   // rows per pass, passes
  constexpr int RB = D::BN / X::VEC, VB = (D::BK * RB + kDsThreads - 1) / kDsThreads;
  static_assert(VA >= 1, "a slice fills the block's row loads");
  auto padded = [&](int m) { return L.at(m / L.ny, m % L.ny, 0); };
  auto packed = [&](int m) { return (long long)(m % L.ny) * ldw + (long long)(m / L.ny) * nz; };
  const int ak = tid % D::BK, ar = tid / D::BK;
  long long base[VA];
#pragma unroll
  for (int v = 0; v < VA; ++v) {
    const int m = min(m0 + ar + v * RP, M - 1);
    base[v] = FWD ? padded(m) : packed(m);
  }
  T ra[VA];
  Vec rb[VB];
  auto load = [&](int k0) {
    const int k = min(k0 + ak, nz - 1);   // columns past nz meet zeros of E
#pragma unroll
    for (int v = 0; v < VA; ++v) ra[v] = in[base[v] + k];
#pragma unroll
    for (int v = 0; v < VB; ++v) {
      const int q = min(tid + v * kDsThreads, D::BK * RB - 1);
      rb[v] = *reinterpret_cast<const Vec*>(E + (long long)(k0 + q / RB) * lde + n0 + (q % RB) * X::VEC);
    }
  };
  auto store = [&](int s) {
#pragma unroll
    for (int v = 0; v < VA; ++v) As[s][ak * SA + ar + v * RP] = ra[v];
#pragma unroll
    for (int v = 0; v < VB; ++v) {
      const int q = tid + v * kDsThreads;
      if (q < D::BK * RB) *reinterpret_cast<Vec*>(&Bs[s][(q / RB) * D::SN + (q % RB) * X::VEC]) = rb[v];
    }
  };
  const int w = tid >> 6, wm = (w >> 1) * WM * X::MT, wn = (w & 1) * WN * X::MT;
  typename X::Acc acc[WM][WN] = {};
  load(0);
  store(0);
  __syncthreads();
  int s = 0;
  for (int k0 = 0; k0 < nz; k0 += D::BK, s ^= 1) {
    const bool more = k0 + D::BK < nz;
    if (more) load(k0 + D::BK);
    ds_mul<T, WM, WN>(As[s], SA, Bs[s], D::SN, wm, wn, acc);
    if (more) store(s ^ 1);
    __syncthreads();
  }
  const int l = tid & 63, lo = l % X::MT, hi = l / X::MT;
#pragma unroll
  for (int p = 0; p < WM; ++p)
#pragma unroll
    for (int e = 0; e < X::NR; ++e) {
      const int m = m0 + wm + p * X::MT + X::row(e, hi);
      if (m >= M) continue;
      T* o = out + (FWD ? packed(m) : padded(m));
#pragma unroll
      for (int q = 0; q < WN; ++q) {
        const int n = n0 + wn + q * X::MT + lo;
        if (n < nz) o[n] = acc[p][q][e];
      }
    }
}

__device__ __forceinline__ double powi(double r, int e) {
  double p = 1.0;
  for (; e > 0; e >>= 1) {
    if (e & 1) p *= r;
    r *= r;
  }
  return p;
}

// The tridiagonal systems along x, in place: -w x_{i-1} + d x_i - w x_{i+1}
// = b_i with d = 2w + lambda, less w in the first and last row at a Neumann
// side.  With r the root of r^2 - (d/w) r + 1 below 1,
//   F = (w/r) (I - r S)(I - r S^T)   (S the shift down)
// is the matrix up to its first and last diagonal entry (w/r and d), so the
// solve is two first-order recurrences, y_i = b_i + r y_{i-1} and x_i =
// (r/w) y_i + r x_{i+1}, and a 2 x 2 system for the two entries' corrections
// cl x_0 and cr x_{n-1}, which are then sources in those rows.
//
// A line's rows are shared out to the wavefronts of a block, LC rows each,
// all loaded at once; the recurrences cross from one to the next by their
// end values (r^LC times the one before), kept in LDS.  One read and one
// write of the array.  The recurrences run in FP64 also for FP32 arrays:
// for the smooth modes 1 - r is a few 1e-3 and its rounding in FP32 would be
// a change of the eigenvalue by 1e-4 of itself.
template <class T, int LC>
__global__ __launch_bounds__(1024) void k_ds_tri(T* __restrict__ W, int n, int nlines, int nz, long long ldw,
                                                 double w, const double* __restrict__ lamy,
                                                 const double* __restrict__ lamz, int open_lo, int open_hi,
                                                 const CgState* __restrict__ st) {
  __shared__ double shy[16][64], shx[16][64], shn[64];
  if (ds_idle(st)) return;
  const int lane = threadIdx.x & 63, c = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nc = blockDim.x >> 6;
  const int line = blockIdx.x * 64 + lane, ln = min(line, nlines - 1);
  const int j = ln / nz, k = ln - j * nz, s = c * LC;
  const int cnt = min(LC, n - s);   // this wavefront's rows
  T* row = W + (long long)s * nz;
  const unsigned off = (unsigned)j * (unsigned)ldw + (unsigned)k;   // arrays below 4 GiB (direct_use)
  T v[LC];
#pragma unroll
  for (int u = 0; u < LC; ++u) v[u] = u < cnt ? (row + (long long)u * nz)[off] : T(0);
  const double lam = lamy[j] + lamz[k], dl = lam / (2.0 * w);
  const double r = 1.0 / (1.0 + dl + sqrt(dl * (2.0 + dl))), kap = r / w;
  double rl = r;
#pragma unroll
  for (int q = 1; q < LC; q *= 2) rl *= rl;   // r^LC
  double y = 0.0;
#pragma unroll
  for (int u = 0; u < LC; ++u)
    if (u < cnt) y = (double)v[u] + r * y;
  shy[c][lane] = y;
  __syncthreads();
  y = 0.0;
  for (int q = 0; q < c; ++q) y = shy[q][lane] + rl * y;
#pragma unroll
  for (int u = 0; u < LC; ++u)
    if (u < cnt) {
      y = (double)v[u] + r * y;
      v[u] = (T)y;
    }
  double x = 0.0;
#pragma unroll
  for (int u = LC - 1; u >= 0; --u) x = kap * (double)v[u] + r * x;
  shx[c][lane] = x;
  if (c == nc - 1) shn[lane] = y;
  __syncthreads();
  double x0 = 0.0;
  x = 0.0;
  for (int q = nc - 1; q >= 0; --q) {
    if (q == c) x = x0;   // the first row past this wavefront's
    x0 = shx[q][lane] + rl * x0;
  }
  // the two diagonal corrections: (I + G C) X = X^ with G the entries of F^-1
  const double xn = kap * shn[lane], rn = powi(r, n), om = 1.0 - r * r;
  const double cl = open_lo ? w * r : -w * (1.0 - r), cr = open_hi ? 0.0 : -w;
  const double u0 = kap * (lam > 0.0 ? (1.0 - rn * rn) / om : (double)n), un = kap * powi(r, n - 1);
  const double m00 = 1.0 + u0 * cl, m01 = un * cr, m10 = un * cl, m11 = 1.0 + kap * cr;
  const double det = m00 * m11 - m01 * m10;
  const double e0 = -cl * (m11 * x0 - m01 * xn) / det, en = -cr * (m00 * xn - m10 * x0) / det;
  const int t = s + LC;   // the row past this wavefront's
  const double pc = powi(rl, c);
  if (t < n) {
    const double ut = kap * (lam > 0.0 ? (pc * rl - rn * powi(r, n - t)) / om : (double)(n - t));
    x += e0 * ut + en * kap * powi(r, n - 1 - t);
  }
  double pw = e0 * pc;
#pragma unroll
  for (int u = 0; u < LC; ++u) {
    if (u < cnt) v[u] = (T)((double)v[u] + (s + u == n - 1 ? pw + en : pw));
    pw *= r;
  }
#pragma unroll
  for (int u = LC - 1; u >= 0; --u) {
    x = kap * (double)v[u] + r * x;
    if (u < cnt && line < nlines) (row + (long long)u * nz)[off] = (T)x;
  }
}

// ------------------------------------------------------- closing sweep -----
// r1 = r - A z, e = om D^-1 r1, x += z + e and the partials of ||r1 - A e||^2,
// marching along x: a block owns FJ x FK columns over a chunk of planes and
// keeps z (two cells around) and e (one cell around) of the planes in
// flight in LDS.  It reads r, z and x once and writes x: 16 bytes per cell
// in FP32, bound by HBM and the latency of its per-plane steps.
// RESID: writes r1 - A e (the residual the next iteration starts from)
// instead of touching x.
// SMOOTH: an iteration of two sweeps alone, z = om_z D^-1 r in place of the
// products' (made from r as it is read), e with a weight of its own.  The
// residual that the products leave is rounding noise, about white in x, and
// after the first sweep these two take it to 0.17 to 0.19 of its norm
// whatever the ratio of the spacings (1 to 16 and to 1/16; the weights are
// the minimax over those).  It costs a RESID and a SMOOTH pass, 127 + 134 us
// at 512x512x128, against 1150 us for products (step 6.34 -> 5.43 ms), and
// 36 + 46 against 270 us at 450x300x40.
template <int FK_>
struct DsFin {
  static constexpr int NTH = 512, FK = FK_, FJ = 1024 / FK_, NU = 2;   // NU columns per thread
  static constexpr int ROWS = NTH / FK;
  static constexpr int ZJ = FJ + 4, ZK = FK + 4, EJ = FJ + 2, EK = FK + 2;
  static constexpr int ZRING = ZJ * ZK - FJ * FK, ERING = EJ * EK - FJ * FK;
  static constexpr int VZ = (ZRING + NTH - 1) / NTH, VE = (ERING + NTH - 1) / NTH;
};

// Position of entry q of the ring of width b around an nj x nk tile, in the
// enlarged plane.
__device__ __forceinline__ void ds_ring(int q, int b, int nj, int nk, int& j, int& k) {
  const int wk = nk + 2 * b, full = b * wk;
  if (q < full) {
    j = q / wk;
    k = q - j * wk;
  } else if (q < 2 * full) {
    q -= full;
    j = nj + b + q / wk;
    k = q % wk;
  } else {
    q -= 2 * full;
    j = b + q / (2 * b);
    const int c = q % (2 * b);
    k = c < b ? c : nk + c;
  }
}

__device__ __forceinline__ int ds_clamp(int i, int n) { return min(max(i, -1), n + 1); }
__device__ __forceinline__ int ds_class(int i, int n) { return (i <= 0 ? 1 : 0) | (i >= n - 1 ? 2 : 0); }

template <int FK, bool RESID, bool SMOOTH, class T>
__global__ __launch_bounds__(512) void k_ds_finish(Params<T> P, const T* __restrict__ R, const T* __restrict__ Z,
                                                   T* __restrict__ X, T* __restrict__ Rout, CgCtl c, int nfi, int njt,
                                                   int nkt) {
  using F = DsFin<FK>;
  __shared__ T sz[3][F::ZJ * F::ZK];
  __shared__ T se[2][F::EJ * F::EK];
  __shared__ T tab_d[64];
  __shared__ T tab_omd[64];
  __shared__ T tab_z[SMOOTH ? 64 : 1];
  const CgState* st = c.st;
  const Layout& L = P.L;
  // uniform over the grid
  if (RESID ? (st->done || st->smoothed != (int)SMOOTH) : SMOOTH ? (st->done || !st->smooth) : ds_idle(st)) {
    if (RESID || SMOOTH || !st->zero_rhs) return;
  }
  int bt, ch;
  if (!xcd_block(njt * nkt, (L.nx + nfi - 1) / nfi, bt, ch)) return;
  const int bid = ch * njt * nkt + bt;
  const int tid = threadIdx.x, kk = tid % F::FK, jr = tid / F::FK;
  const int j0 = (bt / nkt) * F::FJ, k0 = (bt % nkt) * F::FK;
  const int i0 = ch * nfi, i1 = min(L.nx, i0 + nfi);
  if (!RESID && !SMOOTH && st->done) {   // b = 0: the solution is x = 0
    for (int u = 0; u < F::NU; ++u) {
      const int j = j0 + jr + F::ROWS * u, k = k0 + kk;
      if (j < L.ny && k < L.nz)
        for (int i = i0; i < i1; ++i) X[L.at(i, j, k)] = T(0);
    }
    return;
  }
  if (tid < 64) {
    const int cx = tid >> 4, cy = (tid >> 2) & 3, cz = tid & 3;
    auto side = [&](int cl, int a) {
      return P.ih2[a] * (T(!(cl & 1) || P.bc[2 * a] == OUTLET) + T(!(cl & 2) || P.bc[2 * a + 1] == OUTLET));
    };
    const T D = side(cx, 0) + side(cy, 1) + side(cz, 2);
    tab_d[tid] = D;
    tab_omd[tid] = D > T(0) ? T(SMOOTH ? kDsOmegaE : kDsOmega) / D : T(0);
    if (SMOOTH) tab_z[tid] = D > T(0) ? T(kDsOmegaZ) / D : T(0);
  }
  // own columns (u < NU), then ring entries of the z plane and of the e plane
  long long oo[F::NU], zo[F::VZ], ro[F::VE];
  int op[F::NU], oe[F::NU], ocl[F::NU], zp[F::VZ], zcl[F::VZ], ep[F::VE], eq[F::VE], ecl[F::VE];
  bool oin[F::NU], ein[F::VE];
  // A z is formed from differences to the neighbours (a Neumann side's
  // neighbour is the cell itself): for the smooth parts of z they are far
  // smaller than z, and so is their rounding; D z - sum of neighbours rounds
  // relative to z, which A^-1 would turn into an error of the smooth modes.
  int on[F::NU][4], en[F::VE][4];   // LDS positions of the y and z neighbours
  auto neighbours = [&](int q, int j, int k, int (&nb)[4]) {
    nb[0] = j == 0 && P.bc[2] != OUTLET ? q : q - F::ZK;
    nb[1] = j == L.ny - 1 && P.bc[3] != OUTLET ? q : q + F::ZK;
    nb[2] = k == 0 && P.bc[4] != OUTLET ? q : q - 1;
    nb[3] = k == L.nz - 1 && P.bc[5] != OUTLET ? q : q + 1;
  };
#pragma unroll
  for (int u = 0; u < F::NU; ++u) {
    const int jj = jr + F::ROWS * u, j = j0 + jj, k = k0 + kk;
    oo[u] = (long long)(ds_clamp(j, L.ny) + 1) * L.PZ + (ds_clamp(k, L.nz) + 1);
    op[u] = (jj + 2) * F::ZK + kk + 2;
    oe[u] = (jj + 1) * F::EK + kk + 1;
    ocl[u] = (ds_class(j, L.ny) << 2) | ds_class(k, L.nz);
    oin[u] = j < L.ny && k < L.nz;
    neighbours(op[u], j, k, on[u]);
  }
#pragma unroll
  for (int v = 0; v < F::VZ; ++v) {
    const int q = tid + v * F::NTH;
    int a = 0, b = 0;
    if (q < F::ZRING) ds_ring(q, 2, F::FJ, F::FK, a, b);
    zp[v] = q < F::ZRING ? a * F::ZK + b : -1;
    zo[v] = (long long)(ds_clamp(j0 - 2 + a, L.ny) + 1) * L.PZ + (ds_clamp(k0 - 2 + b, L.nz) + 1);
    zcl[v] = (ds_class(j0 - 2 + a, L.ny) << 2) | ds_class(k0 - 2 + b, L.nz);
  }
#pragma unroll
  for (int v = 0; v < F::VE; ++v) {
    const int q = tid + v * F::NTH;
    int a = 0, b = 0;
    if (q < F::ERING) ds_ring(q, 1, F::FJ, F::FK, a, b);
    const int j = j0 - 1 + a, k = k0 - 1 + b;
    ep[v] = q < F::ERING ? a * F::EK + b : -1;
    eq[v] = (a + 1) * F::ZK + b + 1;
    ein[v] = q < F::ERING && (unsigned)j < (unsigned)L.ny && (unsigned)k < (unsigned)L.nz;
    ecl[v] = (ds_class(j, L.ny) << 2) | ds_class(k, L.nz);
    neighbours(eq[v], j, k, en[v]);
    ro[v] = (long long)(ds_clamp(j, L.ny) + 1) * L.PZ + (ds_clamp(k, L.nz) + 1);
  }
  T zv[F::NU], zr[F::VZ], rv[F::NU], rr[F::VE], xv[F::NU];
  // plane i of z with plane i - 1 of r and plane i - 2 of x
  auto load = [&](int i) {
    const long long bz = (long long)(ds_clamp(i, L.nx) + 1) * L.SX, br = (long long)(ds_clamp(i - 1, L.nx) + 1) * L.SX;
#pragma unroll
    for (int u = 0; u < F::NU; ++u) {
      zv[u] = (SMOOTH ? R : Z)[bz + oo[u]];
      rv[u] = R[br + oo[u]];
    }
#pragma unroll
    for (int v = 0; v < F::VZ; ++v) zr[v] = (SMOOTH ? R : Z)[bz + zo[v]];
#pragma unroll
    for (int v = 0; v < F::VE; ++v) rr[v] = R[br + ro[v]];
    if (!RESID) {
      const long long bx = (long long)(ds_clamp(i - 2, L.nx) + 1) * L.SX;
#pragma unroll
      for (int u = 0; u < F::NU; ++u) xv[u] = X[bx + oo[u]];
    }
  };
  const T w0 = P.ih2[0], w1 = P.ih2[1], w2 = P.ih2[2];
  // own z of planes i - 2 .. i, e of planes i - 3 .. i - 1, r1 of i - 2, i - 1
  T z0[F::NU], z1[F::NU], z2[F::NU], e0[F::NU], e1[F::NU], e2[F::NU], q0[F::NU], q1[F::NU];
#pragma unroll
  for (int u = 0; u < F::NU; ++u) z0[u] = z1[u] = z2[u] = e0[u] = e1[u] = e2[u] = q0[u] = q1[u] = T(0);
  double acc[1] = {0.0};
  load(i0 - 2);
  if (SMOOTH) __syncthreads();   // tab_z
  for (int i = i0 - 2; i <= i1 + 1; ++i) {
    T* s2 = sz[(i + 6) % 3];
    T r1[F::NU], rg[F::VE], xo[F::NU];
    if (SMOOTH) {
      const int cz = ds_class(i, L.nx) << 4;
#pragma unroll
      for (int u = 0; u < F::NU; ++u) zv[u] *= tab_z[cz | ocl[u]];
#pragma unroll
      for (int v = 0; v < F::VZ; ++v) zr[v] *= tab_z[cz | zcl[v]];
    }
#pragma unroll
    for (int u = 0; u < F::NU; ++u) {
      z0[u] = z1[u];
      z1[u] = z2[u];
      z2[u] = zv[u];
      s2[op[u]] = zv[u];
      r1[u] = rv[u];
      if (!RESID) xo[u] = xv[u];
    }
#pragma unroll
    for (int v = 0; v < F::VZ; ++v)
      if (zp[v] >= 0) s2[zp[v]] = zr[v];
#pragma unroll
    for (int v = 0; v < F::VE; ++v) rg[v] = rr[v];
    if (i <= i1) load(i + 1);
    __syncthreads();
    // e of plane p = i - 1
    const int p = i - 1;
    const T* s1 = sz[(p + 6) % 3];
    const T* s0 = sz[(p + 5) % 3];
    T* ec = se[p & 1];
    const bool pin = p >= i0 - 1 && (unsigned)p < (unsigned)L.nx;
    const int cx = ds_class(p, L.nx) << 4;
    const T wm = p == 0 && P.bc[0] != OUTLET ? T(0) : w0, wp = p == L.nx - 1 && P.bc[1] != OUTLET ? T(0) : w0;
    auto lap = [&](T zc, T zm, T zq, const int (&nb)[4]) {   // -A z
      return wm * (zm - zc) + wp * (zq - zc) + w1 * ((s1[nb[0]] - zc) + (s1[nb[1]] - zc)) +
             w2 * ((s1[nb[2]] - zc) + (s1[nb[3]] - zc));
    };
#pragma unroll
    for (int u = 0; u < F::NU; ++u) {
      r1[u] = pin && oin[u] ? r1[u] + lap(z1[u], z0[u], z2[u], on[u]) : T(0);
      e0[u] = e1[u];
      e1[u] = e2[u];
      e2[u] = tab_omd[cx | ocl[u]] * r1[u];
      q0[u] = q1[u];
      q1[u] = r1[u];
      ec[oe[u]] = e2[u];
    }
#pragma unroll
    for (int v = 0; v < F::VE; ++v) {
      if (ep[v] < 0) continue;
      const int q = eq[v];
      ec[ep[v]] = pin && ein[v] ? tab_omd[cx | ecl[v]] * (rg[v] + lap(s1[q], s0[q], s2[q], en[v])) : T(0);
    }
    __syncthreads();
    // plane f = i - 2: the residual left, and the iterate
    const int f = i - 2;
    if (f < i0 || f >= i1) continue;
    const T* em = se[f & 1];
    const int cf = ds_class(f, L.nx) << 4;
#pragma unroll
    for (int u = 0; u < F::NU; ++u) {
      if (!oin[u]) continue;
      const T ae = tab_d[cf | ocl[u]] * e1[u] - w0 * (e2[u] + e0[u]) - w1 * (em[oe[u] + F::EK] + em[oe[u] - F::EK]) -
                   w2 * (em[oe[u] + 1] + em[oe[u] - 1]);
      const T r2 = q0[u] - ae;
      const long long o = (long long)(f + 1) * L.SX + oo[u];
      if (RESID) {
        Rout[o] = r2;
      } else {
        X[o] = xo[u] + (z0[u] + e1[u]);
        acc[0] += (double)r2 * (double)r2;
      }
    }
  }
  if (!RESID) {
    const int slots[1] = {S_RR};
    write_partials<1>(acc, c.part, c.stride, slots, bid);
    pad_partials(c, S_RR, bid, njt * nkt * ((L.nx + nfi - 1) / nfi));
  }
}

// One block, after iteration `it` (from 1): has the solve finished?
__global__ __launch_bounds__(256) void k_ds_status(CgCtl c, int it) {
  CgState* st = c.st;
  if (st->done) return;
  const double rr = slot_sum(c.part + (size_t)S_RR * c.stride, c.nb_rr);
  if (threadIdx.x != 0) return;
  st->rr = rr;
  st->iter = it;
  st->nonfinite = !isfinite(rr);
  const bool conv = rr <= st->tol2_bb;
  st->done = conv || st->nonfinite || it >= c.maxit;
  st->noconv = st->done && !conv && !st->nonfinite;
  st->smoothed = st->smooth;
  st->smooth = !st->smoothed && rr <= kDsReach * kDsReach * st->tol2_bb;
}

// ------------------------------------------------------------------- host
struct DsGeom {
  int fk, njt, nkt, nfi, gy;
};

static DsGeom ds_geom(const Layout& L) {
  DsGeom d;
  d.fk = L.nz >= 64 ? 64 : (L.nz > 16 ? 32 : 16);
  const int fj = 1024 / d.fk;
  d.njt = (L.ny + fj - 1) / fj;
  d.nkt = (L.nz + d.fk - 1) / d.fk;
  // about 1024 blocks, of at least four planes (a chunk re-reads four of z)
  const int tiles = d.njt * d.nkt;
  const int want = std::max(1, std::min((L.nx + 3) / 4, (1024 + tiles - 1) / tiles));
  d.nfi = (L.nx + want - 1) / want;
  // few blocks: a chunk's own length is what takes the time (64x32x16 10.6 ->
  // 9.2 us; 96x80x48 in FP64, 144 blocks, 14.4 -> 15.2)
  if (tiles * want < 64) d.nfi = std::max(1, d.nfi / 2);
  d.gy = (L.nx + d.nfi - 1) / d.nfi;
  return d;
}

size_t direct_blocks(const Layout& L) {
  const DsGeom d = ds_geom(L);
  return (size_t)d.njt * d.nkt * d.gy;
}

// Rows of a line per wavefront of k_ds_tri: as few as its sixteen
// wavefronts allow (more lines in flight); 0 for lines past 512 rows (at 64
// rows per wavefront the kernel spills registers).
static int ds_chunk(int nx) {
  for (int lc = 8; lc <= 32; lc *= 2)
    if ((nx + lc - 1) / lc <= 16) return lc;
  return 0;
}

// Which solves are direct: the multigrid configuration with the residual
// criterion (the paper's criterion and the preconditioner study iterate),
// lines of x that the tridiagonal kernel holds, and axes up to the longest
// measured.  There the products are still far the cheaper way (a solve from
// zero, ms, CG against direct; the CG takes 9 to 20 iterations in FP32, 18 to
// 23 in FP64): 8x1024x1000 4.87 against 1.10, 64x64x1900 4.04 / 1.00,
// 4x40x2000 0.99 / 0.26, 200x1000x1000 128 / 18; FP64 64x1000x1000 93 / 11,
// 16x1900x128 6.7 / 1.1, 4x40x2000 3.7 / 0.35.
bool direct_use(const uf_config& c, size_t esize) {
  const double bytes = (double)(c.nx + 3) * (c.ny + 3) * (c.nz + 3) * (double)esize;
  return c.precond == UF_PC_MG && c.cg_criterion == 0 && ds_chunk(c.nx) > 0 && c.ny + c.nz <= 2048 &&
         bytes < 4294967296.0;
}

static int up(int n, int m) { return (n + m - 1) / m * m; }

// Eigenvalues (weight w) and orthonormal eigenvectors v[i * n + c] (column c)
// of the one-dimensional operator on n cells with the given open (outlet)
// sides: theta_m = m pi / n, (m + 1) pi / (n + 1) or (2m + 1) pi / (2n + 1).
// The angles are multiples of one, so a table of sines covers them.  Mode m
// is column n - 1 - m: the products back sum the columns in order, and with
// the smooth modes, which hold most of the solution, coming last the partial
// sums stay small until the end, and so do their roundings (the residual an
// FP32 iteration leaves: 256x256x64 4.4e-6 -> 6.0e-7 ||b||, 512x512x128
// 4.9e-5 -> 4.0e-6; most steps then need one iteration instead of two).
static void axis_modes(int n, double w, bool lo, bool hi, std::vector<double>& lam, std::vector<double>& v) {
  const long long q = (lo && hi) ? n + 1 : (lo || hi) ? 2 * n + 1 : n;   // theta_m = a_m pi / q
  // sines at multiples of pi / (2q)
  std::vector<double> tab(4 * q);
  for (long long t = 0; t < 4 * q; ++t) tab[t] = std::sin(M_PI * (double)t / (double)(2 * q));
  auto sine = [&](long long t) { return tab[t % (4 * q)]; };
  lam.resize(n);
  v.resize((size_t)n * n);
  for (int m = 0; m < n; ++m) {
    const long long a = (lo && hi) ? m + 1 : (lo || hi) ? 2 * m + 1 : m;
    const double s = sine(a);   // sin(theta / 2)
    const int col = n - 1 - m;
    lam[col] = 4.0 * w * s * s;
    const double norm = (lo && hi) ? std::sqrt(2.0 / (n + 1))
                                   : (lo || hi) ? 2.0 / std::sqrt(2.0 * n + 1.0) : std::sqrt((m ? 2.0 : 1.0) / n);
    for (int i = 0; i < n; ++i) {
      const long long cell = lo && !hi ? n - 1 - i : i;   // distance from the closed end
      // sin((i + 1) theta), or cos((cell + 1/2) theta) = sin(pi/2 + ...)
      v[(size_t)i * n + col] = norm * ((lo && hi) ? sine(2 * (i + 1) * a) : sine((2 * cell + 1) * a + q));
    }
  }
}

template <class T>
void direct_setup(Grid& g) {
  const int n[3] = {g.L.nx, g.L.ny, g.L.nz};
  const double h[3] = {g.cfg.dx, g.cfg.dy, g.cfg.dz};
  std::vector<double> lam[3], v;
  std::vector<T> mat;
  for (int a = 1; a < 3; ++a) {
    axis_modes(n[a], 1.0 / (h[a] * h[a]), g.bc[2 * a] == OUTLET, g.bc[2 * a + 1] == OUTLET, lam[a], v);
    const int ld = up(n[a], 128), rows = up(n[a], 16);
    for (int t = 0; t < 2; ++t) {   // [cell][mode] (forward), then [mode][cell] (back)
      mat.assign((size_t)rows * ld, T(0));
      for (int r = 0; r < n[a]; ++r)
        for (int c = 0; c < n[a]; ++c) mat[(size_t)r * ld + c] = T(t == 0 ? v[(size_t)r * n[a] + c] : v[(size_t)c * n[a] + r]);
      void** dst = a == 1 ? &g.ds_y[t] : &g.ds_z[t];
      *dst = galloc(g, mat.size() * sizeof(T));
      upload(g, *dst, mat.data(), mat.size() * sizeof(T));
    }
  }
  for (void*& w : g.ds_w) {
    const size_t bytes = (size_t)g.L.ny * up(g.L.nx * g.L.nz, 4) * sizeof(T);
    w = galloc(g, bytes);
    UF_HIP_CHECK(hipMemsetAsync(w, 0, bytes, g.stream));   // the row padding of W is read
  }
  lam[1].insert(lam[1].end(), lam[2].begin(), lam[2].end());
  g.ds_lam = (double*)galloc(g, lam[1].size() * sizeof(double));
  upload(g, g.ds_lam, lam[1].data(), lam[1].size() * sizeof(double));
}

void direct_free(Grid& g) {
  for (void** p : {&g.ds_y[0], &g.ds_y[1], &g.ds_z[0], &g.ds_z[1], &g.ds_w[0], &g.ds_w[1]}) {
    gfree(g, *p);
    *p = nullptr;
  }
  gfree(g, g.ds_lam);
  g.ds_lam = nullptr;
}

template <class T, bool FWD>
static void launch_row(Grid& g, const T* in, T* out, const T* E, long long ldw) {
  const Layout& L = g.L;
  const int lde = up(L.nz, 128), M = L.nx * L.ny;
  TimedLaunch tl(g, UF_TK_DS_ROW);
  auto go = [&](auto kernel, int bm, int bn) {
    const int mt = (M + bm - 1) / bm, nt = (L.nz + bn - 1) / bn;
    launch_k(g, kernel, xcd_grid(nt, mt), dim3(kDsThreads), L, in, out, E, lde, ldw, mt, nt, (const CgState*)g.st);
  };
  constexpr int MT = Mfma<T>::MT;
  // few rows: the small tile, for the blocks (64x32x16 6.9 -> 4.8 us a launch,
  // 129x97x35 10.1 -> 6.5, 96x80x48 in FP64 7.4 -> 6.0)
  if (M < 256 * 4 * MT) go(k_ds_row<T, 1, 1, FWD>, 2 * MT, 2 * MT);
  else if (L.nz > 2 * MT) go(k_ds_row<T, 2, 2, FWD>, 4 * MT, 4 * MT);
  else go(k_ds_row<T, 2, 1, FWD>, 4 * MT, 2 * MT);
}

template <class T, bool FWD>
static void launch_col(Grid& g, const T* E, const T* in, T* out, long long ldw) {
  const Layout& L = g.L;
  const int lda = up(L.ny, 128), N = L.nx * L.nz;
  TimedLaunch tl(g, UF_TK_DS_COL);
  auto go = [&](auto kernel, int bm, int bn) {
    const int mt = (L.ny + bm - 1) / bm, nt = (N + bn - 1) / bn;
    launch_k(g, kernel, xcd_grid(mt, nt), dim3(kDsThreads), E, lda, in, out, L.ny, L.ny, N, ldw, mt, nt,
             (const CgState*)g.st);
  };
  constexpr int MT = Mfma<T>::MT;
  constexpr bool SPLIT = FWD && sizeof(T) == 4;
  // the large tile halves the LDS traffic per product; the small one wastes
  // less on a ragged ny and gives short axes enough blocks
  if ((long long)up(L.ny, 4 * MT) * 8 <= (long long)L.ny * 9 && (long long)L.ny * N >= 1024LL * 16 * MT * MT) {
    // with a second set of sums the widest tile leaves two wavefronts per
    // SIMD: 368 us at 512x512x128 against 352 with half of it (299 and 310
    // with one set)
    if (SPLIT) go(k_ds_col<T, 2, 1, SPLIT>, 4 * MT, 2 * MT);
    else go(k_ds_col<T, 2, 2, SPLIT>, 4 * MT, 4 * MT);
  } else
    go(k_ds_col<T, 1, 1, SPLIT>, 2 * MT, 2 * MT);
}

template <class T, int LC>
static void launch_tri(Grid& g, T* W, long long ldw) {
  const Layout& L = g.L;
  const int nc = (L.nx + LC - 1) / LC, nlines = L.ny * L.nz;
  TimedLaunch tl(g, UF_TK_DS_TRI);
  launch_k(g, k_ds_tri<T, LC>, dim3((nlines + 63) / 64), dim3(64 * nc), W, L.nx, nlines, L.nz, ldw,
           1.0 / (g.cfg.dx * g.cfg.dx), (const double*)g.ds_lam, (const double*)(g.ds_lam + L.ny),
           g.bc[0] == OUTLET ? 1 : 0, g.bc[1] == OUTLET ? 1 : 0, (const CgState*)g.st);
}

template <bool RESID, bool SMOOTH, class T>
static void launch_finish(Grid& g, const Params<T>& P, const void* R, void* Rout) {
  const DsGeom d = ds_geom(P.L);
  TimedLaunch tl(g, UF_TK_DS_FINISH);
  auto go = [&](auto kernel) {
    launch_k(g, kernel, xcd_grid(d.njt * d.nkt, d.gy), dim3(512), P, (const T*)R, (const T*)g.Z, (T*)g.X, (T*)Rout,
             make_ctl(g), d.nfi, d.njt, d.nkt);
  };
  if (d.fk == 64) go(k_ds_finish<64, RESID, SMOOTH, T>);
  else if (d.fk == 32) go(k_ds_finish<32, RESID, SMOOTH, T>);
  else go(k_ds_finish<16, RESID, SMOOTH, T>);
}

// Iteration t (from 0) of a direct solve; the residual is in resid(g, t).
// After products that left little (CgState::smooth) it is a smoothing
// iteration.  last: the status after iteration t - 1 when the host has it;
// both kinds are enqueued otherwise, and one returns at once.
template <class T>
void launch_direct_iteration(Grid& g, const Params<T>& P, int t, const CgState* last) {
  const Layout& L = P.L;
  const long long ldw = up(L.nx * L.nz, 4);
  T* W0 = (T*)g.ds_w[0];
  T* W1 = (T*)g.ds_w[1];
  if (t > 0) {
    if (!last || !last->smoothed) launch_finish<true, false, T>(g, P, resid(g, t - 1), resid(g, t));
    if (last ? last->smoothed : t > 1) launch_finish<true, true, T>(g, P, resid(g, t - 1), resid(g, t));
    if (!last || last->smooth) launch_finish<false, true, T>(g, P, resid(g, t), nullptr);
  }
  if (t == 0 || !last || !last->smooth) {
    launch_row<T, true>(g, (const T*)resid(g, t), W0, (const T*)g.ds_z[0], ldw);
    launch_col<T, true>(g, (const T*)g.ds_y[0], W0, W1, ldw);
    switch (ds_chunk(L.nx)) {
      case 8: launch_tri<T, 8>(g, W1, ldw); break;
      case 16: launch_tri<T, 16>(g, W1, ldw); break;
      default: launch_tri<T, 32>(g, W1, ldw); break;
    }
    launch_col<T, false>(g, (const T*)g.ds_y[1], W1, W0, ldw);
    launch_row<T, false>(g, W0, (T*)g.Z, (const T*)g.ds_z[1], ldw);
    launch_finish<false, false, T>(g, P, resid(g, t), nullptr);
  }
  hipLaunchKernelGGL(k_ds_status, dim3(1), dim3(256), 0, g.stream, make_ctl(g), t + 1);
}

template void direct_setup<float>(Grid&);
template void direct_setup<double>(Grid&);
template void launch_direct_iteration<float>(Grid&, const Params<float>&, int, const CgState*);
template void launch_direct_iteration<double>(Grid&, const Params<double>&, int, const CgState*);

}  // namespace uf
