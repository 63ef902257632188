// Cell-centred kernels: the k-omega turbulence update (Sec. 3, solved after
// the projection), the porosity -> drag-coefficient map (Sec. 3 drag law),
// and packing between the padded storage (boundary rules applied as values
// are put in) and the compact layouts of the C ABI.
#include "march.h"
#include "turb_model.h"

namespace uf {

constexpr int kCellBlock = 256;

__host__ __device__ inline int cell_gx(const Layout& L) { return (L.ny * L.nz + kCellBlock - 1) / kCellBlock; }

// Logical block (bx, i) of a cell kernel launched on xcd_grid(cell_gx, nx):
// XCD-contiguous ranges of the band-major order (band_map), as the face
// kernels, so that the x-neighbours a stencil reads stay in the XCD's L2.
constexpr int kCellBand = 8;
__device__ __forceinline__ bool cell_block(const Layout& L, int& bx, int& i) {
  const int gx = cell_gx(L), gy = L.nx;
  const int per = (int)(gridDim.x >> 3);
  const int b = (int)(blockIdx.x & 7u) * per + (int)(blockIdx.x >> 3);
  if (b >= gx * gy) return false;
  band_map(gx, gy, kCellBand, b, bx, i);
  return true;
}

// A thread owns cell (i, j, k) of logical block (bx, iplane); threads past
// the plane's cells return.
#define UF_CELL_POINT(L, bx, iplane)                                 \
  const int i = (iplane);                                            \
  const int p = (bx) * kCellBlock + threadIdx.x;                     \
  if (p >= (L).ny * (L).nz) return;                                  \
  const int j = p / (L).nz;                                          \
  const int k = p - j * (L).nz;

#define UF_CELL_THREAD(L)                                            \
  int c_bx, c_by;                                                    \
  if (!cell_block((L), c_bx, c_by)) return;                          \
  UF_CELL_POINT(L, c_bx, c_by)

// k-omega step at one cell.  Velocity gradients: normal derivatives from the
// cell's two faces, cross derivatives as central differences of cell-centred
// velocities (face means; ghost faces beyond the domain).  Strain rate
// S = (grad u + grad u^T)/2, |S|^2 = S_ij S_ij.  Limiter omega~ = max(omega,
// C_lim |S| / sqrt(C_mu/2)) (Wilcox 2006, cited in Sec. 3); eddy viscosity
// nu_t = k / omega~ limited to [0, nu_max - nu] (the paper's von Neumann
// viscosity limiter).  Forward Euler with first-order upwind advection and
// central Laplacians.
// get(a, dx, dj, dk): array a (u, v, w, k, omega) at the cell displaced by
// (dx, dj, dk).  Returns the new eddy viscosity; kn and wn when update_kw.
template <class T, class G>
__device__ __forceinline__ T turb_cell(const Params<T>& P, G get, bool update_kw, T& kn, T& wn) {
  const T h0 = T(0.5) * P.ih[0], h1 = T(0.5) * P.ih[1], h2 = T(0.5) * P.ih[2];
  // gradients G[c][d] = d u_c / d x_d
  const T g00 = (get(0, 1, 0, 0) - get(0, 0, 0, 0)) * P.ih[0];
  const T g11 = (get(1, 0, 1, 0) - get(1, 0, 0, 0)) * P.ih[1];
  const T g22 = (get(2, 0, 0, 1) - get(2, 0, 0, 0)) * P.ih[2];
  auto uc = [&](int dx, int dj, int dk) { return T(0.5) * (get(0, dx, dj, dk) + get(0, dx + 1, dj, dk)); };
  auto vc = [&](int dx, int dj, int dk) { return T(0.5) * (get(1, dx, dj, dk) + get(1, dx, dj + 1, dk)); };
  auto wc = [&](int dx, int dj, int dk) { return T(0.5) * (get(2, dx, dj, dk) + get(2, dx, dj, dk + 1)); };
  const T g01 = (uc(0, 1, 0) - uc(0, -1, 0)) * h1;
  const T g02 = (uc(0, 0, 1) - uc(0, 0, -1)) * h2;
  const T g10 = (vc(1, 0, 0) - vc(-1, 0, 0)) * h0;
  const T g12 = (vc(0, 0, 1) - vc(0, 0, -1)) * h2;
  const T g20 = (wc(1, 0, 0) - wc(-1, 0, 0)) * h0;
  const T g21 = (wc(0, 1, 0) - wc(0, -1, 0)) * h1;
  const T s01 = T(0.5) * (g01 + g10), s02 = T(0.5) * (g02 + g20), s12 = T(0.5) * (g12 + g21);
  const T S2 = g00 * g00 + g11 * g11 + g22 * g22 + T(2) * (s01 * s01 + s02 * s02 + s12 * s12);
  const T lim = P.lim_coef * sqrt(S2);
  const T kk = get(3, 0, 0, 0), ww = get(4, 0, 0, 0);
  const T nut = nmin(nmax(kk / nmax(ww, lim), T(0)), P.cap);
  if (!update_kw) return nut;
  const T u0 = uc(0, 0, 0), u1 = vc(0, 0, 0), u2 = wc(0, 0, 0);
  auto adv = [&](int q) {
    const T c = get(q, 0, 0, 0);
    T a = (nmax(u0, T(0)) * (c - get(q, -1, 0, 0)) + nmin(u0, T(0)) * (get(q, 1, 0, 0) - c)) * P.ih[0];
    a += (nmax(u1, T(0)) * (c - get(q, 0, -1, 0)) + nmin(u1, T(0)) * (get(q, 0, 1, 0) - c)) * P.ih[1];
    a += (nmax(u2, T(0)) * (c - get(q, 0, 0, -1)) + nmin(u2, T(0)) * (get(q, 0, 0, 1) - c)) * P.ih[2];
    return a;
  };
  auto lap = [&](int q) {
    const T c = get(q, 0, 0, 0);
    return (get(q, 1, 0, 0) - T(2) * c + get(q, -1, 0, 0)) * P.ih2[0] +
           (get(q, 0, 1, 0) - T(2) * c + get(q, 0, -1, 0)) * P.ih2[1] +
           (get(q, 0, 0, 1) - T(2) * c + get(q, 0, 0, -1)) * P.ih2[2];
  };
  kn = kk + P.dt * (-adv(3) + T(2) * nut * S2 - T(kCmu) * kk * ww + (P.nu + T(kSigmaStar) * nut) * lap(3));
  wn = ww + P.dt * (-adv(4) + T(2 * kAlpha) * S2 - T(kBeta) * ww * ww + (P.nu + T(kSigma) * nut) * lap(4));
  kn = nmax(kn, P.k_min);
  wn = nmax(wn, P.w_min);
  return nmin(nmax(kn / nmax(wn, lim), T(0)), P.cap);
}

// The step at cell (i, j, k), from memory.
template <class T>
__device__ __forceinline__ void turb_point(const Params<T>& P, const T* __restrict__ U, const T* __restrict__ V, const T* __restrict__ W, const T* __restrict__ K0, const T* __restrict__ W0, T* __restrict__ K1, T* __restrict__ W1, T* __restrict__ NUT, int update_kw, int* nf, int i, int j, int k) {
  const Layout& L = P.L;
  const long long o = L.at(i, j, k);
  const T* q[5] = {U + o, V + o, W + o, K0 + o, W0 + o};
  T kn, wn;
  const T nut = turb_cell(P, [&](int a, int dx, int dj, int dk) { return q[a][dx * L.SX + (long long)dj * L.PZ + dk]; },
                          update_kw != 0, kn, wn);
  if (update_kw) {
    if (!(isfinite(kn) && isfinite(wn))) *nf = 1;   // every writer stores 1: no atomic needed
    store_cell(K1, P, i, j, k, kn, true, P.k_in);
    store_cell(W1, P, i, j, k, wn, true, P.w_in);
  }
  store_cell(NUT, P, i, j, k, nut, false, T(0));
}

template <class T>
__device__ __forceinline__ void turb_cells(const Params<T>& P, const T* __restrict__ U, const T* __restrict__ V, const T* __restrict__ W, const T* __restrict__ K0, const T* __restrict__ W0, T* __restrict__ K1, T* __restrict__ W1, T* __restrict__ NUT, int update_kw, int* nf, int bx, int ib) {
  UF_CELL_POINT(P.L, bx, ib);
  turb_point(P, U, V, W, K0, W0, K1, W1, NUT, update_kw, nf, i, j, k);
}

// The update marching along x (march.h): tiles of the cells off the sides
// along x and y, blocks of their own for the others.
template <class T>
struct TurbArgs {
  const T* in[5];   // u, v, w, k, omega
  T* out[3];        // k, omega, nu_t
  int* nf;
};

__host__ __device__ inline int turb_edges(const Layout& L) { return 2 * L.nz * (L.ny + (L.nx - 2)); }

template <class T>
__device__ __forceinline__ void turb_edge(const Params<T>& P, const TurbArgs<T>& M, int e) {
  const Layout& L = P.L;
  if (e >= turb_edges(L)) return;
  const int r = e / L.nz, k = e - r * L.nz;
  int i, j;
  if (r < 2 * L.ny) {
    i = r < L.ny ? 0 : L.nx - 1;
    j = r < L.ny ? r : r - L.ny;
  } else {
    const int q = r - 2 * L.ny;
    j = q < L.nx - 2 ? 0 : L.ny - 1;
    i = 1 + (q < L.nx - 2 ? q : q - (L.nx - 2));
  }
  turb_point(P, M.in[0], M.in[1], M.in[2], M.in[3], M.in[4], M.out[0], M.out[1], M.out[2], 1, M.nf, i, j, k);
}

template <int SHAPE, class T>
__device__ __forceinline__ void turb_march(const Params<T>& P, const March& G, const TurbArgs<T>& M, T* lds, int tile,
                                           int chunk) {
  const Layout& L = P.L;
  Planes<SHAPE, 5, T> A;
#pragma unroll
  for (int a = 0; a < 5; ++a) A.src[a] = M.in[a];
  int j0, k0;
  const MarchLane c = march_lane<SHAPE>(L, G, tile, L.ny - 2, L.nz + 2, L.nz, L.nz, j0, k0);
  A.init(L, lds, j0, k0, G.TK);
  A.q = c.qa;
  const int i0 = 1 + chunk * G.len;
  march(A, i0, min(L.nx - 1, i0 + G.len), [&](int i) {
    if (!c.active) return;
    T kn, wn;
    const T nut = turb_cell(P, [&](int a, int dx, int dj, int dk) { return A.at(a, dx, dj, dk); }, true, kn, wn);
    if (!(isfinite(kn) && isfinite(wn))) *M.nf = 1;
    const long long o = (long long)(i + 1) * L.SX;   // the ghosts along z copy their cell
    (M.out[0] + o)[c.oc] = kn;
    (M.out[1] + o)[c.oc] = wn;
    (M.out[2] + o)[c.oc] = nut;
  });
}

template <int SHAPE, class T>
__global__ __launch_bounds__(kMarch, 6) void k_turb_march(Params<T> P, March G, TurbArgs<T> M,
                                                           const int* __restrict__ gate) {
  __shared__ T lds[Planes<SHAPE, 5, T>::LDS];
  if (gate && !*gate) return;
  int tile, chunk;
  if (!march_block(G, tile, chunk)) return;
  if (tile < 0) turb_edge(P, M, chunk * kMarch + (int)threadIdx.x);
  else turb_march<SHAPE>(P, G, M, lds, tile, chunk);
}

// gate: as k_project's (the step's k-omega update enqueued with it).
template <class T>
__global__ __launch_bounds__(kCellBlock) void k_turbulence(Params<T> P, const T* __restrict__ U, const T* __restrict__ V, const T* __restrict__ W, const T* __restrict__ K0, const T* __restrict__ W0, T* __restrict__ K1, T* __restrict__ W1, T* __restrict__ NUT, int update_kw, int* nf, const int* __restrict__ gate) {
  if (gate && !*gate) return;
  int bx, ib;
  if (!cell_block(P.L, bx, ib)) return;
  turb_cells(P, U, V, W, K0, W0, K1, W1, NUT, update_kw, nf, bx, ib);
}

// Drag coefficient of each cell: C_d a ((1 - phi)/(phi + e))^b (Sec. 3 drag
// law with the porosity form of its footnote); also keeps phi (compact).
template <class T>
__global__ __launch_bounds__(kCellBlock) void k_porosity(Params<T> P, const T* __restrict__ phi, T* __restrict__ Cc,
                                                         T* __restrict__ PHI, T coef, T e, T b) {
  const Layout& L = P.L;
  UF_CELL_THREAD(L);
  const size_t c = ((size_t)i * L.ny + j) * L.nz + k;
  const T f = phi[c];
  PHI[c] = f;
  store_cell(Cc, P, i, j, k, coef * pow((T(1) - f) / (f + e), b), false, T(0));
}

template <class T>
__global__ __launch_bounds__(kCellBlock) void k_cell_fill(Params<T> P, T* __restrict__ q, T value, int use_inlet,
                                                          T inlet) {
  const Layout& L = P.L;
  UF_CELL_THREAD(L);
  store_cell(q, P, i, j, k, value, use_inlet != 0, inlet);
}

// Copy between the compact layout of a field and the padded storage, one
// pass: the boundary rules of a field put in are applied as its values are
// stored (a second pass over the field to set its ghosts took longer than
// the copy).  A block takes 4 x 256 consecutive values of one x-plane, each
// thread's four loads in flight together (512x512x128, one field: k_pack 78
// + boundary pass 100 to 131 us -> 56 to 74 us in, 66 us out).
enum PackMode { PACK_U = 0, PACK_V = 1, PACK_W = 2, PACK_CELL = 3, PACK_PLAIN = 4, PACK_GET = 5 };
constexpr int kPackLoads = 4;

template <class T, int MODE>
__global__ __launch_bounds__(kCellBlock) void k_pack(Params<T> P, int gx, int ey, int ez, const T* __restrict__ src,
                                                     T* __restrict__ dst, int use_inlet, T inlet, int* nf) {
  const Layout& L = P.L;
  // a state field put in clears the state's non-finite flag
  if (nf && blockIdx.x == 0 && threadIdx.x == 0) *nf = 0;
  const int i = (int)(blockIdx.x / (unsigned)gx), n = ey * ez;
  const int p0 = ((int)blockIdx.x - i * gx) * (kPackLoads * kCellBlock) + threadIdx.x;
  const size_t c0 = (size_t)i * n;
  T v[kPackLoads];
#pragma unroll
  for (int u = 0; u < kPackLoads; ++u) {
    const int p = min(p0 + u * kCellBlock, n - 1), j = p / ez;
    v[u] = MODE == PACK_GET ? src[L.at(i, j, p - j * ez)] : src[c0 + p];
  }
#pragma unroll
  for (int u = 0; u < kPackLoads; ++u) {
    const int p = p0 + u * kCellBlock;
    if (p >= n) break;
    const int j = p / ez, k = p - j * ez;
    if constexpr (MODE <= PACK_W) {
      T val = v[u];
      face_dirichlet<MODE>(P, i, j, k, &val);
      store_face<MODE>(dst, P, i, j, k, val);
    } else if constexpr (MODE == PACK_CELL) {
      store_cell(dst, P, i, j, k, v[u], use_inlet != 0, inlet);
    } else if constexpr (MODE == PACK_PLAIN) {
      dst[L.at(i, j, k)] = v[u];
    } else {
      dst[c0 + p] = v[u];
    }
  }
}

// Sum of the cell-centre wind speed over a box of cells (one FP64 partial per
// block; the caller adds the partials in block order).
template <class T>
__global__ __launch_bounds__(kCellBlock) void k_region_speed(Layout L, const T* __restrict__ U, const T* __restrict__ V,
                                                            const T* __restrict__ W, int i0, int j0, int k0, int ni,
                                                            int nj, int nk, double* __restrict__ part) {
  const long long n = (long long)ni * nj * nk;
  double v[1] = {0.0};
  for (long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x; c < n; c += (long long)gridDim.x * blockDim.x) {
    const int k = k0 + (int)(c % nk);
    const long long r = c / nk;
    const int j = j0 + (int)(r % nj);
    const int i = i0 + (int)(r / nj);
    const long long o = L.at(i, j, k);
    const double uc = 0.5 * ((double)U[o] + (double)U[o + L.SX]);
    const double vc = 0.5 * ((double)V[o] + (double)V[o + L.PZ]);
    const double wc = 0.5 * ((double)W[o] + (double)W[o + 1]);
    v[0] += sqrt(uc * uc + vc * vc + wc * wc);
  }
  block_sum<1>(v);
  if (threadIdx.x == 0) part[blockIdx.x] = v[0];
}

// Pedestrian-plane objective: per column, the cell-centre velocity and the
// porosity interpolated in z at weight t between levels k0 and k0 + 1, the
// speed s = sqrt(|u|^2 + 1e-12), and phi [(s - st)^2 + w max(0, smin - s)^2];
// one FP64 partial per block.
template <class T>
__global__ __launch_bounds__(kCellBlock) void k_plane_objective(Layout L, const T* __restrict__ U,
                                                               const T* __restrict__ V, const T* __restrict__ W,
                                                               const T* __restrict__ PHI, int k0, double t,
                                                               double st, double smin, double wpen,
                                                               double* __restrict__ part) {
  const int n = L.nx * L.ny;
  double v[1] = {0.0};
  for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < n; c += gridDim.x * blockDim.x) {
    const int i = c / L.ny, j = c % L.ny;
    double uc[2], vc[2], wc[2], ph[2];
    for (int q = 0; q < 2; ++q) {
      const long long o = L.at(i, j, k0 + q);
      uc[q] = 0.5 * ((double)U[o] + (double)U[o + L.SX]);
      vc[q] = 0.5 * ((double)V[o] + (double)V[o + L.PZ]);
      wc[q] = 0.5 * ((double)W[o] + (double)W[o + 1]);
      ph[q] = (double)PHI[((size_t)i * L.ny + j) * L.nz + k0 + q];
    }
    const double up = (1.0 - t) * uc[0] + t * uc[1];
    const double vp = (1.0 - t) * vc[0] + t * vc[1];
    const double wp = (1.0 - t) * wc[0] + t * wc[1];
    const double phip = (1.0 - t) * ph[0] + t * ph[1];
    const double s = sqrt(up * up + vp * vp + wp * wp + 1e-12);
    const double lo = fmax(0.0, smin - s);
    v[0] += phip * ((s - st) * (s - st) + wpen * lo * lo);
  }
  block_sum<1>(v);
  if (threadIdx.x == 0) part[blockIdx.x] = v[0];
}

template <class T>
void launch_plane_objective(Grid& g, int k0, double t, double st, double smin, double wpen, double* part,
                            int nblocks) {
  hipLaunchKernelGGL(k_plane_objective<T>, dim3(nblocks), dim3(kCellBlock), 0, g.stream, g.L,
                     (const T*)g.Q[g.cur][0], (const T*)g.Q[g.cur][1], (const T*)g.Q[g.cur][2], (const T*)g.PHI, k0,
                     t, st, smin, wpen, part);
}

// Squared distance between the cell-centre velocity and a desired one over a
// box of cells (one FP64 partial per block).
template <class T>
__global__ __launch_bounds__(kCellBlock) void k_region_field_diff(Layout L, const T* __restrict__ U,
                                                                 const T* __restrict__ V, const T* __restrict__ W,
                                                                 const T* __restrict__ UT, int i0, int j0, int k0,
                                                                 int ni, int nj, int nk, double* __restrict__ part) {
  const long long n = (long long)ni * nj * nk;
  const size_t N = (size_t)L.nx * L.ny * L.nz;
  double v[1] = {0.0};
  for (long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x; c < n; c += (long long)gridDim.x * blockDim.x) {
    const int k = k0 + (int)(c % nk);
    const long long r = c / nk;
    const int j = j0 + (int)(r % nj);
    const int i = i0 + (int)(r / nj);
    const long long o = L.at(i, j, k);
    const size_t q = ((size_t)i * L.ny + j) * L.nz + k;
    const double du = 0.5 * ((double)U[o] + (double)U[o + L.SX]) - (double)UT[q];
    const double dv = 0.5 * ((double)V[o] + (double)V[o + L.PZ]) - (double)UT[N + q];
    const double dw = 0.5 * ((double)W[o] + (double)W[o + 1]) - (double)UT[2 * N + q];
    v[0] += du * du + dv * dv + dw * dw;
  }
  block_sum<1>(v);
  if (threadIdx.x == 0) part[blockIdx.x] = v[0];
}

template <class T>
void launch_region_field_diff(Grid& g, const int box[6], const void* ut, double* part, int nblocks) {
  hipLaunchKernelGGL(k_region_field_diff<T>, dim3(nblocks), dim3(kCellBlock), 0, g.stream, g.L,
                     (const T*)g.Q[g.cur][0], (const T*)g.Q[g.cur][1], (const T*)g.Q[g.cur][2], (const T*)ut, box[0],
                     box[2], box[4], box[1] - box[0], box[3] - box[2], box[5] - box[4], part);
}

template <class T>
void launch_region_speed(Grid& g, const int box[6], double* part, int nblocks) {
  hipLaunchKernelGGL(k_region_speed<T>, dim3(nblocks), dim3(kCellBlock), 0, g.stream, g.L, (const T*)g.Q[g.cur][0],
                     (const T*)g.Q[g.cur][1], (const T*)g.Q[g.cur][2], box[0], box[2], box[4], box[1] - box[0],
                     box[3] - box[2], box[5] - box[4], part);
}

template <class T>
__global__ __launch_bounds__(kCellBlock) void k_check_range(const T* __restrict__ phi, size_t n, int* flag) {
  int bad = 0;
  for (size_t c = (size_t)blockIdx.x * blockDim.x + threadIdx.x; c < n; c += (size_t)gridDim.x * blockDim.x) {
    const T f = phi[c];
    if (!(f >= T(0) && f <= T(1))) bad = 1;
  }
  if (bad) atomicOr(flag, 1);
}

static inline dim3 cell_grid(const Layout& L) { return xcd_grid(cell_gx(L), L.nx); }

template <class T>
void launch_turb(Grid& g, const Params<T>& P, void* const Q[3], const void* K0, const void* W0, void* K1, void* W1,
                 void* NUT, int update_kw, const int* gate) {
  TimedLaunch tl(g, UF_TK_TURB);
  if constexpr (sizeof(T) == 4) if (update_kw && march_pays(P, kMarchTurb)) {
    const Layout& L = P.L;
    const TurbArgs<T> M{{(const T*)Q[0], (const T*)Q[1], (const T*)Q[2], (const T*)K0, (const T*)W0},
                        {(T*)K1, (T*)W1, (T*)NUT}, nf_word(g)};
    const March G = march_geom(L.nx - 2, L.ny - 2, L.nz + 2, turb_edges(L));
    auto go = [&](auto kernel) { launch_k(g, kernel, march_grid(G), dim3(kMarch), P, G, M, gate); };
    if (G.shape == 0) go(k_turb_march<0, T>);
    else if (G.shape == 1) go(k_turb_march<1, T>);
    else go(k_turb_march<2, T>);
    return;
  }
  launch_k(g, k_turbulence<T>, cell_grid(P.L), dim3(kCellBlock), P, (const T*)Q[0],
                     (const T*)Q[1], (const T*)Q[2], (const T*)K0, (const T*)W0, (T*)K1, (T*)W1, (T*)NUT, update_kw,
                     nf_word(g), gate);
}

// The k-omega update of every case of a batch in one persistent launch
// (the cell queue: case c owns [cell0, cell0 + cell_gx * nx)); velocity
// from set sq, k and omega of case c from slot kcs[c] to the other slot,
// nu_t into the case's own array, or into set nut_set's u array when
// nut_set >= 0 (a trial run that leaves the state alone).
template <class T>
__global__ __launch_bounds__(kCellBlock) void k_turb_multi(const MultiCase<T>* __restrict__ mc, CaseStarts cs,
                                                          int band, int sq, const int* __restrict__ kcs,
                                                          int nut_set) {
  const int nb = (int)(gridDim.x >> 3);
  const int xcd = (int)(blockIdx.x & 7u), lid = (int)(blockIdx.x >> 3);
  const int total = cs.start[cs.n];
  const int share = (total + 7) >> 3;
  const int lo = xcd * share, hi = min(total, lo + share);
  for (int lb = lo + lid; lb < hi; lb += nb) {
    const int c = find_case(cs, lb);
    const MultiCase<T>& A = mc[c];
    int bx, ib;
    band_map(cell_gx(A.P.L), A.P.L.nx, band, lb - cs.start[c], bx, ib);
    T* nut = nut_set >= 0 ? A.q[nut_set][0] : A.nut;
    const int kc = kcs[c] & 1;
    turb_cells(A.P, A.q[sq][0], A.q[sq][1], A.q[sq][2], A.k[kc], A.w[kc], A.k[kc ^ 1], A.w[kc ^ 1], nut, 1, A.nf,
               bx, ib);
  }
}

template <class T>
void launch_turb_multi(const MultiCase<T>* mc, const CaseStarts& cs, int band, int blocks, int sq, const int* kcs,
                       int nut_set, hipStream_t stream) {
  hipLaunchKernelGGL(k_turb_multi<T>, dim3((unsigned)blocks), dim3(kCellBlock), 0, stream, mc, cs, band, sq, kcs,
                     nut_set);
}

int cell_queue_blocks(const Layout& L) { return cell_gx(L) * L.nx; }

// Diagnostics of a state, one partial per block and quantity: the largest
// |div_h u| over the cells, the largest dt sum_d |u_d| / h_d with the
// cell-centre velocity (the stability number of the upwind k-omega
// advection), and the number of cells whose eddy viscosity sits at the cap.
// NaN propagates into the maxima.  A block takes kDiagCells x kCellBlock cells
// of a plane at a time, the loads of a thread's cells in flight together
// (230 -> 117 us at 512x512x128, 27 -> 16 at 256x256x64).
constexpr int kDiagCells = 4;

template <class T>
__global__ __launch_bounds__(kCellBlock) void k_diag(Params<T> P, const T* __restrict__ U, const T* __restrict__ V,
                                                     const T* __restrict__ W, const T* __restrict__ NUT, int turb,
                                                     double* __restrict__ part) {
  const Layout& L = P.L;
  const int n = L.ny * L.nz, gx = (n + kDiagCells * kCellBlock - 1) / (kDiagCells * kCellBlock);
  double mdiv = 0.0, mcfl = 0.0, clip = 0.0;
  const double ih0 = 1.0 / (double)P.h[0], ih1 = 1.0 / (double)P.h[1], ih2 = 1.0 / (double)P.h[2];
  for (int b = (int)blockIdx.x; b < gx * L.nx; b += (int)gridDim.x) {
    const int i = b / gx, p0 = (b - i * gx) * kDiagCells * kCellBlock + (int)threadIdx.x;
    T f[kDiagCells][7];
#pragma unroll
    for (int u = 0; u < kDiagCells; ++u) {
      const int p = min(p0 + u * kCellBlock, n - 1), j = p / L.nz;
      const long long o = L.at(i, j, p - j * L.nz);
      f[u][0] = U[o];
      f[u][1] = U[o + L.SX];
      f[u][2] = V[o];
      f[u][3] = V[o + L.PZ];
      f[u][4] = W[o];
      f[u][5] = W[o + 1];
      f[u][6] = turb ? NUT[o] : T(0);
    }
#pragma unroll
    for (int u = 0; u < kDiagCells; ++u) {
      if (p0 + u * kCellBlock >= n) break;
      const double u0 = f[u][0], u1 = f[u][1], v0 = f[u][2], v1 = f[u][3], w0 = f[u][4], w1 = f[u][5];
      const double div = (u1 - u0) * ih0 + (v1 - v0) * ih1 + (w1 - w0) * ih2;
      mdiv = nmax(fabs(div), mdiv);
      const double cfl =
          (double)P.dt * (0.5 * fabs(u0 + u1) * ih0 + 0.5 * fabs(v0 + v1) * ih1 + 0.5 * fabs(w0 + w1) * ih2);
      mcfl = nmax(cfl, mcfl);
      if (turb && f[u][6] >= P.cap) clip += 1.0;
    }
  }
  __shared__ double sh[3][kCellBlock / 64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int o = 32; o > 0; o >>= 1) {
    mdiv = nmax(__shfl_xor(mdiv, o, 64), mdiv);
    mcfl = nmax(__shfl_xor(mcfl, o, 64), mcfl);
    clip += __shfl_xor(clip, o, 64);
  }
  if (lane == 0) {
    sh[0][wv] = mdiv;
    sh[1][wv] = mcfl;
    sh[2][wv] = clip;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int q = 1; q < kCellBlock / 64; ++q) {
      mdiv = nmax(sh[0][q], mdiv);
      mcfl = nmax(sh[1][q], mcfl);
      clip += sh[2][q];
    }
    part[blockIdx.x] = mdiv;
    part[kDiagBlocks + blockIdx.x] = mcfl;
    part[2 * kDiagBlocks + blockIdx.x] = clip;
  }
}

template <class T>
void launch_diag(Grid& g, const Params<T>& P) {
  const int turb = g.cfg.turb_model == UF_TURB_KOMEGA;
  hipLaunchKernelGGL(k_diag<T>, dim3(kDiagBlocks), dim3(kCellBlock), 0, g.stream, P, (const T*)g.Q[g.cur][0],
                     (const T*)g.Q[g.cur][1], (const T*)g.Q[g.cur][2], (const T*)g.NUT, turb, g.diag);
}

template <class T>
void launch_porosity(Grid& g, const Params<T>& P, const void* phi) {
  const uf_config& c = g.cfg;
  hipLaunchKernelGGL(k_porosity<T>, cell_grid(P.L), dim3(kCellBlock), 0, g.stream, P, (const T*)phi, (T*)g.C,
                     (T*)g.PHI, T(c.Cd * c.a), T(c.e), T(c.b));
}

template <class T>
void launch_cell_fill(Grid& g, const Params<T>& P, void* q, double value, int use_inlet, double inlet_value) {
  hipLaunchKernelGGL(k_cell_fill<T>, cell_grid(P.L), dim3(kCellBlock), 0, g.stream, P, (T*)q, T(value), use_inlet,
                     T(inlet_value));
}

template <class T, int MODE>
static void pack_field(Grid& g, const Params<T>& P, int field, const void* src, void* dst, int use_inlet = 0,
                       double inlet = 0.0, int* nf = nullptr) {
  int e[3] = {P.L.nx, P.L.ny, P.L.nz};
  if (field >= 0 && field < 3) e[field] += 1;
  const int gx = (e[1] * e[2] + kPackLoads * kCellBlock - 1) / (kPackLoads * kCellBlock);
  hipLaunchKernelGGL((k_pack<T, MODE>), dim3((unsigned)gx * (unsigned)e[0]), dim3(kCellBlock), 0, g.stream, P, gx,
                     e[1], e[2], (const T*)src, (T*)dst, use_inlet, T(inlet), nf);
}

template <class T>
void launch_pack(Grid& g, const Params<T>& P, const void* src, void* dst, int field, int unpack) {
  if (unpack) pack_field<T, PACK_PLAIN>(g, P, field, src, dst);
  else pack_field<T, PACK_GET>(g, P, field, src, dst);
}

template <class T>
void launch_put(Grid& g, const Params<T>& P, const void* src, void* dst, int field, int* nf) {
  switch (field) {
    case UF_U: pack_field<T, PACK_U>(g, P, field, src, dst, 0, 0.0, nf); break;
    case UF_V: pack_field<T, PACK_V>(g, P, field, src, dst, 0, 0.0, nf); break;
    case UF_W: pack_field<T, PACK_W>(g, P, field, src, dst, 0, 0.0, nf); break;
    case UF_K: pack_field<T, PACK_CELL>(g, P, field, src, dst, 1, g.k_in, nf); break;
    case UF_OMEGA: pack_field<T, PACK_CELL>(g, P, field, src, dst, 1, g.w_in, nf); break;
    case UF_NUT: pack_field<T, PACK_CELL>(g, P, field, src, dst, 0, 0.0, nf); break;
    default: pack_field<T, PACK_PLAIN>(g, P, field, src, dst, 0, 0.0, nf); break;   // pressure: zero ghosts
  }
}

template <class T>
void launch_check_range(Grid& g, const void* phi, size_t n) {
  const int blocks = (int)std::min<size_t>((n + kCellBlock - 1) / kCellBlock, 4096);
  hipLaunchKernelGGL(k_check_range<T>, dim3(blocks), dim3(kCellBlock), 0, g.stream, (const T*)phi, n, g.flag);
}

template void launch_plane_objective<float>(Grid&, int, double, double, double, double, double*, int);
template void launch_plane_objective<double>(Grid&, int, double, double, double, double, double*, int);
template void launch_region_field_diff<float>(Grid&, const int[6], const void*, double*, int);
template void launch_region_field_diff<double>(Grid&, const int[6], const void*, double*, int);
template void launch_region_speed<float>(Grid&, const int[6], double*, int);
template void launch_region_speed<double>(Grid&, const int[6], double*, int);

#define UF_INST(T)                                                                                            \
  template void launch_turb<T>(Grid&, const Params<T>&, void* const[3], const void*, const void*, void*, void*, \
                               void*, int, const int*);                                                     \
  template void launch_diag<T>(Grid&, const Params<T>&);                                                     \
  template void launch_porosity<T>(Grid&, const Params<T>&, const void*);                                    \
  template void launch_put<T>(Grid&, const Params<T>&, const void*, void*, int, int*);                       \
  template void launch_pack<T>(Grid&, const Params<T>&, const void*, void*, int, int);                       \
  template void launch_check_range<T>(Grid&, const void*, size_t);                                           \
  template void launch_cell_fill<T>(Grid&, const Params<T>&, void*, double, int, double);                    \
  template void launch_turb_multi<T>(const MultiCase<T>*, const CaseStarts&, int, int, int, const int*, int, hipStream_t);
UF_INST(float)
UF_INST(double)
#undef UF_INST

}  // namespace uf
