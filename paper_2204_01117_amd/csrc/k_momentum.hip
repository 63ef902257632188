// Momentum stages of the RANS step on the staggered grid (Sec. 3): MacCormack
// semi-Lagrangian advection, explicit (nu + nu_t) diffusion, the porosity drag
// and the pressure-gradient correction of the projection.
//
// Each kernel handles the three face components: a thread owns the faces
// u(i,j,k), v(i,j,k), w(i,j,k) of the cell corner (i,j,k), i in [0, nx],
// (j, k) in [0, ny] x [0, nz], flattened z fastest so that a wavefront
// reads consecutive memory.  Fixed boundary normal faces get their
// Dirichlet value; ghosts are written by store_face.
#include <type_traits>

#include "march.h"

namespace uf {

// ------------------------------------------------------------- advection --
// A NaN velocity clamps the trace to position -1, where the sample is finite:
// every path adds nan_if(), so that such a face is NaN in the predictor's
// field too.
template <int C, class T>
__device__ __forceinline__ T advect_fwd_value(const Params<T>& P, const T* __restrict__ U, const T* __restrict__ V,
                                              const T* __restrict__ W, long long o, int i, int j, int k) {
  T vel[3];
  face_velocity<C>(P.L, U, V, W, o, vel);
  const T* q = C == 0 ? U : (C == 1 ? V : W);
  T mn, mx;
  return sample<C, false>(P.L, q, i, j, k, -(vel[0] * P.dth[0]), -(vel[1] * P.dth[1]), -(vel[2] * P.dth[2]), &mn,
                          &mx) +
         nan_if<T>(any_nan3(vel));
}

template <int C, class T>
__device__ __forceinline__ T advect_corr_value(const Params<T>& P, const T* __restrict__ U, const T* __restrict__ V,
                                               const T* __restrict__ W, const T* __restrict__ qhat, long long o, int i,
                                               int j, int k) {
  T vel[3];
  face_velocity<C>(P.L, U, V, W, o, vel);
  const T* q = C == 0 ? U : (C == 1 ? V : W);
  const T di = vel[0] * P.dth[0], dj = vel[1] * P.dth[1], dk = vel[2] * P.dth[2];
  T mn, mx;
  // forward trace again: same value as stored in qhat, plus the sample range
  const T qh = sample<C, true>(P.L, q, i, j, k, -di, -dj, -dk, &mn, &mx);
  T d0, d1;
  const T qc = sample<C, false>(P.L, qhat, i, j, k, di, dj, dk, &d0, &d1);
  const T qt = qh + T(0.5) * (q[o] - qc);
  return nmin(nmax(qt, mn), mx) + nan_if<T>(any_nan3(vel));
}

template <class T>
__global__ __launch_bounds__(kFaceBlock) void k_advect_fwd(Params<T> P, const T* __restrict__ U, const T* __restrict__ V,
                                                           const T* __restrict__ W, T* __restrict__ Uh,
                                                           T* __restrict__ Vh, T* __restrict__ Wh) {
  UF_FACE_THREAD(P.L);
  const long long o = P.L.at(i, j, k);
  const T a0 = advect_fwd_value<0>(P, U, V, W, o, i, j, k);
  const T a1 = advect_fwd_value<1>(P, U, V, W, o, i, j, k);
  const T a2 = advect_fwd_value<2>(P, U, V, W, o, i, j, k);
  finish_face<0>(P, Uh, i, j, k, a0);
  finish_face<1>(P, Vh, i, j, k, a1);
  finish_face<2>(P, Wh, i, j, k, a2);
}

template <class T>
__global__ __launch_bounds__(kFaceBlock) void k_advect_corr(Params<T> P, const T* __restrict__ U, const T* __restrict__ V,
                                                            const T* __restrict__ W, const T* __restrict__ Uh,
                                                            const T* __restrict__ Vh, const T* __restrict__ Wh,
                                                            T* __restrict__ Uo, T* __restrict__ Vo, T* __restrict__ Wo) {
  UF_FACE_THREAD(P.L);
  const long long o = P.L.at(i, j, k);
  const T a0 = advect_corr_value<0>(P, U, V, W, Uh, o, i, j, k);
  const T a1 = advect_corr_value<1>(P, U, V, W, Vh, o, i, j, k);
  const T a2 = advect_corr_value<2>(P, U, V, W, Wh, o, i, j, k);
  finish_face<0>(P, Uo, i, j, k, a0);
  finish_face<1>(P, Vo, i, j, k, a1);
  finish_face<2>(P, Wo, i, j, k, a2);
}

// The advection kernels with 32-bit offsets (arrays below 4 GiB).  The
// predictor gathers the face velocities of the thread's three faces, then
// issues the trilinear loads of all three components at once, then
// evaluates: two memory round trips instead of one per component.
template <class T>
__device__ __forceinline__ void advect_fwd32_faces(const Params<T>& P, const T* __restrict__ U, const T* __restrict__ V, const T* __restrict__ W, T* __restrict__ Uh, T* __restrict__ Vh, T* __restrict__ Wh, int bx, int ib) {
  UF_FACE_POINT(P.L, bx, ib);
  const Layout& L = P.L;
  const unsigned o = (unsigned)L.at(i, j, k);
  T v0[3], v1[3], v2[3];
  face_velocity32<0>(L, U, V, W, o, v0);
  face_velocity32<1>(L, U, V, W, o, v1);
  face_velocity32<2>(L, U, V, W, o, v2);
  const Tri<T> t0 = tri_corner<0>(L, i, j, k, -(v0[0] * P.dth[0]), -(v0[1] * P.dth[1]), -(v0[2] * P.dth[2]));
  const Tri<T> t1 = tri_corner<1>(L, i, j, k, -(v1[0] * P.dth[0]), -(v1[1] * P.dth[1]), -(v1[2] * P.dth[2]));
  const Tri<T> t2 = tri_corner<2>(L, i, j, k, -(v2[0] * P.dth[0]), -(v2[1] * P.dth[1]), -(v2[2] * P.dth[2]));
  T s0[8], s1[8], s2[8];
  tri_load(U, L, t0.o, s0);
  tri_load(V, L, t1.o, s1);
  tri_load(W, L, t2.o, s2);
  // NaN for a NaN velocity, added rather than selected: a select would let
  // the compiler move the loads under a branch
  const T a0 = tri_eval(t0, s0) + nan_if<T>(any_nan3(v0));
  const T a1 = tri_eval(t1, s1) + nan_if<T>(any_nan3(v1));
  const T a2 = tri_eval(t2, s2) + nan_if<T>(any_nan3(v2));
  finish_face<0>(P, Uh, i, j, k, a0);
  finish_face<1>(P, Vh, i, j, k, a1);
  finish_face<2>(P, Wh, i, j, k, a2);
}

template <class T>
__global__ __launch_bounds__(kFaceBlock) void k_advect_fwd32(Params<T> P, const T* __restrict__ U, const T* __restrict__ V, const T* __restrict__ W, T* __restrict__ Uh, T* __restrict__ Vh, T* __restrict__ Wh) {
  int bx, ib;
  if (!face_block(P.L, bx, ib)) return;
  advect_fwd32_faces(P, U, V, W, Uh, Vh, Wh, bx, ib);
}

// The corrector with 32-bit offsets, one component: the forward trace
// again (its value and the range of its eight samples), the reverse trace
// through the traced field, the correction and the clamp.
template <int C, class T>
__device__ __forceinline__ T advect_corr32_value(const Params<T>& P, const T* __restrict__ U,
                                                 const T* __restrict__ V, const T* __restrict__ W,
                                                 const T* __restrict__ qhat, unsigned o, int i, int j, int k) {
  T vel[3];
  face_velocity32<C>(P.L, U, V, W, o, vel);
  const T* q = C == 0 ? U : (C == 1 ? V : W);
  const T di = vel[0] * P.dth[0], dj = vel[1] * P.dth[1], dk = vel[2] * P.dth[2];
  const Tri<T> fw = tri_corner<C>(P.L, i, j, k, -di, -dj, -dk);
  const Tri<T> bw = tri_corner<C>(P.L, i, j, k, di, dj, dk);
  T sf[8], sb[8];
  tri_load(q, P.L, fw.o, sf);
  tri_load(qhat, P.L, bw.o, sb);
  T mn, mx;
  tri_range(sf, mn, mx);
  const T qh = tri_eval(fw, sf);
  const T qc = tri_eval(bw, sb);
  const T qt = qh + T(0.5) * (vel[C] - qc);
  return nmin(nmax(qt, mn), mx) + nan_if<T>(any_nan3(vel));
}

// The corrector of one component comp of the faces of logical block (bx,
// ib).  The kernels give each component blocks of its own: a thread then
// holds one component's samples (57 registers instead of 110 for all three)
// and twice as many wavefronts hide the gathers' latency (879 -> 781 us per
// launch at 512x512x128).
template <class T>
__device__ __forceinline__ void advect_corr32_component(const Params<T>& P, const T* __restrict__ U, const T* __restrict__ V, const T* __restrict__ W, const T* __restrict__ Uh, const T* __restrict__ Vh, const T* __restrict__ Wh, T* __restrict__ Uo, T* __restrict__ Vo, T* __restrict__ Wo, int comp, int bx, int ib) {
  UF_FACE_POINT(P.L, bx, ib);
  const unsigned o = (unsigned)P.L.at(i, j, k);
  if (comp == 0) {
    const T a = advect_corr32_value<0>(P, U, V, W, Uh, o, i, j, k);
    finish_face<0>(P, Uo, i, j, k, a);
  } else if (comp == 1) {
    const T a = advect_corr32_value<1>(P, U, V, W, Vh, o, i, j, k);
    finish_face<1>(P, Vo, i, j, k, a);
  } else {
    const T a = advect_corr32_value<2>(P, U, V, W, Wh, o, i, j, k);
    finish_face<2>(P, Wo, i, j, k, a);
  }
}

// Single grid, launched on xcd_grid(3 face_gx, nx + 1): the three
// components of a face block are neighbours in the logical order, so they
// run together on one XCD and share the velocity and sample loads in its
// L2 (with the component as a grid dimension of its own each array was
// fetched from HBM three times).
template <class T>
__global__ __launch_bounds__(kFaceBlock) void k_advect_corr32(Params<T> P, const T* __restrict__ U, const T* __restrict__ V, const T* __restrict__ W, const T* __restrict__ Uh, const T* __restrict__ Vh, const T* __restrict__ Wh, T* __restrict__ Uo, T* __restrict__ Vo, T* __restrict__ Wo) {
  const int gx = face_gx(P.L), gy = P.L.nx + 1;
  const int per = (int)(gridDim.x >> 3);
  const int e = (int)(blockIdx.x & 7u) * per + (int)(blockIdx.x >> 3);
  if (e >= 3 * gx * gy) return;
  int bx, ib;
  band_map(gx, gy, kFaceBand, e / 3, bx, ib);
  advect_corr32_component(P, U, V, W, Uh, Vh, Wh, Uo, Vo, Wo, e % 3, bx, ib);
}

// ------------------------------------------------- advection, marching -----
// Arrays: 0 to 2 the velocity, 3 to 5 (corrector) the predictor's field.

template <int C, int SHAPE, class T>
__device__ __forceinline__ T march_fwd(const Params<T>& P, const Planes<SHAPE, 3, T>& A, int i, int j, int k) {
  T vel[3];
  march_velocity<C>(A, vel);
  const T d[3] = {vel[0] * P.dth[0], vel[1] * P.dth[1], vel[2] * P.dth[2]};
  if (march_near(d)) {
    Tri<T> t;
    T v[8];
    march_samples(A, C, -d[0], -d[1], -d[2], t, v);
    return tri_eval(t, v);
  }
  T mn, mx;
  return sample<C, false>(P.L, A.src[C], i, j, k, -d[0], -d[1], -d[2], &mn, &mx) + nan_if<T>(any_nan3(vel));
}

template <int C, int SHAPE, class T>
__device__ __forceinline__ T march_corr(const Params<T>& P, const Planes<SHAPE, 6, T>& A, int i, int j, int k) {
  T vel[3];
  march_velocity<C>(A, vel);
  const T d[3] = {vel[0] * P.dth[0], vel[1] * P.dth[1], vel[2] * P.dth[2]};
  T qh, qc, mn, mx, nan = T(0);
  if (march_near(d)) {
    Tri<T> t;
    T v[8];
    march_samples(A, C, -d[0], -d[1], -d[2], t, v);
    tri_range(v, mn, mx);
    qh = tri_eval(t, v);
    march_samples(A, 3 + C, d[0], d[1], d[2], t, v);
    qc = tri_eval(t, v);
  } else {
    T d0, d1;
    qh = sample<C, true>(P.L, A.src[C], i, j, k, -d[0], -d[1], -d[2], &mn, &mx);
    qc = sample<C, false>(P.L, A.src[3 + C], i, j, k, d[0], d[1], d[2], &d0, &d1);
    nan = nan_if<T>(any_nan3(vel));
  }
  const T qt = qh + T(0.5) * (vel[C] - qc);
  return nmin(nmax(qt, mn), mx) + nan;
}

// ------------------------------------------------------------- diffusion --
template <int C, class T>
__device__ __forceinline__ T diffuse_value(const Params<T>& P, const T* __restrict__ q, const T* __restrict__ nut,
                                           long long o) {
  const Layout& L = P.L;
  const T qc = q[o];
  const T lap = (q[o + L.SX] - T(2) * qc + q[o - L.SX]) * P.ih2[0] +
                (q[o + L.PZ] - T(2) * qc + q[o - L.PZ]) * P.ih2[1] +
                (q[o + 1] - T(2) * qc + q[o - 1]) * P.ih2[2];
  const T nuf = P.nu + T(0.5) * (nut[o - stride<C>(L)] + nut[o]);
  return qc + P.dt * nuf * lap;
}

template <class T>
__device__ __forceinline__ void diffuse_faces(const Params<T>& P, const T* __restrict__ U, const T* __restrict__ V, const T* __restrict__ W, const T* __restrict__ NUT, T* __restrict__ Uo, T* __restrict__ Vo, T* __restrict__ Wo, int bx, int ib) {
  UF_FACE_POINT(P.L, bx, ib);
  const long long o = P.L.at(i, j, k);
  const T a0 = diffuse_value<0>(P, U, NUT, o);
  const T a1 = diffuse_value<1>(P, V, NUT, o);
  const T a2 = diffuse_value<2>(P, W, NUT, o);
  finish_face<0>(P, Uo, i, j, k, a0);
  finish_face<1>(P, Vo, i, j, k, a1);
  finish_face<2>(P, Wo, i, j, k, a2);
}

template <class T>
__global__ __launch_bounds__(kFaceBlock) void k_diffuse(Params<T> P, const T* __restrict__ U, const T* __restrict__ V, const T* __restrict__ W, const T* __restrict__ NUT, T* __restrict__ Uo, T* __restrict__ Vo, T* __restrict__ Wo) {
  int bx, ib;
  if (!face_block(P.L, bx, ib)) return;
  diffuse_faces(P, U, V, W, NUT, Uo, Vo, Wo, bx, ib);
}

// ------------------------------------------------------------ porosity drag
// The factor of a face with velocity vector (a, b, d) between cells of drag
// coefficients c0 and c1.  The speed's sum is written in the fused operations
// it is made of: a batch's kernel and a grid's own give the same bits.
template <class T>
__device__ __forceinline__ T drag_factor(const Params<T>& P, T a, T b, T d, T c0, T c1) {
  const T speed = sqrt(fma(d, d, fma(b, b, a * a)));
  const T cf = T(0.5) * (c0 + c1);
  return nmax(T(0), T(1) - P.dt * cf * speed);
}

template <int C, class T>
__device__ __forceinline__ T drag_value(const Params<T>& P, const T* __restrict__ U, const T* __restrict__ V,
                                        const T* __restrict__ W, const T* __restrict__ Cc, long long o) {
  T vel[3];
  face_velocity<C>(P.L, U, V, W, o, vel);
  return drag_factor(P, vel[0], vel[1], vel[2], Cc[o - stride<C>(P.L)], Cc[o]) * vel[C];
}

template <class T>
__device__ __forceinline__ void drag_faces(const Params<T>& P, const T* __restrict__ U, const T* __restrict__ V, const T* __restrict__ W, const T* __restrict__ Cc, T* __restrict__ Uo, T* __restrict__ Vo, T* __restrict__ Wo, int* nf, int bx, int ib) {
  UF_FACE_POINT(P.L, bx, ib);
  const long long o = P.L.at(i, j, k);
  const T a0 = drag_value<0>(P, U, V, W, Cc, o);
  const T a1 = drag_value<1>(P, U, V, W, Cc, o);
  const T a2 = drag_value<2>(P, U, V, W, Cc, o);
  // a NaN/Inf in an owned face raises the state's non-finite flag (every
  // writer stores 1, so the race is benign)
  if ((owns_face<0, T>(P.L, i, j, k) && !isfinite(a0)) || (owns_face<1, T>(P.L, i, j, k) && !isfinite(a1)) ||
      (owns_face<2, T>(P.L, i, j, k) && !isfinite(a2)))
    *nf = 1;
  finish_face<0>(P, Uo, i, j, k, a0);
  finish_face<1>(P, Vo, i, j, k, a1);
  finish_face<2>(P, Wo, i, j, k, a2);
}

template <class T>
__global__ __launch_bounds__(kFaceBlock) void k_drag(Params<T> P, const T* __restrict__ U, const T* __restrict__ V, const T* __restrict__ W, const T* __restrict__ Cc, T* __restrict__ Uo, T* __restrict__ Vo, T* __restrict__ Wo, int* nf) {
  int bx, ib;
  if (!face_block(P.L, bx, ib)) return;
  drag_faces(P, U, V, W, Cc, Uo, Vo, Wo, nf, bx, ib);
}

template <int C, class T>
__device__ __forceinline__ T project_value(const Params<T>& P, const T* __restrict__ q, const T* __restrict__ p,
                                           long long o) {
  const T grad = (p[o] - p[o - stride<C>(P.L)]) * P.ih[C];
  return q[o] - P.dt_rho * grad;
}

// What a stage reads (the velocity first) and writes.
template <class T>
struct MarchArgs {
  const T* in[6];
  T* out[3];
  int* nf;
};

// Face (i, j, k) of component C of a stage, from memory.
template <int STAGE, int C, class T>
__device__ __forceinline__ void face_from_memory(const Params<T>& P, const MarchArgs<T>& M, int i, int j, int k) {
  const Layout& L = P.L;
  const long long o = L.at(i, j, k);
  const T *U = M.in[0], *V = M.in[1], *W = M.in[2];
  T v;
  if constexpr (STAGE == MS_ADVECT_FWD) v = advect_fwd_value<C>(P, U, V, W, o, i, j, k);
  else if constexpr (STAGE == MS_ADVECT_CORR) v = advect_corr_value<C>(P, U, V, W, M.in[3 + C], o, i, j, k);
  else if constexpr (STAGE == MS_DIFFUSE) v = diffuse_value<C>(P, M.in[C], M.in[3], o);
  else if constexpr (STAGE == MS_DRAG) v = drag_value<C>(P, U, V, W, M.in[3], o);
  else v = project_value<C>(P, M.in[C], M.in[3], o);
  if (STAGE == MS_DRAG && !isfinite(v) && owns_face<C, T>(L, i, j, k)) *M.nf = 1;
  finish_face<C>(P, M.out[C], i, j, k, v);
}

// A stage of a small grid, one component per block: the launch takes as long
// as one thread's chain, which is then a third as long (split_use).
template <int STAGE, class T>
__global__ __launch_bounds__(kFaceBlock) void k_face_split(Params<T> P, MarchArgs<T> M, const int* __restrict__ gate) {
  if (gate && !*gate) return;
  const int gx = face_gx(P.L), e = (int)blockIdx.x, b = e / 3, comp = e - 3 * b;
  UF_FACE_POINT(P.L, b % gx, b / gx);
  if (comp == 0) face_from_memory<STAGE, 0>(P, M, i, j, k);
  else if (comp == 1) face_from_memory<STAGE, 1>(P, M, i, j, k);
  else face_from_memory<STAGE, 2>(P, M, i, j, k);
}

// ------------------------------------------ the stages that march along x --
constexpr int march_arrays(int stage) { return stage == MS_ADVECT_CORR ? 6 : 3; }

template <int STAGE, int C, int SHAPE, int NA, class T>
__device__ __forceinline__ T march_value(const Params<T>& P, const Planes<SHAPE, NA, T>& A, int i, int j, int k) {
  if constexpr (STAGE == MS_ADVECT_FWD) return march_fwd<C>(P, A, i, j, k);
  else return march_corr<C>(P, A, i, j, k);
}

template <int STAGE, int SHAPE, class T>
__device__ __forceinline__ void march_faces(const Params<T>& P, const March& G, const MarchArgs<T>& M, T* lds, int tile,
                                            int chunk) {
  const Layout& L = P.L;
  Planes<SHAPE, march_arrays(STAGE), T> A;
#pragma unroll
  for (int a = 0; a < march_arrays(STAGE); ++a) A.src[a] = M.in[a];
  int j0, k0;
  MarchLane c = march_lane<SHAPE>(L, G, tile, L.ny - 2, L.nz + 3, L.nz, L.nz + 1, j0, k0);
  A.init(L, lds, j0, k0, G.TK);
  const int i0 = 1 + chunk * G.len;
  march(A, i0, min(L.nx - 1, i0 + G.len), [&](int i) {
    if (!c.active) return;
    auto face = [&](auto tag) {
      constexpr int C = decltype(tag)::value;
      A.q = C == 2 ? c.qb : c.qa;
      const T v = march_value<STAGE, C>(P, A, i, c.j, min(max(c.k, 0), C == 2 ? L.nz : L.nz - 1));
      march_put<C>(P, M.out[C], c.k, c.oc, i, v);
    };
    face(std::integral_constant<int, 0>());
    face(std::integral_constant<int, 1>());
    face(std::integral_constant<int, 2>());
  });
}

template <int STAGE, class T>
__device__ __forceinline__ void march_edge(const Params<T>& P, const MarchArgs<T>& M, int e) {
  int i, j, k;
  if (!march_edge_corner(P.L, e, i, j, k)) return;
  face_from_memory<STAGE, 0>(P, M, i, j, k);
  face_from_memory<STAGE, 1>(P, M, i, j, k);
  face_from_memory<STAGE, 2>(P, M, i, j, k);
}

template <int STAGE, int SHAPE, class T>
__global__ __launch_bounds__(kMarch, 6) void k_march(Params<T> P, March G, MarchArgs<T> M) {
  __shared__ T lds[Planes<SHAPE, march_arrays(STAGE), T>::LDS];
  int tile, chunk;
  if (!march_block(G, tile, chunk)) return;
  if (tile < 0) march_edge<STAGE>(P, M, chunk * kMarch + (int)threadIdx.x);
  else march_faces<STAGE, SHAPE>(P, G, M, lds, tile, chunk);
}

// ------------------------------------------------ projection (velocity part)
template <class T>
__device__ __forceinline__ void project_faces(const Params<T>& P, const T* __restrict__ U, const T* __restrict__ V, const T* __restrict__ W, const T* __restrict__ Pp, T* __restrict__ Uo, T* __restrict__ Vo, T* __restrict__ Wo, int bx, int ib) {
  UF_FACE_POINT(P.L, bx, ib);
  const long long o = P.L.at(i, j, k);
  const T a0 = project_value<0>(P, U, Pp, o);
  const T a1 = project_value<1>(P, V, Pp, o);
  const T a2 = project_value<2>(P, W, Pp, o);
  finish_face<0>(P, Uo, i, j, k, a0);
  finish_face<1>(P, Vo, i, j, k, a1);
  finish_face<2>(P, Wo, i, j, k, a2);
}

// gate: when given, the launch does nothing unless *gate is set (a step's
// projection enqueued before the host has read whether the solve ended).
template <class T>
__global__ __launch_bounds__(kFaceBlock) void k_project(Params<T> P, const T* __restrict__ U, const T* __restrict__ V, const T* __restrict__ W, const T* __restrict__ Pp, T* __restrict__ Uo, T* __restrict__ Vo, T* __restrict__ Wo, const int* __restrict__ gate) {
  if (gate && !*gate) return;
  int bx, ib;
  if (!face_block(P.L, bx, ib)) return;
  project_faces(P, U, V, W, Pp, Uo, Vo, Wo, bx, ib);
}

// The projection on large grids: a lane (k from -1 to nz + 1) of the rows and
// planes off the sides along x and y, kProjPlanes planes at a time with all
// their loads in flight, ghosts along z by lanes of their own (march.h);
// blocks of the edges' corners first.  A thread per corner had too few bytes in
// flight (seven loads a thread) and spent half of its instructions on the
// boundary rules: 37 -> 26 us at 256x256x64 in FP32, 273 -> 172 at
// 512x512x128 (5.6 TB/s; two to eight planes: within 4%).
constexpr int kProjPlanes = 4;

template <class T>
__global__ __launch_bounds__(kFaceBlock) void k_project_planes(Params<T> P, int edge, int gx, const T* __restrict__ U,
                                                               const T* __restrict__ V, const T* __restrict__ W,
                                                               const T* __restrict__ Pp, T* __restrict__ Uo,
                                                               T* __restrict__ Vo, T* __restrict__ Wo,
                                                               const int* __restrict__ gate) {
  if (gate && !*gate) return;
  const Layout& L = P.L;
  int b = (int)blockIdx.x;
  if (b < edge) {
    int i, j, k;
    if (!march_edge_corner(L, b * kFaceBlock + (int)threadIdx.x, i, j, k)) return;
    const long long o = L.at(i, j, k);
    finish_face<0>(P, Uo, i, j, k, project_value<0>(P, U, Pp, o));
    finish_face<1>(P, Vo, i, j, k, project_value<1>(P, V, Pp, o));
    finish_face<2>(P, Wo, i, j, k, project_value<2>(P, W, Pp, o));
    return;
  }
  b -= edge;
  const int per = ((int)gridDim.x - edge) >> 3;   // XCD-contiguous, as xcd_block()
  b = (b & 7) * per + (b >> 3);
  const int c = b / gx, p = (b - c * gx) * kFaceBlock + (int)threadIdx.x, w = L.nz + 3;
  const int i0 = 1 + c * kProjPlanes;
  if (i0 > L.nx - 2 || p >= (L.ny - 2) * w) return;
  const int j = p / w, k = p - j * w - 1;
  const unsigned row = (unsigned)(j + 2) * (unsigned)L.PZ + 1u;
  const unsigned oa = row + (unsigned)min(max(k, 0), L.nz - 1), ob = row + (unsigned)min(max(k, 0), L.nz);
  const unsigned oc = row + (unsigned)k;
  T u[kProjPlanes], v[kProjPlanes], wv[kProjPlanes], pc[kProjPlanes], py[kProjPlanes], pb[kProjPlanes], pz[kProjPlanes];
  T px = (Pp + (long long)i0 * L.SX)[oa];
#pragma unroll
  for (int q = 0; q < kProjPlanes; ++q) {
    const long long pl = (long long)(min(i0 + q, L.nx - 2) + 1) * L.SX;
    u[q] = (U + pl)[oa];
    v[q] = (V + pl)[oa];
    wv[q] = (W + pl)[ob];
    pc[q] = (Pp + pl)[oa];
    py[q] = (Pp + pl)[oa - (unsigned)L.PZ];
    pb[q] = (Pp + pl)[ob];
    pz[q] = (Pp + pl)[ob - 1u];
  }
#pragma unroll
  for (int q = 0; q < kProjPlanes; ++q) {
    const int i = i0 + q;
    if (i > L.nx - 2) break;
    march_put<0>(P, Uo, k, oc, i, u[q] - P.dt_rho * ((pc[q] - px) * P.ih[0]));
    march_put<1>(P, Vo, k, oc, i, v[q] - P.dt_rho * ((pc[q] - py[q]) * P.ih[1]));
    march_put<2>(P, Wo, k, oc, i, wv[q] - P.dt_rho * ((pb[q] - pz[q]) * P.ih[2]));
    px = pc[q];
  }
}

// ------------------------------- diffusion and drag, several planes at once --
// As the projection: a thread takes NP planes of its lane with all their
// loads in flight, carries what two planes share, and leaves the edges'
// corners to blocks of their own.  All three components are evaluated at one
// column, k clamped to [0, nz - 1], so the side above must not be an outlet
// (w there is a fixed face).  Diffusion 43 -> 27 us at 256x256x64, 64 -> 49 at
// 450x300x40, 347 -> 287 at 512x512x128; drag 51 -> 35, 70 -> 50, 353 -> 247
// (FP32; one to four planes: within 10%; with their planes in LDS as the
// advection 30, 46 and 290, 39, 49 and 290).  The L1's address path bounds
// them: 18 and 14 loads per lane and plane.
template <int STAGE, class T>
struct PlaneCols;

// u, v, w at the column, its y and z neighbours; nu_t at the column and its
// lower neighbours.
template <class T>
struct PlaneCols<MS_DIFFUSE, T> {
  static constexpr int NP = 4;
  T qm[3], qc[3], nm;                          // plane i - 1; plane i; nu_t of plane i - 1
  T up[NP][3], nb[NP][3][4], nc[NP], ny[NP], nz[NP];
  __device__ __forceinline__ void start(const T* const (&in)[6], long long pm, long long pc, unsigned o, unsigned PZ) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      qm[a] = (in[a] + pm)[o];
      qc[a] = (in[a] + pc)[o];
    }
    nm = (in[3] + pm)[o];
  }
  __device__ __forceinline__ void load(int q, const T* const (&in)[6], long long pc, long long pp, unsigned o,
                                       unsigned PZ) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      up[q][a] = (in[a] + pp)[o];
      nb[q][a][0] = (in[a] + pc)[o - PZ];
      nb[q][a][1] = (in[a] + pc)[o + PZ];
      nb[q][a][2] = (in[a] + pc)[o - 1u];
      nb[q][a][3] = (in[a] + pc)[o + 1u];
    }
    nc[q] = (in[3] + pc)[o];
    ny[q] = (in[3] + pc)[o - PZ];
    nz[q] = (in[3] + pc)[o - 1u];
  }
  __device__ __forceinline__ void eval(const Params<T>& P, int q, T v[3]) {
    const T nlo[3] = {nm, ny[q], nz[q]};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const T c = qc[a];
      const T lap = (up[q][a] - T(2) * c + qm[a]) * P.ih2[0] + (nb[q][a][1] - T(2) * c + nb[q][a][0]) * P.ih2[1] +
                    (nb[q][a][3] - T(2) * c + nb[q][a][2]) * P.ih2[2];
      const T nuf = P.nu + T(0.5) * (nlo[a] + nc[q]);
      v[a] = c + P.dt * nuf * lap;
      qm[a] = c;
      qc[a] = up[q][a];
    }
    nm = nc[q];
  }
};

// The columns of u, v, w and the drag coefficient that the three faces'
// velocity vectors average.
template <class T>
struct PlaneCols<MS_DRAG, T> {
  static constexpr int NP = 4;
  T u[3], vm[2], wm[2], cm;                    // u of plane i at 0, -y, -z; v, w, C of plane i - 1
  T un[NP][3], v[NP][4], w[NP][4], c[NP][3];
  __device__ __forceinline__ void start(const T* const (&in)[6], long long pm, long long pc, unsigned o, unsigned PZ) {
    u[0] = (in[0] + pc)[o];
    u[1] = (in[0] + pc)[o - PZ];
    u[2] = (in[0] + pc)[o - 1u];
    vm[0] = (in[1] + pm)[o];
    vm[1] = (in[1] + pm)[o + PZ];
    wm[0] = (in[2] + pm)[o];
    wm[1] = (in[2] + pm)[o + 1u];
    cm = (in[3] + pm)[o];
  }
  __device__ __forceinline__ void load(int q, const T* const (&in)[6], long long pc, long long pp, unsigned o,
                                       unsigned PZ) {
    un[q][0] = (in[0] + pp)[o];
    un[q][1] = (in[0] + pp)[o - PZ];
    un[q][2] = (in[0] + pp)[o - 1u];
    v[q][0] = (in[1] + pc)[o];
    v[q][1] = (in[1] + pc)[o + PZ];
    v[q][2] = (in[1] + pc)[o - 1u];
    v[q][3] = (in[1] + pc)[o - 1u + PZ];
    w[q][0] = (in[2] + pc)[o];
    w[q][1] = (in[2] + pc)[o + 1u];
    w[q][2] = (in[2] + pc)[o - PZ];
    w[q][3] = (in[2] + pc)[o - PZ + 1u];
    c[q][0] = (in[3] + pc)[o];
    c[q][1] = (in[3] + pc)[o - PZ];
    c[q][2] = (in[3] + pc)[o - 1u];
  }
  __device__ __forceinline__ void eval(const Params<T>& P, int q, T r[3]) {
    const T h = T(0.25);
    const T v0 = h * (vm[0] + vm[1] + v[q][0] + v[q][1]), w0 = h * (wm[0] + wm[1] + w[q][0] + w[q][1]);
    r[0] = drag_factor(P, u[0], v0, w0, cm, c[q][0]) * u[0];
    const T u1 = h * (u[1] + un[q][1] + u[0] + un[q][0]), w1 = h * (w[q][2] + w[q][3] + w[q][0] + w[q][1]);
    r[1] = drag_factor(P, u1, v[q][0], w1, c[q][1], c[q][0]) * v[q][0];
    const T u2 = h * (u[2] + un[q][2] + u[0] + un[q][0]), v2 = h * (v[q][2] + v[q][3] + v[q][0] + v[q][1]);
    r[2] = drag_factor(P, u2, v2, w[q][0], c[q][2], c[q][0]) * w[q][0];
#pragma unroll
    for (int m = 0; m < 3; ++m) u[m] = un[q][m];
    vm[0] = v[q][0];
    vm[1] = v[q][1];
    wm[0] = w[q][0];
    wm[1] = w[q][1];
    cm = c[q][0];
  }
};

template <int STAGE, class T>
__global__ __launch_bounds__(kFaceBlock) void k_planes(Params<T> P, int edge, int gx, MarchArgs<T> M) {
  using F = PlaneCols<STAGE, T>;
  const Layout& L = P.L;
  int b = (int)blockIdx.x;
  if (b < edge) {
    march_edge<STAGE>(P, M, b * kFaceBlock + (int)threadIdx.x);
    return;
  }
  b -= edge;
  const int per = ((int)gridDim.x - edge) >> 3;   // XCD-contiguous, as xcd_block()
  b = (b & 7) * per + (b >> 3);
  const int c = b / gx, p = (b - c * gx) * kFaceBlock + (int)threadIdx.x, w = L.nz + 3;
  const int i0 = 1 + c * F::NP;
  if (i0 > L.nx - 2 || p >= (L.ny - 2) * w) return;
  const int j = p / w, k = p - j * w - 1;
  const unsigned PZ = (unsigned)L.PZ, row = (unsigned)(j + 2) * PZ + 1u;
  const unsigned o = row + (unsigned)min(max(k, 0), L.nz - 1), oc = row + (unsigned)k;
  F f;
  f.start(M.in, (long long)i0 * L.SX, (long long)(i0 + 1) * L.SX, o, PZ);
#pragma unroll
  for (int q = 0; q < F::NP; ++q) {
    const long long pl = (long long)(min(i0 + q, L.nx - 2) + 1) * L.SX;
    f.load(q, M.in, pl, pl + L.SX, o, PZ);
  }
#pragma unroll
  for (int q = 0; q < F::NP; ++q) {
    const int i = i0 + q;
    if (i > L.nx - 2) break;
    T v[3];
    f.eval(P, q, v);
    // a NaN/Inf raises the state's non-finite flag (every writer stores 1, so
    // the race is benign)
    if (STAGE == MS_DRAG && !(isfinite(v[0]) && isfinite(v[1]) && isfinite(v[2]))) *M.nf = 1;
    march_put<0>(P, M.out[0], k, oc, i, v[0]);
    march_put<1>(P, M.out[1], k, oc, i, v[1]);
    march_put<2>(P, M.out[2], k, oc, i, v[2]);
  }
}

// ------------------------------------------------------------ initial state
// Initial state: the inflow profile on every face (fixed faces keep their
// boundary value).
template <int C, class T>
__global__ __launch_bounds__(kFaceBlock) void k_face_init(Params<T> P, T* __restrict__ q) {
  UF_FACE_THREAD(P.L);
  if (!owns_face<C, T>(P.L, i, j, k)) return;
  T val;
  if (!face_dirichlet<C>(P, i, j, k, &val)) val = inflow_comp(P, C, k);
  store_face<C>(q, P, i, j, k, val);
}

// ------------------------------------------------- several grids at once --
// One launch of a face stage for every case of a batch: the cases' logical
// blocks form one queue (case c owns [start[c], start[c + 1])),
// which a persistent grid walks -- every XCD takes a contiguous share and
// its blocks stride through it -- each block running the stage's per-block
// body with its case's parameters and buffers (read from the case table).
// Sets: sin is read, saux is the predictor's output the corrector reads,
// sout is written.
template <int S, class T>
__global__ __launch_bounds__(kFaceBlock) void k_faces_multi(const MultiCase<T>* __restrict__ mc, CaseStarts cs,
                                                            int band, int sin, int saux, int sout) {
  // the corrector's queue holds three entries (components) per face block
  constexpr int NC = S == MS_ADVECT_CORR ? 3 : 1;
  const int nb = (int)(gridDim.x >> 3);
  const int xcd = (int)(blockIdx.x & 7u), lid = (int)(blockIdx.x >> 3);
  const int total = NC * cs.start[cs.n];
  const int share = (total + 7) >> 3;
  const int lo = xcd * share, hi = min(total, lo + share);
  for (int le = lo + lid; le < hi; le += nb) {
    const int lb = le / NC;
    const int c = find_case(cs, lb);
    const MultiCase<T>& A = mc[c];
    int bx, ib;
    band_map(face_gx(A.P.L), A.P.L.nx + 1, band, lb - cs.start[c], bx, ib);
    T* const* qi = A.q[sin];
    T* const* qo = A.q[sout];
    if (S == MS_ADVECT_FWD) {
      advect_fwd32_faces(A.P, qi[0], qi[1], qi[2], qo[0], qo[1], qo[2], bx, ib);
    } else if (S == MS_ADVECT_CORR) {
      T* const* qa = A.q[saux];
      advect_corr32_component(A.P, qi[0], qi[1], qi[2], qa[0], qa[1], qa[2], qo[0], qo[1], qo[2], le - NC * lb, bx,
                              ib);
    } else if (S == MS_DIFFUSE) {
      diffuse_faces(A.P, qi[0], qi[1], qi[2], A.nut, qo[0], qo[1], qo[2], bx, ib);
    } else if (S == MS_DRAG) {
      drag_faces(A.P, qi[0], qi[1], qi[2], A.cc, qo[0], qo[1], qo[2], A.nf, bx, ib);
    } else {
      project_faces(A.P, qi[0], qi[1], qi[2], A.x, qo[0], qo[1], qo[2], bx, ib);
    }
  }
}

template <class T>
void launch_faces_multi(int stage, const MultiCase<T>* mc, const CaseStarts& cs, int band, int blocks, int sin,
                        int saux, int sout, hipStream_t stream) {
  const dim3 grid((unsigned)blocks), blk(kFaceBlock);
  switch (stage) {
    case MS_ADVECT_FWD:
      hipLaunchKernelGGL((k_faces_multi<MS_ADVECT_FWD, T>), grid, blk, 0, stream, mc, cs, band, sin, saux, sout);
      break;
    case MS_ADVECT_CORR:
      hipLaunchKernelGGL((k_faces_multi<MS_ADVECT_CORR, T>), grid, blk, 0, stream, mc, cs, band, sin, saux, sout);
      break;
    case MS_DIFFUSE:
      hipLaunchKernelGGL((k_faces_multi<MS_DIFFUSE, T>), grid, blk, 0, stream, mc, cs, band, sin, saux, sout);
      break;
    case MS_DRAG:
      hipLaunchKernelGGL((k_faces_multi<MS_DRAG, T>), grid, blk, 0, stream, mc, cs, band, sin, saux, sout);
      break;
    default:
      hipLaunchKernelGGL((k_faces_multi<MS_PROJECT, T>), grid, blk, 0, stream, mc, cs, band, sin, saux, sout);
      break;
  }
}

// ----------------------------------------------------------------- launchers
static inline dim3 face_grid(const Layout& L) { return xcd_grid(face_gx(L), L.nx + 1); }

template <int STAGE, class T>
static void launch_march(Grid& g, const Params<T>& P, void* const Q[3], void* const H[3], void* const O[3]) {
  const Layout& L = P.L;
  MarchArgs<T> M{{(const T*)Q[0], (const T*)Q[1], (const T*)Q[2]}, {(T*)O[0], (T*)O[1], (T*)O[2]}, nf_word(g)};
  if (H)
    for (int c = 0; c < 3; ++c) M.in[3 + c] = (const T*)H[c];
  const March G = march_geom(L.nx - 2, L.ny - 2, L.nz + 3, march_edges(L));
  auto go = [&](auto kernel) { launch_k(g, kernel, march_grid(G), dim3(kMarch), P, G, M); };
  if (G.shape == 0) go(k_march<STAGE, 0, T>);
  else if (G.shape == 1) go(k_march<STAGE, 1, T>);
  else go(k_march<STAGE, 2, T>);
}

// Several planes per thread: below about half a million cells there are too few
// threads (129x97x35 diffusion 10.0 against 8.9 us, drag 9.5 against 9.4,
// projection 9.7 against 9.6; 160x128x32 10.8, 10.4 and 9.7 against 11.1, 11.1
// and 10.6).
constexpr double kPlanesFaces = 4.5e5;

template <class T>
static bool planes_use(const Params<T>& P) {
  const Layout& L = P.L;
  return L.nx > 3 && L.ny > 3 && (double)L.nx * L.ny * L.nz >= kPlanesFaces && P.bc[4] != INLET && P.bc[5] != INLET;
}

template <int STAGE, class T>
static void launch_planes(Grid& g, const Params<T>& P, void* const Q[3], const void* cells, void* const O[3]) {
  const Layout& L = P.L;
  const MarchArgs<T> M{{(const T*)Q[0], (const T*)Q[1], (const T*)Q[2], (const T*)cells},
                       {(T*)O[0], (T*)O[1], (T*)O[2]}, nf_word(g)};
  constexpr int NP = PlaneCols<STAGE, T>::NP;
  const int edge = 8 * ((march_edges(L) + 8 * kFaceBlock - 1) / (8 * kFaceBlock));
  const int gx = ((L.ny - 2) * (L.nz + 3) + kFaceBlock - 1) / kFaceBlock, nc = (L.nx - 2 + NP - 1) / NP;
  launch_k(g, k_planes<STAGE, T>, dim3((unsigned)(edge + 8 * ((gx * nc + 7) / 8))), dim3(kFaceBlock), P, edge, gx, M);
}

// One component per block on small grids, us against three per thread:
// 64x32x16 predictor 7.1 -> 5.2, diffusion 6.3 -> 4.5, drag 6.5 -> 4.8,
// projection 6.5 -> 4.8; 96x64x32 10.7 -> 8.6 and 7.8, 7.7, 7.5 -> 7.9, 7.5,
// 7.9; 96x80x48 in FP64 16.3 -> 13.3 and 11.4, 10.7, 10.0 -> 10.9, 12.3, 10.4.
constexpr double kSplitPredictor = 4e5, kSplitFaces = 1e5;

template <class T>
static bool split_use(const Params<T>& P, double below) {
  return (double)P.L.nx * P.L.ny * P.L.nz < below;
}

template <int STAGE, class T>
static void launch_split(Grid& g, const Params<T>& P, void* const Q[3], const void* cells, void* const O[3],
                         const int* gate = nullptr) {
  const MarchArgs<T> M{{(const T*)Q[0], (const T*)Q[1], (const T*)Q[2], (const T*)cells},
                       {(T*)O[0], (T*)O[1], (T*)O[2]}, nf_word(g)};
  launch_k(g, k_face_split<STAGE, T>, dim3(3u * (unsigned)face_gx(P.L) * (unsigned)(P.L.nx + 1)), dim3(kFaceBlock), P, M,
           gate);
}

template <class T>
void launch_advect(Grid& g, const Params<T>& P, void* const Qin[3], void* const Qhat[3], void* const Qout[3]) {
  const dim3 grid = face_grid(P.L);
  if constexpr (sizeof(T) == 4) if (march_pays(P, kMarchFaces)) {
    {
      TimedLaunch tl(g, UF_TK_ADVECT_FWD);
      launch_march<MS_ADVECT_FWD, T>(g, P, Qin, nullptr, Qhat);
    }
    TimedLaunch tl(g, UF_TK_ADVECT_CORR);
    launch_march<MS_ADVECT_CORR, T>(g, P, Qin, Qhat, Qout);
    return;
  }
  if (offsets_fit_32(P.L, sizeof(T))) {
    if (split_use(P, kSplitPredictor)) {
      TimedLaunch tl(g, UF_TK_ADVECT_FWD);
      launch_split<MS_ADVECT_FWD, T>(g, P, Qin, nullptr, Qhat);
    } else {
      TimedLaunch tl(g, UF_TK_ADVECT_FWD);
      launch_k(g, k_advect_fwd32<T>, grid, dim3(kFaceBlock), P, (const T*)Qin[0], (const T*)Qin[1],
               (const T*)Qin[2], (T*)Qhat[0], (T*)Qhat[1], (T*)Qhat[2]);
    }
    TimedLaunch tl(g, UF_TK_ADVECT_CORR);
    launch_k(g, k_advect_corr32<T>, xcd_grid(3 * face_gx(P.L), P.L.nx + 1), dim3(kFaceBlock), P, (const T*)Qin[0], (const T*)Qin[1],
             (const T*)Qin[2], (const T*)Qhat[0], (const T*)Qhat[1], (const T*)Qhat[2], (T*)Qout[0], (T*)Qout[1],
             (T*)Qout[2]);
    return;
  }
  {
    TimedLaunch tl(g, UF_TK_ADVECT_FWD);
    launch_k(g, k_advect_fwd<T>, grid, dim3(kFaceBlock), P, (const T*)Qin[0], (const T*)Qin[1],
                       (const T*)Qin[2], (T*)Qhat[0], (T*)Qhat[1], (T*)Qhat[2]);
  }
  TimedLaunch tl(g, UF_TK_ADVECT_CORR);
  launch_k(g, k_advect_corr<T>, grid, dim3(kFaceBlock), P, (const T*)Qin[0], (const T*)Qin[1],
                     (const T*)Qin[2], (const T*)Qhat[0], (const T*)Qhat[1], (const T*)Qhat[2], (T*)Qout[0],
                     (T*)Qout[1], (T*)Qout[2]);
}

template <class T>
void launch_diffuse(Grid& g, const Params<T>& P, void* const Qin[3], void* const Qout[3]) {
  TimedLaunch tl(g, UF_TK_DIFFUSE);
  if (planes_use(P) && P.bc[5] != OUTLET) return launch_planes<MS_DIFFUSE, T>(g, P, Qin, g.NUT, Qout);
  if (split_use(P, kSplitFaces)) return launch_split<MS_DIFFUSE, T>(g, P, Qin, g.NUT, Qout);
  launch_k(g, k_diffuse<T>, face_grid(P.L), dim3(kFaceBlock), P, (const T*)Qin[0],
                     (const T*)Qin[1], (const T*)Qin[2], (const T*)g.NUT, (T*)Qout[0], (T*)Qout[1], (T*)Qout[2]);
}

template <class T>
void launch_drag(Grid& g, const Params<T>& P, void* const Qin[3], void* const Qout[3]) {
  TimedLaunch tl(g, UF_TK_DRAG);
  if (planes_use(P) && P.bc[5] != OUTLET) return launch_planes<MS_DRAG, T>(g, P, Qin, g.C, Qout);
  if (split_use(P, kSplitFaces)) return launch_split<MS_DRAG, T>(g, P, Qin, g.C, Qout);
  launch_k(g, k_drag<T>, face_grid(P.L), dim3(kFaceBlock), P, (const T*)Qin[0], (const T*)Qin[1],
                     (const T*)Qin[2], (const T*)g.C, (T*)Qout[0], (T*)Qout[1], (T*)Qout[2], nf_word(g));
}

template <class T>
void launch_project(Grid& g, const Params<T>& P, void* const Qin[3], void* const Qout[3], const int* gate) {
  TimedLaunch tl(g, UF_TK_PROJECT);
  const Layout& L = P.L;
  if (planes_use(P)) {
    const int edge = 8 * ((march_edges(L) + 8 * kFaceBlock - 1) / (8 * kFaceBlock));
    const int gx = ((L.ny - 2) * (L.nz + 3) + kFaceBlock - 1) / kFaceBlock;
    const int nc = (L.nx - 2 + kProjPlanes - 1) / kProjPlanes;
    launch_k(g, k_project_planes<T>, dim3((unsigned)(edge + 8 * ((gx * nc + 7) / 8))), dim3(kFaceBlock), P, edge, gx,
             (const T*)Qin[0], (const T*)Qin[1], (const T*)Qin[2], (const T*)g.X, (T*)Qout[0], (T*)Qout[1],
             (T*)Qout[2], gate);
    return;
  }
  if (split_use(P, kSplitFaces)) return launch_split<MS_PROJECT, T>(g, P, Qin, g.X, Qout, gate);
  launch_k(g, k_project<T>, face_grid(P.L), dim3(kFaceBlock), P, (const T*)Qin[0],
                     (const T*)Qin[1], (const T*)Qin[2], (const T*)g.X, (T*)Qout[0], (T*)Qout[1], (T*)Qout[2], gate);
}

template <class T>
void launch_face_init(Grid& g, const Params<T>& P, void* const Q[3]) {
  const dim3 grid = face_grid(P.L);
  hipLaunchKernelGGL((k_face_init<0, T>), grid, dim3(kFaceBlock), 0, g.stream, P, (T*)Q[0]);
  hipLaunchKernelGGL((k_face_init<1, T>), grid, dim3(kFaceBlock), 0, g.stream, P, (T*)Q[1]);
  hipLaunchKernelGGL((k_face_init<2, T>), grid, dim3(kFaceBlock), 0, g.stream, P, (T*)Q[2]);
}

#define UF_INST(T)                                                                                   \
  template void launch_advect<T>(Grid&, const Params<T>&, void* const[3], void* const[3], void* const[3]); \
  template void launch_diffuse<T>(Grid&, const Params<T>&, void* const[3], void* const[3]);          \
  template void launch_drag<T>(Grid&, const Params<T>&, void* const[3], void* const[3]);             \
  template void launch_project<T>(Grid&, const Params<T>&, void* const[3], void* const[3], const int*); \
  template void launch_face_init<T>(Grid&, const Params<T>&, void* const[3]);                      \
  template void launch_faces_multi<T>(int, const MultiCase<T>*, const CaseStarts&, int, int, int, int, int, hipStream_t);
UF_INST(float)
UF_INST(double)
#undef UF_INST

}  // namespace uf
