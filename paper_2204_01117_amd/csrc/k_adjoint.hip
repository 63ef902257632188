// Reverse (discrete adjoint) of the momentum stages of one step (Sec. 3),
// for gradients of a design objective (Sec. 4) with respect to the state
// and the porosity.  Each kernel is the transpose of the forward kernel's
// Jacobian at the recomputed forward state, evaluated in the forward's own
// precision:
//
//   * projection: the step's projection is its own transpose (b = -(rho/dt)
//     div u*, A p = b, u = u* - (dt/rho) grad p with A symmetric and div =
//     -grad^T), so its reverse runs the forward solve and projection on the
//     adjoint with homogeneous boundary values (launched by the host);
//   * drag and MacCormack advection: the transpose of the trilinear samples
//     and of the drag coefficient scatters with atomic adds (their order is
//     not fixed, so the FP32 result may differ in the last bits between
//     runs); the velocity-vector part is stored per face and gathered;
//   * diffusion: the transpose is a gather over every padded position;
//   * ghosts: every ghost is written from its nearest interior face by the
//     side rules (copy, negation at a no-slip wall, a constant at an
//     inlet), so its adjoint is folded back into that face with the sign of
//     the rule; fixed boundary faces hold constants and carry no adjoint.
//
// An adjoint array holds the derivative of the objective with respect to
// the interior faces a stage computes; positions outside that set are read
// as zero (adj_in).
#include <type_traits>

#include "march.h"
#include "turb_model.h"

namespace uf {

static inline dim3 adj_face_grid(const Layout& L) { return xcd_grid(face_gx(L), L.nx + 1); }

template <class T>
__device__ __forceinline__ void add_to(T* p, T v) {
  unsafeAtomicAdd(p, v);
}

// Adjoint of face (i,j,k) of component C: zero unless it is an interior
// face whose value the stage computes (inside the face range, not fixed).
template <int C, class T>
__device__ __forceinline__ T adj_in(const Params<T>& P, const T* __restrict__ a, int i, int j, int k) {
  int ext[3];
  face_ext<C>(P.L, ext);
  if (i < 0 || j < 0 || k < 0 || i >= ext[0] || j >= ext[1] || k >= ext[2]) return T(0);
  T v;
  if (face_dirichlet<C>(P, i, j, k, &v)) return T(0);
  return a[P.L.at(i, j, k)];
}

// Reverse of face_velocity in two parts.  A reverse kernel stores, per face
// of component C, the adjoint vb[cp] of each velocity component the face
// saw (VelAdj, nine padded arrays, written at every position of the face
// thread range); k_vel_gather then adds to each face of component cp its own
// entry and a quarter of the entries of the four faces of each other
// component that averaged it.  Plain stores and a gather instead of nine
// atomic adds per face and component.
template <class T>
struct VelAdj {
  T* a[3][3];   // a[C][cp]: adjoint of velocity component cp seen at faces of component C
};

template <int C, class T>
__device__ __forceinline__ void vel_store(const VelAdj<T>& V, long long o, const T vb[3], bool accumulate) {
#pragma unroll
  for (int cp = 0; cp < 3; ++cp) {
    T* q = V.a[C][cp] + o;
    *q = accumulate ? *q + vb[cp] : vb[cp];
  }
}

// Inside the face thread range (where VelAdj entries are written)?
__device__ __forceinline__ bool in_face_range(const Layout& L, int i, int j, int k) {
  return i >= 0 && j >= 0 && k >= 0 && i <= L.nx && j <= L.ny && k <= L.nz;
}

// Value of an array at (i + di, j + dj, k + dk), zero outside the face thread
// range; base: the array's plane i; p: the position in a plane.
template <class T>
struct GatherAt {
  const Layout& L;
  int i, j, k, p;
  __device__ __forceinline__ T operator()(const T* __restrict__ a, int di, int dj, int dk) const {
    const bool ok = in_face_range(L, i + di, j + dj, k + dk);
    const int ip = i + di >= 0 && i + di <= L.nx ? i + di : i;   // uniform over the block
    const T v = (a + (long long)(ip + 1) * L.SX)[ok ? p + dj * L.PZ + dk : p];
    return ok ? v : T(0);
  }
};

template <int CP, class T>
__device__ __forceinline__ T vel_gather_value(const VelAdj<T>& V, const GatherAt<T>& at) {
  T s = at(V.a[CP][CP], 0, 0, 0);
  const int e2[3] = {CP == 0, CP == 1, CP == 2};
#pragma unroll
  for (int C = 0; C < 3; ++C) {
    if (C == CP) continue;
    const int ec[3] = {C == 0, C == 1, C == 2};
    // faces o of component C whose average of component CP reads (i,j,k):
    // o = t + e_C, t + e_C - e_CP, t, t - e_CP
    T q = at(V.a[C][CP], ec[0], ec[1], ec[2]);
    q += at(V.a[C][CP], ec[0] - e2[0], ec[1] - e2[1], ec[2] - e2[2]);
    q += at(V.a[C][CP], 0, 0, 0);
    q += at(V.a[C][CP], -e2[0], -e2[1], -e2[2]);
    s += T(0.25) * q;
  }
  return s;
}

// One thread per padded position, gx blocks per plane: G_cp += the gathered
// velocity adjoint.  All 27 loads are issued at once, at clamped positions
// (tested one by one, with 64-bit index divisions, the kernel took 138 us at
// 256x256x64 in FP32; 59).
template <class T>
__global__ __launch_bounds__(256) void k_vel_gather(Params<T> P, int gx, VelAdj<T> V, T* __restrict__ G0,
                                                    T* __restrict__ G1, T* __restrict__ G2) {
  const Layout& L = P.L;
  const int pl = (int)blockIdx.x / gx, p = ((int)blockIdx.x - pl * gx) * 256 + (int)threadIdx.x;
  if (p >= (int)L.SX) return;
  const int jp = p / L.PZ;
  const GatherAt<T> at{L, pl - 1, jp - 1, p - jp * L.PZ - 1, p};
  const long long o = (long long)pl * L.SX + p;
  const T g0 = G0[o], g1 = G1[o], g2 = G2[o];
  const T s0 = vel_gather_value<0>(V, at), s1 = vel_gather_value<1>(V, at), s2 = vel_gather_value<2>(V, at);
  G0[o] = g0 + s0;
  G1[o] = g1 + s1;
  G2[o] = g2 + s2;
}

// Cell and fractions of a trace position (i + si, j + sj, k + sk), clamped
// exactly as in sample().
template <int C, class T>
struct SamplePos {
  long long o;      // offset of the lower corner
  T t[3];           // fractions
  bool live[3];     // the position was not clamped along this axis
  __device__ __forceinline__ SamplePos(const Layout& L, int i, int j, int k, T si, T sj, T sk) {
    AxisPos<T> a[3];
    trace_pos<C>(L, i, j, k, si, sj, sk, a);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      t[q] = a[q].t;
      live[q] = a[q].live;
    }
    o = L.at(a[0].c, a[1].c, a[2].c);
  }
};

// Offset of the smallest (want_max false) or largest of the eight samples
// around a position (the first one in corner order on a tie).
template <int C, class T>
__device__ __forceinline__ long long sample_extreme(const Layout& L, const T* __restrict__ q, int i, int j, int k,
                                                    T si, T sj, T sk, bool want_max) {
  const SamplePos<C, T> s(L, i, j, k, si, sj, sk);
  const long long offs[8] = {0, L.SX, L.PZ, L.SX + L.PZ, 1, L.SX + 1, L.PZ + 1, L.SX + L.PZ + 1};
  long long best = s.o;
  T bv = q[s.o];
#pragma unroll
  for (int n = 1; n < 8; ++n) {
    const T v = q[s.o + offs[n]];
    if (want_max ? v > bv : v < bv) {
      bv = v;
      best = s.o + offs[n];
    }
  }
  return best;
}

// ------------------------------------------------------------- advection --
// A trilinear scatter of one lane, made by all lanes of the wavefront
// together.  Lanes are consecutive along z, so lane L's upper layer of
// samples (z index k0 + 1) is usually lane L+1's lower layer: when their
// corners are one apart, L+1 adds L's four upper weights to its own lower
// ones (one shuffle each) and L skips those atomics -- four atomic adds per
// sample instead of eight.  Both lanes decide from the same two corners.
template <class T>
struct Scatter8 {
  long long o;   // lower corner
  T w[8];        // weights times the adjoint, corner order 000 100 010 110 001 101 011 111
  bool on;
};

template <int C, class T>
__device__ __forceinline__ void sample_weights(const Layout& L, const T* __restrict__ q, int i, int j, int k, T si,
                                               T sj, T sk, T wbar, T grad[3], Scatter8<T>& sc) {
  const SamplePos<C, T> s(L, i, j, k, si, sj, sk);
  const long long o = s.o, SX = L.SX, PZ = L.PZ;
  const T ti = s.t[0], tj = s.t[1], tk = s.t[2];
  const T s000 = q[o], s100 = q[o + SX], s010 = q[o + PZ], s110 = q[o + SX + PZ];
  const T s001 = q[o + 1], s101 = q[o + SX + 1], s011 = q[o + PZ + 1], s111 = q[o + SX + PZ + 1];
  const T ui = T(1) - ti, uj = T(1) - tj, uk = T(1) - tk;
  grad[0] = s.live[0] ? uj * uk * (s100 - s000) + tj * uk * (s110 - s010) + uj * tk * (s101 - s001) +
                            tj * tk * (s111 - s011)
                      : T(0);
  grad[1] = s.live[1] ? ui * uk * (s010 - s000) + ti * uk * (s110 - s100) + ui * tk * (s011 - s001) +
                            ti * tk * (s111 - s101)
                      : T(0);
  grad[2] = s.live[2] ? ui * uj * (s001 - s000) + ti * uj * (s101 - s100) + ui * tj * (s011 - s010) +
                            ti * tj * (s111 - s110)
                      : T(0);
  sc.o = o;
  sc.on = wbar != T(0);
  sc.w[0] = wbar * ui * uj * uk;
  sc.w[1] = wbar * ti * uj * uk;
  sc.w[2] = wbar * ui * tj * uk;
  sc.w[3] = wbar * ti * tj * uk;
  sc.w[4] = wbar * ui * uj * tk;
  sc.w[5] = wbar * ti * uj * tk;
  sc.w[6] = wbar * ui * tj * tk;
  sc.w[7] = wbar * ti * tj * tk;
}

// Called by every lane of the wavefront (convergent).
template <class T>
__device__ __forceinline__ void paired_scatter(T* __restrict__ qbar, const Layout& L, const Scatter8<T>& sc) {
  const int lane = (int)(threadIdx.x & 63u);
  const long long mine = sc.on ? sc.o : -2LL;   // corners are >= 0: -2 never matches
  const long long prev = __shfl_up(mine, 1u);
  const long long next = __shfl_down(mine, 1u);
  T r[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) r[q] = __shfl_up(sc.w[4 + q], 1u);
  if (!sc.on) return;
  const bool take = lane > 0 && prev >= 0 && prev + 1 == sc.o;
  const bool give = lane < 63 && next == sc.o + 1;
  const long long SX = L.SX, PZ = L.PZ;
  const long long lo[4] = {0, SX, PZ, SX + PZ};
#pragma unroll
  for (int q = 0; q < 4; ++q) add_to(qbar + sc.o + lo[q], take ? sc.w[q] + r[q] : sc.w[q]);
  if (!give) {
#pragma unroll
    for (int q = 0; q < 4; ++q) add_to(qbar + sc.o + lo[q] + 1, sc.w[4 + q]);
  }
}

// Reverse of the corrector: out = clamp(qh + (q - qc)/2, min, max) with
// qh sampled from q at the back-traced point and qc from qhat at the
// forward-traced point.  A clamped output is one of the eight samples of q.
// The two trilinear scatters are returned (sb into q's adjoint, sf into
// qhat's); the face's own half goes into vb[C] (gathered back to it).
template <int C, class T>
__device__ __forceinline__ void advect_corr_adj(const Params<T>& P, const T* __restrict__ U, const T* __restrict__ V,
                                                const T* __restrict__ W, const T* __restrict__ qhat, T ob,
                                                T* __restrict__ Gq, long long o, int i, int j, int k, T vb[3],
                                                Scatter8<T>& sb, Scatter8<T>& sf) {
  vb[0] = vb[1] = vb[2] = T(0);
  sb = Scatter8<T>();
  sf = Scatter8<T>();
  if (ob == T(0)) return;
  T vel[3];
  face_velocity<C>(P.L, U, V, W, o, vel);
  const T* q = C == 0 ? U : (C == 1 ? V : W);
  const T di = vel[0] * P.dth[0], dj = vel[1] * P.dth[1], dk = vel[2] * P.dth[2];
  T mn, mx, d0, d1;
  const T qh = sample<C, true>(P.L, q, i, j, k, -di, -dj, -dk, &mn, &mx);
  const T qc = sample<C, false>(P.L, qhat, i, j, k, di, dj, dk, &d0, &d1);
  const T qt = qh + T(0.5) * (q[o] - qc);
  if (qt < mn || qt > mx) {
    add_to(Gq + sample_extreme<C>(P.L, q, i, j, k, -di, -dj, -dk, qt > mx), ob);
    return;
  }
  T gb[3], gf[3];
  sample_weights<C>(P.L, q, i, j, k, -di, -dj, -dk, ob, gb, sb);
  sample_weights<C>(P.L, qhat, i, j, k, di, dj, dk, T(-0.5) * ob, gf, sf);
  vb[0] = -ob * P.dth[0] * (gb[0] + T(0.5) * gf[0]);
  vb[1] = -ob * P.dth[1] * (gb[1] + T(0.5) * gf[1]);
  vb[2] = -ob * P.dth[2] * (gb[2] + T(0.5) * gf[2]);
  vb[C] += T(0.5) * ob;
}

// Reverse of the predictor: qhat = q sampled at the back-traced point.
template <int C, class T>
__device__ __forceinline__ void advect_fwd_adj(const Params<T>& P, const T* __restrict__ U, const T* __restrict__ V,
                                               const T* __restrict__ W, T ob, long long o, int i, int j, int k,
                                               T vb[3], Scatter8<T>& sb) {
  vb[0] = vb[1] = vb[2] = T(0);
  sb = Scatter8<T>();
  if (ob == T(0)) return;
  T vel[3];
  face_velocity<C>(P.L, U, V, W, o, vel);
  const T* q = C == 0 ? U : (C == 1 ? V : W);
  T g[3];
  sample_weights<C>(P.L, q, i, j, k, -(vel[0] * P.dth[0]), -(vel[1] * P.dth[1]), -(vel[2] * P.dth[2]), ob, g, sb);
  vb[0] = -ob * P.dth[0] * g[0];
  vb[1] = -ob * P.dth[1] * g[1];
  vb[2] = -ob * P.dth[2] * g[2];
}

// The face-thread mapping without the early exit of lanes past the last
// corner (the paired scatter needs every lane of the wavefront): such lanes
// carry no adjoint and write nothing.
#define UF_FACE_THREAD_ALL(L)                                        \
  int f_bx, f_by;                                                    \
  if (!face_block((L), f_bx, f_by)) return;                          \
  const int i = f_by;                                                \
  const int p_raw = f_bx * kFaceBlock + threadIdx.x;                 \
  const bool lane_valid = p_raw < ((L).ny + 1) * ((L).nz + 1);       \
  const int p = lane_valid ? p_raw : 0;                              \
  const int j = p / ((L).nz + 1);                                    \
  const int k = p - j * ((L).nz + 1);

template <class T>
__global__ __launch_bounds__(kFaceBlock) void k_advect_corr_adj(Params<T> P, const T* __restrict__ U,
                                                                const T* __restrict__ V, const T* __restrict__ W,
                                                                const T* __restrict__ Uh, const T* __restrict__ Vh,
                                                                const T* __restrict__ Wh, const T* __restrict__ A0,
                                                                const T* __restrict__ A1, const T* __restrict__ A2,
                                                                T* __restrict__ GU, T* __restrict__ GV,
                                                                T* __restrict__ GW, T* __restrict__ HU,
                                                                T* __restrict__ HV, T* __restrict__ HW,
                                                                VelAdj<T> VA) {
  UF_FACE_THREAD_ALL(P.L);
  const long long o = P.L.at(i, j, k);
  T vb[3];
  Scatter8<T> sb, sf;
  advect_corr_adj<0>(P, U, V, W, Uh, lane_valid ? adj_in<0>(P, A0, i, j, k) : T(0), GU, o, i, j, k, vb, sb, sf);
  if (lane_valid) vel_store<0>(VA, o, vb, false);
  paired_scatter(GU, P.L, sb);
  paired_scatter(HU, P.L, sf);
  advect_corr_adj<1>(P, U, V, W, Vh, lane_valid ? adj_in<1>(P, A1, i, j, k) : T(0), GV, o, i, j, k, vb, sb, sf);
  if (lane_valid) vel_store<1>(VA, o, vb, false);
  paired_scatter(GV, P.L, sb);
  paired_scatter(HV, P.L, sf);
  advect_corr_adj<2>(P, U, V, W, Wh, lane_valid ? adj_in<2>(P, A2, i, j, k) : T(0), GW, o, i, j, k, vb, sb, sf);
  if (lane_valid) vel_store<2>(VA, o, vb, false);
  paired_scatter(GW, P.L, sb);
  paired_scatter(HW, P.L, sf);
}

template <class T>
__global__ __launch_bounds__(kFaceBlock) void k_advect_fwd_adj(Params<T> P, const T* __restrict__ U,
                                                               const T* __restrict__ V, const T* __restrict__ W,
                                                               const T* __restrict__ H0, const T* __restrict__ H1,
                                                               const T* __restrict__ H2, T* __restrict__ GU,
                                                               T* __restrict__ GV, T* __restrict__ GW,
                                                               VelAdj<T> VA) {
  UF_FACE_THREAD_ALL(P.L);
  const long long o = P.L.at(i, j, k);
  T vb[3];
  Scatter8<T> sb;
  advect_fwd_adj<0>(P, U, V, W, lane_valid ? adj_in<0>(P, H0, i, j, k) : T(0), o, i, j, k, vb, sb);
  if (lane_valid) vel_store<0>(VA, o, vb, true);
  paired_scatter(GU, P.L, sb);
  advect_fwd_adj<1>(P, U, V, W, lane_valid ? adj_in<1>(P, H1, i, j, k) : T(0), o, i, j, k, vb, sb);
  if (lane_valid) vel_store<1>(VA, o, vb, true);
  paired_scatter(GV, P.L, sb);
  advect_fwd_adj<2>(P, U, V, W, lane_valid ? adj_in<2>(P, H2, i, j, k) : T(0), o, i, j, k, vb, sb);
  if (lane_valid) vel_store<2>(VA, o, vb, true);
  paired_scatter(GW, P.L, sb);
}

// ------------------------------------------- advection, marching along x --
// A trace shorter than a cell scatters a face's adjoint over the 3 x 3 x 3
// positions around the face with the hat function's weights, max(0, 1 - |m -
// s|) per axis.  A thread marches along x and keeps the sums of its column in
// registers, nine neighbours along y and z in each plane; the plane that is
// complete goes to LDS, every position of the tile with its
// halo adds the up to nine sums that concern it, and one atomic add per
// position takes them to memory.  The scatter with eight atomic adds per
// sample (four, where neighbouring lanes share) took 1228 us for the
// corrector and 623 for the predictor at 256x256x64 in FP32, as LDS atomics
// 1167 and 625 (about 160 cycles for a wavefront's ds_add_f32), these sums
// 395 and 277 (registers and the nine writes and reads per sample bound them).
template <int SHAPE, int NB, class T>
struct Collect {
  using S = MarchShape<SHAPE>;
  static constexpr int ROWS = S::TJ + 4, PITCH = S::TKM + 4, PL = ROWS * PITCH, LDS = 9 * PL;
  T* lds;            // [3 y][3 z][PL]: the complete plane's sums by column, zero beyond the tile
  T sum[NB][2][9];   // of the column, before plane i is added: planes i - 1 and i
  int own;           // the thread's column; -1: none
  __device__ __forceinline__ void init(T* mem, bool on, int jj, int kk) {
    lds = mem;
    own = on ? (jj + 2) * PITCH + kk + 2 : -1;
    for (int e = threadIdx.x; e < LDS; e += kMarch) lds[e] = T(0);
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int q = 0; q < 9; ++q) sum[b][m][q] = T(0);
  }
  // Adds wbar at the position displaced by (si, sj, sk) from the face of plane
  // i to array b; plane i - 1 is then complete and goes to LDS.
  __device__ __forceinline__ void add(int b, T si, T sj, T sk, T wbar) {
    const T wx[3] = {fmax(-si, T(0)), T(1) - fabs(si), fmax(si, T(0))};
    const T wy[3] = {fmax(-sj, T(0)), T(1) - fabs(sj), fmax(sj, T(0))};
    const T wz[3] = {fmax(-sk, T(0)), T(1) - fabs(sk), fmax(sk, T(0))};
#pragma unroll
    for (int y = 0; y < 3; ++y) {
#pragma unroll
      for (int z = 0; z < 3; ++z) {
        const T w = wbar * wy[y] * wz[z];
        T* u = sum[b][0] + 3 * y + z;
        T* v = sum[b][1] + 3 * y + z;
        if (own >= 0) lds[(3 * y + z) * PL + own] = *u + w * wx[0];
        *u = *v + w * wx[1];
        *v = w * wx[2];
      }
    }
  }
  // The plane in LDS added to the padded plane out.
  template <class A>
  __device__ __forceinline__ void flush(const A& planes, T* __restrict__ out) const {
#pragma unroll
    for (int v = 0; v < A::NV; ++v) {
      if (planes.le[v] < 0) continue;
      const int r = planes.le[v] / A::PITCH, c = planes.le[v] - r * A::PITCH;
      const T* p = lds + r * PITCH + c;   // source (y, z) of sum (y', z') is at row r + 2 - y', column c + 2 - z'
      T x = T(0);
#pragma unroll
      for (int y = 0; y < 3; ++y)
#pragma unroll
        for (int z = 0; z < 3; ++z) x += p[(3 * y + z) * PL + (2 - y) * PITCH + 2 - z];
      if (x != T(0)) add_to(out + planes.off[v], x);
    }
  }
};

// The gradient of a near sample along the axes.
template <class T>
__device__ __forceinline__ void tri_grad(const Tri<T>& t, const T v[8], T grad[3]) {
  const T ti = t.ti, tj = t.tj, tk = t.tk, ui = T(1) - ti, uj = T(1) - tj, uk = T(1) - tk;
  grad[0] = uj * uk * (v[1] - v[0]) + tj * uk * (v[3] - v[2]) + uj * tk * (v[5] - v[4]) + tj * tk * (v[7] - v[6]);
  grad[1] = ui * uk * (v[2] - v[0]) + ti * uk * (v[3] - v[1]) + ui * tk * (v[6] - v[4]) + ti * tk * (v[7] - v[5]);
  grad[2] = ui * uj * (v[4] - v[0]) + ti * uj * (v[5] - v[1]) + ui * tj * (v[6] - v[2]) + ti * tj * (v[7] - v[3]);
}

template <class T>
struct AdvectAdj {
  const T* q[3];      // the state
  const T* qhat[3];   // the predictor's field (corrector)
  const T* a[3];      // adjoint of the stage's output
  T* g[3];            // adjoint of the state
  T* h[3];            // adjoint of qhat (corrector)
  VelAdj<T> va;
};

// A scatter of one lane by itself (a trace that leaves the neighbouring
// cells).
template <class T>
__device__ __forceinline__ void lone_scatter(T* __restrict__ qbar, const Layout& L, const Scatter8<T>& sc) {
  if (!sc.on) return;
  const long long SX = L.SX, PZ = L.PZ;
  const long long lo[4] = {0, SX, PZ, SX + PZ};
#pragma unroll
  for (int q = 0; q < 8; ++q) add_to(qbar + sc.o + lo[q & 3] + (q >> 2), sc.w[q]);
}

// The reverse of the corrector (CORR) or the predictor of component C at the
// faces of a tile.
template <bool CORR, int C, int SHAPE, class T>
__device__ __forceinline__ void march_advect_adj(const Params<T>& P, const March& G, const AdvectAdj<T>& M, T* lds,
                                                 T* acc, int tile, int chunk) {
  constexpr int NA = CORR ? 4 : 3, NB = CORR ? 2 : 1;
  const Layout& L = P.L;
  Planes<SHAPE, NA, T> A;
#pragma unroll
  for (int a = 0; a < 3; ++a) A.src[a] = M.q[a];
  if constexpr (CORR) A.src[3] = M.qhat[C];
  Collect<SHAPE, NB, T> K;
  T* out[NB];
  out[0] = M.g[C];
  if constexpr (CORR) out[1] = M.h[C];
  int j0, k0;
  MarchLane c = march_lane<SHAPE>(L, G, tile, L.ny - 2, L.nz + 3, L.nz + 1, L.nz + 1, j0, k0);
  const bool on = c.active && c.k >= 0 && c.k <= L.nz;
  A.init(L, lds, j0, k0, G.TK);
  A.q = c.qa;
  K.init(acc, on, c.j - j0, c.k - k0);
  const int i0 = 1 + chunk * G.len, i1 = min(L.nx - 1, i0 + G.len);
  A.load(i0 - 1);
  A.store(A.s[0]);
  A.load(i0);
  A.store(A.s[1]);
  A.load(i0 + 1);
  // plane i is computed while i < i1, plane i - 1 is complete then
  for (int i = i0; i <= i1 + 1; ++i) {
    if (i < i1) A.store(A.s[2]);
    lds_barrier();
    if (i + 1 < i1) A.load(i + 2);
    // what depends on the lane alone stays in the loop: hoisted, it spills
    asm volatile("" : "+v"(c.j), "+v"(c.k));
    T sc[4] = {T(0), T(0), T(0), T(0)};   // displacement and adjoint of the face's scatters
    if (on && i < i1) {
      const long long o = L.at(i, c.j, c.k);
      const T ob = adj_in<C>(P, M.a[C], i, c.j, c.k);
      T vb[3] = {T(0), T(0), T(0)};
      if (ob != T(0)) {
        T vel[3];
        march_velocity<C>(A, vel);
        const T d[3] = {vel[0] * P.dth[0], vel[1] * P.dth[1], vel[2] * P.dth[2]};
        if (fabs(d[0]) < T(1) && fabs(d[1]) < T(1) && fabs(d[2]) < T(1)) {
          Tri<T> tf;
          T vf[8], gb[3];
          march_samples(A, C, -d[0], -d[1], -d[2], tf, vf);
          tri_grad(tf, vf, gb);
          if constexpr (CORR) {
            Tri<T> tb;
            T vt[8], gf[3], mn, mx;
            march_samples(A, 3, d[0], d[1], d[2], tb, vt);
            tri_range(vf, mn, mx);
            const T qt = tri_eval(tf, vf) + T(0.5) * (vel[C] - tri_eval(tb, vt));
            if (qt < mn || qt > mx) {   // clamped: one of the eight samples
              add_to(M.g[C] + sample_extreme<C>(L, M.q[C], i, c.j, c.k, -d[0], -d[1], -d[2], qt > mx), ob);
            } else {
              tri_grad(tb, vt, gf);
              sc[3] = ob;
#pragma unroll
              for (int q = 0; q < 3; ++q) vb[q] = -ob * P.dth[q] * (gb[q] + T(0.5) * gf[q]);
              vb[C] += T(0.5) * ob;
            }
          } else {
            sc[3] = ob;
#pragma unroll
            for (int q = 0; q < 3; ++q) vb[q] = -ob * P.dth[q] * gb[q];
          }
#pragma unroll
          for (int q = 0; q < 3; ++q) sc[q] = d[q];
        } else {
          Scatter8<T> sb, sf;
          if constexpr (CORR) {
            advect_corr_adj<C>(P, M.q[0], M.q[1], M.q[2], M.qhat[C], ob, M.g[C], o, i, c.j, c.k, vb, sb, sf);
            lone_scatter(M.h[C], L, sf);
          } else {
            advect_fwd_adj<C>(P, M.q[0], M.q[1], M.q[2], ob, o, i, c.j, c.k, vb, sb);
          }
          lone_scatter(M.g[C], L, sb);
        }
      }
      vel_store<C>(M.va, o, vb, !CORR);
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      if (b == 0) {
        K.add(0, -sc[0], -sc[1], -sc[2], sc[3]);
      } else {
        lds_barrier();
        K.add(b, sc[0], sc[1], sc[2], T(-0.5) * sc[3]);
      }
      lds_barrier();
      K.flush(A, out[b] + (long long)i * L.SX);   // padded plane of i - 1
    }
    A.rotate();
  }
}

template <bool CORR, int SHAPE, class T>
__global__ __launch_bounds__(kMarch, 4) void k_advect_adj_march(Params<T> P, March G, AdvectAdj<T> M) {
  __shared__ T lds[Planes<SHAPE, CORR ? 4 : 3, T>::LDS];
  __shared__ T acc[Collect<SHAPE, CORR ? 2 : 1, T>::LDS];
  const Layout& L = P.L;
  int tile, chunk;
  if (!march_block(G, tile, chunk)) return;
  if (tile >= 0) {
    const int C = chunk % 3;
    if (C == 0) march_advect_adj<CORR, 0, SHAPE>(P, G, M, lds, acc, tile, chunk / 3);
    else if (C == 1) march_advect_adj<CORR, 1, SHAPE>(P, G, M, lds, acc, tile, chunk / 3);
    else march_advect_adj<CORR, 2, SHAPE>(P, G, M, lds, acc, tile, chunk / 3);
    return;
  }
  int i = 0, j = 0, k = 0;
  const bool valid = march_edge_corner(L, chunk * kMarch + (int)threadIdx.x, i, j, k);
  const long long o = L.at(i, j, k);
  auto face = [&](auto tag) {
    constexpr int C = decltype(tag)::value;
    const T ob = valid ? adj_in<C>(P, M.a[C], i, j, k) : T(0);
    T vb[3];
    Scatter8<T> sb, sf;
    if constexpr (CORR) advect_corr_adj<C>(P, M.q[0], M.q[1], M.q[2], M.qhat[C], ob, M.g[C], o, i, j, k, vb, sb, sf);
    else advect_fwd_adj<C>(P, M.q[0], M.q[1], M.q[2], ob, o, i, j, k, vb, sb);
    if (valid) vel_store<C>(M.va, o, vb, !CORR);
    paired_scatter(M.g[C], L, sb);
    if constexpr (CORR) paired_scatter(M.h[C], L, sf);
  };
  face(std::integral_constant<int, 0>());
  face(std::integral_constant<int, 1>());
  face(std::integral_constant<int, 2>());
}

// ------------------------------------------------------------- diffusion --
// Transpose of out = q + dt nu_f lap(q) at one padded position (interior
// or ghost) of component C: the position's own row plus the rows of its
// six neighbours.  Loads at clamped positions, so that all are in flight.
template <int C, class T>
__device__ __forceinline__ T diffuse_adj_value(const Params<T>& P, const T* __restrict__ a, const T* __restrict__ nut,
                                               int i, int j, int k, long long o) {
  const Layout& L = P.L;
  // adjoint of the face displaced by (di, dj, dk) (adj_in) and its viscosity
  auto tap = [&](int di, int dj, int dk, T& nu) -> T {
    int ext[3];
    face_ext<C>(L, ext);
    const int f[3] = {i + di, j + dj, k + dk};
    bool ok = f[0] >= 0 && f[1] >= 0 && f[2] >= 0 && f[0] < ext[0] && f[1] < ext[1] && f[2] < ext[2];
    if ((f[C] == 0 && P.bc[2 * C] != OUTLET) || (f[C] == ext[C] - 1 && P.bc[2 * C + 1] != OUTLET)) ok = false;   // fixed
    const long long q = ok ? o + (long long)di * L.SX + (long long)dj * L.PZ + dk : L.at(0, 0, 0);
    const T v = a[q];
    nu = P.nu + T(0.5) * (nut[q - stride<C>(L)] + nut[q]);
    return ok ? v : T(0);
  };
  T nu;
  const T self = tap(0, 0, 0, nu);
  T s = self != T(0) ? self * (T(1) - T(2) * P.dt * nu * (P.ih2[0] + P.ih2[1] + P.ih2[2])) : T(0);
  const int d[3][3] = {{1, 0, 0}, {0, 1, 0}, {0, 0, 1}};
#pragma unroll
  for (int ax = 0; ax < 3; ++ax) {
#pragma unroll
    for (int sg = -1; sg <= 1; sg += 2) {
      const T an = tap(sg * d[ax][0], sg * d[ax][1], sg * d[ax][2], nu);
      s += an != T(0) ? an * P.dt * nu * P.ih2[ax] : T(0);
    }
  }
  return s;
}

// One thread per padded position, gx blocks per plane; every position of the
// three outputs is written (zero outside [-1, extent] of the component).
// Tested tap by tap, with 64-bit index divisions, it took 154 us at
// 256x256x64 in FP32; 131 here (63 loads a position bound it).
template <class T>
__global__ __launch_bounds__(256) void k_diffuse_adj(Params<T> P, int gx, const T* __restrict__ A0,
                                                     const T* __restrict__ A1, const T* __restrict__ A2,
                                                     const T* __restrict__ NUT, T* __restrict__ G0,
                                                     T* __restrict__ G1, T* __restrict__ G2) {
  const Layout& L = P.L;
  const int pl = (int)blockIdx.x / gx, p = ((int)blockIdx.x - pl * gx) * 256 + (int)threadIdx.x;
  if (p >= (int)L.SX) return;
  const int jp = p / L.PZ, i = pl - 1, j = jp - 1, k = p - jp * L.PZ - 1;
  const long long o = (long long)pl * L.SX + p;
  const bool in_x = i <= L.nx, in_y = j <= L.ny, in_z = k <= L.nz;   // lower bound -1 always holds
  // component C reaches index extent along its own axis (extent + 1 = n + 1 for the normal axis)
  const T g0 = diffuse_adj_value<0>(P, A0, NUT, i, j, k, o);
  const T g1 = diffuse_adj_value<1>(P, A1, NUT, i, j, k, o);
  const T g2 = diffuse_adj_value<2>(P, A2, NUT, i, j, k, o);
  G0[o] = in_y && in_z ? g0 : T(0);
  G1[o] = in_x && in_z ? g1 : T(0);
  G2[o] = in_x && in_y ? g2 : T(0);
}

// ------------------------------------------------------------ porosity drag
// Reverse of out = max(0, 1 - dt c_f |V|) V_C: the velocity part through
// face_velocity and the drag-coefficient part, half to each adjacent cell.
template <int C, class T>
__device__ __forceinline__ void drag_adj(const Params<T>& P, const T* __restrict__ U, const T* __restrict__ V,
                                         const T* __restrict__ W, const T* __restrict__ Cc, T ob,
                                         T* __restrict__ Cbar, long long o, T vb[3]) {
  vb[0] = vb[1] = vb[2] = T(0);
  if (ob == T(0)) return;
  T vel[3];
  face_velocity<C>(P.L, U, V, W, o, vel);
  const T speed = sqrt(vel[0] * vel[0] + vel[1] * vel[1] + vel[2] * vel[2]);
  const T cf = T(0.5) * (Cc[o - stride<C>(P.L)] + Cc[o]);
  const T fac = T(1) - P.dt * cf * speed;
  if (!(fac > T(0))) return;   // the face is stopped: no dependence on either input
  const T g = speed > T(0) ? P.dt * cf * vel[C] / speed : T(0);
  vb[0] = -ob * g * vel[0];
  vb[1] = -ob * g * vel[1];
  vb[2] = -ob * g * vel[2];
  vb[C] += ob * fac;
  const T cb = T(-0.5) * ob * P.dt * speed * vel[C];
  if (cb != T(0)) {
    add_to(Cbar + o - stride<C>(P.L), cb);
    add_to(Cbar + o, cb);
  }
}

template <class T>
__global__ __launch_bounds__(kFaceBlock) void k_drag_adj(Params<T> P, const T* __restrict__ U, const T* __restrict__ V,
                                                         const T* __restrict__ W, const T* __restrict__ Cc,
                                                         const T* __restrict__ A0, const T* __restrict__ A1,
                                                         const T* __restrict__ A2, T* __restrict__ Cbar,
                                                         VelAdj<T> VA) {
  UF_FACE_THREAD(P.L);
  const long long o = P.L.at(i, j, k);
  T vb[3];
  drag_adj<0>(P, U, V, W, Cc, adj_in<0>(P, A0, i, j, k), Cbar, o, vb);
  vel_store<0>(VA, o, vb, false);
  drag_adj<1>(P, U, V, W, Cc, adj_in<1>(P, A1, i, j, k), Cbar, o, vb);
  vel_store<1>(VA, o, vb, false);
  drag_adj<2>(P, U, V, W, Cc, adj_in<2>(P, A2, i, j, k), Cbar, o, vb);
  vel_store<2>(VA, o, vb, false);
}

// ---------------------------------------------------------------- ghosts --
// Sign with which the ghost across side (a, hi) of component c follows its
// neighbour (see face_rule): +1 for a copy, -1 at a no-slip wall, 0 where it
// is the inflow constant.
template <class T>
__device__ __forceinline__ T rule_sign(const Params<T>& P, int c, int a, int hi) {
  if (a == c) return T(1);
  const int kind = P.bc[2 * a + hi];
  if (kind == INLET) return T(0);
  if (kind == WALL) return T(-1);
  return T(1);
}

// Reverse of store_face for face (i,j,k) of component C: the adjoint held
// at each ghost written from this face is added to it with the rule's sign
// and the ghost cleared; a fixed face ends with zero.
template <int C, class T>
__device__ __forceinline__ void fold_face(T* __restrict__ q, const Params<T>& P, int i, int j, int k) {
  const Layout& L = P.L;
  const long long o = L.at(i, j, k);
  int ext[3];
  face_ext<C>(L, ext);
  const bool lo0 = i == 0, hi0 = i == ext[0] - 1;
  const bool lo1 = j == 0, hi1 = j == ext[1] - 1;
  const bool lo2 = k == 0, hi2 = k == ext[2] - 1;
  // an interior face has no ghost and is never fixed: nothing to do
  if (!(lo0 || hi0 || lo1 || hi1 || lo2 || hi2)) return;
  T acc = q[o];
  auto take = [&](long long gpos, T s) {
    acc += s * q[gpos];
    q[gpos] = T(0);
  };
  if (lo2) take(o - 1, rule_sign(P, C, 2, 0));
  if (hi2) take(o + 1, rule_sign(P, C, 2, 1));
  if (lo1) take(o - L.PZ, rule_sign(P, C, 1, 0));
  if (hi1) take(o + L.PZ, rule_sign(P, C, 1, 1));
  if (lo0) take(o - L.SX, rule_sign(P, C, 0, 0));
  if (hi0) take(o + L.SX, rule_sign(P, C, 0, 1));
  if (int(lo0 | hi0) + int(lo1 | hi1) + int(lo2 | hi2) >= 2) {
    for (int ox = -1; ox <= 1; ++ox) {
      if ((ox == -1 && !lo0) || (ox == 1 && !hi0)) continue;
      for (int oy = -1; oy <= 1; ++oy) {
        if ((oy == -1 && !lo1) || (oy == 1 && !hi1)) continue;
        for (int oz = -1; oz <= 1; ++oz) {
          if ((oz == -1 && !lo2) || (oz == 1 && !hi2)) continue;
          if (int(ox != 0) + int(oy != 0) + int(oz != 0) < 2) continue;
          T s = T(1);
          if (ox) s *= rule_sign(P, C, 0, ox > 0);
          if (oy) s *= rule_sign(P, C, 1, oy > 0);
          if (oz) s *= rule_sign(P, C, 2, oz > 0);
          take(L.at(i + ox, j + oy, k + oz), s);
        }
      }
    }
  }
  T fixed;
  if (face_dirichlet<C>(P, i, j, k, &fixed)) acc = T(0);
  q[o] = acc;
}

// The corners whose faces lie on or next to a side: an axis of n cells has
// edge_count(n) such indices 0, n - 1, n (0 and 1 for one cell), edge_index
// the s-th, the others from 1 on.
__host__ __device__ __forceinline__ int edge_count(int n) { return n < 2 ? 2 : 3; }
__device__ __forceinline__ int edge_index(int n, int s) { return s == 0 ? 0 : n + 1 - edge_count(n) + s; }

// Corners with an edge index along x (k fastest), then those left with one
// along y, then those left with one along z.
static long long fold_corners(const Layout& L) {
  const long long ex = edge_count(L.nx), ey = edge_count(L.ny), ez = edge_count(L.nz);
  const long long ix = L.nx + 1 - ex, iy = L.ny + 1 - ey;
  return ex * (L.ny + 1) * (L.nz + 1) + ix * ey * (L.nz + 1) + ix * iy * ez;
}

// Only those corners have anything to fold (a thread for every corner took 41
// us at 256x256x64, six times per reverse step; 16).
template <class T>
__global__ __launch_bounds__(kFaceBlock) void k_fold(Params<T> P, T* __restrict__ Q0, T* __restrict__ Q1,
                                                     T* __restrict__ Q2, int n) {
  const Layout& L = P.L;
  int e = (int)blockIdx.x * kFaceBlock + (int)threadIdx.x;
  if (e >= n) return;
  const int ex = edge_count(L.nx), ey = edge_count(L.ny), ez = edge_count(L.nz);
  const int ix = L.nx + 1 - ex, iy = L.ny + 1 - ey, nk = L.nz + 1;
  const int na = ex * (L.ny + 1) * nk, nb = ix * ey * nk;
  int i, j, k;
  if (e < na) {
    const int r = e / nk, s = r / (L.ny + 1);
    k = e - r * nk;
    i = edge_index(L.nx, s);
    j = r - s * (L.ny + 1);
  } else if (e < na + nb) {
    e -= na;
    const int r = e / nk, s = r / ix;
    k = e - r * nk;
    i = 1 + r - s * ix;
    j = edge_index(L.ny, s);
  } else {
    e -= na + nb;
    const int r = e / ez;
    k = edge_index(L.nz, e - r * ez);
    i = 1 + r / iy;
    j = 1 + r % iy;
  }
  if (owns_face<0, T>(L, i, j, k)) fold_face<0>(Q0, P, i, j, k);
  if (owns_face<1, T>(L, i, j, k)) fold_face<1>(Q1, P, i, j, k);
  if (owns_face<2, T>(L, i, j, k)) fold_face<2>(Q2, P, i, j, k);
}

// Drag-coefficient adjoint of each cell (its face-adjacent ghosts copy it)
// chained to the porosity: c = coef ((1 - phi)/(phi + e))^b, evaluated in
// FP64 (dc/dphi is very large in nearly solid cells), added to phibar.
template <class T>
__global__ __launch_bounds__(256) void k_drag_coef_adj(Params<T> P, const T* __restrict__ Cbar,
                                                       const T* __restrict__ PHI, double* __restrict__ phibar,
                                                       double coef, double e, double b) {
  const Layout& L = P.L;
  const long long n = (long long)L.nx * L.ny * L.nz;
  for (long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x; c < n; c += (long long)gridDim.x * blockDim.x) {
    const int k = (int)(c % L.nz);
    const long long r = c / L.nz;
    const int j = (int)(r % L.ny);
    const int i = (int)(r / L.ny);
    const long long o = L.at(i, j, k);
    double cb = (double)Cbar[o];
    if (i == 0) cb += (double)Cbar[o - L.SX];
    if (i == L.nx - 1) cb += (double)Cbar[o + L.SX];
    if (j == 0) cb += (double)Cbar[o - L.PZ];
    if (j == L.ny - 1) cb += (double)Cbar[o + L.PZ];
    if (k == 0) cb += (double)Cbar[o - 1];
    if (k == L.nz - 1) cb += (double)Cbar[o + 1];
    if (cb == 0.0) continue;
    const double f = (double)PHI[c];
    const double rr = (1.0 - f) / (f + e);
    const double dcdphi = -coef * b * pow(rr, b - 1.0) * (1.0 + e) / ((f + e) * (f + e));
    phibar[c] += cb * dcdphi;
  }
}

// -------------------------------------------------------- k-omega reverse
// Velocity gradients and |S|^2 at cell o, the same expressions as the
// forward turbulence update.
template <class T>
struct Strain {
  T g[3][3];   // g[c][d] = d u_c / d x_d
  T S2;
};

template <class T>
__device__ __forceinline__ Strain<T> strain_at(const Params<T>& P, const T* __restrict__ U, const T* __restrict__ V,
                                               const T* __restrict__ W, long long o) {
  const Layout& L = P.L;
  const long long SX = L.SX, PZ = L.PZ;
  const T h0 = T(0.5) * P.ih[0], h1 = T(0.5) * P.ih[1], h2 = T(0.5) * P.ih[2];
  auto uc = [&](long long q) { return T(0.5) * (U[q] + U[q + SX]); };
  auto vc = [&](long long q) { return T(0.5) * (V[q] + V[q + PZ]); };
  auto wc = [&](long long q) { return T(0.5) * (W[q] + W[q + 1]); };
  Strain<T> s;
  s.g[0][0] = (U[o + SX] - U[o]) * P.ih[0];
  s.g[1][1] = (V[o + PZ] - V[o]) * P.ih[1];
  s.g[2][2] = (W[o + 1] - W[o]) * P.ih[2];
  s.g[0][1] = (uc(o + PZ) - uc(o - PZ)) * h1;
  s.g[0][2] = (uc(o + 1) - uc(o - 1)) * h2;
  s.g[1][0] = (vc(o + SX) - vc(o - SX)) * h0;
  s.g[1][2] = (vc(o + 1) - vc(o - 1)) * h2;
  s.g[2][0] = (wc(o + SX) - wc(o - SX)) * h0;
  s.g[2][1] = (wc(o + PZ) - wc(o - PZ)) * h1;
  const T s01 = T(0.5) * (s.g[0][1] + s.g[1][0]), s02 = T(0.5) * (s.g[0][2] + s.g[2][0]);
  const T s12 = T(0.5) * (s.g[1][2] + s.g[2][1]);
  s.S2 = s.g[0][0] * s.g[0][0] + s.g[1][1] * s.g[1][1] + s.g[2][2] * s.g[2][2] +
         T(2) * (s01 * s01 + s02 * s02 + s12 * s12);
  return s;
}

// nu_t = min(max(k / max(omega, lim), 0), cap), lim = lim_coef |S|, and its
// derivatives where it is not clipped.
template <class T>
struct Nut {
  T nut, dk, dw, dS2;
};

template <class T>
__device__ __forceinline__ Nut<T> nut_of(const Params<T>& P, T kk, T ww, T S2) {
  Nut<T> n;
  const T root = sqrt(S2);
  const T lim = P.lim_coef * root;
  const bool den_w = ww != ww || ww > lim;   // which argument nmax returns
  const T den = den_w ? ww : lim;
  const T r = kk / den;
  n.nut = nmin(nmax(r, T(0)), P.cap);
  const bool live = r > T(0) && r < P.cap;
  n.dk = live ? T(1) / den : T(0);
  const T dden = live ? -r / den : T(0);
  n.dw = den_w ? dden : T(0);
  n.dS2 = (!den_w && root > T(0)) ? dden * P.lim_coef / (T(2) * root) : T(0);
  return n;
}

// Reverse of the k-omega update at one cell (the forward runs on the new
// velocity U and the old k, omega).  kb, wb, nb: adjoints of the new k,
// omega and nu_t; writes the adjoints of the old k and omega (atomic: the
// advection and Laplacian stencils reach the neighbours) and of U.
// Writes, per cell, the adjoints of its velocity gradients (SB.a[0]: the
// diagonal ones times 2 g_dd, SB.a[1]: the symmetric pairs 01, 02, 12 times
// g_cd + g_dc, all times the |S|^2 adjoint) and of its cell-centre velocity
// (SB.a[2]); k_strain_gather moves them to the faces.
template <class T>
__global__ __launch_bounds__(256) void k_turb_adj(Params<T> P, const T* __restrict__ U, const T* __restrict__ V,
                                                  const T* __restrict__ W, const T* __restrict__ K0,
                                                  const T* __restrict__ W0, const T* __restrict__ KB1,
                                                  const T* __restrict__ WB1, const T* __restrict__ NB1,
                                                  T* __restrict__ KB0, T* __restrict__ WB0, VelAdj<T> SB) {
  const Layout& L = P.L;
  const long long n = (long long)L.nx * L.ny * L.nz;
  for (long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x; c < n; c += (long long)gridDim.x * blockDim.x) {
    const int k = (int)(c % L.nz);
    const long long rr = c / L.nz;
    const int j = (int)(rr % L.ny);
    const int i = (int)(rr / L.ny);
    const long long o = L.at(i, j, k);
    const T kb1 = KB1[o], wb1 = WB1[o], nb1 = NB1[o];
    if (kb1 == T(0) && wb1 == T(0) && nb1 == T(0)) {
#pragma unroll
      for (int q = 0; q < 9; ++q) SB.a[q / 3][q % 3][o] = T(0);
      continue;
    }
    const long long st[3] = {L.SX, (long long)L.PZ, 1LL};
    // forward recompute
    const Strain<T> s = strain_at(P, U, V, W, o);
    const T kk = K0[o], ww = W0[o];
    const Nut<T> nu0 = nut_of(P, kk, ww, s.S2);
    const T vel[3] = {T(0.5) * (U[o] + U[o + L.SX]), T(0.5) * (V[o] + V[o + L.PZ]), T(0.5) * (W[o] + W[o + 1])};
    auto adv = [&](const T* q) {
      const T cq = q[o];
      T a = (nmax(vel[0], T(0)) * (cq - q[o - L.SX]) + nmin(vel[0], T(0)) * (q[o + L.SX] - cq)) * P.ih[0];
      a += (nmax(vel[1], T(0)) * (cq - q[o - L.PZ]) + nmin(vel[1], T(0)) * (q[o + L.PZ] - cq)) * P.ih[1];
      a += (nmax(vel[2], T(0)) * (cq - q[o - 1]) + nmin(vel[2], T(0)) * (q[o + 1] - cq)) * P.ih[2];
      return a;
    };
    auto lap = [&](const T* q) {
      const T cq = q[o];
      return (q[o + L.SX] - T(2) * cq + q[o - L.SX]) * P.ih2[0] + (q[o + L.PZ] - T(2) * cq + q[o - L.PZ]) * P.ih2[1] +
             (q[o + 1] - T(2) * cq + q[o - 1]) * P.ih2[2];
    };
    const T lapK = lap(K0), lapW = lap(W0);
    const T knr = kk + P.dt * (-adv(K0) + T(2) * nu0.nut * s.S2 - T(kCmu) * kk * ww +
                               (P.nu + T(kSigmaStar) * nu0.nut) * lapK);
    const T wnr = ww + P.dt * (-adv(W0) + T(2 * kAlpha) * s.S2 - T(kBeta) * ww * ww + (P.nu + T(kSigma) * nu0.nut) * lapW);
    const bool kfree = knr != knr || knr > P.k_min, wfree = wnr != wnr || wnr > P.w_min;
    const T kn = kfree ? knr : P.k_min, wn = wfree ? wnr : P.w_min;
    // the new eddy viscosity
    const Nut<T> nu1 = nut_of(P, kn, wn, s.S2);
    T s2b = nb1 * nu1.dS2;
    const T bk = kfree ? kb1 + nb1 * nu1.dk : T(0);
    const T bw = wfree ? wb1 + nb1 * nu1.dw : T(0);
    // through the explicit update
    const T nutb = bk * P.dt * (T(2) * s.S2 + T(kSigmaStar) * lapK) + bw * P.dt * T(kSigma) * lapW;
    s2b += bk * P.dt * T(2) * nu0.nut + bw * P.dt * T(2 * kAlpha);
    T kkb = bk * (T(1) - P.dt * T(kCmu) * ww) + nutb * nu0.dk;
    T wwb = -bk * P.dt * T(kCmu) * kk + bw * (T(1) - P.dt * T(2 * kBeta) * ww) + nutb * nu0.dw;
    s2b += nutb * nu0.dS2;
    T velb[3] = {T(0), T(0), T(0)};
    // advection and Laplacian of q with weight cw = (adjoint) dt and diffusivity dq
    auto stencil_adj = [&](const T* q, T* QB, T cw, T dq, T& centre) {
      if (cw == T(0)) return;
      const T cq = q[o];
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const T up = nmax(vel[a], T(0)), dn = nmin(vel[a], T(0));
        centre += cw * (-(up - dn) * P.ih[a] - T(2) * dq * P.ih2[a]);
        add_to(QB + o - st[a], cw * (up * P.ih[a] + dq * P.ih2[a]));
        add_to(QB + o + st[a], cw * (-dn * P.ih[a] + dq * P.ih2[a]));
        const T slope = vel[a] > T(0) ? cq - q[o - st[a]] : (vel[a] < T(0) ? q[o + st[a]] - cq : T(0));
        velb[a] -= cw * slope * P.ih[a];
      }
    };
    stencil_adj(K0, KB0, bk * P.dt, P.nu + T(kSigmaStar) * nu0.nut, kkb);
    stencil_adj(W0, WB0, bw * P.dt, P.nu + T(kSigma) * nu0.nut, wwb);
    add_to(KB0 + o, kkb);
    add_to(WB0 + o, wwb);
    SB.a[0][0][o] = T(2) * s.g[0][0] * s2b;
    SB.a[0][1][o] = T(2) * s.g[1][1] * s2b;
    SB.a[0][2][o] = T(2) * s.g[2][2] * s2b;
    SB.a[1][0][o] = (s.g[0][1] + s.g[1][0]) * s2b;
    SB.a[1][1][o] = (s.g[0][2] + s.g[2][0]) * s2b;
    SB.a[1][2][o] = (s.g[1][2] + s.g[2][1]) * s2b;
    SB.a[2][0][o] = velb[0];
    SB.a[2][1][o] = velb[1];
    SB.a[2][2][o] = velb[2];
  }
}

// Transpose of the velocity gradients and cell-centre velocities of
// k_turb_adj, as a gather over every padded face position t of component C:
// g_CC of cells t - e_C (+) and t (-); the centred cross differences
// d u_C / d x_d of cells t -/+ e_d and t -/+ e_d - e_C; the cell-centre
// velocity of cells t and t - e_C.  Cells outside the grid give nothing.
template <int C, class T>
__device__ __forceinline__ T strain_gather_value(const Params<T>& P, const VelAdj<T>& SB, int i, int j, int k) {
  const Layout& L = P.L;
  auto val = [&](int a, int b, int ci, int cj, int ck) -> T {
    if (ci < 0 || cj < 0 || ck < 0 || ci >= L.nx || cj >= L.ny || ck >= L.nz) return T(0);
    return SB.a[a][b][L.at(ci, cj, ck)];
  };
  const int ec[3] = {C == 0, C == 1, C == 2};
  T s = (val(0, C, i - ec[0], j - ec[1], k - ec[2]) - val(0, C, i, j, k)) * P.ih[C];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    if (d == C) continue;
    const int pair = (C + d == 1) ? 0 : ((C + d == 2) ? 1 : 2);   // 01, 02, 12
    const int ed[3] = {d == 0, d == 1, d == 2};
    const T q = T(0.25) * P.ih[d];
    s += q * (val(1, pair, i - ed[0], j - ed[1], k - ed[2]) +
              val(1, pair, i - ed[0] - ec[0], j - ed[1] - ec[1], k - ed[2] - ec[2]) -
              val(1, pair, i + ed[0], j + ed[1], k + ed[2]) -
              val(1, pair, i + ed[0] - ec[0], j + ed[1] - ec[1], k + ed[2] - ec[2]));
  }
  s += T(0.5) * (val(2, C, i, j, k) + val(2, C, i - ec[0], j - ec[1], k - ec[2]));
  return s;
}

template <class T>
__global__ __launch_bounds__(256) void k_strain_gather(Params<T> P, VelAdj<T> SB, T* __restrict__ G0,
                                                       T* __restrict__ G1, T* __restrict__ G2, long long nelem) {
  const Layout& L = P.L;
  for (long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x; p < nelem;
       p += (long long)gridDim.x * blockDim.x) {
    const int i = (int)(p / L.SX) - 1;
    const long long r = p - (long long)(i + 1) * L.SX;
    const int j = (int)(r / L.PZ) - 1;
    const int k = (int)(r - (long long)(j + 1) * L.PZ) - 1;
    G0[p] += strain_gather_value<0>(P, SB, i, j, k);
    G1[p] += strain_gather_value<1>(P, SB, i, j, k);
    G2[p] += strain_gather_value<2>(P, SB, i, j, k);
  }
}

// Reverse of store_cell for a cell field: each face-adjacent ghost's
// adjoint goes to its cell, except across an inlet side when the ghost held
// the inlet constant (use_inlet); ghosts cleared.
template <class T>
__global__ __launch_bounds__(256) void k_cell_fold(Params<T> P, T* __restrict__ q, int use_inlet) {
  const Layout& L = P.L;
  const long long n = (long long)L.nx * L.ny * L.nz;
  for (long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x; c < n; c += (long long)gridDim.x * blockDim.x) {
    const int k = (int)(c % L.nz);
    const long long rr = c / L.nz;
    const int j = (int)(rr % L.ny);
    const int i = (int)(rr / L.ny);
    const int idx[3] = {i, j, k}, nn[3] = {L.nx, L.ny, L.nz};
    const long long st[3] = {L.SX, (long long)L.PZ, 1LL};
    const long long o = L.at(i, j, k);
    T acc = q[o];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
#pragma unroll
      for (int hi = 0; hi < 2; ++hi) {
        if (idx[a] != (hi ? nn[a] - 1 : 0)) continue;
        const long long gpos = o + (hi ? st[a] : -st[a]);
        if (!(use_inlet && P.bc[2 * a + hi] == INLET)) acc += q[gpos];
        q[gpos] = T(0);
      }
    }
    q[o] = acc;
  }
}

// Adjoint of the eddy viscosity the diffusion read: face f of component C
// uses nu + (nu_t[c - e_C] + nu_t[c]) / 2 times dt lap(q)_f, so each cell
// gathers half of dt lap(q)_f a_f from the two faces beside it along each
// axis; a ghost cell copies its interior neighbour, so a boundary cell also
// takes the half that went to its ghost.  Writes nb at interior cells.
template <int C, class T>
__device__ __forceinline__ T nut_face_term(const Params<T>& P, const T* __restrict__ q, const T* __restrict__ a,
                                           int i, int j, int k) {
  const T ab = adj_in<C>(P, a, i, j, k);
  if (ab == T(0)) return T(0);
  const Layout& L = P.L;
  const long long o = L.at(i, j, k);
  const T qc = q[o];
  const T lp = (q[o + L.SX] - T(2) * qc + q[o - L.SX]) * P.ih2[0] +
               (q[o + L.PZ] - T(2) * qc + q[o - L.PZ]) * P.ih2[1] + (q[o + 1] - T(2) * qc + q[o - 1]) * P.ih2[2];
  return T(0.5) * P.dt * lp * ab;
}

template <class T>
__global__ __launch_bounds__(256) void k_diffuse_nut_adj(Params<T> P, const T* __restrict__ Q0,
                                                         const T* __restrict__ Q1, const T* __restrict__ Q2,
                                                         const T* __restrict__ A0, const T* __restrict__ A1,
                                                         const T* __restrict__ A2, T* __restrict__ NB) {
  const Layout& L = P.L;
  const long long n = (long long)L.nx * L.ny * L.nz;
  for (long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x; c < n; c += (long long)gridDim.x * blockDim.x) {
    const int k = (int)(c % L.nz);
    const long long rr = c / L.nz;
    const int j = (int)(rr % L.ny);
    const int i = (int)(rr / L.ny);
    T s = T(0);
    {
      const T lo = nut_face_term<0>(P, Q0, A0, i, j, k), hi = nut_face_term<0>(P, Q0, A0, i + 1, j, k);
      s += lo + hi + (i == 0 ? lo : T(0)) + (i == L.nx - 1 ? hi : T(0));
    }
    {
      const T lo = nut_face_term<1>(P, Q1, A1, i, j, k), hi = nut_face_term<1>(P, Q1, A1, i, j + 1, k);
      s += lo + hi + (j == 0 ? lo : T(0)) + (j == L.ny - 1 ? hi : T(0));
    }
    {
      const T lo = nut_face_term<2>(P, Q2, A2, i, j, k), hi = nut_face_term<2>(P, Q2, A2, i, j, k + 1);
      s += lo + hi + (k == 0 ? lo : T(0)) + (k == L.nz - 1 ? hi : T(0));
    }
    NB[L.at(i, j, k)] = s;
  }
}

// ---------------------------------------------------------- objective seed
// Derivative of a region objective with respect to the faces of the state:
// each face is half of the cell-centre velocity of its two cells, so
// dJ/du_f = (dJ/dU_c[C] + dJ/dU_c'[C]) / 2 over the adjacent cells inside
// the grid.  kind 0 (mean speeds): dJ/dU_c = (sum over the regions holding
// c of coef_r) U_c / |U_c|; kind 2 (desired field): (sum of coef_r)
// (U_c - U_target,c).  coef_r is precomputed by the host.  The plane
// objective has a kernel of its own.

// The plane objective at column (i, j): the cell-centre velocity and the
// porosity interpolated between layers k0 and k0 + 1 with weight t, and
// s = sqrt(|u_p|^2 + 1e-12), as the forward evaluates them.
struct PlaneSeed {
  int k0;
  double t, st, smin, wpen, area;
};

template <class T>
__device__ __forceinline__ void plane_column(const Layout& L, const T* __restrict__ U, const T* __restrict__ V,
                                             const T* __restrict__ W, const T* __restrict__ PHI, const PlaneSeed& ps,
                                             int i, int j, double up[3], double& phip, double& s) {
  double uc[2], vc[2], wc[2], ph[2];
  for (int q = 0; q < 2; ++q) {
    const long long o = L.at(i, j, ps.k0 + q);
    uc[q] = 0.5 * ((double)U[o] + (double)U[o + L.SX]);
    vc[q] = 0.5 * ((double)V[o] + (double)V[o + L.PZ]);
    wc[q] = 0.5 * ((double)W[o] + (double)W[o + 1]);
    ph[q] = (double)PHI[((size_t)i * L.ny + j) * L.nz + ps.k0 + q];
  }
  up[0] = (1.0 - ps.t) * uc[0] + ps.t * uc[1];
  up[1] = (1.0 - ps.t) * vc[0] + ps.t * vc[1];
  up[2] = (1.0 - ps.t) * wc[0] + ps.t * wc[1];
  phip = (1.0 - ps.t) * ph[0] + ps.t * ph[1];
  s = sqrt(up[0] * up[0] + up[1] * up[1] + up[2] * up[2] + 1e-12);
}

template <class T>
__device__ __forceinline__ T seed_cell(const Params<T>& P, const T* __restrict__ U, const T* __restrict__ V,
                                       const T* __restrict__ W, const int* __restrict__ boxes,
                                       const double* __restrict__ coef, int nreg, int kind,
                                       const T* __restrict__ ut, int C, int i, int j, int k) {
  const Layout& L = P.L;
  double cs = 0.0;
  for (int r = 0; r < nreg; ++r) {
    const int* b = boxes + 6 * r;
    if (i >= b[0] && i < b[1] && j >= b[2] && j < b[3] && k >= b[4] && k < b[5]) cs += coef[r];
  }
  if (cs == 0.0) return T(0);
  const long long o = L.at(i, j, k);
  const double uc[3] = {0.5 * ((double)U[o] + (double)U[o + L.SX]), 0.5 * ((double)V[o] + (double)V[o + L.PZ]),
                        0.5 * ((double)W[o] + (double)W[o + 1])};
  if (kind == 0) {
    const double s = sqrt(uc[0] * uc[0] + uc[1] * uc[1] + uc[2] * uc[2]);
    return s > 0.0 ? T(cs * uc[C] / s) : T(0);
  }
  const size_t n = (size_t)L.nx * L.ny * L.nz;
  const size_t cidx = ((size_t)i * L.ny + j) * L.nz + k;
  return T(cs * (uc[C] - (double)ut[(size_t)C * n + cidx]));
}

constexpr int kSeedFaces = 4;   // faces of a thread, a block apart

// The faces of component C in plane i, from face p0 of the plane on.
template <int C, class T>
__device__ __forceinline__ void seed_faces(const Params<T>& P, const T* __restrict__ U, const T* __restrict__ V,
                                           const T* __restrict__ W, const int* __restrict__ boxes,
                                           const double* __restrict__ coef, int nreg, int kind,
                                           const T* __restrict__ ut, T* __restrict__ out, int i, int p0) {
  const Layout& L = P.L;
  const int e1 = L.ny + (C == 1), e2 = L.nz + (C == 2), n = e1 * e2;
  const int nC = C == 0 ? L.nx : (C == 1 ? L.ny : L.nz);
  T* row = out + (size_t)i * n;
#pragma unroll
  for (int u = 0; u < kSeedFaces; ++u) {
    const int p = p0 + u * 256;
    if (p >= n) return;
    const int j = p / e2, k = p - j * e2;
    const int m = C == 0 ? i : (C == 1 ? j : k);
    T s = T(0);
    if (m > 0) s += seed_cell(P, U, V, W, boxes, coef, nreg, kind, ut, C, i - (C == 0), j - (C == 1), k - (C == 2));
    if (m < nC) s += seed_cell(P, U, V, W, boxes, coef, nreg, kind, ut, C, i, j, k);
    row[p] = T(0.5) * s;
  }
}

// gx blocks per plane of faces normal to x: nx + 1 planes of u, nx of v, nx
// of w, in the order of the output, faces of a plane by 32-bit index.
template <class T>
__global__ __launch_bounds__(256) void k_objective_seed(Params<T> P, int gx, const T* __restrict__ U,
                                                        const T* __restrict__ V, const T* __restrict__ W,
                                                        const int* __restrict__ boxes,
                                                        const double* __restrict__ coef, int nreg, int kind,
                                                        const T* __restrict__ ut, T* __restrict__ out) {
  const Layout& L = P.L;
  const size_t n0 = (size_t)(L.nx + 1) * L.ny * L.nz, n1 = (size_t)L.nx * (L.ny + 1) * L.nz;
  const int plane = (int)blockIdx.x / gx;
  const int p0 = ((int)blockIdx.x - plane * gx) * (256 * kSeedFaces) + (int)threadIdx.x;
  if (plane <= L.nx)
    seed_faces<0>(P, U, V, W, boxes, coef, nreg, kind, ut, out, plane, p0);
  else if (plane <= 2 * L.nx)
    seed_faces<1>(P, U, V, W, boxes, coef, nreg, kind, ut, out + n0, plane - L.nx - 1, p0);
  else
    seed_faces<2>(P, U, V, W, boxes, coef, nreg, kind, ut, out + n0 + n1, plane - 2 * L.nx - 1, p0);
}

// Zeros, 16 bytes at a time from the first aligned element on.
template <class T>
__global__ __launch_bounds__(256) void k_seed_zero(T* __restrict__ out, size_t n) {
  constexpr size_t V = 16 / sizeof(T);
  const size_t head = min(n, (size_t)((16 - ((uintptr_t)out & 15)) & 15) / sizeof(T));
  const size_t nv = (n - head) / V, tail = head + nv * V;
  uint4* q = reinterpret_cast<uint4*>(out + head);
  const size_t t = (size_t)blockIdx.x * 256 + threadIdx.x, nt = (size_t)gridDim.x * 256;
  for (size_t v = t; v < nv; v += nt) q[v] = make_uint4(0, 0, 0, 0);
  if (t < head) out[t] = T(0);
  if (t < n - tail) out[tail + t] = T(0);
}

// The plane objective's seed on the two layers of cells beside the plane:
// dJ/ds = area phi_p (2 (s - s_t) - 2 w max(0, s_min - s)), ds/du_p = u_p /
// s; and its direct porosity weight dJ/dphi_p = area ((s - s_t)^2 + w max(0,
// s_min - s)^2), split (1 - t) / t onto the two layers.  A block evaluates
// 16 x 16 columns, one per thread, into LDS and writes the faces of the
// 15 x 15 of them whose lower neighbours it has too.  The rest of the seed
// is zero and is written before (k_seed_zero, 51 MB at 256x256x64 in FP32).
// One kernel over all faces spent its time on those, in index arithmetic and
// in roots and quotients that every wavefront evaluated for the two of its
// faces that need them: 119 us and 8 for the porosity; these two take 10 and
// 14 us (the chain of a column's loads, root and quotients bounds the
// second: 324 blocks).
constexpr int kPlaneTile = 16;

template <class T>
__global__ __launch_bounds__(256) void k_plane_seed(Layout L, int gx, const T* __restrict__ U, const T* __restrict__ V,
                                                    const T* __restrict__ W, const T* __restrict__ PHI, PlaneSeed ps,
                                                    T* __restrict__ out, double* __restrict__ phibar) {
  __shared__ T col[3][2][kPlaneTile][kPlaneTile + 1];
  const int a = threadIdx.x / kPlaneTile, b = threadIdx.x % kPlaneTile;
  const int bi = (int)blockIdx.x / gx, bj = (int)blockIdx.x - bi * gx;
  const int i = bi * (kPlaneTile - 1) + a - 1, j = bj * (kPlaneTile - 1) + b - 1;
  const bool in = i >= 0 && i < L.nx && j >= 0 && j < L.ny, own = a > 0 && b > 0;
  T c[3][2] = {};
  if (in) {
    double up[3], phip, s;
    plane_column(L, U, V, W, PHI, ps, i, j, up, phip, s);
    const double lo = fmax(0.0, ps.smin - s);
    const double dJds = ps.area * phip * (2.0 * (s - ps.st) - 2.0 * ps.wpen * lo);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      c[q][0] = T((1.0 - ps.t) * dJds * up[q] / s);
      c[q][1] = T(ps.t * dJds * up[q] / s);
    }
    if (phibar && own) {
      const double d = ps.area * ((s - ps.st) * (s - ps.st) + ps.wpen * lo * lo);
      const size_t base = ((size_t)i * L.ny + j) * L.nz + ps.k0;
      phibar[base] += (1.0 - ps.t) * d;
      phibar[base + 1] += ps.t * d;
    }
  }
#pragma unroll
  for (int q = 0; q < 3; ++q)
#pragma unroll
    for (int m = 0; m < 2; ++m) col[q][m][a][b] = c[q][m];
  __syncthreads();
  if (!own || i > L.nx || j > L.ny) return;
  const size_t n0 = (size_t)(L.nx + 1) * L.ny * L.nz, n1 = (size_t)L.nx * (L.ny + 1) * L.nz;
  T* u = out + ((size_t)i * L.ny + j) * L.nz + ps.k0;
  T* v = out + n0 + ((size_t)i * (L.ny + 1) + j) * L.nz + ps.k0;
  T* w = out + n0 + n1 + ((size_t)i * L.ny + j) * (L.nz + 1) + ps.k0;
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    // the sum over the face's cells, from zero in their order
    if (j < L.ny) u[m] = T(0.5) * (T(0) + col[0][m][a - 1][b] + c[0][m]);
    if (i < L.nx) v[m] = T(0.5) * (T(0) + col[1][m][a][b - 1] + c[1][m]);
  }
  if (!in) return;
  w[0] = T(0.5) * (T(0) + c[2][0]);
  w[1] = T(0.5) * (T(0) + c[2][0] + c[2][1]);
  w[2] = T(0.5) * (T(0) + c[2][1]);
}

// ----------------------------------------------------------------- launchers
template <class T>
static VelAdj<T> vel_adj(const Grid& g) {
  VelAdj<T> V;
  for (int c = 0; c < 3; ++c)
    for (int cp = 0; cp < 3; ++cp) V.a[c][cp] = (T*)g.AV[c][cp];
  return V;
}

template <class T>
static void launch_vel_gather(Grid& g, const Params<T>& P, void* const G[3]) {
  const int gx = (int)((P.L.SX + 255) / 256);
  hipLaunchKernelGGL(k_vel_gather<T>, dim3((unsigned)gx * (unsigned)(P.L.nx + 3)), dim3(256), 0, g.stream, P, gx,
                     vel_adj<T>(g), (T*)G[0], (T*)G[1], (T*)G[2]);
}

template <bool CORR, class T>
static void launch_march_adj(Grid& g, const Params<T>& P, const AdvectAdj<T>& M) {
  const Layout& L = P.L;
  March G = march_geom(L.nx - 2, L.ny - 2, L.nz + 3, march_edges(L));
  G.len = 8;   // a chunk adds two planes to its neighbours' (4 planes: 451 + 295 us, 8: 395 + 277, 16: 382 + 281)
  G.nch = 3 * ((L.nx - 2 + G.len - 1) / G.len);   // a block computes one component
  auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, march_grid(G), dim3(kMarch), 0, g.stream, P, G, M); };
  if (G.shape == 0) go(k_advect_adj_march<CORR, 0, T>);
  else if (G.shape == 1) go(k_advect_adj_march<CORR, 1, T>);
  else go(k_advect_adj_march<CORR, 2, T>);
}

template <class T>
void launch_advect_adj(Grid& g, const Params<T>& P, void* const Qin[3], void* const Qhat[3], void* const Aout[3],
                       void* const Gq[3], void* const Ghat[3]) {
  const dim3 grid = adj_face_grid(P.L);
  if constexpr (sizeof(T) == 4) if (march_pays(P, kMarchFaces)) {
    AdvectAdj<T> M;
    for (int c = 0; c < 3; ++c) {
      M.q[c] = (const T*)Qin[c];
      M.qhat[c] = (const T*)Qhat[c];
      M.a[c] = (const T*)Aout[c];
      M.g[c] = (T*)Gq[c];
      M.h[c] = (T*)Ghat[c];
    }
    M.va = vel_adj<T>(g);
    launch_march_adj<true>(g, P, M);
    launch_fold<T>(g, P, Ghat);
    for (int c = 0; c < 3; ++c) M.a[c] = (const T*)Ghat[c];
    launch_march_adj<false>(g, P, M);
    launch_vel_gather<T>(g, P, Gq);
    return;
  }
  hipLaunchKernelGGL(k_advect_corr_adj<T>, grid, dim3(kFaceBlock), 0, g.stream, P, (const T*)Qin[0],
                     (const T*)Qin[1], (const T*)Qin[2], (const T*)Qhat[0], (const T*)Qhat[1], (const T*)Qhat[2],
                     (const T*)Aout[0], (const T*)Aout[1], (const T*)Aout[2], (T*)Gq[0], (T*)Gq[1], (T*)Gq[2],
                     (T*)Ghat[0], (T*)Ghat[1], (T*)Ghat[2], vel_adj<T>(g));
  // qhat's ghosts came from its interior faces: fold them before its reverse
  launch_fold<T>(g, P, Ghat);
  hipLaunchKernelGGL(k_advect_fwd_adj<T>, grid, dim3(kFaceBlock), 0, g.stream, P, (const T*)Qin[0],
                     (const T*)Qin[1], (const T*)Qin[2], (const T*)Ghat[0], (const T*)Ghat[1], (const T*)Ghat[2],
                     (T*)Gq[0], (T*)Gq[1], (T*)Gq[2], vel_adj<T>(g));
  launch_vel_gather<T>(g, P, Gq);
}

template <class T>
void launch_diffuse_adj(Grid& g, const Params<T>& P, void* const Aout[3], void* const Gin[3]) {
  const int gx = (int)((P.L.SX + 255) / 256);
  hipLaunchKernelGGL(k_diffuse_adj<T>, dim3((unsigned)gx * (unsigned)(P.L.nx + 3)), dim3(256), 0, g.stream, P, gx,
                     (const T*)Aout[0], (const T*)Aout[1], (const T*)Aout[2], (const T*)g.NUT, (T*)Gin[0], (T*)Gin[1],
                     (T*)Gin[2]);
}

template <class T>
void launch_drag_adj(Grid& g, const Params<T>& P, void* const Qin[3], void* const Aout[3], void* const Gin[3],
                     void* Cbar) {
  hipLaunchKernelGGL(k_drag_adj<T>, adj_face_grid(P.L), dim3(kFaceBlock), 0, g.stream, P, (const T*)Qin[0],
                     (const T*)Qin[1], (const T*)Qin[2], (const T*)g.C, (const T*)Aout[0], (const T*)Aout[1],
                     (const T*)Aout[2], (T*)Cbar, vel_adj<T>(g));
  launch_vel_gather<T>(g, P, Gin);
}

template <class T>
void launch_fold(Grid& g, const Params<T>& P, void* const A[3]) {
  const long long n = fold_corners(P.L);
  hipLaunchKernelGGL(k_fold<T>, dim3((unsigned)((n + kFaceBlock - 1) / kFaceBlock)), dim3(kFaceBlock), 0, g.stream, P,
                     (T*)A[0], (T*)A[1], (T*)A[2], (int)n);
}

template <class T>
void launch_drag_coef_adj(Grid& g, const Params<T>& P, const void* Cbar, double* phibar) {
  const long long n = (long long)P.L.nx * P.L.ny * P.L.nz;
  const int blocks = (int)std::min<long long>((n + 255) / 256, 8192);
  const uf_config& c = g.cfg;
  hipLaunchKernelGGL(k_drag_coef_adj<T>, dim3(blocks), dim3(256), 0, g.stream, P, (const T*)Cbar, (const T*)g.PHI,
                     phibar, c.Cd * c.a, c.e, c.b);
}

template <class T>
void launch_objective_seed(Grid& g, const Params<T>& P, const int* boxes_dev, const double* coef_dev, int nreg,
                           int kind, const void* ut, void* out, const double plane[6], double* phibar) {
  const Layout& L = P.L;
  void* const* Q = g.Q[g.cur];
  if (!plane) {
    const int gx = (std::max((L.ny + 1) * L.nz, L.ny * (L.nz + 1)) + 256 * kSeedFaces - 1) / (256 * kSeedFaces);
    hipLaunchKernelGGL(k_objective_seed<T>, dim3((unsigned)gx * (unsigned)(3 * L.nx + 1)), dim3(256), 0, g.stream, P,
                       gx, (const T*)Q[0], (const T*)Q[1], (const T*)Q[2], boxes_dev, coef_dev, nreg, kind,
                       (const T*)ut, (T*)out);
    return;
  }
  const size_t n = (size_t)(L.nx + 1) * L.ny * L.nz + (size_t)L.nx * (L.ny + 1) * L.nz +
                   (size_t)L.nx * L.ny * (L.nz + 1);
  const PlaneSeed ps{(int)plane[0], plane[1], plane[2], plane[3], plane[4], plane[5]};
  const size_t zb = (n * sizeof(T) / 16 + 1023) / 1024 + 1;   // four stores per thread
  hipLaunchKernelGGL(k_seed_zero<T>, dim3((unsigned)zb), dim3(256), 0, g.stream, (T*)out, n);
  constexpr int own = kPlaneTile - 1;
  const int gx = L.ny / own + 1;
  hipLaunchKernelGGL(k_plane_seed<T>, dim3((unsigned)gx * (unsigned)(L.nx / own + 1)), dim3(256), 0, g.stream, L, gx,
                     (const T*)Q[0], (const T*)Q[1], (const T*)Q[2], (const T*)g.PHI, ps, (T*)out, phibar);
}

static inline int cell_blocks(const Layout& L) {
  const long long n = (long long)L.nx * L.ny * L.nz;
  return (int)std::min<long long>((n + 255) / 256, 8192);
}

template <class T>
void launch_turb_adj(Grid& g, const Params<T>& P, void* const Unew[3], const void* K0, const void* W0,
                     const void* KB1, const void* WB1, const void* NB1, void* KB0, void* WB0, void* const G[3]) {
  // the per-cell values go through the velocity-adjoint arrays, which the
  // next reverse kernel overwrites (its gather reads interior cells only here)
  hipLaunchKernelGGL(k_turb_adj<T>, dim3(cell_blocks(P.L)), dim3(256), 0, g.stream, P, (const T*)Unew[0],
                     (const T*)Unew[1], (const T*)Unew[2], (const T*)K0, (const T*)W0, (const T*)KB1, (const T*)WB1,
                     (const T*)NB1, (T*)KB0, (T*)WB0, vel_adj<T>(g));
  const long long n = (long long)g.nelem;
  const int blocks = (int)std::min<long long>((n + 255) / 256, 16384);
  hipLaunchKernelGGL(k_strain_gather<T>, dim3(blocks), dim3(256), 0, g.stream, P, vel_adj<T>(g), (T*)G[0], (T*)G[1],
                     (T*)G[2], n);
}

template <class T>
void launch_cell_fold(Grid& g, const Params<T>& P, void* q, int use_inlet) {
  hipLaunchKernelGGL(k_cell_fold<T>, dim3(cell_blocks(P.L)), dim3(256), 0, g.stream, P, (T*)q, use_inlet);
}

template <class T>
void launch_diffuse_nut_adj(Grid& g, const Params<T>& P, void* const Qin[3], void* const Aout[3], void* NB) {
  hipLaunchKernelGGL(k_diffuse_nut_adj<T>, dim3(cell_blocks(P.L)), dim3(256), 0, g.stream, P, (const T*)Qin[0],
                     (const T*)Qin[1], (const T*)Qin[2], (const T*)Aout[0], (const T*)Aout[1], (const T*)Aout[2],
                     (T*)NB);
}

#define UF_INST(T)                                                                                             \
  template void launch_advect_adj<T>(Grid&, const Params<T>&, void* const[3], void* const[3], void* const[3],  \
                                     void* const[3], void* const[3]);                                           \
  template void launch_diffuse_adj<T>(Grid&, const Params<T>&, void* const[3], void* const[3]);                \
  template void launch_drag_adj<T>(Grid&, const Params<T>&, void* const[3], void* const[3], void* const[3],    \
                                   void*);                                                                      \
  template void launch_fold<T>(Grid&, const Params<T>&, void* const[3]);                                        \
  template void launch_drag_coef_adj<T>(Grid&, const Params<T>&, const void*, double*);                        \
  template void launch_objective_seed<T>(Grid&, const Params<T>&, const int*, const double*, int, int,         \
                                         const void*, void*, const double*, double*);                           \
  template void launch_turb_adj<T>(Grid&, const Params<T>&, void* const[3], const void*, const void*,         \
                                   const void*, const void*, const void*, void*, void*, void* const[3]);        \
  template void launch_cell_fold<T>(Grid&, const Params<T>&, void*, int);                                      \
  template void launch_diffuse_nut_adj<T>(Grid&, const Params<T>&, void* const[3], void* const[3], void*);
UF_INST(float)
UF_INST(double)
#undef UF_INST

}  // namespace uf
