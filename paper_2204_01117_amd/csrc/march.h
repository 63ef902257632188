// Stages that march along x: a block owns a tile of TJ x TK columns (one per
// thread) over a chunk of planes and keeps the planes i - 1, i and i + 1 of
// the arrays it reads, with a halo of one column, in LDS.  Plane i + 2 is in
// flight into registers while plane i is computed.
//
// Why: a stage that gathers its neighbours from memory issues up to 75 loads
// per corner (corrector), and though nearly all of them hit, the L1's address
// path (about nine cycles for a wavefront's load of a misaligned row) is busy
// 75 to 95% of the time.  Here an element is loaded about 1.4 times per tile
// and stored to LDS, and the gathers are LDS reads.  What then bounds a stage
// is instruction issue, so the tile's shape is a compile-time constant
// (neighbours are immediate offsets), and the rules of the boundary stay out
// of the loop: the planes and rows beside the sides along x and y are left to
// blocks of their own, a thread per corner (with the rules in the loop the
// predictor took 55 us at 256x256x64, without 37),
// and the ghosts beyond the sides along z, of which nearly every
// wavefront has some, have lanes that evaluate the nearest face and store it
// by the side's rule (MarchLane): one store per component without a branch.
//
// Measured (FP32, us per launch, a thread per corner -> marching):
//                256x256x64   450x300x40   512x512x128
//   predictor     69 ->  37    98 ->  48   479 -> 273
//   corrector    113 ->  62   139 ->  78   751 -> 457
//   k-omega       54 ->  46    75 ->  62   451 -> 352
// (the gathering kernels depend on the flow too: 124, 166 and 860 us for the
// corrector of a less regular state; these do not).
#pragma once
#include "face_ops.h"

namespace uf {

constexpr int kMarch = 512;   // threads of a block

// Shapes: TJ rows of up to TKM columns (TJ * TKM <= kMarch), LDS rows of
// TKM + 2.
template <int SHAPE>
struct MarchShape;
template <>
struct MarchShape<0> {
  static constexpr int TJ = 7, TKM = 73;
};
template <>
struct MarchShape<1> {
  static constexpr int TJ = 11, TKM = 46;
};
template <>
struct MarchShape<2> {
  static constexpr int TJ = 22, TKM = 23;
};

// Tiles over ni planes of nj x nk lanes (rows and planes from 1, lanes from k
// = -1) and nedge columns or corners for the threads of the edge blocks:
// shape, lanes per tile row, ntj x ntk tiles and nch chunks of len planes;
// shape -1: none fits.
struct March {
  int shape, TK, ntj, ntk, len, nch;
  int edge;   // blocks of the edges, the first of the launch (a multiple of 8)
};

inline March march_geom(int ni, int nj, int nk, int nedge) {
  const int tj[3] = {MarchShape<0>::TJ, MarchShape<1>::TJ, MarchShape<2>::TJ};
  const int tkm[3] = {MarchShape<0>::TKM, MarchShape<1>::TKM, MarchShape<2>::TKM};
  March G{};
  G.shape = -1;
  double best = 0.0;
  for (int s = 0; s < 3; ++s) {
    const int ntk = (nk + tkm[s] - 1) / tkm[s], ntj = (nj + tj[s] - 1) / tj[s];
    const int tk = (nk + ntk - 1) / ntk;
    // the last tile holds the two ghost lanes and the face they evaluate
    if (ntk > 1 && nk - (ntk - 1) * tk < 4) continue;
    // threads with a lane; the wider rows unless they waste a tenth more
    const double use = (double)nj * nk / ((double)ntj * ntk);
    if (use > 1.1 * best) {
      best = use;
      G.shape = s;
      G.ntk = ntk;
      G.ntj = ntj;
      G.TK = tk;
    }
  }
  // a chunk re-reads two planes, but a block takes 3 to 4 us for a plane when
  // it has its CU to itself, so many short chunks are better than few long
  // ones: about 3000 blocks (corrector in us: 200x200x40 3 planes 28, 6: 30,
  // 12: 39; 256x256x64 2: 67, 4: 62, 8: 63, 12: 72; 512x512x128 3: 501, 6:
  // 463, 8: 458, 24: 483)
  G.len = (int)std::min(8LL, std::max(2LL, ((long long)G.ntj * G.ntk * ni + 2999) / 3000));
  G.nch = (ni + G.len - 1) / G.len;
  G.edge = 8 * ((nedge + 8 * kMarch - 1) / (8 * kMarch));
  return G;
}

// Where marching is the faster way: with too few blocks a CU cannot hide the
// time a block takes per plane.  In FP32 from a quarter of a million corners
// for the advection (predictor and corrector together, us, against a thread
// per corner: 96x64x32 20.5 against 22.4, 129x97x35 24.3 against 30.3,
// 256x256x64 101 against 197) and from 2.5 million cells for
// the k-omega update, whose gathers are fewer (200x200x40 21.5 against 18.8,
// 256x256x64 46.5 against 53.7).  In FP64 the planes in LDS leave one block
// per CU.
template <class T>
inline bool march_pays(const Params<T>& P, double from) {
  const Layout& L = P.L;
  return sizeof(T) == 4 && L.nx > 3 && L.ny > 3 && (double)L.nx * L.ny * L.nz >= from && P.bc[4] != INLET &&
         P.bc[5] != INLET && march_geom(L.nx - 2, L.ny - 2, L.nz + 3, 0).shape >= 0 &&
         march_geom(L.nx - 2, L.ny - 2, L.nz + 2, 0).shape >= 0;
}
constexpr double kMarchFaces = 2.5e5, kMarchTurb = 2.5e6;

// The planes of NA arrays in LDS and this thread's column.
template <int SHAPE, int NA, class T>
struct Planes {
  using S = MarchShape<SHAPE>;
  static constexpr int PITCH = S::TKM + 2, PL = (S::TJ + 2) * PITCH;
  static constexpr int NV = (PL + kMarch - 1) / kMarch;   // elements of a plane per thread
  static constexpr int LDS = 3 * NA * PL;
  const T* src[NA];
  T* lds;                // [slot][array][PL]
  T r[NA][NV];
  unsigned off[NV];      // this thread's elements within a plane of memory
  int le[NV];            // and in LDS; -1: none
  long long SX;
  int s[3];              // slots of planes i - 1, i, i + 1 (element offsets)
  int q;                 // the column being evaluated, in an LDS plane

  // Tile rows j0 - 1 .., columns k0 - 1 .. (TK + 2 of them; k0 from -1),
  // clamped to the padded plane.
  __device__ __forceinline__ void init(const Layout& L, T* mem, int j0, int k0, int TK) {
    lds = mem;
    SX = L.SX;
    const int w = TK + 2, n = (S::TJ + 2) * w;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const int e = (int)threadIdx.x + v * kMarch, a = e / w, b = e - a * w;
      le[v] = e < n ? a * PITCH + b : -1;
      off[v] = (unsigned)min(j0 + a, L.ny + 2) * (unsigned)L.PZ + (unsigned)min(max(k0 + b, 0), L.nz + 2);
    }
    s[0] = 0;
    s[1] = NA * PL;
    s[2] = 2 * NA * PL;
  }
  __device__ __forceinline__ void load(int i) {
#pragma unroll
    for (int a = 0; a < NA; ++a) {
      const T* p = src[a] + (long long)(i + 1) * SX;
#pragma unroll
      for (int v = 0; v < NV; ++v) r[a][v] = p[off[v]];
    }
  }
  __device__ __forceinline__ void store(int slot) {
#pragma unroll
    for (int v = 0; v < NV; ++v)
      if (le[v] >= 0) {
#pragma unroll
        for (int a = 0; a < NA; ++a) lds[slot + a * PL + le[v]] = r[a][v];
      }
  }
  __device__ __forceinline__ void rotate() {
    const int t = s[0];
    s[0] = s[1];
    s[1] = s[2];
    s[2] = t;
  }
  // Array a at (i + dx, j + dj, k + dk).
  __device__ __forceinline__ T at(int a, int dx, int dj, int dk) const {
    return lds[s[dx + 1] + q + a * PL + dj * PITCH + dk];
  }
};

// A barrier for what is in LDS alone: __syncthreads() would also wait for
// the loads of the next plane and the stores of the last.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Runs body(i) for every plane of the block's chunk with planes i - 1, i, i +
// 1 in LDS; planes i0 - 1 .. i1 must exist.  Every thread of the block.
template <int SHAPE, int NA, class T, class F>
__device__ __forceinline__ void march(Planes<SHAPE, NA, T>& A, int i0, int i1, F body) {
  A.load(i0 - 1);
  A.store(A.s[0]);
  A.load(i0);
  A.store(A.s[1]);
  A.load(i0 + 1);
  for (int i = i0; i < i1; ++i) {
    A.store(A.s[2]);
    lds_barrier();
    if (i + 1 < i1) A.load(i + 2);
    body(i);
    lds_barrier();
    A.rotate();
  }
}

// A thread's lane: position (j, k) of the padded plane, k from -1 on.  Its
// column in a plane of memory is oc; qa and qb are the LDS columns of the
// nearest k in [0, na) and in [0, nb).
struct MarchLane {
  int j, k, qa, qb;
  unsigned oc;
  bool active;
};

// nj x nk lanes.
template <int SHAPE>
__device__ __forceinline__ MarchLane march_lane(const Layout& L, const March& G, int tile, int nj, int nk, int na,
                                                int nb, int& j0, int& k0) {
  using S = MarchShape<SHAPE>;
  const int tj = tile / G.ntk, jj = (int)threadIdx.x / G.TK, kk = (int)threadIdx.x - jj * G.TK;
  j0 = 1 + tj * S::TJ;
  k0 = (tile - tj * G.ntk) * G.TK - 1;
  MarchLane c;
  c.j = j0 + jj;
  c.k = k0 + kk;
  c.active = jj < S::TJ && c.j <= nj && c.k < nk - 1;
  const int row = (min(jj, S::TJ - 1) + 1) * (S::TKM + 2) + 1 - k0;
  // (a lane past the end, whose result nobody stores, stays inside its tile)
  c.qa = row + max(k0, min(max(c.k, 0), na - 1));
  c.qb = row + max(k0, min(max(c.k, 0), nb - 1));
  c.oc = (unsigned)(c.j + 1) * (unsigned)L.PZ + (unsigned)(c.k + 1);
  return c;
}

// Stores the value v of component C, evaluated at the face nearest to the lane
// at k, off the sides along x and y and with no inlet along z.  out: the
// padded array; oc: the lane's column in a plane of it.
template <int C, class T>
__device__ __forceinline__ void march_put(const Params<T>& P, T* __restrict__ out, int k, unsigned oc, int i, T v) {
  const Layout& L = P.L;
  T* p = out + (long long)(i + 1) * L.SX;
  if (C == 2) {
    if ((k <= 0 && P.bc[4] != OUTLET) || (k >= L.nz && P.bc[5] != OUTLET)) v = T(0);   // fixed faces
    p[oc] = v;
  } else {
    if ((k < 0 && P.bc[4] == WALL) || (k >= L.nz && P.bc[5] == WALL)) v = -v;
    if (k <= L.nz) p[oc] = v;
  }
}

// face_velocity() of the thread's column.
template <int C, int SHAPE, int NA, class T>
__device__ __forceinline__ void march_velocity(const Planes<SHAPE, NA, T>& A, T vel[3]) {
  constexpr int ec[3] = {C == 0, C == 1, C == 2};
#pragma unroll
  for (int cp = 0; cp < 3; ++cp) {
    if (cp == C) {
      vel[cp] = A.at(cp, 0, 0, 0);
    } else {
      const int e[3] = {cp == 0, cp == 1, cp == 2};
      vel[cp] = T(0.25) * (A.at(cp, -ec[0], -ec[1], -ec[2]) + A.at(cp, e[0] - ec[0], e[1] - ec[1], e[2] - ec[2]) +
                           A.at(cp, 0, 0, 0) + A.at(cp, e[0], e[1], e[2]));
    }
  }
}

// Are all three displacements of every lane shorter than a cell?  The trace
// position of a face is then within the padded array (the clamps of
// trace_axis() do nothing: -1 < n + s < ext for 0 <= n <= ext - 1), its cell
// is the face's or the one before it, and floor() is a comparison.  Stable
// time steps keep it so; other wavefronts take the general path.  False for
// a NaN.
template <class T>
__device__ __forceinline__ bool march_near(const T d[3]) {
  return __all(fabs(d[0]) < T(1) && fabs(d[1]) < T(1) && fabs(d[2]) < T(1));
}

// The samples and weights of array a at the position displaced by s, near.
template <int SHAPE, int NA, class T>
__device__ __forceinline__ void march_samples(const Planes<SHAPE, NA, T>& A, int a, T si, T sj, T sk, Tri<T>& t, T v[8]) {
  constexpr int PITCH = Planes<SHAPE, NA, T>::PITCH, PL = Planes<SHAPE, NA, T>::PL;
  const bool bi = si < T(0), bj = sj < T(0), bk = sk < T(0);
  t.ti = si + (bi ? T(1) : T(0));
  t.tj = sj + (bj ? T(1) : T(0));
  t.tk = sk + (bk ? T(1) : T(0));
  const int q = A.q + (bj ? -PITCH : 0) + (bk ? -1 : 0);
  const T* lo = A.lds + (q + (bi ? A.s[0] : A.s[1])) + a * PL;
  const T* hi = A.lds + (q + (bi ? A.s[1] : A.s[2])) + a * PL;
  v[0] = lo[0];
  v[1] = hi[0];
  v[2] = lo[PITCH];
  v[3] = hi[PITCH];
  v[4] = lo[1];
  v[5] = hi[1];
  v[6] = lo[PITCH + 1];
  v[7] = hi[PITCH + 1];
}

// The corners beside the sides along x (i = 0, nx - 1, nx) and y (j = 0, ny -
// 1, ny), which the tiles leave out: corner e of them.
__host__ __device__ inline int march_edges(const Layout& L) { return 3 * (L.nz + 1) * ((L.ny + 1) + (L.nx - 2)); }

__device__ __forceinline__ bool march_edge_corner(const Layout& L, int e, int& i, int& j, int& k) {
  if (e >= march_edges(L)) return false;
  const int r = e / (L.nz + 1);
  k = e - r * (L.nz + 1);
  if (r < 3 * (L.ny + 1)) {
    const int s = r / (L.ny + 1);
    i = s == 0 ? 0 : L.nx - 2 + s;
    j = r - s * (L.ny + 1);
  } else {
    const int q = r - 3 * (L.ny + 1), s = q / (L.nx - 2);
    j = s == 0 ? 0 : L.ny - 2 + s;
    i = 1 + q - s * (L.nx - 2);
  }
  return true;
}

// The logical block of a marching launch: an edge block (tile -1, chunk its
// number; dealt over the XCDs) or a tile of a chunk (neighbouring tiles on
// one XCD, as xcd_block()).  False for padding blocks.
__device__ __forceinline__ bool march_block(const March& G, int& tile, int& chunk) {
  int b = (int)blockIdx.x;
  if (b < G.edge) {
    tile = -1;
    chunk = b;
    return true;
  }
  b -= G.edge;
  const int per = ((int)gridDim.x - G.edge) >> 3, nt = G.ntj * G.ntk;
  b = (b & 7) * per + (b >> 3);
  if (b >= nt * G.nch) return false;
  chunk = b / nt;
  tile = b - chunk * nt;
  return true;
}

inline dim3 march_grid(const March& G) {
  return dim3((unsigned)(G.edge + 8 * ((G.ntj * G.ntk * G.nch + 7) / 8)));
}

}  // namespace uf
