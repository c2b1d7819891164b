// Small meshes inside one workgroup: the coarse end of the V-cycle (from an
// N0^3 mesh, N0 <= 16, down to 2^3 and back) as one kernel, and whole solves of
// meshes up to 16^3.  They compute what the level-by-level kernels compute
// (Chebyshev-Jacobi smoothing, residual, full-weighting restriction, exact
// solve on 2^3, trilinear prolongation, PCG, refinement), but one launch takes
// the place of ~7 per level and ~10 per iteration, and no vector leaves the CU.
//
// A thread owns four consecutive nodes of a row (16^3: 960 of 1024 threads,
// 8^3: 112 of 128, 4^3: 12 of one wave), one on the coarser levels (small_v).
// Its right-hand side, iterates, inverse diagonal and Krylov vectors stay in its
// registers on every level;
// LDS holds, per level, two copies of the vector the neighbours read (boundary
// positions 0) and kappa.  A stencil takes nine row reads of four values and
// the row halos from the neighbouring lanes, instead of 29 scalar reads a
// node.  The order of every fp32 sum is that of the level-by-level kernels and
// of the earlier scalar form, so a V-cycle keeps its bits: rounding in the inner
// solve shows in Y = Q_l - Q_{l-1} of the finer levels, where it cancels least.
// Bound: LDS latency and the barriers between steps.
// Measured, scalar form with its vectors in LDS (and, for 16^3 and fp64, a launch
// per step) -> this one: a 16^3 / 8^3 pair alone 690 -> 434 us a call, 1131
// pairs 1.69 -> 1.07 ms, 13001 samples of 8^3 1.33 -> 0.94 ms, a plain fp64
// MLMC run on 4^3 to 16^3 (262 samples, Jacobi) 2.85 -> 0.45 ms.
#include "common.hpp"
#include "kernels.hpp"

#include <type_traits>

namespace mlmc {
namespace {

constexpr int kMaxLv = 4;   // 16, 8, 4, 2

struct SmallArgs {
  int degree;
  double c1[16], c2[16];
  size_t gstride;             // grid stride of the N0 level in global memory
  const void* kap[kMaxLv];    // global kappa of each level (element layout, per-sample n^3)
};

__host__ __device__ constexpr int lds_stride(int n) { return ((n + 1) * n * n + n + 1 + 63) / 64 * 64; }

__device__ __forceinline__ int lg2(int n) { return 31 - __clz(n); }

template <class T>
struct V4 { typedef T type __attribute__((ext_vector_type(4))); };
template <class T>
__device__ __forceinline__ void ld4(const T* p, T* d) {
  typedef typename V4<T>::type vt;
  const vt v = *reinterpret_cast<const vt*>(p);
#pragma unroll
  for (int q = 0; q < 4; ++q) d[q] = v[q];
}
template <class T>
__device__ __forceinline__ void st4(T* p, const T* d) {
  typedef typename V4<T>::type vt;
  vt v;
#pragma unroll
  for (int q = 0; q < 4; ++q) v[q] = d[q];
  *reinterpret_cast<vt*>(p) = v;
}

// value of the previous / next lane of the wave (0 beyond its ends)
__device__ __forceinline__ int lane_prev(int x) { return __builtin_amdgcn_update_dpp(0, x, 0x138, 0xF, 0xF, true); }
__device__ __forceinline__ int lane_next(int x) { return __builtin_amdgcn_update_dpp(0, x, 0x130, 0xF, 0xF, true); }
__device__ __forceinline__ float lane_prev(float x) { return __int_as_float(lane_prev(__float_as_int(x))); }
__device__ __forceinline__ float lane_next(float x) { return __int_as_float(lane_next(__float_as_int(x))); }
__device__ __forceinline__ double lane_prev(double x) {
  const long long v = __double_as_longlong(x);
  return __longlong_as_double(((long long)lane_prev((int)(v >> 32)) << 32) | (unsigned)lane_prev((int)v));
}
__device__ __forceinline__ double lane_next(double x) {
  const long long v = __double_as_longlong(x);
  return __longlong_as_double(((long long)lane_next((int)(v >> 32)) << 32) | (unsigned)lane_next((int)v));
}

// N consecutive values
template <int N, class T>
__device__ __forceinline__ void ldv(const T* p, T* d) {
  if constexpr (N == 1) d[0] = *p;
  else ld4(p, d);
}
template <int N, class T>
__device__ __forceinline__ void stv(T* p, const T* d) {
  if constexpr (N == 1) *p = d[0];
  else st4(p, d);
}

// The thread's V = 4 or 1 nodes on the n^3 mesh (n >= 4): lanes of a row are
// consecutive, so the row halos move between lanes.
template <int n, int V = 4>
struct Own {
  static constexpr int G = n / V, NV = (n - 1) * n * G;   // vectors of planes 1 .. n-1
  int gx, pos;
  bool has;       // row j >= 1: holds interior nodes
  __device__ Own() {
    const int v = (int)threadIdx.x;
    gx = v & (G - 1);
    pos = n * n + V * v;
    has = v < NV && ((v / G) & (n - 1)) != 0;
  }
  // columns c = 0 .. V+1: nodes i0-1 .. i0+V of a node row, 0 beyond the mesh
  template <class T>
  __device__ void urow(const T* row, T (&q)[V + 2]) const {
    ldv<V>(row, q + 1);
    if constexpr (G > 1) {
      const T l = lane_prev(q[V]), r = lane_next(q[1]);
      q[0] = gx == 0 ? T(0) : l;
      q[V + 1] = gx == G - 1 ? T(0) : r;
    } else {
      q[0] = q[V + 1] = T(0);
    }
  }
  // columns 0 .. V: elements i0-1 .. i0+V-1 of an element row
  template <class T>
  __device__ void krow(const T* row, T (&q)[V + 1]) const {
    ldv<V>(row, q + 1);
    if constexpr (G > 1) {
      const T l = lane_prev(q[V]);
      q[0] = gx == 0 ? T(0) : l;
    } else {
      q[0] = T(0);
    }
  }
};

// the 8-element kappa sums of the thread's nodes, one element after another
template <int n, int V, class T>
__device__ __forceinline__ void ksum4(const Own<n, V>& o, const T* kap, T (&ks)[V]) {
#pragma unroll
  for (int v = 0; v < V; ++v) ks[v] = T(0);
#pragma unroll
  for (int dz = 0; dz < 2; ++dz)
#pragma unroll
    for (int dy = 0; dy < 2; ++dy) {
      T K[V + 1];
      o.krow(kap + o.pos - n - n * n + n * dy + n * n * dz, K);
#pragma unroll
      for (int v = 0; v < V; ++v) {
        ks[v] += K[v];
        ks[v] += K[v + 1];
      }
    }
}

// A u at the thread's nodes (u in LDS, grid layout), element by element: kappa
// times the sum of its three edge diagonals and its corner
template <int n, int V, class T>
__device__ __forceinline__ void q1v(const Own<n, V>& o, const T* u, const T* kap, T (&au)[V]) {
  constexpr int n2 = n * n;
  const T* up = u + o.pos;
  const T* kp = kap + o.pos - n - n2;
  T f[V], ks[V], M[3][V + 2];   // M: the rows of the node's own plane
#pragma unroll
  for (int r = 0; r < 3; ++r) o.urow(up + n * (r - 1), M[r]);
#pragma unroll
  for (int v = 0; v < V; ++v) f[v] = ks[v] = T(0);
#pragma unroll
  for (int sz = 0; sz < 2; ++sz) {
    T K[2][V + 1], Q[3][V + 2];
    o.krow(kp + n2 * sz, K[0]);
    o.krow(kp + n2 * sz + n, K[1]);
#pragma unroll
    for (int r = 0; r < 3; ++r) o.urow(up + n2 * (2 * sz - 1) + n * (r - 1), Q[r]);
#pragma unroll
    for (int v = 0; v < V; ++v)
#pragma unroll
      for (int sy = 0; sy < 2; ++sy)
#pragma unroll
        for (int sx = 0; sx < 2; ++sx) {
          const T kv = K[sy][v + sx];
          const T g = (M[2 * sy][v + 2 * sx] + Q[1][v + 2 * sx]) + (Q[2 * sy][v + 1] + Q[2 * sy][v + 2 * sx]);
          ks[v] += kv;
          f[v] += kv * g;
        }
  }
  const T h = T(1) / T(n);
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const T a = h * (ks[v] * M[1][v + 1] * (T(1) / T(3)) - f[v] * (T(1) / T(12)));
    au[v] = (v > 0 || o.gx != 0) ? a : T(0);
  }
}

// As q1v, with the kappa sums as a result and one element row at a time: about 35
// values live (the rows of the own plane are read twice), for a kernel held to 64
// registers
template <int n, int V, class T>
__device__ __forceinline__ void q1v_lean(const Own<n, V>& o, const T* u, const T* kap, T (&au)[V], T (&ks)[V]) {
  constexpr int n2 = n * n;
  const T* up = u + o.pos;
  const T* kp = kap + o.pos - n - n2;
  T f[V];
#pragma unroll
  for (int v = 0; v < V; ++v) f[v] = ks[v] = T(0);
#pragma unroll
  for (int sz = 0; sz < 2; ++sz) {
    T Q1[V + 2];
    o.urow(up + n2 * (2 * sz - 1), Q1);
#pragma unroll
    for (int sy = 0; sy < 2; ++sy) {
      T K[V + 1], M[V + 2], Q[V + 2];
      o.krow(kp + n2 * sz + n * sy, K);
      o.urow(up + n * (2 * sy - 1), M);
      o.urow(up + n2 * (2 * sz - 1) + n * (2 * sy - 1), Q);
#pragma unroll
      for (int v = 0; v < V; ++v)
#pragma unroll
        for (int sx = 0; sx < 2; ++sx) {
          const T kv = K[v + sx];
          const T g = (M[v + 2 * sx] + Q1[v + 2 * sx]) + (Q[v + 1] + Q[v + 2 * sx]);
          ks[v] += kv;
          f[v] += kv * g;
        }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  T uc[V];
  ldv<V>(up, uc);
  const T h = T(1) / T(n);
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const T a = h * (ks[v] * uc[v] * (T(1) / T(3)) - f[v] * (T(1) / T(12)));
    au[v] = (v > 0 || o.gx != 0) ? a : T(0);
  }
}

// A u in the operation order of the LDS-tiled stencil engine's apply (16^3
// solves: the PCG operator those meshes had there)
template <int n, class T>
__device__ __forceinline__ void q1v_chain(const Own<n>& o, const T* u, const T* kap, T (&au)[4]) {
  constexpr int n2 = n * n;
  const T* up = u + o.pos;
  const T* kp = kap + o.pos - n - n2;
  T K[2][2][5], Z[2][5], ks[4], fr[4], uc[4];
#pragma unroll
  for (int dz = 0; dz < 2; ++dz)
#pragma unroll
    for (int dy = 0; dy < 2; ++dy) o.krow(kp + n2 * dz + n * dy, K[dz][dy]);
  {
    T C[5];
#pragma unroll
    for (int c = 0; c < 5; ++c) {
      Z[0][c] = K[0][0][c] + K[1][0][c];
      Z[1][c] = K[0][1][c] + K[1][1][c];
      C[c] = Z[0][c] + Z[1][c];
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) ks[v] = C[v] + C[v + 1];
  }
  {
    T Rm[6], Rp[6];
    o.urow(up - n, Rm);
    ld4(up, uc);
    o.urow(up + n, Rp);
#pragma unroll
    for (int v = 0; v < 4; ++v)
      fr[v] = Z[0][v] * Rm[v] + Z[0][v + 1] * Rm[v + 2] + Z[1][v] * Rp[v] + Z[1][v + 1] * Rp[v + 2];
  }
#pragma unroll
  for (int dz = 0; dz < 2; ++dz) {
    T Q[3][6];
#pragma unroll
    for (int r = 0; r < 3; ++r) o.urow(up + n2 * (2 * dz - 1) + n * (r - 1), Q[r]);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      fr[v] = fma(K[dz][0][v] + K[dz][0][v + 1], Q[0][v + 1], fr[v]);
      fr[v] = fma(K[dz][0][v], Q[0][v], fr[v]);
      fr[v] = fma(K[dz][0][v + 1], Q[0][v + 2], fr[v]);
      fr[v] = fma(K[dz][0][v] + K[dz][1][v], Q[1][v], fr[v]);
      fr[v] = fma(K[dz][0][v + 1] + K[dz][1][v + 1], Q[1][v + 2], fr[v]);
      fr[v] = fma(K[dz][1][v] + K[dz][1][v + 1], Q[2][v + 1], fr[v]);
      fr[v] = fma(K[dz][1][v], Q[2][v], fr[v]);
      fr[v] = fma(K[dz][1][v + 1], Q[2][v + 2], fr[v]);
    }
  }
  const T h12 = (T(1) / T(n)) * (T(1) / T(12));
#pragma unroll
  for (int v = 0; v < 4; ++v) au[v] = (v > 0 || o.gx != 0) ? h12 * fma(ks[v] * uc[v], T(4), -fr[v]) : T(0);
}

// The same one element row at a time: fewer values live (62 registers in fp64),
// more row reads.  For the true residual of fp64 solves, and their operator in
// workgroups of 16 waves.
template <int n, class T>
__device__ __forceinline__ void q1v_rows(const Own<n>& o, const T* u, const T* kap, T (&au)[4]) {
  constexpr int n2 = n * n;
  const T* up = u + o.pos;
  T f[4], ks[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) f[v] = ks[v] = T(0);
#pragma unroll 1
  for (int e = 0; e < 4; ++e) {
    const int dz = e >> 1, dy = e & 1, oz = n2 * (2 * dz - 1), oy = n * (2 * dy - 1);
    T K[5], s[6], q[6];
    o.krow(kap + o.pos - n - n2 + n * dy + n2 * dz, K);
    // s: the neighbours on the element's far columns, edge along y + along z + corner
    o.urow(up + oy, s);
    o.urow(up + oz, q);
#pragma unroll
    for (int c = 0; c < 6; ++c) s[c] += q[c];
    o.urow(up + oy + oz, q);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      f[v] = fma(K[v], (s[v] + q[v]) + q[v + 1], f[v]);
      f[v] = fma(K[v + 1], (s[v + 2] + q[v + 2]) + q[v + 1], f[v]);
      ks[v] += K[v] + K[v + 1];
    }
  }
  T uc[4];
  ld4(up, uc);
  const T h12 = T(1) / T(12 * n);
#pragma unroll
  for (int v = 0; v < 4; ++v) au[v] = (v > 0 || o.gx != 0) ? h12 * fma(ks[v] * uc[v], T(4), -f[v]) : T(0);
}

// r <- r - A u at the thread's nodes in fp64, for the refinement of mixed-precision
// solves, one row of u at a time (few values live beside the fp32 state).  The
// operations, each rounding included, are those of the refinement these meshes
// had before whole solves took its place (16^3: the LDS-tiled engine's, 8^3 and
// 4^3: element by element): the first refinement's r is what is left of a
// cancellation, and how it rounds shows in Y of a pair through the solve that
// follows (one-sample 32^3 / 16^3 pairs: up to 1e-8 of a nearly cancelling Y).
template <int n>
__device__ __forceinline__ void residual4(const Own<n>& o, const double* u, const double* kap, double (&r)[4]) {
  constexpr int n2 = n * n;
  constexpr double h = 1.0 / n;
  const double* up = u + o.pos;
  const double* kp = kap + o.pos - n - n2;
  double f[4], ks[4], K0[5], K1[5], q[6];
  if constexpr (n == 16) {
    {
      double C[5];
#pragma unroll
      for (int dy = 0; dy < 2; ++dy) {
        o.krow(kp + n * dy, K0);
        o.krow(kp + n * dy + n2, K1);
        o.urow(up + n * (2 * dy - 1), q);
#pragma unroll
        for (int c = 0; c < 5; ++c) {
          K0[c] += K1[c];
          C[c] = dy ? C[c] + K0[c] : K0[c];
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          // that engine's threads own two nodes: which of the first two products
          // is the rounded one differs between them
          if (dy == 0)
            f[v] = v & 1 ? fma(K0[v], q[v], K0[v + 1] * q[v + 2]) : fma(K0[v + 1], q[v + 2], K0[v] * q[v]);
          else
            f[v] = fma(K0[v + 1], q[v + 2], fma(K0[v], q[v], f[v]));
        }
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) ks[v] = C[v] + C[v + 1];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int dz = 0; dz < 2; ++dz) {
      const double* z = up + n2 * (2 * dz - 1);
      o.krow(kp + n2 * dz, K0);
      o.krow(kp + n2 * dz + n, K1);
      o.urow(z - n, q);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        f[v] = fma(K0[v] + K0[v + 1], q[v + 1], f[v]);
        f[v] = fma(K0[v], q[v], f[v]);
        f[v] = fma(K0[v + 1], q[v + 2], f[v]);
      }
      __builtin_amdgcn_sched_barrier(0);
      o.urow(z, q);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        f[v] = fma(K0[v] + K1[v], q[v], f[v]);
        f[v] = fma(K0[v + 1] + K1[v + 1], q[v + 2], f[v]);
      }
      __builtin_amdgcn_sched_barrier(0);
      o.urow(z + n, q);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        f[v] = fma(K1[v] + K1[v + 1], q[v + 1], f[v]);
        f[v] = fma(K1[v], q[v], f[v]);
        f[v] = fma(K1[v + 1], q[v + 2], f[v]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    ld4(up, q);
#pragma unroll
    for (int v = 0; v < 4; ++v) r[v] = fma(-(h * (1.0 / 12.0)), fma(ks[v] * q[v], 4.0, -f[v]), r[v]);
  } else {
#pragma unroll
    for (int v = 0; v < 4; ++v) f[v] = ks[v] = 0.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int sz = e >> 1, sy = e & 1, oz = n2 * (2 * sz - 1), oy = n * (2 * sy - 1);
      double m[6], w[6];
      o.krow(kp + n2 * sz + n * sy, K0);
      o.urow(up + oy, m);
      o.urow(up + oz, w);
      o.urow(up + oy + oz, q);
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int sx = 0; sx < 2; ++sx) {
          const double kv = K0[v + sx];
          const double g = (m[v + 2 * sx] + w[v + 2 * sx]) + (q[v + 1] + q[v + 2 * sx]);
          ks[v] += kv;
          f[v] = fma(kv, g, f[v]);
        }
      __builtin_amdgcn_sched_barrier(0);
    }
    ld4(up, q);
#pragma unroll
    for (int v = 0; v < 4; ++v) r[v] = fma(-h, fma(ks[v] * q[v], 1.0 / 3.0, -(f[v] * (1.0 / 12.0))), r[v]);
  }
  if (o.gx == 0) r[0] = 0.0;
}

// D, the Jacobi diagonal, from the kappa sums
template <int n, class T>
__device__ __forceinline__ T diag_of(T ks) {
  const T h = T(1) / T(n);
  return h * ks * (T(1) / T(3));
}

// Jacobi scaling by what a node keeps of its diagonal D: fp32 divides by D (the
// scalar form's rounding), fp64 multiplies by 1 / D
__device__ __forceinline__ float keep_diag(float d) { return d; }
__device__ __forceinline__ double keep_diag(double d) { return 1.0 / d; }
__device__ __forceinline__ float scale_diag(float x, float kept) { return x / kept; }
__device__ __forceinline__ double scale_diag(double x, double kept) { return x * kept; }

// threads of a workgroup: one per vector of the finest mesh
template <int NL>
constexpr int small_threads() { return NL == 4 ? 1024 : (NL == 3 ? 128 : 64); }

// nodes per thread on level L: One (below the finest mesh, where the workgroup
// has a thread per node), else four.  Those levels are chains of short phases, and one
// node's stencil is shorter than four's: 13000 samples of 8^3 816 -> 798 us, 32 pairs
// of 32^3 / 16^3 945 -> 927, 1024 of 64^3 39.1 -> 38.9 ms.  Not in the whole solve of 16^3,
// which spills 38 registers then in place of 27 (one pair with 8^3: 307 against 327 us)
template <int NL, int L, bool One>
constexpr int small_v() {
  constexpr int n = (1 << NL) >> L;
  return One && L > 0 && n * n * (n - 1) <= small_threads<NL>() ? 1 : 4;
}

// LDS of the levels of a V-cycle from 2^NL down: two vectors and kappa each
template <class T, int NL>
struct Levels {
  T* X[NL][2];
  T* K[NL];
  __device__ T* carve(T* p) {
#pragma unroll
    for (int l = 0; l < NL; ++l) {
      const int n = (1 << NL) >> l;
      X[l][0] = p; p += lds_stride(n);
      X[l][1] = p; p += lds_stride(n);
      K[l] = p; p += n * n * n;
    }
    return p;
  }
  __device__ T* x(int l, int c) const { return c ? X[l][1] : X[l][0]; }
};
template <class T>
size_t levels_bytes(int n0) {
  size_t tot = 0;
  for (int n = n0; n >= 2; n /= 2) tot += (size_t)2 * lds_stride(n) + (size_t)n * n * n;
  return tot * sizeof(T);
}

// per level, the thread's right-hand side, iterate and diagonal (keep_diag)
template <class T, int NL>
struct Nodes {
  T b[NL][4], x[NL][4], dg[NL][4];
};

// the diagonals of the levels (kappa in LDS)
template <class T, int NL, int L, bool One = true>
__device__ __forceinline__ void form_diag(const Levels<T, NL>& lv, Nodes<T, NL>& nd) {
  constexpr int n = (1 << NL) >> L;
  if constexpr (n > 2) {
    constexpr int V = small_v<NL, L, One>();
    const Own<n, V> o;
#pragma unroll
    for (int v = 0; v < V; ++v) nd.dg[L][v] = T(1);
    if (o.has) {
      T ks[V];
      ksum4<n>(o, lv.K[L], ks);
#pragma unroll
      for (int v = 0; v < V; ++v) nd.dg[L][v] = keep_diag(diag_of<n>(ks[v]));
    }
    form_diag<T, NL, L + 1, One>(lv, nd);
  }
}

// One V-cycle from level L: nd.b[L] the right-hand side, nd.x[L] the result (and
// an LDS copy in lv.x(L, return value) for L > 0).  Called by every thread.
// Lean: few registers, the diagonals formed where they are used.
template <class T, int NL, int L, bool Lean = false, bool One = true>
__device__ int vcycle_small(const SmallArgs& a, const Levels<T, NL>& lv, Nodes<T, NL>& nd) {
  constexpr int n = (1 << NL) >> L;
  constexpr int V = small_v<NL, L, One>();
  const Own<n, V> o;
  T (&b)[4] = nd.b[L];
  T (&x)[4] = nd.x[L];
  T (&dg)[4] = nd.dg[L];
  const T* kap = lv.K[L];
  int c = 0;
  T xo[V];
  // pre-smoothing from 0
#pragma unroll
  for (int v = 0; v < V; ++v) x[v] = T(0);
  if (o.has) {
    if constexpr (Lean) {
      T ks[V];
      ksum4<n>(o, kap, ks);
#pragma unroll
      for (int v = 0; v < V; ++v) dg[v] = diag_of<n>(ks[v]);
    }
#pragma unroll
    for (int v = 0; v < V; ++v) x[v] = (v > 0 || o.gx != 0) ? scale_diag(T(a.c2[0]) * b[v], dg[v]) : T(0);
    stv<V>(lv.x(L, c) + o.pos, x);
  }
  __syncthreads();
  // one smoothing step: x <- x + c1 (x - xo) + c2 D^-1 (b - A x)
  auto smooth = [&](T c1, T c2, bool use_xo) {
    if (o.has) {
      T au[V];
      if constexpr (Lean) {
        T ks[V];
        q1v_lean<n>(o, lv.x(L, c), kap, au, ks);
#pragma unroll
        for (int v = 0; v < V; ++v) dg[v] = diag_of<n>(ks[v]);
      } else {
        q1v<n>(o, lv.x(L, c), kap, au);
      }
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const T prev = use_xo ? x[v] - xo[v] : x[v];
        const T xn = x[v] + c1 * prev + scale_diag(c2 * (b[v] - au[v]), dg[v]);
        xo[v] = x[v];
        x[v] = (v > 0 || o.gx != 0) ? xn : T(0);
      }
    }
  };
  auto publish = [&] {
    c ^= 1;
    if (o.has) stv<V>(lv.x(L, c) + o.pos, x);
    __syncthreads();
  };
  for (int st = 1; st < a.degree; ++st) {
    smooth(T(a.c1[st]), T(a.c2[st]), st > 1);
    publish();
  }
  // the residual into the other copy
  if (o.has) {
    T t[V];
    if constexpr (Lean) {
      T ks[V];
      q1v_lean<n>(o, lv.x(L, c), kap, t, ks);
    } else {
      q1v<n>(o, lv.x(L, c), kap, t);
    }
#pragma unroll
    for (int v = 0; v < V; ++v) t[v] = b[v] - t[v];
    stv<V>(lv.x(L, c ^ 1) + o.pos, t);
  }
  __syncthreads();
  const T* t = lv.x(L, c ^ 1);
  constexpr int nc = n / 2, n2 = n * n;
  const T* xc;
  if constexpr (nc > 2) {
    // full weighting: coarse node (I, J, K) from fine (2I + dx, 2J + dy, 2K + dz)
    constexpr int VC = small_v<NL, L + 1, One>();
    const Own<nc, VC> oc;
    T (&bc)[4] = nd.b[L + 1];
#pragma unroll
    for (int v = 0; v < VC; ++v) bc[v] = T(0);
    if (oc.has) {
      constexpr int lc = nc == 4 ? 2 : 3;
      const int I0 = oc.pos & (nc - 1), J = (oc.pos >> lc) & (nc - 1), K = oc.pos >> (2 * lc);
      const T* tp = t + 2 * I0 + n * 2 * J + n2 * 2 * K;
#pragma unroll
      for (int dz = -1; dz <= 1; ++dz) {
        T az[VC];
#pragma unroll
        for (int v = 0; v < VC; ++v) az[v] = T(0);
#pragma unroll
        for (int dy = -1; dy <= 1; ++dy) {
          const T* row = tp + n * dy + n2 * dz;
          T f[2 * VC + 1];
          f[0] = row[-1];   // of use where I0 > 0 only
          ldv<VC>(row, f + 1);
          ldv<VC>(row + VC, f + 1 + VC);
#pragma unroll
          for (int v = 0; v < VC; ++v)
            az[v] += (dy == 0 ? T(1) : T(0.5)) * (T(0.5) * (f[2 * v] + f[2 * v + 2]) + f[2 * v + 1]);
        }
#pragma unroll
        for (int v = 0; v < VC; ++v) bc[v] += (dz == 0 ? T(1) : T(0.5)) * az[v];
      }
      if (oc.gx == 0) bc[0] = T(0);
    }
    const int cc = vcycle_small<T, NL, L + 1, Lean, One>(a, lv, nd);
    xc = lv.x(L + 1, cc);
  } else {
    // 2^3: one unknown, A_11 = (h / 3) sum of the 8 kappa, h = 1/2
    if (threadIdx.x == 0) {
      const T* k = lv.K[L + 1];
      T acc = T(0);
#pragma unroll
      for (int dz = -1; dz <= 1; ++dz) {
        T az = T(0);
#pragma unroll
        for (int dy = -1; dy <= 1; ++dy) {
          const T* row = t + 2 + n * (2 + dy) + n2 * (2 + dz);
          az += (dy == 0 ? T(1) : T(0.5)) * (T(0.5) * (row[-1] + row[1]) + row[0]);
        }
        acc += (dz == 0 ? T(1) : T(0.5)) * az;
      }
      const T ks = ((k[0] + k[1]) + (k[2] + k[3])) + ((k[4] + k[5]) + (k[6] + k[7]));
      lv.X[L + 1][0][7] = acc / (T(0.5) * ks * (T(1) / T(3)));
    }
    __syncthreads();
    xc = lv.X[L + 1][0];
  }
  // the coarse-grid correction: along x, then y, then z
  if (o.has) {
    constexpr int lf = n == 16 ? 4 : (n == 8 ? 3 : 2), c2n = nc * nc;
    const int j = (o.pos >> lf) & (n - 1), k = o.pos >> (2 * lf);
    T pl[2][V];
#pragma unroll
    for (int z = 0; z < 2; ++z) {
      T rw[2][V];
#pragma unroll
      for (int y = 0; y < 2; ++y) {
        if constexpr (V == 4) {
          const T* row = xc + 2 * o.gx + nc * ((j + y) >> 1) + c2n * ((k + z) >> 1);
          const T p0 = row[0], p1 = row[1], p2 = row[2];
          rw[y][0] = p0;
          rw[y][1] = T(0.5) * (p0 + p1);
          rw[y][2] = p1;
          rw[y][3] = T(0.5) * (p1 + p2);
        } else {
          const T* row = xc + (o.gx >> 1) + nc * ((j + y) >> 1) + c2n * ((k + z) >> 1);
          const T p0 = row[0], p1 = row[1];
          rw[y][0] = (o.gx & 1) ? T(0.5) * (p0 + p1) : p0;
        }
      }
#pragma unroll
      for (int v = 0; v < V; ++v) pl[z][v] = (j & 1) ? T(0.5) * (rw[0][v] + rw[1][v]) : rw[0][v];
    }
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const T e = (k & 1) ? T(0.5) * (pl[0][v] + pl[1][v]) : pl[0][v];
      x[v] += (v > 0 || o.gx != 0) ? e : T(0);
    }
  }
  publish();
  for (int st = 0; st < a.degree; ++st) {
    smooth(st == 0 ? T(0) : T(a.c1[st]), T(a.c2[st]), st > 0);
    if (L > 0 || st + 1 < a.degree) publish();
  }
  return c;
}

// Lean: two workgroups of 16^3 per CU (64 registers, 60 KB of LDS each)
template <class T, int NL, bool Lean>
__global__ void __launch_bounds__(small_threads<NL>(), Lean ? 8 : 1) k_vsmall(SmallArgs a, const T* __restrict__ bglob,
                                                                T* __restrict__ xglob,
                                                                const int* __restrict__ active) {
  constexpr int n = 1 << NL, TPB = small_threads<NL>();
  const int smp = blockIdx.x;
  if (active && !active[smp]) return;
  extern __shared__ __align__(32) unsigned char smem[];
  Levels<T, NL> lv;
  T* end = lv.carve(reinterpret_cast<T*>(smem));
  const int tid = (int)threadIdx.x;
  const Own<n> o;
  Nodes<T, NL> nd;
#pragma unroll
  for (int v = 0; v < 4; ++v) nd.b[0][v] = T(0);
  if (o.has) {
    ld4(bglob + (size_t)smp * a.gstride + o.pos, nd.b[0]);
    if (o.gx == 0) nd.b[0][0] = T(0);
  }
  // zero everything (boundary positions must read as 0), then load kappa
  for (T* q = reinterpret_cast<T*>(smem) + 4 * tid; q < end; q += 4 * TPB) {
    const T z[4] = {T(0), T(0), T(0), T(0)};
    st4(q, z);
  }
  __syncthreads();
#pragma unroll
  for (int l = 0; l < NL; ++l) {
    const int ne = ((1 << NL) >> l) * ((1 << NL) >> l) * ((1 << NL) >> l);
    const T* kg = reinterpret_cast<const T*>(a.kap[l]) + (size_t)smp * ne;
    for (int q = 4 * tid; q < ne; q += 4 * TPB) {
      T k[4];
      ld4(kg + q, k);
      st4(lv.K[l] + q, k);
    }
  }
  __syncthreads();
  if constexpr (!Lean) form_diag<T, NL, 0>(lv, nd);
  vcycle_small<T, NL, 0, Lean>(a, lv, nd);
  if (o.has) st4(xglob + (size_t)smp * a.gstride + o.pos, nd.x[0]);
}

// --------------------------------------------- whole solve in one workgroup
// One workgroup per sample runs a sample's whole solve: the fp64 iterative
// refinement around the fp32 GMG-PCG (mixed precision), or the fp64 PCG with
// its confirmations by the true residual; the same methods as the level-by-level
// kernels.  Sums are taken over the workgroup in a fixed order, so a sample's
// result does not depend on its batch.
struct SolveSmallArgs {
  SmallArgs v;
  double rtol2, inner_tol2, bconst;
  int max_iter, max_outer;
};

template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_move(double x) {
  const long long v = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(v & 0xffffffffll), CTRL, ROWS, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(v >> 32), CTRL, ROWS, 0xF, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Sum of v over the workgroup, the same value in every thread: a tree over each
// wave (all lanes active), then the waves in order.  Two partial arrays take
// turns, so one barrier per sum is enough.
template <int TPB>
struct AllSum {
  double (*ws)[16];
  int turn = 0;
  __device__ double operator()(double v) {
    v += dpp_move<0x111, 0xF>(v);
    v += dpp_move<0x112, 0xF>(v);
    v += dpp_move<0x114, 0xF>(v);
    v += dpp_move<0x118, 0xF>(v);
    v += dpp_move<0x142, 0xA>(v);
    v += dpp_move<0x143, 0xC>(v);   // lane 63 holds the wave's sum
    double* w = ws[turn];
    turn ^= 1;
    if ((threadIdx.x & 63) == 63) w[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int q = 0; q < TPB / 64; ++q) t += w[q];
    return t;
  }
};

template <class T>
__device__ __forceinline__ double dot4(const T (&a)[4], const T (&b)[4]) {
  double s = 0.0;
#pragma unroll
  for (int v = 0; v < 4; ++v) s += (double)a[v] * (double)b[v];
  return s;
}

// coarse kappa of every level from level 0, the mean of the 8 children in the order of k_coarsen
template <class T, int NL>
__device__ __forceinline__ void coarsen_lds(const Levels<T, NL>& lv) {
#pragma unroll
  for (int l = 1; l < NL; ++l) {
    const int nc = (1 << NL) >> l, nf = 2 * nc, f2 = nf * nf, nce = nc * nc * nc, lc = lg2(nc);
    for (int E = threadIdx.x; E < nce; E += blockDim.x) {
      const int EX = E & (nc - 1), EY = (E >> lc) & (nc - 1), EZ = E >> (2 * lc);
      const T* f = lv.K[l - 1] + 2 * EX + nf * 2 * EY + f2 * 2 * EZ;
      const T sv = ((f[0] + f[1]) + (f[nf] + f[nf + 1])) + ((f[f2] + f[f2 + 1]) + (f[f2 + nf] + f[f2 + nf + 1]));
      lv.K[l][E] = sv * T(0.125);
    }
    __syncthreads();
  }
}

// Preconditioned CG on A d = r (nd.b[0]) in the precision T, from d = 0: to
// ||r||^2 <= tol2 (bb given) or max_iter iterations (counted in total).  GMG:
// one V-cycle; else Jacobi.  pbuf: the LDS vector the operator reads.
template <class T, int NL, bool GMG, class Sum>
__device__ void pcg_small(const SmallArgs& a, const Levels<T, NL>& lv, Nodes<T, NL>& nd, T* pbuf, T (&d)[4],
                          double tol2, int max_iter, int& total, Sum& sum) {
  constexpr int n = 1 << NL;
  const Own<n> o;
  T (&r)[4] = nd.b[0];
  T (&z)[4] = nd.x[0];
  T p[4];
  double rz = 0.0;
  bool first = true;
  while (total < max_iter) {
    if (GMG) {
      vcycle_small<T, NL, 0, false, NL != 4>(a, lv, nd);
    } else {
#pragma unroll
      for (int v = 0; v < 4; ++v) z[v] = scale_diag(r[v], nd.dg[0][v]);
    }
    const double rzn = sum(dot4(r, z));
    const T beta = first ? T(0) : (T)(rzn / rz);
    rz = rzn;
#pragma unroll
    for (int v = 0; v < 4; ++v) p[v] = first ? z[v] : fma(beta, p[v], z[v]);
    first = false;
    if (o.has) st4(pbuf + o.pos, p);
    __syncthreads();
    T q[4] = {T(0), T(0), T(0), T(0)};
    if (o.has) {
      if constexpr (sizeof(T) == 8 && NL == 4) q1v_rows<n>(o, pbuf, lv.K[0], q);
      else if constexpr (NL == 4) q1v_chain<n>(o, pbuf, lv.K[0], q);
      else q1v<n>(o, pbuf, lv.K[0], q);
    }
    const T alpha = (T)(rz / sum(dot4(p, q)));
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      d[v] = fma(alpha, p[v], d[v]);
      r[v] = fma(-alpha, q[v], r[v]);
    }
    const double rr = sum(dot4(r, r));
    ++total;
    if (rr <= tol2 || !isfinite(rr)) break;   // a NaN or Inf residual ends the sample's solve
  }
}

// a sample's grid vector: u at the thread's nodes (0 on row 0), 0 outside planes 1 .. n-1
template <int NL>
__device__ __forceinline__ void store_u(const Own<(1 << NL)>& o, double* ug, const double (&u)[4]) {
  constexpr int n = 1 << NL, n2 = n * n, TPB = small_threads<NL>();
  const int tid = (int)threadIdx.x;
  const double z[4] = {0.0, 0.0, 0.0, 0.0};
  if (tid < Own<n>::NV) st4(ug + o.pos, u);
  for (int q = 4 * tid; q < n2; q += 4 * TPB) st4(ug + q, z);
  for (int q = n2 * n + 4 * tid; q < lds_stride(n); q += 4 * TPB) st4(ug + q, z);
}

// Mixed precision, GMG.  In registers the fp32 Krylov vectors; the refinement stages the iterate in fp64 over the two finest
// vectors of the V-cycle, which hold nothing then.
template <int NL>
__global__ void __launch_bounds__(small_threads<NL>(), NL == 2 ? 1 : 4) k_solve_small(SolveSmallArgs a, const double* __restrict__ kap,
                                                     const double* __restrict__ bvec, double* __restrict__ uglob,
                                                     int* __restrict__ active, int* __restrict__ iters,
                                                     double* __restrict__ rr_out, const int* __restrict__ rows) {
  constexpr int n = 1 << NL, n2 = n * n, ne = n2 * n, TPB = small_threads<NL>();
  constexpr int S = lds_stride(n);
  const int smp = rows ? rows[blockIdx.x] : (int)blockIdx.x, tid = (int)threadIdx.x;
  extern __shared__ __align__(32) unsigned char smem[];
  __shared__ double ws[2][16];
  Levels<float, NL> lv;
  float* end = lv.carve(reinterpret_cast<float*>(smem));
  AllSum<TPB> sum{ws};
  const Own<n> o;
  auto zero = [&](float* from, float* to) {
    const float z[4] = {0.f, 0.f, 0.f, 0.f};
    for (float* q = from + 4 * tid; q < to; q += 4 * TPB) st4(q, z);
  };
  zero(reinterpret_cast<float*>(smem), end);
  __syncthreads();
  const double* kg = kap + (size_t)smp * ne;
  for (int q = 4 * tid; q < ne; q += 4 * TPB) {
    double k[4];
    ld4(kg + q, k);
    const float f[4] = {(float)k[0], (float)k[1], (float)k[2], (float)k[3]};
    st4(lv.K[0] + q, f);
  }
  __syncthreads();
  coarsen_lds<float, NL>(lv);
  Nodes<float, NL> nd;
  form_diag<float, NL, 0, NL != 4>(lv, nd);
  const double* bg = bvec ? bvec + (size_t)smp * a.v.gstride : nullptr;
  // the right-hand side at the thread's nodes, 0 on the boundary
  auto rhs = [&](double (&b)[4]) {
#pragma unroll
    for (int v = 0; v < 4; ++v) b[v] = 0.0;
    if (o.has) {
      if (bg) {
        ld4(bg + o.pos, b);
      } else {
#pragma unroll
        for (int v = 0; v < 4; ++v) b[v] = a.bconst;
      }
      if (o.gx == 0) b[0] = 0.0;
    }
  };
  double r64[4];
  rhs(r64);
  const double bb = sum(dot4(r64, r64));
  // the iterate stays in the output between refinements (registers are what
  // bounds the workgroups per CU)
  double* ug = uglob + (size_t)smp * a.v.gstride;
  {
    const double z4[4] = {0.0, 0.0, 0.0, 0.0};
    store_u<NL>(o, ug, z4);
  }
  int total = 0;
  bool done = false;
  double rr_last = bb;
  double* U = reinterpret_cast<double*>(lv.X[0][0]);   // both copies of the finest vector: S doubles
  for (int outer = 0; outer < a.max_outer && total < a.max_iter && !done; ++outer) {
    // inner fp32 GMG-PCG on A d = fp32(r), from d = 0, to the inner tolerance
#pragma unroll
    for (int v = 0; v < 4; ++v) nd.b[0][v] = (float)r64[v];
    const double tol2 = a.inner_tol2 * sum(dot4(nd.b[0], nd.b[0]));
    float d[4] = {0.f, 0.f, 0.f, 0.f};
    pcg_small<float, NL, true>(a.v, lv, nd, lv.X[0][0], d, tol2, a.max_iter, total, sum);
    // fp64 refinement: u += d, r = b - A u (fp64 kappa from global memory)
    zero(lv.X[0][0], lv.X[0][0] + 2 * S);
    __syncthreads();
    if (o.has) {
      double u[4];
      ld4(ug + o.pos, u);
#pragma unroll
      for (int v = 0; v < 4; ++v) u[v] += (double)d[v];
      st4(ug + o.pos, u);
      st4(U + o.pos, u);
    }
    __syncthreads();
    rhs(r64);
    if (o.has) residual4<n>(o, U, kg, r64);
    rr_last = sum(dot4(r64, r64));
    done = rr_last <= a.rtol2 * bb || !isfinite(rr_last);
    zero(lv.X[0][0], lv.X[0][0] + 2 * S);   // (every thread is past the operator: the sum's barrier)
    __syncthreads();
  }
  if (tid == 0) {
    active[smp] = done ? 0 : 1;
    iters[smp] = total;
    if (rr_out) rr_out[smp] = rr_last;
  }
}

// fp64: GMG-PCG (4^3, 8^3) or Jacobi-PCG (up to 16^3) to rtol on the recurrence,
// confirmed by the true residual, at most max_outer times.  Kappa in LDS where
// it fits beside the vectors, else (16^3) read from global memory.
template <int NL, bool GMG>
__global__ void __launch_bounds__(small_threads<NL>()) k_solve_small64(SolveSmallArgs a, const double* __restrict__ kap,
                                                     const double* __restrict__ bvec, double* __restrict__ uglob,
                                                     int* __restrict__ active, int* __restrict__ iters,
                                                     double* __restrict__ rr_out) {
  static_assert(!GMG || NL <= 3, "the fp64 levels of 16^3 exceed the LDS of a workgroup");
  constexpr int n = 1 << NL, n2 = n * n, ne = n2 * n, TPB = small_threads<NL>();
  const int smp = blockIdx.x, tid = (int)threadIdx.x;
  extern __shared__ __align__(32) unsigned char smem[];
  __shared__ double ws[2][16];
  AllSum<TPB> sum{ws};
  const Own<n> o;
  const double* kg = kap + (size_t)smp * ne;
  Levels<double, NL> lv;
  double* end;
  if constexpr (GMG) {
    end = lv.carve(reinterpret_cast<double*>(smem));
  } else {
    lv.X[0][0] = reinterpret_cast<double*>(smem);
    end = lv.X[0][0] + lds_stride(n);
    lv.K[0] = NL < 4 ? end : const_cast<double*>(kg);
    if (NL < 4) end += ne;
  }
  const double z4[4] = {0.0, 0.0, 0.0, 0.0};
  for (double* q = reinterpret_cast<double*>(smem) + 4 * tid; q < end; q += 4 * TPB) st4(q, z4);
  __syncthreads();
  if (GMG || NL < 4) {
    for (int q = 4 * tid; q < ne; q += 4 * TPB) {
      double k[4];
      ld4(kg + q, k);
      st4(lv.K[0] + q, k);
    }
    __syncthreads();
  }
  Nodes<double, NL> nd;
  if constexpr (GMG) {
    coarsen_lds<double, NL>(lv);
    form_diag<double, NL, 0>(lv, nd);
  } else {
#pragma unroll
    for (int v = 0; v < 4; ++v) nd.dg[0][v] = 0.0;
    if (o.has) {
      double ks[4];
      ksum4<n>(o, lv.K[0], ks);
#pragma unroll
      for (int v = 0; v < 4; ++v) nd.dg[0][v] = keep_diag((1.0 / n) * ks[v] * (1.0 / 3.0));
    }
  }
  const double* bg = bvec ? bvec + (size_t)smp * a.v.gstride : nullptr;
  double (&r)[4] = nd.b[0];
  auto rhs = [&] {
#pragma unroll
    for (int v = 0; v < 4; ++v) r[v] = 0.0;
    if (o.has) {
      if (bg) {
        ld4(bg + o.pos, r);
      } else {
#pragma unroll
        for (int v = 0; v < 4; ++v) r[v] = a.bconst;
      }
      if (o.gx == 0) r[0] = 0.0;
    }
  };
  double u[4] = {0.0, 0.0, 0.0, 0.0};
  rhs();
  const double bb = sum(dot4(r, r));
  const double tol2 = a.rtol2 * bb;
  int total = 0;
  bool done = false;
  double rr_last = bb;
  for (int outer = 0; outer < a.max_outer && total < a.max_iter && !done; ++outer) {
    pcg_small<double, NL, GMG>(a.v, lv, nd, lv.X[0][0], u, tol2, a.max_iter, total, sum);
    // the true residual; a sample above its tolerance goes on from it
    __syncthreads();
    if (o.has) st4(lv.X[0][0] + o.pos, u);
    __syncthreads();
    rhs();
    if (o.has) {
      double au[4];
      q1v_rows<n>(o, lv.X[0][0], lv.K[0], au);
#pragma unroll
      for (int v = 0; v < 4; ++v) r[v] -= au[v];
    }
    rr_last = sum(dot4(r, r));
    done = rr_last <= tol2 || !isfinite(rr_last);
  }
  double* ug = uglob + (size_t)smp * a.v.gstride;
  store_u<NL>(o, ug, u);
  if (tid == 0) {
    active[smp] = done ? 0 : 1;
    iters[smp] = total;
    if (rr_out) rr_out[smp] = rr_last;
  }
}

SmallArgs small_args(int n0, int degree, const double* c1, const double* c2) {
  SmallArgs a{};
  a.degree = degree;
  for (int s = 0; s < degree; ++s) {
    a.c1[s] = c1[s];
    a.c2[s] = c2[s];
  }
  a.gstride = grid_stride(n0);
  return a;
}

}  // namespace

template <class T>
hipError_t launch_vsmall(int n0, int B, int degree, const double* c1, const double* c2, const T* const* kap_levels,
                         const T* b, T* x, const int* active, hipStream_t st) {
  if (degree < 1 || degree > 16) return hipErrorInvalidValue;
  SmallArgs a = small_args(n0, degree, c1, c2);
  int l = 0;
  for (int n = n0; n >= 2 && l < kMaxLv; n /= 2, ++l) a.kap[l] = kap_levels[l];
  const size_t lds = levels_bytes<T>(n0);
  switch (n0) {
    case 4: k_vsmall<T, 2, false><<<dim3(B), dim3(small_threads<2>()), lds, st>>>(a, b, x, active); break;
    case 8: k_vsmall<T, 3, false><<<dim3(B), dim3(small_threads<3>()), lds, st>>>(a, b, x, active); break;
    case 16:
      if constexpr (sizeof(T) == 4) {
        // more workgroups than half the CUs: two per CU, so that the launches of
        // other lanes, which such a batch has, run beside this one (1024 samples
        // of 64^3 over four lanes: 39.6 -> 39.1 ms, though alone a launch of 256
        // takes 18.6 us in place of 16.8); else all the registers the compiler
        // wants (32 pairs of 32^3: 1.10 ms against 1.13)
        if (B > 128) k_vsmall<T, 4, true><<<dim3(B), dim3(small_threads<4>()), lds, st>>>(a, b, x, active);
        else k_vsmall<T, 4, false><<<dim3(B), dim3(small_threads<4>()), lds, st>>>(a, b, x, active);
        break;
      }
      return hipErrorInvalidValue;   // above the LDS of a workgroup in fp64
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_solve_small(int n, int B, int degree, const double* c1, const double* c2, const double* kap,
                              const double* bvec, double bconst, double* u, int* active, int* iters, double rtol,
                              double inner_rtol, int max_iter, int max_outer, hipStream_t st, double* rr_out,
                              const int* rows) {
  if (degree < 1 || degree > 16 || B <= 0) return hipErrorInvalidValue;
  SolveSmallArgs a{};
  a.v = small_args(n, degree, c1, c2);
  a.rtol2 = rtol * rtol;
  a.inner_tol2 = inner_rtol * inner_rtol;
  a.bconst = bconst;
  a.max_iter = max_iter;
  a.max_outer = max_outer;
  const size_t lds = levels_bytes<float>(n);
#define MLMC_SMALL(NL) \
  k_solve_small<NL><<<dim3(B), dim3(small_threads<NL>()), lds, st>>>(a, kap, bvec, u, active, iters, rr_out, rows)
  if (n == 4) MLMC_SMALL(2);
  else if (n == 8) MLMC_SMALL(3);
  else if (n == 16) MLMC_SMALL(4);
  else return hipErrorInvalidValue;
#undef MLMC_SMALL
  return hipGetLastError();
}

hipError_t launch_solve_small64(int n, int B, bool gmg, int degree, const double* c1, const double* c2,
                                const double* kap, const double* bvec, double bconst, double* u, int* active,
                                int* iters, double rtol, int max_iter, int max_outer, hipStream_t st,
                                double* rr_out) {
  if (degree < 1 || degree > 16 || B <= 0) return hipErrorInvalidValue;
  SolveSmallArgs a{};
  a.v = small_args(n, degree, c1, c2);
  a.rtol2 = rtol * rtol;
  a.bconst = bconst;
  a.max_iter = max_iter;
  a.max_outer = max_outer;
  const size_t lds = gmg ? levels_bytes<double>(n)
                         : ((size_t)lds_stride(n) + (n < 16 ? (size_t)n * n * n : 0)) * sizeof(double);
#define MLMC_SMALL(NL, GMG) \
  k_solve_small64<NL, GMG><<<dim3(B), dim3(small_threads<NL>()), lds, st>>>(a, kap, bvec, u, active, iters, rr_out)
  if (n == 4) { if (gmg) MLMC_SMALL(2, true); else MLMC_SMALL(2, false); }
  else if (n == 8) { if (gmg) MLMC_SMALL(3, true); else MLMC_SMALL(3, false); }
  else if (n == 16 && !gmg) MLMC_SMALL(4, false);
  else return hipErrorInvalidValue;
#undef MLMC_SMALL
  return hipGetLastError();
}

template hipError_t launch_vsmall<float>(int, int, int, const double*, const double*, const float* const*,
                                         const float*, float*, const int*, hipStream_t);
template hipError_t launch_vsmall<double>(int, int, int, const double*, const double*, const double* const*,
                                          const double*, double*, const int*, hipStream_t);

}  // namespace mlmc
