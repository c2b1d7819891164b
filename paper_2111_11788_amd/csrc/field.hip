// K2: log-normal KLE coefficient on fp64 MFMA.
//
// kappa_b(e) = exp( sum_m Xi[b][m] Phi[e][m] ),  Xi[b][m] = xi_b,m sqrt(lambda_m),
// Phi[e][m] = phi_i(x_e) phi_j(y_e) phi_k(z_e) for mode m = (i, j, k) evaluated
// at the element centroid (the KLE of the log-field in Sec. 5.2).  The sum is
// a dense [B x M] . [M x n^3] contraction; Phi is never stored in HBM -- each
// workgroup builds its [elements x modes] tile in LDS from the separable 1D
// tables tab[x][q] = phi_q((x + 1/2)/n) and feeds it to
// v_mfma_f64_16x16x4_f64 with the xi tile.  exp (and the optional fp32 copy)
// is applied in the epilogue, so g never round-trips through memory.
//
// Operand layout of v_mfma_f64_16x16x4_f64 (64 lanes, checked on gfx950 with a
// probe of encoded operands): lane l supplies A[l % 16][l / 16] and
// B[l / 16][l % 16]; accumulator element r of lane l holds D[l / 16 + 4 r][l % 16].
// Rows = samples, columns = elements, K = modes.  An optional row map sends
// row r to batch slot rowmap[r] (xi read from and kappa written to that slot).
// The default evaluation for 64^3 to 256^3 meshes factorises the same sum
// over the three axes and keeps only the final per-plane contraction, a
// [n x K1] . [K1 x n] product, on the same instruction (k_field_plane_mfma);
// below 64^3 both sums of the row-wise form run on it (k_field_rows).
#include <algorithm>

#include "common.hpp"
#include "kernels.hpp"

namespace mlmc {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int kKc = 16;   // modes per LDS stage (4 MFMA k-steps)

// BS samples x BE elements per workgroup of 4 waves; each wave owns a
// 16-sample x 64-element strip (four 16x16 accumulator tiles).
template <int BS>
__global__ void __launch_bounds__(256) k_field(int n, int M, int64_t count,
                                               const double* __restrict__ xi,
                                               const double* __restrict__ sqrtlam,
                                               const int* __restrict__ triples,
                                               const double* __restrict__ tab, int K1,
                                               double* __restrict__ kappa, float* __restrict__ kappa32,
                                               const int* __restrict__ rowmap) {
  constexpr int WS = BS / 16;          // waves along samples
  constexpr int WE = 4 / WS;           // waves along elements
  constexpr int BE = 64 * WE;          // elements per workgroup
  __shared__ double xs[BS][kKc + 1];
  __shared__ double ph[BE][kKc + 1];

  // The tile's BE elements are consecutive and n is a power of two, so the
  // tile covers TR = max(1, BE / n) whole or partial x-rows; the y-z factor
  // phi_j(y) phi_k(z) of a mode is shared by every element of a row.
  // TR = min(BE / n, n^2) <= 32 over all powers of two n (n = 8: 32 rows)
  __shared__ double wyz[32][kKc];
  const int ne = n * n * n;                  // <= 2^27 for the meshes in use
  const int e0 = (int)blockIdx.x * BE;
  const int64_t s0 = (int64_t)blockIdx.y * BS;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int ws = wave % WS, we = wave / WS;
  const int lg = 31 - __clz(n);
  const int TR = BE > n ? (BE / n < n * n ? BE / n : n * n) : 1;
  const int row0 = e0 >> lg;                 // first x-row (ey + n ez) of the tile

  d4 acc[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) acc[t] = d4{0.0, 0.0, 0.0, 0.0};

  for (int m0 = 0; m0 < M; m0 += kKc) {
    // stage Xi (scaled by sqrt(lambda)), the y-z factors of the tile rows,
    // then the Phi tile = phi_i(x) * y-z factor
    for (int q = tid; q < BS * kKc; q += 256) {
      const int r = q / kKc, c = q % kKc;
      const int64_t s = s0 + r;
      const int m = m0 + c;
      const int64_t row = (s < count && rowmap) ? rowmap[s] : s;
      xs[r][c] = (s < count && m < M) ? xi[row * M + m] * sqrtlam[m] : 0.0;
    }
    for (int q = tid; q < TR * kKc; q += 256) {
      const int tr = q / kKc, c = q % kKc;
      const int m = m0 + c;
      const int xr = row0 + tr;              // x-row index ey + n ez
      double v = 0.0;
      if (m < M && xr < n * n) {
        const int ey = xr & (n - 1), ez = xr >> lg;
        v = tab[ey * K1 + triples[3 * m + 1]] * tab[ez * K1 + triples[3 * m + 2]];
      }
      wyz[tr][c] = v;
    }
    __syncthreads();
    for (int q = tid; q < BE * kKc; q += 256) {
      const int r = q / kKc, c = q % kKc;
      const int e = e0 + r;
      const int m = m0 + c;
      double v = 0.0;
      if (e < ne && m < M) v = tab[(e & (n - 1)) * K1 + triples[3 * m]] * wyz[(e >> lg) - row0][c];
      ph[r][c] = v;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < kKc; kk += 4) {
      const double a = xs[16 * ws + (lane & 15)][kk + (lane >> 4)];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const double b = ph[64 * we + 16 * t + (lane & 15)][kk + (lane >> 4)];
        acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc[t], 0, 0, 0);
      }
    }
    __syncthreads();
  }

#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int64_t e = (int64_t)e0 + 64 * we + 16 * t + (lane & 15);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t s = s0 + 16 * ws + (lane >> 4) + 4 * r;
      if (s < count && e < ne) {
        const int64_t row = rowmap ? rowmap[s] : s;
        const double k = exp(acc[t][r]);
        kappa[row * (int64_t)ne + e] = k;
        if (kappa32) kappa32[row * (int64_t)ne + e] = (float)k;
      }
    }
  }
}

// ---------------------------------------------------------------- bf16 MFMA
// The same contraction with bf16 operands and fp32 accumulation on
// v_mfma_f32_16x16x32_bf16 (gfx950): lane l supplies A[l % 16][8 (l / 16) + v]
// and B[8 (l / 16) + v][l % 16], v = 0..7, and accumulator element r holds
// D[4 (l / 16) + r][l % 16] (checked on gfx950 with a probe of one-hot
// operands).  Xi sqrt(lambda) and Phi are formed in fp64 and rounded to bf16
// (unit roundoff 2^-8), so |g - g_exact| <= (2 u + u^2 + M 2^-24) sum_m
// |Xi_m Phi_m|; kappa = exp(g) is evaluated in fp64 from the fp32 sum.  This
// changes the coefficient field itself (a model perturbation of up to ~1% in
// kappa for |g| of a few units), not just the route to it.
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));
constexpr int kKb = 32;        // modes per stage (one MFMA k-step)
constexpr int kKbPad = 40;     // LDS row pitch in bf16 (16-byte aligned rows)

template <int BS>
__global__ void __launch_bounds__(256) k_field_bf16(int n, int M, int64_t count,
                                                    const double* __restrict__ xi,
                                                    const double* __restrict__ sqrtlam,
                                                    const int* __restrict__ triples,
                                                    const double* __restrict__ tab, int K1,
                                                    double* __restrict__ kappa, float* __restrict__ kappa32,
                                                    const int* __restrict__ rowmap) {
  constexpr int WS = BS / 16;
  constexpr int WE = 4 / WS;
  constexpr int BE = 64 * WE;
  __shared__ __align__(16) __bf16 xs[BS][kKbPad];
  __shared__ __align__(16) __bf16 ph[BE][kKbPad];
  __shared__ double wyz[32][kKb];
  const int ne = n * n * n;
  const int e0 = (int)blockIdx.x * BE;
  const int64_t s0 = (int64_t)blockIdx.y * BS;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int ws = wave % WS, we = wave / WS;
  const int lg = 31 - __clz(n);
  const int TR = BE > n ? (BE / n < n * n ? BE / n : n * n) : 1;
  const int row0 = e0 >> lg;

  f4 acc[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) acc[t] = f4{0.f, 0.f, 0.f, 0.f};

  for (int m0 = 0; m0 < M; m0 += kKb) {
    for (int q = tid; q < BS * kKb; q += 256) {
      const int r = q / kKb, c = q % kKb;
      const int64_t s = s0 + r;
      const int m = m0 + c;
      const int64_t row = (s < count && rowmap) ? rowmap[s] : s;
      xs[r][c] = (__bf16)(float)((s < count && m < M) ? xi[row * M + m] * sqrtlam[m] : 0.0);
    }
    for (int q = tid; q < TR * kKb; q += 256) {
      const int tr = q / kKb, c = q % kKb;
      const int m = m0 + c;
      const int xr = row0 + tr;
      double v = 0.0;
      if (m < M && xr < n * n) {
        const int ey = xr & (n - 1), ez = xr >> lg;
        v = tab[ey * K1 + triples[3 * m + 1]] * tab[ez * K1 + triples[3 * m + 2]];
      }
      wyz[tr][c] = v;
    }
    __syncthreads();
    for (int q = tid; q < BE * kKb; q += 256) {
      const int r = q / kKb, c = q % kKb;
      const int e = e0 + r;
      const int m = m0 + c;
      double v = 0.0;
      if (e < ne && m < M) v = tab[(e & (n - 1)) * K1 + triples[3 * m]] * wyz[(e >> lg) - row0][c];
      ph[r][c] = (__bf16)(float)v;
    }
    __syncthreads();
    const bf8 a = *reinterpret_cast<const bf8*>(&xs[16 * ws + (lane & 15)][8 * (lane >> 4)]);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const bf8 b = *reinterpret_cast<const bf8*>(&ph[64 * we + 16 * t + (lane & 15)][8 * (lane >> 4)]);
      acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[t], 0, 0, 0);
    }
    __syncthreads();
  }

#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int64_t e = (int64_t)e0 + 64 * we + 16 * t + (lane & 15);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t s = s0 + 16 * ws + 4 * (lane >> 4) + r;
      if (s < count && e < ne) {
        const int64_t row = rowmap ? rowmap[s] : s;
        const double k = exp((double)acc[t][r]);
        kappa[row * (int64_t)ne + e] = k;
        if (kappa32) kappa32[row * (int64_t)ne + e] = (float)k;
      }
    }
  }
}

// ------------------------------------------------------------ separable form
// The modes are products phi_i(x) phi_j(y) phi_k(z), so on one x-row of
// elements (fixed ey, ez)
//   g[s][ex] = sum_a phi_a(x_ex) H[s][a],
//   H[s][a]  = sum over the modes m with x-factor a of xi[s][m] sqrt(lambda_m) phi_j(y) phi_k(z):
// M products per sample and row, then K1 (distinct x-factors, <= 16 for 512
// modes at correlation length 0.1) per element, against M per element for the
// dense contraction.  A workgroup takes S samples and R consecutive x-rows:
// it stages the samples' xi in x-grouped mode order into LDS once, then per
// row forms w (the row's y-z factors, sqrt(lambda) included), H and the row's
// elements.  Every sum runs in a fixed order, so a sample's field does not
// depend on its batch.
constexpr int kSepRows = 16;   // x-rows per workgroup

__global__ void __launch_bounds__(256) k_field_sep(int n, int M, int K1, int S, int64_t count,
                                                   const double* __restrict__ xi,
                                                   const double* __restrict__ sqrtlam,
                                                   const int* __restrict__ triples,
                                                   const int* __restrict__ xperm, const int* __restrict__ xoff,
                                                   const double* __restrict__ tab, double* __restrict__ kappa,
                                                   float* __restrict__ kappa32, const int* __restrict__ rowmap) {
  extern __shared__ double fsm[];
  double* X = fsm;            // [S][M]: xi of the block, x-grouped order
  double* w = X + S * M;      // [M]
  double* H = w + M;          // [S][K1]
  double* T = H + S * K1;     // [K1][n]: phi_a(x_ex), transposed so a row's lanes read consecutive words
  const int lg = 31 - __clz(n);
  const int nrows = n * n;
  const int row0 = (int)blockIdx.x * kSepRows;
  const int64_t s0 = (int64_t)blockIdx.y * S;
  const int tid = (int)threadIdx.x;
  for (int q = tid; q < S * M; q += 256) {
    const int s = q / M, p = q - (q / M) * M;
    double v = 0.0;
    if (s0 + s < count) {
      const int64_t r = rowmap ? rowmap[s0 + s] : s0 + s;
      v = xi[r * M + xperm[p]];
    }
    X[q] = v;
  }
  for (int q = tid; q < K1 * n; q += 256) {
    const int a = q >> lg, ex = q & (n - 1);
    T[q] = tab[ex * K1 + a];
  }
  const int64_t ne = (int64_t)n * n * n;
  for (int row = row0; row < row0 + kSepRows && row < nrows; ++row) {
    const int ey = row & (n - 1), ez = row >> lg;
    __syncthreads();   // X staged; the previous row's H no longer read
    for (int p = tid; p < M; p += 256) {
      const int m = xperm[p];
      w[p] = sqrtlam[m] * (tab[ey * K1 + triples[3 * m + 1]] * tab[ez * K1 + triples[3 * m + 2]]);
    }
    __syncthreads();
    for (int q = tid; q < S * K1; q += 256) {
      const int s = q / K1, a = q - (q / K1) * K1;
      const double* x = X + s * M;
      double hv = 0.0;
      for (int p = xoff[a]; p < xoff[a + 1]; ++p) hv += x[p] * w[p];
      H[q] = hv;
    }
    __syncthreads();
    for (int q = tid; q < S * n; q += 256) {
      const int s = q >> lg, ex = q & (n - 1);
      if (s0 + s >= count) continue;
      const double* hs = H + s * K1;
      double g = 0.0;
      for (int a = 0; a < K1; ++a) g += hs[a] * T[a * n + ex];
      const int64_t r = rowmap ? rowmap[s0 + s] : s0 + s;
      const double k = exp(g);
      const int64_t e = (int64_t)row * n + ex;
      kappa[r * ne + e] = k;
      if (kappa32) kappa32[r * ne + e] = (float)k;
    }
  }
}

// ------------------------------------------ separable form, one z-plane per workgroup
// The same sum factorised over all three axes: on the element plane ez of
// sample s,
//   A[a][b]   = sum over the modes m = (a, b, c) of sqrt(lambda_m) xi[s][m] phi_c(z_ez)
//   B[ey][a]  = sum_b A[a][b] phi_b(y_ey)
//   g[ey][ex] = sum_a B[ey][a] phi_a(x_ex)
// so an element costs K1 multiply-adds and the exponential, and the plane's
// M + n K1^2 other products are shared by its n^2 elements.  The element
// contraction g = B Phi_x (n x K1 by K1 x n, K1 padded to a multiple of 4
// with zeros) runs on v_mfma_f64_16x16x4f64: wave w owns the 16-column tiles
// w, w + 4, ... (CTW = n / 64 of them) and keeps their Phi_x operands in
// registers (lane l: phi_{4 ks + l/16} of column 16 t + l % 16); B is formed
// RB rows at a time into LDS (odd row pitch), and per 16-row tile the wave
// loads its A operands once and runs KS k-steps per column tile; the
// accumulator's rows (l/16 + 4 r) and column (l % 16) go through exp to
// kappa.  Every sum runs in a fixed order (A over the modes in x-grouped
// order, B over b, g in the MFMA's k-steps), so a sample's field does not
// depend on its batch.  (The same form with the element sums on the VALU
// measured 706 / 902 us against 574 / 612 us here for 64^3 x 1024 / 256^3 x 16.)
template <int KS, int CTW>
__global__ void __launch_bounds__(256) k_field_plane_mfma(int n, int M, int K1, int RB, int64_t count,
                                                          const double* __restrict__ xi,
                                                          const double* __restrict__ sqrtlam,
                                                          const int* __restrict__ triples,
                                                          const int* __restrict__ xperm,
                                                          const int* __restrict__ xoff,
                                                          const double* __restrict__ tab,
                                                          double* __restrict__ kappa, float* __restrict__ kappa32,
                                                          const int* __restrict__ rowmap) {
  constexpr int KP = 4 * KS, KPS = KP + 1;
  extern __shared__ double fsm[];
  double* wv = fsm;                                   // [M] sqrt(lambda) xi phi_c(z), x-grouped order
  double* A = wv + M;                                 // [K1][K1]
  double* Bm = A + K1 * K1;                           // [RB][KPS]
  int* bv = reinterpret_cast<int*>(Bm + RB * KPS);    // [M] y-factor of each mode
  const int ez = (int)blockIdx.x;
  const int64_t s = (int64_t)blockIdx.y;
  if (s >= count) return;
  const int64_t r = rowmap ? rowmap[s] : s;
  const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int p = tid; p < M; p += 256) {
    const int m = xperm[p];
    const int b = triples[3 * m + 1], c = triples[3 * m + 2];
    wv[p] = sqrtlam[m] * xi[r * M + m] * tab[ez * K1 + c];
    bv[p] = b;
  }
  double ph[CTW][KS];
#pragma unroll
  for (int t = 0; t < CTW; ++t)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int a = 4 * ks + (lane >> 4), ex = 16 * (wave + 4 * t) + (lane & 15);
      ph[t][ks] = a < K1 ? tab[ex * K1 + a] : 0.0;
    }
  __syncthreads();
  for (int q = tid; q < K1 * K1; q += 256) {
    const int a = q / K1, b = q - a * K1;
    double acc = 0.0;
    for (int p = xoff[a]; p < xoff[a + 1]; ++p)
      if (bv[p] == b) acc += wv[p];
    A[q] = acc;
  }
  const int64_t ne = (int64_t)n * n * n;
  double* kr = kappa + r * ne + (int64_t)ez * n * n;
  float* kr32 = kappa32 ? kappa32 + r * ne + (int64_t)ez * n * n : nullptr;
  for (int y0 = 0; y0 < n; y0 += RB) {
    __syncthreads();   // A formed; the previous rows' B no longer read
    for (int q = tid; q < RB * KP; q += 256) {
      const int yr = q / KP, a = q - yr * KP;
      double acc = 0.0;
      if (a < K1) {
        const double* ty = tab + (y0 + yr) * K1;
        const double* Aa = A + a * K1;
        for (int b = 0; b < K1; ++b) acc = fma(Aa[b], ty[b], acc);
      }
      Bm[yr * KPS + a] = acc;
    }
    __syncthreads();
    for (int rt = 0; rt < RB / 16; ++rt) {
      double av[KS];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) av[ks] = Bm[(16 * rt + (lane & 15)) * KPS + 4 * ks + (lane >> 4)];
#pragma unroll
      for (int t = 0; t < CTW; ++t) {
        d4 acc = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av[ks], ph[t][ks], acc, 0, 0, 0);
        const int ex = 16 * (wave + 4 * t) + (lane & 15);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int64_t e = (int64_t)(y0 + 16 * rt + (lane >> 4) + 4 * q) * n + ex;
          const double k = exp(acc[q]);
          kr[e] = k;
          if (kr32) kr32[e] = (float)k;
        }
      }
    }
  }
}

template <int KS, int CTW>
void launch_field_plane_mfma(int n, int M, int K1, int64_t count, const double* xi, const double* sqrtlam,
                             const int* triples, const int* xperm, const int* xoff, const double* tab,
                             double* kappa, float* kappa32, const int* rowmap, hipStream_t st) {
  constexpr int KPS = 4 * KS + 1;
  // B rows per pass: a power of two of 16 rows or more within 2048 values
  int RB = 16;
  while (RB * 2 <= n && RB * 2 * KPS <= 2048) RB *= 2;
  const size_t lds = ((size_t)M + (size_t)K1 * K1 + (size_t)RB * KPS) * sizeof(double) + (size_t)M * sizeof(int);
  dim3 grid((unsigned)n, (unsigned)count);
  k_field_plane_mfma<KS, CTW><<<grid, dim3(256), lds, st>>>(n, M, K1, RB, count, xi, sqrtlam, triples, xperm, xoff,
                                                            tab, kappa, kappa32, rowmap);
}

// ------------------------------ the separable form on meshes below 64^3, on MFMA
// The sums of k_field_sep, each in its order, on v_mfma_f64_16x16x4f64, which
// adds its four products one after another as fused multiply-adds (so padding
// with zeros changes nothing): the field has the bits of k_field_sep.  That
// matters: a change in the last bit of kappa shows in Y = Q_l - Q_{l-1} of a
// mixed-precision pair by up to 1e-8 of a nearly cancelling one.
// A workgroup takes 16 samples and 16 element rows (fixed y, z).
//   H[s][row][a] = sum over the modes m of x-factor a of xi[s][m] w[m][row]: a
//     16 x 16 product of the samples' xi (staged in LDS) and the rows' factors
//     w = sqrt(lambda_m) (phi_b(y) phi_c(z)), which each lane forms as it needs
//     them; a wave takes every fourth a.
//   g[row][ex] = sum_a H[row][a] phi_a(x_ex), SP samples at a time through LDS
//     (over the xi).  Rows of fewer than 16 elements are packed PACK = 16 / n to
//     a tile row: its operand is the PACK rows of H one after another, and the
//     Phi_x operand is block diagonal (zero where a column belongs to another
//     row), so a tile holds 256 elements on every mesh.
// Bound: the 12 bytes written per element and the fp64 exponential (25 million
// elements, 32^3 x 777, M = 256: 91 us a call, 3.3 TB/s, against 731 us with
// k_field_sep, whose sums read both operands from LDS; 13001 samples of 8^3, M =
// 128: 207 -> 42 us; one of 16^3: 48 -> 6.4 us).  Chunks of 256 modes: 40 KB of LDS,
// four workgroups per CU; 128 modes and five per CU, with spills, measured 111 us on
// the first of these against 107.  Stores past the caches: 107 -> 91 us there, and no
// reader of kappa measured slower (1131 pairs of 16^3 / 8^3: 982 -> 966 us a call).
// modes of a chunk, samples of a pass, and the doubles that xi and H share
constexpr int kRowsChunk = 256;
__host__ __device__ constexpr int field_rows_chunk(int M) { return M < kRowsChunk ? M : kRowsChunk; }
__host__ __device__ constexpr int field_rows_sp(int KS) { return KS == 2 ? 16 : 8; }
__host__ __device__ constexpr int field_rows_shared(int KS, int pack, int M) {
  const int x = 16 * (field_rows_chunk(M) | 1), h = field_rows_sp(KS) * 16 / pack * (4 * KS * pack + 1);
  return x > h ? x : h;
}
template <int KS, int PACK, int CT>
__global__ void __launch_bounds__(256) k_field_rows(int n, int M, int K1, int64_t count,
                                                    const double* __restrict__ xi,
                                                    const double* __restrict__ sqrtlam,
                                                    const int* __restrict__ triples,
                                                    const int* __restrict__ xperm, const int* __restrict__ xoff,
                                                    const double* __restrict__ tab, double* __restrict__ kappa,
                                                    float* __restrict__ kappa32, const int* __restrict__ rowmap) {
  constexpr int KP = 4 * KS, KT = KP * PACK, PITCH = KT + 1, SP = field_rows_sp(KS);
  extern __shared__ double fsm[];
  const int lg = 31 - __clz(n), CH = field_rows_chunk(M), XP = CH | 1, lgp = CH > 1 ? 32 - __clz(CH - 1) : 0;
  double* tz = fsm;                                   // [n][K1] the table
  double* sl = tz + n * K1;                           // [CH] sqrt(lambda) of the chunk's modes
  double* X = sl + CH;                                // [16][XP] xi of the chunk's modes; then
  double* Hb = X;                                     // [SP * 16 / PACK][PITCH] H
  int* bc = reinterpret_cast<int*>(X + field_rows_shared(KS, PACK, M));   // [CH] their y- and z-factors
  const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6, lc = lane & 15, lk = lane >> 4;
  const int rows = n * n / 16;                        // row tiles of a sample
  const int64_t s0 = (int64_t)(blockIdx.x / rows) * 16;
  const int row0 = (int)(blockIdx.x % rows) * 16;
  for (int q = tid; q < n * K1; q += 256) tz[q] = tab[q];
  // block-diagonal Phi_x: lane l supplies row k = 4 ks + l / 16 of column l % 16
  double ph[CT][KS * PACK];
#pragma unroll
  for (int t = 0; t < CT; ++t)
#pragma unroll
    for (int ks = 0; ks < KS * PACK; ++ks) {
      const int k = 4 * ks + lk, col = 16 * t + lc;
      const int pr = k / KP, a = k - pr * KP;          // packed row and x-factor of this k
      ph[t][ks] = (PACK == 1 || (col >> lg) == pr) && a < K1 ? tab[(col & (n - 1)) * K1 + a] : 0.0;
    }
  d4 h[KS];   // H of the x-factors wave, wave + 4, ..: samples lk + 4 q, row lc
#pragma unroll
  for (int i = 0; i < KS; ++i) h[i] = d4{0.0, 0.0, 0.0, 0.0};
  for (int c0 = 0; c0 < M; c0 += CH) {   // a chunk of modes, in x-grouped order
    if (c0) __syncthreads();             // the chunk before is no longer read
    const int p = tid & ((1 << lgp) - 1);   // the threads stage 2^lgp modes of 256 >> lgp samples at a time
    if (p < CH && c0 + p < M) {
      const int m = xperm[c0 + p];
      if (tid >> lgp == 0) {
        sl[p] = sqrtlam[m];
        bc[p] = triples[3 * m + 1] | (triples[3 * m + 2] << 16);
      }
      for (int s = tid >> lgp; s < 16; s += 256 >> lgp) {
        double v = 0.0;
        if (s0 + s < count) {
          const int64_t r = rowmap ? rowmap[s0 + s] : s0 + s;
          v = xi[r * M + m];
        }
        X[s * XP + p] = v;
      }
    }
    __syncthreads();
    const double* ty = tz + ((row0 + lc) & (n - 1)) * K1;
    const double* tt = tz + ((row0 + lc) >> lg) * K1;
    const double* x = X + lc * XP;
#pragma unroll
    for (int i = 0; i < KS; ++i) {
      const int a = wave + 4 * i;
      if (a < K1) {
        const int from = xoff[a] - c0, to = xoff[a + 1] - c0;
        const int p1 = to < CH ? to : CH;
        for (int p0 = from > 0 ? from : 0; p0 < p1; p0 += 4) {
          const bool in = p0 + lk < p1;
          const int p = in ? p0 + lk : p0;
          const double xv = x[p], w = sl[p] * (ty[bc[p] & 0xffff] * tt[bc[p] >> 16]);
          h[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(in ? xv : 0.0, in ? w : 0.0, h[i], 0, 0, 0);
        }
      }
    }
  }
  const int64_t ne = (int64_t)1 << (3 * lg);
#pragma unroll
  for (int f = 0; f < 16 / SP; ++f) {   // samples f SP ..
    if (s0 + f * SP >= count) break;    // uniform over the workgroup
    __syncthreads();                    // the xi or the H before are no longer read
#pragma unroll
    for (int i = 0; i < KS; ++i)
#pragma unroll
      for (int q = 0; q < SP / 4; ++q) {
        const int rho = (lk + 4 * q) * 16 + lc;
        Hb[(rho / PACK) * PITCH + (rho % PACK) * KP + wave + 4 * i] = h[i][f * (SP / 4) + q];
      }
    __syncthreads();
    for (int t = wave; t < SP / PACK && s0 + f * SP + t * PACK < count; t += 4) {   // a tile: PACK samples
      double av[KS * PACK];
#pragma unroll
      for (int ks = 0; ks < KS * PACK; ++ks) av[ks] = Hb[(16 * t + lc) * PITCH + 4 * ks + lk];
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        d4 acc = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int ks = 0; ks < KS * PACK; ++ks)
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av[ks], ph[c][ks], acc, 0, 0, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int rho = (16 * t + lk + 4 * q) * PACK + (PACK > 1 ? lc >> lg : 0);
          const int64_t s = s0 + f * SP + (rho >> 4);
          if (s < count) {
            const int64_t r = rowmap ? rowmap[s] : s;
            const double k = exp(acc[q]);
            const int64_t at = r * ne + (row0 + (rho & 15)) * n + ((16 * c + lc) & (n - 1));
            __builtin_nontemporal_store(k, kappa + at);
            if (kappa32) __builtin_nontemporal_store((float)k, kappa32 + at);
          }
        }
      }
    }
  }
}

// LDS of k_field_rows (at most 49 KiB); 0 where the mesh has another form or
// k_field_sep, whose sums these are, would not run
size_t field_rows_lds(int n, int M, int K1) {
  if (n < 4 || n > 32 || K1 > 32 || 2 * (int64_t)M + (int64_t)K1 * (n + 1) > 65536 / (int64_t)sizeof(double)) return 0;
  const int KS = K1 <= 8 ? 2 : (K1 <= 16 ? 4 : 8), pack = n < 16 ? 16 / n : 1;
  const int ch = field_rows_chunk(M);
  return ((size_t)n * K1 + (size_t)ch + (size_t)field_rows_shared(KS, pack, M)) * sizeof(double) +
         (size_t)ch * sizeof(int);
}

template <int KS>
void launch_field_rows_n(int n, int M, int K1, size_t lds, int64_t count, const double* xi, const double* sqrtlam,
                         const int* triples, const int* xperm, const int* xoff, const double* tab, double* kappa,
                         float* kappa32, const int* rowmap, hipStream_t st) {
  const dim3 grid((unsigned)((count + 15) / 16 * (n * n / 16)));
#define MLMC_ROWS(PACK, CT)                                                                                        \
  k_field_rows<KS, PACK, CT><<<grid, dim3(256), lds, st>>>(n, M, K1, count, xi, sqrtlam, triples, xperm, xoff, tab, \
                                                           kappa, kappa32, rowmap)
  if (n == 4) MLMC_ROWS(4, 1);
  else if (n == 8) MLMC_ROWS(2, 1);
  else if (n == 16) MLMC_ROWS(1, 1);
  else MLMC_ROWS(1, 2);
#undef MLMC_ROWS
}

template <int KS>
void launch_field_plane_mfma_n(int n, int M, int K1, int64_t count, const double* xi, const double* sqrtlam,
                               const int* triples, const int* xperm, const int* xoff, const double* tab,
                               double* kappa, float* kappa32, const int* rowmap, hipStream_t st) {
  if (n == 64) launch_field_plane_mfma<KS, 1>(n, M, K1, count, xi, sqrtlam, triples, xperm, xoff, tab, kappa, kappa32, rowmap, st);
  else if (n == 128) launch_field_plane_mfma<KS, 2>(n, M, K1, count, xi, sqrtlam, triples, xperm, xoff, tab, kappa, kappa32, rowmap, st);
  else launch_field_plane_mfma<KS, 4>(n, M, K1, count, xi, sqrtlam, triples, xperm, xoff, tab, kappa, kappa32, rowmap, st);
}

}  // namespace

hipError_t launch_field(int n, int M, int64_t count, const double* xi, const double* sqrtlam,
                        const int* triples, const double* tab, int K1, double* kappa,
                        float* kappa32, hipStream_t st, const int* rowmap, bool bf16, const int* xperm,
                        const int* xoff) {
  if (count <= 0) return hipSuccess;
  const int64_t ne = (int64_t)n * n * n;
  if (!bf16 && xperm && xoff && (n == 64 || n == 128 || n == 256) && K1 <= 32 && M <= 2048 && count <= 65535) {
    // one workgroup per sample and element plane (at most 48 KiB of LDS)
    if (K1 <= 8) launch_field_plane_mfma_n<2>(n, M, K1, count, xi, sqrtlam, triples, xperm, xoff, tab, kappa, kappa32, rowmap, st);
    else if (K1 <= 16) launch_field_plane_mfma_n<4>(n, M, K1, count, xi, sqrtlam, triples, xperm, xoff, tab, kappa, kappa32, rowmap, st);
    else launch_field_plane_mfma_n<8>(n, M, K1, count, xi, sqrtlam, triples, xperm, xoff, tab, kappa, kappa32, rowmap, st);
    return hipGetLastError();
  }
  // 4^3 to 32^3: 16 samples and 16 element rows per workgroup
  const size_t rlds = !bf16 && xperm && xoff ? field_rows_lds(n, M, K1) : 0;
  if (rlds && (count + 15) / 16 * (n * n / 16) <= 0x7fffffff) {
    if (K1 <= 8) launch_field_rows_n<2>(n, M, K1, rlds, count, xi, sqrtlam, triples, xperm, xoff, tab, kappa, kappa32, rowmap, st);
    else if (K1 <= 16) launch_field_rows_n<4>(n, M, K1, rlds, count, xi, sqrtlam, triples, xperm, xoff, tab, kappa, kappa32, rowmap, st);
    else launch_field_rows_n<8>(n, M, K1, rlds, count, xi, sqrtlam, triples, xperm, xoff, tab, kappa, kappa32, rowmap, st);
    return hipGetLastError();
  }
  if (!bf16 && xperm && xoff) {
    // samples per workgroup: as many as fit 64 KiB of LDS with the row's
    // factors and the transposed x-table, at most 32 (more workgroups per CU
    // measured faster than larger blocks)
    const int64_t room = (65536 / (int64_t)sizeof(double) - M - (int64_t)K1 * n) / (M + K1);
    int S = (int)std::min<int64_t>({32, room, count});
    const size_t lds = ((size_t)S * M + M + (size_t)S * K1 + (size_t)K1 * n) * sizeof(double);
    if (S >= 1 && (count + S - 1) / S <= 65535) {   // grid y within the launch limit
      dim3 grid((unsigned)(((int64_t)n * n + kSepRows - 1) / kSepRows), (unsigned)((count + S - 1) / S));
      k_field_sep<<<grid, dim3(256), lds, st>>>(n, M, K1, S, count, xi, sqrtlam, triples, xperm, xoff, tab, kappa,
                                                 kappa32, rowmap);
      return hipGetLastError();
    }
    // the block's coefficients and sums exceed the LDS of a workgroup: the dense form
  }
  if (bf16) {
    if (count >= 48) {
      dim3 grid((unsigned)((ne + 63) / 64), (unsigned)((count + 63) / 64));
      k_field_bf16<64><<<grid, dim3(256), 0, st>>>(n, M, count, xi, sqrtlam, triples, tab, K1, kappa, kappa32,
                                                   rowmap);
    } else {
      dim3 grid((unsigned)((ne + 255) / 256), (unsigned)((count + 15) / 16));
      k_field_bf16<16><<<grid, dim3(256), 0, st>>>(n, M, count, xi, sqrtlam, triples, tab, K1, kappa, kappa32,
                                                   rowmap);
    }
    return hipGetLastError();
  }
  if (count >= 48) {
    dim3 grid((unsigned)((ne + 63) / 64), (unsigned)((count + 63) / 64));
    k_field<64><<<grid, dim3(256), 0, st>>>(n, M, count, xi, sqrtlam, triples, tab, K1, kappa, kappa32, rowmap);
  } else {
    dim3 grid((unsigned)((ne + 255) / 256), (unsigned)((count + 15) / 16));
    k_field<16><<<grid, dim3(256), 0, st>>>(n, M, count, xi, sqrtlam, triples, tab, K1, kappa, kappa32, rowmap);
  }
  return hipGetLastError();
}

}  // namespace mlmc
