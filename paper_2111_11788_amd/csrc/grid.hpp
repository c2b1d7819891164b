// Device-side helpers for the grid-layout kernels: vector types and the
// thread geometry of the z-marching stencil engine and of the streaming
// kernels.  Host code uses the same geometry to size partial-sum buffers.
#pragma once

#include "common.hpp"

namespace mlmc {

// Values per thread along x in the z-marching stencil kernels: one 16-byte
// vector of the row segment (4 floats or 2 doubles).
template <class T>
struct ZV { static constexpr int V = 16 / (int)sizeof(T); };

// Geometry of a z-marching launch on an n^3 grid for B samples.
// A thread owns V consecutive nodes i0 .. i0+V-1 of row j and marches over a
// chunk of planes; a workgroup holds `rows` rows of one sample and one plane
// chunk.  Workgroups of a sample are numbered rb + row_blocks * zb.  Partial
// sums are taken per row block and unit of `zu` planes (planes 1 + u zu ..
// (u + 1) zu; a chunk is a whole number of units) and added up in an order that
// does not depend on how the planes are split, and so not on the batch: up to
// 64^3 a workgroup stores every unit's sum, numbered rb + row_blocks * u; above
// (fold) a chunk is 2^k units, aligned, and its workgroup adds them by pairs, the
// pairs by pairs and so on, stores one sum, numbered as the workgroup, and the
// reduction goes on in the same tree over the chunks.
struct ZGeom {
  int n = 0;
  int G = 0;            // vector groups per row (n / V)
  int rows = 0;         // rows per workgroup
  int row_blocks = 0;   // workgroups per plane chunk
  int zc = 1;           // plane chunks
  int zlen = 0;         // planes per chunk
  int zu = 1;           // planes per unit
  bool fold = false;    // one partial sum per chunk
  int threads = 256;    // threads per workgroup
  __host__ __device__ uint32_t blocks() const { return (uint32_t)row_blocks * zc; }
  __host__ __device__ uint32_t parts() const { return fold ? blocks() : (uint32_t)row_blocks * ((n - 1 + zu - 1) / zu); }
  // what a reduction is given: the partial sums, and with fold log2 of the chunks in bits 24..
  uint32_t parts_code() const {
    uint32_t lz = 0;
    while (fold && (1 << lz) < zc) ++lz;
    return parts() | lz << 24;
  }
};

// waves of a launch from which the samples' planes are no longer split
constexpr long kFillWaves = 8192;
// the same for meshes up to 64^3, whose planes split down to a unit: four waves
// per SIMD (2048 and 8192 measured 2.93 and 2.63 ms against 2.42 on a burst of
// 400 served requests, 39.4 and 40.2 ms against 39.4 on 1024 samples of 64^3)
constexpr long kSplitWaves = 4096;

// The planes of a launch of `waves` waves in one chunk, split over workgroups
// while the launch does not fill the chip.
inline void zsplit(ZGeom& g, long waves) {
  const int n = g.n;
  if (n <= 64) {
    // down to one unit: a workgroup's planes are a serial chain of about a
    // microsecond each, and the two planes a chunk stages beyond its own are
    // cheap while the chip is not full (32 pairs of 32^3 / 16^3, mixed: 1.92 ->
    // 1.31 ms with chunks of 4 planes in place of 16; a 64^3 level of three
    // 128^3 samples likewise).  A launch of one to one and a half times the
    // chip's waves is split once: half of its second round would be idle (the
    // 14-row tiles of 256 samples of 64^3: 268 -> 231 us; solves of 300 and 370
    // samples of 64^3 7 to 9% faster, of 1200 of 32^3 10%, fp64 of 140 of 64^3 8% and
    // of 600 of 32^3 2%, but of 760 2% slower)
    g.zu = n == 64 ? 8 : 4;
    g.zlen = (n - 1 + g.zu - 1) / g.zu * g.zu;
    g.zc = 1;
    while ((waves * g.zc < kSplitWaves || (g.zc == 1 && waves > kSplitWaves && 2 * waves <= 3 * kSplitWaves)) &&
           g.zlen % (2 * g.zu) == 0) {
      g.zlen /= 2;
      g.zc = (n - 1 + g.zlen - 1) / g.zlen;
    }
    return;
  }
  // larger meshes: one partial sum per chunk, chunks of at least 8 planes (n / zc,
  // a power of two: n and zc are)
  int zc = 1;
  while (waves * zc < kFillWaves && (n - 1) / (zc * 2) >= 8) zc *= 2;
  g.zc = zc;
  g.zlen = (n - 1 + zc - 1) / zc;
  g.zu = 8;
  g.fold = true;
}

template <class T>
inline ZGeom zgeom(int n, int B) {
  ZGeom g;
  constexpr int V = ZV<T>::V;
  g.n = n;
  g.G = n / V;
  if (g.G < 1) {   // a row narrower than one vector: no z-march geometry (callers check G)
    g.rows = 0;
    g.row_blocks = 0;
    g.zlen = 0;
    return g;
  }
  const int rowthreads = (n - 1) * g.G;
  g.threads = rowthreads >= 256 ? 256 : ((rowthreads + 63) / 64) * 64;
  g.rows = g.threads / g.G;
  if (g.rows < 1) g.rows = 1;
  g.row_blocks = (n - 1 + g.rows - 1) / g.rows;
  zsplit(g, (long)B * g.row_blocks * (g.threads / 64));
  return g;
}

// The geometry of zgeom for a row of 128 vectors (256^3 in fp64): 512 threads,
// four rows.  256 threads would hold two, and stage four.
template <class T>
inline ZGeom zgeom_long(int n, int B) {
  ZGeom g = zgeom<T>(n, B);
  if (g.G != 128) return g;
  g.threads = 512;
  g.rows = 512 / g.G;
  g.row_blocks = (n - 1 + g.rows - 1) / g.rows;
  zsplit(g, (long)B * g.row_blocks * (g.threads / 64));
  return g;
}

// The geometry of zgeom with `rows` rows per workgroup instead of the most
// that fit (rows >= 1, same thread count).
template <class T>
inline ZGeom zgeom_rows(int n, int B, int rows) {
  ZGeom g = zgeom<T>(n, B);
  if (g.G < 1 || rows < 1) return g;
  g.rows = rows;
  g.row_blocks = (n - 1 + rows - 1) / rows;
  zsplit(g, (long)B * g.row_blocks * (g.threads / 64));
  return g;
}

// Tiles of the corrected smoothing step with its operand formed on the fly,
// which stages two rows more than it computes: with rows of 16 lanes (G = 16)
// a 16-row tile stages 18 rows with 16 rows of threads, and the wave that
// takes the extra rows (each formed from the kappa ring and the coarse
// correction) runs a second pass per plane while the others wait at the
// plane's barrier.  14-row tiles stage 16 rows in one pass at about the same
// total work (5 tiles of 63 rows instead of 4): 9.7 -> 9.4 ms per 64^3 x 1024
// step.
template <class T>
inline ZGeom zgeom_tall(int n, int B) {
  const ZGeom g = zgeom<T>(n, B);
  // only where the shorter tiles add at most a quarter more tiles (63 rows:
  // 5 instead of 4; not 31 rows: 3 instead of 2)
  const bool fits = 4 * ((n - 1 + 13) / 14) <= 5 * ((n - 1 + 15) / 16);
  return g.G == 16 && g.threads == 256 && g.rows == 16 && fits ? zgeom_rows<T>(n, B, 14) : g;
}

// The planes of an LDS-engine launch of B samples split further while it is
// below kSplitWaves.  zsplit stops at chunks that keep a sample's partial sums
// few (8 planes at 64^3, 4 below, 16 at 128^3); a launch without sums, and above 64^3
// one whose sums fit `cap` per sample (~0: no sums), goes down to 8 planes above
// 64^3, 4 at 64^3 and 2 below: what a chunk stages beyond its own planes is cheap
// while the chip is not full.  A solve of three 128^3 samples: 2.70 -> 2.36 ms with the
// split above 64^3 (4 planes in place of 8: 2.42), 2.15 ms with the levels below as
// well; 32 pairs of 32^3 / 16^3, mixed: 1.05 -> 1.00 ms.
inline ZGeom zfine(ZGeom g, int B, uint32_t cap = ~0u) {
  if (g.G < 1 || (g.n <= 64 && cap != ~0u)) return g;   // up to 64^3 the sums are per unit of zu planes
  const long waves = (long)B * g.row_blocks * (g.threads / 64);
  const int least = g.n > 64 ? 8 : (g.n == 64 ? 4 : 2);
  while (waves * g.zc < kSplitWaves && g.zlen % (2 * least) == 0 && (cap == ~0u || 2 * g.parts() <= cap)) {
    g.zlen /= 2;
    g.zc = (g.n - 1 + g.zlen - 1) / g.zlen;
  }
  return g;
}

// Streaming kernels cover the flat range [n^2, n^3) of every sample (planes
// 1..n-1, boundary positions included: they hold zero in every vector) in
// 16-byte vectors; `chunks` workgroups per sample.
struct SGeom {
  int n = 0;
  uint32_t vecs = 0;    // 16-byte vectors per sample in the range
  uint32_t chunks = 0;  // workgroups per sample
};

template <class T>
inline SGeom sgeom(int n) {
  SGeom g;
  g.n = n;
  const size_t elems = (size_t)(n - 1) * n * n;
  g.vecs = (uint32_t)(elems * sizeof(T) / 16);
  uint32_t c = (uint32_t)((g.vecs + 256 * 8 - 1) / (256 * 8));   // ~8 vectors per thread
  if (c > 64) c = 64;
  if (c < 1) c = 1;
  g.chunks = c;
  return g;
}

// Largest number of per-sample partial sums any kernel writes for a mesh.
inline uint32_t max_parts(int n, int B) {
  uint32_t m = sgeom<float>(n).chunks;
  if (sgeom<double>(n).chunks > m) m = sgeom<double>(n).chunks;
  if (n >= 4 && zgeom<float>(n, B).parts() > m) m = zgeom<float>(n, B).parts();
  if (zgeom<double>(n, B).parts() > m) m = zgeom<double>(n, B).parts();
  if (n >= 4 && zgeom_tall<float>(n, B).parts() > m) m = zgeom_tall<float>(n, B).parts();
  if (zgeom_tall<double>(n, B).parts() > m) m = zgeom_tall<double>(n, B).parts();
  return m;
}

}  // namespace mlmc
