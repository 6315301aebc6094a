// Catalog reductions and mass assignment (Sec. 2.1 FKP field, Sec. 2.3 TSC painting with
// interlacing).  Mesh coordinates are computed in FP64 with explicitly rounded operations
// (u = (x - o) * (N / L); no fused multiply-add) so that node indices and fractions match
// any other IEEE implementation of the same formula bit for bit.
#include <algorithm>

#include "../../include/pkm.h"
#include "kernels.hpp"
#include "device_common.hpp"

namespace pkm {

namespace {

constexpr int SUM_THREADS = 256;

// The sums of both catalogs in one launch each (blockIdx.y, and blockIdx.x of the second kernel, is the
// catalog): on small meshes launches are a good part of an estimate.
struct SumArgs {
  const double *w[2], *nbar[2];
  int64_t n[2];
};
__global__ void __launch_bounds__(SUM_THREADS) k_catalog_sums(SumArgs args, double* __restrict__ partial) {
  const double* __restrict__ w = args.w[blockIdx.y];
  const double* __restrict__ nbar = args.nbar[blockIdx.y];
  const int64_t n = args.n[blockIdx.y];
  partial += 3 * (size_t)gridDim.x * blockIdx.y;
  __shared__ double s0[SUM_THREADS], s1[SUM_THREADS], s2[SUM_THREADS];
  double a0 = 0.0, a1 = 0.0, a2 = 0.0;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const double wi = w ? w[i] : 1.0;
    const double w2 = wi * wi;
    a0 += w2;
    a1 += w2 * (nbar ? nbar[i] : 1.0);
    a2 = fmax(a2, fabs(wi));
  }
  s0[threadIdx.x] = a0;
  s1[threadIdx.x] = a1;
  s2[threadIdx.x] = a2;
  __syncthreads();
  for (int h = SUM_THREADS / 2; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) {
      s0[threadIdx.x] += s0[threadIdx.x + h];
      s1[threadIdx.x] += s1[threadIdx.x + h];
      s2[threadIdx.x] = fmax(s2[threadIdx.x], s2[threadIdx.x + h]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    partial[3 * blockIdx.x] = s0[0];
    partial[3 * blockIdx.x + 1] = s1[0];
    partial[3 * blockIdx.x + 2] = s2[0];
  }
}

__global__ void __launch_bounds__(SUM_THREADS) k_sum_partials2(const double* __restrict__ partial, int nblk,
                                                               double* __restrict__ out2, double* __restrict__ wmax) {
  partial += 3 * (size_t)nblk * blockIdx.x;
  out2 += 2 * blockIdx.x;
  wmax += blockIdx.x;
  __shared__ double s0[SUM_THREADS], s1[SUM_THREADS], s2[SUM_THREADS];
  double a0 = 0.0, a1 = 0.0, a2 = 0.0;
  for (int b = threadIdx.x; b < nblk; b += SUM_THREADS) {
    a0 += partial[3 * b];
    a1 += partial[3 * b + 1];
    a2 = fmax(a2, partial[3 * b + 2]);
  }
  s0[threadIdx.x] = a0;
  s1[threadIdx.x] = a1;
  s2[threadIdx.x] = a2;
  __syncthreads();
  for (int h = SUM_THREADS / 2; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) {
      s0[threadIdx.x] += s0[threadIdx.x + h];
      s1[threadIdx.x] += s1[threadIdx.x + h];
      s2[threadIdx.x] = fmax(s2[threadIdx.x], s2[threadIdx.x + h]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out2[0] = s0[0];
    out2[1] = s1[0];
    *wmax = s2[0];
  }
}

template <typename T>
__global__ void k_fill(T* __restrict__ p0, T* __restrict__ p1, size_t n, T v) {
  T* p = blockIdx.y ? p1 : p0;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}

__device__ __forceinline__ int wrap(long long c, int n) {
  long long r = c % n;
  return (int)(r < 0 ? r + n : r);
}

// floor(u) wrapped into the mesh.  Nodes inside the mesh, nearly all of them, need neither the 64-bit
// conversion nor the 64-bit remainder, both of which are long instruction sequences (NaN takes the second
// branch).
__device__ __forceinline__ int wrap_floor(double u, int n) {
  const double f = floor(u);
  return f >= 0.0 && f < (double)n ? (int)f : wrap((long long)f, n);
}

// ---------------------------------------------------------------------------------------
// Tile-sorted painting.  Particles are counting-sorted by the tile (TS^3 nodes) holding
// their base node floor(u); each workgroup accumulates one tile plus the halo its window
// reaches, one LDS region per mesh (for TSC (TS + 3)^3 nodes from t0 - 1 on the plain mesh and
// (TS + 2)^3 from t0 on the +1/2 interlaced one; PaintReach), then adds the non-zero region
// cells to the global meshes with atomics (a block may take several tiles of a row at once).  A tap that falls outside its region (only possible
// through FP64 rounding at a cell face) goes straight to a global atomic.
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ void mesh_u(const double* __restrict__ pos, int64_t i, double o0, double o1, double o2,
                                       double scale, double* u) {
  u[0] = __dmul_rn(__dsub_rn(pos[3 * i + 0], o0), scale);
  u[1] = __dmul_rn(__dsub_rn(pos[3 * i + 1], o1), scale);
  u[2] = __dmul_rn(__dsub_rn(pos[3 * i + 2], o2), scale);
}

// Tile counters come in NCOPY copies of ntiles + 1: a block counts into copy blockIdx mod
// NCOPY.  Workgroups are dispatched round-robin over the 8 XCDs, so each copy is then updated
// from one XCD only and its cache lines stay in that XCD's L2 instead of moving between XCDs
// on every atomic.  (Any copy assignment is correct; this one is only faster.)  The rank
// returned carries the copy in its top bits.
constexpr int NCOPY = TILE_COUNT_COPIES;
constexpr int RANK_BITS = 28;

// Each thread takes CPT particles per round (blockDim apart) and issues their counter atomics
// back to back, so CPT atomics per thread are in flight at once: on a random catalog the pass is bound by
// the latency of returning atomics, not by their number.  A catalog in some spatial order has runs of
// particles of one tile, whose atomics on one counter would be done one after the other: the first lane of
// such a run inside a wavefront counts for the whole run and the others take their ranks from it (one
// particle on every node of a 128^3 mesh in mesh order: 511 us before, 24 now; 21 million random particles at
// 512^3 0.85 to 0.90 ms either way).
constexpr int CPT = 4;
__global__ void k_tile_count(const double* __restrict__ pos, int64_t n, int64_t base, double o0, double o1,
                             double o2, double scale, int nmesh, int ts_log2, int ntiles, int* __restrict__ count,
                             int* __restrict__ tile_of, int* __restrict__ rank) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x * CPT;
  const int tpa = nmesh >> ts_log2;
  const int copy = blockIdx.x % NCOPY;
  const int lane = threadIdx.x & 63;
  int* cnt = count + (size_t)copy * (ntiles + 1);
  // (whole blocks stay in the loop: the lanes of a wavefront exchange their tiles)
  for (int64_t b0 = (int64_t)blockIdx.x * blockDim.x * CPT; b0 < n; b0 += stride) {
    const int64_t i0 = b0 + threadIdx.x;
    int tile[CPT], r[CPT];
    unsigned long long heads[CPT];  // lanes at which a run begins
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
      const int64_t i = i0 + (int64_t)j * blockDim.x;
      tile[j] = -1;
      if (i < n) {
        double u[3];
        mesh_u(pos, i, o0, o1, o2, scale, u);
        int tc[3];
        for (int a = 0; a < 3; ++a) tc[a] = wrap_floor(u[a], nmesh) >> ts_log2;
        tile[j] = (tc[0] * tpa + tc[1]) * tpa + tc[2];
      }
    }
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
      const int before = __shfl_up(tile[j], 1);  // (by every lane: an idle source would read as tile 0)
      heads[j] = __ballot(lane == 0 || before != tile[j]);
    }
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
      r[j] = 0;
      if ((heads[j] >> lane & 1) && tile[j] >= 0) {
        const unsigned long long later = lane < 63 ? heads[j] >> (lane + 1) : 0;
        r[j] = atomicAdd(&cnt[tile[j]], later ? __ffsll(later) : 64 - lane);
      }
    }
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
      const int64_t i = i0 + (int64_t)j * blockDim.x;
      if (heads[j] != ~0ull) {  // (uniform)
        const int first = 63 - __clzll(heads[j] & (~0ull >> (63 - lane)));
        r[j] = __shfl(r[j], first) + lane - first;
      }
      if (tile[j] >= 0) {
        tile_of[base + i] = tile[j];
        rank[base + i] = r[j] | (copy << RANK_BITS);
      }
    }
  }
}

// Counting in LDS.  Atomics on global counters are done at the memory side, about 23 a nanosecond, which bound
// k_tile_count for random catalogs.  Here a block counts one contiguous chunk of the catalogs into counters of
// 16 bits that all fit in its LDS (a chunk has fewer than 2^16 particles) and writes them out as a row; the
// scan turns the rows into each chunk's start in every tile.  Keys are the tiles, or the groups of tiles that
// one painting block takes.  21 million random particles at 512^3: 0.85 to 0.91 ms with global counters, 0.20 with
// these, and 0.06 more in the scan of the longer rows.
__global__ void __launch_bounds__(1024)
    k_tile_count_lds(const double* __restrict__ dpos, const double* __restrict__ rpos, int64_t nd, int64_t ntot,
                     int chunk, double o0, double o1, double o2, double scale, int nmesh, int ts_log2, int zt_log2,
                     int nkeys, int pitch, int* __restrict__ rows, int* __restrict__ key_of, int* __restrict__ rank) {
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned* cnt = reinterpret_cast<unsigned*>(smem);
  const int words = (nkeys + 1) / 2;
  for (int i = threadIdx.x; i < words; i += blockDim.x) cnt[i] = 0;
  __syncthreads();
  const int tpa = nmesh >> ts_log2;
  const int64_t first = (int64_t)blockIdx.x * chunk;
  const int64_t last = first + chunk < ntot ? first + chunk : ntot;
  for (int64_t i0 = first + threadIdx.x; i0 < last; i0 += (int64_t)blockDim.x * CPT) {
    double p[CPT][3];
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
      const int64_t i = i0 + (int64_t)j * blockDim.x < last ? i0 + (int64_t)j * blockDim.x : i0;
      const double* q = i < nd ? dpos + 3 * i : rpos + 3 * (i - nd);
      p[j][0] = q[0];
      p[j][1] = q[1];
      p[j][2] = q[2];
    }
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
      const int64_t i = i0 + (int64_t)j * blockDim.x;
      if (i >= last) break;
      double u[3];
      mesh_u(p[j], 0, o0, o1, o2, scale, u);
      int tc[3];
      for (int a = 0; a < 3; ++a) tc[a] = wrap_floor(u[a], nmesh) >> ts_log2;
      const int key = (tc[0] * tpa + tc[1]) * (tpa >> zt_log2) + (tc[2] >> zt_log2);
      const int sh = 16 * (key & 1);
      key_of[i] = key;
      rank[i] = (int)(atomicAdd(&cnt[key >> 1], 1u << sh) >> sh & 0xffff);
    }
  }
  __syncthreads();
  int2* row = reinterpret_cast<int2*>(rows + (size_t)blockIdx.x * pitch);  // (pitch is even)
  for (int i = threadIdx.x; i < words; i += blockDim.x) row[i] = make_int2(cnt[i] & 0xffff, cnt[i] >> 16);
}

constexpr int SCAN_THREADS = 256, SUMS_THREADS = 1024;
// Exclusive scan in three launches: per-block scans (block sums out), one-block scan of
// the block sums, and the addition of the scanned sums.  Coalesced throughout.
template <int NT> __device__ __forceinline__ int block_scan_excl(int v, int* part) {
  part[threadIdx.x] = v;
  __syncthreads();
  for (int d = 1; d < NT; d <<= 1) {
    const int add = (int)threadIdx.x >= d ? part[threadIdx.x - d] : 0;
    __syncthreads();
    part[threadIdx.x] += add;
    __syncthreads();
  }
  return part[threadIdx.x] - v;
}

// Counters are `rows` rows of `pitch`; 32 rows are read at once, as the pass is bound by latency.
constexpr int SCAN_ROWS = 32;
__global__ void __launch_bounds__(SCAN_THREADS) k_scan_blocks(const int* __restrict__ count, int n, int rows, int pitch,
                                                              int* __restrict__ off, int* __restrict__ bsum) {
  __shared__ int part[SCAN_THREADS];
  const int i = blockIdx.x * SCAN_THREADS + threadIdx.x;
  int v = 0;
  if (i < n)
    for (int c0 = 0; c0 < rows; c0 += SCAN_ROWS) {
#pragma unroll
      for (int c = 0; c < SCAN_ROWS; ++c) v += c0 + c < rows ? count[(size_t)(c0 + c) * pitch + i] : 0;
    }
  const int ex = block_scan_excl<SCAN_THREADS>(v, part);
  if (i < n) off[i] = ex;
  if (threadIdx.x == SCAN_THREADS - 1) bsum[blockIdx.x] = ex + v;
}

__global__ void __launch_bounds__(SUMS_THREADS) k_scan_sums(int* __restrict__ bsum, int nb, int* __restrict__ off,
                                                            int n) {
  __shared__ int part[SUMS_THREADS];
  __shared__ int carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  for (int base = 0; base < nb; base += SUMS_THREADS) {
    const int i = base + threadIdx.x;
    const int v = i < nb ? bsum[i] : 0;
    const int ex = block_scan_excl<SUMS_THREADS>(v, part);
    if (i < nb) bsum[i] = carry + ex;
    __syncthreads();
    if (threadIdx.x == SUMS_THREADS - 1) carry += ex + v;
    __syncthreads();
  }
  if (threadIdx.x == 0) off[n] = carry;
}

// Final tile offsets, and the counters turned in place into per-row start offsets:
// count[c][i] <- off[i] + sum over c' < c of count[c'][i].
__global__ void __launch_bounds__(SCAN_THREADS) k_scan_add(const int* __restrict__ bsum, int n, int rows, int pitch,
                                                           int* __restrict__ off, int* __restrict__ count) {
  const int i = blockIdx.x * SCAN_THREADS + threadIdx.x;
  if (i >= n) return;
  int start = off[i] + bsum[blockIdx.x];
  off[i] = start;
  for (int c0 = 0; c0 < rows; c0 += SCAN_ROWS) {
    int v[SCAN_ROWS];
#pragma unroll
    for (int c = 0; c < SCAN_ROWS; ++c) v[c] = c0 + c < rows ? count[(size_t)(c0 + c) * pitch + i] : 0;
#pragma unroll
    for (int c = 0; c < SCAN_ROWS; ++c) {
      if (c0 + c < rows) count[(size_t)(c0 + c) * pitch + i] = start;
      start += v[c];
    }
  }
}

// The three steps in one launch, by one block: where all the counters are few.
constexpr int SCAN_ONE = 1 << 16;
__global__ void __launch_bounds__(SUMS_THREADS) k_scan_one(int n, int rows, int pitch, int* __restrict__ off,
                                                           int* __restrict__ count) {
  __shared__ int part[SUMS_THREADS];
  __shared__ int carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  for (int base = 0; base < n; base += SUMS_THREADS) {
    const int i = base + threadIdx.x;
    int v = 0;
    if (i < n)
      for (int c0 = 0; c0 < rows; c0 += SCAN_ROWS) {
#pragma unroll
        for (int c = 0; c < SCAN_ROWS; ++c) v += c0 + c < rows ? count[(size_t)(c0 + c) * pitch + i] : 0;
      }
    const int ex = block_scan_excl<SUMS_THREADS>(v, part);
    int start = carry + ex;
    if (i < n) {
      off[i] = start;
      for (int c = 0; c < rows; ++c) {
        const int m = count[(size_t)c * pitch + i];
        count[(size_t)c * pitch + i] = start;
        start += m;
      }
    }
    __syncthreads();
    if (threadIdx.x == SUMS_THREADS - 1) carry += ex + v;
    __syncthreads();
  }
  if (threadIdx.x == 0) off[n] = carry;
}

// Scatter each particle's payload (x, y, z, signed weight) to its slot in tile order.  The row of a
// particle's counter is its chunk (chunk > 0) or the copy in the top bits of its rank.
__global__ void k_tile_scatter(const int* __restrict__ tile_of, const int* __restrict__ rank, int64_t nd, int64_t n,
                               int pitch, int chunk, const int* __restrict__ start, const double* __restrict__ dpos,
                               const double* __restrict__ dw, const double* __restrict__ rpos,
                               const double* __restrict__ rw, double alpha, double4* __restrict__ payload) {
  // CPT particles per thread and round, loads first: several offset lookups in flight at once
  const int64_t stride = (int64_t)gridDim.x * blockDim.x * CPT;
  for (int64_t b0 = (int64_t)blockIdx.x * blockDim.x * CPT; b0 < n; b0 += stride) {
    int dst[CPT];
    double4 p[CPT];
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
      const int64_t i = b0 + threadIdx.x + (int64_t)j * blockDim.x;
      dst[j] = -1;
      if (i < n) {
        const bool isd = i < nd;
        const int64_t k = isd ? i : i - nd;
        const double* pos = isd ? dpos : rpos;
        const double* wp = isd ? dw : rw;
        p[j].x = pos[3 * k];
        p[j].y = pos[3 * k + 1];
        p[j].z = pos[3 * k + 2];
        p[j].w = (wp ? wp[k] : 1.0) * (isd ? 1.0 : -alpha);
        const int r = rank[i];
        const int row = chunk > 0 ? (int)((unsigned)i / (unsigned)chunk) : (int)((unsigned)r >> RANK_BITS);
        dst[j] = start[(size_t)row * pitch + tile_of[i]] + (r & ((1 << RANK_BITS) - 1));
      }
    }
#pragma unroll
    for (int j = 0; j < CPT; ++j)
      if (dst[j] >= 0) payload[dst[j]] = p[j];
  }
}

// Taps of the window at u: nodes c + TAP0 + j (j < W) with weights wt[j], where c is the integer returned.
template <int W> constexpr int TAP0 = W == 3 ? -1 : 0;
template <int W> __device__ __forceinline__ double taps(double u, double* wt) {
  if constexpr (W == 1) {
    wt[0] = 1.0;
    return floor(__dadd_rn(u, 0.5));
  } else if constexpr (W == 2) {
    const double c = floor(u);
    const double d = __dsub_rn(u, c);
    wt[0] = 1.0 - d;
    wt[1] = d;
    return c;
  } else {
    const double c = floor(__dadd_rn(u, 0.5));
    const double d = __dsub_rn(u, c);
    const double a = 0.5 - d, b = 0.5 + d;
    wt[0] = 0.5 * a * a;
    wt[1] = 0.75 - d * d;
    wt[2] = 0.5 * b * b;
    return c;
  }
}

// One tap, a times b (the scale sc inside), into the LDS region: FP64 atomic add (FP64 meshes; sc = 1),
// or, for FP32 meshes, an integer add of the tap rounded to a multiple of 1/sc (fixed point; 64-bit integer
// LDS atomics are faster than FP64 ones on gfx950, and FP32 LDS atomics far slower).
// Deterministic mode (FIXED for FP64 too): every tap is rounded to a multiple of 1/sc of one
// scale shared by all tiles, so integer sums of the taps are exact in any order.
// The pass is bound by vector instructions, a third of which were the conversion to 64 bits, so a b is
// split by two fused adds instead: adding 3 2^83 rounds it to a multiple of 2^32 whose quotient is the low
// word of the sum, and adding 3 2^51 to the rest, |rest| <= 2^31, leaves that as a 64-bit integer above the
// constant's own bits.  For |a b| < 2^63 (callers leave out NaN and infinities).
__device__ __forceinline__ long long fixed_product(double a, double b) {
  constexpr double HI = 0x1.8p84, LO = 0x1.8p52;
  const double h = fma(a, b, HI);
  const double l = fma(a, b, -(h - HI)) + LO;
  const unsigned long long hb = __double_as_longlong(h), lb = __double_as_longlong(l);
  return (long long)(lb + (hb << 32) - 0x4338000000000000ull);
}

template <typename T, bool DET>
__device__ __forceinline__ void region_add(double* __restrict__ reg, int i, double a, double b) {
  if constexpr (sizeof(T) == 4 || DET)
    lds_atomic_add<unsigned long long>(reinterpret_cast<unsigned long long*>(reg) + i,
                                       (unsigned long long)fixed_product(a, b));
  else
    lds_atomic_add<double>(reg + i, a * b);
}

// Slabs a0 <= a < a1 (tap index along x) of one particle's taps, wsc = weight times sc, into the
// region of sides rsz, rsz, rz.  c: what taps() gave per axis, wt: its weights, rel: the first tap's node in the region.
template <typename T, int W, bool DET>
__device__ __forceinline__ void scatter_slabs(double* __restrict__ reg, T* __restrict__ mesh,
                                              unsigned long long* __restrict__ acc, const double* c,
                                              const double (*wt)[W], double wsc, int nmesh, const int* rel, int rsz,
                                              int rz, double isc, int a0, int a1) {
  const bool inside = rel[0] >= 0 && rel[0] + W <= rsz && rel[1] >= 0 && rel[1] + W <= rsz && rel[2] >= 0 &&
                      rel[2] + W <= rz;
  for (int a = a0; a < a1; ++a) {
    double w0 = wt[0][0];
#pragma unroll
    for (int j = 1; j < W; ++j) w0 = a == j ? wt[0][j] : w0;
    const double wa = wsc * w0;
    if (inside) {
      const int row = ((rel[0] + a) * rsz + rel[1]) * rz + rel[2];
#pragma unroll
      for (int b = 0; b < W; ++b) {
        const double wab = wa * wt[1][b];
#pragma unroll
        for (int d = 0; d < W; ++d) region_add<T, DET>(reg, row + b * rz + d, wab, wt[2][d]);
      }
      continue;
    }
    // a tap outside the LDS region (FP64 rounding at a cell face): straight to the mesh
    const long long g0 = (long long)c[0] + TAP0<W> + a;
#pragma unroll
    for (int b = 0; b < W; ++b) {
      const double wab = wa * wt[1][b];
#pragma unroll
      for (int d = 0; d < W; ++d) {
        const size_t g = ((size_t)wrap(g0, nmesh) * nmesh + wrap((long long)c[1] + TAP0<W> + b, nmesh)) * nmesh +
                         wrap((long long)c[2] + TAP0<W> + d, nmesh);
        if constexpr (DET)
          atomicAdd(&acc[g], (unsigned long long)fixed_product(wab, wt[2][d]));
        else
          unsafeAtomicAdd(&mesh[g], (T)(wab * wt[2][d] * isc));
      }
    }
  }
}

// Per-axis reach of a window from a particle's base node b = floor(u): the plain mesh's taps
// lie on nodes b + LO1 .. b + LO1 + EXT1 - 1 + (0 .. ts - 1 over the tile's base nodes), the
// interlaced mesh's (taps of u + 1/2) on b + LO2 ..; so the LDS region of a tile of ts base
// nodes per axis is ts + EXT nodes wide from t0 + LO.  NGP: one tap at floor(u + 1/2), in
// {b, b + 1} (plain) and b + 1 (interlaced).  CIC: b, b + 1 (plain) and floor(u + 1/2) + {0, 1}
// within b .. b + 2.  TSC: floor(u + 1/2) + {-1, 0, 1} within b - 1 .. b + 2 (plain) and
// b + 1 + {-1, 0, 1} (interlaced).  A tap that FP64 rounding of u + 1/2 at a cell face moves
// outside goes to the mesh directly (scatter_slabs).
template <int W> struct PaintReach;
template <> struct PaintReach<1> { static constexpr int LO1 = 0, EXT1 = 1, LO2 = 1, EXT2 = 0; };
template <> struct PaintReach<2> { static constexpr int LO1 = 0, EXT1 = 1, LO2 = 0, EXT2 = 2; };
template <> struct PaintReach<3> { static constexpr int LO1 = -1, EXT1 = 3, LO2 = 0, EXT2 = 2; };

// Add the non-zero cells of one column along x (NX cells, (y, z) cell k of the region of z side NZ) to the
// mesh with global atomics (DET: the integer sums to the 64-bit accumulators).  Region node i of an axis is
// mesh node t0 + LO + i, wrapped once at most.
template <typename T, bool DET, int NX, int NZ, int LO>
__device__ __forceinline__ void flush_column(const double* __restrict__ reg, int k, T* __restrict__ mesh,
                                             unsigned long long* __restrict__ acc, const int* t0, int nmesh,
                                             double isc) {
  const int rb = k / NZ, rc = k - rb * NZ;
  int gx = t0[0] + LO, gy = t0[1] + LO + rb, gz = t0[2] + LO + rc;
  gx += gx < 0 ? nmesh : (gx >= nmesh ? -nmesh : 0);
  gy += gy < 0 ? nmesh : (gy >= nmesh ? -nmesh : 0);
  gz += gz < 0 ? nmesh : (gz >= nmesh ? -nmesh : 0);
  const size_t plane = (size_t)nmesh * nmesh, cell = (size_t)gy * nmesh + gz;
  constexpr int CH = 11;  // cells read at once
#pragma unroll 1
  for (int i0 = 0; i0 < NX; i0 += CH) {
    long long q[CH];
#pragma unroll
    for (int i = 0; i < CH; ++i)
      q[i] = i0 + i < NX ? reinterpret_cast<const long long*>(reg)[(i0 + i) * (NX * NZ) + k] : 0;
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      // (as bits: a region holds no -0.0, and a tap that underflows to 0 adds nothing)
      if (q[i] != 0) {
        if constexpr (DET)
          atomicAdd(&acc[gx * plane + cell], (unsigned long long)q[i]);
        else if constexpr (sizeof(T) == 4)
          unsafeAtomicAdd(&mesh[gx * plane + cell], (T)((double)q[i] * isc));
        else
          unsafeAtomicAdd(&mesh[gx * plane + cell], (T)__longlong_as_double(q[i]));
      }
      if (++gx == nmesh) gx = 0;
    }
  }
}

// Units of work of a painting block: each of its particles on each mesh, or (`parts` then has them) in slabs.
// All of PKM_MAX_PARTICLES may lie in one tile (a 16^3 mesh is one): twice that, and a step of the block's
// threads beyond, fit 32 bits only without a sign.
__host__ __device__ constexpr unsigned paint_units(int begin, int end, int parts) {
  return (unsigned)(end - begin) * (unsigned)parts;
}
static_assert((long long)paint_units(0, (int)PKM_MAX_PARTICLES, 2) == 2 * PKM_MAX_PARTICLES &&
                  2 * PKM_MAX_PARTICLES + 1024 < 1ll << 32,
              "a painting block's units must not wrap");

// A painting block takes ZT consecutive tiles of a row along z, whose particles are consecutive too.
template <int W, int TS, int ZT> struct PaintShape {
  using R = PaintReach<W>;
  static constexpr int N1 = TS + R::EXT1, N2 = TS + R::EXT2, Z1 = TS * ZT + R::EXT1, Z2 = TS * ZT + R::EXT2;
  static constexpr int CELLS1 = N1 * N1 * Z1, CELLS2 = N2 * N2 * Z2;
  static constexpr int THREADS = ZT == 4 ? 512 : 256;
};

// DET: the tiles' integer sums go to the 64-bit accumulators acc1 / acc2 (one per mesh) with
// integer atomics at the shared scale *gsc, instead of floating-point atomics to d1 / d2.
template <typename T, int W, int TS, int ZT, bool DET>
__global__ void __launch_bounds__((PaintShape<W, TS, ZT>::THREADS))
    k_paint_tiles(const int* __restrict__ off, int per, const double4* __restrict__ payload, double o0, double o1, double o2,
                  double scale, int nmesh, T* __restrict__ d1, T* __restrict__ d2, const double* __restrict__ wmax_d,
                  const double* __restrict__ wmax_r, double alpha, unsigned long long* __restrict__ acc1,
                  unsigned long long* __restrict__ acc2, const double* __restrict__ gsc) {
  constexpr int ts = TS;
  using R = PaintReach<W>;
  using S = PaintShape<W, TS, ZT>;
  constexpr int n1 = S::N1, n2 = S::N2, z1 = S::Z1, z2 = S::Z2;  // region sides of the two meshes
  extern __shared__ __align__(16) unsigned char smem[];
  const int tpa = nmesh / ts;
  // Consecutive blocks go to consecutive XCDs.  The start of a row of tiles moves on by one from row to row:
  // in the tiles' own order an XCD would take every 8th block of every row, which for rows of 8 or 16 blocks
  // is a fixed range of z, and a survey that fills part of the box loads some XCDs twice as much as others.
  const int row = blockIdx.x / (tpa / ZT);
  const int tile = (row * (tpa / ZT) + (blockIdx.x + row) % (tpa / ZT)) * ZT;
  // `off` has an entry per tile (per = ZT of them a block) or per block (per = 1)
  const int* at = off + tile / ZT * per;
  const int start = at[0], end = at[per];
  if (start == end) return;
  double* r1 = reinterpret_cast<double*>(smem);   // FP64 accumulation for both precisions
  const bool two = d2 != nullptr;
  // A unit of work is one particle on one mesh, or, where that leaves most of the block idle, one slab of
  // its taps (slabs everywhere repeat the weights and cost a dense survey 1.07 -> 1.68 ms; the two
  // loops apart and the fetch ahead took 512^3 with 21 million particles from 0.76 to 0.65 ms, a 128^3 mock from
  // 52 to 43 us).
  const bool fine = (end - start) < (int)blockDim.x / 2;
  const int parts = (two ? 2 : 1) * (fine ? W : 1);
  const unsigned units = paint_units(start, end, parts);
  // (a thread's particle is fetched one unit ahead, the first one while the regions are cleared)
  double4 next = make_double4(0.0, 0.0, 0.0, 0.0);
  if (!fine && threadIdx.x < units) next = payload[start + (threadIdx.x >> two)];
  const int ncells = S::CELLS1 + (two ? S::CELLS2 : 0);
  for (int i = threadIdx.x; i < (ncells + 1) / 2; i += blockDim.x)
    reinterpret_cast<double2*>(smem)[i] = make_double2(0.0, 0.0);
  const int tz = tile % tpa, ty = (tile / tpa) % tpa, tx = tile / (tpa * tpa);
  const int t0[3] = {tx * ts, ty * ts, tz * ts};
  // fixed-point scale (FP32 meshes): no region cell can exceed B = (particles that reach it: those of
  // two neighbouring tiles of the row, or all of the block's where only their sum is known) x (largest
  // |payload weight|), since a particle's taps sum to its weight.  B (1 + 2^-20) sc <= 2^63: all 63 bits, less
  // room for half a unit of rounding a particle, so that a block of four tiles has no coarser sums than
  // one-tile blocks with B sc <= 2^61.
  double sc = 1.0;
  if constexpr (DET) {
    sc = *gsc;
  } else if constexpr (sizeof(T) == 4) {
    int most = at[1] - start;
    for (int k = 2; k <= per; ++k) most = max(most, at[k] - at[k - 2]);
    const double wm = fmax(*wmax_d, wmax_r ? alpha * *wmax_r : 0.0);
    const double bound = (double)most * wm;
    int e = 0;
    if (bound > 0.0) (void)frexp(bound * (1.0 + 0x1p-20), &e);  // bound (1 + 2^-20) < 2^e
    sc = ldexp(1.0, 63 - e);
  }
  const double isc = 1.0 / sc;  // a power of two: exact
  __syncthreads();
  auto paint_unit = [&](const double4& p, bool second, int a0, int a1) {
    double u[3];
    u[0] = __dmul_rn(__dsub_rn(p.x, o0), scale);
    u[1] = __dmul_rn(__dsub_rn(p.y, o1), scale);
    u[2] = __dmul_rn(__dsub_rn(p.z, o2), scale);
    double c[3], wt[3][W];
    int rel[3];
    const double wsc = p.w * sc;
    if constexpr (sizeof(T) == 4 || DET) {  // (taps that are not numbers count as nothing)
      if (!(fabs(wsc) <= 0x1p63)) return;
      if (W > 1 && !(fabs(u[0]) + fabs(u[1]) + fabs(u[2]) < __builtin_huge_val())) return;
    }
    for (int a = 0; a < 3; ++a) {
      const int lo = second ? R::LO2 : R::LO1;
      c[a] = taps<W>(second ? __dadd_rn(u[a], 0.5) : u[a], wt[a]);
      // the region begins at the tile origin t0 plus LO in the particle's frame, which is the mesh's own for
      // base nodes inside the mesh
      const double f = floor(u[a]);
      if (f >= 0.0 && f < (double)nmesh) {
        rel[a] = (int)(c[a] - (double)(t0[a] + lo - TAP0<W>));
      } else {
        const long long cu = (long long)f;
        rel[a] = (int)((long long)c[a] + TAP0<W> - (cu - (wrap(cu, nmesh) - t0[a]) + lo));
      }
    }
    scatter_slabs<T, W, DET>(second ? r1 + S::CELLS1 : r1, second ? d2 : d1, second ? acc2 : acc1, c, wt,
                             wsc, nmesh, rel, second ? n2 : n1, second ? z2 : z1, isc, a0, a1);
  };
  if (fine) {
    for (int j = threadIdx.x; j < (int)units; j += blockDim.x) {
      const int q = two ? j / (2 * W) : j / W, sub = j - q * parts;
      const bool second = sub >= W;
      const int a0 = second ? sub - W : sub;
      paint_unit(payload[start + q], second, a0, a0 + 1);
    }
  } else {
    for (unsigned j = threadIdx.x; j < units; j += blockDim.x) {
      const double4 p = next;
      if (j + blockDim.x < units) next = payload[start + ((j + blockDim.x) >> two)];
      paint_unit(p, two && (j & 1), 0, W);
    }
  }
  __syncthreads();
  for (int j = threadIdx.x; j < n1 * z1 + (two ? n2 * z2 : 0); j += blockDim.x) {
    if (j < n1 * z1)
      flush_column<T, DET, n1, z1, R::LO1>(r1, j, d1, acc1, t0, nmesh, isc);
    else
      flush_column<T, DET, n2, z2, R::LO2>(r1 + S::CELLS1, j - n1 * z1, d2, acc2, t0, nmesh, isc);
  }
}

// Deterministic mode: the shared fixed-point scale.  A node's value is a sum of taps of the
// particles whose base node lies within one window width of it, which belong to at most 8
// tiles (2 per axis for tiles of at least 3 nodes), so |value| <= B = 8 (largest tile count)
// (largest |payload weight|); sc = 2^(60 - e) with B < 2^e keeps every partial and total sum
// below 2^60 in magnitude.
__global__ void k_det_scale(const int* __restrict__ off, int ntiles, const double* __restrict__ wmax_d,
                            const double* __restrict__ wmax_r, double alpha, double* __restrict__ gsc) {
  __shared__ int s[256];
  int m = 0;
  for (int t = threadIdx.x; t < ntiles; t += blockDim.x) m = max(m, off[t + 1] - off[t]);
  s[threadIdx.x] = m;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) s[threadIdx.x] = max(s[threadIdx.x], s[threadIdx.x + h]);
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double wm = fmax(*wmax_d, wmax_r ? alpha * *wmax_r : 0.0);
    const double bound = 8.0 * (double)s[0] * wm;
    int e = 0;
    if (bound > 0.0) (void)frexp(bound, &e);
    *gsc = ldexp(1.0, 60 - e);
  }
}

// Deterministic mode: mesh value = accumulated integer / sc.
template <typename T>
__global__ void k_det_convert(const unsigned long long* __restrict__ acc, T* __restrict__ d, size_t n,
                              const double* __restrict__ gsc) {
  const double isc = 1.0 / *gsc;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
    d[i] = (T)((double)(long long)acc[i] * isc);
}

}  // namespace

hipError_t launch_catalog_sums(const double* const* w, const double* const* nbar, const int64_t* n, int ncat,
                               double* partial, int nblk, double* out2, double* wmax, hipStream_t s) {
  SumArgs args{};
  for (int c = 0; c < ncat; ++c) {
    args.w[c] = w[c];
    args.nbar[c] = nbar[c];
    args.n[c] = n[c];
  }
  k_catalog_sums<<<dim3(nblk, ncat), SUM_THREADS, 0, s>>>(args, partial);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_sum_partials2<<<ncat, SUM_THREADS, 0, s>>>(partial, nblk, out2, wmax);
  return hipGetLastError();
}

template <typename T> hipError_t launch_fill(T* p, T* p1, size_t n, T v, hipStream_t s) {
  if (n == 0) return hipSuccess;
  size_t blocks = (n + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  k_fill<T><<<dim3((unsigned)blocks, p1 ? 2 : 1), 256, 0, s>>>(p, p1, n, v);
  return hipGetLastError();
}

int paint_tiles_per_block(int nmesh, int ts, int ntiles) {
  // More tiles a block (8-node tiles) mean fewer halo cells and fewer, longer rows of atomics, which the memory
  // side takes at about 20 a nanosecond whatever their length (512^3, 2 million uniform particles: 1.30, 1.10,
  // 1.01 ms for 1, 2, 4); fewer mean more blocks to spread a survey's dense part over (128^3 mock 52, 71,
  // 66 us; 256^3 survey 213, 175, 240 us; 512^3 0.80, 0.82, 0.76 ms).
  const int tpa = nmesh / ts;
  if (ts != 8) return 1;
  if (ntiles >= 1 << 18 && tpa % 4 == 0) return 4;
  return ntiles >= 1 << 15 && tpa % 2 == 0 ? 2 : 1;
}

TileSort tile_sort_of(int nmesh, int ts, int ntiles, int64_t ntot, bool det, size_t scratch_bytes) {
  // Counters in LDS where they fit: one per tile, or, on larger meshes, one per painting block (not in the
  // deterministic mode, whose scale goes by the tiles).  256 chunks, one for each CU, or a multiple of that
  // below 2^16 particles; no fewer particles than a quarter of the counters, whose rows the scan and the scatter
  // read again (2 million particles at 512^3, 65536 counters, 123 chunks: count and scans 98 + 16 -> 36 + 27 us).
  constexpr int KEYS = 72 * 1024, CHUNK = (1 << 16) - 1;
  const int zt = paint_tiles_per_block(nmesh, ts, ntiles);
  TileSort t{ntiles, zt, 0, TILE_COUNT_COPIES, ntiles + 1};
  const bool group = ntiles > KEYS && !det;
  const int keys = group ? ntiles / zt : ntiles;
  if (keys > KEYS) return t;
  const int64_t waves = (ntot + 256 * (int64_t)CHUNK - 1) / (256 * (int64_t)CHUNK);
  const int64_t chunk = std::min<int64_t>(std::max<int64_t>({(ntot + 256 * waves - 1) / (256 * std::max<int64_t>(waves, 1)),
                                                             keys / 4, 2048}), CHUNK);
  const int64_t rows = (ntot + chunk - 1) / chunk;
  const int pitch = (keys + 2) & ~1;
  if (rows * (int64_t)pitch * 4 > (int64_t)scratch_bytes) return t;
  return TileSort{keys, group ? 1 : zt, (int)chunk, (int)rows, pitch};
}

hipError_t launch_tile_sort(const TileSort& t, const double* origin, double scale, int nmesh, int ts, int64_t nd,
                            int64_t nr, const double* dpos, const double* dw, const double* rpos, const double* rw,
                            double alpha, int* count, int* tile_of, int* rank, int* off, int* bsum, void* payload,
                            hipStream_t s) {
  const int64_t ntot = nd + nr;
  const int tpa = nmesh / ts;
  if (t.chunk > 0) {
    const int zt = (int)((int64_t)tpa * tpa * tpa / t.keys);
    if (t.rows > 0)
      k_tile_count_lds<<<t.rows, 1024, sizeof(unsigned) * ((t.keys + 1) / 2), s>>>(
          dpos, rpos, nd, ntot, t.chunk, origin[0], origin[1], origin[2], scale, nmesh, __builtin_ctz(ts),
          __builtin_ctz(zt), t.keys, t.pitch, count, tile_of, rank);
  } else {
    auto run = [&](const double* pos, int64_t n, int64_t base) {
      if (n <= 0) return;
      const int64_t blocks = std::min<int64_t>((n + 256 * CPT - 1) / (256 * CPT), 16384);
      k_tile_count<<<(unsigned)blocks, 256, 0, s>>>(pos, n, base, origin[0], origin[1], origin[2], scale, nmesh,
                                                    __builtin_ctz(ts), t.keys, count, tile_of, rank);
    };
    run(dpos, nd, 0);
    run(rpos, nr, nd);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int nblk = (t.keys + SCAN_THREADS - 1) / SCAN_THREADS;
  if ((int64_t)t.rows * t.pitch <= SCAN_ONE) {
    k_scan_one<<<1, SUMS_THREADS, 0, s>>>(t.keys, t.rows, t.pitch, off, count);
  } else {
    k_scan_blocks<<<nblk, SCAN_THREADS, 0, s>>>(count, t.keys, t.rows, t.pitch, off, bsum);
    k_scan_sums<<<1, SUMS_THREADS, 0, s>>>(bsum, nblk, off, t.keys);
    k_scan_add<<<nblk, SCAN_THREADS, 0, s>>>(bsum, t.keys, t.rows, t.pitch, off, count);
  }
  e = hipGetLastError();
  if (e != hipSuccess || ntot == 0) return e;
  const int64_t blocks = std::min<int64_t>((ntot + 256 * CPT - 1) / (256 * CPT), 16384);
  k_tile_scatter<<<(unsigned)blocks, 256, 0, s>>>(tile_of, rank, nd, ntot, t.pitch, t.chunk, count, dpos, dw, rpos, rw,
                                                  alpha, (double4*)payload);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_paint_tiles(const int* off, int per, const void* payload, int ntiles, const double* origin, double scale,
                              int nmesh, int window, int ts, T* d1, T* d2, const double* wmax_d,
                              const double* wmax_r, double alpha, hipStream_t s, unsigned long long* acc,
                              double* gsc) {
  const bool two = d2 != nullptr;
  const double4* pl = (const double4*)payload;
  unsigned long long* acc2 = (acc && two) ? acc + (size_t)nmesh * nmesh * nmesh : nullptr;
  if (acc) {
    k_det_scale<<<1, 256, 0, s>>>(off, ntiles, wmax_d, wmax_r, alpha, gsc);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const int zt = paint_tiles_per_block(nmesh, ts, ntiles);
#define PKM_PAINT(WV, TV, ZV)                                                                                  \
  if (window == WV && ts == TV && zt == ZV) {                                                             \
    using S = PaintShape<WV, TV, ZV>;                                                                          \
    const size_t sm = sizeof(double) * ((S::CELLS1 + (two ? S::CELLS2 : 0) + 1) & ~1);                         \
    if (acc)                                                                                                   \
      k_paint_tiles<T, WV, TV, ZV, true><<<ntiles / ZV, S::THREADS, sm, s>>>(                                  \
          off, per, pl, origin[0], origin[1], origin[2], scale, nmesh, d1, d2, wmax_d, wmax_r, alpha, acc, acc2, gsc); \
    else                                                                                                       \
      k_paint_tiles<T, WV, TV, ZV, false><<<ntiles / ZV, S::THREADS, sm, s>>>(                                 \
          off, per, pl, origin[0], origin[1], origin[2], scale, nmesh, d1, d2, wmax_d, wmax_r, alpha, nullptr, nullptr, \
          nullptr);                                                                                            \
    return hipGetLastError();                                                                                  \
  }
  PKM_PAINT(1, 8, 4) PKM_PAINT(2, 8, 4) PKM_PAINT(3, 8, 4)
  PKM_PAINT(1, 8, 2) PKM_PAINT(2, 8, 2) PKM_PAINT(3, 8, 2)
  PKM_PAINT(1, 8, 1) PKM_PAINT(2, 8, 1) PKM_PAINT(3, 8, 1)
  PKM_PAINT(1, 4, 1) PKM_PAINT(2, 4, 1) PKM_PAINT(3, 4, 1)
  PKM_PAINT(1, 16, 1) PKM_PAINT(2, 16, 1) PKM_PAINT(3, 16, 1)
#undef PKM_PAINT
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_det_convert(const unsigned long long* acc, T* d1, T* d2, int nmesh, const double* gsc,
                              hipStream_t s) {
  const size_t n = (size_t)nmesh * nmesh * nmesh;
  const unsigned blocks = (unsigned)std::min<size_t>((n + 255) / 256, 8192);
  k_det_convert<T><<<blocks, 256, 0, s>>>(acc, d1, n, gsc);
  if (d2) k_det_convert<T><<<blocks, 256, 0, s>>>(acc + n, d2, n, gsc);
  return hipGetLastError();
}

template hipError_t launch_paint_tiles<float>(const int*, int, const void*, int, const double*, double, int, int, int,
                                              float*, float*, const double*, const double*, double, hipStream_t,
                                              unsigned long long*, double*);
template hipError_t launch_paint_tiles<double>(const int*, int, const void*, int, const double*, double, int, int, int,
                                               double*, double*, const double*, const double*, double, hipStream_t,
                                               unsigned long long*, double*);
template hipError_t launch_det_convert<float>(const unsigned long long*, float*, float*, int, const double*,
                                              hipStream_t);
template hipError_t launch_det_convert<double>(const unsigned long long*, double*, double*, int, const double*,
                                               hipStream_t);
template hipError_t launch_fill<unsigned long long>(unsigned long long*, unsigned long long*, size_t, unsigned long long, hipStream_t);
template hipError_t launch_fill<float>(float*, float*, size_t, float, hipStream_t);
template hipError_t launch_fill<int>(int*, int*, size_t, int, hipStream_t);
template hipError_t launch_fill<double>(double*, double*, size_t, double, hipStream_t);

}  // namespace pkm
