// Launch wrappers for the estimator's HIP kernels (definitions in kernels_*.hip).
// Every wrapper enqueues on the given stream and returns the launch status.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pkm {

struct FftShape {
  int n;            // mesh side N
  int e_col;        // elements per thread for the length-N column transforms
  int e_z;          // elements per thread for the length-N/2 line transforms
  uint32_t sched_col;  // radix schedule (4 bits per stage) for length N
  int nst_col;
  uint32_t sched_z;    // radix schedule for length N/2
  int nst_z;
  int tile;         // columns per column-pass tile
  int zlines;       // lines per z-pass block
  int e_post, tile_post;  // checked, and in the limit on k bins; the post-pass has its own shape per side
  int cus;          // compute units of the device (0: unknown)
  bool col_builtin;  // e_col and tile are the built-in choice: the column passes run the
                     // kernels compiled for the side
};

// Field buffers (the weighted fields after their z transform) are kz-major, [kz][x][y] with n/2 kz planes
// of n n complex values plus 256 bytes: a power-of-two plane stride would put the pre-pass's stores,
// which go to every plane, on few HBM channels.
template <typename T> __host__ __device__ constexpr size_t field_plane_stride(int n) {
  return (size_t)n * n + 128 / sizeof(T);
}
// One record of the field tables (device).  A pre-pass entry: the buffers p0 and p1 of a pair (p1 null:
// a field alone), l (or degree), m (or monomial code), the partner's code m2; the column pass
// takes the same entries.  A post-pass line: its field's buffer p0, l, m and the multipole's slot.
struct FieldRec {
  void* p0;
  void* p1;
  int l, m, m2, slot;
};

// Bytes of LDS of the z-pass and column-pass blocks of a shape.
size_t zpass_smem_bytes(const FftShape& fs, bool fp64);
size_t colpass_smem_bytes(const FftShape& fs, bool fp64);

// The post-pass of a side with blocks of `lines` kz lines (0, or more than the side's own: those): lines per
// tile, threads per block, persistent blocks per CU that the registers leave room for, and LDS bytes without
// histograms and thresholds.  false: no such side.
struct PostGeometry {
  int tp, threads, per_cu;
  size_t smem;
};
template <typename T> bool post_geometry(int n, int lines, PostGeometry* g);

// Orthogonal matrix (rows r[0..2], r[3..5], r[6..8]) applied to every unit vector, node
// direction and wave vector alike, before harmonics or monomials are evaluated.  The sums
// over m (or over the monomials of one degree) depend on k.x only, so any orthogonal matrix
// gives the same multipoles; the plan picks one that turns the mean line of sight to
// (1,1,1)/sqrt(3), away from the coordinate poles where FP32 rounding of a direction
// cosine becomes a large, and across the survey correlated, angle error.
struct Frame {
  double r[9];
  float f[9];  // the same, rounded (FP32 passes)
  template <typename T> __host__ __device__ T at(int i) const {
    if constexpr (sizeof(T) == 4) return f[i]; else return (T)r[i];
  }
};

struct BinSpec {
  const long long* thr;  // device, nb+1 integer thresholds on |n|^2
  const int* thr32;      // the same, clamped to the int range (no |n|^2 of a mesh reaches it)
  int nb;
  int hist_copies;       // per-block histogram copies
  int turns;             // wavefronts per copy (they add one after the other)
  int thr_lds;           // stage the thresholds in LDS
};

// Sums of ncat (1 or 2) catalogs: out2[2 c] = sum w^2, out2[2 c + 1] = sum w^2 nbar, wmax[c] = max |w| (w, nbar
// may be null => 1).  partial holds 3 nblk doubles a catalog.
hipError_t launch_catalog_sums(const double* const* w, const double* const* nbar, const int64_t* n, int ncat,
                               double* partial, int nblk, double* out2, double* wmax, hipStream_t s);

// n values each of p and, where it is not null, p1.
template <typename T> hipError_t launch_fill(T* p, T* p1, size_t n, T v, hipStream_t s);

// How the particles are sorted by the tile of their base node.  The counters are `rows` rows of `pitch`: with
// chunk > 0 one row per chunk of that many particles, counted in LDS; else TILE_COUNT_COPIES rows of global
// counters (a block uses one row), zeroed by the caller.  keys: tiles, or groups of the tiles one painting
// block takes; per: entries of the offsets a painting block spans.
struct TileSort {
  int keys, per, chunk, rows, pitch;
};
// scratch_bytes: what the rows of a chunked sort may take.
TileSort tile_sort_of(int nmesh, int ts, int ntiles, int64_t ntot, bool det, size_t scratch_bytes);
// The sort: per particle its key and rank, the offsets (keys + 1 entries) and the payload (x, y, z, w for
// data / -alpha w for randoms; 32 bytes each) in key order.  count: the rows (turned into start offsets).
hipError_t launch_tile_sort(const TileSort& t, const double* origin, double scale, int nmesh, int ts, int64_t nd,
                            int64_t nr, const double* dpos, const double* dw, const double* rpos, const double* rw,
                            double alpha, int* count, int* tile_of, int* rank, int* off, int* bsum, void* payload,
                            hipStream_t s);
constexpr int TILE_COUNT_COPIES = 8;
// Scratch entries needed by the tile scan (block sums).
inline int tile_scan_scratch(int ntiles) { return (ntiles + 255) / 256 + 1; }
// Tile-wise painting from the sorted payload.
template <typename T>
// wmax_d / wmax_r: device pointers to the largest |w| of each catalog (wmax_r null without
// randoms); they bound the per-tile fixed-point accumulation of FP32 meshes.
// acc (deterministic mode, else null): 64-bit accumulators, n^3 per mesh (two meshes when d2 is
// set), zeroed by the caller; the paint then leaves d1 / d2 untouched and writes the shared
// fixed-point scale to *gsc, and launch_det_convert turns the accumulators into the meshes.
hipError_t launch_paint_tiles(const int* off, int per, const void* payload, int ntiles, const double* origin, double scale,
                              int nmesh, int window, int ts, T* d1, T* d2, const double* wmax_d,
                              const double* wmax_r, double alpha, hipStream_t s, unsigned long long* acc = nullptr,
                              double* gsc = nullptr);
template <typename T>
hipError_t launch_det_convert(const unsigned long long* acc, T* d1, T* d2, int nmesh, const double* gsc,
                              hipStream_t s);

// Forward real-to-half-complex transform along z of nbuf real meshes (nbuf <= 2).
template <typename T>
hipError_t launch_zfwd(const FftShape& fs, const T* in0, const T* in1, void* out0, void* out1, int nbuf,
                       const void* tw, hipStream_t s);

// Column transform of nbuf half spectra [x][y][kz] in place along y (axis = 1) or x (axis = 0).
template <typename T>
hipError_t launch_col(const FftShape& fs, void* const* bufs_dev, int nbuf, int axis, bool inverse,
                      const void* tw, hipStream_t s);
// Forward transform along x of the field buffers of `nent` entries in place, their first `planes` kz
// planes; rows whose modes all have |n|^2 >= tmax are left unwritten.  Separates the fields of a pair.
template <typename T>
hipError_t launch_col_fields(const FftShape& fs, const FieldRec* ents_dev, int nent, int planes, int tmax,
                             const void* tw, hipStream_t s);

// x-pass of the forward transforms of the two painted meshes, interlace combine,
// compensation and Nyquist zeroing; writes C and, when g_out != null, G = C inverse-
// transformed along x.
template <typename T>
hipError_t launch_xcombine(const FftShape& fs, void* s1, void* s2, void* c_out, void* g_out, int interlaced,
                           int compensated, const void* invw, const void* phase, const void* tw, hipStream_t s);

// Inverse z transform (half-complex to real) of G, scaled, into a real mesh.
template <typename T>
hipError_t launch_zinv(const FftShape& fs, const void* g_in, T* real_out, double scale, const void* tw,
                       hipStream_t s);

// Inverse z of G, scaled to D_c (or D_c read from real_in != null), then for every entry of the group
// the Y_lm(xhat)-weighted forward transform along z into the field buffers, kz planes below
// kz_live only.  basis 1 (Cartesian decomposition): weights are the monomials xhat^a of degree l and
// index code m instead of Y_lm(xhat).  Entries must come with |m| ascending.
template <typename T>
hipError_t launch_zpre(const FftShape& fs, const void* g_in, const T* real_in, int nent, const FieldRec* ents_dev,
                       double scale, const double* off, double h, const void* ytab,
                       const void* tw, const Frame& frame, int basis, int kz_live, hipStream_t s);

// Last transform pass of every field of the group (along y), sum over m of Y_lm(khat) B_lm per
// multipole slot, product with C and binning over the listed tiles (x << 16 | kz0) of `lines` kz lines.  Odd l
// (spherical basis) are binned as Im[C conj (sum)] instead of Re.  Lines come slot by slot, |m|
// ascending within a slot.  Per block the partial sums are rows of nb bins:
// [count, sum |k|, sum |C|^2] when with_l0, then one row of sum 4 pi Y Re[C conj B] per slot.
// basis 1: the slot sums (p!/a!) khat^a B_a over the monomials a of one degree p, and its row
// holds sum Re[C conj (that sum)] without the 4 pi.
template <typename T>
hipError_t launch_xpost(const FftShape& fs, int lines, int nrecs, const FieldRec* recs_dev, int nslots, int with_l0,
                        const void* c_in, const void* ytab, const BinSpec& bs, double kf,
                        double* partial, int nblocks, const void* tw, const Frame& frame, int basis,
                        const unsigned* tiles_dev, int ntiles, hipStream_t s);
template <typename T>
hipError_t launch_xpost_few(const FftShape& fs, int lines, int nrecs, const FieldRec* recs_dev, int nslots, int with_l0,
                            const void* c_in, const void* ytab, const BinSpec& bs, double kf,
                            double* partial, int nblocks, const void* tw, const Frame& frame, int basis,
                            const unsigned* tiles_dev, int ntiles, hipStream_t s);

// out[map[v]] (+)= sum_b partial[b*nvals + v] (map null -> identity), fixed order.
hipError_t launch_reduce(const double* partial, int nblocks, int nvals, double* out, const int* map, int accumulate,
                         hipStream_t s);

// Global line of sight: (k, mu) cells; partial[block][cell*2 + {0: sum w, 1: sum w |C|^2}].
template <typename T>
hipError_t launch_kmu(const FftShape& fs, const void* c_in, const double* los, const BinSpec& bs,
                      const double* mu_edges, int nmu, double* partial, int nblk, hipStream_t s);

// Device-side normalisation of reduced (k, mu) sums {count, sum |C|^2} per cell into
// P = sum / (I count) - S (NaN when empty) and the integer counts.
hipError_t launch_kmu_finish(const double* sums, int ncells, double norm_I, double shot, double* pk, long long* nm,
                             hipStream_t s);

}  // namespace pkm
