// Column passes: length-N transforms along the strided axis of a buffer, in place, and the x pass
// of the painted meshes with the interlace combine.  Included by one source per precision.
#pragma once

#include "fft_common.hpp"

namespace pkm {

namespace {

// Elements per thread, columns and threads of the compile-time column passes: N / E rows by 16 columns
// (128-byte rows in FP32, 256 in FP64), 8 where that exceeds 1024 threads in FP32 or 512 in FP64 (twice the
// registers: 432, 576, 648 and 768 then have 128-byte rows), or the LDS of a CU.  Rows of 64 bytes fetch their
// 128-byte lines twice: 1024^3 combine 7.35 -> 6.32 ms (5.87 since its rows have uniform bases).
__host__ __device__ constexpr int col_e(int n) { return is_pow2(n) ? (n >= 256 ? 16 : 8) : 12; }
template <typename T> __host__ __device__ constexpr int col_tile(int n) {
  return (n / col_e(n)) * 16 > (sizeof(T) == 4 ? 1024 : 512) || sizeof(cx<T>) * ((size_t)n * 17 + n) > 160 * 1024 ? 8 : 16;
}
template <typename T> __host__ __device__ constexpr int col_threads(int n) { return (n / col_e(n)) * col_tile<T>(n); }

// ------------------------------------------------------------------------------------------
// column pass (length N), in place.  Lane c = tid % tile, t = tid / tile: the tile load leaves
// rows t + pt*e of column c in the thread's registers, which is the transform's own register
// layout, so LDS is used only between radix stages.  Tiles run over the contiguous axis (clen
// elements) within each outer plane; the last tile may be partial.
// ------------------------------------------------------------------------------------------
template <typename T, int E, bool INV, int NC, int TC>
__global__ void __launch_bounds__((NC > 0 ? (NC / E) * TC : XMAX_THREADS)) k_col(int n_rt, int tile_rt, uint32_t sched, int nst,
                                                       void* const* __restrict__ bufs, size_t row_stride,
                                                       size_t outer_stride, int clen,
                                                       const cx<T>* __restrict__ tw) {
  extern __shared__ __align__(16) unsigned char smem[];
  cx<T>* lds = reinterpret_cast<cx<T>*>(smem);
  const int n = NC > 0 ? NC : n_rt;
  const int tile = TC > 0 ? TC : tile_rt;
  const int pt = n / E;
  const int tiles = (clen + tile - 1) / tile;
  const int blk = xcd_tile(blockIdx.x, gridDim.x);
  const int outer = blk / tiles;
  const int c0 = (blk % tiles) * tile;
  cx<T>* buf = reinterpret_cast<cx<T>*>(bufs[blockIdx.y]);
  const int pitch = tile + 1;
  const int tid = threadIdx.x;
  const int c = tid % tile, t = tid / tile;
  buf += (size_t)outer * outer_stride + c0;
  const unsigned off = (unsigned)(t * row_stride + c);
  constexpr bool FULL = NC > 0 && (NC / 2) % (TC > 0 ? TC : 1) == 0;
  const bool live = FULL || c0 + c < clen;
  cx<T> u[E];
#pragma unroll
  for (int e = 0; e < E; ++e)
    u[e] = live ? gload32<T>(buf + pt * e * row_stride, off) : mk<T>(T(0), T(0));
  // generic path: the W_N^j table; compile-time path: the per-stage table only
  cx<T>* twl = lds + (size_t)n * pitch;
  cx<T>* twst = twl;
  if constexpr (NC > 0) ct_twiddles<T, E, NC, NC>(twst, tw); else stage_twiddles<T>(twl, tw, n);
  const LineRt rt{n, sched, nst, pt, n};
  xf_regs<T, E, INV, 0, NC, false, true>(lds, c, pitch, rt, t, u, twst, twl);
  if (!live) return;
#pragma unroll
  for (int e = 0; e < E; ++e) gstore32<T>(buf + pt * e * row_stride, off, u[e]);
}

// ------------------------------------------------------------------------------------------
// column pass of the weighted fields, in place: field buffers [kz][x][y], rows along x, tiles over y
// within a kz plane.  A pair Z = B1 + i B2 arrives as U = Z(kz) in the first buffer and
// V = conj Z(-kz) in the second, both transformed along z only; the transforms along x and y of U
// and V are Z(k) and conj Z(-k), so B1 = U + V and B2 = -i (U - V) (the pre-pass carries the 1/2):
// both tiles are loaded, combined, transformed, and the buffers hold one field each from here on.
// Rows whose modes all lie at or beyond the last k edge (fx^2 + kz^2 >= tmax) belong to no bin and are
// not written: 21% of the bytes with edges up to the Nyquist wavenumber.
// Bound by memory: 512^3, 14 fields: 2.69 ms, 5.3 TB/s (2.75 ms before for every mode; 2.79 with 64-bit addresses
// per row, of which 14 registers a thread spilled: 30% more written);
// 432^3, 44 fields in groups of 16: 2.85 -> 1.89 ms a group; 128^3, 152 fields 454 -> 411..455 us (5.1
// TB/s or more).
// ------------------------------------------------------------------------------------------
template <typename T, int N>
__global__ void __launch_bounds__((col_threads<T>(N)), (sizeof(T) == 4 ? 4 : 2))
    k_col_fields(const FieldRec* __restrict__ ents, int tmax, const cx<T>* __restrict__ tw) {
  constexpr int E = col_e(N), TC = col_tile<T>(N), PT = N / E;
  constexpr int TILES = (N + TC - 1) / TC;  // the last one partial where TC does not divide N
  extern __shared__ __align__(16) unsigned char smem[];
  cx<T>* lds = reinterpret_cast<cx<T>*>(smem);
  cx<T>* twst = lds + N * (TC + 1);
  const int blk = xcd_tile(blockIdx.x, gridDim.x);
  const int kz = blk / TILES, c0 = (blk % TILES) * TC;
  const FieldRec en = ents[blockIdx.y];
  const int tid = threadIdx.x, c = tid % TC, t = tid / TC;
  const bool live = N % TC == 0 || c0 + c < N;
  // (uniform row bases and one 32-bit offset a thread: 64-bit addresses per row would spill)
  const unsigned off = (unsigned)(t * N + (live ? c0 + c : N - 1));
  const bool pair = en.p1 != nullptr;
  const size_t plane = (size_t)kz * field_plane_stride<T>(N);
  cx<T>* b0 = reinterpret_cast<cx<T>*>(en.p0) + plane;
  cx<T>* b1 = reinterpret_cast<cx<T>*>(en.p1) + plane;
  cx<T> u[E], v[E];
#pragma unroll
  for (int e = 0; e < E; ++e) u[e] = gload32<T>(b0 + PT * e * N, off);
  if (pair) {
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = gload32<T>(b1 + PT * e * N, off);
  }
  ct_twiddles<T, E, N, N>(twst, tw);
  auto put = [&](cx<T>* b, const cx<T>* w) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int r = t + PT * e, f = r - (e >= E / 2 ? N : 0);
      if (live && f * f + kz * kz < tmax) gstore32<T>(b + PT * e * N, off, w[e]);
    }
  };
  if (pair) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const cx<T> d = csub<T>(u[e], v[e]);
      u[e] = cadd<T>(u[e], v[e]);
      v[e] = mk<T>(d.y, -d.x);
    }
  }
  __syncthreads();  // (the twiddles; the first exchange synchronises again before it writes)
  ct_fft_regs<T, E, false, 0, N, false>(lds, c, TC + 1, t, u, twst);
  put(b0, u);
  if (!pair) return;
  ct_fft_regs<T, E, false, 0, N, false>(lds, c, TC + 1, t, v, twst);
  put(b1, v);
}

// ------------------------------------------------------------------------------------------
// x pass of the painted meshes + combine + inverse x of C (same lane layout as k_col).  512^3 FP32: 0.60 ms for
// 2.1 GB; three transforms in a row on 16 wavefronts a CU leave the memory idle for part of the time.
// ------------------------------------------------------------------------------------------
template <typename T, int E, int NC, int TC>
__global__ void __launch_bounds__((NC > 0 ? (NC / E) * TC : XMAX_THREADS), (sizeof(T) == 4 ? 4 : 2)) k_xcombine(int n_rt, int tile_rt, uint32_t sched, int nst,
                                                            const cx<T>* __restrict__ s1, const cx<T>* __restrict__ s2,
                                                            cx<T>* __restrict__ cout, cx<T>* __restrict__ gout,
                                                            int interlaced, int compensated,
                                                            const T* __restrict__ invw,
                                                            const cx<T>* __restrict__ phase,
                                                            const cx<T>* __restrict__ tw) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int n = NC > 0 ? NC : n_rt;
  const int tile = TC > 0 ? TC : tile_rt;
  const int nh = n >> 1;
  const int pitch = tile + 1;
  const int pt = n / E;
  cx<T>* lds = reinterpret_cast<cx<T>*>(smem);
  const int tiles = (nh + tile - 1) / tile;
  const int blk = xcd_tile(blockIdx.x, gridDim.x);
  const int y = blk / tiles;
  const int kz0 = (blk % tiles) * tile;
  const size_t rs = (size_t)n * nh;
  const int tid = threadIdx.x;
  const int c = tid % tile, t = tid / tile;
  constexpr bool FULL = NC > 0 && (NC / 2) % (TC > 0 ? TC : 1) == 0;
  const bool live = FULL || kz0 + c < nh;
  const int kz = live ? kz0 + c : nh - 1;  // lanes past the row repeat its last column and write nothing
  const size_t base = (size_t)y * nh;
  const unsigned off = (unsigned)(t * rs + kz);
  cx<T> a1[E];
  cx<T> a2[E];
#pragma unroll
  for (int e = 0; e < E; ++e) a1[e] = gload32<T>(s1 + base + pt * e * rs, off);
  if (interlaced) {
#pragma unroll
    for (int e = 0; e < E; ++e) a2[e] = gload32<T>(s2 + base + pt * e * rs, off);
  }
  // generic path: the W_N^j table; compile-time path: the per-stage table only
  cx<T>* twl = lds + (size_t)n * pitch;
  cx<T>* twst = twl;
  if constexpr (NC > 0) ct_twiddles<T, E, NC, NC>(twst, tw); else stage_twiddles<T>(twl, tw, n);
  const LineRt rt{n, sched, nst, pt, n};
  xf_regs<T, E, false, 0, NC, false, true>(lds, c, pitch, rt, t, a1, twst, twl);
  if (interlaced) {
    xf_regs<T, E, false, 0, NC, false, true>(lds, c, pitch, rt, t, a2, twst, twl);
    const cx<T> pyz = cmul<T>(phase[y], phase[kz]);
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int x = t + pt * e;
      const cx<T> b = cmul<T>(a2[e], cmul<T>(phase[x], pyz));
      a1[e] = mk<T>(T(0.5) * (a1[e].x + b.x), T(0.5) * (a1[e].y + b.y));
    }
  }
  const bool ynyq = (y == nh);
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int x = t + pt * e;
    cx<T> v = a1[e];
    if (compensated) v = cscale<T>(v, invw[x] * invw[y] * invw[kz]);
    if (ynyq || x == nh) v = mk<T>(T(0), T(0));
    a1[e] = v;
    if (live) gstore32<T>(cout + base + pt * e * rs, off, v);
  }
  if (gout == nullptr) return;
  xf_regs<T, E, true, 0, NC, false, true>(lds, c, pitch, rt, t, a1, twst, twl);
  if (!live) return;
#pragma unroll
  for (int e = 0; e < E; ++e) gstore32<T>(gout + base + pt * e * rs, off, a1[e]);
}

}  // namespace

// LDS of a column block: n rows of `tile` columns (one spare column per row), and the twiddles:
// the W_N^j table (N entries) or the per-stage table, which has fewer.
template <typename T> inline size_t colsmem(int n, int tile) {
  return sizeof(cx<T>) * ((size_t)n * (tile + 1) + n);
}

// Compile-time column kernels for shapes other than the built-in one (a caller's or a tuned shape).
#define PKM_TRY_COL_SHAPES(TRY) TRY(64, 8, 8) TRY(128, 8, 8) TRY(256, 8, 8) TRY(512, 8, 8) TRY(1024, 8, 4)

// Blocks and launch of a column kernel: KERN<E, NC, TC> with the built-in shape of the side, one of
// the shapes above, or (NC = 0) the runtime-generic kernel.
#define PKM_COL_LAUNCH(OUTER, CLEN, NBUF, CALL)                                                         \
  auto grid_of = [&](int tile) { return dim3((unsigned)((size_t)(OUTER) * (((CLEN) + tile - 1) / tile)), NBUF); }; \
  if (fs.col_builtin) {                                                                                 \
    switch (fs.n) { PKM_FOR_SIDES(PKM_COL_SIDE_##CALL) default: return hipErrorInvalidValue; }            \
    return hipGetLastError();                                                                           \
  }                                                                                                     \
  PKM_TRY_COL_SHAPES(PKM_COL_TRY_##CALL)                                                                 \
  {                                                                                                     \
    constexpr int NC = 0, TC = 0;                                                                       \
    const int thr = (fs.n / fs.e_col) * fs.tile;                                                          \
    const size_t sm = colsmem<T>(fs.n, fs.tile);                                                          \
    const dim3 grid = grid_of(fs.tile);                                                                   \
    PKM_DISPATCH_E(fs.e_col, PKM_COL_RUN_##CALL)                                                          \
  }                                                                                                     \
  return hipGetLastError();
#define PKM_COL_BIND(RUN, NV, EV, TV)                              \
  {                                                                \
    constexpr int NC = NV, E = EV, TC = TV;                        \
    constexpr int thr = (NC / E) * TC;                             \
    const size_t sm = colsmem<T>(NC, TC);                          \
    const dim3 grid = grid_of(TC);                                 \
    RUN;                                                           \
  }

#define PKM_COL_RUN_FWD                                                                                        \
  (k_col<T, E, false, NC, TC><<<grid, thr, sm, s>>>(fs.n, fs.tile, fs.sched_col, fs.nst_col, bufs_dev,         \
                                                    row_stride, outer_stride, clen, (const cx<T>*)tw))
#define PKM_COL_RUN_INV                                                                                       \
  (k_col<T, E, true, NC, TC><<<grid, thr, sm, s>>>(fs.n, fs.tile, fs.sched_col, fs.nst_col, bufs_dev,         \
                                                   row_stride, outer_stride, clen, (const cx<T>*)tw))
#define PKM_COL_RUN_XC                                                                                    \
  (k_xcombine<T, E, NC, TC><<<grid, thr, sm, s>>>(                                                        \
      fs.n, fs.tile, fs.sched_col, fs.nst_col, (const cx<T>*)s1, (const cx<T>*)s2, (cx<T>*)c_out,         \
      (cx<T>*)g_out, interlaced, compensated, (const T*)invw, (const cx<T>*)phase, (const cx<T>*)tw))
#define PKM_COL_SIDE_FWD(NV) case NV: PKM_COL_BIND(PKM_COL_RUN_FWD, NV, col_e(NV), col_tile<T>(NV)) break;
#define PKM_COL_SIDE_INV(NV) case NV: PKM_COL_BIND(PKM_COL_RUN_INV, NV, col_e(NV), col_tile<T>(NV)) break;
#define PKM_COL_SIDE_XC(NV) case NV: PKM_COL_BIND(PKM_COL_RUN_XC, NV, col_e(NV), col_tile<T>(NV)) break;
#define PKM_COL_TRY(RUN, NV, EV, TV) \
  if (fs.n == NV && fs.e_col == EV && fs.tile == TV) { PKM_COL_BIND(RUN, NV, EV, TV) return hipGetLastError(); }
#define PKM_COL_TRY_FWD(NV, EV, TV) PKM_COL_TRY(PKM_COL_RUN_FWD, NV, EV, TV)
#define PKM_COL_TRY_INV(NV, EV, TV) PKM_COL_TRY(PKM_COL_RUN_INV, NV, EV, TV)
#define PKM_COL_TRY_XC(NV, EV, TV) PKM_COL_TRY(PKM_COL_RUN_XC, NV, EV, TV)

template <typename T>
hipError_t launch_col(const FftShape& fs, void* const* bufs_dev, int nbuf, int axis, bool inverse, const void* tw,
                      hipStream_t s) {
  // half spectra [x][y][kz]: rows along y (axis 1) or x (axis 0), tiles over kz
  const size_t n = fs.n, nh = fs.n / 2, plane = n * nh;
  const size_t row_stride = axis == 1 ? nh : plane, outer_stride = axis == 1 ? plane : nh;
  const int clen = (int)nh;
  if (inverse) {
    PKM_COL_LAUNCH(n, clen, nbuf, INV)
  }
  PKM_COL_LAUNCH(n, clen, nbuf, FWD)
}

template <typename T>
hipError_t launch_col_fields(const FftShape& fs, const FieldRec* ents_dev, int nent, int planes, int tmax,
                             const void* tw, hipStream_t s) {
#define PKM_COL_SIDE_FLD(NV)                                                                                  \
  case NV: {                                                                                                  \
    constexpr int TC = col_tile<T>(NV);                                                                          \
    const dim3 grid((unsigned)planes * ((NV + TC - 1) / TC), nent);                                           \
    k_col_fields<T, NV><<<grid, (NV / col_e(NV)) * TC, colsmem<T>(NV, TC), s>>>(ents_dev, tmax,               \
                                                                               (const cx<T>*)tw);             \
    break;                                                                                                    \
  }
  switch (fs.n) { PKM_FOR_SIDES(PKM_COL_SIDE_FLD) default: return hipErrorInvalidValue; }
#undef PKM_COL_SIDE_FLD
  return hipGetLastError();
}

template <typename T>
hipError_t launch_xcombine(const FftShape& fs, void* s1, void* s2, void* c_out, void* g_out, int interlaced,
                           int compensated, const void* invw, const void* phase, const void* tw, hipStream_t s) {
  PKM_COL_LAUNCH(fs.n, fs.n / 2, 1, XC)
}

#define PKM_COLUMNS_INST(T)                                                                                    \
  template hipError_t launch_col<T>(const FftShape&, void* const*, int, int, bool, const void*, hipStream_t);  \
  template hipError_t launch_col_fields<T>(const FftShape&, const FieldRec*, int, int, int, const void*,       \
                                           hipStream_t);                                                       \
  template hipError_t launch_xcombine<T>(const FftShape&, void*, void*, void*, void*, int, int, const void*,   \
                                         const void*, const void*, hipStream_t);

}  // namespace pkm
