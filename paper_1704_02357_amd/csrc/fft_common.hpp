// Helpers shared by the transform kernels: global accesses, twiddle staging, line transforms
// over LDS, the packed real split and the field-buffer geometry.
#pragma once

#include "kernels.hpp"
#include "device_common.hpp"

namespace pkm {

namespace {

constexpr double FOUR_PI = 12.566370614359172953850573533118;
constexpr int ZPAD = 3;  // z-line LDS layout: one spare slot per 8 complex
__host__ __device__ constexpr int zpitch(int nh) { return nh + (nh >> ZPAD) + 1; }
// z-pass blocks: up to 512 threads in FP32, 256 in FP64
template <typename T> __host__ __device__ constexpr int zmax_threads() { return sizeof(T) == 4 ? 512 : 256; }
constexpr int XMAX_THREADS = 512;

// Global-memory accesses through address-space-1 pointers (buffer pointers read from a
// device array would otherwise be generic and compile to flat instructions).
#define PKM_GLOBAL __attribute__((address_space(1)))
template <typename T> __device__ __forceinline__ cx<T> gload(const cx<T>* p, size_t i) {
  const PKM_GLOBAL T* q = (const PKM_GLOBAL T*)(const void*)p;
  return mk<T>(q[2 * i], q[2 * i + 1]);
}
// The same with a wave-uniform pointer and a 32-bit element offset (scalar base, vector offset).
template <typename T> __device__ __forceinline__ cx<T> gload32(const cx<T>* p, unsigned i) {
  const PKM_GLOBAL T* q = (const PKM_GLOBAL T*)((const PKM_GLOBAL char*)(const void*)p + i * (unsigned)sizeof(cx<T>));
  return mk<T>(q[0], q[1]);
}
template <typename T> __device__ __forceinline__ void gstore32(cx<T>* p, unsigned i, cx<T> v) {
  PKM_GLOBAL T* q = (PKM_GLOBAL T*)((PKM_GLOBAL char*)(void*)p + i * (unsigned)sizeof(cx<T>));
  q[0] = v.x;
  q[1] = v.y;
}
// A value the compiler takes as new at this point: what is computed from it is computed here, and not
// kept in registers across the loops around it.
template <typename V> __device__ __forceinline__ V fresh(V v) {
  asm volatile("" : "+v"(v));
  return v;
}
template <typename T> __device__ __forceinline__ void gstore(cx<T>* p, size_t i, cx<T> v) {
  PKM_GLOBAL T* q = (PKM_GLOBAL T*)(void*)p;
  q[2 * i] = v.x;
  q[2 * i + 1] = v.y;
}

// Workgroups are dispatched round-robin over the 8 XCDs (each with its own L2).  Remap so
// that consecutive logical tiles (which share 128-byte rows when a tile is narrower than
// that, and neighbouring rows otherwise) run on the same XCD one after the other.
__device__ __forceinline__ int xcd_tile(int b, int nblk) {
  if (nblk % 8) return b;
  return (b % 8) * (nblk / 8) + b / 8;
}

// Copy the twiddle table into LDS (n entries); returns the LDS copy.
template <typename T>
__device__ __forceinline__ cx<T>* stage_twiddles(cx<T>* dst, const cx<T>* __restrict__ tw, int n) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) dst[i] = tw[i];
  return dst;
}

__device__ __forceinline__ int tdiv(int i, int tile) { return (tile & (tile - 1)) == 0 ? i >> (__ffs(tile) - 1) : i / tile; }
__device__ __forceinline__ int tmod(int i, int tile) { return (tile & (tile - 1)) == 0 ? i & (tile - 1) : i % tile; }

// G contiguous lines of nh complex: element i = tid + j*bs is line i / nh, entry i % nh.
template <typename T, int E>
__device__ __forceinline__ void lines_to_lds(cx<T>* lds, const cx<T>* __restrict__ src, int nh, int lp, int bs) {
  cx<T> v[E];
#pragma unroll
  for (int j = 0; j < E; ++j) v[j] = gload<T>(src, threadIdx.x + j * bs);
#pragma unroll
  for (int j = 0; j < E; ++j) {
    const int i = threadIdx.x + j * bs;
    lds[tdiv(i, nh) * lp + padi<ZPAD>(tmod(i, nh))] = v[j];
  }
}

// Runtime description of one line transform (generic path).
struct LineRt {
  int L;           // line length
  uint32_t sched;  // radix schedule
  int nst;
  int pt;          // threads per line
  int ntw;         // entries of the W_ntw^j table
};

// Line transform with the line in registers on entry and exit (element e = position
// t + pt*e).  LC > 0: compile-time schedule (WAVE = the line lies inside one wavefront);
// LC = 0: generic schedule through the LDS line, block-wide barriers.
template <typename T, int E, bool INV, int PAD, int LC, bool WAVE, bool FINE = false>
__device__ __forceinline__ void xf_regs(cx<T>* lds, int off, int es, const LineRt& rt, int t, cx<T>* u,
                                        const cx<T>* twst, const cx<T>* __restrict__ twl) {
  if constexpr (LC > 0) {
    ct_fft_regs<T, E, INV, PAD, LC, WAVE, FINE>(lds, off, es, t, u, twst);
  } else {
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) lds[off + padi<PAD>(t + rt.pt * e) * es] = u[e];
    __syncthreads();
    lds_fft<T, E, INV, PAD>(lds, off, es, rt.L, rt.sched, rt.nst, t, rt.pt, twl, rt.ntw);
#pragma unroll
    for (int e = 0; e < E; ++e) u[e] = lds[off + padi<PAD>(t + rt.pt * e) * es];
  }
}
// LDS entries of the per-stage twiddle table (compile-time path only).
template <int E, int LC> __host__ __device__ constexpr int twst_size() { return LC > 0 ? ct_tw_total(E, LC) : 0; }

// Forward split of a packed half-length transform: X_k = E_k + W_N^k O_k.
template <typename T>
__device__ __forceinline__ cx<T> r2c_split(const cx<T>* line, int k, int nh, const cx<T>* __restrict__ tw) {
  const cx<T> zk = line[padi<ZPAD>(k)];
  const cx<T> zm = cconj<T>(line[padi<ZPAD>(k == 0 ? 0 : nh - k)]);
  const cx<T> e = mk<T>(T(0.5) * (zk.x + zm.x), T(0.5) * (zk.y + zm.y));
  const cx<T> d = mk<T>(T(0.5) * (zk.x - zm.x), T(0.5) * (zk.y - zm.y));
  const cx<T> o = mk<T>(d.y, -d.x);  // d / i
  return cadd<T>(e, cmul<T>(tw[k], o));
}

// Inverse split: Z_k = E_k + i O_k with E_k = (X_k + conj X_{nh-k})/2,
// O_k = (X_k - conj X_{nh-k}) conj(W_N^k) / 2; X_{nh} = 0 and X_0 taken real.
template <typename T>
__device__ __forceinline__ cx<T> c2r_split(const cx<T>* line, int k, int nh, const cx<T>* __restrict__ tw) {
  cx<T> xk = line[padi<ZPAD>(k)];
  cx<T> xp;
  if (k == 0) {
    xk.y = T(0);
    xp = mk<T>(T(0), T(0));
  } else {
    xp = cconj<T>(line[padi<ZPAD>(nh - k)]);
  }
  const cx<T> e = mk<T>(T(0.5) * (xk.x + xp.x), T(0.5) * (xk.y + xp.y));
  const cx<T> d = mk<T>(T(0.5) * (xk.x - xp.x), T(0.5) * (xk.y - xp.y));
  const cx<T> o = cmul<T>(d, cconj<T>(tw[k]));
  return mk<T>(e.x - o.y, e.y + o.x);  // e + i o
}

__device__ __forceinline__ int sfreq(int j, int n) { return j < (n >> 1) ? j : j - n; }

// Histogram in LDS: `copies` copies of nvals doubles; wave w uses copy w % copies.
__device__ __forceinline__ void hist_zero(double* h, int total) {
  for (int i = threadIdx.x; i < total; i += blockDim.x) h[i] = 0.0;
}
__device__ __forceinline__ void hist_flush(const double* h, int copies, int nvals, double* out) {
  for (int v = threadIdx.x; v < nvals; v += blockDim.x) {
    double s = 0.0;
    for (int c = 0; c < copies; ++c) s += h[c * nvals + v];
    out[v] = s;
  }
}

// Sides the field passes and the column passes are compiled for: every 2^a 3^b with a >= 2 in
// [16, 1024], which is every side a plan accepts.
#ifndef PKM_FOR_SIDES
#define PKM_FOR_SIDES(X)                                                                              \
  X(16) X(24) X(32) X(36) X(48) X(64) X(72) X(96) X(108) X(128) X(144) X(192) X(216) X(256) X(288)    \
  X(324) X(384) X(432) X(512) X(576) X(648) X(768) X(864) X(972) X(1024)
#endif

// CALL with E the run-time number of elements per thread.
#define PKM_DISPATCH_E(EVAL, CALL)                  \
  switch (EVAL) {                                   \
    case 4: { constexpr int E = 4; CALL; break; }   \
    case 6: { constexpr int E = 6; CALL; break; }   \
    case 8: { constexpr int E = 8; CALL; break; }   \
    case 12: { constexpr int E = 12; CALL; break; } \
    case 16: { constexpr int E = 16; CALL; break; } \
    default: return hipErrorInvalidValue;           \
  }

constexpr bool is_pow2(int n) { return (n & (n - 1)) == 0; }
// Radix stages of the compile-time transform.
__host__ __device__ constexpr int ct_stages(int e, int L) {
  int m = 1, k = 0;
  while (m < L) {
    m *= ct_radix(e, L / m);
    ++k;
  }
  return k;
}
// Elements per thread of a full-length line in the field passes (they carry the harmonic state
// of E points): 8 for powers of two; for lengths with a factor 3, 12, or in FP64 6 where that
// costs at most one more radix stage (12 points of FP64 state leave one wave per SIMD).  FP32 lines of
// 1024 take 16: they then lie inside one wavefront (8 would spread them over two and synchronise blocks
// at every stage; pre-pass 32 against 23 ms per 11 fields, post-pass 20 against 16); 128 and 256 do worse with 16
// (pre-pass of 153 fields at 128^3 543 against 383 us, of 14 at 256^3 283 against 278).
template <typename T> __host__ __device__ constexpr int line_e(int n) {
  if (n == 1024 && sizeof(T) == 4) return 16;
  if (is_pow2(n)) return 8;
  if (sizeof(T) == 8 && ct_stages(6, n) <= ct_stages(12, n) + 1) return 6;
  return 12;
}

}  // namespace

}  // namespace pkm
