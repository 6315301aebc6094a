// Pre-pass of the weighted fields: D_c from G (inverse z), then for every entry of the group the
// harmonic weighting and the forward z transform.  Included by one source per precision.
#pragma once

#include "fft_common.hpp"

namespace pkm {

namespace {

// Geometry of a pre-pass block: E points per thread, PT threads per line and G lines, consecutive y of
// one x plane.  G consecutive y of a kz go out as one piece: 128 bytes (16 lines in FP32, 8 in FP64)
// where the threads that the registers leave room for allow it.
template <typename T, int N> struct PreShape {
  static constexpr int E = line_e<T>(N);
  static constexpr int PT = N / E;
  // threads at MINW wavefronts per SIMD
  static constexpr int MINW = sizeof(T) == 4 ? (E <= 8 ? 4 : E <= 12 ? 3 : 2) : (E <= 8 ? 2 : 1);
  static constexpr int lines() {
    int g = 64 / (int)sizeof(T);
    while (g > 1 && (N % g || PT * g > 256 * MINW)) g /= 2;
    return g;
  }
  static constexpr int G = lines();
  static constexpr int THREADS = PT * G;
  static constexpr bool WAVE = 64 % PT == 0;  // a line lies inside one wavefront
  // line pitch: 64 / G modulo the complex values of one row of LDS banks, so that the lanes of a
  // transposed read (G lines by 64 / G kz) spread evenly over the banks
  static constexpr int BANKS = 256 / (int)sizeof(cx<T>);
  static constexpr int PITCH = (ct_line_slots<T, E, N>() - 64 / G + BANKS - 1) / BANKS * BANKS + 64 / G;
  // line regions: two where they fit (a field is then transformed in one while the stores of the previous
  // one still read the other)
  static constexpr size_t REGION = (size_t)G * PITCH;
  static constexpr int REGIONS = sizeof(cx<T>) * (2 * REGION + twst_size<E, N>()) <= 160 * 1024 ? 2 : 1;
  static constexpr size_t SMEM = sizeof(cx<T>) * (REGIONS * REGION + twst_size<E, N>());
};

// ------------------------------------------------------------------------------------------
// One full-length complex transform serves two real fields: an entry pairs two fields f1, f2 of one
// multipole (+m and -m, or two monomials) as Z = FT[D_c (w1 + i w2)] / 2, whose planes kz >= 0 go to the
// first field's buffer and the conjugates of the planes kz = -j <= 0 to plane j of the second's; the
// column pass separates them.  Nothing has to be split here, a line is transformed inside its wavefront,
// and a transform has half the points of harmonic state of a packed real line.  A field without a
// partner keeps its kz >= 0 planes only (the rest mirrors them).  Entries come |m|-major, so the
// recurrence of one continues from the previous one; for |m| > 0 it carries the 1/2 of a pair.
// Finished lines are parked in LDS and stored transposed, G consecutive y per piece.  Planes at and
// beyond the last k edge (kz_live) are not written.
// 512^3, 14 fields of l <= 4: 2.93 -> 2.55 ms (bound by the stores and by the harmonics and butterflies between
// them; stores of 64 bytes a piece took 2.8 ms); 384^3 FP64 3.81 -> 2.98 ms; 432^3, 44 fields in groups of 16:
// 5.22 -> 2.40 ms a group (a kernel of run-time lengths before); 256^3 345 -> 278 us.  128^3, 152 fields of
// l <= 16: 329 -> 368 us, 3.5 TB/s written and vector units 45% busy: all blocks are resident at once and each takes
// its 80 entries one after the other, a barrier an entry.
// ------------------------------------------------------------------------------------------
template <typename T, int N>
__global__ void __launch_bounds__((PreShape<T, N>::THREADS), (PreShape<T, N>::MINW))
    k_zpre(const cx<T>* __restrict__ gin, const T* __restrict__ real_in, int nent,
           const FieldRec* __restrict__ ents, T scale, double off0, double off1, double off2, double h,
           const T* __restrict__ ytab, const cx<T>* __restrict__ tw, Frame fr, int cart, int kz_live) {
  using S = PreShape<T, N>;
  constexpr int E = S::E, PT = S::PT, G = S::G, nh = N / 2;
  extern __shared__ __align__(16) unsigned char smem[];
  cx<T>* lds = reinterpret_cast<cx<T>*>(smem);
  cx<T>* twst = lds + S::REGIONS * S::REGION;
  const int tid = threadIdx.x;
  const int t = tid % PT, g = tid / PT;
  const int line = blockIdx.x * G + g;
  const int ix = line / N, iy = line % N;
  ct_twiddles<T, E, N, N>(twst, tw);
  HRun<T, E> hr;
  if (real_in) {
    const T* src = real_in + (size_t)line * N;
#pragma unroll
    for (int e = 0; e < E; ++e) hr.cr[e] = src[t + PT * e];
    __syncthreads();
  } else {
    // Hermitian extension of the half line (kz = N/2 zero, kz = 0 real), inverse transform, real part
    const cx<T>* src = gin + (size_t)line * nh;
    cx<T> u[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int p = t + PT * e;
      if (e < E / 2) {
        u[e] = gload<T>(src, p);
        if (p == 0) u[e].y = T(0);
      } else {
        u[e] = p == nh ? mk<T>(T(0), T(0)) : cconj<T>(gload<T>(src, p == nh ? 0 : N - p));
      }
    }
    __syncthreads();
    ct_fft_regs<T, E, true, AUTO_PAD, N, S::WAVE>(lds, g * S::PITCH, 1, t, u, twst);
#pragma unroll
    for (int e = 0; e < E; ++e) hr.cr[e] = u[e].x * scale;
  }
  // unit vectors from the observer to this thread's nodes (x, y fixed by the line), formed
  // in FP64 and rounded once: in FP32 the distance to a far observer rounds the same way for
  // whole planes of nodes, and the slope of high-degree harmonics near the pole would turn
  // that common bias into a systematic error of the multipoles
  const double px = off0 + ix * h, py = off1 + iy * h;
  const double pxy2 = px * px + py * py;
  const double ax = fr.r[0] * px + fr.r[1] * py, ay = fr.r[3] * px + fr.r[4] * py, az = fr.r[6] * px + fr.r[7] * py;
  T ux[E], uy[E], uz[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const double pz = off2 + (t + PT * e) * h;
    const double rr = pxy2 + pz * pz;
    const bool zero = !(rr > 0.0);
    const double inv = zero ? 0.0 : (sizeof(T) == 4 ? rsqrt(rr) : 1.0 / sqrt(rr));
    ux[e] = (T)((ax + fr.r[2] * pz) * inv);
    uy[e] = (T)((ay + fr.r[5] * pz) * inv);
    uz[e] = (T)((az + fr.r[8] * pz) * inv);
    // a node at the observer has no direction: its weighted value is zero for every field
    if (zero) hr.cr[e] = T(0);
    hr.ci[e] = T(0);
  }
  auto dir = [&](int v, T& x, T& y, T& z) { x = ux[v]; y = uy[v]; z = uz[v]; };
  hrun_init(hr);
  constexpr size_t plane = field_plane_stride<T>(N);
  // transposed stores: element tid + e THREADS of the block's N x G values is line `gg`, k = k0 + PT e
  const int gg = tid % G, k0 = tid / G;
  const unsigned out_off = (unsigned)(k0 * plane) + blockIdx.x * G + gg;
  // the planes of a pair's second buffer run downwards: plane PT E - k = (PT - k0) + PT (E - 1 - e)
  const unsigned out_neg = (unsigned)((PT - k0) * plane) + blockIdx.x * G + gg;
  const bool all = kz_live == nh;
  for (int f = 0; f < nent; ++f) {
    const FieldRec en = ents[f];
    const int l = en.l, m = en.m;
    const bool pair = en.p1 != nullptr;
    cx<T> u[E];
    if (!cart) {
      hrun_to<T, E>(hr, l, m < 0 ? -m : m, m == 0 ? T(1) : T(0.5), ytab, dir);
#pragma unroll
      for (int e = 0; e < E; ++e) {
        u[e] = mk<T>(hr.q1[e] * hr.cr[e], hr.q1[e] * hr.ci[e]);
        if (!pair) u[e] = mk<T>(m == 0 ? u[e].x : T(2) * (m < 0 ? u[e].y : u[e].x), T(0));
      }
    } else {
      T w[E];
      monomial_eval<T, E>(l, m, pair ? T(0.5) : T(1), dir, w);
#pragma unroll
      for (int e = 0; e < E; ++e) u[e] = mk<T>(hr.cr[e] * w[e], T(0));
      if (pair) {
        monomial_eval<T, E>(l, en.m2, T(0.5), dir, w);
#pragma unroll
        for (int e = 0; e < E; ++e) u[e].y = hr.cr[e] * w[e];
      }
    }
    // Two regions: the barrier below orders the last reads of this one (two fields ago) before the
    // transform that reuses it; one region: a barrier after its reads does.
    cx<T>* park = lds + (S::REGIONS == 2 && (f & 1) ? S::REGION : 0);
    if (S::REGIONS == 1 && f > 0) __syncthreads();
    ct_fft_regs<T, E, false, AUTO_PAD, N, S::WAVE>(park, g * S::PITCH, 1, t, u, twst);
    if constexpr (S::WAVE) ct_sync<true>(); else __syncthreads();
    {
      cx<T>* p = park + g * S::PITCH;
#pragma unroll
      for (int e = 0; e < E; ++e) p[t + PT * e] = u[e];
    }
    __syncthreads();
    // kz = k below N/2, -(N - k) above, the Nyquist plane between
    const cx<T>* q = park + gg * S::PITCH;
    cx<T>* p0 = reinterpret_cast<cx<T>*>(en.p0);
#pragma unroll
    for (int e = 0; e < E / 2; ++e) {
      const int k = k0 + PT * e;
      if (all || k < kz_live) gstore32<T>(p0 + e * PT * plane, out_off, q[k]);
    }
    if (pair) {
      cx<T>* p1 = reinterpret_cast<cx<T>*>(en.p1);
#pragma unroll
      for (int e = E / 2; e < E; ++e) {
        const int k = k0 + PT * e, j = N - k;
        if (j < nh && (all || j < kz_live))
          gstore32<T>(p1 + (E - 1 - e) * PT * plane, out_neg, cconj<T>(q[k]));
      }
      if (k0 == 0) gstore32<T>(p1, out_off, cconj<T>(q[0]));
    }
  }
}

}  // namespace

template <typename T>
hipError_t launch_zpre(const FftShape& fs, const void* g_in, const T* real_in, int nent, const FieldRec* ents_dev,
                       double scale, const double* off, double h, const void* ytab,
                       const void* tw, const Frame& frame, int basis, int kz_live, hipStream_t s) {
#define PKM_PRE_SIDE(NV)                                                                                       \
  case NV: {                                                                                                   \
    using S = PreShape<T, NV>;                                                                                 \
    k_zpre<T, NV><<<NV * NV / S::G, S::THREADS, S::SMEM, s>>>(                                                 \
        (const cx<T>*)g_in, real_in, nent, ents_dev, (T)scale, off[0], off[1], off[2], h,            \
        (const T*)ytab, (const cx<T>*)tw, frame, basis == 1, kz_live);                                         \
    break;                                                                                                     \
  }
  switch (fs.n) { PKM_FOR_SIDES(PKM_PRE_SIDE) default: return hipErrorInvalidValue; }
#undef PKM_PRE_SIDE
  return hipGetLastError();
}

#define PKM_PRE_INST(T)                                                                                           \
  template hipError_t launch_zpre<T>(const FftShape&, const void*, const T*, int, const FieldRec*, double, const double*, double, const void*, const void*, const Frame&, int, \
                                     int, hipStream_t);

}  // namespace pkm
