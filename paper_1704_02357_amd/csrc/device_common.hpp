// Device-side building blocks shared by the estimator's kernels (gfx950, wave64):
// complex arithmetic, small-radix DFTs, an LDS-resident Stockham FFT over a batch of
// lines, the real/complex packing of a real-input transform, the real spherical-harmonic
// recurrence and the integer k-bin search.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pkm {

template <typename T> struct vec2;
template <> struct vec2<float> { using type = float2; };
template <> struct vec2<double> { using type = double2; };
template <typename T> using cx = typename vec2<T>::type;

template <typename T> __device__ __forceinline__ cx<T> mk(T re, T im) { cx<T> r; r.x = re; r.y = im; return r; }
template <typename T> __device__ __forceinline__ cx<T> cadd(cx<T> a, cx<T> b) { return mk<T>(a.x + b.x, a.y + b.y); }
template <typename T> __device__ __forceinline__ cx<T> csub(cx<T> a, cx<T> b) { return mk<T>(a.x - b.x, a.y - b.y); }
template <typename T> __device__ __forceinline__ cx<T> cmul(cx<T> a, cx<T> b) {
  return mk<T>(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
template <typename T> __device__ __forceinline__ cx<T> cconj(cx<T> a) { return mk<T>(a.x, -a.y); }
template <typename T> __device__ __forceinline__ cx<T> cscale(cx<T> a, T s) { return mk<T>(a.x * s, a.y * s); }
// multiply by -i (forward) or +i (inverse)
template <typename T, bool INV> __device__ __forceinline__ cx<T> rot_mi(cx<T> a) {
  return INV ? mk<T>(-a.y, a.x) : mk<T>(a.y, -a.x);
}

// ---------------------------------------------------------------------------------------
// Radix-R DFT on registers: y_s = sum_t x_t exp(-+2 pi i s t / R), R in {2,3,4,6,8,12,16}.
// ---------------------------------------------------------------------------------------
template <typename T, bool INV> __device__ __forceinline__ void dft2(cx<T>* v) {
  cx<T> a = v[0], b = v[1];
  v[0] = cadd<T>(a, b);
  v[1] = csub<T>(a, b);
}

template <typename T, bool INV> __device__ __forceinline__ void dft4(cx<T>* v) {
  cx<T> a0 = cadd<T>(v[0], v[2]), b0 = csub<T>(v[0], v[2]);
  cx<T> a1 = cadd<T>(v[1], v[3]), b1 = rot_mi<T, INV>(csub<T>(v[1], v[3]));
  v[0] = cadd<T>(a0, a1);
  v[2] = csub<T>(a0, a1);
  v[1] = cadd<T>(b0, b1);
  v[3] = csub<T>(b0, b1);
}

// a times a constant.  Rounded to 24 bits, sqrt(1/2), sqrt(3)/2 and cos(pi/8) are 1.7e-8, 1.8e-8 and 3.1e-8 too
// small, always the same way, and the power of a line shrinks by what the constants of its butterflies lack
// (4.1e-8 at 128 points, 5.0e-8 at 144, twiddles included), which no average over modes removes.  FINE carries the
// constant's remainder inside the one rounding: 2.4e-8 and 0.8e-8.  The transforms of the painted meshes take it,
// whose error goes into P_0; the passes over the weighted fields, bound by vector instructions, lose 2 to 3% with it
// where radices 3, 6 and 12 run.  FP32 against FP64, 128^3 survey, 60 seeds: P_l 1.84e-7 -> 1.39e-7; 432^3, l <= 8:
// 2.9e-7 -> 1.6e-7; times unchanged.
template <typename T, bool FINE> __device__ __forceinline__ T times_c(T a, double c) {
  if (FINE && sizeof(T) == 4 && (double)(T)c != c) return (T)__builtin_fmaf(a, (T)c, a * (T)(c - (double)(T)c));
  return a * (T)c;
}

template <typename T, bool INV, bool FINE> __device__ __forceinline__ void dft3(cx<T>* v) {
  const T h = T(0.5);
  const double s3 = INV ? -0.86602540378443864676 : 0.86602540378443864676;
  cx<T> t1 = cadd<T>(v[1], v[2]);
  cx<T> t2 = csub<T>(v[1], v[2]);
  cx<T> m = mk<T>(v[0].x - h * t1.x, v[0].y - h * t1.y);
  // forward: y1 = m - i s3 t2, y2 = m + i s3 t2
  cx<T> it = mk<T>(times_c<T, FINE>(t2.y, s3), times_c<T, FINE>(t2.x, -s3));  // -i * s3 * t2
  v[0] = cadd<T>(v[0], t1);
  v[1] = cadd<T>(m, it);
  v[2] = csub<T>(m, it);
}

template <typename T, bool INV, bool FINE> __device__ __forceinline__ void dft6(cx<T>* v) {
  // split t -> (t, t+3): a_t = x_t + x_{t+3}, b_t = (x_t - x_{t+3}) W6^t
  cx<T> a[3], b[3];
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    a[t] = cadd<T>(v[t], v[t + 3]);
    b[t] = csub<T>(v[t], v[t + 3]);
  }
  const double s1 = INV ? 0.86602540378443864676 : -0.86602540378443864676;
  auto rot = [&](cx<T> a, T c) { return mk<T>(a.x * c - times_c<T, FINE>(a.y, s1), times_c<T, FINE>(a.x, s1) + a.y * c); };
  b[1] = rot(b[1], T(0.5));    // W6^1
  b[2] = rot(b[2], T(-0.5));   // W6^2
  dft3<T, INV, FINE>(a);
  dft3<T, INV, FINE>(b);
  v[0] = a[0]; v[2] = a[1]; v[4] = a[2];
  v[1] = b[0]; v[3] = b[1]; v[5] = b[2];
}

template <typename T, bool INV, bool FINE> __device__ __forceinline__ void dft8(cx<T>* v) {
  cx<T> a[4], b[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    a[t] = cadd<T>(v[t], v[t + 4]);
    b[t] = csub<T>(v[t], v[t + 4]);
  }
  const double r = 0.70710678118654752440;
  // b_t *= W8^t
  const T p1 = times_c<T, FINE>(b[1].x + b[1].y, r), m1 = times_c<T, FINE>(b[1].x - b[1].y, r);
  const T p3 = times_c<T, FINE>(b[3].x + b[3].y, r), m3 = times_c<T, FINE>(b[3].x - b[3].y, r);
  b[1] = INV ? mk<T>(m1, p1) : mk<T>(p1, -m1);
  b[2] = rot_mi<T, INV>(b[2]);
  b[3] = INV ? mk<T>(-p3, m3) : mk<T>(-m3, -p3);
  dft4<T, INV>(a);
  dft4<T, INV>(b);
  v[0] = a[0]; v[2] = a[1]; v[4] = a[2]; v[6] = a[3];
  v[1] = b[0]; v[3] = b[1]; v[5] = b[2]; v[7] = b[3];
}

// a * exp(-+2 pi i j / 12) for the constant (cos, sin) of that angle, one of them +-1/2.
template <typename T, bool INV, bool FINE> __device__ __forceinline__ cx<T> rot_c(cx<T> a, double c, double s) {
  const double ss = INV ? s : -s;
  return mk<T>(times_c<T, FINE>(a.x, c) - times_c<T, FINE>(a.y, ss), times_c<T, FINE>(a.x, ss) + times_c<T, FINE>(a.y, c));
}

// 12 = 4 x 3: t = t0 + 4 t1, s = s1 + 3 s0; DFTs of 3 over t1, twiddles W12^(t0 s1), DFTs of 4.
template <typename T, bool INV, bool FINE> __device__ __forceinline__ void dft12(cx<T>* v) {
  const double h = 0.86602540378443864676;
  cx<T> a[4][3];
#pragma unroll
  for (int t0 = 0; t0 < 4; ++t0) {
#pragma unroll
    for (int t1 = 0; t1 < 3; ++t1) a[t0][t1] = v[t0 + 4 * t1];
    dft3<T, INV, FINE>(a[t0]);
  }
  a[1][1] = rot_c<T, INV, FINE>(a[1][1], h, 0.5);      // W12^1
  a[1][2] = rot_c<T, INV, FINE>(a[1][2], 0.5, h);      // W12^2
  a[2][1] = rot_c<T, INV, FINE>(a[2][1], 0.5, h);      // W12^2
  a[2][2] = rot_c<T, INV, FINE>(a[2][2], -0.5, h);     // W12^4
  a[3][1] = rot_mi<T, INV>(a[3][1]);             // W12^3
  a[3][2] = mk<T>(-a[3][2].x, -a[3][2].y);       // W12^6
#pragma unroll
  for (int s1 = 0; s1 < 3; ++s1) {
    cx<T> b[4];
#pragma unroll
    for (int t0 = 0; t0 < 4; ++t0) b[t0] = a[t0][s1];
    dft4<T, INV>(b);
#pragma unroll
    for (int s0 = 0; s0 < 4; ++s0) v[s1 + 3 * s0] = b[s0];
  }
}

// The rotations of a DFT of 16, always FINE: the two such DFTs of a length of 256 took 5.3e-8 of a line's power with
// rounded constants, where radices 8, 8 and 4 take 4.1e-8; 1.0e-8 now (the remainder of sin(pi/8) is left out).  1024
// points: 5.3e-8, 5.0e-8 with radices 8, 8, 8 and 2, 3.1e-8 now (1.4e-8 with FINE radix-8 stages).
// a * exp(-+2 pi i j / 16): j = 1 and 9 (FIRST: the larger constant on the diagonal; the sign of both with 9) or 3.
template <typename T, bool INV, bool FIRST> __device__ __forceinline__ cx<T> rot_16(cx<T> a, double sign) {
  const double c1 = 0.92387953251128675613, c3 = 0.38268343236508977173;
  const T s3 = (T)(sign * c3);
  const T px = times_c<T, true>(a.x, sign * c1), py = times_c<T, true>(a.y, sign * c1);
  // forward: (x + i y)(c - i s)
  if constexpr (FIRST) return INV ? mk<T>(px - a.y * s3, a.x * s3 + py) : mk<T>(px + a.y * s3, py - a.x * s3);
  else return INV ? mk<T>(a.x * s3 - py, px + a.y * s3) : mk<T>(a.x * s3 + py, a.y * s3 - px);
}
// j = 2, and 6 (the same times -+i)
template <typename T, bool INV> __device__ __forceinline__ cx<T> rot_8(cx<T> a) {
  const double r = 0.70710678118654752440;
  const T p = times_c<T, true>(a.x + a.y, r), m = times_c<T, true>(a.x - a.y, r);
  return INV ? mk<T>(m, p) : mk<T>(p, -m);
}

// 16 = 4 x 4: t = t0 + 4 t1, s = s1 + 4 s0; DFTs of 4 over t1, twiddles W16^(t0 s1), DFTs of 4.
template <typename T, bool INV> __device__ __forceinline__ void dft16(cx<T>* v) {
  cx<T> a[4][4];
#pragma unroll
  for (int t0 = 0; t0 < 4; ++t0) {
#pragma unroll
    for (int t1 = 0; t1 < 4; ++t1) a[t0][t1] = v[t0 + 4 * t1];
    dft4<T, INV>(a[t0]);
  }
  a[1][1] = rot_16<T, INV, true>(a[1][1], 1.0);             // W16^1
  a[1][2] = rot_8<T, INV>(a[1][2]);                         // W16^2
  a[1][3] = rot_16<T, INV, false>(a[1][3], 1.0);            // W16^3
  a[2][1] = rot_8<T, INV>(a[2][1]);                         // W16^2
  a[2][2] = rot_mi<T, INV>(a[2][2]);                        // W16^4
  a[2][3] = rot_mi<T, INV>(rot_8<T, INV>(a[2][3]));         // W16^6
  a[3][1] = rot_16<T, INV, false>(a[3][1], 1.0);            // W16^3
  a[3][2] = rot_mi<T, INV>(rot_8<T, INV>(a[3][2]));         // W16^6
  a[3][3] = rot_16<T, INV, true>(a[3][3], -1.0);            // W16^9
#pragma unroll
  for (int s1 = 0; s1 < 4; ++s1) {
    cx<T> b[4];
#pragma unroll
    for (int t0 = 0; t0 < 4; ++t0) b[t0] = a[t0][s1];
    dft4<T, INV>(b);
#pragma unroll
    for (int s0 = 0; s0 < 4; ++s0) v[s1 + 4 * s0] = b[s0];
  }
}

template <typename T, int R, bool INV, bool FINE = false> __device__ __forceinline__ void dft_r(cx<T>* v) {
  if constexpr (R == 2) dft2<T, INV>(v);
  else if constexpr (R == 3) dft3<T, INV, FINE>(v);
  else if constexpr (R == 4) dft4<T, INV>(v);
  else if constexpr (R == 6) dft6<T, INV, FINE>(v);
  else if constexpr (R == 8) dft8<T, INV, FINE>(v);
  else if constexpr (R == 12) dft12<T, INV, FINE>(v);
  else dft16<T, INV>(v);
}

// ---------------------------------------------------------------------------------------
// Stockham (decimation-in-time, autosorting) FFT of a batch of lines resident in LDS.
// Element i of a line sits at lds[off + i*es].  Each line is processed by Pt = L/E threads;
// this thread is number t of its line.  At a stage of radix R and span m, butterfly b
// (b = t + q*Pt, q < E/R) reads x_s = in[b + s L/R], multiplies by W_{mR}^{s k} (k = b mod m),
// applies the radix-R DFT and writes y_s to out[(b/m) m R + k + s m].  The stage runs in
// place: all reads finish at a barrier before any write.  Twiddles come from
// tw[j] = exp(-2 pi i j / Ntw); W_{mR}^{q} = tw[q * Ntw/(mR)].  The caller must hold a
// barrier between filling the lines and calling this; it returns after a barrier.
// ---------------------------------------------------------------------------------------
// Physical LDS slot of element i: with PAD > 0 one spare slot follows every 2^PAD elements,
// which breaks the power-of-two strides of the first Stockham stages across LDS banks.
template <int PAD> __host__ __device__ __forceinline__ constexpr int padi(int i) {
  return PAD > 0 ? i + (i >> PAD) : i;
}

template <typename T, int E, int R, bool INV, int PAD>
__device__ __forceinline__ void stockham_stage(cx<T>* lds, int off, int es, int L, int m, int t, int Pt,
                                               const cx<T>* __restrict__ tw, int Ntw) {
  constexpr int NB = E / R;
  cx<T> v[E];
  const int Lr = L / R;
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    const int b = t + q * Pt;
#pragma unroll
    for (int s = 0; s < R; ++s) v[q * R + s] = lds[off + padi<PAD>(b + s * Lr) * es];
  }
  __syncthreads();
  const int step = Ntw / (m * R);
  const bool pow2 = (m & (m - 1)) == 0;
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    const int b = t + q * Pt;
    const int k = pow2 ? (b & (m - 1)) : b % m;
    const int base = (b - k) * R + k;  // (b/m) m R + k
    if (k != 0) {
#pragma unroll
      for (int s = 1; s < R; ++s) {
        cx<T> w = tw[s * k * step];
        if (INV) w.y = -w.y;
        v[q * R + s] = cmul<T>(v[q * R + s], w);
      }
    }
    dft_r<T, R, INV, true>(&v[q * R]);  // (only transforms of the painted meshes come here)
#pragma unroll
    for (int s = 0; s < R; ++s) lds[off + padi<PAD>(base + s * m) * es] = v[q * R + s];
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------------------
// Compile-time Stockham FFT for L = 2^a 3^b with the line held in registers on entry and
// exit.  At each stage the first of the radices 12, 8, 6, 4, 3, 2 that divides both E and the
// remaining length, or 16 where that saves a stage (E = 16 and 16, 256 or 1024 left); spans, strides and twiddle offsets are constants.  Element e of the register array u is position t + PT*e of the line (PT = L/E
// threads per line, this thread number t).  The first stage reads its inputs straight from
// u and the last stage's outputs are exactly the positions t + PT*e again, so only the
// exchanges between stages go through LDS (at lds[off + padi<PAD>(i)*es]).
//
// Twiddles come from a per-stage table (ct_twiddles): the stage of span M and radix R keeps
// W_{MR}^{sk} at offset ct_tw_off(M) + k(R-1) + (s-1), so lanes with consecutive k read
// consecutive entries instead of the strided, bank-conflicting reads of a W_N^j table.
//
// WAVE = true when every line lies inside one wavefront: the stage exchanges then need only
// a wavefront-level ordering (LDS operations of one wave complete in issue order).
// ---------------------------------------------------------------------------------------
__host__ __device__ constexpr int ct_radix(int e, int rem) {
  return (e % 16 == 0 && (rem == 16 || rem == 256 || rem == 1024)) ? 16
         : (e % 12 == 0 && rem % 12 == 0) ? 12
         : (e % 8 == 0 && rem % 8 == 0)   ? 8
         : (e % 6 == 0 && rem % 6 == 0) ? 6
         : (e % 4 == 0 && rem % 4 == 0) ? 4
         : (e % 3 == 0 && rem % 3 == 0) ? 3
                                        : 2;
}
// Offset of the twiddles of the stage with span mstage (all stages with span < mstage).
__host__ __device__ constexpr int ct_tw_off(int e, int L, int mstage) {
  int m = 1, sz = 0;
  while (m < mstage && m < L) {
    const int r = ct_radix(e, L / m);
    if (m > 1) sz += m * (r - 1);
    m *= r;
  }
  return sz;
}
__host__ __device__ constexpr int ct_tw_total(int e, int L) { return ct_tw_off(e, L, L); }
__host__ __device__ constexpr int ct_last_radix(int e, int L) {
  int m = 1, r = 2;
  while (m < L) {
    r = ct_radix(e, L / m);
    m *= r;
  }
  return r;
}

// Fill the per-stage table from tw[j] = exp(-2 pi i j / NTW) (NTW a multiple of L).
template <typename T, int E, int L, int NTW>
__device__ __forceinline__ void ct_twiddles(cx<T>* dst, const cx<T>* __restrict__ tw) {
  constexpr int total = ct_tw_total(E, L);
  for (int i = threadIdx.x; i < total; i += blockDim.x) {
    int m = 1, off = 0;
    for (;;) {
      const int r = ct_radix(E, L / m);
      if (m > 1) {
        const int sz = m * (r - 1);
        if (i < off + sz) {
          const int j = i - off;
          const int k = j / (r - 1), s = j % (r - 1) + 1;
          dst[i] = tw[s * k * (NTW / (m * r))];
          break;
        }
        off += sz;
      }
      m *= r;
    }
  }
}

// Ordering of LDS accesses between the threads that share a line.
template <bool WAVE> __device__ __forceinline__ void ct_sync() {
  if constexpr (WAVE) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
}

// Spare slots of one exchange: element i sits at i + a (i >> s).
struct Pad {
  int s, a;
  __host__ __device__ constexpr int operator()(int i) const { return i + a * (i >> s); }
};
// Most lanes of a group that fall on one LDS bank (a slot of 8 or 16 bytes covers 2 or 4 of the 64 banks;
// 32 or 16 lanes are served at a time).
__host__ __device__ constexpr int ct_hits(Pad pad, int banks, int PT, int t0, bool scatter, int M, int R) {
  int count[32] = {};
  int worst = 0;
  for (int i = 0; i < (PT < banks ? PT : banks); ++i) {
    const int t = t0 + i, b = pad(scatter ? (t - t % M) * R + t % M : t) % banks;
    worst = ++count[b] > worst ? count[b] : worst;
  }
  return worst;
}
// Whether the slot of i + K is that of i plus the constant pad(K), for every i of a stage: then one
// address register and immediate offsets serve it.  Writes: i mod M R < M and K = s M < M R.  Reads: i is
// any position, so K must be a multiple of the spacing.
__host__ __device__ constexpr bool ct_sep_w(Pad p, int M, int MR) {
  const int span = 1 << p.s;
  return p.a == 0 || M % span == 0 || (span % M == 0 && (MR % span == 0 || span % MR == 0));
}
__host__ __device__ constexpr bool ct_sep_r(Pad p, int K) { return p.a == 0 || K % (1 << p.s) == 0; }
// The spare slots of the exchange after the stage that ends at span X (the writes of that stage, the
// reads of the next) of a length-L line in LDS slots of one element: those with the fewest bank
// conflicts, then constant offsets, then the least space (at most one quarter more).
__host__ __device__ constexpr Pad ct_exchange_pad(int bytes, int E, int L, int X) {
  const int banks = 256 / bytes, PT = L / E;
  int M = 1, R = ct_radix(E, L);
  while (M * R < X) {
    M *= R;
    R = ct_radix(E, L / M);
  }
  const int R2 = ct_radix(E, L / X);
  Pad best{0, 0};
  int best_cost = 1 << 30;
  for (int s = 1; s <= 9; ++s)
    for (int a = 0; a <= 8; ++a) {
      const Pad p{s, a};
      if (a * ((L - 1) >> s) * 4 > L || (a == 0 && s > 1)) continue;
      int cost = 0;
      for (int t0 = 0; t0 < PT && t0 <= banks; t0 += banks)
        cost += 64 * (ct_hits(p, banks, PT, t0, true, M, R) + ct_hits(p, banks, PT, t0, false, M, R));
      bool sep = ct_sep_w(p, M, M * R) && ct_sep_r(p, L / R2);
      if (E / R2 > 1) sep = sep && ct_sep_r(p, PT);
      cost += (sep ? 0 : 32) + a * ((L - 1) >> s) * 16 / L;
      if (cost < best_cost) {
        best_cost = cost;
        best = p;
      }
    }
  return best;
}
// PAD of the compile-time transforms: padi's, or AUTO_PAD for the choice above (es = 1 only).
constexpr int AUTO_PAD = 64;
template <typename T, int E, int PAD, int L, int X> __host__ __device__ constexpr Pad ct_pad_of() {
  if constexpr (PAD == AUTO_PAD) return ct_exchange_pad((int)sizeof(cx<T>), E, L, X);
  else if constexpr (PAD > 0) return Pad{PAD, 1};
  else return Pad{0, 0};
}
// LDS slots of a line with AUTO_PAD.
template <typename T, int E, int L> __host__ __device__ constexpr int ct_line_slots() {
  int slots = L;
  for (int m = ct_radix(E, L); m < L; m *= ct_radix(E, L / m)) {
    const int n = ct_exchange_pad((int)sizeof(cx<T>), E, L, m)(L - 1) + 1;
    slots = n > slots ? n : slots;
  }
  return slots;
}

// Stage of span M: inputs v[q*R + s] = x[b + s*L/R], b = t + q*PT.
template <typename T, int E, int PAD, int L, int M>
__device__ __forceinline__ void ct_gather(const cx<T>* lds, int off, int es, int t, cx<T>* v) {
  constexpr int R = ct_radix(E, L / M), PT = L / E, NB = E / R, LR = L / R;
  constexpr Pad pad = ct_pad_of<T, E, PAD, L, M>();
  const cx<T>* p = lds + off + pad(t) * es;
#pragma unroll
  for (int q = 0; q < NB; ++q)
#pragma unroll
    for (int s = 0; s < R; ++s) {
      if (ct_sep_r(pad, q * PT + s * LR)) v[q * R + s] = p[pad(q * PT + s * LR) * es];
      else v[q * R + s] = lds[off + pad(t + q * PT + s * LR) * es];
    }
}
template <typename T, int E, bool INV, int L, int M, bool FINE = false>
__device__ __forceinline__ void ct_butterflies(int t, cx<T>* v, const cx<T>* twst) {
  constexpr int R = ct_radix(E, L / M), PT = L / E, NB = E / R, OFF = ct_tw_off(E, L, M);
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    if constexpr (M > 1) {
      const int k = (t + q * PT) % M;  // a mask when M is a power of two
#pragma unroll
      for (int s = 1; s < R; ++s) {
        cx<T> w = twst[OFF + k * (R - 1) + (s - 1)];
        if (INV) w.y = -w.y;
        v[q * R + s] = cmul<T>(v[q * R + s], w);
      }
    }
    dft_r<T, R, INV, FINE>(&v[q * R]);
  }
}
// Outputs y_s of butterfly b go to (b/M) M R + (b mod M) + s M.
template <typename T, int E, int PAD, int L, int M>
__device__ __forceinline__ void ct_scatter(cx<T>* lds, int off, int es, int t, const cx<T>* v) {
  constexpr int R = ct_radix(E, L / M), PT = L / E, NB = E / R;
  constexpr Pad pad = ct_pad_of<T, E, PAD, L, M * R>();
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    const int b = t + q * PT;
    const int k = b % M;
    const int base = (b - k) * R + k;
    cx<T>* p = lds + off + pad(base) * es;
#pragma unroll
    for (int s = 0; s < R; ++s) {
      if (ct_sep_w(pad, M, M * R)) p[pad(s * M) * es] = v[q * R + s];
      else lds[off + pad(base + s * M) * es] = v[q * R + s];
    }
  }
}
template <typename T, int E, bool INV, int PAD, int L, bool WAVE, int M, bool FINE = false>
__device__ __forceinline__ void ct_rest(cx<T>* lds, int off, int es, int t, cx<T>* v, const cx<T>* twst) {
  ct_butterflies<T, E, INV, L, M, FINE>(t, v, twst);
  constexpr int R = ct_radix(E, L / M);
  if constexpr (M * R < L) {
    ct_sync<WAVE>();
    ct_scatter<T, E, PAD, L, M>(lds, off, es, t, v);
    ct_sync<WAVE>();
    ct_gather<T, E, PAD, L, M * R>(lds, off, es, t, v);
    ct_rest<T, E, INV, PAD, L, WAVE, M * R, FINE>(lds, off, es, t, v, twst);
  }
}

// Transform of u in place (registers).  The caller must have finished every read of the
// line's LDS slots by the threads of the line (ct_sync<WAVE> or stronger) and the twiddle
// table must be visible.  On return the LDS slots hold intermediate data.
template <typename T, int E, bool INV, int PAD, int L, bool WAVE, bool FINE = false>
__device__ __forceinline__ void ct_fft_regs(cx<T>* lds, int off, int es, int t, cx<T>* u, const cx<T>* twst) {
  constexpr int R0 = ct_radix(E, L), NB0 = E / R0;
  constexpr int RL = ct_last_radix(E, L), NBL = E / RL;
  cx<T> v[E];
#pragma unroll
  for (int q = 0; q < NB0; ++q)
#pragma unroll
    for (int s = 0; s < R0; ++s) v[q * R0 + s] = u[q + s * NB0];
  ct_rest<T, E, INV, PAD, L, WAVE, 1, FINE>(lds, off, es, t, v, twst);
#pragma unroll
  for (int q = 0; q < NBL; ++q)
#pragma unroll
    for (int s = 0; s < RL; ++s) u[q + s * NBL] = v[q * RL + s];
}

// ct_fft_regs in two parts, so that a caller can refill the registers it loaded the line into while the
// later stages run.
template <typename T, int E, bool INV, int L>
__device__ __forceinline__ void ct_first_stage(const cx<T>* u, cx<T>* v) {
  constexpr int R0 = ct_radix(E, L), NB0 = E / R0;
#pragma unroll
  for (int q = 0; q < NB0; ++q) {
#pragma unroll
    for (int s = 0; s < R0; ++s) v[q * R0 + s] = u[q + s * NB0];
    dft_r<T, R0, INV>(&v[q * R0]);
  }
}
template <typename T, int E, bool INV, int PAD, int L, bool WAVE>
__device__ __forceinline__ void ct_later_stages(cx<T>* lds, int off, int t, cx<T>* v, cx<T>* u, const cx<T>* twst) {
  constexpr int R0 = ct_radix(E, L);
  constexpr int RL = ct_last_radix(E, L), NBL = E / RL;
  if constexpr (R0 < L) {
    ct_sync<WAVE>();
    ct_scatter<T, E, PAD, L, 1>(lds, off, 1, t, v);
    ct_sync<WAVE>();
    ct_gather<T, E, PAD, L, R0>(lds, off, 1, t, v);
    ct_rest<T, E, INV, PAD, L, WAVE, R0>(lds, off, 1, t, v, twst);
  }
#pragma unroll
  for (int q = 0; q < NBL; ++q)
#pragma unroll
    for (int s = 0; s < RL; ++s) u[q + s * NBL] = v[q * RL + s];
}

// Same as ct_fft_regs with the input line already in LDS (filled and made visible by the caller).
template <typename T, int E, bool INV, int PAD, int L, bool WAVE, bool FINE = false>
__device__ __forceinline__ void ct_fft_lds_in(cx<T>* lds, int off, int es, int t, cx<T>* u, const cx<T>* twst) {
  constexpr int RL = ct_last_radix(E, L), NBL = E / RL;
  cx<T> v[E];
  ct_gather<T, E, PAD, L, 1>(lds, off, es, t, v);
  ct_rest<T, E, INV, PAD, L, WAVE, 1, FINE>(lds, off, es, t, v, twst);
#pragma unroll
  for (int q = 0; q < NBL; ++q)
#pragma unroll
    for (int s = 0; s < RL; ++s) u[q + s * NBL] = v[q * RL + s];
}

// Radix schedule packed 4 bits per stage (stage 0 in the low bits), nst stages.
template <typename T, int E, bool INV, int PAD = 0>
__device__ __forceinline__ void lds_fft(cx<T>* lds, int off, int es, int L, uint32_t sched, int nst, int t, int Pt,
                                        const cx<T>* __restrict__ tw, int Ntw) {
  int m = 1;
  for (int st = 0; st < nst; ++st) {
    const int r = (sched >> (4 * st)) & 15;
    if constexpr (E % 8 == 0) {
      if (r == 8) { stockham_stage<T, E, 8, INV, PAD>(lds, off, es, L, m, t, Pt, tw, Ntw); m *= 8; continue; }
    }
    if constexpr (E % 6 == 0) {
      if (r == 6) { stockham_stage<T, E, 6, INV, PAD>(lds, off, es, L, m, t, Pt, tw, Ntw); m *= 6; continue; }
    }
    if constexpr (E % 4 == 0) {
      if (r == 4) { stockham_stage<T, E, 4, INV, PAD>(lds, off, es, L, m, t, Pt, tw, Ntw); m *= 4; continue; }
    }
    if constexpr (E % 3 == 0) {
      if (r == 3) { stockham_stage<T, E, 3, INV, PAD>(lds, off, es, L, m, t, Pt, tw, Ntw); m *= 3; continue; }
    }
    if constexpr (E % 2 == 0) {
      if (r == 2) { stockham_stage<T, E, 2, INV, PAD>(lds, off, es, L, m, t, Pt, tw, Ntw); m *= 2; continue; }
    }
  }
}

// ---------------------------------------------------------------------------------------
// Real spherical harmonics in Cartesian form, no trigonometry:
//   Y_lm(u) = q_l^{|m|}(u_z) * Re/Im[(u_x + i u_y)^{|m|}]   (Re for m >= 0, Im for m < 0)
// where q_l^m = N_lm P_l^m(t) / (1 - t^2)^{m/2} obeys
//   q_m^m = c_m,  q_{m+1}^m = a_{m+1,m} t q_m^m,  q_l^m = a_lm t q_{l-1}^m - b_lm q_{l-2}^m.
// The coefficient table (built in FP64 on the host, rounded to T) is laid out per |m|:
// tab[m*STRIDE + 0] = c_m, tab[m*STRIDE + 2*(l-m)-1] = a_lm, tab[m*STRIDE + 2*(l-m)] = b_lm.
// ---------------------------------------------------------------------------------------
constexpr int YLM_LMAX = 16;
constexpr int YLM_STRIDE = 2 * YLM_LMAX + 2;

// Cartesian decomposition (Sec. 2.1, the monomial form the spherical-harmonic expansion
// replaces): a field of degree p is weighted by the monomial u_x^i u_y^j u_z^(p-i-j), its
// index packed as code = 32 i + j.  out = coef * monomial for NV directions.
__host__ __device__ constexpr int cart_code(int i, int j) { return 32 * i + j; }

// dir(v, x, y, z) gives direction v.
template <typename T, int NV, typename DIR>
__device__ __forceinline__ void monomial_eval(int p, int code, T coef, DIR dir, T* out) {
  const int i = code >> 5, j = code & 31;
#pragma unroll
  for (int v = 0; v < NV; ++v) out[v] = coef;
  // (a loop per axis: p is uniform, and one loop choosing the factor would take two selects a point and factor:
  // 384^3 FP64, l <= 4, pre-pass 4.01 -> 3.50 ms, post-pass 2.60 -> 2.32)
  int q = 0;
  auto until = [&](int end, auto pick) {
    for (; q < end; ++q) {
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        T x, y, z;
        dir(v, x, y, z);
        out[v] *= pick(x, y, z);
      }
    }
  };
  until(i, [](T x, T, T) { return x; });
  until(i + j, [](T, T y, T) { return y; });
  until(p, [](T, T, T z) { return z; });
}

// p! / (i! j! (p-i-j)!), exact in integers for p <= 16 (at most 2018016)
__device__ __forceinline__ int multinomial(int p, int code) {
  const int i = code >> 5, j = code & 31;
  long long c = 1;
  for (int q = 1; q <= i; ++q) c = c * (p - i + q) / q;          // binom(p, i)
  for (int q = 1; q <= j; ++q) c = c * (p - i - j + q) / q;      // binom(p - i, j)
  return (int)c;
}

// Running evaluation of the real Y_lm at NV points over a sequence of (l, |m|).  The state keeps
// c = c0 (ux + i uy)^am, where c0 is what the caller put there (1, or the field value the
// harmonics weight), and the recurrence pair (q_{l-1}^am, q_l^am), so that
// Y_{l,+m} c0 = q1 cr and Y_{l,-m} c0 = q1 ci (c0 real).  An entry with the same |m| and a larger l
// continues the recurrence, one with a larger |m| costs complex multiplies and a restart of the
// recurrence; |m| may only grow between resets of the state.  Control flow depends only on
// (l, |m|), which are wave-uniform.  f scales the start of the recurrence (every q is linear in it).
template <typename T, int NV> struct HRun {
  T cr[NV], ci[NV], q0[NV], q1[NV];
  int am, l;
};

// The caller sets cr, ci; this starts the state at |m| = 0 with no degree evaluated.
template <typename T, int NV> __device__ __forceinline__ void hrun_init(HRun<T, NV>& s) {
  s.am = 0;
  s.l = -1;
}

// dir(v, &x, &y, &z): the unit vector of point v.
template <typename T, int NV, typename DIR>
__device__ __forceinline__ void hrun_to(HRun<T, NV>& s, int ell, int am, T f, const T* __restrict__ tab, DIR dir) {
  if (am != s.am || s.l < am || ell < s.l) {
    for (int j = s.am; j < am; ++j) {
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        T x, y, z;
        dir(v, x, y, z);
        const T nr = s.cr[v] * x - s.ci[v] * y;
        s.ci[v] = s.cr[v] * y + s.ci[v] * x;
        s.cr[v] = nr;
      }
    }
    s.am = am;
    const T c0 = tab[am * YLM_STRIDE] * f;
#pragma unroll
    for (int v = 0; v < NV; ++v) { s.q1[v] = c0; s.q0[v] = T(0); }
    s.l = am;
  }
  const T* c = tab + am * YLM_STRIDE;
  int l = s.l + 1;
  // two degrees per iteration with the pair's roles swapped in between (no register copies)
  for (; l + 1 <= ell; l += 2) {
    const int j = l - am;
    const T a1 = c[2 * j - 1], b1 = c[2 * j];  // b = 0 for j = 1
    const T a2 = c[2 * j + 1], b2 = c[2 * j + 2];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      T x, y, z;
      dir(v, x, y, z);
      s.q0[v] = a1 * z * s.q1[v] - b1 * s.q0[v];  // q_l
      s.q1[v] = a2 * z * s.q0[v] - b2 * s.q1[v];  // q_{l+1}
    }
  }
  if (l <= ell) {
    const int j = l - am;
    const T a = c[2 * j - 1], b = c[2 * j];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      T x, y, z;
      dir(v, x, y, z);
      const T q2 = a * z * s.q1[v] - b * s.q0[v];
      s.q0[v] = s.q1[v];
      s.q1[v] = q2;
    }
  }
  s.l = ell;
}

// The same at one degree, for |m| in ascending order: q at (ell, am) from q_am^am upwards each time, so that
// between calls only the powers and q live in registers.  The caller starts with cr = 1, ci = 0, am = -1.
// TIGHT keeps the points apart (fewest registers at once).
template <typename T, int NV> struct HFixed {
  T cr[NV], ci[NV], q[NV];
  int am;
};
template <typename T, int NV, bool TIGHT, typename DIR>
__device__ __forceinline__ void hfixed_to(HFixed<T, NV>& s, int ell, int am, const T* __restrict__ tab, DIR dir) {
  if (am == s.am) return;
  for (int j = s.am < 0 ? 0 : s.am; j < am; ++j) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      T x, y, z;
      dir(v, x, y, z);
      const T nr = s.cr[v] * x - s.ci[v] * y;
      s.ci[v] = s.cr[v] * y + s.ci[v] * x;
      s.cr[v] = nr;
      if (TIGHT) __builtin_amdgcn_sched_barrier(0);
    }
  }
  s.am = am;
  const T* c = tab + am * YLM_STRIDE;
  T p[NV];
  const T c0 = c[0];
#pragma unroll
  for (int v = 0; v < NV; ++v) { s.q[v] = c0; p[v] = T(0); }
  int j = 1;
  // two degrees per iteration with the pair's roles swapped in between (no register copies)
  for (; j + 1 <= ell - am; j += 2) {
    const T a1 = c[2 * j - 1], b1 = c[2 * j];  // b = 0 for j = 1
    const T a2 = c[2 * j + 1], b2 = c[2 * j + 2];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      T x, y, z;
      dir(v, x, y, z);
      p[v] = a1 * z * s.q[v] - b1 * p[v];
      s.q[v] = a2 * z * p[v] - b2 * s.q[v];
      if (TIGHT) __builtin_amdgcn_sched_barrier(0);
    }
  }
  if (j <= ell - am) {
    const T a = c[2 * j - 1], b = c[2 * j];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      T x, y, z;
      dir(v, x, y, z);
      s.q[v] = a * z * s.q[v] - b * p[v];
      if (TIGHT) __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// Atomic add to an LDS location (native ds_add_f32 / ds_add_f64; a plain atomicAdd through a
// generic pointer may compile to a flat atomic).
template <typename T> __device__ __forceinline__ void lds_atomic_add(T* p, T v) {
  typedef __attribute__((address_space(3))) T LT;
  __hip_atomic_fetch_add((LT*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

}  // namespace pkm
