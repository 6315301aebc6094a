// z passes of the painted meshes and of the caller's transforms, reductions and the global
// line-of-sight binning (Sec. 2.1, Sec. 2.3).
//
// Data layout.  A real mesh is R[x][y][z] (z contiguous).  A half spectrum is
// H[x][y][kz] with kz in [0, N/2) contiguous: the kz = N/2 plane is never stored because
// the combined field is zero on every Nyquist plane and those modes belong to no k bin.
// x and y indices are frequencies in FFT order (j < N/2 -> j, else j - N).
//
// Passes of an estimate (each one read and one write of every element, tiles staged through LDS):
//   z pass   : real lines -> half-complex lines (length-N/2 complex FFT + split), this file.
//   column   : length-N transforms along y or x over tiles of adjacent columns (columns.hpp).
//   xcombine : forward x of both painted meshes + interlace combine + compensation +
//              Nyquist zero, then inverse x of C (columns.hpp).
//   zpre     : inverse z of G to the real field D_c, Y_lm(xhat) weighting and full-length forward z
//              of two fields at a time (fields_pre.hpp).
//   xpost    : last transform of every field of a group (along y), sum_m Y_lm(khat) B_lm,
//              product with C, and binning into per-block partial sums (fields_post.hpp).
// Both harmonic passes evaluate Y_lm for the direction turned by the plan's Frame (any
// orthogonal frame gives the same sums over m), or the monomials of the Cartesian decomposition.
//
// The z kernels take two extra template constants: NC (mesh side) and TC (lines per block).  For
// the built-in shapes of the power-of-two meshes and of 384 and 768 (radix-3 schedules) the
// launchers instantiate them with the plan's values, so all index arithmetic and the radix
// schedule fold to constants; NC = TC = 0 selects the runtime-generic path used for the other
// sizes and shapes.
#include <algorithm>

#include "fft_common.hpp"

namespace pkm {

namespace {

// ------------------------------------------------------------------------------------------
// z pass, forward (real -> half complex)
// ------------------------------------------------------------------------------------------
// LDS of the z passes: G padded lines, the W_N^j table (N entries; the splits read the
// first N/2), and on the compile-time path the per-stage table of the length-N/2 transform.
template <typename T, int E, int NC, int TC>
__global__ void __launch_bounds__(zmax_threads<T>()) k_zfwd(int n_rt, int g_rt, uint32_t sched, int nst,
                                                        const T* __restrict__ in0, const T* __restrict__ in1,
                                                        void* __restrict__ out0, void* __restrict__ out1,
                                                        const cx<T>* __restrict__ tw) {
  extern __shared__ __align__(16) unsigned char smem[];
  cx<T>* lds = reinterpret_cast<cx<T>*>(smem);
  const int n = NC > 0 ? NC : n_rt;
  const int G = TC > 0 ? TC : g_rt;
  const int nh = n >> 1;
  const int lp = zpitch(nh);
  const int pt = nh / E;
  const int bs = pt * G;
  constexpr bool WAVE = NC > 0 && NC / 2 / E <= 64;
  const T* in = blockIdx.y ? in1 : in0;
  void* out = blockIdx.y ? out1 : out0;
  const size_t line0 = (size_t)blockIdx.x * G;
  const int tid = threadIdx.x;
  cx<T>* twl = stage_twiddles<T>(lds + (size_t)G * lp, tw, n);
  cx<T>* twst = twl + n;
  if constexpr (NC > 0) ct_twiddles<T, E, NC / 2, NC>(twst, tw);
  lines_to_lds<T, E>(lds, reinterpret_cast<const cx<T>*>(in) + line0 * nh, nh, lp, bs);
  __syncthreads();
  const int t = tid % pt, g = tid / pt;
  cx<T>* line = lds + g * lp;
  if constexpr (NC > 0) {
    cx<T> u[E];
    ct_fft_lds_in<T, E, false, ZPAD, NC / 2, WAVE, true>(lds, g * lp, 1, t, u, twst);
#pragma unroll
    for (int e = 0; e < E; ++e) line[padi<ZPAD>(t + pt * e)] = u[e];
    ct_sync<WAVE>();
  } else {
    lds_fft<T, E, false, ZPAD>(lds, g * lp, 1, nh, sched, nst, t, pt, twl, n);
  }
  const size_t ob = (line0 + g) * nh;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int k = t + pt * e;
    gstore<T>((cx<T>*)out, ob + k, r2c_split<T>(line, k, nh, twl));
  }
}

// ------------------------------------------------------------------------------------------
// z pass, inverse (half complex -> real): packed half-length transform
// ------------------------------------------------------------------------------------------
template <typename T, int E, int NC, int TC>
__global__ void __launch_bounds__(zmax_threads<T>()) k_zinv(int n_rt, int g_rt, uint32_t sched, int nst,
                                                        const cx<T>* __restrict__ gin, T* __restrict__ real_out,
                                                        T scale, const cx<T>* __restrict__ tw) {
  extern __shared__ __align__(16) unsigned char smem[];
  cx<T>* lds = reinterpret_cast<cx<T>*>(smem);
  const int n = NC > 0 ? NC : n_rt;
  const int G = TC > 0 ? TC : g_rt;
  const int nh = n >> 1;
  const int lp = zpitch(nh);
  const int pt = nh / E;
  const int bs = pt * G;
  constexpr bool WAVE = NC > 0 && NC / 2 / E <= 64;
  const size_t line0 = (size_t)blockIdx.x * G;
  const int tid = threadIdx.x;
  const int t = tid % pt, g = tid / pt;
  cx<T>* line = lds + g * lp;
  cx<T>* twl = stage_twiddles<T>(lds + (size_t)G * lp, tw, n);
  cx<T>* twst = twl + n;
  if constexpr (NC > 0) ct_twiddles<T, E, NC / 2, NC>(twst, tw);
  const LineRt rt{nh, sched, nst, pt, n};
  lines_to_lds<T, E>(lds, gin + line0 * nh, nh, lp, bs);
  __syncthreads();
  cx<T> z[E];
#pragma unroll
  for (int e = 0; e < E; ++e) z[e] = c2r_split<T>(line, t + pt * e, nh, twl);
  xf_regs<T, E, true, ZPAD, NC / 2, WAVE, true>(lds, g * lp, 1, rt, t, z, twst, twl);
  cx<T>* dst = reinterpret_cast<cx<T>*>(real_out) + (line0 + g) * nh;
#pragma unroll
  for (int e = 0; e < E; ++e) gstore<T>(dst, t + pt * e, cscale<T>(z[e], scale));
}

// ------------------------------------------------------------------------------------------
// fixed-order reduction of per-block partial sums
// ------------------------------------------------------------------------------------------
// A block sums V neighbouring values: thread t the rows t / V, t / V + 256 / V, ... of value t % V.
constexpr int RED_THREADS = 256;
template <int V>
__global__ void __launch_bounds__(RED_THREADS) k_reduce(const double* __restrict__ partial, int nblocks, int nvals,
                                                        double* __restrict__ out, const int* __restrict__ map,
                                                        int accumulate) {
  __shared__ double s[RED_THREADS];
  const int v = blockIdx.x * V + threadIdx.x % V;
  double a = 0.0;
  if (v < nvals)
#pragma unroll 8
    for (int b = threadIdx.x / V; b < nblocks; b += RED_THREADS / V) a += partial[(size_t)b * nvals + v];
  s[threadIdx.x] = a;
  __syncthreads();
  for (int hh = RED_THREADS / 2; hh >= V; hh >>= 1) {
    if ((int)threadIdx.x < hh) s[threadIdx.x] += s[threadIdx.x + hh];
    __syncthreads();
  }
  if (threadIdx.x < V && v < nvals) {
    const int o = map ? map[v] : v;
    out[o] = accumulate ? out[o] + s[threadIdx.x] : s[threadIdx.x];
  }
}

// ------------------------------------------------------------------------------------------
// global line of sight (k, mu) binning of |C|^2
// ------------------------------------------------------------------------------------------
// A thread walks KMU_ROWS consecutive y at one (x, kz), its k and mu bins and their limits in registers: from
// row to row a mode mostly stays in its cell, so the search, the exact mu and the two LDS atomics are needed
// only where it leaves it, and lanes (consecutive kz, often one cell) meet less on an address; `copies` of the
// histogram spread the lanes that still do.  One thread per mode with 64-bit index divisions, a search and
// a division and square root each took 0.91 ms at 512^3 in FP32, 0.28 now (reading C alone takes 0.1).
constexpr int KMU_ROWS = 32;
// doubles between copies: 4 modulo the 32 of a row of LDS banks
__host__ __device__ constexpr int kmu_pitch(int nvals) { return (nvals + 31) / 32 * 32 + 4; }

template <typename T>
__global__ void __launch_bounds__(256) k_kmu(int n, const cx<T>* __restrict__ cin, double l0, double l1, double l2,
                      const long long* __restrict__ thr, int nb, const double* __restrict__ mue, int nmu, int copies,
                      double* __restrict__ partial) {
  extern __shared__ __align__(16) unsigned char smem[];
  double* hist = reinterpret_cast<double*>(smem);
  const int nvals = 2 * nb * nmu, pitch = kmu_pitch(nvals);
  // limits of k bin b in klim[b + 1], klim[b + 2] and of mu bin j in mlim[j + 1], mlim[j + 2], the ranges
  // below (bin -1) and above the edges included; the last mu bin has no upper limit
  double* mlim = hist + copies * pitch;
  int* klim = reinterpret_cast<int*>(mlim + nmu + 2);
  hist_zero(hist, copies * pitch);
  for (int i = threadIdx.x; i < nb + 3; i += blockDim.x) {
    const long long t = i == 0 ? INT_MIN : i == nb + 2 ? INT_MAX : thr[i - 1];
    klim[i] = (int)(t < INT_MAX ? t : INT_MAX);
  }
  for (int i = threadIdx.x; i < nmu + 2; i += blockDim.x)
    mlim[i] = i == 0 ? -__builtin_huge_val() : i == nmu + 1 ? __builtin_huge_val() : mue[i - 1];
  __syncthreads();
  const int nh = n >> 1;
  const int segs = (n + KMU_ROWS - 1) / KMU_ROWS;
  const int items = n * segs * nh;
  double* h = hist + (threadIdx.x & (copies - 1)) * pitch;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < items; i += gridDim.x * blockDim.x) {
    const int kz = i % nh, xs = i / nh, x = xs / segs, y0 = (xs - x * segs) * KMU_ROWS;
    if (x == nh) continue;
    const int fx = sfreq(x, n), n2xz = fx * fx + kz * kz;
    const double dx = __dmul_rn((double)fx, l0), dz = __dmul_rn((double)kz, l2);
    const double omega = kz == 0 ? 1.0 : 2.0;
    const cx<T>* c = cin + ((size_t)x * n + y0) * nh + kz;
    // largest index whose limit is <= v, of limits [0] = -inf .. [top] = inf
    auto find = [](const auto* lim, int top, auto v) {
      int lo = 0;
      while (top - lo > 1) { const int mid = (lo + top) >> 1; if (lim[mid] <= v) lo = mid; else top = mid; }
      return lo;
    };
    const int f0 = sfreq(y0, n), s2 = n2xz + f0 * f0;
    int kb = find(klim, nb + 2, s2) - 1, klo = klim[kb + 1], khi = klim[kb + 2];
    int mb = find(mlim, nmu + 1, fabs(dx + (double)f0 * l1 + dz) * rsqrt((double)max(s2, 1))) - 1;
    double mlo = mlim[mb + 1], mhi = mlim[mb + 2];
    int count = 0;
    double sum = 0.0;
    auto put = [&]() {
      if (count == 0) return;
      double* q = h + 2 * (kb * nmu + mb);
      lds_atomic_add<double>(q, omega * count);
      lds_atomic_add<double>(q + 1, omega * sum);
      count = 0;
      sum = 0.0;
    };
    constexpr int CH = 8;  // rows loaded ahead
    for (int r0 = 0; r0 < KMU_ROWS && y0 + r0 < n; r0 += CH) {
      cx<T> v[CH];
#pragma unroll
      for (int r = 0; r < CH; ++r) v[r] = y0 + r0 + r < n ? gload<T>(c, (size_t)(r0 + r) * nh) : mk<T>(T(0), T(0));
#pragma unroll
      for (int r = 0; r < CH; ++r) {
        const int y = y0 + r0 + r;
        const int fy = sfreq(y, n), n2 = n2xz + fy * fy;
        if (y >= n || y == nh || n2 == 0) continue;
        const double dot = fabs(__dadd_rn(__dadd_rn(dx, __dmul_rn((double)fy, l1)), dz));
        const double near = dot * rsqrt((double)n2);
        if (n2 < klo || n2 >= khi || near < mlo + 1e-12 || near >= mhi - 1e-12) {
          put();
          while (n2 >= khi) { klo = khi; khi = klim[++kb + 2]; }
          while (n2 < klo) { khi = klo; klo = klim[--kb + 1]; }
          while (near >= mhi) { mlo = mhi; mhi = mlim[++mb + 2]; }
          while (near < mlo) { mhi = mlo; mlo = mlim[--mb + 1]; }
          // The exactly rounded mu decides; further from the limits than the error of the reciprocal root
          // both give the same bin.
          if (near < mlo + 1e-12 || near >= mhi - 1e-12) {
            mb = find(mlim, nmu + 1, __ddiv_rn(dot, __dsqrt_rn((double)n2))) - 1;
            mlo = mlim[mb + 1];
            mhi = mlim[mb + 2];
          }
        }
        if (kb >= 0 && kb < nb && mb >= 0) {
          ++count;
          sum += (double)v[r].x * (double)v[r].x + (double)v[r].y * (double)v[r].y;
        }
      }
    }
    put();
  }
  __syncthreads();
  for (int v = threadIdx.x; v < nvals; v += blockDim.x) {
    double t = 0.0;
    for (int k = 0; k < copies; ++k) t += hist[k * pitch + v];
    partial[(size_t)blockIdx.x * nvals + v] = t;
  }
}

// Normalisation of reduced (k, mu) sums on the device, FP64 with explicitly rounded
// operations (the host form of the same formula gives identical bits):
// pk[i] = sum_i / (I cnt_i) - S (NaN for an empty cell), nm[i] = cnt_i.
__global__ void k_kmu_finish(const double* __restrict__ sums, int ncells, double norm_I, double shot,
                             double* __restrict__ pk, long long* __restrict__ nm) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= ncells) return;
  const double cnt = sums[2 * i];
  nm[i] = __double2ll_rn(cnt);
  pk[i] = cnt > 0.0 ? __dsub_rn(__ddiv_rn(sums[2 * i + 1], __dmul_rn(norm_I, cnt)), shot)
                    : __longlong_as_double(0x7ff8000000000000LL);
}

}  // namespace

// ------------------------------------------------------------------------------------------
// launchers
// ------------------------------------------------------------------------------------------
static int zthreads(const FftShape& fs) { return (fs.n / 2 / fs.e_z) * fs.zlines; }
// LDS sizes.  Twiddles: the generic path stages the W_N^j table (N entries); the per-stage
// table of the compile-time path has fewer than L entries for a length-L transform.
static size_t zsmem(const FftShape& fs, size_t cs) {
  return cs * ((size_t)fs.zlines * zpitch(fs.n / 2) + fs.n + fs.n / 2);
}
size_t zpass_smem_bytes(const FftShape& fs, bool fp64) {
  // (two line regions a block, as when the pre-pass shared the shape: the limit that callers' shapes are held to;
  // the z passes take one)
  const size_t cs = fp64 ? sizeof(double2) : sizeof(float2);
  return cs * (2 * (size_t)fs.zlines * zpitch(fs.n / 2) + fs.n + fs.n / 2);
}
size_t colpass_smem_bytes(const FftShape& fs, bool fp64) {
  return (fp64 ? sizeof(double2) : sizeof(float2)) * ((size_t)fs.n * (fs.tile + 1) + fs.n);
}

// Compile-time instantiations: (N, E, TC) triples matching the plan's shape rules for FP32
// and FP64 at the power-of-two sizes and at 384 and 768; anything else runs the generic
// kernels.
#define PKM_TRY(NV, EV, TV, EARG, TARG, CALL)      \
  if (fs.n == NV && (EARG) == EV && (TARG) == TV) { \
    constexpr int NC = NV, E = EV, TC = TV;         \
    CALL;                                           \
    return hipGetLastError();                       \
  }

#define PKM_TRY_Z(CALL)                        \
  PKM_TRY(64, 8, 64, fs.e_z, fs.zlines, CALL)  \
  PKM_TRY(128, 8, 32, fs.e_z, fs.zlines, CALL) \
  PKM_TRY(256, 8, 16, fs.e_z, fs.zlines, CALL) \
  PKM_TRY(512, 8, 16, fs.e_z, fs.zlines, CALL) \
  PKM_TRY(512, 8, 8, fs.e_z, fs.zlines, CALL)  \
  PKM_TRY(1024, 8, 8, fs.e_z, fs.zlines, CALL) \
  PKM_TRY(1024, 8, 4, fs.e_z, fs.zlines, CALL) \
  PKM_TRY(384, 6, 8, fs.e_z, fs.zlines, CALL)  \
  PKM_TRY(768, 6, 8, fs.e_z, fs.zlines, CALL)  \
  PKM_TRY(768, 6, 4, fs.e_z, fs.zlines, CALL)  \
  PKM_TRY(512, 4, 4, fs.e_z, fs.zlines, CALL)

template <typename T>
hipError_t launch_zfwd(const FftShape& fs, const T* in0, const T* in1, void* out0, void* out1, int nbuf,
                       const void* tw, hipStream_t s) {
  const int lines = fs.n * fs.n;
  dim3 grid(lines / fs.zlines, nbuf);
  const size_t sm = zsmem(fs, sizeof(cx<T>));
  PKM_TRY_Z((k_zfwd<T, E, NC, TC><<<grid, zthreads(fs), sm, s>>>(fs.n, fs.zlines, fs.sched_z, fs.nst_z, in0, in1,
                                                                   out0, out1, (const cx<T>*)tw)));
  PKM_DISPATCH_E(fs.e_z, (k_zfwd<T, E, 0, 0><<<grid, zthreads(fs), sm, s>>>(fs.n, fs.zlines, fs.sched_z, fs.nst_z, in0,
                                                                          in1, out0, out1, (const cx<T>*)tw)));
  return hipGetLastError();
}

template <typename T>
hipError_t launch_zinv(const FftShape& fs, const void* g_in, T* real_out, double scale, const void* tw,
                       hipStream_t s) {
  const int blocks = fs.n * fs.n / fs.zlines;
  const size_t sm = zsmem(fs, sizeof(cx<T>));
  PKM_TRY_Z((k_zinv<T, E, NC, TC><<<blocks, zthreads(fs), sm, s>>>(
      fs.n, fs.zlines, fs.sched_z, fs.nst_z, (const cx<T>*)g_in, real_out, (T)scale, (const cx<T>*)tw)));
  PKM_DISPATCH_E(fs.e_z, (k_zinv<T, E, 0, 0><<<blocks, zthreads(fs), sm, s>>>(
                             fs.n, fs.zlines, fs.sched_z, fs.nst_z, (const cx<T>*)g_in, real_out, (T)scale,
                             (const cx<T>*)tw)));
  return hipGetLastError();
}

hipError_t launch_reduce(const double* partial, int nblocks, int nvals, double* out, const int* map, int accumulate,
                         hipStream_t s) {
  if (nvals <= 0) return hipSuccess;
  // A block of one value reads 8 bytes of every row; of eight, 64, and has an eighth of the blocks (1656 rows at
  // 128^3 in FP32: 100 values 8 us with one a block, 9 with eight; 300 values 10 and 9, 1500 27 and 12; 768 rows
  // of 5000 values 38 and 13).
  if (nvals >= 256)
    k_reduce<8><<<(nvals + 7) / 8, RED_THREADS, 0, s>>>(partial, nblocks, nvals, out, map, accumulate);
  else
    k_reduce<1><<<nvals, RED_THREADS, 0, s>>>(partial, nblocks, nvals, out, map, accumulate);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_kmu(const FftShape& fs, const void* c_in, const double* los, const BinSpec& bs,
                      const double* mu_edges, int nmu, double* partial, int nblk, hipStream_t s) {
  const int pitch = kmu_pitch(2 * bs.nb * nmu);
  int copies = 8;  // within 40 KB: four blocks a CU
  while (copies > 1 && sizeof(double) * copies * (size_t)pitch > 40 * 1024) copies /= 2;
  const size_t sm = sizeof(double) * ((size_t)copies * pitch + nmu + 2) + sizeof(int) * (size_t)(bs.nb + 3);
  k_kmu<T><<<nblk, 256, sm, s>>>(fs.n, (const cx<T>*)c_in, los[0], los[1], los[2], bs.thr, bs.nb, mu_edges, nmu,
                                 copies, partial);
  return hipGetLastError();
}

hipError_t launch_kmu_finish(const double* sums, int ncells, double norm_I, double shot, double* pk, long long* nm,
                             hipStream_t s) {
  if (ncells <= 0) return hipSuccess;
  k_kmu_finish<<<(ncells + 255) / 256, 256, 0, s>>>(sums, ncells, norm_I, shot, pk, nm);
  return hipGetLastError();
}

#define PKM_INST(T)                                                                                           \
  template hipError_t launch_zfwd<T>(const FftShape&, const T*, const T*, void*, void*, int, const void*,     \
                                     hipStream_t);                                                            \
  template hipError_t launch_zinv<T>(const FftShape&, const void*, T*, double, const void*, hipStream_t);     \
  template hipError_t launch_kmu<T>(const FftShape&, const void*, const double*, const BinSpec&, const double*, \
                                    int, double*, int, hipStream_t);
PKM_INST(float)
PKM_INST(double)

}  // namespace pkm
