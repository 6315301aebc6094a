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
    ct_fft_lds_in<T, E, false, ZPAD, NC / 2, WAVE>(lds, g * lp, 1, t, u, twst);
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
  xf_regs<T, E, true, ZPAD, NC / 2, WAVE>(lds, g * lp, 1, rt, t, z, twst, twl);
  cx<T>* dst = reinterpret_cast<cx<T>*>(real_out) + (line0 + g) * nh;
#pragma unroll
  for (int e = 0; e < E; ++e) gstore<T>(dst, t + pt * e, cscale<T>(z[e], scale));
}

// ------------------------------------------------------------------------------------------
// fixed-order reduction of per-block partial sums
// ------------------------------------------------------------------------------------------
constexpr int RED_THREADS = 256;
__global__ void __launch_bounds__(RED_THREADS) k_reduce(const double* __restrict__ partial, int nblocks, int nvals,
                                                        double* __restrict__ out, const int* __restrict__ map,
                                                        int accumulate) {
  __shared__ double s[RED_THREADS];
  const int v = blockIdx.x;
  double a = 0.0;
  for (int b = threadIdx.x; b < nblocks; b += RED_THREADS) a += partial[(size_t)b * nvals + v];
  s[threadIdx.x] = a;
  __syncthreads();
  for (int hh = RED_THREADS / 2; hh > 0; hh >>= 1) {
    if ((int)threadIdx.x < hh) s[threadIdx.x] += s[threadIdx.x + hh];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const int o = map ? map[v] : v;
    out[o] = accumulate ? out[o] + s[0] : s[0];
  }
}

// ------------------------------------------------------------------------------------------
// global line of sight (k, mu) binning of |C|^2
// ------------------------------------------------------------------------------------------
template <typename T>
__global__ void k_kmu(int n, const cx<T>* __restrict__ cin, double l0, double l1, double l2,
                      const long long* __restrict__ thr, int nb, const double* __restrict__ mue, int nmu,
                      double* __restrict__ partial) {
  extern __shared__ __align__(16) unsigned char smem[];
  double* hist = reinterpret_cast<double*>(smem);
  const int nvals = 2 * nb * nmu;
  hist_zero(hist, nvals);
  __syncthreads();
  const int nh = n >> 1;
  const size_t total = (size_t)n * n * nh;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += stride) {
    const int kz = (int)(i % nh);
    const size_t xy = i / nh;
    const int y = (int)(xy % n), x = (int)(xy / n);
    if (x == nh || y == nh) continue;
    const int fx = sfreq(x, n), fy = sfreq(y, n);
    const long long n2 = (long long)fx * fx + (long long)fy * fy + (long long)kz * kz;
    if (n2 == 0) continue;
    const int kb = kbin_of(n2, thr, nb);
    if (kb < 0) continue;
    const double dot = __dadd_rn(__dadd_rn(__dmul_rn((double)fx, l0), __dmul_rn((double)fy, l1)),
                                 __dmul_rn((double)kz, l2));
    const double mu = __ddiv_rn(fabs(dot), __dsqrt_rn((double)n2));
    // mu bin: last edge <= mu -> last bin; else largest j with mue[j] <= mu
    int mb;
    if (mu >= mue[nmu]) mb = nmu - 1;
    else if (mu < mue[0]) mb = -1;
    else {
      int lo = 0, hi = nmu;
      while (hi - lo > 1) { const int mid = (lo + hi) >> 1; if (mue[mid] <= mu) lo = mid; else hi = mid; }
      mb = lo;
    }
    if (mb < 0) continue;
    const cx<T> v = cin[i];
    const double p2 = (double)v.x * (double)v.x + (double)v.y * (double)v.y;
    const double omega = (kz == 0) ? 1.0 : 2.0;
    const int cell = kb * nmu + mb;
    lds_atomic_add<double>(&hist[2 * cell], omega);
    lds_atomic_add<double>(&hist[2 * cell + 1], omega * p2);
  }
  __syncthreads();
  hist_flush(hist, 1, nvals, partial + (size_t)blockIdx.x * nvals);
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
  // shapes are held to the LDS of two line regions per block
  const size_t cs = fp64 ? sizeof(double2) : sizeof(float2);
  return cs * (2 * (size_t)fs.zlines * zpitch(fs.n / 2) + fs.n + fs.n / 2);
}
size_t colpass_smem_bytes(const FftShape& fs, bool fp64) {
  return (fp64 ? sizeof(double2) : sizeof(float2)) * ((size_t)fs.n * (fs.tile + 1) + fs.n);
}

#define PKM_DISPATCH_E(EVAL, CALL)                  \
  switch (EVAL) {                                   \
    case 4: { constexpr int E = 4; CALL; break; }   \
    case 6: { constexpr int E = 6; CALL; break; }   \
    case 8: { constexpr int E = 8; CALL; break; }   \
    case 12: { constexpr int E = 12; CALL; break; } \
    case 16: { constexpr int E = 16; CALL; break; } \
    default: return hipErrorInvalidValue;           \
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
  k_reduce<<<nvals, RED_THREADS, 0, s>>>(partial, nblocks, nvals, out, map, accumulate);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_kmu(const FftShape& fs, const void* c_in, const double* los, const BinSpec& bs,
                      const double* mu_edges, int nmu, double* partial, int nblk, hipStream_t s) {
  const size_t sm = sizeof(double) * 2 * (size_t)bs.nb * nmu;
  k_kmu<T><<<nblk, 256, sm, s>>>(fs.n, (const cx<T>*)c_in, los[0], los[1], los[2], bs.thr, bs.nb, mu_edges, nmu,
                                 partial);
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
