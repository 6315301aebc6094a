// Post-pass of the weighted fields: the last transform of every field (along y), the sum over m
// with Y_lm(khat), the product with C and the k binning.  Included by one source per precision.
#pragma once

#include <type_traits>

#include "fft_common.hpp"

namespace pkm {

namespace {

// A post-pass tile is TP whole y lines (consecutive kz) of one x plane: 256 threads.  A line wider than
// a wavefront synchronises its whole block at every radix stage, so such a tile is one line.
template <typename T, int N> struct PostShape {
  static constexpr int E = line_e<T>(N);
  static constexpr int PT = N / E;
  static constexpr bool WAVE = 64 % PT == 0;  // a line lies inside one wavefront
  static constexpr int lines() {
    if (PT > 64) return 1;
    int tp = (N <= 128 ? 64 : 256) / PT;
    while (tp & (tp - 1)) tp &= tp - 1;
    return tp < 16 ? tp : 16;
  }
  static constexpr int TP = lines();
  static constexpr int THREADS = PT * TP;
  static constexpr int PITCH = ct_line_slots<T, E, N>();
  static constexpr int CPITCH = N + 1;  // the tile's C, [line][y]
  // LDS of a block of `tp` lines without histograms and thresholds
  __host__ __device__ static constexpr size_t smem(int tp) {
    return sizeof(cx<T>) * ((size_t)tp * (PITCH + CPITCH) + twst_size<E, N>());
  }
  // Sides to 128 leave a few wavefronts per SIMD for the whole grid: latency bounds them, so they keep
  // the points' chains interleaved; longer ones keep the registers low.
  static constexpr bool TIGHT = N > 128;
  // wavefronts per SIMD the registers are bounded for
  static constexpr int MINW = sizeof(T) == 4 ? (E <= 8 && N > 128 ? 3 : 2) : (E <= 8 && N > 128 ? 2 : 1);
  // Merge the l = 0 values of neighbouring lanes before their atomics: 512^3 1.61 -> 1.33 ms (merging the values of
  // the other slots as well: 1.36).  12 and 16 points a thread spill more for it (432^3 1.57 -> 1.64, 1024^3 21.0 ->
  // 22.8 ms).
  static constexpr bool MERGE = E <= 8;
  // persistent blocks of `tp` lines per CU (threads the registers above leave room for)
  static constexpr int per_cu(int tp) {
    const int wide = (PT * tp + 63) / 64 * 64;
    return 256 * MINW / wide > 0 ? 256 * MINW / wide : 1;
  }
};

// Tiles of a persistent post-pass block.  When the grid is a multiple of 8, block b (dispatched to XCD
// b mod 8) walks a contiguous eighth of the tiles, so the blocks of one XCD work on neighbouring tiles at the
// same time; a block may find none left.
struct TileWalk {
  int first, step, end, chunk0;
  __device__ TileWalk(int nt) {
    const int G = gridDim.x, b = blockIdx.x;
    if (G % 8 == 0) {
      const int x = b % 8;
      chunk0 = (int)((long long)nt * x / 8);
      first = b / 8;
      step = G / 8;
      end = (int)((long long)nt * (x + 1) / 8) - chunk0;
    } else {
      chunk0 = 0;
      first = b;
      step = G;
      end = nt;
    }
  }
  __device__ int tile(int j) const { return chunk0 + j; }
};

// k bins of E elements at once: all searches step together, so their reads of the thresholds
// overlap.  -1 for modes outside [thr[0], thr[nb]).
template <int E> __device__ __forceinline__ void kbins(const int* thr, int nb, const int* n2, int* bin) {
  int hi[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    bin[e] = 0;
    hi[e] = nb;
  }
  for (int w = nb; w > 1; w = (w + 1) >> 1) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int mid = (bin[e] + hi[e]) >> 1;
      const bool up = thr[mid] <= n2[e];
      bin[e] = up ? mid : bin[e];
      hi[e] = up ? hi[e] : mid;
    }
  }
  const int lo = thr[0], top = thr[nb];
#pragma unroll
  for (int e = 0; e < E; ++e) bin[e] = n2[e] >= lo && n2[e] < top ? bin[e] : -1;
}

// Neighbouring lanes hold neighbouring y, whose modes are often in one bin, and their atomics on it are done
// one after the other.  Lanes that are partners in a quad (CTRL: the quad permutation, 0xB1 and 0x4E pair lanes 1
// and 2 apart) and share a bin add their values first: the lower lane takes the sum, the upper one no bin.
template <int CTRL> __device__ __forceinline__ int quad_from(int v) {
  return __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true);
}
template <int CTRL> __device__ __forceinline__ double quad_from(double v) {
  return __hiloint2double(quad_from<CTRL>(__double2hiint(v)), quad_from<CTRL>(__double2loint(v)));
}
template <int CTRL, typename... V> __device__ __forceinline__ void quad_merge(int& bin, V&... v) {
  const bool same = quad_from<CTRL>(bin) == bin;
  ((v += same ? quad_from<CTRL>(v) : V(0)), ...);
  if (same && (threadIdx.x & (CTRL == 0xB1 ? 1 : 2))) bin = 0xffff;
}

// ------------------------------------------------------------------------------------------
// The post-pass.  Thread (t, c) transforms line kz0 + c and holds y = t + PT e, the transform's own
// register layout, so each line is loaded straight into registers (whole contiguous lines, the
// next one prefetched during the current one) and LDS carries only the stage exchanges, the tile's C and
// the histograms.  Lines come slot by slot (a slot is one multipole): one complex accumulator per
// element holds sum_m Y_lm(khat) B_lm of the current slot and is folded against C into the FP64
// bins after the slot's last line.  Only tiles that hold modes below the last k edge are listed
// (`tiles`, x and kz0 packed).  Registers bound the wavefronts in flight: the unit vectors are rebuilt
// from the mode numbers (linear in fy) where the recurrence needs them.
// 512^3, 14 fields of l <= 4: 2.64 ms as packed half lines over every mode, 1.33 now (4.5 TB/s; the rest is
// the harmonics and the exchanges); 432^3, 44 fields of l <= 8 in groups of 16: 5.85 -> 1.57 ms a group (a kernel of
// run-time lengths before); 1024^3 18.9 -> 14.6; 384^3 FP64 2.60 -> 1.5; 256^3 337 -> 221 us; 128^3, 152 fields of
// l <= 16: 297 -> 248 us; 64^3 FP64, l <= 4: 31 -> 23 us.
// ALL: blocks of all TP lines.  Else of as many (fewer) as the launch has threads for: requests whose
// histograms leave no room for TP lines in the LDS of a CU.
// ------------------------------------------------------------------------------------------
template <typename T, int N, bool CART, bool ALL>
__global__ void __launch_bounds__((PostShape<T, N>::THREADS), (PostShape<T, N>::MINW))
    k_xpost(int nrecs, const FieldRec* __restrict__ recs, int nslots, int with_l0,
            double kf, const cx<T>* __restrict__ cin, const T* __restrict__ ytab, const int* __restrict__ thr,
            int nb, int copies, int turns, int thr_lds, double* __restrict__ partial,
            const cx<T>* __restrict__ tw, Frame frm, const unsigned* __restrict__ tiles, int ntiles) {
  using S = PostShape<T, N>;
  constexpr int E = S::E, PT = S::PT, nh = N / 2;
  // (constants of the front end where ALL: the offset left to the optimiser costs the 12-point kernels 4 scalar
  // registers more to spill, 576^3 FP32 post-pass 5.59 -> 5.83 ms)
  const auto TP = [] {
    if constexpr (ALL) return std::integral_constant<int, S::TP>{};
    else return (int)blockDim.x / PT;
  }();
  const auto line_lds = [] {
    if constexpr (ALL) return std::integral_constant<size_t, S::smem(S::TP)>{};
    else return S::smem((int)blockDim.x / PT);
  }();
  extern __shared__ __align__(16) unsigned char smem[];
  cx<T>* exch = reinterpret_cast<cx<T>*>(smem);
  cx<T>* cst = exch + TP * S::PITCH;
  cx<T>* twst = cst + TP * S::CPITCH;
  double* hist = reinterpret_cast<double*>(smem + line_lds);
  const int l0rows = with_l0 ? 3 : 0;
  const int nvals = (l0rows + nslots) * nb;
  int* thr_l = reinterpret_cast<int*>(hist + (size_t)copies * nvals);
  hist_zero(hist, copies * nvals);
  if (thr_lds)
    for (int i = threadIdx.x; i <= nb; i += blockDim.x) thr_l[i] = thr[i];
  ct_twiddles<T, E, N, N>(twst, tw);
  __syncthreads();
  const int tid = threadIdx.x;
  const int c = tid / PT, t = tid % PT;
  // histogram of this wavefront: waves that share a copy add in turn, between barriers, so the sums
  // are taken in one order whatever the number of copies
  const int wave = tid >> 6;
  double* h = hist + (wave / turns) * nvals;
  const int my_turn = wave % turns;
  const int* thr_p = thr_lds ? thr_l : thr;
  constexpr size_t plane = field_plane_stride<T>(N);
  const TileWalk walk(ntiles);
  cx<T> nxt[E];
  // (lines past the last kz of a partial tile repeat that kz; their modes are in no bin)
  auto fetch = [&](unsigned tl, const void* buf) {
    const int kz0 = (int)(tl & 0xffff);
    const cx<T>* b = reinterpret_cast<const cx<T>*>(buf) + (size_t)kz0 * plane + (size_t)(tl >> 16) * N;
    const int cc = (ALL && nh % S::TP == 0) || kz0 + c < nh ? c : nh - 1 - kz0;
    const unsigned off = (unsigned)(cc * plane + t);
#pragma unroll
    for (int e = 0; e < E; ++e) nxt[e] = gload32<T>(b, off + (unsigned)(PT * e));
  };
  int j = walk.first;
  // the records run two ahead: the line of the next one is fetched as soon as the registers of this one's
  // are free, and the one after it is read meanwhile (tables are padded by a copy of the first record)
  FieldRec rec = recs[0], nx = recs[1];
  if (j < walk.end && nslots > 0) fetch(tiles[walk.tile(j)], rec.p0);
  for (; j < walk.end; j += walk.step) {
    const unsigned tl = tiles[walk.tile(j)];
    const int x = (int)(tl >> 16), kz0 = (int)(tl & 0xffff), kz = kz0 + c;
    // C of the tile: TP consecutive kz per y row, kept in LDS for the whole tile
    __syncthreads();  // the previous tile's reads of it are done
#pragma unroll
    for (int q = 0; q < E; ++q) {
      const int i = tid + q * (PT * TP), y = i / TP, cc = i % TP;
      const int k = kz0 + cc < nh ? kz0 + cc : nh - 1;
      cst[cc * S::CPITCH + y] = gload32<T>(cin + (size_t)x * (N * nh), (unsigned)(y * nh + k));
    }
    const int fx = sfreq(x, N);
    T ki[E];
    unsigned binp[(E + 1) / 2];  // 16 bits each, 0xffff: none
    {
      int n2[E], bin[E];
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int y = t + PT * e;
        const int fy = sfreq(y, N);
        n2[e] = fx * fx + fy * fy + kz * kz;
        ki[e] = n2[e] > 0 ? T(1) / sqrt((T)n2[e]) : T(0);
        if (y == nh || kz >= nh || n2[e] == 0) n2[e] = -1;  // (in no bin: the thresholds are >= 0)
      }
      kbins<E>(thr_p, nb, n2, bin);
#pragma unroll
      for (int e = 0; e < E; e += 2)
        binp[e / 2] = (unsigned)(bin[e] & 0xffff) | (e + 1 < E ? (unsigned)bin[e + 1] << 16 : 0u);
    }
    auto bin_of = [&](int e) { return (int)((binp[e / 2] >> (16 * (e & 1))) & 0xffff); };
    // Turned unit wave vectors: the mode (fx, fy, kz) turned by the frame is linear in fy, so one fused
    // add and a product by 1 / |k| give a component.  Its part in fx and kz is formed in FP64 and rounded
    // once, and fy is exact: splitting fy between the two (t here, PT e there) would cancel at small |k|
    // and cost an order of magnitude at l = 16.
    const T a0 = (T)(frm.r[0] * fx + frm.r[2] * kz), a1 = (T)(frm.r[3] * fx + frm.r[5] * kz),
            a2 = (T)(frm.r[6] * fx + frm.r[8] * kz);
    const T tf = (T)t;
    auto dir = [&](int e, T& vx, T& vy, T& vz) {
      const T fy = (S::TIGHT ? fresh(tf) : tf) + (T)(PT * e - (e >= E / 2 ? N : 0));
      vx = (a0 + frm.at<T>(1) * fy) * ki[e];
      vy = (a1 + frm.at<T>(4) * fy) * ki[e];
      vz = (a2 + frm.at<T>(7) * fy) * ki[e];
    };
    __syncthreads();  // C staged
    const unsigned tl_next = tiles[walk.tile(j + walk.step < walk.end ? j + walk.step : j)];
    for (int li = 0, slot = 0; slot < nslots || (slot == 0 && with_l0); ++slot) {
      cx<T> acc[E];
      HFixed<T, E> hr;
      hr.am = -1;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        acc[e] = mk<T>(T(0), T(0));
        hr.cr[e] = T(1);
        hr.ci[e] = T(0);
      }
      const int l_slot = rec.l;
      for (; li < nrecs && rec.slot == slot; ++li) {
        const int l = rec.l, m = rec.m;
        cx<T> u[E], v[E];
        ct_first_stage<T, E, false, N>(nxt, v);
        fetch(li + 1 < nrecs ? tl : tl_next, nx.p0);
        rec = nx;
        nx = recs[li + 2 < nrecs ? li + 2 : li + 2 - nrecs < nrecs ? li + 2 - nrecs : 0];
        ct_later_stages<T, E, false, AUTO_PAD, N, S::WAVE>(exch, c * S::PITCH, t, v, u, twst);
        __builtin_amdgcn_sched_barrier(0);  // (the last stage's inputs and twiddles are not held across the harmonics)
        T y[E];
        if constexpr (!CART) {
          hfixed_to<T, E, S::TIGHT>(hr, l, m < 0 ? -m : m, ytab, dir);
          if (m < 0) {
#pragma unroll
            for (int e = 0; e < E; ++e) y[e] = hr.q[e] * hr.ci[e];
          } else {
#pragma unroll
            for (int e = 0; e < E; ++e) y[e] = hr.q[e] * hr.cr[e];
          }
        } else {
          monomial_eval<T, E>(l, m, (T)multinomial(l, m), dir, y);
        }
#pragma unroll
        for (int e = 0; e < E; ++e) acc[e] = mk<T>(acc[e].x + y[e] * u[e].x, acc[e].y + y[e] * u[e].y);
      }
      // even l: Re[C conj acc]; odd l (spherical basis only): Im[C conj acc], the part of
      // the shell average that survives when a mode and its mirror are summed
      const bool odd = !CART && (l_slot & 1);
      const bool l0 = with_l0 && slot == 0;
      double* hs = h + (l0rows + slot) * nb;
      // Hermitian weight; the spherical sum also carries the 4 pi of the addition theorem
      const double w = kz == 0 ? 1.0 : 2.0, wfold = w * (CART ? 1.0 : FOUR_PI);
      for (int tr = 0; tr < turns; ++tr) {
        if (tr == my_turn) {
#pragma unroll
          for (int e = 0; e < E; ++e) {
            if constexpr (S::TIGHT) __builtin_amdgcn_sched_barrier(0);
            int b = bin_of(e);
            if constexpr (!S::MERGE)
              if (b == 0xffff) continue;
            const cx<T> cv = cst[c * S::CPITCH + t + PT * e];
            const double cr = cv.x, ci = cv.y;
            auto folded = [&]() {
              const double ar = acc[e].x, ai = acc[e].y;
              return wfold * (odd ? ci * ar - cr * ai : cr * ar + ci * ai);
            };
            auto k_sum = [&]() {
              const int fy = t + PT * e - (e >= E / 2 ? N : 0);
              return w * kf * sqrt((double)(fx * fx + fy * fy + kz * kz));
            };
            if (S::MERGE && l0) {  // (lanes with no bin stay: their neighbours read them)
              int cnt = kz == 0 ? 1 : 2;
              double v = folded(), ks = k_sum(), p0 = w * (cr * cr + ci * ci);
              quad_merge<0xB1>(b, v, cnt, ks, p0);
              quad_merge<0x4E>(b, v, cnt, ks, p0);
              if (b == 0xffff) continue;
              if (nslots > 0) lds_atomic_add<double>(&hs[b], v);
              lds_atomic_add<double>(&h[b], (double)cnt);
              lds_atomic_add<double>(&h[nb + b], ks);
              lds_atomic_add<double>(&h[2 * nb + b], p0);
              continue;
            }
            if (b == 0xffff) continue;
            if (nslots > 0) lds_atomic_add<double>(&hs[b], folded());
            if (l0) {
              lds_atomic_add<double>(&h[b], w);
              lds_atomic_add<double>(&h[nb + b], k_sum());
              lds_atomic_add<double>(&h[2 * nb + b], w * (cr * cr + ci * ci));
            }
          }
        }
        if (turns > 1) __syncthreads();
      }
    }
  }
  __syncthreads();
  hist_flush(hist, copies, nvals, partial + (size_t)blockIdx.x * nvals);
}

// One launch of the post-pass of a side with blocks of `lines` lines: ALL blocks of all its lines, or fewer.
template <typename T, int N, bool ALL>
void post_run(int lines, int nrecs, const FieldRec* recs_dev, int nslots, int with_l0, const void* c_in,
              const void* ytab, const BinSpec& bs, double kf, double* partial, int nblocks, const void* tw,
              const Frame& frame, int basis, const unsigned* tiles_dev, int ntiles, hipStream_t s) {
  using S = PostShape<T, N>;
  const int nvals = ((with_l0 ? 3 : 0) + nslots) * bs.nb;
  const size_t sm = S::smem(lines) + sizeof(double) * (size_t)bs.hist_copies * nvals +
                    (bs.thr_lds ? sizeof(int) * (size_t)(bs.nb + 1) : 0);
  auto run = [&](auto kern) {
    kern<<<nblocks, S::PT * lines, sm, s>>>(nrecs, recs_dev, nslots, with_l0, kf, (const cx<T>*)c_in, (const T*)ytab,
                                            bs.thr32, bs.nb, bs.hist_copies, bs.turns, bs.thr_lds, partial,
                                            (const cx<T>*)tw, frame, tiles_dev, ntiles);
  };
  if (basis == 1) run(k_xpost<T, N, true, ALL>); else run(k_xpost<T, N, false, ALL>);
}

}  // namespace

#define PKM_POST_ARGS                                                                                        \
  lines, nrecs, recs_dev, nslots, with_l0, c_in, ytab, bs, kf, partial, nblocks, tw, frame, basis, tiles_dev, ntiles, s

template <typename T> bool post_geometry(int n, int lines, PostGeometry* g) {
#define PKM_POST_SIDE(NV)                                                                                    \
  case NV: {                                                                                                 \
    using S = PostShape<T, NV>;                                                                              \
    const int tp = lines > 0 && lines < S::TP ? lines : S::TP;                                               \
    *g = PostGeometry{tp, S::PT * tp, S::per_cu(tp), S::smem(tp)};                                           \
    return true;                                                                                             \
  }
  switch (n) { PKM_FOR_SIDES(PKM_POST_SIDE) default: return false; }
#undef PKM_POST_SIDE
}

template <typename T>
hipError_t launch_xpost(const FftShape& fs, int lines, int nrecs, const FieldRec* recs_dev, int nslots, int with_l0,
                        const void* c_in, const void* ytab, const BinSpec& bs, double kf,
                        double* partial, int nblocks, const void* tw, const Frame& frame, int basis,
                        const unsigned* tiles_dev, int ntiles, hipStream_t s) {
  if (nslots < 0 || nblocks < 1 || lines < 1) return hipErrorInvalidValue;
#define PKM_POST_SIDE(NV)                                                                                    \
  case NV: {                                                                                                 \
    constexpr int TP = PostShape<T, NV>::TP;                                                                 \
    if (lines < TP) return launch_xpost_few<T>(fs, PKM_POST_ARGS);                                           \
    if (lines > TP) return hipErrorInvalidValue;                                                             \
    post_run<T, NV, true>(PKM_POST_ARGS);                                                                    \
    break;                                                                                                   \
  }
  switch (fs.n) { PKM_FOR_SIDES(PKM_POST_SIDE) default: return hipErrorInvalidValue; }
#undef PKM_POST_SIDE
  return hipGetLastError();
}

// Blocks of fewer lines than the side's own (checked by launch_xpost); sources of their own, which compile
// beside the others.
template <typename T>
hipError_t launch_xpost_few(const FftShape& fs, int lines, int nrecs, const FieldRec* recs_dev, int nslots,
                            int with_l0, const void* c_in, const void* ytab, const BinSpec& bs, double kf,
                            double* partial, int nblocks, const void* tw, const Frame& frame, int basis,
                            const unsigned* tiles_dev, int ntiles, hipStream_t s) {
#define PKM_POST_SIDE(NV)                                                                                    \
  case NV:                                                                                                   \
    if constexpr (PostShape<T, NV>::TP > 1) {                                                                \
      post_run<T, NV, false>(PKM_POST_ARGS);                                                                 \
      return hipGetLastError();                                                                              \
    }                                                                                                        \
    return hipErrorInvalidValue;
  switch (fs.n) { PKM_FOR_SIDES(PKM_POST_SIDE) default: return hipErrorInvalidValue; }
#undef PKM_POST_SIDE
}

#define PKM_POST_PARAMS                                                                                       \
  const FftShape&, int, int, const FieldRec*, int, int, const void*, const void*, const BinSpec&, double,     \
      double*, int, const void*, const Frame&, int, const unsigned*, int, hipStream_t
#define PKM_POST_INST(T)                                                                                      \
  extern template hipError_t launch_xpost_few<T>(PKM_POST_PARAMS);                                            \
  template bool post_geometry<T>(int, int, PostGeometry*);                                                    \
  template hipError_t launch_xpost<T>(PKM_POST_PARAMS);
#define PKM_POST_FEW_INST(T) template hipError_t launch_xpost_few<T>(PKM_POST_PARAMS);

}  // namespace pkm
