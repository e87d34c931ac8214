// General pencil-pass kernels of the spectral Poisson solve (gfx950).
//
// One launch transforms every pencil (1D line) of a field along one axis.  A
// workgroup of 256 threads takes a tile of P pencils: it loads the tile from
// HBM with unit-stride runs (along the pencil when the pencil is contiguous,
// across pencils otherwise) straight into the complex FFT input in LDS, runs a
// mixed-radix Stockham FFT there (radices 2..16 in FP32, 2..10 in FP64, any
// larger prime by a stage of its own) and writes the result with unit-stride
// runs again.  The strides of the input and output sides are independent, so
// a pass can also transpose.
//
// What bounds them: at the sizes of one solve (1 to 16 million points, resident
// in the 256 MB cache) a pass is one or two rounds of workgroups, each a chain
// of load, stages (two barriers and a trip through LDS each) and store, so its
// time is the length of that chain, not bytes or flops.  Hence few stages of
// large radix, no run-time divisions, no raw copy of the tile beside the FFT
// input, LDS rows that every access pattern takes without bank conflicts, and
// tiles narrowed where there are fewer of them than CUs.  Measured on one
// MI355X, whole solves, against stages of radix <= 8 with a raw tile and direct
// prime sums: 120 x 96 x 80 FP64 Neumann 123 -> 83 us, 96 x 80 x 100 FP64 free
// space 139 -> 97 us, 128^3 FP32 semi-unbounded gradient 381 -> 239 us, 127^3
// FP32 periodic (a prime) 971 -> 111 us.
//
// The sandwich pass (last axis of the forward transform) loads, transforms,
// multiplies by the spectral multiplier (Table 1 eigenvalues or the Green's
// spectrum, Section 2.2 step 2), applies the spectral derivative (step 3,
// eq. ft_sd), transforms back and stores, so the spectrum of that axis never
// leaves LDS.
#include <algorithm>
#include <mutex>

#include "hp_device.hpp"
#include "hp_faces.hpp"
#include "hp_gendft.hpp"
#include "hp_internal.hpp"
#include "hp_wavefft.hpp"

namespace hp {

// ----------------------------------------------------------- index helpers
// Quotients by run-time divisors d <= 8192 of small numbers (x d < 2^32), one
// multiply instead of the division sequence: m = ceil(2^32 / d).
__device__ __forceinline__ unsigned div_magic(int d) { return 0xffffffffu / (unsigned)d + 1u; }
__device__ __forceinline__ int div_by(int x, int d, unsigned m) {
  return d > 1 ? (int)__umulhi((unsigned)x, m) : x;
}

// ------------------------------------------------------------- LDS tile
// The FFT data of a tile: element m of transform f (a pencil pair, or a
// complex pencil) at row m, column f.  Rows hold nf = 2^lg transforms and, from
// two on, one pad element: consecutive lanes take consecutive columns, so
// every access of a stage is a set of whole rows whatever its stride, and the
// accesses along m (rows read one column at a time) step over all banks.
// Pointers carry the LDS address space, so that functions that are not inlined
// use LDS instructions and not generic ones.
#define HP_LDS __attribute__((address_space(3)))
#define HP_GLB __attribute__((address_space(1)))
template <typename T>
struct V2 {
  typedef T t __attribute__((ext_vector_type(2)));
  // the same in global memory, aligned to one element only
  typedef T u __attribute__((ext_vector_type(2), aligned(sizeof(T))));
};
template <typename T>
using GC = const HP_GLB typename V2<T>::t*;  // complex table or field in global memory
template <typename T>
__device__ __forceinline__ GC<T> glb(const void* p) {
  return (GC<T>)p;
}
template <typename T>
__device__ __forceinline__ C2<T> ldc(GC<T> p, long long i) {
  const typename V2<T>::t v = p[i];
  return {v.x, v.y};
}
template <typename T>
__device__ __forceinline__ void stc(void* p, long long i, C2<T> c) {
  typename V2<T>::t v;
  v.x = c.re;
  v.y = c.im;
  ((HP_GLB typename V2<T>::t*)p)[i] = v;
}
template <typename T>
struct LTile {
  HP_LDS typename V2<T>::t* z;
  int S, lg;
  __device__ __forceinline__ C2<T> get(int i) const {
    const typename V2<T>::t v = z[i];
    return {v.x, v.y};
  }
  __device__ __forceinline__ void put(int i, C2<T> c) const {
    typename V2<T>::t v;
    v.x = c.re;
    v.y = c.im;
    z[i] = v;
  }
};
__host__ __device__ constexpr int tile_row(int nf, bool pad) { return nf > 1 && pad ? nf + 1 : nf; }

template <typename T>
__device__ __forceinline__ LTile<T> lds_tile(unsigned char* smem, int nf, int L, int index, bool pad = true) {
  LTile<T> z;
  z.lg = 31 - __builtin_clz((unsigned)nf);
  z.S = tile_row(nf, pad);
  z.z = (HP_LDS typename V2<T>::t*)smem + (size_t)index * L * z.S;
  return z;
}

// ------------------------------------------------------------- Stockham FFT
// Kernel modes.  Complex elements per thread of one stage: 16 (FP32) / 8
// (FP64), fewer registers and more resident waves, or (GM_BIG) 32 / 16 for
// tiles of long transforms.  GM_SMALL has no prime stage, whose accumulators
// would set the registers of every kernel that holds it (FP64: 184 against
// 82, two resident waves per SIMD against five).
enum GenMode : int { GM_SMALL = 0, GM_PRIME = 1, GM_BIG = 2 };
template <typename T, int MODE>
struct Maxe {
  static constexpr int v = (MODE == GM_BIG ? 32 : 16) / (sizeof(T) == 8 ? 2 : 1);
};

// Butterflies of radix R a thread holds: rounded down in the smaller budget
// (its registers are the kernel's), up in the larger one (every length fits).
template <typename T>
__host__ __device__ constexpr int stage_slots(int R, int maxe) {
  return maxe > (sizeof(T) == 4 ? 16 : 8) ? (maxe + R - 1) / R : (maxe / R > 1 ? maxe / R : 1);
}

// One radix-R stage over the nf transforms of a tile.  Butterfly j of a
// transform reads x[j + t L/R] (t < R), twiddles input t by W_{Ns R}^{t k}
// (k = j mod Ns; no twiddles in the first stage, Ns = 1), and writes output t'
// to (j / Ns) Ns R + k + t' Ns.  All reads finish (barrier) before any write,
// so the stage is in place.
template <typename T, int R, int MAXE>
__device__ __attribute__((noinline)) void fft_stage(LTile<T> Z, int L, int Ns, GC<T> tw) {
  constexpr int MB = stage_slots<T>(R, MAXE);
  const int nbl = L / R;
  const int total = nbl << Z.lg;
  const int mask = (1 << Z.lg) - 1;
  const unsigned mN = div_magic(Ns);
  const int twstep = nbl / Ns;
  const int rstep = nbl * Z.S, wstep = Ns * Z.S;
  C2<T> v[MB][R];
  int ob[MB];
#pragma unroll
  for (int b = 0; b < MB; ++b) {
    const int idx = threadIdx.x + b * kThreads;
    ob[b] = -1;
    if (idx < total) {
      const int f = idx & mask, j = idx >> Z.lg;
      const int k = j - div_by(j, Ns, mN) * Ns;
      const int src = j * Z.S + f;
#pragma unroll
      for (int t = 0; t < R; ++t) v[b][t] = Z.get(src + t * rstep);
      if (Ns > 1) {
        const int e = k * twstep;
#pragma unroll
        for (int t = 1; t < R; ++t) v[b][t] = cmul(v[b][t], ldc<T>(tw, t * e));
      }
      ob[b] = ((j - k) * R + k) * Z.S + f;
    }
  }
  __syncthreads();
#pragma unroll
  for (int b = 0; b < MB; ++b) {
    if (ob[b] >= 0) {
      dft_any<T, R>(v[b]);
#pragma unroll
      for (int t = 0; t < R; ++t) Z.put(ob[b] + t * wstep, v[b][t]);
    }
  }
  __syncthreads();
}

// One stage of a prime radix R that has no register DFT, by the even and odd
// parts of the butterfly's inputs (s_t = x_t + x_{R-t}, d_t = x_t - x_{R-t}
// after the stage twiddles):
//   X_u, X_{R-u} = x_0 + sum_t s_t cos(2 pi t u / R) -+ i sum_t d_t sin(2 pi t u / R),
// t = 1 .. h = (R - 1) / 2, a quarter of the products of the direct sum and
// half its terms per accumulator.  First the parts replace the inputs in
// place (each pair belongs to one thread); then a thread accumulates kPrimeB
// values u of one butterfly, so one read of s_t and d_t serves 4 kPrimeB
// multiply-adds, the factors coming from a table of R values in LDS; the
// outputs are written after all reads.
constexpr int kPrimeB = 4;
// TABLE false: the factors come from the twiddle table instead (tiles that
// leave no LDS for them: coupled fields of lengths above 4096).
template <typename T, int MAXE, bool TABLE>
__device__ __attribute__((noinline)) void fft_stage_prime(LTile<T> Z, HP_LDS typename V2<T>::t* wR,
                                                          int L, int R, int Ns, GC<T> tw) {
  // items per thread: blocks of kPrimeB outputs u of one butterfly (the last
  // block of a butterfly may be partly unused: at most 1.5 slots per element)
  constexpr int MBP = MAXE * 3 / 16 > 2 ? MAXE * 3 / 16 : 2;
  const int nbl = L / R, h = (R - 1) / 2;
  const int mask = (1 << Z.lg) - 1;
  const int twstep = nbl / Ns;
  const int rstep = nbl * Z.S;
  const unsigned mN = div_magic(Ns), mB = div_magic(nbl);
  if constexpr (TABLE)
    for (int e = threadIdx.x; e < R; e += kThreads) {
      const C2<T> w = ldc<T>(tw, e * nbl);
      typename V2<T>::t c;
      c.x = w.re;
      c.y = -w.im;  // (cos, sin) of 2 pi e / R
      wR[e] = c;
    }
  const int total1 = (nbl * h) << Z.lg;
  for (int idx = threadIdx.x; idx < total1; idx += kThreads) {
    const int f = idx & mask, r = idx >> Z.lg;
    const int t1 = div_by(r, nbl, mB), j = r - t1 * nbl;
    const int t = t1 + 1;
    const int ia = j * Z.S + f + t * rstep, ib = j * Z.S + f + (R - t) * rstep;
    C2<T> x = Z.get(ia), y = Z.get(ib);
    if (Ns > 1) {
      const int e = (j - div_by(j, Ns, mN) * Ns) * twstep;
      x = cmul(x, ldc<T>(tw, t * e));
      y = cmul(y, ldc<T>(tw, (R - t) * e));
    }
    Z.put(ia, cadd(x, y));
    Z.put(ib, csub(x, y));
  }
  __syncthreads();
  const int nb = (h + 1 + kPrimeB - 1) / kPrimeB;
  const int total = (nbl * nb) << Z.lg;
  C2<T> C[MBP][kPrimeB], D[MBP][kPrimeB];
  int ob[MBP], u0[MBP];
#pragma unroll
  for (int b = 0; b < MBP; ++b) {
    const int idx = threadIdx.x + b * kThreads;
    ob[b] = -1;
    u0[b] = 0;
    if (idx < total) {
      const int f = idx & mask, r = idx >> Z.lg;
      const int ub = div_by(r, nbl, mB), j = r - ub * nbl;
      const int k = j - div_by(j, Ns, mN) * Ns;
      u0[b] = ub * kPrimeB;
      ob[b] = ((j - k) * R + k) * Z.S + f;
      const int src = j * Z.S + f;
      const C2<T> x0 = Z.get(src);
      unsigned e[kPrimeB];
#pragma unroll
      for (int q = 0; q < kPrimeB; ++q) {
        C[b][q] = x0;
        D[b][q] = {(T)0, (T)0};
        e[q] = 0;
      }
      int ia = src, ib = src + R * rstep;
#pragma unroll 1
      for (int t = 1; t <= h; ++t) {
        ia += rstep;
        ib -= rstep;
        const C2<T> s = Z.get(ia), d = Z.get(ib);
#pragma unroll
        for (int q = 0; q < kPrimeB; ++q) {
          // t u mod R, stepped by u <= h + kPrimeB - 1 < R
          e[q] += (unsigned)(u0[b] + q);
          e[q] = min(e[q], e[q] - (unsigned)R);
          typename V2<T>::t w;
          if constexpr (TABLE) {
            w = wR[e[q]];
          } else {
            w = tw[e[q] * nbl];
            w.y = -w.y;
          }
          C[b][q].re += s.re * w.x;
          C[b][q].im += s.im * w.x;
          D[b][q].re += d.re * w.y;
          D[b][q].im += d.im * w.y;
        }
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int b = 0; b < MBP; ++b) {
    if (ob[b] >= 0) {
#pragma unroll
      for (int q = 0; q < kPrimeB; ++q) {
        const int u = u0[b] + q;
        if (u > h) continue;
        const C2<T> c = C[b][q], d = D[b][q];
        Z.put(ob[b] + u * Ns * Z.S, {c.re + d.im, c.im - d.re});
        if (u > 0) Z.put(ob[b] + (R - u) * Ns * Z.S, {c.re - d.im, c.im + d.re});
      }
    }
  }
  __syncthreads();
}

// Forward FFT of the tile's transforms (caller has synchronised the input).
// A backward FFT is this one with real and imaginary parts exchanged on both
// sides, which the loads and stores around it do.
template <typename T, int MODE>
__device__ __forceinline__ void fft_lds(LTile<T> Z, HP_LDS typename V2<T>::t* wR, unsigned char* smem,
                                        const PassArgs& a) {
  HP_LDS char* lds0 = (HP_LDS char*)smem;
  (void)lds0;
  constexpr int ME = Maxe<T, MODE>::v;
  const GC<T> tw = glb<T>(a.tw);
  const int L = a.L;
  int Ns = 1;
  for (int s = 0; s < a.nstage; ++s) {
    const int R = a.radix[s];
    switch (R) {
      case 2: fft_stage<T, 2, ME>(Z, L, Ns, tw); break;
      case 3: fft_stage<T, 3, ME>(Z, L, Ns, tw); break;
      case 4: fft_stage<T, 4, ME>(Z, L, Ns, tw); break;
      case 5: fft_stage<T, 5, ME>(Z, L, Ns, tw); break;
      case 6: fft_stage<T, 6, ME>(Z, L, Ns, tw); break;
      case 7: fft_stage<T, 7, ME>(Z, L, Ns, tw); break;
      case 8: fft_stage<T, 8, ME>(Z, L, Ns, tw); break;
      case 9: fft_stage<T, 9, ME>(Z, L, Ns, tw); break;
      case 10: fft_stage<T, 10, ME>(Z, L, Ns, tw); break;
      default:
        if constexpr (sizeof(T) == 4) {  // (kMaxRadix64: registers)
          if (R == 11) { fft_stage<T, 11, ME>(Z, L, Ns, tw); break; }
          if (R == 12) { fft_stage<T, 12, ME>(Z, L, Ns, tw); break; }
          if (R == 13) { fft_stage<T, 13, ME>(Z, L, Ns, tw); break; }
          if (R == 14) { fft_stage<T, 14, ME>(Z, L, Ns, tw); break; }
          if (R == 15) { fft_stage<T, 15, ME>(Z, L, Ns, tw); break; }
          if (R == 16) { fft_stage<T, 16, ME>(Z, L, Ns, tw); break; }
        }
        if constexpr (MODE == GM_BIG) {
          // (wR: the LDS after the tiles; no table where that is too short)
          const int room = (a.lds_bytes - (int)((HP_LDS char*)wR - lds0)) / (int)sizeof(C2<T>);
          if (room < R) { fft_stage_prime<T, ME, false>(Z, wR, L, R, Ns, tw); break; }
        }
        if constexpr (MODE != GM_SMALL) fft_stage_prime<T, ME, true>(Z, wR, L, R, Ns, tw);
        break;
    }
    Ns *= R;
  }
}

constexpr bool xform_inverse_fft(int x) {
  return x == X_C2C_B || x == X_C2R || x == X_PAIR_B || x == X_DCT3 || x == X_DST3;
}
__device__ __forceinline__ bool xform_complex_in(int x) { return x == X_C2C_F || x == X_C2C_B; }

// ----------------------------------------------------------- tile addressing
struct Tile {
  int o, p0, np;
};

template <typename T>
__device__ __forceinline__ Tile tile_of(const PassArgs& a, int Np) {
  const int tiles_p = (Np + a.P - 1) / a.P;
  const int ei = (int)sizeof(T) * (xform_complex_in(a.xf) || a.xf == X_C2R ? 2 : 1);
  const int eo = (int)sizeof(T) * (xform_complex_in(a.xf) || a.xf == X_R2C ? 2 : 1);
  const int b = off_lines(a, ei, eo) ? xcd_block(blockIdx.x, gridDim.x) : (int)blockIdx.x;
  Tile t;
  t.o = b / tiles_p;
  t.p0 = (b - t.o * tiles_p) * a.P;
  t.np = min(a.P, Np - t.p0);
  return t;
}

// Element e of a tile of nf = 2^lg columns and cnt rows -> (column, row):
// runs along the rows (jfast: the pencil axis is contiguous in memory) or
// across the columns.
__device__ __forceinline__ void tile_fj(int e, int lg, int cnt, unsigned mc, int jfast, int& f, int& j) {
  if (jfast) {
    f = div_by(e, cnt, mc);
    j = e - f * cnt;
  } else {
    j = e >> lg;
    f = e - (j << lg);
  }
}

// ---------------------------------------------------------------- loading
// Each thread takes kLoadBatch elements per round and issues all their loads
// before the first is used, so a tile costs one memory latency per round
// instead of one per element.  The values go straight to their places in the
// FFT input: the symmetric extension of a real-to-real transform is written
// while loading, so there is no raw copy of the tile.
constexpr int kLoadBatch = 4;

template <typename T>
__device__ __forceinline__ void zero_rows(LTile<T> Z, int m0, int m1) {
  const int total = (m1 - m0) << Z.lg;
  for (int e = threadIdx.x; e < total; e += kThreads) {
    const int m = e >> Z.lg;
    Z.put((m0 + m) * Z.S + e - (m << Z.lg), {(T)0, (T)0});
  }
}

// FFT input of transform XC from element s of the pair (a + ib) in column f:
//   DST-I   [0, x_0..x_{n-1}, 0, -x_{n-1}..-x_0]
//   DCT-I   [x_0..x_{n-1}, x_{n-2}..x_1]
//   DCT-II  [x_0..x_{n-1}, x_{n-1}..x_0] (DST-II: (-1)^s x_s)
//   DCT-III e^{+i pi s/2n} x_s below n, 0 at n, the conjugate twist above
//           (DST-III: x reversed), for the backward FFT (parts exchanged)
//   others  x_s (rows beyond the input zeroed by extend_zeros)
template <typename T, int XC>
__device__ __forceinline__ void extend(LTile<T> Z, int f, int s, C2<T> v, const PassArgs& a, int n) {
  const int L = a.L;
  auto put = [&](int m, C2<T> z) { Z.put(m * Z.S + f, z); };
  if constexpr (XC == X_DST1) {
    put(s + 1, v);
    put(L - 1 - s, {-v.re, -v.im});
  } else if constexpr (XC == X_DCT1) {
    put(s, v);
    if (s > 0 && s < n - 1) put(L - s, v);
  } else if constexpr (XC == X_DCT2 || XC == X_DST2) {
    if (XC == X_DST2 && (s & 1)) v = {-v.re, -v.im};
    put(s, v);
    put(L - 1 - s, v);
  } else if constexpr (XC == X_DCT3 || XC == X_DST3) {
    const int m = XC == X_DST3 ? n - 1 - s : s;
    const C2<T> w = ldc<T>(glb<T>(a.qtw), m);  // e^{-i pi m / 2n}
    const C2<T> lo = cmul(v, cconj(w)), hi = cmul(v, w);
    put(m, {lo.im, lo.re});
    if (m > 0) put(L - m, {hi.im, hi.re});
  } else {
    put(s, v);
  }
}

// The rows of the FFT input that no element reaches.
template <typename T, int XC>
__device__ __forceinline__ void extend_zeros(LTile<T> Z, const PassArgs& a, int n, int cnt) {
  if constexpr (XC == X_DST1) {
    zero_rows<T>(Z, 0, 1);
    zero_rows<T>(Z, n + 1, n + 2);
  } else if constexpr (XC == X_DCT3 || XC == X_DST3) {
    zero_rows<T>(Z, n, n + 1);
  } else if constexpr (XC == X_R2C || XC == X_PAIR_F || XC == X_DHT) {
    zero_rows<T>(Z, cnt, a.L);
  }
}

__device__ __forceinline__ bool has_face_terms(const PassArgs& a) {
  return a.face[0][0] || a.face[0][1] || a.face[1][0] || a.face[1][1] || a.face[2][0] || a.face[2][1];
}

// Whether element j of pencil p or p + 1 is the first or last unknown of an axis.
__device__ __forceinline__ bool beside_face(const PassArgs& a, int j, int p, int o) {
  bool hit = false;
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    const int hi = a.nunk[b] - 1;
    if (a.ax_j == b) hit |= j <= 0 || j >= hi;
    if (a.ax_p == b) hit |= p <= 0 || p + 1 >= hi;
    if (a.ax_o == b) hit |= o <= 0 || o >= hi;
  }
  return hit;
}

// Real pencils, two per column, with boundary terms when present (first
// passes only: forward transforms).
template <typename T, int XC>
__device__ __forceinline__ void load_real_x(LTile<T> Z, const void* src, const PassArgs& a, const Tile& t, int n,
                                            int cnt, bool faces) {
  const int jfast = a.in_jfast;
  const int total = cnt << Z.lg;
  const unsigned mc = div_magic(cnt);
  const HP_GLB T* in = (const HP_GLB T*)src + (long long)t.o * a.in_so + (long long)t.p0 * a.in_sp;
  // adjacent pencils adjacent in memory, every pair complete: one load a pair
  const bool pairs = a.in_sp == 1 && !jfast && (t.np & 1) == 0;
  for (int e0 = threadIdx.x; e0 < total; e0 += kLoadBatch * kThreads) {
    C2<T> v[kLoadBatch];
    int ff[kLoadBatch], jj[kLoadBatch];
    // unconditional loads from clamped (in-tile) addresses; the pencils
    // beyond np are zeroed where the values are kept
    if (pairs) {
#pragma unroll
      for (int u = 0; u < kLoadBatch; ++u) {
        tile_fj(min(e0 + u * kThreads, total - 1), Z.lg, cnt, mc, 0, ff[u], jj[u]);
        const typename V2<T>::u w =
            *(const HP_GLB typename V2<T>::u*)(in + (long long)jj[u] * a.in_sj + min(2 * ff[u], t.np - 2));
        v[u] = {w.x, w.y};
      }
    } else {
#pragma unroll
      for (int u = 0; u < kLoadBatch; ++u) {
        tile_fj(min(e0 + u * kThreads, total - 1), Z.lg, cnt, mc, jfast, ff[u], jj[u]);
        const HP_GLB T* row = in + (long long)jj[u] * a.in_sj;
        v[u].re = row[(long long)min(2 * ff[u], t.np - 1) * a.in_sp];
        v[u].im = row[(long long)min(2 * ff[u] + 1, t.np - 1) * a.in_sp];
      }
    }
#pragma unroll
    for (int u = 0; u < kLoadBatch; ++u) {
      if (e0 + u * kThreads >= total) continue;
      const int p = 2 * ff[u];
      extend<T, XC>(Z, ff[u], jj[u], {p < t.np ? v[u].re : (T)0, p + 1 < t.np ? v[u].im : (T)0}, a, n);
    }
  }
  extend_zeros<T, XC>(Z, a, n, cnt);
  if (faces) {
    // boundary terms: the elements next to a face are read back from their
    // (first) place in the FFT input and extended again
    __syncthreads();
    for (int e = threadIdx.x; e < total; e += kThreads) {
      int f, j;
      tile_fj(e, Z.lg, cnt, mc, 0, f, j);
      const int p = 2 * f;
      if (p >= t.np || !beside_face(a, j, t.p0 + p, t.o)) continue;
      C2<T> v = Z.get((XC == X_DST1 ? j + 1 : j) * Z.S + f);
      if (XC == X_DST2 && (j & 1)) v = {-v.re, -v.im};
      v.re = (T)((double)v.re + face_terms<T>(a, j, t.p0 + p, t.o));
      if (p + 1 < t.np) v.im = (T)((double)v.im + face_terms<T>(a, j, t.p0 + p + 1, t.o));
      extend<T, XC>(Z, f, j, v, a, n);
    }
  }
}

template <typename T>
__device__ __forceinline__ void load_real(LTile<T> Z, const void* src, int x, const PassArgs& a, const Tile& t, int n,
                                          int cnt, bool faces) {
  switch (x) {
    case X_DST1: load_real_x<T, X_DST1>(Z, src, a, t, n, cnt, faces); break;
    case X_DST2: load_real_x<T, X_DST2>(Z, src, a, t, n, cnt, faces); break;
    case X_DST3: load_real_x<T, X_DST3>(Z, src, a, t, n, cnt, faces); break;
    case X_DCT1: load_real_x<T, X_DCT1>(Z, src, a, t, n, cnt, faces); break;
    case X_DCT2: load_real_x<T, X_DCT2>(Z, src, a, t, n, cnt, faces); break;
    case X_DCT3: load_real_x<T, X_DCT3>(Z, src, a, t, n, cnt, faces); break;
    default: load_real_x<T, X_R2C>(Z, src, a, t, n, cnt, faces); break;  // R2C, paired, Hartley: as they are
  }
}

// ------------------------------------------------ series derivatives (FanJob)
// Extends coefficient k (value v, the factor applied) of the input into the
// derivative's FFT input; the thread of the first (last) coefficient also
// writes the places beside it that no coefficient reaches.
template <typename T, int XD>
__device__ __forceinline__ void extend_derivative(LTile<T> Z, int f, int k, C2<T> v, const FanJob& q,
                                                  const PassArgs& a) {
  const int s = q.basis == FB_HARTLEY ? fan_place<true>(q, k) : fan_place<false>(q, k);
  if (s >= 0 && s < q.nd) extend<T, XD>(Z, f, s, v, a, q.nd);
  if (q.basis == FB_SINE || q.basis == FB_COSINE) {
    const C2<T> zero = {(T)0, (T)0};
    if (k == 0 && q.shift < 0) extend<T, XD>(Z, f, 0, zero, a, q.nd);
    if (k == q.n - 1 && s + 1 < q.nd) extend<T, XD>(Z, f, s + 1, zero, a, q.nd);
  }
}

// The coefficients of a pencil tile times their factors, as the FFT input of
// the derivative's transform.
template <typename T, int XD>
__device__ __forceinline__ void load_derivative_x(LTile<T> Z, const FanJob& q, const PassArgs& a, const Tile& t) {
  const int cnt = q.n, jfast = a.in_jfast;
  const int total = cnt << Z.lg;
  const unsigned mc = div_magic(cnt);
  const HP_GLB T* in = (const HP_GLB T*)q.in + (long long)t.o * a.in_so + (long long)t.p0 * a.in_sp;
  for (int e0 = threadIdx.x; e0 < total; e0 += kLoadBatch * kThreads) {
    C2<T> v[kLoadBatch];
    int ff[kLoadBatch], jj[kLoadBatch];
#pragma unroll
    for (int u = 0; u < kLoadBatch; ++u) {
      tile_fj(min(e0 + u * kThreads, total - 1), Z.lg, cnt, mc, jfast, ff[u], jj[u]);
      const HP_GLB T* row = in + (long long)jj[u] * a.in_sj;
      v[u].re = row[(long long)min(2 * ff[u], t.np - 1) * a.in_sp];
      v[u].im = row[(long long)min(2 * ff[u] + 1, t.np - 1) * a.in_sp];
    }
#pragma unroll
    for (int u = 0; u < kLoadBatch; ++u) {
      if (e0 + u * kThreads >= total) continue;
      const int p = 2 * ff[u];
      const T m = (T)(q.basis == FB_HARTLEY ? fan_factor<true>(q, jj[u]) : fan_factor<false>(q, jj[u]));
      extend_derivative<T, XD>(Z, ff[u], jj[u], {p < t.np ? m * v[u].re : (T)0, p + 1 < t.np ? m * v[u].im : (T)0}, q,
                               a);
    }
  }
  extend_zeros<T, XD>(Z, a, q.nd, q.nd);
}

template <typename T>
__device__ __forceinline__ void load_derivative(LTile<T> Z, const FanJob& q, const PassArgs& a, const Tile& t) {
  switch (q.xd) {
    case X_DST1: load_derivative_x<T, X_DST1>(Z, q, a, t); break;
    case X_DST3: load_derivative_x<T, X_DST3>(Z, q, a, t); break;
    case X_DCT1: load_derivative_x<T, X_DCT1>(Z, q, a, t); break;
    case X_DCT3: load_derivative_x<T, X_DCT3>(Z, q, a, t); break;
    default: load_derivative_x<T, X_DHT>(Z, q, a, t); break;
  }
}

// Complex pencils, one per column, zero beyond nin; swap: for the backward FFT.
template <typename T>
__device__ __forceinline__ void load_c2c(LTile<T> Z, const void* src, const PassArgs& a, const Tile& t, bool swap) {
  const int cnt = a.nin, jfast = a.in_jfast;
  const int total = cnt << Z.lg;
  const unsigned mc = div_magic(cnt);
  const GC<T> in = glb<T>(src) + (long long)t.o * a.in_so + (long long)t.p0 * a.in_sp;
  for (int e0 = threadIdx.x; e0 < total; e0 += kLoadBatch * kThreads) {
    C2<T> v[kLoadBatch];
    int ff[kLoadBatch], jj[kLoadBatch];
#pragma unroll
    for (int u = 0; u < kLoadBatch; ++u) {
      tile_fj(min(e0 + u * kThreads, total - 1), Z.lg, cnt, mc, jfast, ff[u], jj[u]);
      v[u] = ldc<T>(in, (long long)min(ff[u], t.np - 1) * a.in_sp + (long long)jj[u] * a.in_sj);
    }
#pragma unroll
    for (int u = 0; u < kLoadBatch; ++u) {
      if (e0 + u * kThreads >= total) continue;
      const C2<T> w = ff[u] < t.np ? v[u] : C2<T>{(T)0, (T)0};
      Z.put(jj[u] * Z.S + ff[u], swap ? C2<T>{w.im, w.re} : w);
    }
  }
  zero_rows<T>(Z, cnt, a.L);
}

// Half spectra A, B (L/2 + 1 bins) of the two pencils of a column, completed
// to A + iB by Hermitian symmetry, for the backward FFT.
template <typename T>
__device__ __forceinline__ void load_half(LTile<T> Z, const void* src, const PassArgs& a, const Tile& t) {
  const int cnt = a.nin, jfast = a.in_jfast, L = a.L;
  const int total = cnt << Z.lg;
  const unsigned mc = div_magic(cnt);
  const GC<T> in = glb<T>(src) + (long long)t.o * a.in_so + (long long)t.p0 * a.in_sp;
  constexpr int U = kLoadBatch / 2;
  for (int e0 = threadIdx.x; e0 < total; e0 += U * kThreads) {
    C2<T> va[U], vb[U];
    int ff[U], jj[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      tile_fj(min(e0 + u * kThreads, total - 1), Z.lg, cnt, mc, jfast, ff[u], jj[u]);
      const GC<T> row = in + (long long)jj[u] * a.in_sj;
      va[u] = ldc<T>(row, (long long)min(2 * ff[u], t.np - 1) * a.in_sp);
      vb[u] = ldc<T>(row, (long long)min(2 * ff[u] + 1, t.np - 1) * a.in_sp);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (e0 + u * kThreads >= total) continue;
      const int m = jj[u], p = 2 * ff[u];
      const bool self = m == 0 || 2 * m == L;
      C2<T> A = p < t.np ? va[u] : C2<T>{(T)0, (T)0}, B = p + 1 < t.np ? vb[u] : C2<T>{(T)0, (T)0};
      if (self) A.im = B.im = (T)0;
      Z.put(m * Z.S + ff[u], {A.im + B.re, A.re - B.im});
      if (!self) Z.put((L - m) * Z.S + ff[u], {B.re - A.im, A.re + B.im});
    }
  }
}

// ---------------------------------------------------------------- storing
// Output k of the two pencils of column f from the transformed tile.
template <typename T, int XC>
__device__ __forceinline__ C2<T> real_out(LTile<T> Z, const PassArgs& a, int n, int f, int k) {
  if constexpr (XC == X_DST1) {
    const C2<T> v = Z.get((k + 1) * Z.S + f);
    return {-v.im, v.re};
  } else if constexpr (XC == X_DCT1) {
    return Z.get(k * Z.S + f);
  } else if constexpr (XC == X_DCT2 || XC == X_DST2) {
    const int kk = XC == X_DST2 ? n - 1 - k : k;
    return cmul(Z.get(kk * Z.S + f), ldc<T>(glb<T>(a.qtw), kk));
  } else if constexpr (XC == X_DHT) {
    // Z = X_a + i X_b with X_a, X_b Hermitian; H = Re X - Im X per pencil
    const C2<T> u = Z.get(k * Z.S + f), w = Z.get((k == 0 ? 0 : a.L - k) * Z.S + f);
    return {(T)0.5 * ((u.re + w.re) - (u.im - w.im)), (T)0.5 * ((u.im + w.im) + (u.re - w.re))};
  } else {  // DCT-III, DST-III, C2R, paired backward: the parts exchanged back
    const C2<T> v = Z.get(k * Z.S + f);
    if (XC == X_DST3 && (k & 1)) return {-v.im, -v.re};
    return {v.im, v.re};
  }
}

template <typename T, int XC>
__device__ __forceinline__ void store_real_x(LTile<T> Z, void* dst, const PassArgs& a, const Tile& t, int n,
                                             int cnt) {
  const int jfast = a.out_jfast;
  const int total = cnt << Z.lg;
  const unsigned mc = div_magic(cnt);
  HP_GLB T* out = (HP_GLB T*)dst + (long long)t.o * a.out_so + (long long)t.p0 * a.out_sp;
  const bool pairs = a.out_sp == 1 && !jfast && (t.np & 1) == 0;
  for (int e = threadIdx.x; e < total; e += kThreads) {
    int f, k;
    tile_fj(e, Z.lg, cnt, mc, jfast, f, k);
    if (2 * f >= t.np) continue;
    const C2<T> v = real_out<T, XC>(Z, a, n, f, k);
    HP_GLB T* row = out + (long long)k * a.out_sj;
    if (pairs) {
      typename V2<T>::u w;
      w.x = v.re;
      w.y = v.im;
      *(HP_GLB typename V2<T>::u*)(row + 2 * f) = w;
    } else {
      row[(long long)(2 * f) * a.out_sp] = v.re;
      if (2 * f + 1 < t.np) row[(long long)(2 * f + 1) * a.out_sp] = v.im;
    }
  }
}

// Complex pencils (swap: the parts exchanged back after a backward FFT).
template <typename T>
__device__ __forceinline__ void store_c2c(LTile<T> Z, void* dst, const PassArgs& a, const Tile& t, bool swap) {
  const int cnt = a.nout, jfast = a.out_jfast;
  const int total = cnt << Z.lg;
  const unsigned mc = div_magic(cnt);
  C2<T>* out = (C2<T>*)dst + (long long)t.o * a.out_so + (long long)t.p0 * a.out_sp;
  for (int e = threadIdx.x; e < total; e += kThreads) {
    int f, k;
    tile_fj(e, Z.lg, cnt, mc, jfast, f, k);
    if (f >= t.np) continue;
    const C2<T> v = Z.get(k * Z.S + f);
    stc<T>(out, (long long)f * a.out_sp + (long long)k * a.out_sj, swap ? C2<T>{v.im, v.re} : v);
  }
}

// Half spectra of the two pencils of every column (X_R2C).
template <typename T>
__device__ __forceinline__ void store_half(LTile<T> Z, void* dst, const PassArgs& a, const Tile& t) {
  const int cnt = a.nout, jfast = a.out_jfast;
  const int total = cnt << Z.lg;
  const unsigned mc = div_magic(cnt);
  C2<T>* out = (C2<T>*)dst + (long long)t.o * a.out_so + (long long)t.p0 * a.out_sp;
  for (int e = threadIdx.x; e < total; e += kThreads) {
    int f, k;
    tile_fj(e, Z.lg, cnt, mc, jfast, f, k);
    if (2 * f >= t.np) continue;
    const C2<T> zk = Z.get(k * Z.S + f), zc = cconj(Z.get((k == 0 ? 0 : a.L - k) * Z.S + f));
    const C2<T> s = cadd(zk, zc), d = csub(zk, zc);
    C2<T>* row = out + (long long)k * a.out_sj;
    stc<T>(row, (long long)(2 * f) * a.out_sp, {s.re * (T)0.5, s.im * (T)0.5});
    // (zk - zc) / (2 i)
    if (2 * f + 1 < t.np) stc<T>(row, (long long)(2 * f + 1) * a.out_sp, {d.im * (T)0.5, -d.re * (T)0.5});
  }
}

template <typename T>
__device__ __forceinline__ void store_real(LTile<T> Z, int x, void* dst, const PassArgs& a, const Tile& t, int n,
                                           int cnt) {
  switch (x) {
    case X_DST1: store_real_x<T, X_DST1>(Z, dst, a, t, n, cnt); break;
    case X_DST2: store_real_x<T, X_DST2>(Z, dst, a, t, n, cnt); break;
    case X_DST3: store_real_x<T, X_DST3>(Z, dst, a, t, n, cnt); break;
    case X_DCT1: store_real_x<T, X_DCT1>(Z, dst, a, t, n, cnt); break;
    case X_DCT2: store_real_x<T, X_DCT2>(Z, dst, a, t, n, cnt); break;
    case X_DHT: store_real_x<T, X_DHT>(Z, dst, a, t, n, cnt); break;
    default: store_real_x<T, X_DCT3>(Z, dst, a, t, n, cnt); break;  // DCT-III, C2R, paired backward
  }
}

template <typename T>
__device__ __forceinline__ void store_out(LTile<T> Z, int x, void* dst, const PassArgs& a, const Tile& t) {
  switch (x) {
    case X_C2C_F: store_c2c<T>(Z, dst, a, t, false); break;
    case X_C2C_B: store_c2c<T>(Z, dst, a, t, true); break;
    case X_R2C: store_half<T>(Z, dst, a, t); break;
    default: store_real<T>(Z, x, dst, a, t, a.n, a.nout); break;
  }
}

// -------------------------------------------------------- spectral multiply
// Spectral indices per logical axis.
struct KIdx {
  int k0, k1, k2;
};

__device__ __forceinline__ double eigen_multiplier(const PassArgs& a, const KIdx& k) {
  double lam = ((const HP_GLB double*)a.lam[0])[k.k0];
  if (a.lam[1]) lam += ((const HP_GLB double*)a.lam[1])[k.k1];
  if (a.lam[2]) lam += ((const HP_GLB double*)a.lam[2])[k.k2];
  return lam == 0.0 ? 0.0 : a.norm / lam;
}

template <typename T>
__device__ __forceinline__ T multiplier(const PassArgs& a, const KIdx& k) {
  if (a.mult == M_EIGEN) return (T)eigen_multiplier(a, k);
  if (a.mult == M_GREEN) {
    const int i0 = min(k.k0, a.gM[0] - k.k0);
    const int i1 = min(k.k1, a.gM[1] - k.k1);
    return ((const HP_GLB T*)a.green)[(long long)i0 * a.g_s[0] + (long long)i1 * a.g_s[1] +
                                      (long long)k.k2 * a.g_s[2]];
  }
  return (T)1;
}

// Spectral indices of element m of pencil p (tile-relative pencils beyond the
// last one are clamped: their values are never stored).
__device__ __forceinline__ KIdx spectral_index(const PassArgs& a, int m, int p, int o) {
  p = min(p, a.Np - 1);
  auto of = [&](int ax) { return a.ax_j == ax ? m : (a.ax_p == ax ? p : (a.ax_o == ax ? o : 0)); };
  return {of(0), of(1), of(2)};
}

template <typename T>
__device__ __forceinline__ T kval(const PassArgs& a, int axis, const KIdx& k) {
  return ((const HP_GLB T*)a.kvec[axis])[axis == 0 ? k.k0 : (axis == 1 ? k.k1 : k.k2)];
}

// ------------------------------------------------------------ pass bodies
template <typename T, int MODE>
__device__ __forceinline__ void oneway(const PassArgs& a, unsigned char* smem, const Tile& t, int field) {
  if (!a.in[field]) return;  // absent field (zero upstream gradient): uniform per block
  const int x = a.xf;
  const bool cplx = xform_complex_in(x);
  const int nf = cplx ? a.P : a.P / 2;
  const LTile<T> Z = lds_tile<T>(smem, nf, a.L, 0);
  if (cplx) load_c2c<T>(Z, a.in[field], a, t, x == X_C2C_B);
  else if (x == X_C2R) load_half<T>(Z, a.in[field], a, t);
  else load_real<T>(Z, a.in[field], x, a, t, a.n, a.nin, has_face_terms(a));
  __syncthreads();
  fft_lds<T, MODE>(Z, Z.z + (size_t)a.L * Z.S, smem, a);
  store_out<T>(Z, x, a.out[field], a, t);
}

// Spectral values of the forward transform XF times the multiplier, as the
// input of the backward transform XB.  In place without a barrier: output k
// is read from bins that only its own thread replaces (the sine and cosine
// transforms read one bin below n and write it and its mirror above n; a
// Hartley output reads bins k and L - k, both handled by one thread).
template <typename T, int XF, int XB>
__device__ __forceinline__ void multiply_r2r(LTile<T> Z, const PassArgs& a, const Tile& t) {
  const int rows = XF == X_DHT ? a.n / 2 + 1 : a.n;
  const int total = rows << Z.lg;
  auto scaled = [&](C2<T> s, int m, int f) {
    return C2<T>{s.re * multiplier<T>(a, spectral_index(a, m, t.p0 + 2 * f, t.o)),
                 s.im * multiplier<T>(a, spectral_index(a, m, t.p0 + 2 * f + 1, t.o))};
  };
  for (int e = threadIdx.x; e < total; e += kThreads) {
    const int m = e >> Z.lg, f = e - (m << Z.lg);
    const C2<T> v = scaled(real_out<T, XF>(Z, a, a.n, f, m), m, f);
    if constexpr (XF == X_DHT) {
      const int mm = m == 0 ? 0 : a.L - m;
      if (mm != m) {
        const C2<T> w = scaled(real_out<T, XF>(Z, a, a.n, f, mm), mm, f);
        extend<T, XB>(Z, f, mm, w, a, a.n);
      }
    }
    extend<T, XB>(Z, f, m, v, a, a.n);
  }
  extend_zeros<T, XB>(Z, a, a.n, a.n);
}

// Real-to-real sandwich (Dirichlet / Neumann / Hartley): forward R2R, multiply
// by the FD2 / PS multiplier, backward R2R, along the same axis.
template <typename T, int MODE>
__device__ __forceinline__ void sandwich_r2r(const PassArgs& a, unsigned char* smem, const Tile& t, int field) {
  const LTile<T> Z = lds_tile<T>(smem, a.P / 2, a.L, 0);
  HP_LDS typename V2<T>::t* wR = Z.z + (size_t)a.L * Z.S;
  load_real<T>(Z, a.in[field], a.xf, a, t, a.n, a.nin, has_face_terms(a));
  __syncthreads();
  fft_lds<T, MODE>(Z, wR, smem, a);
  switch (a.xf) {
    case X_DST1: multiply_r2r<T, X_DST1, X_DST1>(Z, a, t); break;
    case X_DST2: multiply_r2r<T, X_DST2, X_DST3>(Z, a, t); break;
    case X_DCT1: multiply_r2r<T, X_DCT1, X_DCT1>(Z, a, t); break;
    case X_DCT2: multiply_r2r<T, X_DCT2, X_DCT3>(Z, a, t); break;
    default: multiply_r2r<T, X_DHT, X_DHT>(Z, a, t); break;
  }
  __syncthreads();
  fft_lds<T, MODE>(Z, wR, smem, a);
  store_out<T>(Z, a.xb, a.out[field], a, t);
}

// Green's rows of a semi-unbounded plan's free axis.  Paired real pencils 2f,
// 2f + 1 of the tile belong to different bounded modes, so they take different
// real-even rows G_a, G_b.  The FFT Z of a + ib holds the Hermitian spectra
// X_a = (Z_m + conj Z_-m) / 2 and X_b = (Z_m - conj Z_-m) / 2i; G_a X_a + i G_b X_b
// recombines to Z'_m = A Z_m + B conj Z_-m with A = (G_a + G_b) / 2,
// B = (G_a - G_b) / 2, the same A, B at -m.  One thread per bin pair (m, L - m).
// ODD: also the rows of the kernel's derivative into D (bins i b_a, i b_b, b odd
// in m): Z'_m = i (A Z_m + B conj Z_-m) and Z'_-m = -i (A Z_-m + B conj Z_m),
// A, B from b_a, b_b at m.  Both with parts exchanged for the backward FFT.
template <typename T, bool ODD>
__device__ __forceinline__ void multiply_rows(LTile<T> S, LTile<T> D, const PassArgs& a, const Tile& t,
                                              const FanJob* q) {
  const int L = a.L, half = L / 2;
  const unsigned mh = div_magic(half + 1);
  auto row = [&](const void* g, int p, int m) -> T {
    p = min(p, a.Np - 1);
    const long long sj = a.ax_j == 0 ? a.g_s[0] : (a.ax_j == 1 ? a.g_s[1] : a.g_s[2]);
    const long long sp = a.ax_p == 0 ? a.g_s[0] : (a.ax_p == 1 ? a.g_s[1] : a.g_s[2]);
    long long off = (long long)m * sj + (long long)p * sp;
    if (a.ax_o >= 0) off += (long long)t.o * (a.ax_o == 0 ? a.g_s[0] : (a.ax_o == 1 ? a.g_s[1] : a.g_s[2]));
    return ((const HP_GLB T*)g)[off];
  };
  for (int e = threadIdx.x; e < ((half + 1) << S.lg); e += kThreads) {
    const int f = div_by(e, half + 1, mh);
    const int m = e - f * (half + 1);
    const int mm = m == 0 ? 0 : L - m;
    const int im = m * S.S + f, imm = mm * S.S + f;
    const C2<T> zm = S.get(im), zmm = S.get(imm);
    if constexpr (ODD) {
      const T sc = (T)q->scale;
      const T ga = sc * row(q->green_odd, t.p0 + 2 * f, m), gb = sc * row(q->green_odd, t.p0 + 2 * f + 1, m);
      const T A = (T)0.5 * (ga + gb), B = (T)0.5 * (ga - gb);
      const C2<T> ym = cadd(cscale(zm, A), cscale(cconj(zmm), B));    // times i, exchanged
      const C2<T> ymm = cadd(cscale(zmm, A), cscale(cconj(zm), B));  // times -i, exchanged
      D.put(im, {ym.re, -ym.im});
      if (mm != m) D.put(imm, {-ymm.re, ymm.im});
    }
    const T ga = row(a.green, t.p0 + 2 * f, m), gb = row(a.green, t.p0 + 2 * f + 1, m);
    const T A = (T)0.5 * (ga + gb), B = (T)0.5 * (ga - gb);
    const C2<T> ym = cadd(cscale(zm, A), cscale(cconj(zmm), B));
    const C2<T> ymm = cadd(cscale(zmm, A), cscale(cconj(zm), B));
    S.put(im, {ym.im, ym.re});
    if (mm != m) S.put(imm, {ymm.im, ymm.re});
  }
}

// ------------------------------------------------------------- fan passes
// One-way fan pass: the derivative first, then the plain transform, which may
// replace the input in place (its tile is this workgroup's alone).
template <typename T, int MODE>
__device__ __forceinline__ void oneway_fan(const PassArgs& a, unsigned char* smem, const Tile& t, const FanJob& q) {
  const LTile<T> Z = lds_tile<T>(smem, a.P / 2, a.L, 0);
  HP_LDS typename V2<T>::t* wR = Z.z + (size_t)a.L * Z.S;
  if (q.deriv) {
    load_derivative<T>(Z, q, a, t);
    __syncthreads();
    fft_lds<T, MODE>(Z, wR, smem, a);
    store_real<T>(Z, q.xd, q.deriv, a, t, q.nd, q.nd);
    __syncthreads();
  }
  load_real<T>(Z, q.in, q.xp, a, t, q.n, q.n, false);
  __syncthreads();
  fft_lds<T, MODE>(Z, wR, smem, a);
  store_real<T>(Z, q.xp, q.plain, a, t, q.n, q.n);
}

// multiply_r2r for both outputs: the multiplied spectrum into Z (plain) and,
// times the derivative's factors, into D.  XD: the derivative's transform
// (the Laplacian's is XB).
template <typename T, int XF, int XB, int XD>
__device__ __forceinline__ void multiply_r2r_fan(LTile<T> Z, LTile<T> D, const PassArgs& a, const Tile& t,
                                                 const FanJob& q) {
  const int rows = XF == X_DHT ? a.n / 2 + 1 : a.n;
  const int total = rows << Z.lg;
  auto axis_w2 = [&](int b, int k) {
    const int bs = b == 0 ? a.basis[0] : (b == 1 ? a.basis[1] : a.basis[2]);
    const int n = b == 0 ? a.nunk[0] : (b == 1 ? a.nunk[1] : a.nunk[2]);
    const double kc = b == 0 ? a.kc[0] : (b == 1 ? a.kc[1] : a.kc[2]);
    const int kk = bs == FB_HARTLEY ? (2 * k < n ? k : (2 * k == n ? 0 : k - n)) : (bs == FB_SINE ? k + 1 : k);
    const double w = kc * (double)kk;
    return w * w;
  };
  // plain and derivative value of bin m of column f from the spectra s
  auto both = [&](C2<T> s, int m, int f, C2<T>& d) {
    const KIdx ka = spectral_index(a, m, t.p0 + 2 * f, t.o), kb = spectral_index(a, m, t.p0 + 2 * f + 1, t.o);
    const double ma = eigen_multiplier(a, ka), mb = eigen_multiplier(a, kb);
    double fa, fb;
    if (q.basis == FB_LAP) {
      fa = -q.scale * (axis_w2(0, ka.k0) + axis_w2(1, ka.k1) + axis_w2(2, ka.k2));
      fb = -q.scale * (axis_w2(0, kb.k0) + axis_w2(1, kb.k1) + axis_w2(2, kb.k2));
    } else {
      fa = fb = XF == X_DHT ? fan_factor<true>(q, m) : fan_factor<false>(q, m);
    }
    d = {s.re * (T)(ma * fa), s.im * (T)(mb * fb)};
    return C2<T>{s.re * (T)ma, s.im * (T)mb};
  };
  for (int e = threadIdx.x; e < total; e += kThreads) {
    const int m = e >> Z.lg, f = e - (m << Z.lg);
    C2<T> d;
    const C2<T> v = both(real_out<T, XF>(Z, a, a.n, f, m), m, f, d);
    if constexpr (XF == X_DHT) {
      const int mm = m == 0 ? 0 : a.L - m;
      if (mm != m) {
        C2<T> dm;
        const C2<T> w = both(real_out<T, XF>(Z, a, a.n, f, mm), mm, f, dm);
        extend<T, XB>(Z, f, mm, w, a, a.n);
        extend_derivative<T, XD>(D, f, mm, dm, q, a);
      }
    }
    extend<T, XB>(Z, f, m, v, a, a.n);
    extend_derivative<T, XD>(D, f, m, d, q, a);
  }
  extend_zeros<T, XB>(Z, a, a.n, a.n);
  extend_zeros<T, XD>(D, a, q.nd, q.nd);
}

// Real-to-real fan sandwich: forward, multiplier, and two backward transforms.
template <typename T, int MODE>
__device__ __forceinline__ void sandwich_r2r_fan(const PassArgs& a, unsigned char* smem, const Tile& t,
                                                 const FanJob& q) {
  const LTile<T> Z = lds_tile<T>(smem, a.P / 2, a.L, 0), D = lds_tile<T>(smem, a.P / 2, a.L, 1);
  HP_LDS typename V2<T>::t* wR = D.z + (size_t)a.L * Z.S;
  load_real<T>(Z, q.in, a.xf, a, t, a.n, a.n, has_face_terms(a));
  __syncthreads();
  fft_lds<T, MODE>(Z, wR, smem, a);
  const bool lap = q.basis == FB_LAP;
  switch (a.xf) {
    case X_DST1:
      if (lap) multiply_r2r_fan<T, X_DST1, X_DST1, X_DST1>(Z, D, a, t, q);
      else multiply_r2r_fan<T, X_DST1, X_DST1, X_DCT1>(Z, D, a, t, q);
      break;
    case X_DST2:
      if (lap) multiply_r2r_fan<T, X_DST2, X_DST3, X_DST3>(Z, D, a, t, q);
      else multiply_r2r_fan<T, X_DST2, X_DST3, X_DCT3>(Z, D, a, t, q);
      break;
    case X_DCT1:
      if (lap) multiply_r2r_fan<T, X_DCT1, X_DCT1, X_DCT1>(Z, D, a, t, q);
      else multiply_r2r_fan<T, X_DCT1, X_DCT1, X_DST1>(Z, D, a, t, q);
      break;
    case X_DCT2:
      if (lap) multiply_r2r_fan<T, X_DCT2, X_DCT3, X_DCT3>(Z, D, a, t, q);
      else multiply_r2r_fan<T, X_DCT2, X_DCT3, X_DST3>(Z, D, a, t, q);
      break;
    default: multiply_r2r_fan<T, X_DHT, X_DHT, X_DHT>(Z, D, a, t, q); break;
  }
  __syncthreads();
  fft_lds<T, MODE>(D, wR, smem, a);
  fft_lds<T, MODE>(Z, wR, smem, a);
  store_real<T>(D, q.xd, q.deriv, a, t, q.nd, q.nd);
  store_real<T>(Z, a.xb, q.plain, a, t, a.n, a.n);
}

// Free-axis fan sandwich (Green's rows): psi and its free-axis derivative.
template <typename T, int MODE>
__device__ __forceinline__ void sandwich_rows_fan(const PassArgs& a, unsigned char* smem, const Tile& t,
                                                  const FanJob& q) {
  const LTile<T> Z = lds_tile<T>(smem, a.P / 2, a.L, 0), D = lds_tile<T>(smem, a.P / 2, a.L, 1);
  HP_LDS typename V2<T>::t* wR = D.z + (size_t)a.L * Z.S;
  load_real<T>(Z, q.in, X_PAIR_F, a, t, a.n, a.nin, false);
  __syncthreads();
  fft_lds<T, MODE>(Z, wR, smem, a);
  multiply_rows<T, true>(Z, D, a, t, &q);
  __syncthreads();
  fft_lds<T, MODE>(D, wR, smem, a);
  fft_lds<T, MODE>(Z, wR, smem, a);
  store_real<T>(D, X_PAIR_B, q.deriv, a, t, a.n, a.nout);
  store_real<T>(Z, X_PAIR_B, q.plain, a, t, a.n, a.nout);
}

// Complex sandwich (periodic after R2C, unbounded, 1D periodic pairs):
// every coupled field of the tile is resident: S_c (one LDS tile each) plus a
// work tile W where there are derivative inputs or outputs.
template <typename T, int MODE>
__device__ __forceinline__ void sandwich_c2c(const PassArgs& a, unsigned char* smem, const Tile& t) {
  const bool pair = a.xf == X_PAIR_F;
  const int nf = pair ? a.P / 2 : a.P;
  const int L = a.L;
  const bool adj = diff_is_adjoint(a.diff);
  const int nS = adj ? a.n_out : a.n_in;
  // independent fields (no derivative coupling) take their field from blockIdx.y
  const int fb = (a.diff == D_NONE) ? (int)blockIdx.y : 0;
  const int tiles = a.diff == D_NONE ? nS : nS + 1;
  const LTile<T> S = lds_tile<T>(smem, nf, L, 0, !a.tight);
  const LTile<T> W = lds_tile<T>(smem, nf, L, a.diff == D_NONE ? 0 : nS, !a.tight);
  const int tileC = L * S.S;  // LDS elements of a tile
  HP_LDS typename V2<T>::t* wR = S.z + (size_t)tiles * tileC;
  const int total = L << S.lg;
  const unsigned mL = div_magic(L);
  auto tile = [&](int c) { return LTile<T>{S.z + (size_t)c * tileC, S.S, S.lg}; };

  auto load_into = [&](LTile<T> dst, const void* src) {
    if (pair) load_real<T>(dst, src, X_PAIR_F, a, t, a.n, a.nin, false);
    else load_c2c<T>(dst, src, a, t, false);
    __syncthreads();
    fft_lds<T, MODE>(dst, wR, smem, a);
  };
  // element e of a tile -> column f, bin m (rows first: the multipliers' rows
  // are contiguous along m)
  auto each = [&](auto&& body) {
    for (int e = threadIdx.x; e < total; e += kThreads) {
      const int f = div_by(e, L, mL), m = e - f * L;
      body(m * S.S + f, spectral_index(a, m, t.p0 + f, t.o));
    }
  };

  for (int c = 0; c < nS; ++c) {
    if (a.in[fb + c]) {
      load_into(tile(c), a.in[fb + c]);
    } else {
      zero_rows<T>(tile(c), 0, L);
      __syncthreads();
    }
  }
  // spectral Laplacian: the first derivative i k_b (Nyquist zeroed) twice per axis
  auto lap_of = [&](const KIdx& k) -> T {
    T s = (T)0;
    for (int b = 0; b < 3; ++b)
      if (a.kvec[b]) {
        const T kb = kval<T>(a, b, k);
        s -= kb * kb;
      }
    return s;
  };
  // Transposed derivative inputs: curl (symmetric), minus the divergence
  // (gradient), minus the gradient (divergence) or the Laplacian (symmetric).
  if (adj) {
    const int nextra = a.n_in - nS;
    for (int i = 0; i < nextra; ++i) {
      const void* src = a.in[nS + i];
      if (!src) continue;
      load_into(W, src);
      each([&](int z, const KIdx& k) {
        const C2<T> g = W.get(z);
        auto acc = [&](int c, C2<T> v) {
          const int q = z + c * tileC;
          S.put(q, cadd(S.get(q), v));
        };
        if (a.diff == D_ADJ_CURL && nS == 1) {
          // 2D curl of a scalar, (d_y, -d_x): its transpose is -d_y g_0 + d_x g_1
          const T kk = i == 0 ? -kval<T>(a, 1, k) : kval<T>(a, 0, k);
          acc(0, cscale(cmuli(g), kk));
        } else if (a.diff == D_ADJ_CURL) {
          // (C g)_c = i(k_{c+1} g_{c+2} - k_{c+2} g_{c+1}): g_i enters
          // component i+1 with +i k_{i+2} and component i+2 with -i k_{i+1}
          const int c1 = (i + 1) % 3, c2 = (i + 2) % 3;
          const T kc1 = kval<T>(a, c1, k), kc2 = kval<T>(a, c2, k);
          const C2<T> ig = cmuli(g);
          acc(c1, cscale(ig, kc2));
          acc(c2, cscale(ig, -kc1));
        } else if (a.diff == D_ADJ_DIV) {
          const C2<T> ig = cmuli(g);
          for (int c = 0; c < nS; ++c) acc(c, cscale(ig, -kval<T>(a, c, k)));
        } else if (a.diff == D_ADJ_NABLA) {
          acc(i, cscale(g, lap_of(k)));
        } else {
          acc(0, cscale(cmuli(g), -kval<T>(a, i, k)));
        }
      });
      __syncthreads();
    }
  }
  // The multiplied spectra S keep their parts in place while derivative
  // outputs still read them, and are exchanged for the backward FFT otherwise.
  const bool derivs = a.diff == D_GRAD || a.diff == D_CURL || a.diff == D_DIV || a.diff == D_NABLA;
  if (a.mult == M_GREEN_ROWS) {
    multiply_rows<T, false>(S, S, a, t, nullptr);
  } else {
    // multiply by the spectral multiplier
    each([&](int z, const KIdx& k) {
      const T mu = multiplier<T>(a, k);
      for (int c = 0; c < nS; ++c) {
        const C2<T> v = cscale(S.get(z + c * tileC), mu);
        S.put(z + c * tileC, derivs ? v : C2<T>{v.im, v.re});
      }
    });
  }
  __syncthreads();
  const int xb = pair ? X_PAIR_B : X_C2C_B;
  // derivative outputs (forward GRAD / CURL) through W, then psi in place
  if (derivs) {
    const int nd = a.n_out - a.n_in;
    for (int d = 0; d < nd; ++d) {
      each([&](int z, const KIdx& k) {
        C2<T> v;
        if (a.diff == D_GRAD) {
          v = cscale(cmuli(S.get(z)), kval<T>(a, d, k));
        } else if (a.diff == D_DIV) {
          C2<T> acc = {(T)0, (T)0};
          for (int c = 0; c < a.n_in; ++c) acc = cadd(acc, cscale(S.get(z + c * tileC), kval<T>(a, c, k)));
          v = cmuli(acc);
        } else if (a.diff == D_NABLA) {
          v = cscale(S.get(z + d * tileC), lap_of(k));
        } else if (a.n_in == 1) {
          // 2D curl of a scalar: (d_y psi, -d_x psi)
          v = cscale(cmuli(S.get(z)), d == 0 ? kval<T>(a, 1, k) : -kval<T>(a, 0, k));
        } else {
          const int c1 = (d + 1) % 3, c2 = (d + 2) % 3;
          v = cmuli(csub(cscale(S.get(z + c2 * tileC), kval<T>(a, c1, k)),
                         cscale(S.get(z + c1 * tileC), kval<T>(a, c2, k))));
        }
        W.put(z, {v.im, v.re});
      });
      __syncthreads();
      fft_lds<T, MODE>(W, wR, smem, a);
      store_out<T>(W, xb, a.out[a.n_in + d], a, t);
      __syncthreads();
    }
    for (int c = 0; c < nS; ++c)
      each([&](int z, const KIdx&) {
        const C2<T> v = S.get(z + c * tileC);
        S.put(z + c * tileC, {v.im, v.re});
      });
    __syncthreads();
  }
  for (int c = 0; c < nS; ++c) {
    fft_lds<T, MODE>(tile(c), wR, smem, a);
    store_out<T>(tile(c), xb, a.out[fb + c], a, t);
  }
}

template <typename T, int MODE>
__global__ void __launch_bounds__(kThreads) k_oneway(const PassArgs) {
  extern __shared__ __align__(16) unsigned char smem[];
  const PassArgs& a = kernel_args();
  oneway<T, MODE>(a, smem, tile_of<T>(a, a.Np), blockIdx.y);
}

template <typename T, int MODE>
__global__ void __launch_bounds__(kThreads) k_sandwich_c2c(const PassArgs) {
  extern __shared__ __align__(16) unsigned char smem[];
  const PassArgs& a = kernel_args();
  sandwich_c2c<T, MODE>(a, smem, tile_of<T>(a, a.Np));
}

template <typename T, int MODE>
__global__ void __launch_bounds__(kThreads) k_sandwich_r2r(const PassArgs) {
  extern __shared__ __align__(16) unsigned char smem[];
  const PassArgs& a = kernel_args();
  sandwich_r2r<T, MODE>(a, smem, tile_of<T>(a, a.Np), blockIdx.y);
}

// KIND: 0 one-way, 1 real-to-real sandwich, 2 free-axis sandwich.
template <typename T, int MODE, int KIND>
__global__ void __launch_bounds__(kThreads) k_fan(const PassArgs) {
  extern __shared__ __align__(16) unsigned char smem[];
  const PassArgs& a = kernel_args();
  const FanJob& q = a.fan[blockIdx.y];
  const Tile t = tile_of<T>(a, q.Np);
  if (t.o >= q.No) return;  // fewer tiles than the largest job: whole workgroup
  if constexpr (KIND == 0) oneway_fan<T, MODE>(a, smem, t, q);
  else if constexpr (KIND == 1) sandwich_r2r_fan<T, MODE>(a, smem, t, q);
  else sandwich_rows_fan<T, MODE>(a, smem, t, q);
}

template <typename T, int MODE, int KIND>
static void launch_fan(const PassArgs& a, dim3 grid, hipStream_t s) {
  allow_lds<k_fan<T, MODE, KIND>>();
  hipLaunchKernelGGL((k_fan<T, MODE, KIND>), grid, dim3(kThreads), a.lds_bytes, s, a);
}

template <typename T, int MODE>
static void launch_t(const PassArgs& a, dim3 grid, hipStream_t s) {
  if (a.nfan > 0) {
    if (a.kind == PK_ONEWAY) launch_fan<T, MODE, 0>(a, grid, s);
    else if (a.mult == M_GREEN_ROWS) launch_fan<T, MODE, 2>(a, grid, s);
    else launch_fan<T, MODE, 1>(a, grid, s);
  } else if (a.kind == PK_ONEWAY) {
    allow_lds<k_oneway<T, MODE>>();
    hipLaunchKernelGGL((k_oneway<T, MODE>), grid, dim3(kThreads), a.lds_bytes, s, a);
  } else if (a.xf == X_C2C_F || a.xf == X_PAIR_F) {
    allow_lds<k_sandwich_c2c<T, MODE>>();
    hipLaunchKernelGGL((k_sandwich_c2c<T, MODE>), grid, dim3(kThreads), a.lds_bytes, s, a);
  } else {
    allow_lds<k_sandwich_r2r<T, MODE>>();
    hipLaunchKernelGGL((k_sandwich_r2r<T, MODE>), grid, dim3(kThreads), a.lds_bytes, s, a);
  }
}

// Radices of the register stages (fft_lds); a larger one runs the prime stage.
int max_radix(int prec) { return prec == 0 ? 16 : 10; }

int general_mode(const PassArgs& a, int prec) {
  if (a.big) return GM_BIG;
  for (int s = 0; s < a.nstage; ++s)
    if (a.radix[s] > max_radix(prec)) return GM_PRIME;
  return GM_SMALL;
}

template <typename T>
static void launch_mode(const PassArgs& a, int mode, dim3 grid, hipStream_t s) {
  if (mode == GM_BIG) launch_t<T, GM_BIG>(a, grid, s);
  else if (mode == GM_PRIME) launch_t<T, GM_PRIME>(a, grid, s);
  else launch_t<T, GM_SMALL>(a, grid, s);
}

// Every stage has room for its butterflies in the threads' registers (nf
// transforms of length L in a tile), and the radices make up L.
bool stages_fit(int L, long long nf, const int* radix, int nstage, int big, int prec) {
  const int maxe = (big ? 32 : 16) / (prec == 0 ? 1 : 2);
  long long prod = 1;
  for (int s = 0; s < nstage; ++s) {
    const int R = radix[s];
    if (R < 2) return false;
    prod *= R;
    if (L % prod != 0) return false;
    const long long nbl = L / R;
    if (R <= max_radix(prec)) {
      if (nf * nbl > (long long)(prec == 0 ? stage_slots<float>(R, maxe) : stage_slots<double>(R, maxe)) * kThreads)
        return false;
    } else {
      if (R % 2 == 0) return false;
      const long long nb = ((R - 1) / 2 + 1 + kPrimeB - 1) / kPrimeB;
      if (nf * nbl * nb > (long long)std::max(2, maxe * 3 / 16) * kThreads) return false;
    }
  }
  return prod == L;
}

bool general_fits(const PassArgs& a, int prec) {
  const bool cplx = a.xf == X_C2C_F || a.xf == X_C2C_B;
  const long long nf = cplx ? a.P : a.P / 2;
  if (nf < 1 || (nf & (nf - 1)) || a.L < 1 || a.L > 8192 || a.nin > a.L + 1 || a.nout > a.L + 1) return false;
  return stages_fit(a.L, nf, a.radix, a.nstage, a.big, prec);
}

// Tiles of a pass: nS coupled fields and a work tile where derivatives couple
// them, a fan sandwich's two outputs.
static int pass_tiles(const PassArgs& a) {
  if (a.nfan > 0) return a.kind == PK_SANDWICH ? 2 : 1;
  if (a.kind != PK_SANDWICH || !(a.xf == X_C2C_F || a.xf == X_C2C_B || a.xf == X_PAIR_F)) return 1;
  const int nS = diff_is_adjoint(a.diff) ? a.n_out : a.n_in;
  return a.diff == D_NONE ? nS : nS + 1;
}

// Whether the rows of the tiles of coupled fields leave the pad out: where no more
// than four workgroups share a CU with it, more do without, and the pass has more
// tiles than are resident.  Free-space curl of 150 x 80 x 100 cells, FP64 937 -> 657 us
// (four tiles of 300 x 2, two workgroups and four), FP32 454 -> 402, 100 x 60 x 80 FP32
// 255 -> 214.  Otherwise the bank conflicts cost more: seven and eight workgroups
// 127 -> 134 us (20 x 100 x 100 FP32), every tile resident anyway 127 -> 129 (periodic
// gradient 150 x 80 x 100 FP64), rows of 256 bytes, a turn of the banks each, whose
// accesses along m are served one lane at a time, 146 -> 156 (20 x 100 x 100 FP64).
static bool pass_tight(const PassArgs& a, int P, int prec) {
  const bool cplx = a.xf == X_C2C_F || a.xf == X_C2C_B;
  const int nf = cplx ? P : P / 2, tiles = pass_tiles(a), cs = prec == 0 ? 8 : 16;
  if (a.nfan > 0 || tiles < 2 || nf < 2 || nf * cs >= 256) return false;
  const long long lds = 160 * 1024, row = (long long)tiles * a.L * cs;
  const long long with = lds / (row * (nf + 1));
  return with <= 4 && lds / (row * nf) > with && (long long)((a.Np + P - 1) / P) * a.No > with * kCUs;
}

// LDS bytes of a general pass of tile width P: its FFT tiles (`padded`: with padded
// rows, also where the kernel leaves the pad out) and the table of the largest prime
// stage (left out where it would not fit; the kernel sees the room that is left).
int general_lds_bytes(const PassArgs& a, int P, int prec, bool padded) {
  const bool cplx = a.xf == X_C2C_F || a.xf == X_C2C_B;
  const int nf = cplx ? P : P / 2;
  int table = 0;
  for (int s = 0; s < a.nstage; ++s)
    if (a.radix[s] > max_radix(prec)) table = std::max(table, a.radix[s]);
  const long long cs = prec == 0 ? 8 : 16;
  const long long data = (long long)pass_tiles(a) * a.L * tile_row(nf, padded || !pass_tight(a, P, prec)) * cs;
  if (a.big && data + table * cs > 160 * 1024) table = 0;
  return (int)std::min<long long>(data + table * cs, 1 << 30);
}

hipError_t launch_pass(const PassArgs& pass, int prec, int grid_y, hipStream_t s) {
  PassArgs a = pass;
  a.tight = pass_tight(a, a.P, prec);
  if (!general_fits(a, prec) || general_lds_bytes(a, a.P, prec) > a.lds_bytes) return hipErrorInvalidValue;
  int tiles = ((a.Np + a.P - 1) / a.P) * a.No;
  if (a.nfan > 0) {
    // jobs fit the pass: sizes within the FFT input, a sandwich one job with
    // both outputs
    if (a.nfan > kMaxFan || (a.kind == PK_SANDWICH && (a.nfan != 1 || !a.fan[0].deriv))) return hipErrorInvalidValue;
    for (int i = 0; i < a.nfan; ++i) {
      const FanJob& q = a.fan[i];
      if (!q.in || !q.plain || q.n < 1 || q.n > a.L || (q.deriv && (q.nd < 0 || q.nd > a.L)) || q.Np < 1 || q.No < 1)
        return hipErrorInvalidValue;
      tiles = std::max(tiles, ((q.Np + a.P - 1) / a.P) * q.No);
    }
    grid_y = a.nfan;
  }
  dim3 grid(tiles, grid_y);
  const int mode = general_mode(a, prec);
  if (prec == 0) launch_mode<float>(a, mode, grid, s);
  else launch_mode<double>(a, mode, grid, s);
  return hipGetLastError();
}

// ------------------------------------------------------------ batched passes
// One pass level of a batched plan (the same pass of every problem, any
// lengths): one workgroup per item, consecutive tiles of one problem's pass,
// with the device code of the one-launch-per-pass path.  Launch boundaries
// order the levels.
template <typename T, int MODE>
__global__ void __launch_bounds__(kThreads) k_batched(const PassArgs* passes, const BatchItem* items) {
  extern __shared__ __align__(16) unsigned char smem[];
  const BatchItem bi = items[blockIdx.x];
  const PassArgs& a = passes[__builtin_amdgcn_readfirstlane(bi.pass)];
  const int tiles_p = (a.Np + a.P - 1) / a.P;
  const int n = __builtin_amdgcn_readfirstlane(bi.ntile);
  for (int k = 0; k < n; ++k) {
    const int tile = bi.tile + k;
    Tile t;
    t.o = tile / tiles_p;
    t.p0 = (tile - t.o * tiles_p) * a.P;
    t.np = min(a.P, a.Np - t.p0);
    if (a.kind == PK_ONEWAY) oneway<T, MODE>(a, smem, t, 0);
    else sandwich_r2r<T, MODE>(a, smem, t, 0);
    __syncthreads();  // LDS reuse by the next tile
  }
}

template <typename T, int MODE>
static void launch_batched_t(const PassArgs* passes, const BatchItem* items, int count, int lds, hipStream_t s) {
  allow_lds<k_batched<T, MODE>>();
  hipLaunchKernelGGL((k_batched<T, MODE>), dim3(count), dim3(kThreads), lds, s, passes, items);
}

template <typename T>
static void launch_batched_mode(const PassArgs* passes, const BatchItem* items, int count, int lds, int mode,
                                hipStream_t s) {
  if (mode == GM_BIG) launch_batched_t<T, GM_BIG>(passes, items, count, lds, s);
  else if (mode == GM_PRIME) launch_batched_t<T, GM_PRIME>(passes, items, count, lds, s);
  else launch_batched_t<T, GM_SMALL>(passes, items, count, lds, s);
}

hipError_t launch_batched(const PassArgs* passes, const BatchItem* items, const BatchGroup& g, int prec,
                          int mode, hipStream_t s) {
  if (g.count <= 0) return hipSuccess;
  if (prec == 0) launch_batched_mode<float>(passes, items + g.first, g.count, g.lds, mode, s);
  else launch_batched_mode<double>(passes, items + g.first, g.count, g.lds, mode, s);
  return hipGetLastError();
}

// ------------------------------------------------------ plan-time kernels
// Tabulated integral of the spectral kernel at x >= 0: the nearest table node
// plus the Gauss-Legendre integral of the integrand over the rest (<= step/2).
template <class F>
__device__ double table_integral(double x, const GreenEval& e, F g) {
  int j = (int)(x / e.si_step + 0.5);
  j = min(j, e.si_n - 1);
  const double a = j * e.si_step;
  const double mid = 0.5 * (x + a), half = 0.5 * (x - a);
  double acc = 0.0;
#pragma unroll
  for (int q = 0; q < 8; ++q) acc += e.gl_w[q] * g(mid + half * e.gl_x[q]);
  return e.si[j] + half * acc;
}

// ln(t) + E1(t), t >= 0 (the ln t singularities cancel): the power series
// -gamma - sum_k (-t)^k / (k k!) for t <= 2, else ln t + E1(t) with E1 from its
// continued fraction e^-t / (t + 1 - 1^2 / (t + 3 - 2^2 / (t + 5 - ...)))
// evaluated by the modified Lentz method.
__device__ double log_plus_e1(double t) {
  const double euler = 0.57721566490153286060651209008240243;
  if (t <= 2.0) {
    double term = 1.0, sum = 0.0;
    for (int k = 1; k <= 40; ++k) {
      term *= -t / k;  // (-t)^k / k!
      const double add = term / k;
      sum += add;
      if (fabs(add) < 1e-18 * fabs(sum)) break;
    }
    return -euler - sum;
  }
  const double tiny = 1e-300;
  double b = t + 1.0, c = 1.0 / tiny, d = 1.0 / b, h = d;
  for (int i = 1; i <= 200; ++i) {
    const double an = -(double)i * i;
    b += 2.0;
    d = 1.0 / (an * d + b);
    c = b + an / c;
    const double del = c * d;
    h *= del;
    if (fabs(del - 1.0) < 1e-16) break;
  }
  return log(t) + h * exp(-t);
}

// G(r) of a 2D or 1D free-space kernel (the readings beside the 3D ones).
__device__ double green_value_low(double r, const GreenEval& e) {
  const double pi = M_PI;
  if (e.dim == 2) {
    if (e.kind == 0) {
      const double euler = 0.57721566490153286060651209008240243;
      const double F = r == 0.0 ? 0.0 : table_integral(e.kc * r, e, [](double t) { return (1.0 - j0(t)) / t; });
      return (F - log(0.5 * e.kc) - euler) / (2.0 * pi);
    }
    // (1 / 2 pi) [ln sigma + (ln 2 + ln t + E1(t)) / 2 - e^-t sum_j L_{j-1}(t) / (2 j)], t = rho^2 / 2
    const double t = 0.5 * (r / e.sigma) * (r / e.sigma);
    double S = 0.0;
    switch (e.kind) {  // sum_{j=1}^{m-1} L_{j-1}(t) / (2 j), expanded
      case 4: S = 0.5; break;
      case 6: S = 0.5 + (1.0 - t) / 4.0; break;
      case 8: S = 0.5 + (1.0 - t) / 4.0 + ((0.5 * t - 2.0) * t + 1.0) / 6.0; break;
      case 10:
        S = 0.5 + (1.0 - t) / 4.0 + ((0.5 * t - 2.0) * t + 1.0) / 6.0 +
            (((-t / 6.0 + 1.5) * t - 3.0) * t + 1.0) / 8.0;
        break;
      default: break;
    }
    return (log(e.sigma) + 0.5 * (M_LN2 + log_plus_e1(t)) - exp(-t) * S) / (2.0 * pi);
  }
  // 1D: the spectral cutoff, or Gaussian order 2m: G2 plus
  // (sigma / sqrt(2 pi)) e^{-rho^2/2} sum_{j=1}^{m-1} (-1)^j He_{2j-2}(rho) / (2^j j!)
  // (the twice-integrated Hermite terms of the order-2m source), in t = rho^2
  const double x = fabs(r);
  if (e.kind == 0) {
    const double si = x == 0.0 ? 0.0 : table_integral(e.kc * x, e, [](double t) { return sin(t) / t; });
    return (x * si + cos(e.kc * x) / e.kc) / pi;
  }
  const double t = (x / e.sigma) * (x / e.sigma);
  double C = 1.0;
  switch (e.kind) {
    case 10: C += (((t - 15.0) * t + 45.0) * t - 15.0) / 384.0; [[fallthrough]];
    case 8: C -= ((t - 6.0) * t + 3.0) / 48.0; [[fallthrough]];
    case 6: C += (t - 1.0) / 8.0; [[fallthrough]];
    case 4: C -= 0.5; break;
    default: break;
  }
  return 0.5 * x * erf(x / (M_SQRT2 * e.sigma)) + e.sigma * exp(-0.5 * t) / sqrt(2.0 * pi) * C;
}

// G(r) of the free-space kernel (GreenEval); see the kernel list in hipoisson.h.
__device__ double green_value(double r, const GreenEval& e) {
  if (e.dim != 3) return green_value_low(r, e);
  if (e.kind == 0) {
    // spectral cutoff: -Si(kc r) / (2 pi^2 r); Si from the nearest table node
    // plus the Gauss-Legendre integral of sin(t) / t over the remaining stretch
    if (r == 0.0) return -e.kc / (2.0 * M_PI * M_PI);
    const double x = e.kc * r;
    int j = (int)(x / e.si_step + 0.5);
    j = min(j, e.si_n - 1);
    const double a = j * e.si_step;
    const double mid = 0.5 * (x + a), half = 0.5 * (x - a);
    double acc = 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const double t = mid + half * e.gl_x[q];
      acc += e.gl_w[q] * sin(t) / t;
    }
    return -(e.si[j] + half * acc) / (2.0 * M_PI * M_PI * r);
  }
  // Gaussian order 2m: -(1 / (4 pi sigma)) [erf(rho / sqrt2) / rho
  //                    + sqrt(2 / pi) exp(-rho^2 / 2) S_m(rho^2)], with the
  // Hermite sum S_m expanded in t = rho^2
  const double rho = r / e.sigma, t = rho * rho;
  const double s2pi = 0.79788456080286535587989211986876;  // sqrt(2 / pi)
  const double E = rho == 0.0 ? s2pi : erf(rho / M_SQRT2) / rho;
  double S = 0.0;
  switch (e.kind) {
    case 4: S = 0.5; break;
    case 6: S = (7.0 - t) / 8.0; break;
    case 8: S = ((t - 16.0) * t + 57.0) / 48.0; break;
    case 10: S = (((29.0 - t) * t - 233.0) * t + 561.0) / 384.0; break;
    default: break;
  }
  return -(E + s2pi * exp(-0.5 * t) * S) / (4.0 * M_PI * e.sigma);
}

__global__ void k_green_eval(double* g, int M0, int M1, int M2, double h0, double h1,
                             double h2, const GreenEval e, double scale) {
  const long long total = (long long)M0 * M1 * M2;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total;
       i += (long long)gridDim.x * blockDim.x) {
    const int z = (int)(i % M2);
    const int y = (int)((i / M2) % M1);
    const int x = (int)(i / ((long long)M1 * M2));
    const double dx = min(x, M0 - x) * h0, dy = min(y, M1 - y) * h1, dz = min(z, M2 - z) * h2;
    g[i] = green_value(sqrt(dx * dx + dy * dy + dz * dz), e) * scale;
  }
}

hipError_t launch_green_eval(double* g, const int M[3], const double h[3], const GreenEval& ge,
                             double scale, hipStream_t s) {
  if (ge.kind == 0 && (!ge.si || ge.si_n < 1)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_green_eval, dim3(4096), dim3(256), 0, s, g, M[0], M[1], M[2], h[0], h[1],
                     h[2], ge, scale);
  return hipGetLastError();
}

// Weighted sum of the boundary-augmented source (zero-mode query): grid-stride
// accumulation in FP64, one partial per block.
template <typename T>
__global__ void __launch_bounds__(256) k_zero_mode(const PassArgs a, const T* f, int n0, int n1,
                                                   int n2, int t0, int t1, int t2, double* partial) {
  __shared__ double red[256];
  const long long total = (long long)n0 * n1 * n2;
  double acc = 0.0;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total;
       i += (long long)gridDim.x * blockDim.x) {
    const int i2 = (int)(i % n2), i1 = (int)((i / n2) % n1), i0 = (int)(i / ((long long)n1 * n2));
    double w = 1.0;
    if (t0 && (i0 == 0 || i0 == n0 - 1)) w *= 0.5;
    if (t1 && (i1 == 0 || i1 == n1 - 1)) w *= 0.5;
    if (t2 && (i2 == 0 || i2 == n2 - 1)) w *= 0.5;
    acc += w * ((double)f[i] + face_terms<T>(a, i0, i1, i2));
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

hipError_t launch_zero_mode(const PassArgs& a, const void* f, const int n[3], const int trap[3],
                            double* partial, int nb, int prec, hipStream_t s) {
  if (prec == 0)
    hipLaunchKernelGGL(k_zero_mode<float>, dim3(nb), dim3(256), 0, s, a, (const float*)f, n[0], n[1],
                       n[2], trap[0], trap[1], trap[2], partial);
  else
    hipLaunchKernelGGL(k_zero_mode<double>, dim3(nb), dim3(256), 0, s, a, (const double*)f, n[0],
                       n[1], n[2], trap[0], trap[1], trap[2], partial);
  return hipGetLastError();
}

// ------------------------------------------------- reference streaming copy
// A plain copy with 16-byte nontemporal loads and stores: every workgroup
// copies one contiguous 16 KiB chunk, four accesses in flight per thread (of
// the shapes measured, this one moved the most bytes per second; the
// nontemporal hint keeps the streamed data from displacing cache lines).  The
// bandwidth a kernel doing nothing but streaming reaches on the device: the
// measured ceiling beside the HBM specification.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr int kCopyPer = 4;  // 16-byte accesses per thread

__global__ void __launch_bounds__(256) k_copy16(const u32x4* __restrict__ src,
                                                u32x4* __restrict__ dst, long long n16) {
  const long long base = (long long)blockIdx.x * (kCopyPer * 256) + threadIdx.x;
  u32x4 v[kCopyPer];
#pragma unroll
  for (int k = 0; k < kCopyPer; ++k) {
    const long long i = base + (long long)k * 256;
    if (i < n16) v[k] = __builtin_nontemporal_load(&src[i]);
  }
#pragma unroll
  for (int k = 0; k < kCopyPer; ++k) {
    const long long i = base + (long long)k * 256;
    if (i < n16) __builtin_nontemporal_store(v[k], &dst[i]);
  }
}

__global__ void k_copy_tail(const unsigned char* src, unsigned char* dst, long long n) {
  const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (i < n) dst[i] = src[i];
}

hipError_t launch_copy(const void* src, void* dst, size_t bytes, hipStream_t s) {
  const long long n16 = (long long)(bytes / 16);
  if (n16 > 0) {
    const long long per = (long long)kCopyPer * 256;
    const long long grid = (n16 + per - 1) / per;
    if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_copy16, dim3((unsigned)grid), dim3(256), 0, s, (const u32x4*)src,
                       (u32x4*)dst, n16);
  }
  const long long tail = (long long)(bytes - (size_t)n16 * 16);
  if (tail > 0)
    hipLaunchKernelGGL(k_copy_tail, dim3(1), dim3(64), 0, s, (const unsigned char*)src + n16 * 16,
                       (unsigned char*)dst + n16 * 16, tail);
  return hipGetLastError();
}

// ------------------------------------------ allocation-free zero-mode query
// The per-block partial sums of every component live in this file-scope
// device array instead of plan memory.  Each device holds its own copy (at
// its own address) until the process ends; in host code the name is only a
// stand-in, so host code uses the address that hipGetSymbolAddress returns
// for the device, never the name itself.
static __device__ __align__(256) double scratch[kZeroModeMaxComp * kZeroModeBlocks];

namespace {
std::mutex g_scratch_mu;
void* g_scratch_ptr[64] = {};
}  // namespace

hipError_t zero_mode_scratch(hipStream_t s, double** out) {
  *out = nullptr;
  int dev = 0;
  hipError_t e = hipStreamGetDevice(s, &dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    int cur = 0;
    e = hipGetDevice(&cur);
    if (e != hipSuccess) return e;
    if (cur != dev && (e = hipSetDevice(dev)) != hipSuccess) return e;
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (cur != dev) {
      const hipError_t r = hipSetDevice(cur);
      if (e == hipSuccess) e = r;
    }
    if (e != hipSuccess) return e;
    g_scratch_ptr[dev] = ptr;
  }
  *out = (double*)g_scratch_ptr[dev];
  return hipSuccess;
}

// out[c] = (partials of component c summed in block order) / W[c]; one
// thread per component, so the sum is the same as a host loop over them.
__global__ void k_zero_mode_finish(const double* partial, int nb, int ncomp, double W0, double W1,
                                   double W2, double* out) {
  const int c = threadIdx.x;
  if (c >= ncomp) return;
  const double W = c == 0 ? W0 : (c == 1 ? W1 : W2);
  double sum = 0.0;
  if (W != 0.0) {
    for (int i = 0; i < nb; ++i) sum += partial[(long long)c * nb + i];
    sum /= W;
  }
  out[c] = sum;
}

hipError_t launch_zero_mode_noalloc(const PassArgs* a, const void* const* f, int ncomp,
                                    const int n[3], const int trap[3], const double* W,
                                    double* out, int prec, hipStream_t s) {
  if (ncomp < 1 || ncomp > kZeroModeMaxComp) return hipErrorInvalidValue;
  double* partial = nullptr;
  hipError_t e = zero_mode_scratch(s, &partial);
  if (e != hipSuccess) return e;
  for (int c = 0; c < ncomp; ++c) {
    if (W[c] == 0.0) continue;  // no zero eigenvalue: the finish kernel writes 0
    e = launch_zero_mode(a[c], f[c], n, trap, partial + (long long)c * kZeroModeBlocks,
                         kZeroModeBlocks, prec, s);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_zero_mode_finish, dim3(1), dim3(64), 0, s, partial, kZeroModeBlocks, ncomp,
                     W[0], ncomp > 1 ? W[1] : 0.0, ncomp > 2 ? W[2] : 0.0, out);
  return hipGetLastError();
}

template <typename T>
__global__ void k_octant(const double* spec, int M0, int M1, int K2, double scale, T* out) {
  const int O0 = M0 / 2 + 1, O1 = M1 / 2 + 1;
  const long long total = (long long)O0 * O1 * K2;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total;
       i += (long long)gridDim.x * blockDim.x) {
    const int x = (int)(i % O0);
    const int y = (int)((i / O0) % O1);
    const int z = (int)(i / ((long long)O0 * O1));
    const long long src = ((long long)x * M1 + y) * K2 + z;
    out[i] = (T)(spec[2 * src] * scale);
  }
}

hipError_t launch_octant(const double* spec, const int M[3], double scale, void* out, int prec,
                         hipStream_t s) {
  const int K2 = M[2] / 2 + 1;
  if (prec == 0)
    hipLaunchKernelGGL(k_octant<float>, dim3(2048), dim3(256), 0, s, spec, M[0], M[1], K2, scale,
                       (float*)out);
  else
    hipLaunchKernelGGL(k_octant<double>, dim3(2048), dim3(256), 0, s, spec, M[0], M[1], K2, scale,
                       (double*)out);
  return hipGetLastError();
}

// Green's spectrum rows of the free axis (see launch_semi_green).  The DFT of
// the mirrored samples of G = -exp(-kappa x) / (2 kappa) sums two geometric
// series in q = exp(-kappa h); with s = (-1)^m q^n (n = M / 2) and
// theta = 2 pi m / M it is
//   -(1 - s)(1 - q^2) / (2 kappa ((1 - q)^2 + 4 q sin^2(theta / 2))),
// a sum of positive terms in the denominator (no cancellation).  kappa = 0
// (G = |x| / 2): h n^2 / 2 at m = 0, else -h (1 - (-1)^m) / (4 sin^2(theta / 2)).
// odd: G' = sign(x) exp(-kappa |x|) / 2 sampled at j = 1 .. n - 1 and with
// the opposite sign at M - j (0 at j = 0 and n); its bin m is -i times
// Im sum_{j=1}^{n-1} z^j, z = q e^{i theta}, a geometric series whose sum
// (z - s) / (1 - z) gives the stored b(m) (bin = i b):
//   -q sin(theta) (1 - s) / ((1 - q)^2 + 4 q sin^2(theta / 2)),
// for kappa = 0 (q = 1) -(1 - (-1)^m) cot(theta / 2) / 2, 0 at m = 0.
template <typename T>
__global__ void k_semi_green(T* out, const double* lam1, int n1, const double* lam2, int n2, int M,
                             double h, double scale, int odd) {
  const int K = M / 2 + 1, n = M / 2;
  const long long total = (long long)K * n1 * n2;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total;
       i += (long long)gridDim.x * blockDim.x) {
    const int m = (int)(i % K);
    const long long r = i / K;
    const int i1 = (int)(r % n1), i2 = (int)(r / n1);
    const double lam = lam1[i1] + (lam2 ? lam2[i2] : 0.0);
    const double sh = sinpi((double)m / (double)M);  // sin(theta / 2)
    const double sgn = (m & 1) ? -1.0 : 1.0;
    double v;
    if (odd) {
      const double st = sinpi(2.0 * (double)m / (double)M);  // sin(theta)
      if (lam < 0.0) {
        const double kappa = sqrt(-lam);
        const double q = exp(-kappa * h);
        const double omq = -expm1(-kappa * h);
        const double s = sgn * exp(-kappa * h * n);
        v = -q * st * (1.0 - s) / (omq * omq + 4.0 * q * sh * sh);
      } else {
        v = m == 0 ? 0.0 : -0.5 * (1.0 - sgn) * cospi((double)m / (double)M) / sh;
      }
    } else if (lam < 0.0) {
      const double kappa = sqrt(-lam);
      const double q = exp(-kappa * h);
      const double omq = -expm1(-kappa * h);       // 1 - q
      const double omq2 = -expm1(-2.0 * kappa * h);  // 1 - q^2
      const double s = sgn * exp(-kappa * h * n);
      v = -(1.0 - s) * omq2 / (2.0 * kappa * (omq * omq + 4.0 * q * sh * sh));
    } else if (m == 0) {
      v = 0.5 * h * (double)n * (double)n;
    } else {
      v = -h * (1.0 - sgn) / (4.0 * sh * sh);
    }
    out[i] = (T)(scale * v);
  }
}

hipError_t launch_semi_green(void* out, const double* lam1, int n1, const double* lam2, int n2,
                             int M, double h, double scale, int odd, int prec, hipStream_t s) {
  if (prec == 0)
    hipLaunchKernelGGL(k_semi_green<float>, dim3(1024), dim3(256), 0, s, (float*)out, lam1, n1, lam2,
                       n2, M, h, scale, odd);
  else
    hipLaunchKernelGGL(k_semi_green<double>, dim3(1024), dim3(256), 0, s, (double*)out, lam1, n1,
                       lam2, n2, M, h, scale, odd);
  return hipGetLastError();
}

// Boundary nodes of the fields of a solve (FillArgs): block row blockIdx.y =
// 2 a + side walks face (a, side) of field blockIdx.z only, one thread per
// node, the node's other two coordinates row-major (the face array's own
// index).  A node on several faces of the field's mask is written once, by
// the face of its highest axis.  32-bit node indices within a face: the
// launch refuses faces of 2^30 nodes or more.
template <typename T>
__global__ void k_boundary_fill(const FillArgs p) {
  const int fld = blockIdx.z, axes = p.axes[fld];
  const int N[3] = {p.N[0], p.N[1], p.N[2]};
  const int a = blockIdx.y >> 1, side = blockIdx.y & 1;
  if (a >= p.ndim || !((axes >> a) & 1)) return;
  const int o0 = a == 0 ? 1 : 0, o1 = a == 2 ? 1 : 2;  // the other axes, in order
  const int n1 = N[o1], fsize = N[o0] * N[o1];
  const T* g = (const T*)p.face[fld][a][side];
  T* out = (T*)p.out[fld];
  const long long st[3] = {(long long)N[1] * N[2], (long long)N[2], 1LL};
  for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < fsize; j += gridDim.x * blockDim.x) {
    int c[3];
    c[a] = side ? N[a] - 1 : 0;
    c[o0] = j / n1;
    c[o1] = j - c[o0] * n1;
    bool own = true;
    for (int b = a + 1; b < p.ndim; ++b)
      if (((axes >> b) & 1) && (c[b] == 0 || c[b] == N[b] - 1)) own = false;
    if (!own) continue;
    out[c[0] * st[0] + c[1] * st[1] + c[2] * st[2]] = g ? g[j] : (T)0;
  }
}

hipError_t launch_boundary_fill(const FillArgs& a, int prec, hipStream_t s) {
  if (a.nf < 1 || a.nf > kMaxFill) return hipErrorInvalidValue;
  long long fmax = 1;
  for (int b = 0; b < 3; ++b) fmax = std::max(fmax, (long long)a.N[0] * a.N[1] * a.N[2] / std::max(a.N[b], 1));
  if (fmax >= (1LL << 30)) return hipErrorInvalidValue;
  const dim3 grid((unsigned)std::min<long long>((fmax + 255) / 256, 1024), 6, (unsigned)a.nf);
  if (prec == 0) hipLaunchKernelGGL(k_boundary_fill<float>, grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL(k_boundary_fill<double>, grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace hp
