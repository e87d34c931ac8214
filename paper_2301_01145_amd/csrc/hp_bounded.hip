// Bounded (Dirichlet / Neumann) passes with one FFT per wavefront, for
// FFT lengths L = 32 .. 512 (powers of two), 48, 96 and 192 (hp_wavefft.hpp).
//
// The real-to-real transforms of Table 1 (DST-I/II/III, DCT-I/II/III) run as
// one complex FFT of length L on a pair of real pencils packed as a + ib.  The
// regular types extend each pencil to its symmetry:
//   DST-I   L = 2(n+1): [0, x_0..x_{n-1}, 0, -x_{n-1}..-x_0]
//   DCT-I   L = 2(n-1): [x_0..x_{n-1}, x_{n-2}..x_1]
// and every output is read from a single FFT bin.  The staggered types reorder
// it instead (r2r_build), L = n; types II, and the Hartley transform of a
// periodic axis of a mixed plan, take an output from the bins k and n - k
// (mirror_bin).  Lane g holds bins g + G i, so the outputs stay in the
// lanes that computed them.
//
// Passes (the pencil descriptors are those of the general path, in place in
// the output array): contiguous one-way passes load the pencil pair straight
// into the wavefront's LDS slot; strided passes stage a tile of P pencils
// (runs of P elements along the contiguous axis) through LDS; the sandwich
// pass transforms forward, multiplies by norm / sum_a lambda_a (Table 1,
// eq. pois_spec; 0 where the sum is 0) and transforms back before the tile is
// stored.  Inhomogeneous FD2 boundary terms are added while loading.
#include "hp_device.hpp"
#include "hp_faces.hpp"
#include "hp_internal.hpp"
#include "hp_wavefft.hpp"

namespace hp {

namespace {

__device__ __forceinline__ bool r2r_inverse_fft(int x) { return x == X_DCT3 || x == X_DST3; }

// Rows of a pencil that an FFT of length L transforms at most: the staggered
// types (H) use an FFT of their own length, the regular ones one of 2 (n + 1)
// or 2 (n - 1).
template <int L, bool H>
constexpr int kMaxRows = H ? L : L / 2 + 1;

// FFT input z[m] of the pair (a, b) for transform x of n points (FFT length
// L); get(s, w) is element s of pencil a (w = 0) or b (w = 1).
//
// The staggered types use an FFT of n points, half the symmetric extension
// (Makhoul's reordering; n even): type II transforms v[m] = x[2m], v[n-1-m] =
// x[2m+1] and takes the real part of q[k] V[k] afterwards (r2r_extract); type
// III starts from conj(q[k]) (c[k] - i c[n-k]) and puts the reals back in
// order.  The sine forms alternate signs and reverse the coefficients.  Against
// the extension: 128^3 FP32 Dirichlet 50.2 -> 44.1 us, FP64 77.6 -> 59.4, 256^3
// FP32 224 -> 184, 192^3 (FFT 384: general kernels) 201 -> 112; batches of eight
// 128^3 251 -> 188, of 32 96^3 582 -> 437, of 64 64^3 267 -> 205.  A first and
// last pass of 128^3 is bound by its launch and one memory latency either way.
template <typename T, class Get>
__device__ __forceinline__ C2<T> r2r_build(int x, int m, int n, int L, const C2<T>* q, Get get) {
  switch (x) {
    case X_DST1:
      if (m >= 1 && m <= n) return {get(m - 1, 0), get(m - 1, 1)};
      if (m > n + 1) return {-get(L - m - 1, 0), -get(L - m - 1, 1)};
      return {(T)0, (T)0};
    case X_DCT1: {
      const int s = m < n ? m : L - m;
      return {get(s, 0), get(s, 1)};
    }
    case X_DCT2:
    case X_DST2: {
      const bool even = 2 * m < n;
      const int s = even ? 2 * m : 2 * (n - m) - 1;
      C2<T> z = {get(s, 0), get(s, 1)};
      if (x == X_DST2 && !even) z = {-z.re, -z.im};
      return z;
    }
    case X_DCT3:
    case X_DST3: {
      const int s = x == X_DST3 ? n - 1 - m : m;
      const int sm = m == 0 ? s : (x == X_DST3 ? m - 1 : n - m);
      const C2<T> u = {get(s, 0), get(s, 1)};
      C2<T> um = {get(sm, 0), get(sm, 1)};
      if (m == 0) um = {(T)0, (T)0};
      const C2<T> d = {u.re + um.im, u.im - um.re}, w = q[m];
      return cmul_fixed(d, cconj(w));
    }
    case X_DHT: return {get(m, 0), get(m, 1)};
    default:
      return {(T)0, (T)0};
  }
}

// The bin n - k (0 for k = 0) of every bin k = g + G i that a lane holds:
// element R0 - 1 - i of lane G - g, lane 0's own ones in reverse.  (Types II
// separate the two pencils with it; one lane exchange per component instead
// of a second LDS exchange.)
template <typename T, int L>
__device__ __forceinline__ C2<T> mirror_bin(const C2<T> (&v)[WF<L>::R0], int i, int g) {
  constexpr int R0 = WF<L>::R0, G = WF<L>::G;
  const int from = ((int)(threadIdx.x & 63) & ~(G - 1)) + ((G - g) & (G - 1));
  const C2<T> o = v[(R0 - i) % R0];
  const C2<T> w = {__shfl(v[R0 - 1 - i].re, from, 64), __shfl(v[R0 - 1 - i].im, from, 64)};
  return g == 0 ? o : w;
}

// Output index carried by bin i of the lane (m = g + G i) of transform x (-1: none).
template <int L>
__device__ __forceinline__ int r2r_index(int x, int i, int g, int n) {
  const int m = g + WF<L>::G * i;
  switch (x) {
    case X_DST1: return m < 1 || m > n ? -1 : m - 1;
    case X_DCT1: return m < n ? m : -1;
    case X_DCT3:
    case X_DST3: return 2 * m < n ? 2 * m : 2 * (n - m) - 1;
    case X_DST2: return n - 1 - m;
    default: return m;  // DCT-II, Hartley
  }
}

// That index and the two real outputs (pencils a and b).
template <typename T, int L>
__device__ __forceinline__ int r2r_extract(int x, int i, int g, int n, const C2<T> (&v)[WF<L>::R0], const C2<T>* q,
                                           T& oa, T& ob) {
  const int m = g + WF<L>::G * i;
  const C2<T> z = v[i];
  const int k = r2r_index<L>(x, i, g, n);
  switch (x) {
    case X_DST1:
      oa = -z.im;
      ob = z.re;
      break;
    case X_DCT1:
      oa = z.re;
      ob = z.im;
      break;
    case X_DCT3:
    case X_DST3: {
      const T sg = (x == X_DST3 && 2 * m >= n) ? (T)-1 : (T)1;
      oa = sg * z.re;
      ob = sg * z.im;
    } break;
    case X_DCT2:
    case X_DST2: {
      const C2<T> c = cconj(mirror_bin<T, L>(v, i, g)), w = q[m];
      const C2<T> s = cadd(z, c), d = csub(z, c);
      oa = fma(s.re, w.re, -rounded(s.im * w.im));
      ob = fma(d.re, w.im, rounded(d.im * w.re));
    } break;
    default: {  // Hartley: Re - Im of either pencil's bin, from the bins k and n - k
      const C2<T> c = mirror_bin<T, L>(v, i, g);
      const T h = (T)0.5;
      oa = h * ((z.re + c.re) - (z.im - c.im));
      ob = h * ((z.im + c.im) + (z.re - c.re));
    } break;
  }
  return k;
}

__device__ __forceinline__ bool has_faces(const PassArgs& a) {
  bool f = false;
#pragma unroll
  for (int ax = 0; ax < 3; ++ax) f |= a.face[ax][0] != nullptr || a.face[ax][1] != nullptr;
  return f;
}

// Transform the pair held as reals by get() with transform x; on return
// v[i] holds bin g + G i.
template <typename T, int L, class Get>
__device__ __forceinline__ void r2r_fft(C2<T> (&v)[WF<L>::R0], int x, int n, C2<T>* slot, int g,
                                        const C2<T>* tw, const C2<T>* q, Get get) {
  constexpr int R0 = WF<L>::R0, G = WF<L>::G;
#pragma unroll
  for (int i = 0; i < R0; ++i) v[i] = r2r_build<T>(x, g + G * i, n, L, q, get);
  wave_sync();  // the FFT overwrites the slot the inputs may have come from
  if (r2r_inverse_fft(x)) wave_fft<T, L, true, false, false, true, true>(v, slot, 1, g, tw);
  else wave_fft<T, L, false, false, false, true, true>(v, slot, 1, g, tw);
}

// Runs f with the transform type as a compile-time constant: one branch per
// FFT (uniform per wavefront) instead of a switch per element.  H: one of the
// types of r2r_half, else one of the regular ones (a kernel holds one family).
template <bool H, class F>
__device__ __forceinline__ void with_xform(int x, F&& f) {
  if constexpr (H) {
    switch (x) {
      case X_DST2: f(std::integral_constant<int, X_DST2>{}); break;
      case X_DST3: f(std::integral_constant<int, X_DST3>{}); break;
      case X_DCT2: f(std::integral_constant<int, X_DCT2>{}); break;
      case X_DHT: f(std::integral_constant<int, X_DHT>{}); break;
      default: f(std::integral_constant<int, X_DCT3>{}); break;
    }
  } else {
    if (x == X_DST1) f(std::integral_constant<int, X_DST1>{});
    else f(std::integral_constant<int, X_DCT1>{});
  }
}

// Backward transform of the Table 1 pair that starts with forward type x.
__host__ __device__ constexpr int r2r_partner(int x) {
  return x == X_DST2 ? X_DST3 : (x == X_DCT2 ? X_DCT3 : x);
}

// Multiplier norm / (sum of the eigenvalues) at spectral index k along the
// pencil axis, given the eigenvalue sum `rest` of the other axes.
// (the eigenvalue sum is formed in FP64; an FP32 plan divides in FP32)
template <typename T>
__device__ __forceinline__ T eigen_mult(const PassArgs& a, int k, double rest) {
  const double lam = a.lam[a.ax_j][k] + rest;
  if (lam == 0.0) return (T)0;
  return (T)a.norm / (T)lam;
}

__device__ __forceinline__ double eigen_rest(const PassArgs& a, int p, int o) {
  double r = 0.0;
  if (a.ax_p >= 0) r += a.lam[a.ax_p][p];
  if (a.ax_o >= 0) r += a.lam[a.ax_o][o];
  return r;
}

}  // namespace

constexpr int kR2RContigWaves = 4;

// Boundary terms of the elements j = g + G r of pencil (p, o), added in the order
// of face_terms.  One face after the other for all of them, so that its loads are
// in flight together; element by element each waited for its own (64^3 staggered
// with values on every face 33.6 us, 31.3; 128^3 51.0, 47.7).
template <int NJ, int G, typename T>
__device__ __forceinline__ void add_faces(const PassArgs& a, T (&v)[NJ], int g, int p, int o, int n, bool live) {
  double add[NJ];
#pragma unroll
  for (int r = 0; r < NJ; ++r) add[r] = 0.0;
#pragma unroll
  for (int ax = 0; ax < 3; ++ax) {
#pragma unroll
    for (int side = 0; side < 2; ++side) {
      const T* f = (const T*)a.face[ax][side];
      if (!f) continue;
      const int edge = side == 0 ? 0 : a.nunk[ax] - 1;
      // the whole pencil lies beside the face, or one of its elements
      const bool along = ax != a.ax_j;
      if (along && (ax == a.ax_p ? p : o) != edge) continue;
      const int b0 = ax == 0 ? 1 : 0, b1 = ax == 2 ? 1 : 2;  // the face's axes, ascending
      auto at = [&](int b, int j) {
        return (long long)((a.ax_j == b ? j : (a.ax_p == b ? p : o)) + ((a.face_off >> b) & 1));
      };
      T w[NJ];
#pragma unroll
      for (int r = 0; r < NJ; ++r) {
        const int j = min(g + G * r, n - 1);
        long long off = 0;
        if (a.nunk[b0] > 0) off += at(b0, j) * a.face_s[ax][0];
        if (a.nunk[b1] > 0) off += at(b1, j) * a.face_s[ax][a.nunk[b0] > 0 ? 1 : 0];
        w[r] = (T)0;
        if (live && (along || j == edge)) w[r] = f[off];
      }
#pragma unroll
      for (int r = 0; r < NJ; ++r) add[r] += a.face_w[ax][side] * (double)w[r];
    }
  }
#pragma unroll
  for (int r = 0; r < NJ; ++r)
    if (live) v[r] = (T)((double)v[r] + add[r]);
}

// ----------------------------------------------- contiguous one-way pass
// Pairs (p, p+1) of pencils at one o; the pencil axis is unit stride.  CW
// wavefronts a workgroup (launch_bounded_L).
template <typename T, int L, bool H, int CW>
__global__ void __launch_bounds__(64 * CW) kb_contig(const PassArgs a) {
  constexpr int R0 = WF<L>::R0, G = WF<L>::G, PPW = WF<L>::PPW;
  constexpr int NT = 64 * CW;
  extern __shared__ __align__(16) unsigned char smem[];
  const int n = H ? L : a.n;
  C2<T>* tw = (C2<T>*)smem;
  C2<T>* q = tw + L;
  C2<T>* slots = q + n;
  for (int m = threadIdx.x; m < L; m += NT) tw[m] = ((const C2<T>*)a.tw)[m];
  if (a.qtw)
    for (int m = threadIdx.x; m < n; m += NT) q[m] = ((const C2<T>*)a.qtw)[m];
  __syncthreads();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int qq = lane / G, g = lane % G;
  C2<T>* slot = slots + (wave * PPW + qq) * slot_len(L);
  T* R = (T*)slot;  // the pair's reals: a at R[0..n), b at R[n..2n)
  const int pairs_p = (a.Np + 1) / 2;
  const long long total = (long long)pairs_p * a.No;
  const int blk = off_lines(a, sizeof(T), sizeof(T)) ? xcd_block(blockIdx.x, gridDim.x) : (int)blockIdx.x;
  const long long pr = ((long long)blk * CW + wave) * PPW + qq;
  const bool valid = pr < total;
  const int o = valid ? (int)(pr / pairs_p) : 0;
  const int pa = valid ? 2 * (int)(pr % pairs_p) : 0;
  const bool vb = valid && pa + 1 < a.Np;
  const bool faces = has_faces(a);
  const T* in = (const T*)a.in[0];
  const long long ib = (long long)o * a.in_so + (long long)pa * a.in_sp;
  // every load of the pair is issued before the first is used (n <= kMaxRows,
  // checked at launch): one memory latency per pass, not one per row
  constexpr int NJ = (kMaxRows<L, H> + G - 1) / G;
  T va[NJ], vbv[NJ];
  // (unconditional loads from clamped addresses: pencil pa + 1 only where it
  // exists, rows below n; the conditions apply where the values are kept)
  const long long ibb = ib + (vb ? a.in_sp : 0);
#pragma unroll
  for (int r = 0; r < NJ; ++r) {
    const long long jo = (long long)min(g + G * r, n - 1) * a.in_sj;
    va[r] = in[ib + jo];
    vbv[r] = in[ibb + jo];
  }
  if (faces) {
    add_faces<NJ, G>(a, va, g, pa, o, n, valid);
    add_faces<NJ, G>(a, vbv, g, pa + 1, o, n, vb);
  }
#pragma unroll
  for (int r = 0; r < NJ; ++r) {
    const int j = g + G * r;
    if (j < n) {
      R[j] = valid ? va[r] : (T)0;
      R[n + j] = vb ? vbv[r] : (T)0;
    }
  }
  wave_sync();
  T* out = (T*)a.out[0];
  const long long ob = (long long)o * a.out_so + (long long)pa * a.out_sp;
  with_xform<H>(a.xf, [&](auto XF) {
    constexpr int X = decltype(XF)::value;
    C2<T> v[R0];
    r2r_fft<T, L>(v, X, n, slot, g, tw, q, [&](int s, int w) { return R[w * n + s]; });
#pragma unroll
    for (int i = 0; i < R0; ++i) {
      T oa, obv;
      const int k = r2r_extract<T, L>(X, i, g, n, v, q, oa, obv);
      if (k < 0) continue;
      if (valid) st_stream(&out[ob + (long long)k * a.out_sj], oa);
      if (vb) st_stream(&out[ob + a.out_sp + (long long)k * a.out_sj], obv);
    }
  });
}

// ------------------------------------------- strided one-way and sandwich
// A tile is P pencils (p0 .. p0+P-1, o) whose pencil axis is strided; the
// contiguous axis is p.  The tile [n][P] (reals) is loaded as runs of P,
// wavefront pairs transform columns (2f, 2f+1) in place in it, and it is
// stored as runs of P.  SW: sandwich (forward, multiplier, backward).
//
// Four wavefronts at least load and store the tile, the first W transform it (one
// pair per lane group): the staggered types need half the lanes per pencil that
// their extension took, and with these alone the tile's accesses were a longer
// chain per thread (FP32 32^3 27.3 us, 23.9; 48^3 35.9, 30.6; 64^3 27.8, 25.8).
//
// PERS (persistent): a workgroup walks tiles blockIdx-strided; every thread
// loads its share of the next tile into registers before the current tile's
// FFTs and writes it to LDS after the current tile has been stored.  Chosen
// when there are many more tiles than resident workgroups.
// (Boundary terms enter in the contiguous first pass only.)
__host__ __device__ constexpr int strided_threads(int W) { return 64 * (W < 4 ? 4 : W); }
template <typename T, int L, bool H, int P, int W, bool SW, bool PERS>
__global__ void __launch_bounds__(strided_threads(W)) kb_strided(const PassArgs a) {
  constexpr int R0 = WF<L>::R0, G = WF<L>::G, PPW = WF<L>::PPW;
  constexpr int NT = strided_threads(W), TS = P + 1;
  constexpr int MAXN = kMaxRows<L, H>;           // rows of a tile at most
  constexpr int PER = (MAXN * P + NT - 1) / NT;  // tile elements per thread
  extern __shared__ __align__(16) unsigned char smem[];
  const int n = H ? L : a.n;
  C2<T>* tw = (C2<T>*)smem;
  C2<T>* q = tw + L;
  C2<T>* slots = q + n;
  T* tile = (T*)(slots + W * PPW * slot_len(L));
  const int tiles_p = (a.Np + P - 1) / P;
  const int ntiles = tiles_p * a.No;
  int t = off_lines(a, sizeof(T), sizeof(T)) ? xcd_block(blockIdx.x, gridDim.x) : (int)blockIdx.x;
  if (t >= ntiles) return;  // whole workgroup
  for (int m = threadIdx.x; m < L; m += NT) tw[m] = ((const C2<T>*)a.tw)[m];
  if (a.qtw)
    for (int m = threadIdx.x; m < n; m += NT) q[m] = ((const C2<T>*)a.qtw)[m];
  const T* in = (const T*)a.in[0];
  T* out = (T*)a.out[0];
  T pre[PER];
  auto fetch = [&](int tt) {
    const int o = tt / tiles_p, p0 = (tt % tiles_p) * P;
    const int np = min(P, a.Np - p0);
    const long long ib = (long long)o * a.in_so + (long long)p0 * a.in_sp;
    // unconditional loads from clamped (in-tile) addresses: no branches
    // between the loads, so all of them are in flight at once; put() drops
    // the rows beyond n and zeroes the pencils beyond np
#pragma unroll
    for (int r = 0; r < PER; ++r) {
      const int e = threadIdx.x + r * NT;
      const int j = e / P, c = e - (e / P) * P;
      pre[r] = in[ib + (long long)min(j, n - 1) * a.in_sj + (long long)min(c, np - 1) * a.in_sp];
    }
  };
  auto put = [&](int tt) {
    const int np = min(P, a.Np - (tt % tiles_p) * P);
#pragma unroll
    for (int r = 0; r < PER; ++r) {
      const int e = threadIdx.x + r * NT;
      const int j = e / P, c = e - (e / P) * P;
      if (j < n) tile[j * TS + c] = c < np ? pre[r] : (T)0;
    }
  };
  // the whole tile's loads in flight at once (registers, then LDS)
  fetch(t);
  put(t);
  __syncthreads();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int qq = lane / G, g_lane = lane % G;
  C2<T>* slot = slots + (wave * PPW + qq) * slot_len(L);
  for (;;) {
    const int o = t / tiles_p, p0 = (t % tiles_p) * P;
    const int np = min(P, a.Np - p0);
    const int nxt = PERS ? t + (int)gridDim.x : ntiles;
    if (PERS && nxt < ntiles) fetch(nxt);
    // the FFT's LDS addresses depend only on the lane: keep the compiler from
    // holding them in registers across the tile loop
    int g = g_lane;
    if constexpr (PERS) asm volatile("" : "+v"(g));
    static_assert(P / 2 == W * PPW, "one pair per wavefront lane group");
    if (wave < W) {
      const int f = wave * PPW + qq;  // pair: columns 2f, 2f + 1
      T* ca = tile + 2 * f;
      auto get = [&](int s, int w) { return ca[s * TS + w]; };
      // the sandwich's backward type is the Table 1 partner of its forward
      // type (checked at launch)
      with_xform<H>(a.xf, [&](auto XF) {
        constexpr int XFc = decltype(XF)::value;
        constexpr int XO = SW ? r2r_partner(XFc) : XFc;
        C2<T> v[R0];
        r2r_fft<T, L>(v, XFc, n, slot, g, tw, q, get);
        if constexpr (SW) {
          // spectra times the multiplier, back into the pair's columns
          const int pa = min(p0 + 2 * f, a.Np - 1), pb = min(p0 + 2 * f + 1, a.Np - 1);
          const double ra = eigen_rest(a, pa, o), rb = eigen_rest(a, pb, o);
#pragma unroll
          for (int i = 0; i < R0; ++i) {
            T sa, sb;
            const int k = r2r_extract<T, L>(XFc, i, g, n, v, q, sa, sb);
            if (k < 0) continue;
            ca[k * TS] = sa * eigen_mult<T>(a, k, ra);
            ca[k * TS + 1] = sb * eigen_mult<T>(a, k, rb);
          }
          wave_sync();
          r2r_fft<T, L>(v, XO, n, slot, g, tw, q, get);
        }
        // outputs into the pair's columns (the inputs were consumed above)
#pragma unroll
        for (int i = 0; i < R0; ++i) {
          T oa, obv;
          const int k = r2r_extract<T, L>(XO, i, g, n, v, q, oa, obv);
          if (k < 0) continue;
          ca[k * TS] = oa;
          ca[k * TS + 1] = obv;
        }
      });
      wave_sync();  // the slot is reused by the next pair
    }
    __syncthreads();
    const long long ob = (long long)o * a.out_so + (long long)p0 * a.out_sp;
    for (int e = threadIdx.x; e < n * P; e += NT) {
      const int j = e / P, c = e - (e / P) * P;
      if (c < np) st_stream(&out[ob + (long long)j * a.out_sj + (long long)c * a.out_sp], tile[j * TS + c]);
    }
    t = nxt;
    if (!PERS || t >= ntiles) break;
    __syncthreads();  // the tile has been read out
    put(t);
    __syncthreads();
  }
}

// ------------------------------------------------------- fan passes (FanJob)
// The passes of solves with series derivatives: a pencil pair is read once and
// transformed for the plain output and the derivative along the pencil.  One
// launch holds every array of a pass (job = blockIdx.y): the gradient of a 3D
// Dirichlet solve is 5 launches where one launch per array, with elementwise
// passes for the coefficients, was 16 (128^3 FP32 with its gradient: 81 us, was
// 168).  Rows off the cache lines are stored through the caches, where the parts
// of a line merge (127 points a row: 81 us, 85 streaming); aligned ones as the
// planner says (fan_stream).
namespace {

// Families of types: a kernel holds one (the instances of several need more
// registers than any of theirs alone).
enum Family : int { FAM_REGULAR = 0, FAM_STAGGERED = 1, FAM_HARTLEY = 2 };
__host__ __device__ constexpr int family(int x) {
  return x == X_DHT ? FAM_HARTLEY : (r2r_half(x) ? FAM_STAGGERED : FAM_REGULAR);
}
// The backward (forward) type as a compile-time constant.
template <int FAM, class F>
__device__ __forceinline__ void with_backward(int x, F&& f) {
  if constexpr (FAM == FAM_HARTLEY) {
    f(std::integral_constant<int, X_DHT>{});
  } else if constexpr (FAM == FAM_STAGGERED) {
    if (x == X_DST3) f(std::integral_constant<int, X_DST3>{});
    else f(std::integral_constant<int, X_DCT3>{});
  } else {
    if (x == X_DST1) f(std::integral_constant<int, X_DST1>{});
    else f(std::integral_constant<int, X_DCT1>{});
  }
}
template <int FAM, class F>
__device__ __forceinline__ void with_forward(int x, F&& f) {
  if constexpr (FAM == FAM_HARTLEY) {
    f(std::integral_constant<int, X_DHT>{});
  } else if constexpr (FAM == FAM_STAGGERED) {
    if (x == X_DST2) f(std::integral_constant<int, X_DST2>{});
    else f(std::integral_constant<int, X_DCT2>{});
  } else {
    if (x == X_DST1) f(std::integral_constant<int, X_DST1>{});
    else f(std::integral_constant<int, X_DCT1>{});
  }
}
// The stores of a fan pass, through the caches or streaming.
template <class F>
__device__ __forceinline__ void fan_stores(bool cached, F&& f) {
  if (cached) f(std::false_type{});
  else f(std::true_type{});
}
// Backward type of the derivative of a series with backward type x.
__host__ __device__ constexpr int r2r_other_parity(int x) {
  return x == X_DST1 ? X_DCT1 : (x == X_DCT1 ? X_DST1 : (x == X_DST3 ? X_DCT3 : (x == X_DCT3 ? X_DST3 : x)));
}

}  // namespace

template <typename T, int L, int FAM>
__global__ void __launch_bounds__(64 * kR2RContigWaves) kb_contig_fan(const PassArgs) {
  constexpr bool H = FAM != FAM_REGULAR;
  constexpr int R0 = WF<L>::R0, G = WF<L>::G, PPW = WF<L>::PPW;
  constexpr int NT = 64 * kR2RContigWaves;
  extern __shared__ __align__(16) unsigned char smem[];
  const PassArgs& a = kernel_args();
  const FanJob& job = a.fan[blockIdx.y];
  const int n = H ? L : job.n;
  C2<T>* tw = (C2<T>*)smem;
  C2<T>* q = tw + L;
  C2<T>* slots = q + a.n;
  for (int m = threadIdx.x; m < L; m += NT) tw[m] = ((const C2<T>*)a.tw)[m];
  if (a.qtw)
    for (int m = threadIdx.x; m < a.n; m += NT) q[m] = ((const C2<T>*)a.qtw)[m];
  __syncthreads();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int qq = lane / G, g = lane % G;
  C2<T>* slot = slots + (wave * PPW + qq) * slot_len(L);
  T* R = (T*)slot;  // the pair's reals, pencil b after pencil a
  const int pairs_p = (job.Np + 1) / 2;
  const long long total = (long long)pairs_p * job.No;
  const bool off = off_lines(a, sizeof(T), sizeof(T)), cached = off || !a.stream;
  const int blk = off ? xcd_block(blockIdx.x, gridDim.x) : (int)blockIdx.x;
  const long long pr = ((long long)blk * kR2RContigWaves + wave) * PPW + qq;
  const bool valid = pr < total;
  const int o = valid ? (int)(pr / pairs_p) : 0;
  const int pa = valid ? 2 * (int)(pr % pairs_p) : 0;
  const bool vb = valid && pa + 1 < job.Np;
  const T* in = (const T*)job.in;
  const long long ib = (long long)o * a.in_so + (long long)pa * a.in_sp;
  constexpr int NJ = (kMaxRows<L, H> + G - 1) / G;
  T va[NJ], vbv[NJ];
  const long long ibb = ib + (vb ? a.in_sp : 0);
#pragma unroll
  for (int r = 0; r < NJ; ++r) {
    const long long jo = (long long)min(g + G * r, n - 1) * a.in_sj;
    va[r] = valid ? in[ib + jo] : (T)0;
    vbv[r] = vb ? in[ibb + jo] : (T)0;
  }
  const long long ob = (long long)o * a.out_so + (long long)pa * a.out_sp;
  auto run = [&](auto XC, int cnt, void* dst) __attribute__((always_inline)) {
    constexpr int X = decltype(XC)::value;
    T* out = (T*)dst;
    C2<T> v[R0];
    r2r_fft<T, L>(v, X, cnt, slot, g, tw, q, [&](int s, int w) { return R[w * cnt + s]; });
    fan_stores(cached, [&](auto ST) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < R0; ++i) {
        T oa, obv;
        const int k = r2r_extract<T, L>(X, i, g, cnt, v, q, oa, obv);
        if (k < 0) continue;
        if (valid) st_out<decltype(ST)::value>(&out[ob + (long long)k * a.out_sj], oa);
        if (vb) st_out<decltype(ST)::value>(&out[ob + a.out_sp + (long long)k * a.out_sj], obv);
      }
    });
    wave_sync();  // the slot is filled again
  };
  if (job.deriv) {
    const int nd = H ? L : job.nd;
    // places that no coefficient reaches: the first and the last at most
    if (g == 0) R[0] = R[nd - 1] = R[nd] = R[2 * nd - 1] = (T)0;
    wave_sync();
#pragma unroll
    for (int r = 0; r < NJ; ++r) {
      const int j = g + G * r, s = fan_place<FAM == FAM_HARTLEY>(job, j);
      if (j < n && s >= 0 && s < nd) {
        const T m = (T)fan_factor<FAM == FAM_HARTLEY>(job, j);
        R[s] = m * va[r];
        R[nd + s] = m * vbv[r];
      }
    }
    wave_sync();
    with_backward<FAM>(job.xd, [&](auto XC) __attribute__((always_inline)) { run(XC, nd, job.deriv); });
  }
#pragma unroll
  for (int r = 0; r < NJ; ++r) {
    const int j = g + G * r;
    if (j < n) {
      R[j] = va[r];
      R[n + j] = vbv[r];
    }
  }
  wave_sync();
  with_backward<FAM>(job.xp, [&](auto XC) __attribute__((always_inline)) { run(XC, n, job.plain); });
}

// Strided fan pass and sandwich (kb_strided).  TWO: a tile for either transform;
// otherwise both run in one tile, one after the other, the input of a one-way
// pass or the spectrum of a sandwich waiting in registers for the second one.
// One tile lets more workgroups share a CU (four instead of two at 128 points:
// FP64 128^3, a sandwich 37.8 -> 24.3 us, a one-way pass of two arrays 38.1 ->
// 26.8), and costs two barriers and a store phase where every workgroup is
// resident anyway (64^3: 9.1 -> 9.5): the planner's rule is to_fast_r2r's
// (PassArgs.emit_dbl: two tiles).
template <typename T, int L, int FAM, int P, int W, bool SW, bool TWO>
__global__ void __launch_bounds__(64 * W) kb_strided_fan(const PassArgs) {
  constexpr bool H = FAM != FAM_REGULAR;
  constexpr int R0 = WF<L>::R0, G = WF<L>::G, PPW = WF<L>::PPW;
  constexpr int NT = 64 * W, TS = P + 1;
  constexpr int MAXN = kMaxRows<L, H>;
  constexpr int PER = (MAXN * P + NT - 1) / NT;
  extern __shared__ __align__(16) unsigned char smem[];
  const PassArgs& a = kernel_args();
  const FanJob& job = a.fan[blockIdx.y];
  const int n = H ? L : job.n, nd = H ? L : job.nd;
  C2<T>* tw = (C2<T>*)smem;
  C2<T>* q = tw + L;
  C2<T>* slots = q + a.n;
  T* tile = (T*)(slots + W * PPW * slot_len(L));
  T* dtile = TWO ? tile + n * TS : tile;
  const int tiles_p = (job.Np + P - 1) / P;
  const bool off = off_lines(a, sizeof(T), sizeof(T)), cached = off || !a.stream;
  const int t = off ? xcd_block(blockIdx.x, gridDim.x) : (int)blockIdx.x;
  if (t >= tiles_p * job.No) return;  // whole workgroup
  for (int m = threadIdx.x; m < L; m += NT) tw[m] = ((const C2<T>*)a.tw)[m];
  if (a.qtw)
    for (int m = threadIdx.x; m < a.n; m += NT) q[m] = ((const C2<T>*)a.qtw)[m];
  const int o = t / tiles_p, p0 = (t % tiles_p) * P;
  const int np = min(P, job.Np - p0);
  // the whole tile's loads in flight at once (kb_strided); pencils beyond np are 0
  T pre[PER];
  {
    const T* in = (const T*)job.in;
    const long long ib = (long long)o * a.in_so + (long long)p0 * a.in_sp;
#pragma unroll
    for (int r = 0; r < PER; ++r) {
      const int e = threadIdx.x + r * NT;
      const int j = e / P, c = e - (e / P) * P;
      pre[r] = in[ib + (long long)min(j, n - 1) * a.in_sj + (long long)min(c, np - 1) * a.in_sp];
    }
#pragma unroll
    for (int r = 0; r < PER; ++r) pre[r] = (int)(threadIdx.x + r * NT) % P < np ? pre[r] : (T)0;
  }
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int qq = lane / G, g = lane % G;
  C2<T>* slot = slots + (wave * PPW + qq) * slot_len(L);
  static_assert(P / 2 == W * PPW, "one pair per wavefront lane group");
  const int f = wave * PPW + qq;  // pair: columns 2f, 2f + 1
  T* ca = tile + 2 * f;
  T* da = dtile + 2 * f;
  // transform the pair's columns `col` in place (cnt points)
  auto back = [&](auto XC, T* col, int cnt) __attribute__((always_inline)) {
    constexpr int X = decltype(XC)::value;
    C2<T> v[R0];
    r2r_fft<T, L>(v, X, cnt, slot, g, tw, q, [&](int s, int w) { return col[s * TS + w]; });
#pragma unroll
    for (int i = 0; i < R0; ++i) {
      T oa, obv;
      const int k = r2r_extract<T, L>(X, i, g, cnt, v, q, oa, obv);
      if (k < 0) continue;
      col[k * TS] = oa;
      col[k * TS + 1] = obv;
    }
    wave_sync();  // the slot is used again
  };
  const long long ob = (long long)o * a.out_so + (long long)p0 * a.out_sp;
  auto store = [&](const T* src, int cnt, void* dst) {
    T* out = (T*)dst;
    fan_stores(cached, [&](auto ST) __attribute__((always_inline)) {
      for (int e = threadIdx.x; e < cnt * P; e += NT) {
        const int j = e / P, c = e - (e / P) * P;
        if (c < np) st_out<decltype(ST)::value>(&out[ob + (long long)j * a.out_sj + (long long)c * a.out_sp], src[j * TS + c]);
      }
    });
  };
  auto put_plain = [&] {
#pragma unroll
    for (int r = 0; r < PER; ++r) {
      const int e = threadIdx.x + r * NT;
      const int j = e / P, c = e - (e / P) * P;
      if (j < n) tile[j * TS + c] = pre[r];
    }
  };
  // places that no coefficient reaches: the first and the last at most
  auto zero_ends = [&] {
    if (g == 0) da[0] = da[1] = da[(nd - 1) * TS] = da[(nd - 1) * TS + 1] = (T)0;
    wave_sync();
  };
  // a derivative coefficient into its place
  const bool lap = SW && job.basis == FB_LAP;
  auto place = [&](int k, T va, T vb) {
    const int s = lap ? k : fan_place<FAM == FAM_HARTLEY>(job, k);
    if (s >= 0 && s < nd) {
      da[s * TS] = va;
      da[s * TS + 1] = vb;
    }
  };
  if constexpr (SW) {
    put_plain();
    __syncthreads();
    const int pa = min(p0 + 2 * f, job.Np - 1), pb = min(p0 + 2 * f + 1, job.Np - 1);
    const double ra = eigen_rest(a, pa, o), rb = eigen_rest(a, pb, o);
    auto w2 = [&](int ax, int k) {
      if (ax < 0) return 0.0;
      const double w = a.kc[ax] * (double)(a.basis[ax] == FB_SINE ? k + 1 : (a.basis[ax] == FB_COSINE ? k : signed_index(k, a.nunk[ax])));
      return w * w;
    };
    const double la = lap ? w2(a.ax_p, pa) + w2(a.ax_o, o) : 0.0, lb = lap ? w2(a.ax_p, pb) + w2(a.ax_o, o) : 0.0;
    with_forward<FAM>(a.xf, [&](auto XC) __attribute__((always_inline)) {
      constexpr int XF = decltype(XC)::value;
      constexpr int XB = r2r_partner(XF);
      T wa[TWO ? 1 : R0], wb[TWO ? 1 : R0];  // the derivative's coefficients
      {
        C2<T> v[R0];
        r2r_fft<T, L>(v, XF, n, slot, g, tw, q, [&](int s, int w) { return ca[s * TS + w]; });
        if constexpr (TWO) zero_ends();
#pragma unroll
        for (int i = 0; i < R0; ++i) {
          T sa, sb;
          const int k = r2r_extract<T, L>(XF, i, g, n, v, q, sa, sb);
          if (k < 0) continue;
          const double lam = a.lam[a.ax_j][k];
          const double ma = lam + ra == 0.0 ? 0.0 : a.norm / (lam + ra);
          const double mb = lam + rb == 0.0 ? 0.0 : a.norm / (lam + rb);
          // (the plain value with the multiplier of a solve without derivatives)
          ca[k * TS] = sa * eigen_mult<T>(a, k, ra);
          ca[k * TS + 1] = sb * eigen_mult<T>(a, k, rb);
          const double wj = lap ? w2(a.ax_j, k) : 0.0;
          const double fa = lap ? -job.scale * (wj + la) : fan_factor<FAM == FAM_HARTLEY>(job, k);
          const double fb = lap ? -job.scale * (wj + lb) : fa;
          const T va = sa * (T)(ma * fa), vb = sb * (T)(mb * fb);
          if constexpr (TWO) {
            place(k, va, vb);
          } else {
            wa[i] = va;
            wb[i] = vb;
          }
        }
        wave_sync();
      }
      back(std::integral_constant<int, XB>{}, ca, n);
      if constexpr (!TWO) {
        __syncthreads();
        store(tile, n, job.plain);
        __syncthreads();
        zero_ends();
#pragma unroll
        for (int i = 0; i < R0; ++i) {
          const int k = r2r_index<L>(XF, i, g, n);
          if (k >= 0) place(k, wa[i], wb[i]);
        }
        wave_sync();
      }
      if (lap) back(std::integral_constant<int, XB>{}, da, nd);
      else back(std::integral_constant<int, r2r_other_parity(XB)>{}, da, nd);
    });
    __syncthreads();
    if constexpr (TWO) store(tile, n, job.plain);
    store(dtile, nd, job.deriv);
  } else {
    if constexpr (TWO) {
      put_plain();
      __syncthreads();
      if (job.deriv) {
        zero_ends();
        for (int k = g; k < n; k += G) {
          const T m = (T)fan_factor<FAM == FAM_HARTLEY>(job, k);
          place(k, m * ca[k * TS], m * ca[k * TS + 1]);
        }
        wave_sync();
        with_backward<FAM>(job.xd, [&](auto XC) __attribute__((always_inline)) { back(XC, da, nd); });
      }
    } else {
      if (job.deriv) {
#pragma unroll
        for (int r = 0; r < PER; ++r) {
          const int e = threadIdx.x + r * NT;
          const int k = e / P, c = e - (e / P) * P;
          if (k >= n) continue;
          const int s = fan_place<FAM == FAM_HARTLEY>(job, k);
          if (s >= 0 && s < nd) tile[s * TS + c] = (T)fan_factor<FAM == FAM_HARTLEY>(job, k) * pre[r];
          // the places beside the first and the last coefficient's
          if (FAM != FAM_HARTLEY && k == 0 && s > 0) tile[c] = (T)0;
          if (FAM != FAM_HARTLEY && k == n - 1 && s + 1 < nd) tile[(s + 1) * TS + c] = (T)0;
        }
        __syncthreads();
        with_backward<FAM>(job.xd, [&](auto XC) __attribute__((always_inline)) { back(XC, ca, nd); });
        __syncthreads();
        store(tile, nd, job.deriv);
        __syncthreads();
      }
      put_plain();
      __syncthreads();
    }
    with_backward<FAM>(job.xp, [&](auto XC) __attribute__((always_inline)) { back(XC, ca, n); });
    __syncthreads();
    if (TWO && job.deriv) store(dtile, nd, job.deriv);
    store(tile, n, job.plain);
  }
}

// ------------------------------------------ batched solve
// A pass level of a batched plan (one pass of every problem) is one launch, one
// workgroup of kBatchWaves wavefronts per work item (consecutive tiles of one
// pass of one problem).  The tile bodies are those of kb_contig / kb_strided
// with the transform length and type as compile-time constants:
//   contiguous pass: a tile is kBatchWaves * PPW pencil pairs (one per lane
//     group) taken in (o, pair) order;
//   strided pass / sandwich: a tile is P = 32 pencils adjacent along the
//     contiguous axis (16 pairs), transformed by W = min(P / (2 PPW),
//     kBatchWaves) wavefronts, each lane group taking P / (2 W PPW) pairs in
//     turn; the workgroup holds S = kBatchWaves / W tiles at once (one per
//     group of W wavefronts).
// LDS: twiddles [L] | quarter twists [MAXN] | exchange slots | S tiles.
// Four wavefronts per workgroup keep the exchange slots small enough for
// three or four workgroups per CU at every length.  Stores go through the
// caches, never slower than streaming (64 problems of 64^3: 267 us, 279; 64 of
// 128^3, beyond the caches: 1918, 1917).
constexpr int kBatchWaves = 4;

namespace {

template <int L, bool H>
struct BW {
  static constexpr int PPW = WF<L>::PPW;
  static constexpr int P = 32;  // FP32 pencils per strided tile (128-byte runs)
  static constexpr int W = (P / 2) / PPW < kBatchWaves ? (P / 2) / PPW : kBatchWaves;
  static constexpr int PPL = (P / 2) / (W * PPW);  // pairs per lane group
  static constexpr int S = kBatchWaves / W;
  static constexpr int MAXN = kMaxRows<L, H>;
  static constexpr int TS = P + 1;
  static_assert(W >= 1 && kBatchWaves % W == 0 && PPL * W * PPW == P / 2, "batched strided tile");
};

// The fields of a pass that the tile bodies read.  The pass table and the work
// list are read through the constant address space: they do not change while
// the launch runs, so the reads are scalar loads into scalar registers.
struct BwArgs {
  int L, n, Np, No;
  long long in_sj, in_sp, in_so, out_sj, out_sp, out_so;
  const float* in;
  float* out;
  const C2<float>* tw;
  const C2<float>* qtw;
  const double* lam_j;  // eigenvalues along the pencil axis (sandwich)
  const double* lam_p;  // along the tile axis (null: none)
  const double* lam_o;  // along the outer axis (null: none)
  double norm;
};

using ConstPass = const __attribute__((address_space(4))) PassArgs;
using ConstItem = const __attribute__((address_space(4))) BatchItem;

__device__ __forceinline__ BwArgs bw_args(ConstPass* a) {
  BwArgs b;
  b.L = a->L;
  b.n = a->n;
  b.Np = a->Np;
  b.No = a->No;
  b.in_sj = a->in_sj;
  b.in_sp = a->in_sp;
  b.in_so = a->in_so;
  b.out_sj = a->out_sj;
  b.out_sp = a->out_sp;
  b.out_so = a->out_so;
  b.in = (const float*)a->in[0];
  b.out = (float*)a->out[0];
  b.tw = (const C2<float>*)a->tw;
  b.qtw = (const C2<float>*)a->qtw;
  const int aj = a->ax_j, ap = a->ax_p, ao = a->ax_o;
  b.lam_j = aj >= 0 ? a->lam[aj] : nullptr;
  b.lam_p = ap >= 0 ? a->lam[ap] : nullptr;
  b.lam_o = ao >= 0 ? a->lam[ao] : nullptr;
  b.norm = a->norm;
  return b;
}

// Load the twiddles of the pass (and the quarter-wave twists) into LDS.
template <int L>
__device__ __forceinline__ void bw_tables(const BwArgs& a, C2<float>* tw, C2<float>* q, int tid) {
  constexpr int NT = 64 * kBatchWaves;
  for (int m = tid; m < L; m += NT) tw[m] = a.tw[m];
  if (a.qtw)
    for (int m = tid; m < a.n; m += NT) q[m] = a.qtw[m];
}

template <int L, int X>
__device__ __forceinline__ void bw_contig(const BwArgs& a, unsigned char* smem, int tile, int ntile) {
  constexpr bool H = r2r_half(X);
  constexpr int R0 = WF<L>::R0, G = WF<L>::G, PPW = WF<L>::PPW;
  using T = float;
  const int n = H ? L : a.n;
  C2<T>* tw = (C2<T>*)smem;
  C2<T>* q = tw + L;
  C2<T>* slots = q + BW<L, H>::MAXN;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int qq = lane / G, g = lane % G;
  C2<T>* slot = slots + (wave * PPW + qq) * slot_len(L);
  T* R = (T*)slot;
  // (every axis has at most 256 points: 32 bits count the pairs)
  const unsigned pairs_p = (a.Np + 1) / 2, total = pairs_p * a.No;
  for (int k = 0; k < ntile; ++k) {
    const unsigned pr = ((tile + k) * kBatchWaves + wave) * PPW + qq;
    const bool valid = pr < total;
    const int o = valid ? (int)(pr / pairs_p) : 0;
    const int pa = valid ? 2 * (int)(pr % pairs_p) : 0;
    const bool vb = valid && pa + 1 < a.Np;
    const long long ib = (long long)o * a.in_so + (long long)pa * a.in_sp;
    // every load of the pair in flight at once (compile-time trip count,
    // addresses clamped to the array), the tables' loads behind them
    constexpr int NJ = (BW<L, H>::MAXN + G - 1) / G;
    T va[NJ], vbv[NJ];
    const long long ibb = ib + (vb ? a.in_sp : 0);
#pragma unroll
    for (int r = 0; r < NJ; ++r) {
      const long long jo = (long long)min(g + r * G, n - 1) * a.in_sj;
      va[r] = a.in[ib + jo];
      vbv[r] = a.in[ibb + jo];
    }
    if (k == 0) bw_tables<L>(a, tw, q, tid);
#pragma unroll
    for (int r = 0; r < NJ; ++r) {
      const int j = g + r * G;
      if (j < n) {
        R[j] = valid ? va[r] : (T)0;
        R[n + j] = vb ? vbv[r] : (T)0;
      }
    }
    if (k == 0) __syncthreads();
    else wave_sync();
    const long long ob = (long long)o * a.out_so + (long long)pa * a.out_sp;
    C2<T> v[R0];
    r2r_fft<T, L>(v, X, n, slot, g, tw, q, [&](int s, int w) { return R[w * n + s]; });
#pragma unroll
    for (int i = 0; i < R0; ++i) {
      T oa, obv;
      const int kk = r2r_extract<T, L>(X, i, g, n, v, q, oa, obv);
      if (kk < 0) continue;
      if (valid) a.out[ob + (long long)kk * a.out_sj] = oa;
      if (vb) a.out[ob + a.out_sp + (long long)kk * a.out_sj] = obv;
    }
    wave_sync();  // the slot is reused by the next pair
  }
}

template <int L, int XF, int XO, bool SW>
__device__ __forceinline__ void bw_strided(const BwArgs& a, unsigned char* smem, int tile, int ntile) {
  constexpr bool H = r2r_half(XF);
  constexpr int R0 = WF<L>::R0, G = WF<L>::G, PPW = WF<L>::PPW;
  constexpr int P = BW<L, H>::P, W = BW<L, H>::W, S = BW<L, H>::S, TS = BW<L, H>::TS, PPL = BW<L, H>::PPL;
  constexpr int MAXN = BW<L, H>::MAXN, NTS = 64 * W;
  using T = float;
  const int n = H ? L : a.n;
  C2<T>* tw = (C2<T>*)smem;
  C2<T>* q = tw + L;
  C2<T>* slots = q + MAXN;
  T* tiles = (T*)(slots + kBatchWaves * PPW * slot_len(L));
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int sub = wave / W, wv = wave - sub * W;  // tile group and wavefront in it
  const int ts = tid - sub * NTS;                  // thread in the group
  const int qq = lane / G, g = lane % G;
  C2<T>* slot = slots + (wave * PPW + qq) * slot_len(L);
  T* tile_s = tiles + sub * MAXN * TS;
  const int tiles_p = (a.Np + P - 1) / P;
  for (int base = 0; base < ntile; base += S) {
    const bool active = base + sub < ntile;
    const int t = tile + base + sub;
    const int o = active ? t / tiles_p : 0, p0 = active ? (t % tiles_p) * P : 0;
    const int np = active ? min(P, a.Np - p0) : 0;
    const long long ib = (long long)o * a.in_so + (long long)p0 * a.in_sp;
    // a batch of loads in flight per thread before their LDS stores: one load at
    // a time waits out the memory latency once per element.  The staggered types
    // (tiles of exactly [L][P]) take the whole tile at once, the others, whose
    // FFT needs twice the registers, eight rows (a whole tile spilled).
    // Addresses are clamped to the array; np = 0: the group's tile is idle.
    constexpr int U = H ? MAXN * P / NTS : 8;
    for (int e0 = ts; e0 < n * P; e0 += U * NTS) {
      T v8[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = e0 + u * NTS;
        const int j = min(e / P, n - 1), c = max(min(e % P, np - 1), 0);
        v8[u] = a.in[ib + (long long)j * a.in_sj + (long long)c * a.in_sp];
      }
      if (base == 0 && e0 == ts) bw_tables<L>(a, tw, q, tid);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = e0 + u * NTS;
        if (e < n * P) tile_s[(e / P) * TS + e % P] = e % P < np ? v8[u] : (T)0;
      }
    }
    __syncthreads();
    for (int r = 0; r < PPL && active; ++r) {
      const int f = (r * W + wv) * PPW + qq;  // pair: columns 2f, 2f + 1
      T* ca = tile_s + 2 * f;
      auto get = [&](int s, int w) { return ca[s * TS + w]; };
      C2<T> v[R0];
      r2r_fft<T, L>(v, XF, n, slot, g, tw, q, get);
      if constexpr (SW) {
        // multiplier norm / (sum of the eigenvalues), FP64 sum (Table 1)
        const int pa = min(p0 + 2 * f, a.Np - 1), pb = min(p0 + 2 * f + 1, a.Np - 1);
        const double ro = a.lam_o ? a.lam_o[o] : 0.0;
        const double ra = ro + (a.lam_p ? a.lam_p[pa] : 0.0), rb = ro + (a.lam_p ? a.lam_p[pb] : 0.0);
#pragma unroll
        for (int i = 0; i < R0; ++i) {
          T sa, sb;
          const int k = r2r_extract<T, L>(XF, i, g, n, v, q, sa, sb);
          if (k < 0) continue;
          const double la = a.lam_j[k] + ra, lb = a.lam_j[k] + rb;
          ca[k * TS] = la == 0.0 ? (T)0 : sa * ((T)a.norm / (T)la);
          ca[k * TS + 1] = lb == 0.0 ? (T)0 : sb * ((T)a.norm / (T)lb);
        }
        wave_sync();
        r2r_fft<T, L>(v, XO, n, slot, g, tw, q, get);
      }
#pragma unroll
      for (int i = 0; i < R0; ++i) {
        T oa, obv;
        const int k = r2r_extract<T, L>(XO, i, g, n, v, q, oa, obv);
        if (k < 0) continue;
        ca[k * TS] = oa;
        ca[k * TS + 1] = obv;
      }
      wave_sync();  // the slot is reused by the next pair
    }
    __syncthreads();
    const long long ob = (long long)o * a.out_so + (long long)p0 * a.out_sp;
    for (int e = ts; e < n * P; e += NTS) {
      const int j = e / P, c = e - (e / P) * P;
      if (c < np) a.out[ob + (long long)j * a.out_sj + (long long)c * a.out_sp] = tile_s[j * TS + c];
    }
    __syncthreads();  // the tiles are reloaded by the next step
  }
}

// One item of kind KIND: 0 / 1 contiguous pass of type XF / XB, 2 / 3 strided
// pass of type XF / XB, 4 sandwich (XF, multiplier, XB).
template <int L, int XF, int XB, int KIND>
__device__ __forceinline__ void bw_item(const BwArgs& a, unsigned char* smem, int tile, int ntile) {
  if constexpr (KIND == 0) bw_contig<L, XF>(a, smem, tile, ntile);
  else if constexpr (KIND == 1) bw_contig<L, XB>(a, smem, tile, ntile);
  else if constexpr (KIND == 2) bw_strided<L, XF, XF, false>(a, smem, tile, ntile);
  else if constexpr (KIND == 3) bw_strided<L, XB, XB, false>(a, smem, tile, ntile);
  else bw_strided<L, XF, XB, true>(a, smem, tile, ntile);
}

__device__ __forceinline__ BatchItem bw_take(const BatchItem* items) {
  ConstItem* it = (ConstItem*)items + blockIdx.x;
  BatchItem b;
  b.pass = it->pass;
  b.tile = it->tile;
  b.ntile = it->ntile;
  return b;
}

// One pass level of the batch, every transform length in one launch: the
// workgroups of a level are independent, so the lengths run side by side and
// a solve is one launch per level (8 problems of 32 to 128 cells per axis: 85 us
// against 174 with a launch per level and length; 64 problems: 484 and 609).
template <int XF, int XB, int KIND>
__global__ void __launch_bounds__(64 * kBatchWaves, 4)
    k_batched_pass(const PassArgs* passes, const BatchItem* items) {
  extern __shared__ __align__(16) unsigned char smem[];
  const BatchItem bi = bw_take(items);
  const BwArgs a = bw_args((ConstPass*)passes + bi.pass);
  if constexpr (r2r_half(XF)) {
    switch (a.L) {
      case 32: bw_item<32, XF, XB, KIND>(a, smem, bi.tile, bi.ntile); break;
      case 48: bw_item<48, XF, XB, KIND>(a, smem, bi.tile, bi.ntile); break;
      case 64: bw_item<64, XF, XB, KIND>(a, smem, bi.tile, bi.ntile); break;
      case 96: bw_item<96, XF, XB, KIND>(a, smem, bi.tile, bi.ntile); break;
      default: bw_item<128, XF, XB, KIND>(a, smem, bi.tile, bi.ntile); break;
    }
  } else {
    switch (a.L) {
      case 64: bw_item<64, XF, XB, KIND>(a, smem, bi.tile, bi.ntile); break;
      case 96: bw_item<96, XF, XB, KIND>(a, smem, bi.tile, bi.ntile); break;
      case 128: bw_item<128, XF, XB, KIND>(a, smem, bi.tile, bi.ntile); break;
      case 192: bw_item<192, XF, XB, KIND>(a, smem, bi.tile, bi.ntile); break;
      default: bw_item<256, XF, XB, KIND>(a, smem, bi.tile, bi.ntile); break;
    }
  }
}

// One pass level of the batch for one transform length L and one pass kind
// (the passes of every problem that have no dependency left, transform along
// L and are of that kind): one workgroup per item, no queue, no waiting; the
// launch boundaries order the levels.  One instance per (L, kind) holds a
// single tile body, register-allocated like the single-plan kernels (all
// lengths and kinds in one kernel did not fit in 128 VGPRs).
// KIND: 0 / 1 contiguous pass of type XF / XB, 2 / 3 strided pass of type
// XF / XB, 4 sandwich (XF, multiplier, XB).
template <int XF, int XB, int L, int KIND>
__global__ void __launch_bounds__(64 * kBatchWaves, 4)
    k_batched_level(const PassArgs* passes, const BatchItem* items) {
  extern __shared__ __align__(16) unsigned char smem[];
  const BatchItem bi = bw_take(items);
  bw_item<L, XF, XB, KIND>(bw_args((ConstPass*)passes + bi.pass), smem, bi.tile, bi.ntile);
}

template <int XF, int XB, int L, int KIND>
hipError_t bw_launch_group(const PassArgs* passes, const BatchItem* items, int n, int lds, hipStream_t s) {
  if constexpr (L == 0) {
    allow_lds<k_batched_pass<XF, XB, KIND>>();
    hipLaunchKernelGGL((k_batched_pass<XF, XB, KIND>), dim3(n), dim3(64 * kBatchWaves), lds, s, passes, items);
  } else {
    allow_lds<k_batched_level<XF, XB, L, KIND>>();
    hipLaunchKernelGGL((k_batched_level<XF, XB, L, KIND>), dim3(n), dim3(64 * kBatchWaves), lds, s, passes,
                       items);
  }
  return hipGetLastError();
}

template <int XF, int XB, int L>
hipError_t bw_launch_kind(const BatchGroup& g, const PassArgs* passes, const BatchItem* it, hipStream_t s) {
  switch (g.kind) {
    case 0: return bw_launch_group<XF, XB, L, 0>(passes, it, g.count, g.lds, s);
    case 1: return bw_launch_group<XF, XB, L, 1>(passes, it, g.count, g.lds, s);
    case 2: return bw_launch_group<XF, XB, L, 2>(passes, it, g.count, g.lds, s);
    case 3: return bw_launch_group<XF, XB, L, 3>(passes, it, g.count, g.lds, s);
    case 4: return bw_launch_group<XF, XB, L, 4>(passes, it, g.count, g.lds, s);
    default: return hipErrorInvalidValue;
  }
}

template <int XF, int XB>
hipError_t bw_launch_one(const BatchGroup& g, const PassArgs* passes, const BatchItem* items, hipStream_t s) {
  if (g.count <= 0) return hipSuccess;
  const BatchItem* it = items + g.first;
  switch (g.L) {
    case 0: return bw_launch_kind<XF, XB, 0>(g, passes, it, s);
    case 64: return bw_launch_kind<XF, XB, 64>(g, passes, it, s);
    case 96: return bw_launch_kind<XF, XB, 96>(g, passes, it, s);
    case 128: return bw_launch_kind<XF, XB, 128>(g, passes, it, s);
    default: break;
  }
  if constexpr (r2r_half(XF)) {
    if (g.L == 32) return bw_launch_kind<XF, XB, 32>(g, passes, it, s);
    if (g.L == 48) return bw_launch_kind<XF, XB, 48>(g, passes, it, s);
  } else {
    if (g.L == 192) return bw_launch_kind<XF, XB, 192>(g, passes, it, s);
    if (g.L == 256) return bw_launch_kind<XF, XB, 256>(g, passes, it, s);
  }
  return hipErrorInvalidValue;
}

// f(L, H) as compile-time constants for the lengths of batched_wf_length;
// false: no such length.
template <class F>
bool with_batch_length(int L, bool half, F&& f) {
  auto go = [&](auto Lc, auto Hc) {
    f(Lc, Hc);
    return true;
  };
  using std::integral_constant;
  if (half) {
    switch (L) {
      case 32: return go(integral_constant<int, 32>{}, std::true_type{});
      case 48: return go(integral_constant<int, 48>{}, std::true_type{});
      case 64: return go(integral_constant<int, 64>{}, std::true_type{});
      case 96: return go(integral_constant<int, 96>{}, std::true_type{});
      case 128: return go(integral_constant<int, 128>{}, std::true_type{});
      default: return false;
    }
  }
  switch (L) {
    case 64: return go(integral_constant<int, 64>{}, std::false_type{});
    case 96: return go(integral_constant<int, 96>{}, std::false_type{});
    case 128: return go(integral_constant<int, 128>{}, std::false_type{});
    case 192: return go(integral_constant<int, 192>{}, std::false_type{});
    case 256: return go(integral_constant<int, 256>{}, std::false_type{});
    default: return false;
  }
}

}  // namespace

bool batched_wf_length(int L, bool half) {
  return with_batch_length(L, half, [](auto, auto) {});
}

int batched_wf_lds(const PassArgs& a) {
  int lds = -1;
  with_batch_length(a.L, r2r_half(a.xf), [&](auto Lc, auto Hc) {
    constexpr int L = decltype(Lc)::value;
    using B = BW<L, decltype(Hc)::value>;
    lds = (L + B::MAXN + kBatchWaves * B::PPW * slot_len(L)) * 8;
    if (a.fast != FAST_R2R_C) lds += B::S * B::MAXN * B::TS * 4;
  });
  return lds;
}

int batched_wf_tiles(const PassArgs& a) {
  if (a.fast != FAST_R2R_C) return ((a.Np + 31) / 32) * a.No;
  int tiles = 0;
  with_batch_length(a.L, r2r_half(a.xf), [&](auto Lc, auto) {
    const long long pairs = (long long)((a.Np + 1) / 2) * a.No;
    const long long per = (long long)kBatchWaves * WF<decltype(Lc)::value>::PPW;
    tiles = (int)((pairs + per - 1) / per);
  });
  return tiles;
}

int batched_wf_group(const PassArgs& a) {
  if (a.fast == FAST_R2R_C) return 1;
  int s = 1;
  with_batch_length(a.L, r2r_half(a.xf), [&](auto Lc, auto Hc) {
    s = BW<decltype(Lc)::value, decltype(Hc)::value>::S;
  });
  return s;
}

hipError_t launch_batched_group(int xf, const PassArgs* passes, const BatchItem* items,
                                const BatchGroup& g, hipStream_t s) {
  if (xf == X_DCT2) return bw_launch_one<X_DCT2, X_DCT3>(g, passes, items, s);
  if (xf == X_DST2) return bw_launch_one<X_DST2, X_DST3>(g, passes, items, s);
  if (xf == X_DCT1) return bw_launch_one<X_DCT1, X_DCT1>(g, passes, items, s);
  return hipErrorInvalidValue;
}

// ---------------------------------------------------------------- launch
// Pencils per tile of the strided passes: runs of 128 bytes (FP64 at length 32:
// 256, the 16 pairs that one wavefront transforms).
static constexpr int r2r_tile_of(int L, bool f32) { return f32 || L == 32 ? 32 : 16; }
int r2r_tile(int L, int prec) { return r2r_tile_of(L, prec == 0); }

// Wavefronts per strided workgroup: one per pair (PPW pairs per wavefront
// for short transforms).
constexpr int r2r_waves(int P, int ppw) { return (P / 2) / ppw; }

// LDS bytes of a strided pass with `rows` tile rows (n quarter twists); -1: a
// tile's pairs do not fill whole wavefronts (one pair per lane group).
static constexpr int r2r_strided_lds(int L, int n, int rows, int prec) {
  const int cs = prec == 0 ? 8 : 16, es = cs / 2, P = r2r_tile_of(L, prec == 0), ppw = 64 / (L / wf_r0(L));
  if ((P / 2) % ppw != 0) return -1;
  return (L + n + r2r_waves(P, ppw) * ppw * slot_len(L)) * cs + rows * (P + 1) * es;
}
// n: rows of the tile (and quarter twists), nd: rows of a second tile (0: none).
int r2r_lds_bytes(int fast, int L, int n, int nd, int prec) {
  const int R0 = wf_r0(L);
  if (R0 <= 0 || (R0 % 3 == 0 && prec != 0)) return -1;  // 3 x 2^k: FP32 only
  if (fast == FAST_R2R_C) return (L + n + kR2RContigWaves * (64 / (L / R0)) * slot_len(L)) * (prec == 0 ? 8 : 16);
  return r2r_strided_lds(L, n, n + nd, prec);
}
// Whether one tile instead of two (n rows each) lets a fan pass of FFT length L
// have more workgroups on a CU.
static constexpr bool r2r_one_tile(int L, int n, int prec) {
  const int one = r2r_strided_lds(L, n, n, prec), two = r2r_strided_lds(L, n, 2 * n, prec);
  return one > 0 && (160 * 1024) / one > (160 * 1024) / two;
}
bool fan_one_tile(int fast, int L, bool half, int prec) {
  if (wf_r0(L) <= 0 || fast == FAST_R2R_C || (fast == FAST_R2R_SW && wf_r0(L) % 3 == 0)) return false;
  return r2r_one_tile(L, half ? L : L / 2, prec);
}

namespace {

template <typename T, int L, int FAM>
hipError_t launch_fan_L(const PassArgs& a, hipStream_t s) {
  constexpr bool H = FAM != FAM_REGULAR;
  constexpr int PPW = WF<L>::PPW;
  constexpr int P = r2r_tile_of(L, sizeof(T) == 4);
  constexpr int W = r2r_waves(P, PPW);
  if (a.nfan > kMaxFan || a.P != P) return hipErrorInvalidValue;
  long long blocks = 0;
  int rows = 0, drows = 0;
  for (int i = 0; i < a.nfan; ++i) {
    const FanJob& q = a.fan[i];
    if (!q.in || !q.plain || q.n < 1 || q.n > kMaxRows<L, H> || q.Np < 1 || q.No < 1) return hipErrorInvalidValue;
    if (q.deriv && (q.nd < 1 || q.nd > kMaxRows<L, H> || q.basis == FB_ODD)) return hipErrorInvalidValue;
    // one family of types per kernel; all but the regular ones have L points
    if (family(q.xp) != FAM || (q.deriv && family(q.xd) != FAM)) return hipErrorInvalidValue;
    if (q.deriv && q.basis != FB_LAP && (q.basis == FB_HARTLEY) != (FAM == FAM_HARTLEY)) return hipErrorInvalidValue;
    if (H && (q.n != L || a.n != L || (q.deriv && q.nd != L))) return hipErrorInvalidValue;
    const long long per = (long long)kR2RContigWaves * PPW;
    blocks = std::max(blocks, a.fast == FAST_R2R_C ? ((long long)((q.Np + 1) / 2) * q.No + per - 1) / per
                                                   : (long long)((q.Np + P - 1) / P) * q.No);
    rows = std::max(rows, q.n);
    if (q.deriv) drows = std::max(drows, q.nd);
  }
  const bool two = a.emit_dbl != 0;
  rows = std::max(rows, a.n);
  if (r2r_lds_bytes(a.fast, L, two ? rows : std::max(rows, drows), two ? drows : 0, sizeof(T) == 8) > a.lds_bytes ||
      a.lds_bytes > 160 * 1024)
    return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks, a.nfan);
  if (a.fast == FAST_R2R_C) {
    allow_lds<kb_contig_fan<T, L, FAM>>();
    hipLaunchKernelGGL((kb_contig_fan<T, L, FAM>), grid, dim3(64 * kR2RContigWaves), a.lds_bytes, s, a);
    return hipGetLastError();
  }
  if constexpr (W < 1 || (P / 2) % PPW != 0) {
    return hipErrorInvalidValue;
  } else {
    const bool sw = a.fast == FAST_R2R_SW;
    if (sw && (a.xb != r2r_partner(a.xf) || a.nfan != 1 || !a.fan[0].deriv)) return hipErrorInvalidValue;
    auto go = [&](auto S, auto B) {
      constexpr bool SW = decltype(S)::value, TWO = decltype(B)::value;
      allow_lds<kb_strided_fan<T, L, FAM, P, W, SW, TWO>>();
      hipLaunchKernelGGL((kb_strided_fan<T, L, FAM, P, W, SW, TWO>), grid, dim3(64 * W), a.lds_bytes, s, a);
    };
    // (one-tile instances where r2r_one_tile can ask for them)
    constexpr bool kOne = r2r_one_tile(L, H ? L : L / 2, sizeof(T) == 8);
    if constexpr (kOne) {
      if (!two && !sw) { go(std::false_type{}, std::false_type{}); return hipGetLastError(); }
      if constexpr (WF<L>::R0 % 3 != 0) {
        if (!two) { go(std::true_type{}, std::false_type{}); return hipGetLastError(); }
      }
    }
    if (!two) return hipErrorInvalidValue;
    if (sw) go(std::true_type{}, std::true_type{});
    else go(std::false_type{}, std::true_type{});
  }
  return hipGetLastError();
}

// Workgroups of a persistent strided pass; HP_PERSIST=<n>, n > 0, caps them, which
// makes passes of few tiles persistent too (a pass of more than four tiles per
// workgroup is).
template <auto K>
int strided_grid(int nt, int lds, int ntiles) {
  const int nb = persistent_grid<K>(nt, lds, ntiles);
  const char* e = std::getenv("HP_PERSIST");
  const int cap = e ? std::atoi(e) : 0;
  return cap > 0 ? std::min(nb, cap) : nb;
}

template <typename T, int L, bool H>
hipError_t launch_bounded_L(const PassArgs& a, hipStream_t s) {
  constexpr int PPW = WF<L>::PPW;
  const int lds = a.lds_bytes;
  // rows per pencil of every Table 1 type
  if (H ? a.n != L : (a.n < 1 || a.n > L / 2 + 1)) return hipErrorInvalidValue;
  if (a.nfan > 0) {
    if constexpr (H && L >= 64) {  // (shorter Hartley passes stay general)
      if (a.fan[0].xp == X_DHT) return launch_fan_L<T, L, FAM_HARTLEY>(a, s);
    }
    return launch_fan_L<T, L, H ? FAM_STAGGERED : FAM_REGULAR>(a, s);
  }
  if (a.fast == FAST_R2R_C) {
    const long long waves = ((long long)((a.Np + 1) / 2) * a.No + PPW - 1) / PPW;
    auto go = [&](auto C) {
      constexpr int CW = decltype(C)::value;
      allow_lds<kb_contig<T, L, H, CW>>();
      hipLaunchKernelGGL((kb_contig<T, L, H, CW>), dim3((unsigned)((waves + CW - 1) / CW)), dim3(64 * CW), lds, s, a);
    };
    // short staggered pencils (8 or 16 pairs a wavefront): a wavefront a workgroup
    // where that leaves no CU two of them (FP32 32^3 23.9 -> 22.1 us, 128 x 64 x 32 28.0 ->
    // 27.2; but 128 x 128 x 64, 1024 wavefronts, 33.1 -> 34.8)
    if constexpr (H && L <= 64) {
      if (waves <= 256) {
        go(std::integral_constant<int, 1>{});
        return hipGetLastError();
      }
    }
    go(std::integral_constant<int, kR2RContigWaves>{});
    return hipGetLastError();
  }
  constexpr int P = r2r_tile_of(L, sizeof(T) == 4);
  constexpr int W = r2r_waves(P, PPW);
  if (a.P != P) return hipErrorInvalidValue;
  if constexpr (W < 1 || (P / 2) % PPW != 0) {
    return hipErrorInvalidValue;  // the planner keeps such passes on the general kernels
  } else {
    const dim3 grid((unsigned)(((a.Np + P - 1) / P) * a.No));
    const int ntiles = (int)grid.x;
    // radix-12 lengths: the register prefetch of the persistent form would
    // cost occupancy, so their tiles are one workgroup each
    constexpr bool kPers = WF<L>::R0 % 3 != 0;
    if (a.fast == FAST_R2R_SW) {
      if (a.xb != r2r_partner(a.xf)) return hipErrorInvalidValue;
      if constexpr (kPers) {
        allow_lds<kb_strided<T, L, H, P, W, true, true>>();
        const int nb = strided_grid<kb_strided<T, L, H, P, W, true, true>>(strided_threads(W), lds, ntiles);
        if (ntiles > 4 * nb && !std::getenv("HP_R2R_NOPERS")) {
          hipLaunchKernelGGL((kb_strided<T, L, H, P, W, true, true>), dim3(nb), dim3(strided_threads(W)), lds, s, a);
          return hipGetLastError();
        }
      }
      allow_lds<kb_strided<T, L, H, P, W, true, false>>();
      hipLaunchKernelGGL((kb_strided<T, L, H, P, W, true, false>), grid, dim3(strided_threads(W)), lds, s, a);
    } else {
      if constexpr (kPers) {
        allow_lds<kb_strided<T, L, H, P, W, false, true>>();
        const int nb = strided_grid<kb_strided<T, L, H, P, W, false, true>>(strided_threads(W), lds, ntiles);
        if (ntiles > 4 * nb) {
          hipLaunchKernelGGL((kb_strided<T, L, H, P, W, false, true>), dim3(nb), dim3(strided_threads(W)), lds, s, a);
          return hipGetLastError();
        }
      }
      allow_lds<kb_strided<T, L, H, P, W, false, false>>();
      hipLaunchKernelGGL((kb_strided<T, L, H, P, W, false, false>), grid, dim3(strided_threads(W)), lds, s, a);
    }
    return hipGetLastError();
  }
}

template <typename T>
hipError_t launch_bounded_T(const PassArgs& a, hipStream_t s) {
  // 3 x 2^k lengths: FP32 only (radix-12 first stage; FP64 stays on the
  // general kernels, see r2r_lds_bytes)
  if constexpr (sizeof(T) == 4) {
    if (wf_half(a)) {
      if (a.L == 48) return launch_bounded_L<T, 48, true>(a, s);
      if (a.L == 96) return launch_bounded_L<T, 96, true>(a, s);
      if (a.L == 192) return launch_bounded_L<T, 192, true>(a, s);
    } else {
      if (a.L == 96) return launch_bounded_L<T, 96, false>(a, s);
      if (a.L == 192) return launch_bounded_L<T, 192, false>(a, s);
    }
  }
  if (wf_half(a)) {
    switch (a.L) {
      case 32: return launch_bounded_L<T, 32, true>(a, s);
      case 64: return launch_bounded_L<T, 64, true>(a, s);
      case 128: return launch_bounded_L<T, 128, true>(a, s);
      case 256: return launch_bounded_L<T, 256, true>(a, s);
      default: return hipErrorInvalidValue;
    }
  }
  switch (a.L) {
    case 64: return launch_bounded_L<T, 64, false>(a, s);
    case 128: return launch_bounded_L<T, 128, false>(a, s);
    case 256: return launch_bounded_L<T, 256, false>(a, s);
    case 512: return launch_bounded_L<T, 512, false>(a, s);
    default: return hipErrorInvalidValue;
  }
}

// out[0][i] += in[0][i] (+ in[1][i]), i < n_add: the second terms of the
// Dirichlet / Neumann divergence and curl.
template <typename T>
__global__ void __launch_bounds__(256) k_add(PassArgs a) {
  const long long total = a.n_add;
  T* dst = (T*)a.out[0];
  const T* x = (const T*)a.in[0];
  const T* y = (const T*)a.in[1];
  const long long step = (long long)gridDim.x * blockDim.x;
  for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += step) {
    T v = dst[e] + x[e];
    if (y) v += y[e];
    dst[e] = v;
  }
}

template <typename T>
hipError_t launch_add(const PassArgs& a, hipStream_t s) {
  const long long total = a.n_add;
  if (total <= 0) return hipSuccess;
  const long long blocks = (total + 255) / 256;
  const int grid = (int)(blocks < 8192 ? blocks : 8192);
  hipLaunchKernelGGL(k_add<T>, dim3(grid), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace

// One thread per output point; every term reads the three points around it
// along its axis (the faces' values or the one-sided stencils at the ends).
template <typename T>
__global__ void __launch_bounds__(256) k_fd_deriv(FdArgs a) {
  long long total = 1;
  for (int b = 0; b < a.nd; ++b) total *= a.N[b];
  T* out = (T*)a.out;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x) {
    int c[3] = {0, 0, 0};
    long long r = e;
    for (int b = a.nd - 1; b >= 0; --b) {
      c[b] = (int)(r % a.N[b]);
      r /= a.N[b];
    }
    double acc = 0.0;
    for (int k = 0; k < a.nterm; ++k) {
      const FdTerm& t = a.t[k];
      const int ax = t.axis, n = a.N[ax], j = c[ax];
      long long s = 1;
      for (int b = ax + 1; b < a.nd; ++b) s *= a.N[b];
      const T* p = (const T*)t.psi;
      auto v = [&](int i) -> double { return (double)p[e + (long long)(i - j) * s]; };
      // face values at this point's position on the other axes
      long long fo = 0;
      for (int b = 0; b < a.nd; ++b)
        if (b != ax) fo = fo * a.N[b] + c[b];
      const double glo = (t.g_lo && j == 0) ? (double)((const T*)t.g_lo)[fo] : 0.0;
      const double ghi = (t.g_hi && j == n - 1) ? (double)((const T*)t.g_hi)[fo] : 0.0;
      const double h = a.h[ax];
      const int bc = a.bc[ax];
      double d;
      if (bc == FD_PERIODIC) {  // the grid wraps
        d = (v(j + 1 < n ? j + 1 : 0) - v(j > 0 ? j - 1 : n - 1)) / (2.0 * h);
      } else if (bc == FD_DIRICHLET && a.regular) {  // boundary nodes hold g; n >= 3
        if (j == 0) d = (-3.0 * v(0) + 4.0 * v(1) - v(2)) / (2.0 * h);
        else if (j == n - 1) d = (3.0 * v(n - 1) - 4.0 * v(n - 2) + v(n - 3)) / (2.0 * h);
        else d = (v(j + 1) - v(j - 1)) / (2.0 * h);
      } else if (bc == FD_DIRICHLET) {  // quadratic through the face value and two centres
        if (n == 1) d = (ghi - glo) / h;  // (both faces at this one point)
        else if (j == 0) d = (v(1) / 3.0 + v(0) - 4.0 * glo / 3.0) / h;
        else if (j == n - 1) d = (4.0 * ghi / 3.0 - v(n - 1) - v(n - 2) / 3.0) / h;
        else d = (v(j + 1) - v(j - 1)) / (2.0 * h);
      } else {  // Neumann ghosts: centred difference = g (REGULAR), face difference = g
        const double left = j > 0 ? v(j - 1) : (a.regular ? v(1) - 2.0 * h * glo : v(0) - h * glo);
        const double right =
            j < n - 1 ? v(j + 1) : (a.regular ? v(n - 2) + 2.0 * h * ghi : v(n - 1) + h * ghi);
        d = (right - left) / (2.0 * h);
      }
      acc += t.sign * d;
    }
    out[e] = (T)acc;
  }
}

hipError_t launch_fd_deriv(const FdArgs& a, int prec, hipStream_t s) {
  if (prec == 0) hipLaunchKernelGGL(k_fd_deriv<float>, dim3(1024), dim3(256), 0, s, a);
  else hipLaunchKernelGGL(k_fd_deriv<double>, dim3(1024), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_bounded(const PassArgs& a, int prec, hipStream_t s) {
  if (a.fast == FAST_ADD) return prec == 0 ? launch_add<float>(a, s) : launch_add<double>(a, s);
  if (a.fast == FAST_SMALL2D) return launch_small2d(a, prec, s);
  if (prec == 0) return launch_bounded_T<float>(a, s);
  return launch_bounded_T<double>(a, s);
}

}  // namespace hp
