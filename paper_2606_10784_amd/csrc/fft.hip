// Zero-padded 2D FFT convolution of eq. (8) / eq. (10) for gfx950.
//
// The grid product G_grid u is evaluated as
//     [F^-1( F(c) . F(b) )]_restr,   b = u zero-padded from m x m to n x n,
// with n the smallest power of two >= 2m and the spectrum F(c) of the
// circulant kernel resident in HBM as an even-symmetric quarter (Sec.
// III-A/B).  Three passes:
//   rows_fwd : scatter the active grid values of one grid row into LDS,
//              length-n FFT along x, write the row (only rows [y0, y0+nr)
//              that hold active points, compacted);
//   cols_conv: for a block of CW columns: length-n FFT along y (rows >= nr are
//              zero), multiply by the spectrum, inverse FFT, keep nr rows;
//   rows_inv : inverse FFT along x, gather the active points of the row.
// The circulant product commutes with cyclic shifts, so compacting the rows to
// [0, nr) changes nothing.  The 1/n^2 of the inverse DFT is folded into the
// stored spectrum.
//
// Each FFT is an in-LDS Stockham autosort with radix-16 passes (radix 8, 4
// or 2 for the remainder); each thread holds its butterflies in registers
// across a barrier, so a single LDS buffer suffices.  In the column pass the
// first forward pass reads the tile from HBM straight into registers (its
// upper half is the zero padding), the last forward pass, the spectrum
// multiply and the first inverse pass share one register round (the inverse
// runs its radices in reverse order so the butterflies line up), and the last
// inverse pass stores only the kept rows straight to HBM.
#include <hip/hip_ext.h>

#include <type_traits>

#include "aim_internal.h"

namespace aim {

// ---------------------------------------------------------------------------
// small DFTs in registers (forward: e^{-2 pi i/R}, INV: conjugate)
// ---------------------------------------------------------------------------
template <typename V, bool INV>
__device__ __forceinline__ V rot_mi(V a) {      // multiply by -i (forward) or +i (inverse)
  V r;
  if (INV) { r.x = -a.y; r.y = a.x; }
  else { r.x = a.y; r.y = -a.x; }
  return r;
}

template <typename V, bool INV>
__device__ __forceinline__ void dft2(V& a, V& b) {
  V t = a;
  a = cadd(t, b);
  b = csub(t, b);
}

template <typename V, bool INV>
__device__ __forceinline__ void dft4(V& a, V& b, V& c, V& d) {
  V t0 = cadd(a, c), t1 = csub(a, c), t2 = cadd(b, d), t3 = rot_mi<V, INV>(csub(b, d));
  a = cadd(t0, t2);
  c = csub(t0, t2);
  b = cadd(t1, t3);
  d = csub(t1, t3);
}

template <typename T, bool INV>
__device__ __forceinline__ void dft8(cplx<T>* v) {
  using V = cplx<T>;
  const T c = (T)0.70710678118654752440084436210484903928;
  // even / odd halves
  V e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6];
  V o0 = v[1], o1 = v[3], o2 = v[5], o3 = v[7];
  dft4<V, INV>(e0, e1, e2, e3);
  dft4<V, INV>(o0, o1, o2, o3);
  // twiddles w8^k on the odd half
  V w1, w3;
  if (!INV) {
    w1.x = c * (o1.x + o1.y); w1.y = c * (o1.y - o1.x);
    w3.x = c * (o3.y - o3.x); w3.y = -c * (o3.x + o3.y);
  } else {
    w1.x = c * (o1.x - o1.y); w1.y = c * (o1.x + o1.y);
    w3.x = -c * (o3.x + o3.y); w3.y = c * (o3.x - o3.y);
  }
  V w2 = rot_mi<V, INV>(o2);
  v[0] = cadd(e0, o0); v[4] = csub(e0, o0);
  v[1] = cadd(e1, w1); v[5] = csub(e1, w1);
  v[2] = cadd(e2, w2); v[6] = csub(e2, w2);
  v[3] = cadd(e3, w3); v[7] = csub(e3, w3);
}

// 16-point DFT as 4 x 4: n = 4 n1 + n2, k = k1 + 4 k2
template <typename T, bool INV>
__device__ __forceinline__ void dft16(cplx<T>* v) {
  using V = cplx<T>;
  // W16^e, e = 0..9 (forward sign)
  const T c1 = (T)0.92387953251128675612818318939678829, s1 = (T)0.38268343236508977172845998403039887;
  const T c2 = (T)0.70710678118654752440084436210484903;
  dft4<V, INV>(v[0], v[4], v[8], v[12]);
  dft4<V, INV>(v[1], v[5], v[9], v[13]);
  dft4<V, INV>(v[2], v[6], v[10], v[14]);
  dft4<V, INV>(v[3], v[7], v[11], v[15]);
  // after the first stage v[4 k1 + n2] holds A[n2][k1]; twiddle by W16^{n2 k1}
  auto tw = [&](V a, T c, T sn) -> V {   // a * (c - i sn) forward, a * (c + i sn) inverse
    V r;
    if (!INV) { r.x = a.x * c + a.y * sn; r.y = a.y * c - a.x * sn; }
    else { r.x = a.x * c - a.y * sn; r.y = a.y * c + a.x * sn; }
    return r;
  };
  // n2 = 1: k1 = 1,2,3 -> e = 1,2,3
  v[5] = tw(v[5], c1, s1);
  v[9] = tw(v[9], c2, c2);
  v[13] = tw(v[13], s1, c1);
  // n2 = 2: e = 2,4,6
  v[6] = tw(v[6], c2, c2);
  v[10] = rot_mi<V, INV>(v[10]);
  v[14] = tw(v[14], -c2, c2);
  // n2 = 3: e = 3,6,9
  v[7] = tw(v[7], s1, c1);
  v[11] = tw(v[11], -c2, c2);
  v[15] = tw(v[15], -c1, -s1);
  // second stage over n2 for each k1; output X[k1 + 4 k2]
  dft4<V, INV>(v[0], v[1], v[2], v[3]);
  dft4<V, INV>(v[4], v[5], v[6], v[7]);
  dft4<V, INV>(v[8], v[9], v[10], v[11]);
  dft4<V, INV>(v[12], v[13], v[14], v[15]);
  // v[4 k1 + k2] holds X[k1 + 4 k2]: transpose the 4 x 4 block
  V t;
  t = v[1]; v[1] = v[4]; v[4] = t;
  t = v[2]; v[2] = v[8]; v[8] = t;
  t = v[3]; v[3] = v[12]; v[12] = t;
  t = v[6]; v[6] = v[9]; v[9] = t;
  t = v[7]; v[7] = v[13]; v[13] = t;
  t = v[11]; v[11] = v[14]; v[14] = t;
}

// 16-point DFT whose inputs 8..15 are zero: even and odd outputs are two
// 8-point DFTs of v and of v[r] W16^r.
template <typename T, bool INV>
__device__ __forceinline__ void dft16_halfin(cplx<T>* v) {
  using V = cplx<T>;
  const T c1 = (T)0.92387953251128675612818318939678829, s1 = (T)0.38268343236508977172845998403039887;
  const T c2 = (T)0.70710678118654752440084436210484903;
  auto tw = [&](V a, T c, T sn) -> V {   // a * (c - i sn) forward, a * (c + i sn) inverse
    V r;
    if (!INV) { r.x = a.x * c + a.y * sn; r.y = a.y * c - a.x * sn; }
    else { r.x = a.x * c - a.y * sn; r.y = a.y * c + a.x * sn; }
    return r;
  };
  V a[8], o[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) a[r] = v[r];
  o[0] = v[0];
  o[1] = tw(v[1], c1, s1);
  o[2] = tw(v[2], c2, c2);
  o[3] = tw(v[3], s1, c1);
  o[4] = rot_mi<V, INV>(v[4]);
  o[5] = tw(v[5], -s1, c1);
  o[6] = tw(v[6], -c2, c2);
  o[7] = tw(v[7], -c1, s1);
  dft8<T, INV>(a);
  dft8<T, INV>(o);
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    v[2 * k] = a[k];
    v[2 * k + 1] = o[k];
  }
}

// outputs 0..7 of a 16-point DFT: X[k] = E[k] + W16^k O[k] with E, O the
// 8-point DFTs of the even and odd inputs; result in v[0..7].
template <typename T, bool INV>
__device__ __forceinline__ void dft16_halfout(cplx<T>* v) {
  using V = cplx<T>;
  const T c1 = (T)0.92387953251128675612818318939678829, s1 = (T)0.38268343236508977172845998403039887;
  const T c2 = (T)0.70710678118654752440084436210484903;
  auto tw = [&](V a, T c, T sn) -> V {
    V r;
    if (!INV) { r.x = a.x * c + a.y * sn; r.y = a.y * c - a.x * sn; }
    else { r.x = a.x * c - a.y * sn; r.y = a.y * c + a.x * sn; }
    return r;
  };
  V e[8], o[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    e[r] = v[2 * r];
    o[r] = v[2 * r + 1];
  }
  dft8<T, INV>(e);
  dft8<T, INV>(o);
  v[0] = cadd(e[0], o[0]);
  v[1] = cadd(e[1], tw(o[1], c1, s1));
  v[2] = cadd(e[2], tw(o[2], c2, c2));
  v[3] = cadd(e[3], tw(o[3], s1, c1));
  v[4] = cadd(e[4], rot_mi<V, INV>(o[4]));
  v[5] = cadd(e[5], tw(o[5], -s1, c1));
  v[6] = cadd(e[6], tw(o[6], -c2, c2));
  v[7] = cadd(e[7], tw(o[7], -c1, s1));
}

template <typename T, int R, bool INV>
__device__ __forceinline__ void dft_r(cplx<T>* v) {
  if constexpr (R == 16) dft16<T, INV>(v);
  else if constexpr (R == 8) dft8<T, INV>(v);
  else if constexpr (R == 4) dft4<cplx<T>, INV>(v[0], v[1], v[2], v[3]);
  else dft2<cplx<T>, INV>(v[0], v[1]);
}

// LDS index with one pad slot per 16 elements: the radix-16 first pass
// stores with a stride of 16 elements, which the pad turns into 17 so the
// lanes of a wave spread over all banks.
__device__ __forceinline__ int pidx(int i) { return i + (i >> 4); }
__host__ __device__ constexpr int padded(int n) { return n + (n >> 4); }
// The column pass pads one slot per 256 bytes in both precisions: per 16
// FP64 or per 32 FP32 complex values.  In its fused pass consecutive lanes
// step 8 CW values apart (256 B), so the pad shifts each lane by one value
// (4 banks in FP64, 2 in FP32) and a cycle's lanes (16 of 16 B, 32 of 8 B)
// cover distinct banks.  The buffer is sized with padded(), which covers both.
template <typename T>
__device__ __forceinline__ int cidx(int i) { return i + (i >> (sizeof(T) == 4 ? 5 : 4)); }

// w^r for r = 1..R-1 from w = w^1 by a product tree of depth <= 4
template <typename V, int R>
__device__ __forceinline__ void tw_powers(V w1, V* wp) {
  wp[1] = w1;
  if constexpr (R > 2) {
    wp[2] = cmul(w1, w1);
    wp[3] = cmul(wp[2], w1);
  }
  if constexpr (R > 4) {
    wp[4] = cmul(wp[2], wp[2]);
    wp[5] = cmul(wp[4], w1);
    wp[6] = cmul(wp[4], wp[2]);
    wp[7] = cmul(wp[4], wp[3]);
  }
  if constexpr (R > 8) {
    wp[8] = cmul(wp[4], wp[4]);
#pragma unroll
    for (int r = 9; r < 16; ++r) wp[r] = cmul(wp[8], wp[r - 8]);
  }
}

// Twiddles of butterfly j of a Stockham pass (sub-transform length NS):
// input r is multiplied by w^(k r), w = e^{-2 pi i/(NS R)}, k = j mod NS.
template <typename T, int N, bool INV, int NS, int R>
__device__ __forceinline__ void pass_twiddle(cplx<T>* v, int j, const cplx<T>* __restrict__ tw) {
  using V = cplx<T>;
  if constexpr (NS > 1) {
    const int k = j & (NS - 1);
    V w1 = tw[k * (N / (NS * R))];
    if (INV) w1.y = -w1.y;
    V wp[R];
    tw_powers<V, R>(w1, wp);
#pragma unroll
    for (int r = 1; r < R; ++r) v[r] = cmul(v[r], wp[r]);
  }
}

// Base twiddle w^1 of butterfly j of a pass with sub-length NS (forward
// sign), loaded once so a later pass can reuse it without a dependent load.
template <typename T, int N, int NS, int R>
__device__ __forceinline__ cplx<T> tw_base(int j, const cplx<T>* __restrict__ tw) {
  if constexpr (NS > 1) return tw[(j & (NS - 1)) * (N / (NS * R))];
  else return mk<T>(1, 0);
}

// pass_twiddle with the base twiddle already in a register
template <typename T, bool INV, int NS, int R>
__device__ __forceinline__ void apply_twiddle(cplx<T>* v, cplx<T> w1) {
  using V = cplx<T>;
  if constexpr (NS > 1) {
    if (INV) w1.y = -w1.y;
    V wp[R];
    tw_powers<V, R>(w1, wp);
#pragma unroll
    for (int r = 1; r < R; ++r) v[r] = cmul(v[r], wp[r]);
  }
}

// One Stockham pass: sub-transform length NS -> NS*R.  Element i of column c
// lives at buf[pidx(i * NCOL + c)]; butterfly b = j * NCOL + c reads elements
// j + r N/R and writes (j - k) R + k + r NS, k = j mod NS.
template <typename T, int N, int NCOL, int NT, bool INV, int NS, int R>
__device__ __forceinline__ void stockham_pass(cplx<T>* buf, const cplx<T>* __restrict__ tw) {
  using V = cplx<T>;
  constexpr int NB = (N / R) * NCOL;
  constexpr int PER = (NB + NT - 1) / NT;
  V v[PER][R];
  const int tid = threadIdx.x;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int b = tid + q * NT;
    if ((NB % NT) == 0 || b < NB) {
      const int c = b % NCOL, j = b / NCOL;
#pragma unroll
      for (int r = 0; r < R; ++r) v[q][r] = buf[pidx((j + r * (N / R)) * NCOL + c)];
      pass_twiddle<T, N, INV, NS, R>(v[q], j, tw);
      dft_r<T, R, INV>(v[q]);
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int b = tid + q * NT;
    if ((NB % NT) == 0 || b < NB) {
      const int c = b % NCOL, j = b / NCOL;
      const int k = j & (NS - 1);
      const int base = (j / NS) * NS * R + k;
#pragma unroll
      for (int r = 0; r < R; ++r) buf[pidx((base + r * NS) * NCOL + c)] = v[q][r];
    }
  }
  __syncthreads();
}

// Stockham pass with the base twiddle of each butterfly given (w[q] for
// butterfly tid + q NT, forward sign); single column
template <typename T, int N, int NT, bool INV, int NS, int R>
__device__ __forceinline__ void stockham_pass_w(cplx<T>* buf, const cplx<T>* w) {
  using V = cplx<T>;
  constexpr int NB = N / R;
  constexpr int PER = (NB + NT - 1) / NT;
  V v[PER][R];
  const int tid = threadIdx.x;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int j = tid + q * NT;
    if ((NB % NT) == 0 || j < NB) {
#pragma unroll
      for (int r = 0; r < R; ++r) v[q][r] = buf[pidx(j + r * (N / R))];
      apply_twiddle<T, INV, NS, R>(v[q], w[q]);
      dft_r<T, R, INV>(v[q]);
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int j = tid + q * NT;
    if ((NB % NT) == 0 || j < NB) {
      const int k = j & (NS - 1);
      const int base = (j / NS) * NS * R + k;
#pragma unroll
      for (int r = 0; r < R; ++r) buf[pidx(base + r * NS)] = v[q][r];
    }
  }
  __syncthreads();
}

// A chain of single-column Stockham passes from sub-length NS up to NSEND,
// radix 16 (R16) or radix min(16, N/NS); the base twiddles of every pass are
// loaded up front (chain_tw) so no pass waits on a dependent load.
template <int N, int NS, bool R16> constexpr int chain_radix() { return R16 ? 16 : (N / NS >= 16 ? 16 : N / NS); }
template <int N, int NT, int NS, int NSEND, bool R16> constexpr int chain_len() {
  if constexpr (NS >= NSEND) return 0;
  else {
    constexpr int R = chain_radix<N, NS, R16>();
    return (N / R + NT - 1) / NT + chain_len<N, NT, NS * R, NSEND, R16>();
  }
}
template <typename T, int N, int NT, int NS, int NSEND, bool R16>
__device__ __forceinline__ void chain_tw(const cplx<T>* __restrict__ tw, cplx<T>* w) {
  if constexpr (NS < NSEND) {
    constexpr int R = chain_radix<N, NS, R16>();
    constexpr int NB = N / R, PER = (NB + NT - 1) / NT;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int j = threadIdx.x + q * NT;
      w[q] = ((NB % NT) == 0 || j < NB) ? tw_base<T, N, NS, R>(j, tw) : mk<T>(1, 0);
    }
    chain_tw<T, N, NT, NS * R, NSEND, R16>(tw, w + PER);
  }
}
template <typename T, int N, int NT, bool INV, int NS, int NSEND, bool R16>
__device__ __forceinline__ void chain_passes(cplx<T>* buf, const cplx<T>* w) {
  if constexpr (NS < NSEND) {
    constexpr int R = chain_radix<N, NS, R16>();
    stockham_pass_w<T, N, NT, INV, NS, R>(buf, w);
    chain_passes<T, N, NT, INV, NS * R, NSEND, R16>(buf, w + (N / R + NT - 1) / NT);
  }
}

// radix-16 passes, then 8, 4 or 2 for the remainder
template <typename T, int N, int NCOL, int NT, bool INV, int NS>
__device__ __forceinline__ void fft_passes(cplx<T>* buf, const cplx<T>* __restrict__ tw) {
  if constexpr (NS < N) {
    constexpr int R = (N / NS >= 16) ? 16 : (N / NS);
    stockham_pass<T, N, NCOL, NT, INV, NS, R>(buf, tw);
    fft_passes<T, N, NCOL, NT, INV, NS * R>(buf, tw);
  }
}

// radix-16 passes with sub-transform lengths NS, 16 NS, ... below NSEND
template <typename T, int N, int NCOL, int NT, bool INV, int NS, int NSEND>
__device__ __forceinline__ void passes16(cplx<T>* buf, const cplx<T>* __restrict__ tw) {
  if constexpr (NS < NSEND) {
    stockham_pass<T, N, NCOL, NT, INV, NS, 16>(buf, tw);
    passes16<T, N, NCOL, NT, INV, NS * 16, NSEND>(buf, tw);
  }
}

// One in-place Cooley-Tukey pass with stride S and radix R: butterfly
// (block, m) owns positions blk S R + m + S r.  Forward (decimation in
// frequency): R-point DFT, then output k times W_{SR}^{m k}.  Inverse
// (decimation in time, the exact reverse): input k times W_{SR}^{-m k}, then
// the inverse R-point DFT.  Each thread writes back the positions it read, so
// one barrier per pass suffices.
template <typename T, int N, int NCOL, int NT, bool INV, int S, int R>
__device__ __forceinline__ void ct_pass(cplx<T>* buf, const cplx<T>* __restrict__ tw) {
  using V = cplx<T>;
  constexpr int NB = (N / R) * NCOL;
  constexpr int PER = (NB + NT - 1) / NT;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int b = threadIdx.x + q * NT;
    if ((NB % NT) == 0 || b < NB) {
      const int c = b % NCOL, t = b / NCOL;
      const int m = t % S, base = (t / S) * S * R + m;
      V v[R];
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = buf[pidx((base + S * r) * NCOL + c)];
      if (!INV) {
        dft_r<T, R, false>(v);
        pass_twiddle<T, N, false, S, R>(v, m, tw);
      } else {
        pass_twiddle<T, N, true, S, R>(v, m, tw);
        dft_r<T, R, true>(v);
      }
#pragma unroll
      for (int r = 0; r < R; ++r) buf[pidx((base + S * r) * NCOL + c)] = v[r];
    }
  }
  __syncthreads();
}

// ct_pass with the base twiddle of each of the thread's butterflies given
// (w[q] for butterfly tid + q NT, forward sign)
template <typename T, int N, int NCOL, int NT, bool INV, int S, int R>
__device__ __forceinline__ void ct_pass_w(cplx<T>* buf, const cplx<T>* w) {
  using V = cplx<T>;
  constexpr int NB = (N / R) * NCOL;
  constexpr int PER = (NB + NT - 1) / NT;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int b = threadIdx.x + q * NT;
    if ((NB % NT) == 0 || b < NB) {
      const int c = b % NCOL, t = b / NCOL;
      const int m = t % S, base = (t / S) * S * R + m;
      V v[R];
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = buf[cidx<T>((base + S * r) * NCOL + c)];
      if (!INV) {
        dft_r<T, R, false>(v);
        apply_twiddle<T, false, S, R>(v, w[q]);
      } else {
        apply_twiddle<T, true, S, R>(v, w[q]);
        dft_r<T, R, true>(v);
      }
#pragma unroll
      for (int r = 0; r < R; ++r) buf[cidx<T>((base + S * r) * NCOL + c)] = v[r];
    }
  }
  __syncthreads();
}

// radix-16 forward passes with strides S, S/16, ... down to SEND (inclusive)
template <typename T, int N, int NCOL, int NT, int S, int SEND>
__device__ __forceinline__ void dif16_down(cplx<T>* buf, const cplx<T>* __restrict__ tw) {
  if constexpr (S >= SEND && S >= 1) {
    ct_pass<T, N, NCOL, NT, false, S, 16>(buf, tw);
    dif16_down<T, N, NCOL, NT, S / 16, SEND>(buf, tw);
  }
}

// radix-16 inverse passes with strides S, 16 S, ... up to SEND (inclusive)
template <typename T, int N, int NCOL, int NT, int S, int SEND>
__device__ __forceinline__ void dit16_up(cplx<T>* buf, const cplx<T>* __restrict__ tw) {
  if constexpr (S <= SEND && S >= 1) {
    ct_pass<T, N, NCOL, NT, true, S, 16>(buf, tw);
    dit16_up<T, N, NCOL, NT, S * 16, SEND>(buf, tw);
  }
}

// radix of the remainder pass: N = 16^p * last_radix(N), last_radix in 2..16
template <int N> constexpr int last_radix() {
  if constexpr (N <= 16) return N;
  else return last_radix<N / 16>();
}

// ---------------------------------------------------------------------------
// tiles: CB columns per tile; columns kx and N - kx share a tile (and a
// column-pass block) so the even-symmetric quarter spectrum is fetched once.
// Tile b, slot c holds pair q = b*(CB/2) + c/2 + 1 (c odd: the mirror N - q);
// the last slot pair of the last tile holds the self-mirrored columns 0 and
// N/2.
// ---------------------------------------------------------------------------
// CB is the tile width (columns per tile, the row passes' piece); CW the
// columns one column-pass block transforms: as many as fit the LDS budget
// of two blocks per CU.  Tiles are at least 64 bytes wide, so the row
// passes read and write whole 64-byte pieces; where CW is narrower (N >=
// 2048 in either precision) the CB / CW blocks of a tile take CW columns
// each.
template <typename T, int N> struct ColCfg {
  static constexpr int BYTES = 80000;   // padded LDS per column block: two blocks per CU
  static constexpr int CB0 = BYTES / (padded(N) * (int)sizeof(cplx<T>));
  static constexpr int CW1 = CB0 < 2 ? 1 : (CB0 > 16 ? 16 : CB0);
  static constexpr int CW = (CW1 >= 16) ? 16 : (CW1 >= 8 ? 8 : (CW1 >= 4 ? 4 : (CW1 >= 2 ? 2 : 1)));
  // tiles at least 64 bytes wide, so the row passes move whole 64-byte pieces
  static constexpr int CB64 = 64 / (int)sizeof(cplx<T>);
  static constexpr int CB = CW > CB64 ? CW : CB64;
  static constexpr int NT = (N * CW / 16 >= 512) ? 512 : 256;
};

// Column-pass block b -> tile tb and first column c0 within the tile.  The
// K = CB / CW blocks of a tile are 8 apart, which the launch deals to the
// same XCD, so the parts of each tile line meet in one L2.
template <typename T, int N>
__device__ __forceinline__ void col_block_of(int b, int& tb, int& c0) {
  constexpr int CB = ColCfg<T, N>::CB, CW = ColCfg<T, N>::CW, K = CB / CW;   // blocks per tile
  if constexpr (K == 1) {
    tb = b;
    c0 = 0;
  } else {
    static_assert(K * CW == CB && (K & (K - 1)) == 0 && (N / CB) % 8 == 0, "tile split into 2^k blocks");
    tb = (b / (8 * K)) * 8 + (b & 7);
    c0 = ((b >> 3) & (K - 1)) * CW;
  }
}

// For N = 1024 a column-pass block takes a quad of columns p, N - p,
// N/2 - p, N/2 + p (two pairs, p = 1 .. N/4 - 1; the last quad has the pairs
// N/4 and (0, N/2)), which share their row-transform sums (sparse_rows).
// Neighbouring p complete each other's tile lines, so each XCD (blocks are
// dealt round-robin over 8) takes a run of p.
template <int N> __device__ __forceinline__ int quad_of_block(int bid) {
  static_assert(N / 4 % 8 == 0, "whole runs per XCD");
  return (bid & 7) * (N / 32) + (bid >> 3) + 1;
}
// pair and slot offset (tile, first slot) of columns c = 0..3 of quad p
template <int N> __device__ __forceinline__ int quad_pair(int p, int c) {
  return c < 2 ? p : (p == N / 4 ? N / 2 : N / 2 - p);
}

__device__ __forceinline__ void col_of(int b, int c, int N, int CB, int& kx, int& kxq) {
  const int q = b * (CB / 2) + (c >> 1) + 1;
  const int half = c & 1;
  if (q >= N / 2) {            // last pair slot of the last tile
    kx = half ? N / 2 : 0;
    kxq = kx;
  } else {
    kx = half ? N - q : q;
    kxq = q;
  }
}

// XCD-aware row order: consecutive rows go to the same XCD (blocks are
// dealt round-robin over 8 XCDs), so the pieces of a tile line written by
// neighbouring rows meet in one L2.
__device__ __forceinline__ int xcd_row(int bid, int nrows) {
  const int per = (nrows + 7) / 8;
  return (bid & 7) * per + (bid >> 3);
}

// ---------------------------------------------------------------------------
// kernels.  T layout (tiled): [pair][tile][row][CB] with ldt >= nr rows
// per tile (tile_rows); rows nr .. ldt-1 are never read or written
// ---------------------------------------------------------------------------
template <int N> constexpr int row_threads() { return N / 16 < 64 ? 64 : (N / 16 > 256 ? 256 : N / 16); }

// Pass 1: gather active values of a row into a zeroed LDS row, FFT along x.
// Active points have x < N/2, so only that half is cleared and the first pass
// reads inputs 0..7 of its radix-16 butterflies.
template <typename T, int N>
__global__ __launch_bounds__(row_threads<N>()) void k_rows_fwd(
    const cplx<T>* __restrict__ U, int n_act, const int32_t* __restrict__ row_ptr,
    const int32_t* __restrict__ act_ix, int nr, int ldt, cplx<T>* __restrict__ Tb,
    const cplx<T>* __restrict__ tw) {
  using V = cplx<T>;
  static_assert(N >= 32, "row pass assumes at least two forward passes");
  constexpr int NT = row_threads<N>();
  constexpr int CB = ColCfg<T, N>::CB;
  constexpr int NBLK = N / CB;
  __shared__ V buf[padded(N)];
  const int row = xcd_row(blockIdx.x, nr), pair = blockIdx.y;
  const int tid = threadIdx.x;
  if (row >= nr) return;
  constexpr int NW = chain_len<N, NT, 16, N, false>();
  V wt[NW > 0 ? NW : 1];
  chain_tw<T, N, NT, 16, N, false>(tw, wt);
  for (int i = tid; i < N / 2; i += NT) buf[pidx(i)] = mk<T>(0, 0);
  __syncthreads();
  const int a0 = row_ptr[row], a1 = row_ptr[row + 1];
  const V* Up = U + (size_t)pair * n_act;
  for (int a = a0 + tid; a < a1; a += NT) buf[pidx(act_ix[a])] = Up[a];
  __syncthreads();
  {
    constexpr int NB = N / 16, PER = (NB + NT - 1) / NT;
    V v[PER][16];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int j = tid + q * NT;
      if ((NB % NT) == 0 || j < NB) {
#pragma unroll
        for (int r = 0; r < 8; ++r) v[q][r] = buf[pidx(j + r * (N / 16))];
        dft16_halfin<T, false>(v[q]);
      }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int j = tid + q * NT;
      if ((NB % NT) == 0 || j < NB) {
#pragma unroll
        for (int r = 0; r < 16; ++r) buf[pidx(j * 16 + r)] = v[q][r];
      }
    }
    __syncthreads();
  }
  chain_passes<T, N, NT, false, 16, N, false>(buf, wt);
  // groups of CB lanes fill the CB-wide segments of the tiled layout; the LDS
  // reads of a thread are all issued before its stores
  V* out = Tb + (size_t)pair * NBLK * ldt * CB + (size_t)row * CB;
  constexpr int PER = (N + NT - 1) / NT;
  V v[PER];
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int idx = tid + q * NT;
    if ((N % NT) == 0 || idx < N) {
      int kx, kxq;
      col_of(idx / CB, idx % CB, N, CB, kx, kxq);
      v[q] = buf[pidx(kx)];
    }
  }
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int idx = tid + q * NT;
    if ((N % NT) == 0 || idx < N) out[(size_t)(idx / CB) * ldt * CB + idx % CB] = v[q];
  }
}

// Pass 3: inverse FFT along x, gather the active points of the row.  The
// inverse runs its radices in reverse order so that the last pass is radix 16
// and computes only the outputs x < N/2, where the active points lie.
template <typename T, int N>
__global__ __launch_bounds__(row_threads<N>()) void k_rows_inv(
    const cplx<T>* __restrict__ Tb, int nr, int ldt, const int32_t* __restrict__ row_ptr,
    const int32_t* __restrict__ act_ix, cplx<T>* __restrict__ Vout, int n_act,
    const cplx<T>* __restrict__ tw) {
  using V = cplx<T>;
  static_assert(N >= 32, "row pass assumes at least two inverse passes");
  constexpr int NT = row_threads<N>();
  constexpr int CB = ColCfg<T, N>::CB;
  constexpr int NBLK = N / CB;
  constexpr int RL = last_radix<N>();
  __shared__ V buf[padded(N)];
  const int row = xcd_row(blockIdx.x, nr), pair = blockIdx.y;
  const int tid = threadIdx.x;
  if (row >= nr) return;
  const V* in = Tb + (size_t)pair * NBLK * ldt * CB + (size_t)row * CB;
  // base twiddles of the radix-16 passes and of the last pass, loaded with
  // the row
  constexpr int NW = chain_len<N, NT, RL, N / 16, true>();
  constexpr int NS_L = N / 16, PER_L = (NS_L + NT - 1) / NT;
  V wt[NW > 0 ? NW : 1], wl[PER_L];
  chain_tw<T, N, NT, RL, N / 16, true>(tw, wt);
#pragma unroll
  for (int q = 0; q < PER_L; ++q) {
    const int j = tid + q * NT;
    wl[q] = ((NS_L % NT) == 0 || j < NS_L) ? tw_base<T, N, NS_L, 16>(j, tw) : mk<T>(1, 0);
  }
  {
    // all HBM loads of a thread in flight before its LDS stores
    constexpr int PER = (N + NT - 1) / NT;
    V v[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int idx = tid + q * NT;
      if ((N % NT) == 0 || idx < N) v[q] = in[(size_t)(idx / CB) * ldt * CB + idx % CB];
    }
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int idx = tid + q * NT;
      if ((N % NT) == 0 || idx < N) {
        int kx, kxq;
        col_of(idx / CB, idx % CB, N, CB, kx, kxq);
        buf[pidx(kx)] = v[q];
      }
    }
  }
  __syncthreads();
  stockham_pass<T, N, 1, NT, true, 1, RL>(buf, tw);
  chain_passes<T, N, NT, true, RL, N / 16, true>(buf, wt);
  {
    constexpr int NS = NS_L, NB = NS, PER = PER_L;
    V v[PER][16];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int j = tid + q * NT;
      if ((NB % NT) == 0 || j < NB) {
#pragma unroll
        for (int r = 0; r < 16; ++r) v[q][r] = buf[pidx(j + r * NS)];
        apply_twiddle<T, true, NS, 16>(v[q], wl[q]);
        dft16_halfout<T, true>(v[q]);
      }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int j = tid + q * NT;
      if ((NB % NT) == 0 || j < NB) {
#pragma unroll
        for (int r = 0; r < 8; ++r) buf[pidx(j + r * NS)] = v[q][r];
      }
    }
    __syncthreads();
  }
  const int a0 = row_ptr[row], a1 = row_ptr[row + 1];
  V* Vp = Vout + (size_t)pair * n_act;
  for (int a = a0 + tid; a < a1; a += NT) Vp[a] = buf[pidx(act_ix[a])];
}

// Set-up: in-place forward FFT of full rows of length N (row-major array).
template <typename T, int N>
__global__ __launch_bounds__(row_threads<N>()) void k_rows_fft_inplace(cplx<T>* __restrict__ A,
                                                                       const cplx<T>* __restrict__ tw) {
  constexpr int NT = row_threads<N>();
  __shared__ cplx<T> buf[padded(N)];
  cplx<T>* rowp = A + (size_t)blockIdx.x * N;
  for (int i = threadIdx.x; i < N; i += NT) buf[pidx(i)] = rowp[i];
  __syncthreads();
  fft_passes<T, N, 1, NT, false, 1>(buf, tw);
  for (int i = threadIdx.x; i < N; i += NT) rowp[i] = buf[pidx(i)];
}

// Pass 2 (MODE 0): column FFT, spectrum multiply, inverse column FFT, in
// place on CW columns of one tile [row][CB] of T (nr <= N/2 rows kept, the rest is the
// zero padding).  The column FFT is an in-place decimation in frequency, so
// position p holds frequency ky_of_pos(N, p); the spectrum Cq is stored in
// that order, folded over ky -> N - ky ([kxq][spec_row_len(N)]), and the
// inverse is the matching decimation in time.
// MODE 1 (set-up): plain forward FFT of CW consecutive columns of a
// row-major N x N array.
// The column pass of CW columns of one tile [row][CB] (nr kept rows, the rest of the
// column is the zero padding), in place: column FFT, spectrum multiply,
// inverse column FFT (the MODE 0 body of k_cols and of k_cols_group).
template <typename T, int N>
__device__ __forceinline__ void cols_conv_tile(cplx<T>* buf, cplx<T>* __restrict__ tile, int nr, int b, int c0_,
                                               const cplx<T>* __restrict__ Cq, const cplx<T>* __restrict__ tw) {
  using V = cplx<T>;
  constexpr int CB = ColCfg<T, N>::CB;   // tile width (global layout)
  constexpr int CW = ColCfg<T, N>::CW;   // columns of this block, c0 .. c0 + CW - 1 (LDS layout)
  const int c0 = CW == CB ? 0 : c0_;
  constexpr int NT = ColCfg<T, N>::NT;
  const int tid = threadIdx.x;
  static_assert(N >= 32, "column pass assumes at least two forward passes");
  constexpr int RL = last_radix<N>();
  constexpr int S1 = N / 16;
  constexpr int SM = N / 256;                   // middle radix-16 pass stride
  constexpr bool MID = SM >= RL && SM >= 1;
  static_assert(!MID || SM / 16 < RL, "at most one middle pass per direction");
  constexpr int NB1 = S1 * CW, PER1 = (NB1 + NT - 1) / NT;
  constexpr int NBM = (N / 16) * CW, PERM = (NBM + NT - 1) / NT;
  constexpr int NG = N / RL, NBF = NG * CW, PERF = (NBF + NT - 1) / NT;
  // forward pass 1 (stride N/16, radix 16) from HBM: inputs m + S1 r with
  // r >= 8 lie in the zero half
  V v[PER1][16];
#pragma unroll
  for (int q = 0; q < PER1; ++q) {
    const int bb = tid + q * NT;
    if ((NB1 % NT) == 0 || bb < NB1) {
      const int c = bb % CW, m = bb / CW;
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const int i = m + r * S1;
        v[q][r] = i < nr ? tile[(size_t)i * CB + c0 + c] : mk<T>(0, 0);
      }
    }
  }
  // everything else this block reads from HBM does not depend on the data:
  // the spectrum values of the fused pass and the twiddles of the other
  // passes are issued now and consumed passes later, so their latency
  // overlaps the first passes instead of stalling each one (the spectrum
  // only in FP64 up to N = 2048: elsewhere the extra registers would cost
  // a wave per SIMD or spill).
  // The spectrum row is folded (ky and N - ky share a slot): group g holds
  // ky = low + W r with low the base-16 digit reversal of g; a group with
  // low > W/2 reads its mirror group W - low and reverses r (in registers,
  // at the multiply, so a prefetch never waits).
  constexpr int W = N / RL, HS = (W / 2 + 1) * RL;
  auto mirrored = [&](int g, int& lowc) {
    int low = 0;
#pragma unroll
    for (int t = 1, gg = g; t < W; t *= 16, gg >>= 4) low = low * 16 + (gg & 15);
    lowc = low > W / 2 ? W - low : low;
    return low > W / 2;
  };
  auto load_spec_part = [&](int bb, V* cv, int r0, int r1) {
    const int g = bb % NG, c = bb / NG;
    int kx, kxq, lowc;
    col_of(b, c0 + c, N, CB, kx, kxq);
    mirrored(g, lowc);
    const V* Cp = Cq + (size_t)kxq * HS + lowc * RL;
#pragma unroll
    for (int r = 0; r < RL; ++r)
      if (r >= r0 && r < r1) cv[r] = Cp[r];
  };
  auto load_spec = [&](int bb, V* cv) { load_spec_part(bb, cv, 0, RL); };
  constexpr bool PRE = sizeof(T) == 8 && N <= 2048 && PERF * RL <= 16;
  // FP64 above N = 2048 (one block per CU): half of the spectrum loads go
  // out once the first pass has left its values in LDS, so their latency
  // overlaps the middle pass in registers the first pass has freed, and the
  // other half right after the middle pass (all of them at once would spill)
  constexpr bool LATE = sizeof(T) == 8 && !PRE && MID && PERF * RL <= 16;
  V cv[PERF][RL];
  if constexpr (PRE) {
#pragma unroll
    for (int q = 0; q < PERF; ++q) {
      const int bb = tid + q * NT;
      if ((NBF % NT) == 0 || bb < NBF) load_spec(bb, cv[q]);
    }
  }
  V w1[PER1], wm[PERM];
#pragma unroll
  for (int q = 0; q < PER1; ++q) {
    const int bb = tid + q * NT;
    w1[q] = ((NB1 % NT) == 0 || bb < NB1) ? tw_base<T, N, S1, 16>(bb / CW, tw) : mk<T>(1, 0);
  }
  if constexpr (MID) {
#pragma unroll
    for (int q = 0; q < PERM; ++q) {
      const int bb = tid + q * NT;
      wm[q] = ((NBM % NT) == 0 || bb < NBM) ? tw_base<T, N, SM, 16>((bb / CW) % SM, tw) : mk<T>(1, 0);
    }
  }
#pragma unroll
  for (int q = 0; q < PER1; ++q) {
    const int bb = tid + q * NT;
    if ((NB1 % NT) == 0 || bb < NB1) {
      const int c = bb % CW, m = bb / CW;
      dft16_halfin<T, false>(v[q]);
      apply_twiddle<T, false, S1, 16>(v[q], w1[q]);
#pragma unroll
      for (int r = 0; r < 16; ++r) buf[cidx<T>((m + r * S1) * CW + c)] = v[q][r];
    }
  }
  if constexpr (LATE) {
#pragma unroll
    for (int q = 0; q < PERF; ++q) {
      const int bb = tid + q * NT;
      if ((NBF % NT) == 0 || bb < NBF) load_spec_part(bb, cv[q], 0, RL / 2);
    }
  }
  __syncthreads();
  if constexpr (MID) ct_pass_w<T, N, CW, NT, false, SM, 16>(buf, wm);
  if constexpr (LATE) {
#pragma unroll
    for (int q = 0; q < PERF; ++q) {
      const int bb = tid + q * NT;
      if ((NBF % NT) == 0 || bb < NBF) load_spec_part(bb, cv[q], RL / 2, RL);
    }
  }
  // last forward pass (contiguous groups of RL), spectrum multiply in the
  // stored frequency order, first inverse pass; lanes run along the groups
#pragma unroll
  for (int q = 0; q < PERF; ++q) {
    const int bb = tid + q * NT;
    if ((NBF % NT) == 0 || bb < NBF) {
      const int g = bb % NG, c = bb / NG;
      if constexpr (!PRE && !LATE) load_spec(bb, cv[q]);
      V u[RL];
#pragma unroll
      for (int r = 0; r < RL; ++r) u[r] = buf[cidx<T>((g * RL + r) * CW + c)];
      int lowc;
      const bool mir = mirrored(g, lowc);
      dft_r<T, RL, false>(u);
#pragma unroll
      for (int r = 0; r < RL; ++r) u[r] = cmul(u[r], mir ? cv[q][RL - 1 - r] : cv[q][r]);
      dft_r<T, RL, true>(u);
#pragma unroll
      for (int r = 0; r < RL; ++r) buf[cidx<T>((g * RL + r) * CW + c)] = u[r];
    }
  }
  __syncthreads();
  if constexpr (MID) ct_pass_w<T, N, CW, NT, true, SM, 16>(buf, wm);
  // last inverse pass (stride N/16, radix 16) straight to HBM: outputs
  // m + S1 r, only r < 8 can be a kept row
#pragma unroll
  for (int q = 0; q < PER1; ++q) {
    const int bb = tid + q * NT;
    if ((NB1 % NT) == 0 || bb < NB1) {
      const int c = bb % CW, m = bb / CW;
      V u[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) u[r] = buf[cidx<T>((m + r * S1) * CW + c)];
      apply_twiddle<T, true, S1, 16>(u, w1[q]);
      dft16_halfout<T, true>(u);
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const int i = m + r * S1;
        if (i < nr) tile[(size_t)i * CB + c0 + c] = u[r];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Column pass for N = 1024: two waves per column, no block barrier inside
// the transforms.
//
// The frequencies ky = q + 2 k' of one residue q are a 512-point FFT of
// z_q[j] = W_N^{q j} x[j] (rows past N/2 are the zero padding), and the
// inverse adds the two residues.  Wave q of a column transforms residue q in
// place as 8 x 8 x 8 with 8 values per lane: digit a of j = 64 a + 8 b + c in
// the registers, lane = 8 b + c; two exchanges through a wave-private LDS
// buffer bring b, then c, into the registers.  ky order after the forward
// transform: lane = 8 k0 + k1, register k2, k' = k0 + 8 k1 + 64 k2, which is
// the order the spectrum is stored in.
//
// The inputs come from the active points themselves (sparse_rows), not from
// transformed rows: a row holds 10 to 20 active points, so its transform at
// one column is as many products, and the row pass with its write and read
// of the whole tile set falls away.  Measured on a 392-row star, three
// channels of two right-hand sides and one of two: 45.9 + 17.9 us against
// 34.3 + 16.3 us of column pass and 16.3 + 7.3 us of row pass with one launch
// each; the whole TE Calderon product 105.8 against 112.0 us.  Bound by FP64
// issue and by LDS writes (a KB takes 5.8 ns per CU, a read 1.8), which
// overlap only in part at 16 waves per CU; the row sums by the L2-to-CU rate.
// ---------------------------------------------------------------------------
// LDS traffic of one wave stays in program order
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  __builtin_amdgcn_sched_barrier(0);
}

// keeps the compiler from carrying values derived from a across this point
template <typename V> __device__ __forceinline__ void opaque(V& a) { asm volatile("" : "+v"(a.x), "+v"(a.y)); }

template <typename T, int N> struct WaveCols {
  static_assert(N == 1024, "two waves per column, one residue each");
  static constexpr int F = 512, Q = 2;
  static constexpr int CW = 4, NT = 2 * CW * 64;
  static constexpr int EX = 576;                      // 8 x 72: padded exchange buffer of a wave
  static constexpr int LDS = 2 * CW * EX + 64;        // exchange buffers and W_64 table; staging and E are smaller
  static_assert(CW * F + N / 2 <= LDS, "staging and look-up table fit");
};
// staging slot of (row, column c) within column c's F: rows permuted within
// runs of 16, so that lanes along rows and lanes along (row, c) both spread
// over the banks
__device__ __forceinline__ int st_row(int row, int c) { return row ^ (c << 2); }

// v[k] *= base g^k (conjugated when INV)
template <typename T, bool INV>
__device__ __forceinline__ void mul_powers(cplx<T>* v, cplx<T> base, cplx<T> g) {
  using V = cplx<T>;
  auto mul = [](V a, V w) { return INV ? cmulc(a, w) : cmul(a, w); };
  opaque(g);
  V t[4];
  t[0] = base;
  v[0] = mul(v[0], t[0]);
  t[1] = cmul(base, g);
  v[1] = mul(v[1], t[1]);
  V g2 = cmul(g, g);
  t[2] = cmul(base, g2);
  v[2] = mul(v[2], t[2]);
  t[3] = cmul(t[1], g2);
  v[3] = mul(v[3], t[3]);
  g2 = cmul(g2, g2);
#pragma unroll
  for (int k = 4; k < 8; ++k) v[k] = mul(v[k], cmul(t[k - 4], g2));
  __builtin_amdgcn_sched_barrier(0);
}

// Forward transform, spectrum multiply and inverse transform of residue q
// (uniform over the wave) in v.  Cr: the stored spectrum row; w64[8 k + lo]:
// W_64^{k lo} in LDS.
template <typename T, int N>
__device__ __forceinline__ void wave_conv(cplx<T>* v, cplx<T>* ex, int lane, int q, cplx<T> g, const cplx<T>* w64,
                                          const cplx<T>* __restrict__ Cr, const cplx<T>* __restrict__ tw) {
  using V = cplx<T>;
  const int hi = lane >> 3, lo = lane & 7;
  V* e0 = ex + lane;                   // register digit outermost
  V* e1 = ex + hi * 72 + lo;           // + 8 d: digit b; + 9 d: digit k1
  V* e2 = ex + hi * 72 + lo * 9;       // + d: digit c
  const V base = tw[lane * q];
#pragma unroll
  for (int t = 1; t < 8; ++t) v[t] = cmul(v[t], tw[q * t * 64]);   // uniform
  dft8<T, false>(v);
  mul_powers<T, false>(v, base, g);
#pragma unroll
  for (int d = 0; d < 8; ++d) e0[d * 72] = v[d];
  wave_sync();
#pragma unroll
  for (int d = 0; d < 8; ++d) v[d] = e1[8 * d];
  wave_sync();
  dft8<T, false>(v);
#pragma unroll
  for (int k = 1; k < 8; ++k) v[k] = cmul(v[k], w64[8 * k + lo]);
#pragma unroll
  for (int d = 0; d < 8; ++d) e1[9 * d] = v[d];
  wave_sync();
  // stored spectrum slots (ky_of_slot): registers 0..3 of every lane, and for
  // residue 0 slot 256 (lane 0, register 4).  The rest is even: -ky of (lane,
  // r) is (63 - lane, 7 - r) for residue 1; for residue 0 lane digits
  // (8 - k0, 7 - k1) or (0, 8 - k1) and for lane 0 register 8 - r.
  V cv[8];
  {
    const int mir = q ? 63 - lane : (hi ? (8 - hi) * 8 + (7 - lo) : (lo ? 8 - lo : 64));
#pragma unroll
    for (int r = 0; r < 8; ++r) cv[r] = (Cr + q * 264 + (r < 4 ? r : 7 - r) * 64)[r < 4 ? lane : mir];
  }
#pragma unroll
  for (int d = 0; d < 8; ++d) v[d] = e2[d];
  wave_sync();
  dft8<T, false>(v);
#pragma unroll
  for (int r = 0; r < 8; ++r) v[r] = cmul(v[r], cv[r]);
  dft8<T, true>(v);
#pragma unroll
  for (int k = 1; k < 8; ++k) v[k] = cmulc(v[k], w64[8 * k + lo]);
#pragma unroll
  for (int d = 0; d < 8; ++d) e2[d] = v[d];
  wave_sync();
#pragma unroll
  for (int d = 0; d < 8; ++d) v[d] = e1[9 * d];
  wave_sync();
  dft8<T, true>(v);
#pragma unroll
  for (int d = 0; d < 8; ++d) e1[8 * d] = v[d];
  wave_sync();
#pragma unroll
  for (int d = 0; d < 8; ++d) v[d] = e0[d * 72];
  wave_sync();
  mul_powers<T, true>(v, base, g);
  dft8<T, true>(v);
#pragma unroll
  for (int t = 1; t < 8; ++t) v[t] = cmulc(v[t], tw[q * t * 64]);
  __builtin_amdgcn_sched_barrier(0);
}

// xor-reduction step over lane distance D within groups of 2 D lanes whose
// halves already hold their own sums
template <int D> __device__ __forceinline__ int lane_swap(int v) {
  if constexpr (D == 1) return __builtin_amdgcn_mov_dpp(v, 0xB1, 0xf, 0xf, true);        // quad_perm 1,0,3,2
  else if constexpr (D == 2) return __builtin_amdgcn_mov_dpp(v, 0x4E, 0xf, 0xf, true);   // quad_perm 2,3,0,1
  else if constexpr (D == 4) return __builtin_amdgcn_mov_dpp(v, 0x141, 0xf, 0xf, true);  // mirror in 8
  else if constexpr (D == 8) return __builtin_amdgcn_mov_dpp(v, 0x140, 0xf, 0xf, true);  // mirror in 16
  else return __shfl_xor(v, D);
}
template <int D> __device__ __forceinline__ double lane_add(double v) {
  return v + __hiloint2double(lane_swap<D>(__double2hiint(v)), lane_swap<D>(__double2loint(v)));
}
template <int D> __device__ __forceinline__ float lane_add(float v) {
  return v + __int_as_float(lane_swap<D>(__float_as_int(v)));
}

// Row transforms of the active points at the four columns of quad p: for
// each row, sum_i u_i W_N^{kx x_i}.  With w = W_N^{p x} = (wx, wy) the columns
// p and N - p need u w and u conj(w), and N/2 -+ p the same with the sign
// (-1)^x, so one look-up of w and four real products per point serve all
// four columns when points of even and odd x are summed apart (the slots
// alternate even and odd x).  The last quad (columns N/4, 3N/4, 0, N/2) uses
// w = (f, 1) for even and (1, -f) for odd x, f = (-1)^{x div 2}, which keeps
// the plain sums beside those of W_4^x.  E: nx values of w; X: the staging.
template <typename T, int N>
__device__ __forceinline__ void sparse_rows(cplx<T>* E, cplx<T>* X, int p, const SparseIn& in, const cplx<T>* __restrict__ U,
                                            int nr, const cplx<T>* __restrict__ tw) {
  using V = cplx<T>;
  using C = WaveCols<T, N>;
  static_assert(C::NT / 64 == kRowWaves, "row tasks are dealt to this block's waves");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool last = p == N / 4;
  const RowWave rw = in.wave[wave];
  const V* up = U + rw.slot;
  const uint16_t* ip = in.ix + rw.slot;
  {
    constexpr int PER = N / 2 / C::NT;
    V e[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int i = tid + k * C::NT;
      const T f = (i & 2) ? -1 : 1;
      e[k] = last ? ((i & 1) ? mk<T>(1, -f) : mk<T>(f, 1)) : tw[(p * i) & (N - 1)];
    }
#pragma unroll
    for (int k = 0; k < PER; ++k)
      if (tid + k * C::NT < in.nx) E[tid + k * C::NT] = e[k];
  }
  __syncthreads();
  for (int k = rw.task; k < rw.task + rw.ntask; ++k) {
    const RowTask tk = in.task[k];
    // a, b, c, d: sums of u.x w.x, u.y w.y, u.x w.y, u.y w.x over even x; o*: odd
    T a = 0, b = 0, c = 0, d = 0, oa = 0, ob = 0, oc = 0, od = 0;
    auto add = [&](auto nn) {   // nn points per lane, all loads ahead of their uses
      constexpr int n = decltype(nn)::value;
      V u[n];
      int x[n];
#pragma unroll
      for (int j = 0; j < n; ++j) {
        u[j] = up[(unsigned)lane + j * 64];
        x[j] = ip[(unsigned)lane + j * 64];
      }
      up += 64 * n;
      ip += 64 * n;
#pragma unroll
      for (int j = 0; j < n; j += 2) {
        const V w = E[x[j]], v = E[x[j + 1]];
        a += u[j].x * w.x; b += u[j].y * w.y; c += u[j].x * w.y; d += u[j].y * w.x;
        oa += u[j + 1].x * v.x; ob += u[j + 1].y * v.y; oc += u[j + 1].x * v.y; od += u[j + 1].y * v.x;
      }
    };
    for (int t = 8; t <= tk.T; t += 8) add(std::integral_constant<int, 8>());
    if (tk.T & 4) add(std::integral_constant<int, 4>());
    if (tk.T & 2) add(std::integral_constant<int, 2>());
    auto reduce = [&](auto dd) {
      constexpr int D = decltype(dd)::value;
      if ((1 << tk.lg) > D) {
        a = lane_add<D>(a); b = lane_add<D>(b); c = lane_add<D>(c); d = lane_add<D>(d);
        oa = lane_add<D>(oa); ob = lane_add<D>(ob); oc = lane_add<D>(oc); od = lane_add<D>(od);
      }
    };
    reduce(std::integral_constant<int, 1>());
    reduce(std::integral_constant<int, 2>());
    reduce(std::integral_constant<int, 4>());
    reduce(std::integral_constant<int, 8>());
    reduce(std::integral_constant<int, 16>());
    reduce(std::integral_constant<int, 32>());
    const int row = tk.row0 + (lane >> tk.lg);
    if ((lane & ((1 << tk.lg) - 1)) == 0 && row < nr) {
      V o[4];
      if (!last) {
        const V ew = mk<T>(a - b, c + d), ec = mk<T>(a + b, d - c);         // even x: u w, u conj(w)
        const V ow = mk<T>(oa - ob, oc + od), oo = mk<T>(oa + ob, od - oc);   // odd x
        o[0] = cadd(ew, ow);
        o[1] = cadd(ec, oo);
        o[2] = csub(ec, oo);
        o[3] = csub(ew, ow);
      } else {
        o[0] = mk<T>(a - ob, d + oc);
        o[1] = mk<T>(a + ob, d - oc);
        o[2] = mk<T>(c + oa, b + od);
        o[3] = mk<T>(c - oa, b - od);
      }
#pragma unroll
      for (int cc = 0; cc < 4; ++cc) X[cc * C::F + st_row(row, cc)] = o[cc];
    }
  }
}

// The columns of quad p of a pair's tile set Tp: from transformed rows in the
// tiles, in place, or (SP) from the anterpolated active points
template <typename T, int N, bool SP>
__device__ __forceinline__ void cols_wave_quad(cplx<T>* buf, cplx<T>* __restrict__ Tp, int nr, int ldt, int p,
                                               const cplx<T>* __restrict__ Cq, const cplx<T>* __restrict__ tw,
                                               const SparseIn& sp, const cplx<T>* __restrict__ U) {
  using V = cplx<T>;
  using C = WaveCols<T, N>;
  constexpr int F = C::F, CW = C::CW, NT = C::NT;
  constexpr int CB = ColCfg<T, N>::CB;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = wave >> 1, h = wave & 1;     // column of the quad, residue ky mod 2
  V* stc = buf + c * F + st_row(lane, c);    // + a multiple of 64 rows
  // coalesced tile access: thread -> (row, column), PER rows RS apart
  constexpr int PER = F * CW / NT, RS = NT / CW;
  const int cc = tid % CW, rc = tid / CW;
  const int pp = quad_pair<N>(p, cc) - 1;
  V* tcol = Tp + ((size_t)(pp / (CB / 2)) * ldt + rc) * CB + (pp % (CB / 2)) * 2 + (cc & 1);
  V* bcol = buf + cc * F + st_row(rc, cc);   // RS is a multiple of 16
  V z[8];
  if constexpr (SP) {
    sparse_rows<T, N>(buf + CW * F, buf, p, sp, U, nr, tw);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 8; ++t) z[t] = 64 * t + lane < nr ? stc[64 * t] : mk<T>(0, 0);
  } else {
    V in[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) in[q] = q * RS + rc < nr ? tcol[q * RS * CB] : mk<T>(0, 0);
#pragma unroll
    for (int q = 0; q < PER; ++q) bcol[q * RS] = in[q];
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 8; ++t) z[t] = stc[64 * t];
  }
  __syncthreads();
  const int pr = quad_pair<N>(p, c);
  const V* Cr = Cq + (size_t)(pr == N / 2 && !(c & 1) ? 0 : pr) * (N / 2 + 8);   // columns 0, N/2: their own rows
  V* w64 = buf + 2 * CW * C::EX;
  const V g = tw[lane * C::Q];
  if (tid < 64) w64[tid] = tw[(tid >> 3) * (tid & 7) * (N / 64)];
  __syncthreads();
  wave_conv<T, N>(z, buf + wave * C::EX, lane, h, g, w64, Cr, tw);
  // add the two waves' partial outputs: each wave owns the rows of half its
  // registers, gives the other half away, and leaves the sums in the staging
  // for coalesced stores
  __syncthreads();
  auto give = [&](auto hh) {
    constexpr int O = 4 * (1 - decltype(hh)::value);
#pragma unroll
    for (int t = O; t < O + 4; ++t) stc[64 * t] = z[t];
  };
  auto add = [&](auto hh) {
    constexpr int O = 4 * decltype(hh)::value;
#pragma unroll
    for (int t = O; t < O + 4; ++t) stc[64 * t] = cadd(stc[64 * t], z[t]);
  };
  if (h == 0) give(std::integral_constant<int, 0>());
  else give(std::integral_constant<int, 1>());
  __syncthreads();
  if (h == 0) add(std::integral_constant<int, 0>());
  else add(std::integral_constant<int, 1>());
  __syncthreads();
#pragma unroll
  for (int q = 0; q < PER; ++q)
    if (q * RS + rc < nr) tcol[q * RS * CB] = bcol[q * RS];
}

template <typename T, int N, bool SP>
__global__ __launch_bounds__((WaveCols<T, N>::NT), 4) void k_cols_wave(
    cplx<T>* __restrict__ Tb, int nr, int ldt, const cplx<T>* __restrict__ Cq, const cplx<T>* __restrict__ tw,
    SparseIn in) {
  __shared__ cplx<T> buf[WaveCols<T, N>::LDS];
  cols_wave_quad<T, N, SP>(buf, Tb + (size_t)blockIdx.y * N * ldt, nr, ldt, quad_of_block<N>(blockIdx.x), Cq, tw, in,
                           (const cplx<T>*)in.U + (size_t)blockIdx.y * in.nslot);
}

template <typename T, int N, int MODE>
__global__ __launch_bounds__((ColCfg<T, N>::NT)) void k_cols(
    cplx<T>* __restrict__ Tb, int nr, int ldt, const cplx<T>* __restrict__ Cq,
    const cplx<T>* __restrict__ tw) {
  using V = cplx<T>;
  constexpr int CB = ColCfg<T, N>::CB;
  constexpr int CW = ColCfg<T, N>::CW;
  constexpr int NT = ColCfg<T, N>::NT;
  constexpr int NBLK = N / CB;
  __shared__ V buf[padded(N * CW)];
  const int b = blockIdx.x;
  const int pair = blockIdx.y;
  const int tid = threadIdx.x;
  if constexpr (MODE == 0) {
    int tb, c0;
    col_block_of<T, N>(b, tb, c0);
    cols_conv_tile<T, N>(buf, Tb + ((size_t)pair * NBLK + tb) * ldt * CB, nr, tb, c0, Cq, tw);
  } else {
    const int kx0 = b * CW;
    for (int idx = tid; idx < N * CW; idx += NT) {
      const int i = idx / CW, c = idx % CW;
      buf[pidx(idx)] = Tb[(size_t)i * N + kx0 + c];
    }
    __syncthreads();
    fft_passes<T, N, CW, NT, false, 1>(buf, tw);
    for (int idx = tid; idx < N * CW; idx += NT) {
      const int i = idx / CW, c = idx % CW;
      Tb[(size_t)i * N + kx0 + c] = buf[pidx(idx)];
    }
  }
}

// Column passes of several contexts that share one spectrum (same n, k eps
// and precision), one launch: entry e of the batch is a pair's tile set
// (tile base of column block 0, kept rows, tile stride); blockIdx.y picks
// the entry.  Each tile is computed exactly as by k_cols.
struct ColBatch {
  static constexpr int kMax = kColBatchMax;
  void* tile[kMax];
  int nr[kMax];
  int ldt[kMax];
  SparseIn in[kMax];
};

template <typename T, int N>
__global__ __launch_bounds__((ColCfg<T, N>::NT)) void k_cols_group(ColBatch batch, const cplx<T>* __restrict__ Cq,
                                                                 const cplx<T>* __restrict__ tw) {
  using V = cplx<T>;
  constexpr int CB = ColCfg<T, N>::CB;
  __shared__ V buf[padded(N * ColCfg<T, N>::CW)];
  const int e = blockIdx.y;
  int tb, c0;
  col_block_of<T, N>(blockIdx.x, tb, c0);
  V* tile = (V*)batch.tile[e] + (size_t)tb * batch.ldt[e] * CB;
  cols_conv_tile<T, N>(buf, tile, batch.nr[e], tb, c0, Cq, tw);
}

template <typename T, int N, bool SP>
__global__ __launch_bounds__((WaveCols<T, N>::NT), 4) void k_cols_wave_group(
    ColBatch batch, const cplx<T>* __restrict__ Cq, const cplx<T>* __restrict__ tw) {
  __shared__ cplx<T> buf[WaveCols<T, N>::LDS];
  const int e = blockIdx.y;
  cols_wave_quad<T, N, SP>(buf, (cplx<T>*)batch.tile[e], batch.nr[e], batch.ldt[e],
                           quad_of_block<N>(blockIdx.x), Cq, tw, batch.in[e], (const cplx<T>*)batch.in[e].U);
}

// ---------------------------------------------------------------------------
// launchers with run-time size dispatch
// ---------------------------------------------------------------------------
#define AIM_FOR_SIZES(X) X(32) X(64) X(128) X(256) X(512) X(1024) X(2048) X(4096)

template <typename T>
aim_status launch_rows_fwd(int n, const cplx<T>* U, int n_act, const int32_t* row_ptr,
                           const int32_t* act_ix, int nr, int ldt, int pairs, cplx<T>* Tb,
                           const cplx<T>* tw, hipStream_t s) {
  if (ldt < nr) return AIM_E_ARG;
  dim3 g(8 * ((nr + 7) / 8), pairs);
  switch (n) {
#define CASE(NN)                                                                               \
  case NN:                                                                                     \
    hipLaunchKernelGGL((k_rows_fwd<T, NN>), g, dim3(row_threads<NN>()), 0, s, U, n_act, row_ptr, \
                       act_ix, nr, ldt, Tb, tw);                                               \
    break;
    AIM_FOR_SIZES(CASE)
#undef CASE
    default: return AIM_E_ARG;
  }
  return hipGetLastError() == hipSuccess ? AIM_OK : AIM_E_HIP;
}

template <typename T>
aim_status launch_rows_inv(int n, const cplx<T>* Tb, int nr, int ldt, const int32_t* row_ptr,
                           const int32_t* act_ix, int pairs, cplx<T>* V, int n_act,
                           const cplx<T>* tw, hipStream_t s) {
  if (ldt < nr) return AIM_E_ARG;
  dim3 g(8 * ((nr + 7) / 8), pairs);
  switch (n) {
#define CASE(NN)                                                                               \
  case NN:                                                                                     \
    hipLaunchKernelGGL((k_rows_inv<T, NN>), g, dim3(row_threads<NN>()), 0, s, Tb, nr, ldt,      \
                       row_ptr, act_ix, V, n_act, tw);                                         \
    break;
    AIM_FOR_SIZES(CASE)
#undef CASE
    default: return AIM_E_ARG;
  }
  return hipGetLastError() == hipSuccess ? AIM_OK : AIM_E_HIP;
}

// The column pass: from transformed rows in Tb, or from the active points of
// `in` (in.nslot > 0, n = kWaveCols).  mode 1: the set-up FFT.
template <typename T, int N>
void cols_wave(cplx<T>* Tb, int nr, int ldt, int pairs, const cplx<T>* Cq, const cplx<T>* tw, const SparseIn& in,
               hipStream_t s, hipEvent_t ev_start, hipEvent_t ev_stop) {
  const dim3 g(N / WaveCols<T, N>::CW, pairs), b(WaveCols<T, N>::NT);
  if (in.nslot > 0)
    hipExtLaunchKernelGGL((k_cols_wave<T, N, true>), g, b, 0, s, ev_start, ev_stop, 0, Tb, nr, ldt, Cq, tw, in);
  else
    hipExtLaunchKernelGGL((k_cols_wave<T, N, false>), g, b, 0, s, ev_start, ev_stop, 0, Tb, nr, ldt, Cq, tw, in);
}
template <typename T, int N>
void cols_wave_group(const ColBatch& bt, int count, bool sparse, const cplx<T>* Cq, const cplx<T>* tw,
                     hipStream_t s) {
  const dim3 g(N / WaveCols<T, N>::CW, count), b(WaveCols<T, N>::NT);
  if (sparse)
    hipLaunchKernelGGL((k_cols_wave_group<T, N, true>), g, b, 0, s, bt, Cq, tw);
  else
    hipLaunchKernelGGL((k_cols_wave_group<T, N, false>), g, b, 0, s, bt, Cq, tw);
}

template <typename T>
aim_status launch_cols(int n, int mode, cplx<T>* Tb, int nr, int ldt, int pairs, const cplx<T>* Cq,
                       const cplx<T>* tw, const SparseIn& in, hipStream_t s, hipEvent_t ev_start, hipEvent_t ev_stop) {
  // kept rows lie in the unpadded half
  if (mode == 0 && (nr < 1 || nr > n / 2 || ldt < nr)) return AIM_E_ARG;
  if (in.nslot > 0 && (mode != 0 || n != kWaveCols || in.nx > n / 2)) return AIM_E_ARG;
  switch (n) {
#define CASE(NN)                                                                                                     \
  case NN: {                                                                                                         \
    if (mode != 0)                                                                                                   \
      hipLaunchKernelGGL((k_cols<T, NN, 1>), dim3(NN / ColCfg<T, NN>::CW, pairs), dim3(ColCfg<T, NN>::NT), 0, s, Tb, \
                         nr, ldt, Cq, tw);                                                                           \
    else if constexpr (NN == kWaveCols)                                                                           \
      cols_wave<T, NN>(Tb, nr, ldt, pairs, Cq, tw, in, s, ev_start, ev_stop);                                        \
    else                                                                                                             \
      hipExtLaunchKernelGGL((k_cols<T, NN, 0>), dim3(NN / ColCfg<T, NN>::CW, pairs), dim3(ColCfg<T, NN>::NT), 0, s,  \
                            ev_start, ev_stop, 0, Tb, nr, ldt, Cq, tw);                                              \
    break;                                                                                                           \
  }
    AIM_FOR_SIZES(CASE)
#undef CASE
    default: return AIM_E_ARG;
  }
  return hipGetLastError() == hipSuccess ? AIM_OK : AIM_E_HIP;
}

// columns per tile of the column pass (tile layout of the intermediate)
int col_block(int n, bool f32) {
  switch (n) {
#define CASE(NN) \
  case NN: return f32 ? ColCfg<float, NN>::CB : ColCfg<double, NN>::CB;
    AIM_FOR_SIZES(CASE)
#undef CASE
  }
  return 0;
}

// grouped column pass over `count` tile sets (count <= ColBatch::kMax), all
// of them from transformed rows or all from active points
template <typename T>
aim_status launch_cols_group(int n, int count, void* const* tiles, const int* nr, const int* ldt, const SparseIn* in,
                             const cplx<T>* Cq, const cplx<T>* tw, hipStream_t s) {
  if (count < 1 || count > ColBatch::kMax) return AIM_E_ARG;
  ColBatch bt;
  const bool sparse = in[0].nslot > 0;
  for (int e = 0; e < ColBatch::kMax; ++e) {
    const int q = e < count ? e : 0;
    if (nr[q] < 1 || nr[q] > n / 2 || ldt[q] < nr[q] || (in[q].nslot > 0) != sparse || in[q].nx > n / 2) return AIM_E_ARG;
    bt.tile[e] = tiles[q];
    bt.nr[e] = nr[q];
    bt.ldt[e] = ldt[q];
    bt.in[e] = in[q];
  }
  if (sparse && n != kWaveCols) return AIM_E_ARG;
  switch (n) {
#define CASE(NN)                                                                                              \
  case NN:                                                                                                    \
    if constexpr (NN == kWaveCols)                                                                         \
      cols_wave_group<T, NN>(bt, count, sparse, Cq, tw, s);                                                   \
    else                                                                                                      \
      hipLaunchKernelGGL((k_cols_group<T, NN>), dim3(NN / ColCfg<T, NN>::CW, count), dim3(ColCfg<T, NN>::NT), 0, \
                         s, bt, Cq, tw);                                                                      \
    break;
    AIM_FOR_SIZES(CASE)
#undef CASE
    default: return AIM_E_ARG;
  }
  return hipGetLastError() == hipSuccess ? AIM_OK : AIM_E_HIP;
}

aim_status launch_rows_fft_inplace(int n, double2* A, const double2* tw, hipStream_t s) {
  switch (n) {
#define CASE(NN)                                                                                   \
  case NN:                                                                                         \
    hipLaunchKernelGGL((k_rows_fft_inplace<double, NN>), dim3(NN), dim3(row_threads<NN>()), 0, s, A, tw); \
    break;
    AIM_FOR_SIZES(CASE)
#undef CASE
    default: return AIM_E_ARG;
  }
  return hipGetLastError() == hipSuccess ? AIM_OK : AIM_E_HIP;
}

template aim_status launch_rows_fwd<double>(int, const double2*, int, const int32_t*, const int32_t*, int, int, int,
                                            double2*, const double2*, hipStream_t);
template aim_status launch_rows_fwd<float>(int, const float2*, int, const int32_t*, const int32_t*, int, int, int,
                                           float2*, const float2*, hipStream_t);
template aim_status launch_rows_inv<double>(int, const double2*, int, int, const int32_t*, const int32_t*, int,
                                            double2*, int, const double2*, hipStream_t);
template aim_status launch_rows_inv<float>(int, const float2*, int, int, const int32_t*, const int32_t*, int,
                                           float2*, int, const float2*, hipStream_t);
template aim_status launch_cols<double>(int, int, double2*, int, int, int, const double2*, const double2*,
                                        const SparseIn&, hipStream_t, hipEvent_t, hipEvent_t);
template aim_status launch_cols<float>(int, int, float2*, int, int, int, const float2*, const float2*,
                                       const SparseIn&, hipStream_t, hipEvent_t, hipEvent_t);
template aim_status launch_cols_group<double>(int, int, void* const*, const int*, const int*, const SparseIn*,
                                              const double2*, const double2*, hipStream_t);
template aim_status launch_cols_group<float>(int, int, void* const*, const int*, const int*, const SparseIn*,
                                             const float2*, const float2*, hipStream_t);

}  // namespace aim
