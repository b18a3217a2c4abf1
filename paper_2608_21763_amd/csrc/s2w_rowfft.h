// Real transforms of whole rows in registers, for every transform length of the library
// (M = L/2 = 16 .. 512 packed slots).
//
// A row's complex transform of M = N1 * N2 points (n = N2 n1 + n2, k = k1 + N1 k2) is a decimation
// in frequency: radix-4 stages with the twiddles after each, a radix-2 stage last where log2 M is
// odd, the first stages (N1 points) and the last ones (N2 points) each in registers and one
// exchange through the row's own LDS buffer between them.  Every product is written as an explicit
// fused multiply-add: half-precision words formed from spectra turn over with the last bit, so
// the rounding must not depend on what the compiler contracts.
// TPR consecutive lanes of one wavefront own a row, E = M / TPR values each, so the steps of a
// row are ordered by the wavefront alone (wave_sync) and the buffer serves every exchange in
// place; a workgroup barrier is needed only where the data come from or go to other lanes.
// nt <= M always (L >= 2 nt - 1), so the packed series z[n] = x[2n] + i x[2n+1] is zero for
// n >= M/2: the forward transform's first pass takes half of its inputs as zeros and the inverse
// transform's second pass forms only half of its outputs.
#pragma once

#include "s2w_device.h"
#include "s2w_wave.h"

namespace s2w {

template <int M_>
struct RowFft {
  static constexpr int M = M_;
  static constexpr int N1 = M >= 64 ? 16 : 4;
  static constexpr int N2 = M / N1;                     // 32, 16, 8, 4 (M = 64), 8, 4
  static constexpr int TPR = N2 < N1 ? N2 : N1;         // lanes per row
  static constexpr int CA = N2 / TPR;                   // first-pass columns per lane
  static constexpr int CB = N1 / TPR;                   // second-pass columns per lane
  static constexpr int E = M / TPR;                     // values per lane
  static constexpr int ROWS = 256 / TPR;                // rows of a 256-thread workgroup
  static constexpr int GA = ROWS / 16;                  // groups of 16 rows
  static constexpr int LD = (N1 * (N2 + 1)) | 1;        // row stride in LDS (odd: column reads spread)
  static_assert(CA * N1 == E && CB * N2 == E && TPR * CB == N1, "row split");
};

// a * w (DIR < 0) or a * conj(w), with the rounding fixed: the product with Im w is rounded, the one
// with Re w is fused.
template <int DIR>
__device__ __forceinline__ float2 tmul(float2 a, float2 w) {
  const float s = DIR < 0 ? w.y : -w.y;
  return make_float2(__builtin_fmaf(a.x, w.x, -(a.y * s)), __builtin_fmaf(a.y, w.x, a.x * s));
}

// exp(-2 pi i m / 64), 0 <= m < 64; folds to constants where m is one
__device__ __forceinline__ float2 w64(int m) {
  constexpr float Q[17] = {1.0f,
                           0.99518472667219693f,
                           0.98078528040323044f,
                           0.95694033573220882f,
                           0.92387953251128674f,
                           0.88192126434835505f,
                           0.83146961230254524f,
                           0.77301045336273699f,
                           0.70710678118654752f,
                           0.63439328416364549f,
                           0.55557023301960222f,
                           0.47139673682599764f,
                           0.38268343236508977f,
                           0.29028467725446233f,
                           0.19509032201612825f,
                           0.09801714032956060f,
                           0.0f};
  const int q = (m >> 4) & 3, r = m & 15;
  const float c = Q[r], s = Q[16 - r];  // cos, sin of 2 pi r / 64
  return q == 0   ? make_float2(c, -s)
         : q == 1 ? make_float2(-s, -c)
         : q == 2 ? make_float2(-c, s)
                  : make_float2(s, c);
}

// Short DFTs in registers, natural order; HZ: x2 = x3 = 0 (not read).
template <int DIR, bool HZ>
__device__ __forceinline__ void dft4v(float2& x0, float2& x1, float2& x2, float2& x3) {
  if constexpr (HZ) {  // x2 = x3 = 0
    const float2 a = x0, b = x1;
    const float2 j = DIR < 0 ? make_float2(b.y, -b.x) : make_float2(-b.y, b.x);
    x0 = cadd(a, b);
    x1 = cadd(a, j);
    x2 = csub(a, b);
    x3 = csub(a, j);
  } else {
    dft4<DIR>(x0, x1, x2, x3);
  }
}

// N points (4, 8, 16 or 32) with constant twiddles
template <int N, int DIR>
__device__ __forceinline__ void dft_reg(float2* v) {
  if constexpr (N == 2) {
    const float2 a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
  } else if constexpr (N == 4) {
    dft4<DIR>(v[0], v[1], v[2], v[3]);
  } else {
    // n = N/4 a + p: radix 4 over a, W_N^{p k}, then N/4 points over p for each k
    constexpr int P = N / 4;
    float2 t[N];
#pragma unroll
    for (int p = 0; p < P; ++p) {
      float2 x[4] = {v[p], v[p + P], v[p + 2 * P], v[p + 3 * P]};
      dft4<DIR>(x[0], x[1], x[2], x[3]);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        t[P * k + p] = p * k ? tmul<DIR>(x[k], w64(p * k * (64 / N))) : x[k];
      }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) dft_reg<P, DIR>(t + P * k);
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int q = 0; q < P; ++q) v[k + 4 * q] = t[P * k + q];
  }
}

// Twiddle table of the lengths whose twiddles do not fit the registers: exp(-2 pi i k / 1024), in LDS.
template <int M>
constexpr int kTwLds = M == 512 ? 1024 : 1;

template <int M>
__device__ __forceinline__ void fill_tw_lds(float2* t) {  // a barrier follows before the first use
  if (M == 512)
    for (int k = threadIdx.x; k < 1024; k += 256) {
      const float2 w = c_tw[k & 511];
      t[k] = k >= 512 ? make_float2(-w.x, -w.y) : w;
    }
}

// A lane's twiddles: the first pass' ones of its columns c + TPR j and the real pre- and post-steps'
// W_L^{c + TPR e}, in registers except for M = 512.
template <int M>
struct RowTw {
  using F = RowFft<M>;
  static constexpr bool LDS = M == 512;
  static constexpr int NT = F::N1 == 16 ? 15 : 3;  // per column
  float2 a[LDS ? 1 : F::CA * NT];
  float2 r[LDS ? 1 : F::E];
  const float2* t;
  int c;

  // exp(-2 pi i n / M), 0 <= n < M
  __device__ __forceinline__ static float2 wm(int n) {
    const int k = n * (TWN / M);
    const float2 w = c_tw[k & (TWN / 2 - 1)];
    return k >= TWN / 2 ? make_float2(-w.x, -w.y) : w;
  }
  __device__ __forceinline__ void init(int lane, const float2* lds) {
    t = lds;
    c = lane;
    if constexpr (!LDS) {
#pragma unroll
      for (int j = 0; j < F::CA; ++j) {
        const int n2 = c + F::TPR * j;
        if constexpr (F::N1 == 4) {
#pragma unroll
          for (int k = 1; k < 4; ++k) a[NT * j + k - 1] = wm(n2 * k);
        } else {
#pragma unroll
          for (int k = 1; k < 4; ++k) {
#pragma unroll
            for (int m = 0; m < 4; ++m) a[NT * j + 3 * m + k - 1] = wm((F::N2 * m + n2) * k);
            a[NT * j + 12 + k - 1] = wm(4 * n2 * k);
          }
        }
      }
#pragma unroll
      for (int e = 0; e < F::E; ++e) r[e] = c_tw[(c + F::TPR * e) * (TWN / (2 * M))];
    }
  }
  // first stage, W_M^{(N2 m + n2) k}; N1 = 4: W_M^{n2 k} (m = 0)
  __device__ __forceinline__ float2 stage1(int j, int m, int k) const {
    if constexpr (LDS) return t[2 * k * (F::N2 * m + c + F::TPR * j)];
    else return a[NT * j + 3 * m + k - 1];
  }
  // second stage, W_{M/4}^{n2 k}
  __device__ __forceinline__ float2 stage2(int j, int k) const {
    if constexpr (LDS) return t[8 * k * (c + F::TPR * j)];
    else return a[NT * j + 12 + k - 1];
  }
  // W_L^{c + TPR e}
  __device__ __forceinline__ float2 real(int e) const {
    if constexpr (LDS) return t[c + F::TPR * e];
    else return r[e];
  }
};

// First pass of column j: v[n1] -> the N1 outputs with their twiddles, natural order in k1.
// HZ: v[n1] = 0 for n1 >= N1/2 (not read).
template <int M, int DIR, bool HZ>
__device__ __forceinline__ void row_pass1(float2* v, int j, const RowTw<M>& tw) {
  auto turn = [](float2 x, float2 w) { return tmul<DIR>(x, w); };
  if constexpr (RowFft<M>::N1 == 4) {
    dft4v<DIR, HZ>(v[0], v[1], v[2], v[3]);
#pragma unroll
    for (int k = 1; k < 4; ++k) v[k] = turn(v[k], tw.stage1(j, 0, k));
  } else {
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      dft4v<DIR, HZ>(v[m], v[4 + m], v[8 + m], v[12 + m]);
#pragma unroll
      for (int k = 1; k < 4; ++k) v[4 * k + m] = turn(v[4 * k + m], tw.stage1(j, m, k));
    }
    float2 t[16];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      dft4<DIR>(v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int k1 = k + 4 * q;
        t[k1] = q ? turn(v[4 * k + q], tw.stage2(j, q)) : v[4 * k + q];
      }
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = t[i];
  }
}

// Pre-step of the inverse real transform (irfft_pre_w with the rounding fixed)
__device__ __forceinline__ float2 row_pre(const float2* X, int k, int M, float2 w) {
  const float2 xk = X[k], xm = X[k ? M - k : 0];
  const float2 d = make_float2(xk.x - xm.x, xk.y + xm.y);
  const float2 o = tmul<+1>(d, w);
  const float2 z = make_float2((xk.x + xm.x) - o.y, (xk.y - xm.y) + o.x);
  return k ? z : make_float2(xk.x + xk.y, xk.x - xk.y);
}

// Packed spectrum in the row buffer X -> z (unnormalised, times L): lane c gets
// u[i][k2] = z[c + TPR i + N1 k2] for k2 < N2/2 (the rest is truncated).  X is overwritten.
template <int M>
__device__ __forceinline__ void row_inverse(float2* X, int c, const RowTw<M>& tw,
                                            float2 (&u)[RowFft<M>::CB][RowFft<M>::N2]) {
  using F = RowFft<M>;
  float2 v[F::CA][F::N1];
#pragma unroll
  for (int j = 0; j < F::CA; ++j)
#pragma unroll
    for (int n1 = 0; n1 < F::N1; ++n1)
      v[j][n1] = row_pre(X, F::N2 * n1 + c + F::TPR * j, M, tw.real(F::CA * n1 + j));
  wave_sync();
#pragma unroll
  for (int j = 0; j < F::CA; ++j) {
    row_pass1<M, +1, false>(v[j], j, tw);
#pragma unroll
    for (int k1 = 0; k1 < F::N1; ++k1) X[k1 * (F::N2 + 1) + c + F::TPR * j] = v[j][k1];
  }
  wave_sync();
#pragma unroll
  for (int i = 0; i < F::CB; ++i)
#pragma unroll
    for (int n2 = 0; n2 < F::N2; ++n2) u[i][n2] = X[(c + F::TPR * i) * (F::N2 + 1) + n2];
  wave_sync();
#pragma unroll
  for (int i = 0; i < F::CB; ++i) dft_reg<F::N2, +1>(u[i]);
}

// Lane c's v[j][n1] = z[N2 n1 + c + TPR j], n1 < N1/2 (zero beyond) -> packed spectrum in natural
// order in the row buffer X.  The row's lanes must be past their reads of X.
template <int M>
__device__ __forceinline__ void row_forward(float2* X, int c, const RowTw<M>& tw,
                                            float2 (&v)[RowFft<M>::CA][RowFft<M>::N1]) {
  using F = RowFft<M>;
#pragma unroll
  for (int j = 0; j < F::CA; ++j) {
    row_pass1<M, -1, true>(v[j], j, tw);
#pragma unroll
    for (int k1 = 0; k1 < F::N1; ++k1) X[k1 * (F::N2 + 1) + c + F::TPR * j] = v[j][k1];
  }
  wave_sync();
  float2 u[F::CB][F::N2];
#pragma unroll
  for (int i = 0; i < F::CB; ++i)
#pragma unroll
    for (int n2 = 0; n2 < F::N2; ++n2) u[i][n2] = X[(c + F::TPR * i) * (F::N2 + 1) + n2];
  wave_sync();
#pragma unroll
  for (int i = 0; i < F::CB; ++i) {
    dft_reg<F::N2, -1>(u[i]);
#pragma unroll
    for (int k2 = 0; k2 < F::N2; ++k2) X[c + F::TPR * i + F::N1 * k2] = u[i][k2];
  }
  wave_sync();
  // post-step of the real transform, slots k and M - k of a lane together and in place; k = 0 goes
  // with k = M/2 (whose partner is itself: the conjugate)
#pragma unroll
  for (int e = 0; e < F::E / 2; ++e) {
    const int k = c + F::TPR * e;
    const bool first = e == 0 && c == 0;
    const int k2 = first ? M / 2 : M - k;
    const float2 zk = X[k], zm = X[k2];
    const float2 zc = cconj(zm);
    const float2 ev = cscale(cadd(zk, zc), 0.5f);
    const float2 d = csub(zk, zc);
    const float2 t = tmul<-1>(make_float2(0.5f * d.y, -0.5f * d.x), tw.real(e));  // W_L^k d / (2i)
    float2 xk = cadd(ev, t), xm = cconj(csub(ev, t));
    if (first) {
      xk = make_float2(zk.x + zk.y, zk.x - zk.y);
      xm = zc;
    }
    X[k] = xk;
    X[k2] = xm;
  }
  wave_sync();
}

}  // namespace s2w
