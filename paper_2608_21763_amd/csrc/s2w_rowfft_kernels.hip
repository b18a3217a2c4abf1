// Row-transform kernels on the register transforms of s2w_rowfft.h: operator setup, the batched
// source and output transforms and the batched mid-chain, for every transform length.
//
// A unit of every kernel is GA x 16 rows: GA consecutive values of an outer index a and 16 of an
// inner index b, the one that is contiguous on the far side (subfaults, grid rows or ruptures of
// a spectrum store), so that spectra move as 128-byte runs of 16 and time rows as runs of a row.
#include <algorithm>

#include "s2w_half.h"
#include "s2w_internal.h"
#include "s2w_rowfft.h"

namespace s2w {

hipError_t upload_twiddles_rows() { return upload_tw_table(); }

namespace {

constexpr int ilog2c(int v) { return v <= 1 ? 0 : 1 + ilog2c(v / 2); }

// Destination of the forward transforms of a unit.
enum RfftOut {
  OUT_RUN = 0,   // complex64, 16 values of b contiguous per slot
  OUT_ROW = 1,   // complex64, the slots of a row contiguous
  OUT_MAX = 2,   // largest |Re|, |Im| of a grid row and slot over its columns (no spectra)
  OUT_G = 3,     // scaled half words of the elastic store (+ 0: bf16, + 1: f16), columns along b
  OUT_F = 5      // the same of the acoustic store, grid rows along b
};

struct RfftArgs {
  const float* in;  // row (a, b) at in + a * in_a + b * in_b, nt samples
  int64_t in_a, in_b;
  int na, na_out, nb, nb_out;  // rows a < na, b < nb exist (others are zero); a < na_out, b < nb_out are written
  int nt;
  float scale;
  void* out;  // slot l of row (a, b) at out + a * oa + b * ob + l * ol
  int64_t oa, ob, ol;
  int nau, nbu;  // units along a and b
  // OUT_MAX and the half words: the grid row is a (elastic, columns along b) or b (columns along a).  A
  // workgroup (of nwg) keeps one unit index of the grid rows and runs over one of `splits` ranges of the other
  int elastic, splits, nfix, nwg;
  uint32_t* mx;     // [grid row of this call][slot]: largest value (float bits)
  float* down;      // inverse scales [grid row][slot]
  int64_t row0;
  int ncp16;        // elastic words: column blocks of 16 (row-block-major store); 0: strided words
};

// Zero-padded forward real FFT of time rows (Alg. 2 steps 1-2), one unit at a time, the next
// unit's samples loaded under the transform of the current one.
//
// Bound by HBM at setup (4 nt bytes read, 4 or 8 M written per row) and by the latency of one unit on
// few rows.  The register transform replaced a radix-4 one in LDS with a barrier per stage and 4- and
// 8-byte strided stores: 512 grid rows of 963 + 64 columns x 256 steps into half words took 2.9 ms
// (16 rows per launch), now 0.51 ms in all; one unit of 16 short rows 12.6, now 3.8 us.
template <int M, int OUT>
__device__ __forceinline__ void rfft_units(const RfftArgs& p, int wg, int nwg, float2* X, float2* twl) {
  using F = RowFft<M>;
  constexpr int LOGM = ilog2c(M), Q = F::GA * M / 16, H = F::N1 / 2;
  constexpr bool GW = OUT == OUT_G || OUT == OUT_G + 1, FW = OUT == OUT_F || OUT == OUT_F + 1;
  constexpr bool FIX = GW || FW || OUT == OUT_MAX;
  constexpr int HT = OUT == OUT_G || OUT == OUT_F ? 1 : 2;
  const int tid = threadIdx.x;
  const int row = tid / F::TPR, c = tid % F::TPR, ga = row >> 4, br = row & 15;  // transform
  const int r = tid & 15, lq = tid >> 4;                                        // stores by run
  float2* Xr = X + row * F::LD;
  fill_tw_lds<M>(twl);
  RowTw<M> tw;
  tw.init(c, twl);
  // units u = fixed * nloop + step; with FIX a workgroup's fixed index is its grid rows
  const bool loop_b = !FIX || p.elastic;
  const int nloop = loop_b ? p.nbu : p.nau;
  int64_t u, u1, du, f = 0;
  int split = 0;
  if (FIX) {
    // workgroups go round the eight XCDs; neighbours in the fixed index (grid rows whose words
    // share cache lines) are given to one XCD
    const int at = (wg & 7) * (nwg >> 3) + (wg >> 3);
    if (at >= p.nfix * p.splits) return;
    f = at % p.nfix;
    split = at / p.nfix;
    u = f * nloop + (int64_t)nloop * split / p.splits;
    u1 = f * nloop + (int64_t)nloop * (split + 1) / p.splits;
    du = 1;
  } else {
    u = wg;
    u1 = (int64_t)p.nau * p.nbu;
    du = nwg;
  }
  if (kTwLds<M> > 1) __syncthreads();  // the twiddle table
  const bool even = !(p.nt & 1);
  auto unit = [&](int64_t v, int& a0, int& b0) {
    const int f = (int)(v / nloop), s = (int)(v - (int64_t)f * nloop);
    a0 = (loop_b ? f : s) * F::GA;
    b0 = (loop_b ? s : f) * 16;
  };
  float2 pv[F::CA][H];
  auto fetch = [&](int64_t v) {
    int a0, b0;
    unit(v, a0, b0);
    const int a = a0 + ga, b = b0 + br;
    const bool live = a < p.na && b < p.nb;
    const float* x = p.in + (live ? a * p.in_a + b * p.in_b : 0);
#pragma unroll
    for (int j = 0; j < F::CA; ++j)
#pragma unroll
      for (int n1 = 0; n1 < H; ++n1) {
        const int m0 = 2 * (F::N2 * n1 + c + F::TPR * j);
        float2 xv = make_float2(0.f, 0.f);
        if (even) {  // rows of an even length: the pair is one aligned 8-byte load
          if (live && m0 < p.nt) xv = *reinterpret_cast<const float2*>(x + m0);
        } else {
          if (live && m0 < p.nt) xv.x = x[m0];
          if (live && m0 + 1 < p.nt) xv.y = x[m0 + 1];
        }
        pv[j][n1] = xv;
      }
  };
  // half words: scale multipliers of this thread's stores, the same in all its units; the first range of
  // the grid rows leaves the inverses.  Elastic words go four columns (16 bytes) at a time, thread -> column
  // quad tid % 4 of slot and grid row (tid / 4 + 64 k); the acoustic ones by single words (their
  // alignment is the caller's first row's)
  constexpr int NUP = GW ? Q / 4 : (FW ? Q : 1);
  float up[NUP];
  if ((GW || FW) && u < u1) {
    int a0, b0;
    unit(u, a0, b0);
#pragma unroll
    for (int k = 0; k < NUP; ++k) {
      const int q = GW ? (tid >> 2) + 64 * k : lq + 16 * k, l = q & (M - 1);
      const int g = GW ? a0 + (q >> LOGM) : b0 + r, ng = GW ? p.na : p.nb;
      float dn;
      pow2_scale(__uint_as_float(p.mx[(int64_t)min(g, ng - 1) * M + l]), up[k], dn);
      if (split == 0 && g < ng && (GW ? (tid & 3) == 0 : q < M)) p.down[(p.row0 + g) * M + l] = dn;
    }
  }
  float mx[OUT == OUT_MAX ? F::E : 1];
  if (OUT == OUT_MAX) {
#pragma unroll
    for (int e = 0; e < F::E; ++e) mx[e] = 0.f;
  }
  if (u < u1) fetch(u);
  for (; u < u1; u += du) {
    int a0, b0;
    unit(u, a0, b0);
    float2 v[F::CA][F::N1];
#pragma unroll
    for (int j = 0; j < F::CA; ++j)
#pragma unroll
      for (int n1 = 0; n1 < H; ++n1) v[j][n1] = make_float2(pv[j][n1].x * p.scale, pv[j][n1].y * p.scale);
    if (u + du < u1) fetch(u + du);
    row_forward<M>(Xr, c, tw, v);
    if (OUT == OUT_MAX) {
#pragma unroll
      for (int e = 0; e < F::E; ++e) {
        const float2 z = Xr[c + F::TPR * e];
        mx[e] = fmaxf(mx[e], fmaxf(fabsf(z.x), fabsf(z.y)));
      }
      wave_sync();
      continue;
    }
    __syncthreads();
    if (OUT == OUT_ROW) {
      float2* out = (float2*)p.out;
#pragma unroll 4
      for (int i = tid; i < F::ROWS * M; i += 256) {
        const int rr = i >> LOGM, l = i & (M - 1);
        const int a = a0 + (rr >> 4), b = b0 + (rr & 15);
        if (a < p.na_out && b < p.nb_out) out[a * p.oa + b * p.ob + l] = X[rr * F::LD + l];
      }
    } else if constexpr (GW) {
#pragma unroll
      for (int k = 0; k < NUP; ++k) {
        const int q = (tid >> 2) + 64 * k, l = q & (M - 1), g2 = q >> LOGM, c4 = 4 * (tid & 3);
        if (a0 + g2 >= p.na_out) continue;
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float2 z = X[(g2 * 16 + c4 + i) * F::LD + l];
          w[i] = pack_half2<HT>(z.x * up[k], z.y * up[k]);
        }
        const int64_t g = p.row0 + a0 + g2;
        *reinterpret_cast<uint4*>((uint32_t*)p.out + l * p.ol + ((g >> 4) * p.ncp16 + (b0 >> 4)) * 256 +
                                  (g & 15) * 16 + c4) = make_uint4(w[0], w[1], w[2], w[3]);
      }
    } else {
#pragma unroll
      for (int k = 0; k < Q; ++k) {
        const int q = lq + 16 * k, l = q & (M - 1), g2 = q >> LOGM;
        const int a = a0 + g2, b = b0 + r;
        if (a >= p.na_out || b >= p.nb_out) continue;
        const float2 z = X[(g2 * 16 + r) * F::LD + l];
        if constexpr (FW)
          ((uint32_t*)p.out)[a * p.oa + p.row0 + b + l * p.ol] = pack_half2<HT>(z.x * up[k], z.y * up[k]);
        else
          ((float2*)p.out)[a * p.oa + b + l * p.ol] = z;
      }
    }
    __syncthreads();  // the next unit refills X
  }
  if (OUT == OUT_MAX) {
    // the rows of one grid row together through LDS, then one atomic per grid row and slot
    float* W = reinterpret_cast<float*>(X);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < F::E; ++e) W[row * M + c + F::TPR * e] = mx[e];
    __syncthreads();
    const int ng = p.elastic ? F::GA : 16, nr = p.elastic ? 16 : F::GA;  // grid rows of a unit, rows of each
    for (int i = tid; i < ng * M; i += 256) {
      const int gr = i >> LOGM, l = i & (M - 1);
      float m = 0.f;
      for (int k = 0; k < nr; ++k) m = fmaxf(m, W[(p.elastic ? gr * 16 + k : k * 16 + gr) * M + l]);
      const int64_t g = f * ng + gr;
      if (g < (p.elastic ? p.na : p.nb)) atomicMax(p.mx + g * M + l, __float_as_uint(m));
    }
  }
}

#define S2W_RFFT_LDS(M_)                                        \
  __shared__ float2 X[RowFft<M_>::ROWS * RowFft<M_>::LD];       \
  __shared__ float2 twl[kTwLds<M_>]

template <int M, int OUT>
__global__ __launch_bounds__(256, M <= 256 ? 3 : 2) void k_rfft_units(const RfftArgs p) {
  S2W_RFFT_LDS(M);
  rfft_units<M, OUT>(p, blockIdx.x, gridDim.x, X, twl);
}

// Half-precision setup, both operators in one launch, the elastic one by the first workgroups: the maxima of the grid
// rows, and their words.
template <int M>
__global__ __launch_bounds__(256, M <= 256 ? 3 : 2) void k_rfft_max(const RfftArgs g, const RfftArgs f) {
  S2W_RFFT_LDS(M);
  const bool e = (int)blockIdx.x < g.nwg;
  RfftArgs p{};
  p.in = e ? g.in : f.in;
  p.in_a = e ? g.in_a : f.in_a;
  p.in_b = e ? g.in_b : f.in_b;
  p.na = e ? g.na : f.na;
  p.nb = e ? g.nb : f.nb;
  p.nt = g.nt;
  p.scale = g.scale;
  p.nau = e ? g.nau : f.nau;
  p.nbu = e ? g.nbu : f.nbu;
  p.elastic = e;
  p.splits = e ? g.splits : f.splits;
  p.nfix = e ? g.nfix : f.nfix;
  p.mx = e ? g.mx : f.mx;
  rfft_units<M, OUT_MAX>(p, e ? blockIdx.x : blockIdx.x - g.nwg, e ? g.nwg : f.nwg, X, twl);
}
template <int M, int HG, int HF>
__global__ __launch_bounds__(256, M <= 256 ? 3 : 2) void k_rfft_words(const RfftArgs g, const RfftArgs f) {
  S2W_RFFT_LDS(M);
  if ((int)blockIdx.x < g.nwg)
    rfft_units<M, OUT_G + HG - 1>(g, blockIdx.x, g.nwg, X, twl);
  else
    rfft_units<M, OUT_F + HF - 1>(f, blockIdx.x - g.nwg, f.nwg, X, twl);
}
#undef S2W_RFFT_LDS

// Inverse real FFT (Alg. 2 steps 4-5: keep n < nt) of summed partial spectra,
//   out[b * ob + a * oa + n] = scale * IFFT(tau[l][b] * sum_s part[s * p_s + a * pa + b * pb + l * pl])[n].
// ROW: the slots of a row are contiguous (pl = 1), else 16 values of b are (pb = 1).
struct IrfftArgs {
  const float2* part;
  int splits;
  int64_t p_s, pa, pb, pl;
  int na, nb;
  const float* tau;
  int64_t tau_l;
  float* out;
  int64_t oa, ob;
  int nt;
  float scale;
  int nau, nbu;
};

template <int M, bool ROW>
__global__ __launch_bounds__(256, 2) void k_irfft_units(const IrfftArgs p) {
  using F = RowFft<M>;
  constexpr int LOGM = ilog2c(M), Q = F::GA * M / 16;
  __shared__ float2 X[F::ROWS * F::LD];
  const int tid = threadIdx.x;
  const int row = tid / F::TPR, c = tid % F::TPR, ga = row >> 4, br = row & 15;
  const int r = tid & 15, lq = tid >> 4;
  float2* Xr = X + row * F::LD;
  __shared__ float2 twl[kTwLds<M>];
  fill_tw_lds<M>(twl);
  RowTw<M> tw;
  tw.init(c, twl);
  const int64_t units = (int64_t)p.nau * p.nbu;
  for (int64_t u = blockIdx.x; u < units; u += gridDim.x) {
    const int a0 = (int)(u / p.nbu) * F::GA, b0 = (int)(u % p.nbu) * 16;
    // all loads of one split in flight together, splits added in order; loads are unconditional
    // (rows past the end read the last one and are zeroed)
    constexpr int QC = Q < 16 ? Q : 16;
#pragma unroll 1
    for (int k0 = 0; k0 < Q; k0 += QC) {
      const float2* src[QC];
      float2 sum[QC];
#pragma unroll
      for (int k = 0; k < QC; ++k) {
        const int q = ROW ? tid + 256 * (k0 + k) : lq + 16 * (k0 + k);
        const int l = q & (M - 1), rr = ROW ? q >> LOGM : (q >> LOGM) * 16 + r;
        const int a = a0 + (rr >> 4), b = b0 + (rr & 15);
        src[k] = p.part + (a < p.na ? a : p.na - 1) * p.pa + (b < p.nb ? b : p.nb - 1) * p.pb + l * p.pl;
        sum[k] = *src[k];
      }
      for (int t = 1; t < p.splits; ++t) {
        float2 w[QC];
#pragma unroll
        for (int k = 0; k < QC; ++k) w[k] = src[k][t * p.p_s];
#pragma unroll
        for (int k = 0; k < QC; ++k) sum[k] = cadd(sum[k], w[k]);
      }
#pragma unroll
      for (int k = 0; k < QC; ++k) {
        const int q = ROW ? tid + 256 * (k0 + k) : lq + 16 * (k0 + k);
        const int l = q & (M - 1), rr = ROW ? q >> LOGM : (q >> LOGM) * 16 + r;
        const int a = a0 + (rr >> 4), b = b0 + (rr & 15);
        const bool ok = a < p.na && b < p.nb;
        const float td = p.tau ? p.tau[l * p.tau_l + (b < p.nb ? b : p.nb - 1)] : 1.f;
        X[rr * F::LD + l] = ok ? make_float2(sum[k].x * td, sum[k].y * td) : make_float2(0.f, 0.f);
      }
    }
    __syncthreads();
    float2 z[F::CB][F::N2];
    row_inverse<M>(Xr, c, tw, z);
    const int a = a0 + ga, b = b0 + br;
    if (a < p.na && b < p.nb) {
      float* dst = p.out + a * p.oa + b * p.ob;
#pragma unroll
      for (int i = 0; i < F::CB; ++i)
#pragma unroll
        for (int k2 = 0; k2 < F::N2 / 2; ++k2) {
          const int m0 = 2 * (c + F::TPR * i + F::N1 * k2);
          const float2 y = make_float2(z[i][k2].x * p.scale, z[i][k2].y * p.scale);
          if (m0 + 1 < p.nt && !(p.nt & 1)) {
            *reinterpret_cast<float2*>(dst + m0) = y;
          } else {
            if (m0 < p.nt) dst[m0] = y.x;
            if (m0 + 1 < p.nt) dst[m0 + 1] = y.y;
          }
        }
    }
    __syncthreads();  // the next unit refills X
  }
}

// Fixed-order sum of partial spectra and inverse real FFT of one row per workgroup,
//   out[o * nt + n] = scale * IFFT(sum_p part[p][o][.])[n],  n < nt  (part rows of M slots, nop per partial).
// QL threads share a pair of slots: thread q sums partials q, q + QL, ... (eight loads in flight; past
// the end the last one, not added), then the QL sums are added in order through LDS.
//
// Bound by latency: the sum and the transform are a few microseconds each whatever their bytes.  128
// partials of 4 x 32 slots 5.5 + 4.2 us as two launches, 4.7 as one; 256 of 32 x 256 (17 MB) 16 -> 11; 64 of
// 60 x 256 10 + 7 -> 7.6.
template <int M>
__global__ __launch_bounds__(1024) void k_sum_irfft_rows(const v4f* __restrict__ part, int nparts, int64_t p_s,
                                                         float* __restrict__ out, int nt, float scale) {
  using F = RowFft<M>;
  constexpr int I = M / 2, QL = 1024 / I;
  __shared__ v4f sh[QL][I];
  __shared__ float2 X[F::LD];
  const int tid = threadIdx.x, it = tid % I, q = tid / I;
  const v4f* src = part + (int64_t)blockIdx.x * I + it;
  v4f s = v4f{0.f, 0.f, 0.f, 0.f};
  for (int p = q; p < nparts; p += 8 * QL) {
    v4f a[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) a[u] = src[(int64_t)min(p + u * QL, nparts - 1) * p_s];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (p + u * QL < nparts) s += a[u];
  }
  sh[q][it] = s;
  __syncthreads();
  if (q == 0) {
    for (int k = 1; k < QL; ++k) s += sh[k][it];
    X[2 * it] = make_float2(s.x, s.y);
    X[2 * it + 1] = make_float2(s.z, s.w);
  }
  __syncthreads();
  if (tid >= F::TPR) return;
  RowTw<M> tw;
  tw.init(tid, nullptr);
  float2 z[F::CB][F::N2];
  row_inverse<M>(X, tid, tw, z);
  float* dst = out + (int64_t)blockIdx.x * nt;
#pragma unroll
  for (int i = 0; i < F::CB; ++i)
#pragma unroll
    for (int k2 = 0; k2 < F::N2 / 2; ++k2) {
      const int m0 = 2 * (tid + F::TPR * i + F::N1 * k2);
      if (m0 < nt) dst[m0] = z[i][k2].x * scale;
      if (m0 + 1 < nt) dst[m0 + 1] = z[i][k2].y * scale;
    }
}

// Batched mid-chain round trip on U[g][l][b] (complex, b < bp), in place: for GA grid rows and 16
// ruptures, inverse FFT -> truncate -> D_t -> zero-pad -> FFT (Alg. 1 line 3; Alg. 2 steps 4-5 and
// 1-2), times the store's scale sF[g][l], written as complex64 (PACK = 0) or as bfloat16 high and
// low terms of the real and imaginary parts in two words (PACK = 1).  The next unit's rows are
// loaded under the transforms of the current one (M = 512: 32 values per lane leave no registers
// for that; the second workgroup of the CU covers the loads).  CMAX: the grid is a multiple of the rupture
// blocks (nbb), so a workgroup keeps its ruptures; it leaves the largest |Re|, |Im| of every
// (slot, rupture) it writes in cmax[blockIdx / nbb][l][b] (b < bp; zero for b >= B).
//
// Bound by HBM (16 M bytes read and written per grid row and rupture) and the LDS passes; the generic
// LDS transforms it replaced spent a barrier and two LDS passes per radix-4 stage.  240 x 9,001 grid
// rows x 500 steps (M = 512), 64 ruptures: 9.1 -> 1.3 ms (3.6 TB/s); 9,440 rows x 100 steps (M = 128),
// 33 ruptures with snapshots: 0.58 -> 0.29 ms.
//
// FLAT (few ruptures, bp 8 or 16): U is [l][g][b] and a unit GA x 16 consecutive values of g * bp + b, so
// that 8 ruptures fill a unit; every workgroup keeps its ruptures and leaves maxima.
struct MidArgs {
  float2* U;
  const float* sF;
  int ngrid, B, bp, nt, mode;
  float mscale;
  float* cmax;
  int nbb, units;
  DispOut disp;
};

typedef float mid_f2 __attribute__((ext_vector_type(2)));
typedef __bf16 mid_b2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t mid_bf16x2(float a, float b) {
  const mid_f2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, mid_b2));
}

template <int M, bool PACK, bool DISP, bool CMAX, bool FLAT = false>
__global__ __launch_bounds__(256, 2) void k_mid_units(const MidArgs p) {
  using F = RowFft<M>;
  // NG: grid rows of a unit, at most
  constexpr int LOGM = ilog2c(M), Q = F::GA * M / 16, NG = FLAT ? F::ROWS / 8 : F::GA, NS = (NG * M + 255) / 256;
  static_assert(!FLAT || (CMAX && !PACK && !DISP), "flat units");
  __shared__ float2 X[F::ROWS * F::LD];
  __shared__ float fsl[NG * M];
  __shared__ short dtab[DISP ? 512 : 1];
  const int tid = threadIdx.x;
  if (DISP) disp_fill_cols(p.disp, p.nt, dtab);  // ordered by the first unit's barrier
  const int row = tid / F::TPR, c = tid % F::TPR, ga = row >> 4, br = row & 15;
  const int r = tid & 15, lq = tid >> 4;
  float2* Xr = X + row * F::LD;
  __shared__ float2 twl[kTwLds<M>];
  fill_tw_lds<M>(twl);
  RowTw<M> tw;
  tw.init(c, twl);
  float2 pre[Q];
  float fs[NS];
  float cmx[CMAX ? Q : 1];
  if (CMAX) {
#pragma unroll
    for (int k = 0; k < Q; ++k) cmx[k] = 0.f;
  }
  const int rows = p.ngrid * p.bp;  // FLAT
  // loads are unconditional: rows and ruptures past the end read the last one and are zeroed
  auto fetch = [&](int u) {
    const int g0 = FLAT ? u * F::ROWS / p.bp : (u / p.nbb) * F::GA, b = (u % p.nbb) * 16 + r;
#pragma unroll
    for (int k = 0; k < Q; ++k) {
      const int q = lq + 16 * k, l = q & (M - 1), g = g0 + (q >> LOGM);
      if (FLAT) {  // scalar base per k, 32-bit lane offset
        const int fr = u * F::ROWS + (q >> LOGM) * 16 + r;
        const float2 v = (p.U + (int64_t)((16 * k) & (M - 1)) * rows)[(uint32_t)(lq * rows + min(fr, rows - 1))];
        pre[k] = fr < rows && r % p.bp < p.B ? v : make_float2(0.f, 0.f);
        continue;
      }
      const int gc = F::GA == 1 || g < p.ngrid ? g : p.ngrid - 1;
      const float2 v = p.U[((int64_t)gc * M + l) * p.bp + (b < p.B ? b : p.B - 1)];
      pre[k] = b < p.B && (F::GA == 1 || g < p.ngrid) ? v : make_float2(0.f, 0.f);
    }
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      const int q = tid + 256 * k, g = g0 + (q >> LOGM);
      fs[k] = p.sF && q < NG * M && g < p.ngrid ? p.sF[(int64_t)g0 * M + q] : 1.f;
    }
  };
  constexpr bool AHEAD = M < 512;
  int u = blockIdx.x;
  if (AHEAD && u < p.units) fetch(u);
  for (; u < p.units; u += gridDim.x) {
    const int g0 = (u / p.nbb) * F::GA, b0 = (u % p.nbb) * 16;
    if (!AHEAD) fetch(u);
#pragma unroll
    for (int k = 0; k < Q; ++k) {
      const int q = lq + 16 * k;
      X[((q >> LOGM) * 16 + r) * F::LD + (q & (M - 1))] = pre[k];
    }
#pragma unroll
    for (int k = 0; k < NS; ++k)
      if (tid + 256 * k < NG * M) fsl[tid + 256 * k] = fs[k];
    __syncthreads();
    if (AHEAD && u + (int)gridDim.x < p.units) fetch(u + gridDim.x);
    {
      float2 z[F::CB][F::N2];
      row_inverse<M>(Xr, c, tw, z);
      const DispRows dr{p.disp.base + (int64_t)(g0 + ga) * p.disp.grid_stride + (int64_t)b0 * p.disp.row_stride,
                        p.disp.row_stride, g0 + ga < p.ngrid ? p.B - b0 : 0, p.disp.scale};
#pragma unroll
      for (int i = 0; i < F::CB; ++i)
#pragma unroll
        for (int k2 = 0; k2 < F::N2 / 2; ++k2) {
          const int n = c + F::TPR * i + F::N1 * k2;
          Xr[n] = z[i][k2];
          if (DISP) {
            if (2 * n < p.nt) disp_put(&dr, dtab, br, 2 * n, z[i][k2].x);
            if (2 * n + 1 < p.nt) disp_put(&dr, dtab, br, 2 * n + 1, z[i][k2].y);
          }
        }
    }
    wave_sync();
    float2 v[F::CA][F::N1];
#pragma unroll
    for (int j = 0; j < F::CA; ++j)
#pragma unroll
      for (int n1 = 0; n1 < F::N1 / 2; ++n1) {
        const int n = F::N2 * n1 + c + F::TPR * j, m0 = 2 * n, m1 = m0 + 1;
        const float2 z = Xr[n];
        float a = z.x, b = z.y;
        // neighbours are read unconditionally (clamped index) and selected
        if (p.mode == MID_BACKWARD) {
          const float zp = Xr[n > 0 ? n - 1 : 0].y;
          b -= a;
          a -= n > 0 ? zp : 0.f;
        } else if (p.mode == MID_BACKWARD_T) {
          const float zn = Xr[n + 1 < M / 2 ? n + 1 : n].x;
          a -= m1 < p.nt ? b : 0.f;
          b -= m1 + 1 < p.nt ? zn : 0.f;  // m1 + 1 < nt <= M implies n + 1 < M/2
        }
        v[j][n1] = make_float2((m0 < p.nt ? a : 0.f) * p.mscale, (m1 < p.nt ? b : 0.f) * p.mscale);
      }
    wave_sync();
    row_forward<M>(Xr, c, tw, v);
    __syncthreads();
    const int b = FLAT ? r % p.bp : b0 + r;
    if (b < p.B) {
#pragma unroll
      for (int k = 0; k < Q; ++k) {
        const int q = lq + 16 * k, l = q & (M - 1), g2 = q >> LOGM;
        const int rr = g2 * 16 + r, fr = u * F::ROWS + rr;  // FLAT
        if (FLAT ? fr >= rows : (F::GA > 1 && g0 + g2 >= p.ngrid)) continue;
        const float f = fsl[FLAT ? rr / p.bp * M + l : q];
        const float2 x = X[(g2 * 16 + r) * F::LD + l];
        const float2 y = make_float2(x.x * f, x.y * f);
        float2* dst = FLAT ? (p.U + (int64_t)((16 * k) & (M - 1)) * rows) + (uint32_t)(lq * rows + fr) : p.U + ((int64_t)(g0 + g2) * M + l) * p.bp + b;
        if (PACK) {
          const uint32_t h = mid_bf16x2(y.x, y.y);
          const uint32_t lo = mid_bf16x2(y.x - __uint_as_float(h << 16), y.y - __uint_as_float(h & 0xffff0000u));
          *reinterpret_cast<uint2*>(dst) = make_uint2(h, lo);
        } else {
          *dst = y;
        }
        if (CMAX) cmx[k] = fmaxf(cmx[k], fmaxf(fabsf(y.x), fabsf(y.y)));
      }
    }
    __syncthreads();  // the next unit refills X
  }
  if (FLAT) {
    float* o = p.cmax + (int64_t)blockIdx.x * M * p.bp + r;
    constexpr int QM = M / 16;
#pragma unroll
    for (int k = 0; k < QM; ++k) {
      float m = cmx[k];
#pragma unroll
      for (int g2 = 1; g2 < F::GA; ++g2) m = fmaxf(m, cmx[k + QM * g2]);
      if (p.bp == 8) m = fmaxf(m, __shfl_xor(m, 8, 64));
      if (r < p.bp) o[(int64_t)(lq + 16 * k) * p.bp] = m;  // zero for b >= B
    }
  } else if (CMAX) {
    const int b = (int)(blockIdx.x % p.nbb) * 16 + r;
    if (b < p.bp) {
      float* o = p.cmax + (int64_t)(blockIdx.x / p.nbb) * M * p.bp + b;
      constexpr int QM = M / 16;  // slots of one grid row per thread; GA rows share a slot
#pragma unroll
      for (int k = 0; k < QM; ++k) {
        float m = cmx[k];
#pragma unroll
        for (int g2 = 1; g2 < F::GA; ++g2) m = fmaxf(m, cmx[k + QM * g2]);
        o[(int64_t)(lq + 16 * k) * p.bp] = b < p.B ? m : 0.f;
      }
    }
  }
}

#define S2W_BY_M(M_, CALL_)     \
  switch (M_) {                 \
    case 16: CALL_(16); break;   \
    case 32: CALL_(32); break;   \
    case 64: CALL_(64); break;   \
    case 128: CALL_(128); break; \
    case 256: CALL_(256); break; \
    case 512: CALL_(512); break; \
    default: return hipErrorInvalidValue; \
  }
// M = 256 has batched kernels of its own
#define S2W_BY_M_BATCH(M_, CALL_) \
  switch (M_) {                  \
    case 16: CALL_(16); break;   \
    case 32: CALL_(32); break;   \
    case 64: CALL_(64); break;   \
    case 128: CALL_(128); break; \
    case 512: CALL_(512); break; \
    default: return hipErrorInvalidValue; \
  }

int rows_ga(int M) { return M >= 256 ? 1 : (M == 128 ? 2 : 4); }  // RowFft<M>::GA
static_assert(RowFft<512>::GA == 1 && RowFft<256>::GA == 1 && RowFft<128>::GA == 2 && RowFft<64>::GA == 4 &&
                  RowFft<32>::GA == 4 && RowFft<16>::GA == 4,
              "rows_ga");

}  // namespace

hipError_t launch_rfft_units(const float* in, int64_t in_a, int64_t in_b, int na, int na_out, int nb, int nb_out,
                             float2* out, int64_t oa, int64_t ob, int64_t ol, const Geometry& g, float scale,
                             hipStream_t st) {
  if (na_out == 0 || nb_out == 0) return hipSuccess;
  if (na < 0 || nb < 0 || na_out < na || nb_out < nb || g.nt < 1 || g.nt > g.M || (ob != 1 && ol != 1))
    return hipErrorInvalidValue;
  RfftArgs a{};
  a.in = in;
  a.in_a = in_a;
  a.in_b = in_b;
  a.na = na;
  a.na_out = na_out;
  a.nb = nb;
  a.nb_out = nb_out;
  a.nt = g.nt;
  a.scale = scale;
  a.out = out;
  a.oa = oa;
  a.ob = ob;
  a.ol = ol;
  const int ga = rows_ga(g.M);
  a.nau = (na_out + ga - 1) / ga;
  a.nbu = (nb_out + 15) / 16;
  const int64_t units = (int64_t)a.nau * a.nbu;
  const dim3 grid((unsigned)std::min<int64_t>(units, 256 * 8));
#define S2W_CALL(M_)                                                                                  \
  if (ol == 1)                                                                                        \
    hipLaunchKernelGGL((k_rfft_units<M_, OUT_ROW>), grid, dim3(256), 0, st, a);                       \
  else                                                                                                \
    hipLaunchKernelGGL((k_rfft_units<M_, OUT_RUN>), grid, dim3(256), 0, st, a)
  S2W_BY_M(g.M, S2W_CALL)
#undef S2W_CALL
  return hipGetLastError();
}

// One operator's side of the setup: n grid rows from in[row][c.cols][nt], in `wgs` workgroups at least where there
// are that many units.
static RfftArgs quant_args(const QuantStore& c, bool elastic, const float* in, int n, int64_t row0, uint32_t* mx,
                           const Geometry& g) {
  const int ga = rows_ga(g.M);
  RfftArgs a{};
  a.in = in;
  a.elastic = elastic;
  a.in_a = elastic ? (int64_t)c.cols * g.nt : g.nt;
  a.in_b = elastic ? g.nt : (int64_t)c.cols * g.nt;
  a.na = elastic ? n : c.cols;
  a.na_out = elastic ? n : c.pad;
  a.nb = elastic ? c.cols : n;
  a.nb_out = elastic ? c.pad : n;
  a.nt = g.nt;
  a.scale = 1.f;
  a.out = c.words;
  a.oa = c.w_col;
  a.ol = elastic ? (int64_t)c.row_blocks * (c.pad / 16) * 256 : c.w_slot;
  a.ncp16 = c.pad / 16;
  a.nau = (a.na_out + ga - 1) / ga;
  a.nbu = (a.nb_out + 15) / 16;
  a.mx = mx;
  a.down = c.down;
  a.row0 = row0;
  return a;
}
static void quant_grid(RfftArgs& a, int wgs) {
  const int nloop = a.elastic ? a.nbu : a.nau;
  a.nfix = a.elastic ? a.nau : a.nbu;
  a.splits = std::max(1, std::min(nloop, (wgs + a.nfix - 1) / a.nfix));
  // a multiple of eight, so that every XCD gets a whole share (the rest returns at once)
  a.nwg = (int)(((int64_t)a.nfix * a.splits + 7) / 8 * 8);
}

hipError_t launch_quant_spectra(const QuantStore& G, const QuantStore& F, int64_t nrows, int64_t row0, uint32_t* mx,
                                int64_t mx_words, const Geometry& g, hipStream_t st) {
  if (g.nt < 1 || g.nt > g.M || G.pad < G.cols || F.pad < F.cols || G.pad % 16 || mx_words < 2 * g.M)
    return hipErrorInvalidValue;
  // a pass over the largest |Re|, |Im| of every (grid row, slot), then one that writes the scaled
  // words: the transform is done twice instead of keeping 8-byte spectra between the passes.  Three launches,
  // both operators in one: a few rows are a chain of launches and of one unit's latency
  // (963 + 64 columns x 256 steps, 1, 16 and 512 rows:
  // 19, 43 and 514 us, with eight launches 39, 62 and 544; 16 + 4 x 16, 1 row: 12, with eight 26).
  for (int64_t r0 = 0; r0 < nrows;) {
    const int n = (int)std::min<int64_t>(nrows - r0, mx_words / (2 * g.M));
    hipError_t e = launch_zero_strided(mx, 2 * (int64_t)n * g.M, 1, 1, st);
    if (e != hipSuccess) return e;
    RfftArgs a = quant_args(G, true, G.in + r0 * G.cols * g.nt, n, row0 + r0, mx, g);
    RfftArgs b = quant_args(F, false, F.in + r0 * F.cols * g.nt, n, row0 + r0, mx + (int64_t)n * g.M, g);
    quant_grid(a, 4096);
    quant_grid(b, 4096);
#define S2W_CALL(M_) hipLaunchKernelGGL((k_rfft_max<M_>), dim3((unsigned)(a.nwg + b.nwg)), dim3(256), 0, st, a, b)
    S2W_BY_M(g.M, S2W_CALL)
#undef S2W_CALL
    // Both word passes keep the grid rows too, consecutive ones on one XCD: their 64-byte runs (elastic,
    // row-block-major) or single words (acoustic) are neighbours in the store and meet in one L2
    quant_grid(a, 1536);
    const dim3 grid((unsigned)(a.nwg + b.nwg));
#define S2W_WORDS(M_, G_, F_) hipLaunchKernelGGL((k_rfft_words<M_, G_, F_>), grid, dim3(256), 0, st, a, b)
#define S2W_CALL(M_)                                                  \
  if (G.ht == 1) {                                                    \
    if (F.ht == 1) S2W_WORDS(M_, 1, 1); else S2W_WORDS(M_, 1, 2);     \
  } else {                                                            \
    if (F.ht == 1) S2W_WORDS(M_, 2, 1); else S2W_WORDS(M_, 2, 2);     \
  }
    S2W_BY_M(g.M, S2W_CALL)
#undef S2W_CALL
#undef S2W_WORDS
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    r0 += n;
  }
  return hipSuccess;
}

hipError_t launch_irfft_units(const float2* part, int splits, int64_t p_s, int64_t pa, int64_t pb, int64_t pl, int na,
                              int nb, const float* tau, int64_t tau_l, float* out, int64_t oa, int64_t ob,
                              const Geometry& g, float scale, hipStream_t st) {
  if (na == 0 || nb == 0) return hipSuccess;
  if (na < 0 || nb < 0 || splits < 1 || g.nt < 1 || g.nt > g.M || (pb != 1 && pl != 1)) return hipErrorInvalidValue;
  IrfftArgs a;
  a.part = part;
  a.splits = splits;
  a.p_s = p_s;
  a.pa = pa;
  a.pb = pb;
  a.pl = pl;
  a.na = na;
  a.nb = nb;
  a.tau = tau;
  a.tau_l = tau_l;
  a.out = out;
  a.oa = oa;
  a.ob = ob;
  a.nt = g.nt;
  a.scale = scale;
  const int ga = rows_ga(g.M);
  a.nau = (na + ga - 1) / ga;
  a.nbu = (nb + 15) / 16;
  const dim3 grid((unsigned)std::min<int64_t>((int64_t)a.nau * a.nbu, 256 * 8));
#define S2W_CALL(M_)                                                              \
  if (pl == 1)                                                                    \
    hipLaunchKernelGGL((k_irfft_units<M_, true>), grid, dim3(256), 0, st, a);     \
  else                                                                            \
    hipLaunchKernelGGL((k_irfft_units<M_, false>), grid, dim3(256), 0, st, a)
  S2W_BY_M(g.M, S2W_CALL)
#undef S2W_CALL
  return hipGetLastError();
}

// Up to four rounds of eight loads per thread (512 partials of 4 x 256 slots, eight rounds, stay with the sum
// of their own over more workgroups); a row of 512 slots does not fit the registers of 1,024 threads.
bool sum_irfft_rows_fits(int M, int nparts) { return M <= 256 && (int64_t)nparts * M <= 65536; }

hipError_t launch_sum_irfft_rows(const float2* part, int nparts, int nrows, int nop, float* out, const Geometry& g,
                                 hipStream_t st) {
  if (nparts < 1 || nrows < 1 || nrows > nop || g.nt < 1 || g.nt > g.M || !sum_irfft_rows_fits(g.M, nparts))
    return hipErrorInvalidValue;
#define S2W_CALL(M_)                                                                                             \
  hipLaunchKernelGGL((k_sum_irfft_rows<M_>), dim3((unsigned)nrows), dim3(1024), 0, st, (const v4f*)part, nparts, \
                     (int64_t)nop * (M_ / 2), out, g.nt, 1.0f / (float)g.L)
  switch (g.M) {
    case 16: S2W_CALL(16); break;
    case 32: S2W_CALL(32); break;
    case 64: S2W_CALL(64); break;
    case 128: S2W_CALL(128); break;
    default: S2W_CALL(256); break;
  }
#undef S2W_CALL
  return hipGetLastError();
}

hipError_t launch_mid_units(float2* U, const float* sF, int B, int bp, bool adjoint, bool pack_bf16,
                            const Geometry& g, hipStream_t st, float* cmax, int64_t cmax_floats, int* cmax_groups,
                            const DispOut* disp) {
  if (cmax_groups) *cmax_groups = 0;
  const int ga = rows_ga(g.M);
  const int64_t nbb = (B + 15) / 16, units = (g.ngrid + ga - 1) / ga * nbb;
  if (B < 1 || bp < B || g.nt > g.M || units > 0x7fffffff || (pack_bf16 && cmax) || (adjoint && (pack_bf16 || disp)))
    return hipErrorInvalidValue;
  MidArgs a{};
  a.U = U;
  a.sF = sF;
  a.ngrid = g.ngrid;
  a.B = B;
  a.bp = bp;
  a.nt = g.nt;
  a.mode = g.diff ? (adjoint ? MID_BACKWARD_T : MID_BACKWARD) : MID_NONE;
  a.mscale = (float)(1.0 / ((double)g.L * (g.diff ? (double)g.dt : 1.0)));
  a.cmax = cmax;
  a.nbb = (int)nbb;
  a.units = (int)units;
  if (disp) a.disp = *disp;
  int64_t nblk = std::min<int64_t>(units, 256 * 8);
  if (cmax) {
    // whole groups of nbb workgroups, as many as the partial maxima fit
    const int64_t groups = std::min<int64_t>(std::max<int64_t>(1, nblk / nbb), cmax_floats / ((int64_t)g.M * bp));
    if (groups < 1) return hipErrorInvalidValue;
    nblk = groups * nbb;
    if (cmax_groups) *cmax_groups = (int)groups;
  }
  const dim3 grid((unsigned)nblk);
  const bool d = a.disp.base != nullptr;
#define S2W_MID(M_, P_, D_, C_) hipLaunchKernelGGL((k_mid_units<M_, P_, D_, C_>), grid, dim3(256), 0, st, a)
#define S2W_CALL(M_)                                                     \
  if (pack_bf16) {                                                       \
    if (d) S2W_MID(M_, true, true, false);                               \
    else S2W_MID(M_, true, false, false);                                \
  } else if (cmax) {                                                     \
    if (d) S2W_MID(M_, false, true, true);                               \
    else S2W_MID(M_, false, false, true);                                \
  } else {                                                               \
    if (d) S2W_MID(M_, false, true, false);                              \
    else S2W_MID(M_, false, false, false);                               \
  }
  S2W_BY_M_BATCH(g.M, S2W_CALL)
#undef S2W_CALL
#undef S2W_MID
  return hipGetLastError();
}

hipError_t launch_mid_flat(float2* U, const float* sF, int B, int bp, const Geometry& g, hipStream_t st, float* cmax,
                           int64_t cmax_floats, int* cmax_groups) {
  if ((bp != 8 && bp != 16) || B < 1 || B > bp || g.nt > g.M || !cmax || (int64_t)g.ngrid * bp > (1 << 24))
    return hipErrorInvalidValue;
  const int rows = 16 * rows_ga(g.M);
  MidArgs a{};
  a.U = U;
  a.sF = sF;
  a.ngrid = g.ngrid;
  a.B = B;
  a.bp = bp;
  a.nt = g.nt;
  a.mode = g.diff ? MID_BACKWARD : MID_NONE;
  a.mscale = (float)(1.0 / ((double)g.L * (g.diff ? (double)g.dt : 1.0)));
  a.cmax = cmax;
  a.nbb = 1;
  a.units = (int)(((int64_t)g.ngrid * bp + rows - 1) / rows);
  const int64_t nblk = std::min<int64_t>(std::min<int64_t>(a.units, 256 * 4), cmax_floats / ((int64_t)g.M * bp));
  if (nblk < 1) return hipErrorInvalidValue;
  *cmax_groups = (int)nblk;
#define S2W_CALL(M_) \
  hipLaunchKernelGGL((k_mid_units<M_, false, false, true, true>), dim3((unsigned)nblk), dim3(256), 0, st, a)
  S2W_BY_M_BATCH(g.M, S2W_CALL)
#undef S2W_CALL
  return hipGetLastError();
}

}  // namespace s2w
