// Per-bin complex matrix-vector products of one BLTT operator for a few inputs (Alg. 2 step 3
// when the batch is too small to feed the matrix cores): the product streams the operator
// store once, so it is bound by HBM bandwidth.
//   yh[b][l][r] = sum_c K[r][l][c] x[b][l][c]      (slot 0: componentwise, the packed real bins)
// K is the store Fs[r][l][c] (complex64, c padded to an even ncp with zeros), x the transformed
// inputs [b][l][c] with the same padding.  One wavefront per (r, l), lanes over c two complex
// values at a time (16-byte loads), a butterfly sum across the wavefront at the end.  A workgroup
// keeps the inputs of one slot in registers, whole or a chunk of columns at a time, and streams the rows
// of that slot.
#include <algorithm>
#include <type_traits>

#include "s2w_internal.h"

namespace s2w {

typedef float gv_f4 __attribute__((ext_vector_type(4)));

// re + i im += k (x) x over two complex values; slot 0 multiplies componentwise
__device__ __forceinline__ void gv_mac(const float4& k, const float4& x, bool dc, float& re, float& im) {
  if (dc) {
    re += k.x * x.x + k.z * x.z;
    im += k.y * x.y + k.w * x.w;
  } else {
    re += k.x * x.x - k.y * x.y + k.z * x.z - k.w * x.w;
    im += k.x * x.y + k.y * x.x + k.z * x.w + k.w * x.z;
  }
}

// Sum of 2 NB values over the wavefront; value 2 b + (0 re, 1 im) goes to, or unless it is the first is added
// to, out[b * b_step + (0, 1)] (floats) for b < B.  The pairs of lanes are those of a butterfly
// (32, 16, ... 1), but while a lane holds several values it keeps one half of them and hands the
// other half over, so that 8 values take 10 exchanges instead of 48 (same sums, same order).
template <int NB>
__device__ __forceinline__ void gv_store(float (&re)[NB], float (&im)[NB], int lane, int B, float* out,
                                         int64_t b_step, bool first) {
  float v[2 * NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    v[2 * b] = re[b];
    v[2 * b + 1] = im[b];
  }
  int m = 32, idx = 0;
#pragma unroll
  for (int n = NB; n >= 1; n >>= 1, m >>= 1) {  // 2 n values held; the upper lanes keep the upper half
    const bool up = lane & m;
#pragma unroll
    for (int i = 0; i < n; ++i) {
      const float lo = v[i], hi = v[i + n];
      const float keep = up ? hi : lo, give = up ? lo : hi;
      v[i] = keep + __shfl_xor(give, m, 64);
    }
    idx += up ? n : 0;
  }
#pragma unroll
  for (; m >= 1; m >>= 1) v[0] += __shfl_xor(v[0], m, 64);
  // one lane of those that hold value idx = 2 b + (0 re, 1 im)
  constexpr int SHARE = 32 / NB;  // lanes with the same value
  if ((lane & (SHARE - 1)) == 0 && (idx >> 1) < B) {
    float& o = out[(idx >> 1) * b_step + (idx & 1)];
    o = first ? v[0] : o + v[0];
  }
}

// The sums of a workgroup's rows collect in LDS and leave as runs of rows: written one by one (8 bytes
// of a row of M values each, its neighbours by other workgroups) they cost more than their bytes.
constexpr int kGvRows = 128;
template <int NB>
__device__ __forceinline__ void gv_flush(const float2 (&res)[NB][kGvRows], int B, float2* yh, int nrow, int M, int l,
                                         int r0, int n) {
  __syncthreads();
  for (int b = 0; b < B; ++b)
    for (int i = threadIdx.x; i < n; i += 256) {
      typedef float f2 __attribute__((ext_vector_type(2)));
      const float2 v = res[b][i];
      __builtin_nontemporal_store(f2{v.x, v.y}, reinterpret_cast<f2*>(yh + ((int64_t)b * M + l) * nrow + r0 + i));
    }
  __syncthreads();
}

// Workgroup per (slot l, range of rows).  Columns go in chunks of cw <= 64 NI float4 (WHOLE: one chunk), rows in
// chunks of kGvRows: the inputs of a column chunk sit in registers (a lane needs the same ones for every row; from
// LDS they took as long as the row's own bytes), each wavefront streams that part of its rows, the next row
// loaded under the sums of the current one, and the sums of a row's chunks are added in order in LDS.
//
// Bound by HBM.  963 columns x 9,440 rows x 256 slots (18.6 GB), whole call, before and after whole
// butterflies per value, 8-byte stores scattered over the outputs, inputs read from LDS and a copy of the
// next row's registers went: one input 3.25 -> 2.86 ms (6.5 TB/s), two 3.5 -> 2.92, four 5.4 -> 3.06.  Two
// wavefronts per SIMD are enough: with three or four demanded the inputs spill.  Five inputs take the matrix
// cores' path (3.67 ms).  2,100 columns x 20,000 rows x 16 slots (5.4 GB): one input 0.86, four 0.91 ms; with the
// inputs in LDS 0.84 and, past 64 KB of them, read through L2 2.82.
template <int NB, int NI, bool WHOLE>
__global__ __launch_bounds__(256, 2) void k_bltt_gemv_row(const float4* __restrict__ K, const float4* __restrict__ X,
                                                          float2* __restrict__ yh, int nrow, int M, int nc4, int cw,
                                                          int B, int nsplit) {
  __shared__ float2 res[NB][kGvRows];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // row addresses are scalar
  const int l = blockIdx.x % M, split = blockIdx.x / M;
  gv_f4 xr[NB][NI];  // inputs of the column chunk, zeros past B and its end
  auto inputs = [&](int c0, int n) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int t = 0; t < NI; ++t) {
        const int i = lane + 64 * t;
        xr[b][t] = gv_f4{0.f, 0.f, 0.f, 0.f};
        if (b < B && i < n) xr[b][t] = reinterpret_cast<const gv_f4*>(X)[((int64_t)b * M + l) * nc4 + c0 + i];
      }
  };
  if (WHOLE) inputs(0, nc4);  // in flight under the divisions
  const int r0 = (int)((int64_t)nrow * split / nsplit), r1 = (int)((int64_t)nrow * (split + 1) / nsplit);
  // loads past the range repeat its last row, loads past the chunk its last value (times zero inputs)
  auto load = [&](int r, int c0, int n, gv_f4 (&q)[NI]) {
    const gv_f4* a = reinterpret_cast<const gv_f4*>(K + ((int64_t)min(r, r1 - 1) * M + l) * nc4 + c0);
#pragma unroll
    for (int t = 0; t < NI; ++t) q[t] = __builtin_nontemporal_load(a + min(lane + 64 * t, n - 1));
  };
  auto macs = [&](const gv_f4 (&q)[NI], auto dc, float (&re)[NB], float (&im)[NB]) {
#pragma unroll
    for (int t = 0; t < NI; ++t)
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const float4 x = make_float4(xr[b][t].x, xr[b][t].y, xr[b][t].z, xr[b][t].w);
        gv_mac(make_float4(q[t].x, q[t].y, q[t].z, q[t].w), x, dc(), re[b], im[b]);
      }
  };
  auto sums = [&](int rc, int r, bool first, const gv_f4 (&q)[NI]) {
    if (r >= r1) return;
    float re[NB], im[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) re[b] = im[b] = 0.f;
    if (l == 0)
      macs(q, std::true_type{}, re, im);
    else
      macs(q, std::false_type{}, re, im);
    gv_store<NB>(re, im, lane, B, reinterpret_cast<float*>(&res[0][r - rc]), 2 * kGvRows, first);
  };
  static_assert(kGvRows % 8 == 0, "a chunk is whole turns of the loop");
  gv_f4 q0[NI], q1[NI];
  auto rows = [&](int rc, int re1, int c0, int n, bool first) {  // q0 holds this wavefront's first row
    for (int r = rc + wave; r - wave < re1; r += 8) {
      load(r + 4, c0, n, q1);
      sums(rc, r, first, q0);
      load(r + 8, c0, n, q0);
      sums(rc, r + 4, first, q1);
    }
  };
  if (WHOLE && r0 < r1) load(r0 + wave, 0, nc4, q0);
  for (int rc = r0; rc < r1; rc += kGvRows) {
    const int re1 = min(rc + kGvRows, r1);
    if (WHOLE) {
      rows(rc, re1, 0, nc4, true);
    } else {
      for (int c0 = 0; c0 < nc4; c0 += cw) {
        const int n = min(cw, nc4 - c0);
        inputs(c0, n);
        load(rc + wave, c0, n, q0);
        rows(rc, re1, c0, n, c0 == 0);
      }
    }
    gv_flush<NB>(res, B, yh, nrow, M, l, rc, re1 - rc);
  }
}

// NI: float4 per lane (past the chunk's end a lane sums zeros).  Chunks are 257 to 448 float4, whole rows at most 512, or
// 640 of one and two inputs.
template <int NB>
static void gv_launch(dim3 grid, hipStream_t st, bool whole, const float4* K, const float4* X, float2* yh, int nrow,
                      int M, int nc4, int cw, int B, int nsplit) {
  const int ni = (cw + 63) / 64;
#define S2W_GV(NI_, W_) \
  hipLaunchKernelGGL((k_bltt_gemv_row<NB, NI_, W_>), grid, dim3(256), 0, st, K, X, yh, nrow, M, nc4, cw, B, nsplit)
  if (!whole) {
    if (ni <= 5) S2W_GV(5, false);
    else if (ni == 6) S2W_GV(6, false);
    else S2W_GV(7, false);
  } else if (ni <= 2) S2W_GV(2, true);
  else if (ni == 3) S2W_GV(3, true);
  else if (ni == 4) S2W_GV(4, true);
  else if (ni == 5) S2W_GV(5, true);
  else if (ni == 6) S2W_GV(6, true);
  else if (ni == 7) S2W_GV(7, true);
  else if (ni == 8) S2W_GV(8, true);
  else if constexpr (NB <= 2) {
    if (ni == 9) S2W_GV(9, true);
    else S2W_GV(10, true);
  }
#undef S2W_GV
}

hipError_t launch_bltt_gemv(const float2* K, const float2* X, float2* yh, int nrow, int M, int ncp, int B, int ncu,
                            hipStream_t st) {
  if (B < 1 || B > 4 || (ncp & 1) || nrow < 1 || M < 1) return hipErrorInvalidValue;
  const int nc4 = ncp / 2;
  const float4* k4 = reinterpret_cast<const float4*>(K);
  const float4* x4 = reinterpret_cast<const float4*>(X);
  // Up to 512 float4 a row's inputs stay in registers (640 of one and two inputs: 600 x 1,100 x 256 slots 215, in two
  // chunks 229 us); longer rows go in equal chunks of at most 448 (with 512, four inputs spill: 400 x 2,048 x
  // 256 365 against 320 us).
  const int nch = nc4 <= (B <= 2 ? 640 : 512) ? 1 : (nc4 + 447) / 448, cw = (nc4 + nch - 1) / nch;
  // Row ranges per slot: about 16 workgroups per CU, but with several chunks, whose inputs each workgroup reads
  // again for every 128 rows, whole rounds of two per CU with about that many rows each (100 x 8,000 x 256, one and
  // four inputs: 388, 767 us with 16 ranges of 6 rows, 291, 349 with two of 50).
  int64_t splits = (int64_t)ncu * 16 / M;
  if (nch > 1) {
    const int64_t round = std::max(1, 2 * ncu / M);
    splits = round * std::max<int64_t>(1, (nrow + kGvRows / 2 * round) / (kGvRows * round));
  }
  const int nsplit = (int)std::max<int64_t>(1, std::min<int64_t>(splits, (nrow + 3) / 4));
  const dim3 grid((unsigned)((int64_t)M * nsplit));
  if (B == 1)
    gv_launch<1>(grid, st, nch == 1, k4, x4, yh, nrow, M, nc4, cw, B, nsplit);
  else if (B == 2)
    gv_launch<2>(grid, st, nch == 1, k4, x4, yh, nrow, M, nc4, cw, B, nsplit);
  else
    gv_launch<4>(grid, st, nch == 1, k4, x4, yh, nrow, M, nc4, cw, B, nsplit);
  return hipGetLastError();
}

}  // namespace s2w
