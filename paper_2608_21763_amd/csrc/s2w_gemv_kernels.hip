// Per-bin complex matrix-vector products of one BLTT operator for a few inputs (Alg. 2 step 3
// when the batch is too small to feed the matrix cores): the product streams the operator
// store once, so it is bound by HBM bandwidth.
//   yh[b][l][r] = sum_c K[r][l][c] x[b][l][c]      (slot 0: componentwise, the packed real bins)
// K is the store Fs[r][l][c] (complex64, c padded to an even ncp with zeros), x the transformed
// inputs [b][l][c] with the same padding.  One wavefront per (r, l), lanes over c two complex
// values at a time (16-byte loads), a butterfly sum across the wavefront at the end.  A workgroup
// keeps the inputs of one slot and streams the rows of that slot: in registers up to 1,024 columns,
// in LDS while they fit in 60 KB; otherwise the inputs are read through L2.
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

// Sum of 2 NB values over the wavefront; value 2 b + (0 re, 1 im) goes to out[b * b_step + (0, 1)] (floats)
// for b < B.  The pairs of lanes are those of a butterfly
// (32, 16, ... 1), but while a lane holds several values it keeps one half of them and hands the
// other half over, so that 8 values take 10 exchanges instead of 48 (same sums, same order).
template <int NB>
__device__ __forceinline__ void gv_store(float (&re)[NB], float (&im)[NB], int lane, int B, float* out,
                                         int64_t b_step) {
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
  if ((lane & (SHARE - 1)) == 0 && (idx >> 1) < B)
    out[(idx >> 1) * b_step + (idx & 1)] = v[0];
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

// One wavefront per (r, l) (tasks in store order), the inputs read through L2.
template <int NB>
__global__ __launch_bounds__(256) void k_bltt_gemv(const float4* __restrict__ K, const float4* __restrict__ X,
                                                   float2* __restrict__ yh, int nrow, int M, int nc4, int B) {
  const int lane = threadIdx.x & 63;
  const int64_t tasks = (int64_t)nrow * M;
  const int64_t nwave = (int64_t)gridDim.x * 4;
  for (int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); t < tasks; t += nwave) {
    const int r = (int)(t / M), l = (int)(t - (int64_t)r * M);
    const bool dc = (l == 0);
    const float4* a = K + t * nc4;
    float re[NB], im[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) re[b] = im[b] = 0.f;
#pragma unroll 4
    for (int i = lane; i < nc4; i += 64) {
      const gv_f4 kv = __builtin_nontemporal_load(reinterpret_cast<const gv_f4*>(a + i));  // streamed once
      const float4 k = make_float4(kv.x, kv.y, kv.z, kv.w);
#pragma unroll
      for (int b = 0; b < NB; ++b)
        if (b < B) gv_mac(k, X[((int64_t)b * M + l) * nc4 + i], dc, re[b], im[b]);
    }
    gv_store<NB>(re, im, lane, B, reinterpret_cast<float*>(yh + (int64_t)l * nrow + r), 2 * (int64_t)M * nrow);
  }
}

// Workgroup per (slot l, range of rows): the inputs of slot l sit in LDS, and each wavefront
// streams whole store rows (r, l) of its range, one at a time.
template <int NB>
__global__ __launch_bounds__(256) void k_bltt_gemv_lds(const float4* __restrict__ K, const float4* __restrict__ X,
                                                       float2* __restrict__ yh, int nrow, int M, int nc4, int B,
                                                       int nsplit) {
  extern __shared__ float4 xs[];  // [b][i], b < B, i < nc4
  __shared__ float2 res[NB][kGvRows];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l = blockIdx.x % M, split = blockIdx.x / M;
  const bool dc = (l == 0);
  for (int j = threadIdx.x; j < B * nc4; j += 256) {
    const int b = j / nc4, i = j - b * nc4;
    xs[j] = X[((int64_t)b * M + l) * nc4 + i];
  }
  __syncthreads();
  const int r0 = (int)((int64_t)nrow * split / nsplit), r1 = (int)((int64_t)nrow * (split + 1) / nsplit);
  for (int rc = r0; rc < r1; rc += kGvRows) {
    const int re1 = min(rc + kGvRows, r1);
    for (int r = rc + wave; r < re1; r += 4) {
      const float4* a = K + ((int64_t)r * M + l) * nc4;
      float re[NB], im[NB];
#pragma unroll
      for (int b = 0; b < NB; ++b) re[b] = im[b] = 0.f;
#pragma unroll 4
      for (int i = lane; i < nc4; i += 64) {
        const gv_f4 kv = __builtin_nontemporal_load(reinterpret_cast<const gv_f4*>(a + i));  // streamed once
        const float4 k = make_float4(kv.x, kv.y, kv.z, kv.w);
#pragma unroll
        for (int b = 0; b < NB; ++b)
          if (b < B) gv_mac(k, xs[b * nc4 + i], dc, re[b], im[b]);
      }
      gv_store<NB>(re, im, lane, B, reinterpret_cast<float*>(&res[0][r - rc]), 2 * kGvRows);
    }
    gv_flush<NB>(res, B, yh, nrow, M, l, rc, re1 - rc);
  }
}

// As k_bltt_gemv_lds for rows of at most 512 float4 (ncol <= 1024): a whole row (NI float4 per lane) in
// flight, the next one loaded under the sums of the current one, and the inputs of the slot in registers
// (a lane needs the same ones for every row; from LDS they took as long as the row's own bytes).
//
// Bound by HBM.  963 columns x 9,440 rows x 256 slots (18.6 GB), whole call, before and after whole
// butterflies per value, 8-byte stores scattered over the outputs, inputs read from LDS and a copy of the
// next row's registers went: one input 3.25 -> 2.86 ms (6.5 TB/s), two 3.5 -> 2.92, four 5.4 -> 3.06.  Two
// wavefronts per SIMD are enough: with three or four demanded the inputs spill.  Five inputs take the matrix
// cores' path (3.67 ms).
template <int NB, int NI>
__global__ __launch_bounds__(256, 2) void k_bltt_gemv_row(const float4* __restrict__ K, const float4* __restrict__ X,
                                                          float2* __restrict__ yh, int nrow, int M, int nc4, int B,
                                                          int nsplit) {
  __shared__ float2 res[NB][kGvRows];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l = blockIdx.x % M, split = blockIdx.x / M;
  gv_f4 xr[NB][NI];  // zeros past B and nc4
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int t = 0; t < NI; ++t) {
      const int i = lane + 64 * t;
      xr[b][t] = gv_f4{0.f, 0.f, 0.f, 0.f};
      if (b < B && i < nc4) xr[b][t] = reinterpret_cast<const gv_f4*>(X)[((int64_t)b * M + l) * nc4 + i];
    }
  const int r0 = (int)((int64_t)nrow * split / nsplit), r1 = (int)((int64_t)nrow * (split + 1) / nsplit);
  // loads past the range repeat its last row, loads past nc4 its last value (times zero inputs)
  auto load = [&](int r, gv_f4 (&q)[NI]) {
    const gv_f4* a = reinterpret_cast<const gv_f4*>(K + ((int64_t)min(r, r1 - 1) * M + l) * nc4);
#pragma unroll
    for (int t = 0; t < NI; ++t) q[t] = __builtin_nontemporal_load(a + min(lane + 64 * t, nc4 - 1));
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
  auto sums = [&](int rc, int r, const gv_f4 (&q)[NI]) {
    if (r >= r1) return;
    float re[NB], im[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) re[b] = im[b] = 0.f;
    if (l == 0)
      macs(q, std::true_type{}, re, im);
    else
      macs(q, std::false_type{}, re, im);
    gv_store<NB>(re, im, lane, B, reinterpret_cast<float*>(&res[0][r - rc]), 2 * kGvRows);
  };
  static_assert(kGvRows % 8 == 0, "a chunk is whole turns of the loop");
  gv_f4 q0[NI], q1[NI];
  if (r0 < r1) load(r0 + wave, q0);
  for (int rc = r0; rc < r1; rc += kGvRows) {
    const int re1 = min(rc + kGvRows, r1);
    for (int r = rc + wave; r - wave < re1; r += 8) {
      load(r + 4, q1);
      sums(rc, r, q0);
      load(r + 8, q0);
      sums(rc, r + 4, q1);
    }
    gv_flush<NB>(res, B, yh, nrow, M, l, rc, re1 - rc);
  }
}

hipError_t launch_bltt_gemv(const float2* K, const float2* X, float2* yh, int nrow, int M, int ncp, int B, int ncu,
                            hipStream_t st) {
  if (B < 1 || B > 4 || (ncp & 1) || nrow < 1 || M < 1) return hipErrorInvalidValue;
  const int nc4 = ncp / 2;
  const float4* k4 = reinterpret_cast<const float4*>(K);
  const float4* x4 = reinterpret_cast<const float4*>(X);
  const size_t lds = (size_t)B * nc4 * sizeof(float4);
  // inputs of a slot in LDS; enough row ranges per slot for about 16 workgroups per CU
  const int nsplit = (int)std::max<int64_t>(1, std::min<int64_t>((int64_t)ncu * 16 / M, (nrow + 3) / 4));
  if (nc4 <= 512 || lds <= 60 * 1024) {  // 4 KB more hold the results
    const dim3 grid((unsigned)((int64_t)M * nsplit));
    if (nc4 <= 512) {  // whole rows in flight, 2, 3, 4 or 8 float4 per lane (past the row's end a lane sums zeros)
#define S2W_GVR(NB_, NI_)                                                                                              \
  hipLaunchKernelGGL((k_bltt_gemv_row<NB_, NI_>), grid, dim3(256), 0, st, k4, x4, yh, nrow, \
                     M, nc4, B, nsplit)
#define S2W_GVN(NB_)                                                                        \
  if (nc4 <= 128) S2W_GVR(NB_, 2); else if (nc4 <= 192) S2W_GVR(NB_, 3); else if (nc4 <= 256) S2W_GVR(NB_, 4); else S2W_GVR(NB_, 8)
      if (B == 1) {
        S2W_GVN(1);
      } else if (B == 2) {
        S2W_GVN(2);
      } else {
        S2W_GVN(4);
      }
#undef S2W_GVN
#undef S2W_GVR
    } else {
#define S2W_GV2(NB_) \
  hipLaunchKernelGGL((k_bltt_gemv_lds<NB_>), grid, dim3(256), lds, st, k4, x4, yh, nrow, M, nc4, B, nsplit)
      if (B == 1) S2W_GV2(1); else if (B == 2) S2W_GV2(2); else S2W_GV2(4);
#undef S2W_GV2
    }
    return hipGetLastError();
  }
  const int64_t tasks = (int64_t)nrow * M;
  const int64_t blocks = std::min<int64_t>((tasks + 3) / 4, (int64_t)ncu * 16);
  const dim3 grid((unsigned)blocks);
  if (B == 1)
    hipLaunchKernelGGL((k_bltt_gemv<1>), grid, dim3(256), 0, st, k4, x4, yh, nrow, M, nc4, B);
  else if (B == 2)
    hipLaunchKernelGGL((k_bltt_gemv<2>), grid, dim3(256), 0, st, k4, x4, yh, nrow, M, nc4, B);
  else
    hipLaunchKernelGGL((k_bltt_gemv<4>), grid, dim3(256), 0, st, k4, x4, yh, nrow, M, nc4, B);
  return hipGetLastError();
}

}  // namespace s2w
