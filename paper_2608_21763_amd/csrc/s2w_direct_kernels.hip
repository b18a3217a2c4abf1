// Direct time-domain evaluation of the map, no FFT: each block lower-triangular Toeplitz
// product is computed from its defining sum in the channel form of eq. (4),
//
//   out[r][n] = sum_c sum_{k=0}^{n} A(c, r, k) x_c[n - k],   n < Nt,
//
// on the float32 matrix cores.  This is the paper's direct reference evaluation (Sec. II-C2)
// of eq. (1) (rows r = grid points, channels c = subfaults, A = the elastic blocks), of eq. (2)
// (rows = observers, channels = grid points, A = the acoustic blocks), and, with the time axis
// reversed, of their transposes (the correlations of the adjoint).
//
// As a matrix product, for one channel c the operator row A(c, r, .) (Nt lags) multiplies the
// Toeplitz matrix T_c[k][n] = x_c[n - k] (zero for k > n).  With the time axis cut into blocks
// of 16, the block (kb, nb) of T_c is zero for kb > nb and depends only on d = nb - kb, so one
// channel is a sum over the 136 block pairs kb <= nb (Nt = 256) of 16 x 16 x 16 products: the
// upper triangle of T is never multiplied, except inside the diagonal blocks.
//
// MFMA v_mfma_f32_16x16x4_f32 fragments, lane l = 16 kq + li of 64:
//   A (16 x 4): row li, K entry kq;  B (4 x 16): column li, K entry kq;
//   D (16 x 16): column li, rows 4 kq .. 4 kq + 3.
// K order inside a block of 16 lags: in step q (0..3) lane group kq carries lag 16 kb + 4 kq + q,
// so a lane reads its four operator values of a block as one float4 and the matching Toeplitz
// entries x[16 d + li - 4 kq - q] from the channel's LDS copy.  Lag blocks are taken in pairs
// (m, P - 1 - m), one long and one short, so that every pair has the same number of products over
// the next pair's operator loads.
//
// Bound by the float32 matrix cores (157 TFLOP/s).  240 channels x 9,440 rows x 200 steps (1.06e11
// operations): 1.07 ms while the wait before the products was for the next pair's loads too (they sat
// behind a condition) and neighbouring blocks were paired, 0.95 ms now; two rounds of workgroups on 512
// slots would take 0.72.
#include "s2w_device.h"
#include "s2w_internal.h"

namespace s2w {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kDirectXs = 16 + 512;  // LDS floats per staged channel: 16 zeros, then x[0 .. ntp)

struct DirectArgs {
  const float* A;   // A(c, r, k) at A + c*a_c + r*a_r + k (k < ntp; zeros at k >= nt)
  int64_t a_c, a_r;
  int R;            // rows written (loads clamp below it)
  int nchan;
  const float* X;   // x_c[p] at X + c*x_c + (rev ? nt - 1 - p : p), p < nt
  int64_t x_c;
  int rev;
  float* out;       // out + split*o_s + r*o_r + n, n < nt
  int64_t o_s, o_r;
  int nt, ntp;      // ntp: nt rounded up to 16
  int nrt;          // row tiles (64 * RW rows each)
  int splits;       // channel splits, one partial output each (WC waves' sums added up)
  int nranges;      // ranges of 16 output blocks (Nt > 256 needs two)
};

// Workgroup: four waves in WC groups of 4 / WC; the waves of a group own 16 RW rows each and share
// the staged channel, the groups take channels in turn.  Grid: row tile x channel split x output
// range.  WC > 1 is for few rows (a tile of 64 would leave waves without any): the groups' sums are
// added through LDS at the end, group by group.
template <int RW, int WC>
__global__ __launch_bounds__(256, 2) void k_direct(const DirectArgs p) {
  constexpr int GT = 256 / WC, NX = 512 / GT;  // threads of a group, staged values per thread
  __shared__ float xs_all[2][WC][kDirectXs];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, kq = lane >> 4;
  const int group = wave / (4 / WC), gt = tid % GT;
  int q = blockIdx.x;
  const int range = q % p.nranges;
  q /= p.nranges;
  const int split = q % p.splits;
  const int rt = q / p.splits;
  const int c0 = (int)((int64_t)p.nchan * split / p.splits);
  const int c1 = (int)((int64_t)p.nchan * (split + 1) / p.splits);
  const int nbt = p.ntp >> 4;                 // blocks of 16 output steps
  const int nb0 = 16 * range, nb1 = min(nb0 + 16, nbt);
  const int npairs = (nb1 + 1) >> 1;          // pairs of lag blocks touching the range
  const int r0 = rt * (64 * RW / WC) + (wave % (4 / WC)) * 16 * RW;

  // this lane's operator rows (clamped: rows past R are loaded but never written)
  const float* arow[RW];
#pragma unroll
  for (int rb = 0; rb < RW; ++rb) arow[rb] = p.A + (int64_t)min(r0 + 16 * rb + li, p.R - 1) * p.a_r + 4 * kq;

  f32x4 acc[RW][16];
#pragma unroll
  for (int rb = 0; rb < RW; ++rb)
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[rb][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  for (int i = tid; i < 16 * 2 * WC; i += 256) xs_all[i / 16 % 2][i / 32][i % 16] = 0.f;
  // staged channel values: thread t of a group holds x[t + GT h] (past nt the last one, stored as zero)
  auto load_x = [&](int c, float (&v)[NX]) {
    const float* xc = p.X + (int64_t)c * p.x_c;
#pragma unroll
    for (int h = 0; h < NX; ++h) {
      const int t = min(gt + GT * h, p.nt - 1);
      v[h] = xc[p.rev ? p.nt - 1 - t : t];
    }
  };
  auto store_x = [&](int buf, const float (&v)[NX]) {
#pragma unroll
    for (int h = 0; h < NX; ++h) {
      const int t = gt + GT * h;
      if (t < p.ntp) xs_all[buf][group][16 + t] = t < p.nt ? v[h] : 0.f;
    }
  };
  // lag blocks of pair m: m and nb1 - 1 - m (none when they meet)
  auto lag_of = [&](int m, int h) { return h == 0 ? m : nb1 - 1 - m; };
  auto load_a = [&](int c, int m, float4 (&a)[2][RW]) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int kb = lag_of(m, h);
#pragma unroll
      for (int rb = 0; rb < RW; ++rb)
        a[h][rb] = *reinterpret_cast<const float4*>(arow[rb] + (int64_t)c * p.a_c + 16 * kb);
    }
  };
  auto products = [&](const float* xb, int m, const float4 (&a)[2][RW]) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int kb = lag_of(m, h);
      if (h == 1 && kb == m) continue;
#pragma unroll
      for (int jg = 0; jg < 16; jg += 4) {  // four blocks' Toeplitz entries in flight ahead of their products
        if (nb0 + jg + 3 < kb || nb0 + jg >= nb1) continue;
        float b[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float* t = xb + 16 + 16 * max(nb0 + jg + i - kb, 0) + li - 4 * kq;
#pragma unroll
          for (int k = 0; k < 4; ++k) b[i][k] = t[-k];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int j = jg + i, nb = nb0 + j;
          if (nb < kb || nb >= nb1) continue;
#pragma unroll
          for (int rb = 0; rb < RW; ++rb)
            acc[rb][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[h][rb].x, b[i][0], acc[rb][j], 0, 0, 0);
#pragma unroll
          for (int rb = 0; rb < RW; ++rb)
            acc[rb][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[h][rb].y, b[i][1], acc[rb][j], 0, 0, 0);
#pragma unroll
          for (int rb = 0; rb < RW; ++rb)
            acc[rb][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[h][rb].z, b[i][2], acc[rb][j], 0, 0, 0);
#pragma unroll
          for (int rb = 0; rb < RW; ++rb)
            acc[rb][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[h][rb].w, b[i][3], acc[rb][j], 0, 0, 0);
        }
      }
    }
  };

  if (c0 < c1) {
    float xv[NX];
    const int nstep = (c1 - c0 + WC - 1) / WC;
    const int cl = c1 - 1;  // a group past its last channel loads that one and adds nothing
    load_x(min(c0 + group, cl), xv);
    store_x(0, xv);
    float4 a0[2][RW], a1[2][RW];
    load_a(min(c0 + group, cl), 0, a0);
    __syncthreads();
    int st = 0, m = 0;  // channel step and pair of the current products
    // The next pair's operator loads go out ahead of this pair's products, always: behind a condition
    // the wait before the products would be for them instead of for the pair's own.
    auto turn = [&](const float4 (&cur)[2][RW], float4 (&nxt)[2][RW]) {
      const int cc = c0 + st * WC + group;
      const bool last = m + 1 == npairs;
      if (m == 0) load_x(min(cc + WC, cl), xv);
      load_a(min(last ? cc + WC : cc, cl), last ? 0 : m + 1, nxt);
      if (WC == 1 || cc < c1) products(xs_all[st & 1][group], m, cur);
      m = last ? 0 : m + 1;
      if (last) {
        store_x(++st & 1, xv);
        __syncthreads();
      }
    };
    while (st < nstep) {
      turn(a0, a1);
      if (st == nstep) break;
      turn(a1, a0);
    }
  }
  if constexpr (WC > 1) {  // the first group adds the others' sums, four output blocks at a time
    constexpr int GW = 4 / WC;
    __shared__ f32x4 sum[4 - GW][RW * 4][64];
#pragma unroll
    for (int jg = 0; jg < 16; jg += 4) {
      if (nb0 + jg >= nb1) break;
      __syncthreads();
      if (group > 0)
#pragma unroll
        for (int rb = 0; rb < RW; ++rb)
#pragma unroll
          for (int i = 0; i < 4; ++i) sum[wave - GW][rb * 4 + i][lane] = acc[rb][jg + i];
      __syncthreads();
      if (group == 0)
#pragma unroll
        for (int g = 0; g < WC - 1; ++g)
#pragma unroll
          for (int rb = 0; rb < RW; ++rb)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[rb][jg + i] += sum[g * GW + wave][rb * 4 + i][lane];
    }
    if (group > 0) return;
  }
  float* ow = p.out + (int64_t)split * p.o_s;
#pragma unroll
  for (int rb = 0; rb < RW; ++rb)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = r0 + 16 * rb + 4 * kq + v;
      if (r >= p.R) continue;
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int n = 16 * (nb0 + j) + li;
        if (nb0 + j < nb1 && n < p.nt) ow[(int64_t)r * p.o_r + n] = acc[rb][j][v];
      }
    }
}

// Row tile of a product with R rows: 64 rw rows, or 32 and 16 with the waves in groups by channel
// when R fits: 16 rows, 9,440 channels, 200 steps take 321 us in 64-row tiles, 87 in 16-row ones.
int direct_tile_rows(int rw, int R) { return R <= 16 ? 16 : R <= 32 ? 32 : 64 * rw; }

hipError_t launch_direct(int rw, const float* A, int64_t a_c, int64_t a_r, int R, int nchan, const float* X,
                         int64_t x_c, bool rev, float* out, int64_t o_s, int64_t o_r, int nt, int splits,
                         hipStream_t st) {
  if ((rw != 1 && rw != 2) || nt < 1 || nt > 512 || R < 1 || nchan < 1 || splits < 1 || splits > nchan ||
      (a_c & 3) || (a_r & 3) || ((uintptr_t)A & 15))
    return hipErrorInvalidValue;
  const int rows = direct_tile_rows(rw, R);
  DirectArgs a;
  a.A = A;
  a.a_c = a_c;
  a.a_r = a_r;
  a.R = R;
  a.nchan = nchan;
  a.X = X;
  a.x_c = x_c;
  a.rev = rev ? 1 : 0;
  a.out = out;
  a.o_s = o_s;
  a.o_r = o_r;
  a.nt = nt;
  a.ntp = (nt + 15) / 16 * 16;
  a.nrt = (R + rows - 1) / rows;
  a.splits = splits;
  a.nranges = (a.ntp / 16 + 15) / 16;
  const int64_t blocks = (int64_t)a.nrt * splits * a.nranges;
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks);
  if (rows == 16)
    hipLaunchKernelGGL((k_direct<1, 4>), grid, dim3(256), 0, st, a);
  else if (rows == 32)
    hipLaunchKernelGGL((k_direct<1, 2>), grid, dim3(256), 0, st, a);
  else if (rows == 64)
    hipLaunchKernelGGL((k_direct<1, 1>), grid, dim3(256), 0, st, a);
  else
    hipLaunchKernelGGL((k_direct<2, 1>), grid, dim3(256), 0, st, a);
  return hipGetLastError();
}

// Fixed-order sum over partials with an optional backward difference and time reversal:
//   S(r, p)  = sum_{q < parts} part[q*p_s + r*p_r + (rev ? nt - 1 - p : p)]
//   out[r*o_r + p] = diff ? (S(r, p) - S(r, p - 1)) * scale : S(r, p) * scale,  S(r, -1) = 0.
// Between the two products it forms D_t of the seafloor field (forward) or, on the time-reversed
// correlation, D_t^T (the adjoint); at the end it sums the output partials.  In the forward map
// S is the seafloor displacement m of eq. (1), which `disp` may capture at selected steps.
// A thread sums four consecutive steps (16-byte loads; p_s and p_r are multiples of 4, partial rows
// whole fours).  The partials are dealt to PL threads and their sums added through LDS, in order.
template <int PL>
__global__ __launch_bounds__(256) void k_direct_reduce(const float* __restrict__ part, int parts, int64_t p_s,
                                                       int64_t p_r, int R, int nt, int rev, int diff, float scale,
                                                       float* __restrict__ out, int64_t o_r, DispOut disp) {
  constexpr int IT = 256 / PL;  // fours of steps per workgroup
  const int item = threadIdx.x % IT, pl = threadIdx.x / IT;
  const int n4 = (nt + 3) / 4;
  const int64_t i = (int64_t)blockIdx.x * IT + item;
  const bool on = i < (int64_t)R * n4;
  const int r = on ? (int)(i / n4) : 0, t0 = on ? 4 * (int)(i - (int64_t)r * n4) : 0;
  const float* pr = part + (int64_t)r * p_r + t0;
  const int prev = diff && t0 > 0 ? -1 : 0;  // the step before the four, for the difference
  float s[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
  for (int q = pl; q < parts; q += PL) {
    const float4 v = *reinterpret_cast<const float4*>(pr + (int64_t)q * p_s);
    if (diff) s[0] += pr[(int64_t)q * p_s + prev];
    s[1] += v.x;
    s[2] += v.y;
    s[3] += v.z;
    s[4] += v.w;
  }
  if constexpr (PL > 1) {
    __shared__ float sum[PL][5][IT];
#pragma unroll
    for (int k = 0; k < 5; ++k) sum[pl][k][item] = s[k];
    __syncthreads();
    if (pl > 0) return;
    for (int g = 1; g < PL; ++g)
#pragma unroll
      for (int k = 0; k < 5; ++k) s[k] += sum[g][k][item];
  }
  if (!on) return;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int t = t0 + k, n = rev ? nt - 1 - t : t;
    if (t >= nt) break;
    float v = s[k + 1];
    if (disp.base && r < disp.rows) {
      const int c = disp_col(disp, n);
      if (c >= 0) disp.base[(int64_t)r * disp.row_stride + c] = v * disp.scale;
    }
    if (diff && t > 0) v -= s[k];
    out[(int64_t)r * o_r + n] = v * scale;
  }
}

hipError_t launch_direct_reduce(const float* part, int parts, int64_t p_s, int64_t p_r, int R, int nt, bool rev,
                                bool diff, float scale, float* out, int64_t o_r, hipStream_t st,
                                const DispOut* disp) {
  if (parts < 1 || R < 1 || nt < 1 || (p_s & 3) || (p_r & 3) || p_r < (nt + 3) / 4 * 4 || (rev && diff))
    return hipErrorInvalidValue;
  const int64_t items = (int64_t)R * ((nt + 3) / 4);
  const DispOut d = disp ? *disp : DispOut{};
  // Threads per sum: as many as 860 workgroups allow, a chain of all partials in one thread where the rows fill the
  // chip by themselves.  us with 1 / 4 / 8 / 16 / 32 (one step per thread and all partials in one chain): 16 x 200, 512
  // partials 78 / 23 / 13 / 8 / 5 (122); 300 x 100, 170 partials 29 / 10 / 7 / 7 / 10 (43); 200 x 512, 128 partials 31 / 12 /
  // 10 / 11 / 26 (48); 964 x 374, 32 partials 9 / 9 / 10 / 12 / 40 (12); 9,440 x 200, 13 partials 19 / 20 / 21 / 33 / 194 (35).
  int pl = 32;
  while (pl > 1 && (pl > parts || items * pl > 860 * 256)) pl = pl == 4 ? 1 : pl / 2;
#define S2W_REDUCE(PL_)                                                                                               \
  hipLaunchKernelGGL((k_direct_reduce<PL_>), dim3((unsigned)((items + 256 / PL_ - 1) / (256 / PL_))), dim3(256), 0, st, \
                     part, parts, p_s, p_r, R, nt, rev ? 1 : 0, diff ? 1 : 0, scale, out, o_r, d)
  if (pl == 32) S2W_REDUCE(32);
  else if (pl == 16) S2W_REDUCE(16);
  else if (pl == 8) S2W_REDUCE(8);
  else if (pl == 4) S2W_REDUCE(4);
  else S2W_REDUCE(1);
#undef S2W_REDUCE
  return hipGetLastError();
}

// Time-domain store rows: out[s][k] = in[s][k] for k < nt, 0 for nt <= k < ntp (series s < n).
__global__ __launch_bounds__(256) void k_pad_series(const float* __restrict__ in, int64_t n, int nt, int ntp,
                                                    float* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n * ntp) return;
  const int64_t s = i / ntp;
  const int k = (int)(i % ntp);
  out[i] = k < nt ? in[s * nt + k] : 0.f;
}

hipError_t launch_pad_series(const float* in, int64_t n, int nt, int ntp, float* out, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int64_t items = n * ntp;
  hipLaunchKernelGGL(k_pad_series, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, st, in, n, nt, ntp, out);
  return hipGetLastError();
}

}  // namespace s2w
