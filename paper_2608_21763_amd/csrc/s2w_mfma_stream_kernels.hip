// Per-bin products of the batched half-precision path for a few ruptures (at most 32): the
// operator streams once from HBM straight into matrix-core fragments, and nothing else moves much.
//
// Both kernels read operator fragments with plain 16-byte loads in registers, no LDS and no barrier on
// the operator's way, so every wavefront keeps its own loads in flight.  The 256-row tiles of the
// large batches spend their LDS copies, barriers and matrix instructions on 128 or more columns, of
// which 8 ruptures fill 16.  Every output takes the same products in the same order as in those
// tiles, so the results are the same bits.
#include <algorithm>

#include "s2w_half.h"
#include "s2w_internal.h"
#include "s2w_wave.h"

namespace s2w {

// ---------------------------------------------------------------------------------------------
// Elastic product (eq. 1 per bin), as k_gemm_g4:
//   U(g, l, b) = sG[g][l] * sig_down[l][b] * sum_j Gq[g][l][j] (x) Sq[l][j][b]
// at U + g*u_g + l*u_l + b: [l][g][b] where the mid-chain and the acoustic product can take it (a row
// block leaves as one contiguous KB), else [g][l][b].
// A wavefront owns one slot and streams units of 64 grid rows (four 16-row blocks of nks KB each,
// contiguous); operator and activation fragments (k_prep_act; from L2, once per four row blocks) come
// in groups of GRP K steps, the next group (of the same or the next unit) loaded under the products
// of the current one.  The eight wavefronts of a workgroup take eight consecutive slots of the same rows.
//
// Bound by HBM, and by its dislike of mixed traffic: a read stream of 18.9 GB at 6.7 to 7.0 TB/s falls to 5.2
// TB/s when 1 KB is written after every 61 KB read (1.6 % of the traffic), and comes back to 6.5 TB/s when
// the same bytes leave in bursts of 128 KB per CU with non-temporal stores.  So the products of NU units
// collect in 128 KB of LDS and leave together.  963 x 18,880 x 256 slots, bf16, 8 ruptures (18.6 GB):
// 4.15 (256 x 128 tiles) -> 3.43 (products stored row block by row block) -> 2.98 ms.
template <int HT, int H, int NF>
__global__ __launch_bounds__(512) void k_gemm_gs(const uint4* __restrict__ Gq, const float* __restrict__ sG,
                                                 const uint4* __restrict__ Bop, const float* __restrict__ sig_down,
                                                 float2* __restrict__ U, int64_t u_g, int64_t u_l, int ngrid, int M,
                                                 int nks, int B, int bp, int splits) {
  constexpr int MF = 4, GRP = 2, NU = NF == 1 ? 4 : (NF == 2 ? 2 : 1);
  constexpr int UW = 16 * MF * 16 * NF;  // floats of a unit's products
  __shared__ float res[8][NU * UW];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // slot groups of eight; all workgroups of a group on one XCD (group mod 8) where there are that many
  const int ng8 = M >> 3;
  int grp, split;
  if (ng8 >= 8) {
    const int q = blockIdx.x >> 3;
    grp = (blockIdx.x & 7) + 8 * (q / splits);
    split = q % splits;
  } else {
    grp = blockIdx.x % ng8;
    split = blockIdx.x / ng8;
  }
  const int l = 8 * grp + wave;
  const int ng16 = (ngrid + 15) >> 4, nu = (ng16 + MF - 1) / MF;
  const int u0 = (int)((int64_t)nu * split / splits), u1 = (int)((int64_t)nu * (split + 1) / splits);
  if (u0 >= u1) return;
  const int ngrp = (nks + GRP - 1) / GRP;
  const uint4* slot = Gq + (int64_t)l * ng16 * nks * 64 + (lane & 15) * 4 + (lane >> 4);
  const uint4* act = Bop + (int64_t)l * nks * NF * H * 64 + lane;
  struct Group {
    uint4 a[GRP][MF], b[GRP][NF * H];
  };
  int lu = u0, lg = 0;  // next group to load
  auto load = [&](Group& f) {  // steps, rows and units past the end repeat the last one (never used)
    const uint4* row[MF];
#pragma unroll
    for (int a = 0; a < MF; ++a) row[a] = slot + (int64_t)min(MF * lu + a, ng16 - 1) * nks * 64;
#pragma unroll
    for (int i = 0; i < GRP; ++i) {
      const int64_t ks = min(lg * GRP + i, nks - 1);
#pragma unroll
      for (int a = 0; a < MF; ++a) f.a[i][a] = ntload(row[a] + ks * 64);
#pragma unroll
      for (int b = 0; b < NF * H; ++b) f.b[i][b] = act[(ks * NF * H + b) * 64];
    }
    if (++lg == ngrp) {
      lg = 0;
      lu = min(lu + 1, u1 - 1);
    }
  };
  float dn[NF];
#pragma unroll
  for (int b = 0; b < NF; ++b) {
    const int rup = (16 * b + (lane & 15)) >> 1;
    dn[b] = rup < B ? sig_down[(int64_t)l * bp + rup] : 0.f;
  }
  f32x4 acc[MF][NF];
  auto clear = [&]() {
#pragma unroll
    for (int a = 0; a < MF; ++a)
#pragma unroll
      for (int b = 0; b < NF; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  clear();
  int cu = u0, cg = 0;  // group in the products
  auto products = [&](const Group& f) {
#pragma unroll
    for (int i = 0; i < GRP; ++i) {
      if (cg * GRP + i < nks) {
#pragma unroll
        for (int a = 0; a < MF; ++a) {
          const uint4 av = op_word<HT>(f.a[i][a]);
#pragma unroll
          for (int b = 0; b < NF; ++b)
#pragma unroll
            for (int h = 0; h < H; ++h) acc[a][b] = mfma16<kActT<HT>>(av, f.b[i][b * H + h], acc[a][b]);
        }
      }
    }
    if (++cg < ngrp) return;
    const int g0 = 16 * MF * cu;
    float sg[MF][4];
#pragma unroll
    for (int a = 0; a < MF; ++a)
#pragma unroll
      for (int r = 0; r < 4; ++r) sg[a][r] = sG[(int64_t)min(g0 + 16 * a + 4 * (lane >> 4) + r, ngrid - 1) * M + l];
    float* mine = res[wave] + (cu - u0) % NU * UW;
#pragma unroll
    for (int a = 0; a < MF; ++a)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int b = 0; b < NF; ++b)
          mine[(16 * a + 4 * (lane >> 4) + r) * (16 * NF) + 16 * b + (lane & 15)] = acc[a][b][r] * sg[a][r] * dn[b];
    clear();
    cg = 0;
    ++cu;
    const int n = (cu - u0) % NU ? (cu - u0) % NU : NU;  // units held
    if (n < NU && cu < u1) return;
    __syncthreads();  // all wavefronts at the same unit: one burst of the workgroup
    const int gf = 16 * MF * (cu - n), rows = min(16 * MF * n, ngrid - gf);
    const f32x4* from = reinterpret_cast<const f32x4*>(res[wave]);
    for (int i = lane; i < rows * 4 * NF; i += 64) {  // 2 bp = 16 NF floats per row
      const int r = i / (4 * NF), c = i - r * (4 * NF);
      __builtin_nontemporal_store(from[i], reinterpret_cast<f32x4*>(U + (gf + r) * u_g + l * u_l) + c);
    }
    wave_sync();  // other lanes of this wavefront write the next unit's products over what the burst reads
  };
  Group f0, f1;
  load(f0);
  for (int64_t t = (int64_t)(u1 - u0) * ngrp; t > 0; t -= 2) {
    load(f1);
    products(f0);
    if (t == 1) break;
    load(f0);
    products(f1);
  }
}

bool gemm_gs_fits(int hterms, int B) { return hterms * ((2 * B + 15) / 16) <= 6 && B <= 32; }

// One workgroup of eight wavefronts per CU, one round: two and four rounds of smaller workgroups
// (bursts less in step) took 3.07 and 3.17 where this takes 2.98 ms.
static int gs_splits(int ngrid, int M, int ncu) {
  const int nu = (ngrid + 63) / 64, ng8 = M / 8;
  return std::max(1, std::min((ncu + ng8 - 1) / ng8, nu));
}

// Not where slots and rows give eight workgroups or fewer and each has a long chain of products (K steps x columns
// x terms): the tiles share a slot's out over more (whole call, 900 subfaults x 64 rows, bfloat16 products, 16 and 64
// slots: 24 ruptures 111 and 142 us streamed, 82 and 110 in tiles; 8 ruptures 64 and 98, 78 and 102).
bool gemm_gs_pays(int hterms, int B, int ngrid, int M, int nks, int ncu) {
  return gemm_gs_fits(hterms, B) &&
         (M / 8 * gs_splits(ngrid, M, ncu) > 8 || nks * ((2 * B + 15) / 16) * hterms <= 200);
}

template <int HT, int H>
static hipError_t gemm_gs_h(const uint4* Gq, const float* sG, const uint4* Bop, const float* sig_down, float2* U,
                            int64_t u_g, int64_t u_l, int ngrid, int M, int nks, int ncb, int B, int bp, int ncu,
                            hipStream_t st) {
  const int ng8 = M / 8, splits = gs_splits(ngrid, M, ncu);
  const dim3 grid((unsigned)(ng8 * splits));
#define S2W_GS(NF_)                                                                                                  \
  hipLaunchKernelGGL((k_gemm_gs<HT, H, NF_>), grid, dim3(512), 0, st, Gq, sG, Bop, sig_down, U, u_g, u_l, ngrid, \
                     M, nks, B, bp, splits)
  if (ncb == 1) S2W_GS(1);
  else if (ncb == 2) S2W_GS(2);
  else if (ncb == 3) S2W_GS(3);
  else S2W_GS(4);
#undef S2W_GS
  return hipGetLastError();
}

hipError_t launch_gemm_gs(int ht, int hterms, const uint4* Gq, const float* sG, const uint4* Bop, const float* sig_down,
                          float2* U, int64_t u_g, int64_t u_l, int ngrid, int M, int nks, int B, int bp, int ncu, hipStream_t st) {
  const int ncb = (2 * B + 15) / 16;
  if ((M & 7) || B < 1 || bp < B || ngrid < 1 || !gemm_gs_fits(hterms, B) || bp != 8 * ncb) return hipErrorInvalidValue;
  if (ht == 1 && hterms == 2) return gemm_gs_h<1, 2>(Gq, sG, Bop, sig_down, U, u_g, u_l, ngrid, M, nks, ncb, B, bp, ncu, st);
  if (ht == 2 && hterms == 1) return gemm_gs_h<2, 1>(Gq, sG, Bop, sig_down, U, u_g, u_l, ngrid, M, nks, ncb, B, bp, ncu, st);
  if (ht == 3 && hterms == 1) return gemm_gs_h<3, 1>(Gq, sG, Bop, sig_down, U, u_g, u_l, ngrid, M, nks, ncb, B, bp, ncu, st);
  return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------------------------
// Acoustic product (eq. 2 per bin), as k_gemm_fw, float16 products:
//   part[split][l][o][n] = sum_{g in split} Fq[l][o][g] (x) up[l][b] V[l][g][b]
// A wavefront owns 16 observers of one slot and range of grid rows and all ruptures: operator
// fragments (four consecutive grid rows a lane) and complex64 activations come straight into
// registers, GRP K steps of 16 grid rows at a time, the next ones under the products of the current
// ones, and are converted there.  The wavefronts of a workgroup share the activations through L1.
//
// Bound by HBM.  64 observers x 18,880 x 256 slots, bf16, 8 ruptures (1.2 + 0.3 GB): 0.74 -> 0.42 ms.
struct FSArgs {
  const uint32_t* Fq;
  const float2* V;
  const float* up;  // [l][bp]
  float* part;
  int ngrid, ngq, noq, nobs, M, B, bp, nks, nog, splits;
};

template <int HT, int NF>
__global__ __launch_bounds__(256) void k_gemm_fs(const FSArgs p) {
  constexpr int GRP = NF == 1 ? 4 : 2;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int x = blockIdx.x & 7;
  int q = blockIdx.x >> 3;
  const int og = q % p.nog;
  q /= p.nog;
  const int split = q % p.splits, l = x + 8 * (q / p.splits);
  const int o0 = 16 * (og * (int)(blockDim.x >> 6) + wave);
  if (o0 >= p.noq) return;
  const bool dc = (l == 0);
  const int ks0 = (int)((int64_t)p.nks * split / p.splits), ks1 = (int)((int64_t)p.nks * (split + 1) / p.splits);
  const int n = lane & 15, kg = lane >> 4, cim = lane & 1;
  const uint32_t* A = p.Fq + ((int64_t)l * p.noq + o0 + n) * p.ngq + 4 * kg;
  const float2* V = p.V + (int64_t)l * p.ngrid * p.bp;
  int bx[NF];
  float up[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    bx[f] = min(8 * f + (n >> 1), p.bp - 1);
    up[f] = p.up[(int64_t)l * p.bp + bx[f]];
  }
  f32x4 acc[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) acc[f] = f32x4{0.f, 0.f, 0.f, 0.f};
  struct Group {
    uint4 a[GRP];
    float2 v[GRP][NF][4];
  };
  auto load = [&](int ks, Group& r) {  // steps past the range repeat its last (never used)
#pragma unroll
    for (int i = 0; i < GRP; ++i) {
      const int k = min(ks + i, ks1 - 1);
      r.a[i] = ntload(reinterpret_cast<const uint4*>(A + 16 * (int64_t)k));
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float2* row = V + (int64_t)min(16 * k + 4 * kg + e, p.ngrid - 1) * p.bp;
#pragma unroll
        for (int f = 0; f < NF; ++f) r.v[i][f][e] = row[bx[f]];
      }
    }
  };
  auto products = [&](int ks, const Group& r) {
#pragma unroll
    for (int i = 0; i < GRP; ++i) {
      if (ks + i >= ks1) break;
      const uint4 av = op_word<HT>(r.a[i]);
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        uint32_t w[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool ok = 16 * (ks + i) + 4 * kg + e < p.ngrid;
          const float vx = ok ? r.v[i][f][e].x * up[f] : 0.f, vy = ok ? r.v[i][f][e].y * up[f] : 0.f;
          // column re: (x, -y) (DC: (x, 0)); column im: (y, x) (DC: (0, y))
          w[e] = pack_half2<2>(cim ? (dc ? 0.f : vy) : vx, cim ? (dc ? vy : vx) : (dc ? 0.f : -vy));
        }
        acc[f] = mfma16<2>(av, make_uint4(w[0], w[1], w[2], w[3]), acc[f]);
      }
    }
  };
  if (ks0 < ks1) {
    Group g0, g1;
    load(ks0, g0);
    for (int ks = ks0; ks < ks1; ks += 2 * GRP) {
      load(ks + GRP, g1);
      products(ks, g0);
      load(ks + 2 * GRP, g0);
      products(ks + GRP, g1);
    }
  }
  float* ow = p.part + (((int64_t)split * p.M + l) * p.noq) * (2 * (int64_t)p.bp);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int o = o0 + 4 * kg + r;
#pragma unroll
    for (int f = 0; f < NF; ++f)
      if (o < p.nobs && 8 * f + (n >> 1) < p.B) ow[(int64_t)o * (2 * p.bp) + 16 * f + n] = acc[f][r];
  }
}

hipError_t launch_gemm_fs(int ht, const uint32_t* Fq, const float2* V, const float* up, float* part, int ngrid, int ngq,
                          int M, int noq, int nobs, int B, int bp, int splits, hipStream_t st) {
  if ((M & 7) || ngq % 16 || ngq < ngrid || noq % 16 || nobs > noq || B < 1 || B > 16 || B > bp || !up || splits < 1 ||
      (ht != 2 && ht != 3))
    return hipErrorInvalidValue;
  FSArgs a;
  a.Fq = Fq;
  a.V = V;
  a.up = up;
  a.part = part;
  a.ngrid = ngrid;
  a.ngq = ngq;
  a.noq = noq;
  a.nobs = nobs;
  a.M = M;
  a.B = B;
  a.bp = bp;
  a.nks = ngq / 16;
  a.splits = std::min(splits, a.nks);
  const int nob = (nobs + 15) / 16, nw = std::min(4, nob);
  a.nog = (nob + nw - 1) / nw;
  const dim3 grid((unsigned)((int64_t)M * a.nog * a.splits)), blk(64 * nw);
  if (ht == 2) {
    if (B <= 8) hipLaunchKernelGGL((k_gemm_fs<2, 1>), grid, blk, 0, st, a);
    else hipLaunchKernelGGL((k_gemm_fs<2, 2>), grid, blk, 0, st, a);
  } else {
    if (B <= 8) hipLaunchKernelGGL((k_gemm_fs<3, 1>), grid, blk, 0, st, a);
    else hipLaunchKernelGGL((k_gemm_fs<3, 2>), grid, blk, 0, st, a);
  }
  return hipGetLastError();
}

}  // namespace s2w
