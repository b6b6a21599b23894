// Weight-streaming GEMM for one or two row blocks (up to 32 rows: the layers of
// one or two drafting rows and of a chain's verify forward), bf16 weights:
//   Y[m][n] = sum_k X[m][k] * W[n][k]
// over the packed weight tiles and the activations' hi/lo fragment planes of
// the wide kernel (gemm_wide.hip), to the same precision.
//
// Bound by streaming W once.  A workgroup owns CT weight tiles and a K range; its
// NW waves take every NW-th k-step each, all CT tiles of it, so a k-step's
// activation fragments (2 KB a row block) are loaded by exactly one wave of the
// workgroup, straight into registers beside the CT weight fragments, D k-steps
// ahead.  There is no LDS and no barrier until the waves' sums meet at the end
// (added in wave order).  The skinny kernel (gemm.hip) stages fp32 activations
// through LDS, split by every workgroup, with a barrier per chunk: in a step of 16
// rows of the 8B shape gate/up takes 33.5 us here against 36.9 there (a bare read of its
// weights in this launch shape 31.0), QKV 10.3 against 12.0, down 18.5 against 19.4.
//
// O ends with the residual update (EPI_RESID): one tile over all of K per
// workgroup, so no sum crosses workgroups (10.4 us with the epilogue, against 13.1
// for K splits that meet behind a ticket).  The RMSNorm that follows is deferred: the epilogue
// leaves x times the norm's gain as the next projection's planes and each
// tile's row sums of squares, and gate/up scales its sums by
// rsqrt(sum / d + eps): the norm factor of a row is one number.  Down is three
// times longer and keeps its K split (4 splits 18.5 us, 2 of the same tiles 26.8); the next
// RMSNorm's launch adds its partials.
#include "common.h"
#include "kernels.h"
#include "mfma.h"

#include <algorithm>

namespace dk {

namespace {

DEVI float silu_r(float x) { return x / (1.f + expf(-x)); }

// hi and lo bf16 parts of four values as 8 bytes each
DEVI void split_quad(const float (&v)[4], uint2 &hi, uint2 &lo) {
  const float f[8] = {v[0], v[1], v[2], v[3], 0.f, 0.f, 0.f, 0.f};
  bf16x8 h, l;
  split8(f, h, l);
  const u32x4 hu = __builtin_bit_cast(u32x4, h), lu = __builtin_bit_cast(u32x4, l);
  hi = make_uint2(hu[0], hu[1]);
  lo = make_uint2(lu[0], lu[1]);
}

// 8-byte place of columns k .. k + 3 of row m in a plane of KS k-steps
DEVI size_t quad_at(int m, int k, int KS) {
  return (((size_t)(m >> 4) * KS + (k >> 5)) * 64 + 16 * ((k >> 3) & 3) + (m & 15)) * 2 + ((k >> 2) & 1);
}

template <int CT, int MT, int NW, int D, int EPI>
__global__ __launch_bounds__(NW * 64) void gemm_rows_kernel(GemmArgs a, int nrb) {
  static_assert(EPI != EPI_SWIGLU || CT % 2 == 0, "(gate, up) pairs stay in one workgroup");
  constexpr int T = CT * MT;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, cc = lane & 15;
  const int grp = blockIdx.x, ky = blockIdx.y, KS = a.KS;
  const int spw = (KS + a.ksplit - 1) / a.ksplit;
  const int s0 = min(KS, ky * spw), s1 = min(KS, s0 + spw);
  __shared__ floatx4 red[NW][T][64];
  __shared__ float rs_part[EPI == EPI_SWIGLU ? NW * 4 : 1][MT * 16];

  // tiles and row blocks past the end are clamped: they only feed outputs that are never stored
  const u32x4 *wsrc[CT], *xsrc[2 * MT];
#pragma unroll
  for (int c = 0; c < CT; ++c)
    wsrc[c] = (const u32x4 *)a.P + (size_t)(a.tile0 + min(grp * CT + c, a.ntiles - 1)) * KS * 64;
#pragma unroll
  for (int f = 0; f < 2 * MT; ++f)
    xsrc[f] = (const u32x4 *)a.xf + ((size_t)(f / MT) * nrb + min(f % MT, nrb - 1)) * KS * 64;

  // fragment of k-step s; past the range nothing is fetched (a descriptor without records) and zeros return
  auto frag = [&](const u32x4 *p, int s, int aux) {
    const bool in = s < s1;
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, in ? KS * 1024 : 0, 0x00020000);
    const int so = in ? s * 1024 : 0;
    return __builtin_bit_cast(u32x4, aux ? __builtin_amdgcn_raw_buffer_load_b128(r, lane * 16, so, 2)
                                         : __builtin_amdgcn_raw_buffer_load_b128(r, lane * 16, so, 0));
  };
  u32x4 wr[D][CT], xr[D][2 * MT];
  auto load = [&](int d, int i) {  // this wave's i-th k-step
    const int s = s0 + i * NW + wave;
#pragma unroll
    for (int f = 0; f < 2 * MT; ++f) xr[d][f] = frag(xsrc[f], s, 0);
#pragma unroll
    for (int c = 0; c < CT; ++c) wr[d][c] = frag(wsrc[c], s, 2);  // non-temporal
  };
  const int n = (s1 - s0 + NW - 1) / NW;  // uniform over the waves
#pragma unroll
  for (int d = 0; d < D; ++d) {
    load(d, d);
    __builtin_amdgcn_sched_barrier(0);
  }

  // what the epilogue needs besides the sums, in flight behind the first k-steps
  const int n0 = grp * CT * 16 + 4 * g;  // EPI_RESID: CT = 1, wave mt finishes rows 16 mt ..
  const int rm = min(wave * 16 + cc, a.M - 1);
  float4 res = make_float4(0.f, 0.f, 0.f, 0.f);
  bf16_t gain[4] = {};
  if constexpr (EPI == EPI_RESID) {
    if (wave < MT && grp < a.ntiles) {
      res = *(const float4 *)(a.res_in + (size_t)rm * a.ldy + n0);
#pragma unroll
      for (int e = 0; e < 4; ++e) gain[e] = ((const bf16_t *)a.res_gain)[n0 + e];
    }
  }
  if constexpr (EPI == EPI_SWIGLU) {  // row sums of squares: thread (q, m) adds the groups q, q + 4 NW, ...
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int m = min(mt * 16 + (tid & 15), a.M - 1);
      float t = 0.f;
#pragma unroll 8
      for (int q = tid >> 4; q < a.rs_ng; q += NW * 4) t += a.rs_ssq[(size_t)q * a.M + m];
      rs_part[tid >> 4][mt * 16 + (tid & 15)] = t;
    }
  }

  floatx4 acc[CT][MT];
#pragma unroll
  for (int c = 0; c < CT; ++c)
#pragma unroll
    for (int m = 0; m < MT; ++m) acc[c][m] = floatx4{0.f, 0.f, 0.f, 0.f};
  auto step = [&](int d, int i, bool more) {
#pragma unroll
    for (int m = 0; m < 2 * MT; ++m)  // hi of every row block, then lo
#pragma unroll
      for (int c = 0; c < CT; ++c)
        acc[c][m % MT] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wr[d][c]),
                                                                __builtin_bit_cast(bf16x8, xr[d][m]), acc[c][m % MT],
                                                                0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    if (more) load(d, i + D);
    __builtin_amdgcn_sched_barrier(0);
  };
  int i = 0;
  for (; i + 2 * D <= n; i += D)
#pragma unroll
    for (int d = 0; d < D; ++d) step(d, i + d, true);
  // fewer than 2 D k-steps are left (zeros past the end)
  for (; i < n; i += D)
#pragma unroll
    for (int d = 0; d < D; ++d) step(d, i + d, i + D < n);

#pragma unroll
  for (int c = 0; c < CT; ++c)
#pragma unroll
    for (int m = 0; m < MT; ++m) red[wave][c * MT + m][lane] = acc[c][m];
  __syncthreads();
  auto total = [&](int t) {
    floatx4 v = red[0][t][lane];
#pragma unroll
    for (int q = 1; q < NW; ++q) v += red[q][t][lane];
    return v;
  };

  if constexpr (EPI == EPI_STORE) {
    for (int t = wave; t < T; t += NW) {
      const int tile = grp * CT + t / MT, m = (t % MT) * 16 + cc;
      if (tile >= a.ntiles || m >= a.M) continue;
      const floatx4 v = total(t);
      const int col = tile * 16 + 4 * g;
      float *y = a.Y + (size_t)ky * a.ysplit + (size_t)m * a.ldy + col;
      if (col + 4 <= a.N && (a.ldy & 3) == 0) {
        *(floatx4 *)y = v;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (col + e < a.N) y[e] = v[e];
      }
    }
  } else if constexpr (EPI == EPI_SWIGLU) {
    for (int t = wave; t < T / 2; t += NW) {  // pair t / MT, row block t % MT
      const int tile = grp * CT + t / MT * 2, m = (t % MT) * 16 + cc;
      if (tile + 1 >= a.ntiles || m >= a.M) continue;
      const floatx4 vg = total((t / MT * 2) * MT + t % MT), vu = total((t / MT * 2 + 1) * MT + t % MT);
      float ss = 0.f;
#pragma unroll
      for (int q = 0; q < NW * 4; ++q) ss += rs_part[q][m];
      const float rs = 1.0f / sqrtf(ss / (float)a.rs_d + a.rs_eps);
      float o[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = silu_r(vg[e] * rs) * (vu[e] * rs);
      uint2 hi, lo;
      split_quad(o, hi, lo);
      const int KSo = a.N / 32;
      const size_t at = quad_at(m, tile * 8 + 4 * g, KSo);
      ((uint2 *)a.yf)[at] = hi;
      ((uint2 *)a.yf)[(size_t)nrb * KSo * 128 + at] = lo;
    }
  } else {  // EPI_RESID
    if (wave >= MT || grp >= a.ntiles) return;
    const floatx4 v = total(wave);
    const int m = wave * 16 + cc;
    const float x[4] = {res.x + v[0], res.y + v[1], res.z + v[2], res.w + v[3]};
    float ss = 0.f, xg[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      ss = fmaf(x[e], x[e], ss);
      xg[e] = x[e] * to_f32(gain[e]);
    }
    ss += __shfl_xor(ss, 16, 64);
    ss += __shfl_xor(ss, 32, 64);
    if (m >= a.M) return;
    *(float4 *)(a.res_out + (size_t)m * a.ldy + n0) = make_float4(x[0], x[1], x[2], x[3]);
    uint2 hi, lo;
    split_quad(xg, hi, lo);
    const int KSo = a.N / 32;
    const size_t at = quad_at(m, n0, KSo);
    ((uint2 *)a.yf)[at] = hi;
    ((uint2 *)a.yf)[(size_t)nrb * KSo * 128 + at] = lo;
    if (g == 0) a.res_ssq[(size_t)grp * a.M + m] = ss;
  }
}

template <int CT, int MT, int NW, int D>
bool launch_ct(int epi, const GemmArgs &a, const GemmPlan &p, int nrb, hipStream_t st) {
  const dim3 grid(p.groups, p.ksplit), block(NW * 64);
  if (epi == EPI_STORE) hipLaunchKernelGGL((gemm_rows_kernel<CT, MT, NW, D, EPI_STORE>), grid, block, 0, st, a, nrb);
  else if constexpr (CT == 1) {
    if (epi != EPI_RESID) return false;
    hipLaunchKernelGGL((gemm_rows_kernel<CT, MT, NW, D, EPI_RESID>), grid, block, 0, st, a, nrb);
  } else if constexpr (CT % 2 == 0) {
    if (epi != EPI_SWIGLU) return false;
    hipLaunchKernelGGL((gemm_rows_kernel<CT, MT, NW, D, EPI_SWIGLU>), grid, block, 0, st, a, nrb);
  } else {
    return false;
  }
  return true;
}

// k-steps in flight per wave: by registers, and none of the tile sizes gained from more
template <int MT>
bool launch_mt(int epi, const GemmArgs &a, const GemmPlan &p, int nrb, hipStream_t st) {
  switch (p.nw) {
    case 1: return launch_ct<1, MT, 8, 8>(epi, a, p, nrb, st);
    case 2: return launch_ct<2, MT, 8, 6>(epi, a, p, nrb, st);
    case 3: return launch_ct<3, MT, 8, 4>(epi, a, p, nrb, st);
    case 4: return launch_ct<4, MT, 8, 4>(epi, a, p, nrb, st);
    case 6: return launch_ct<6, MT, 4, 4>(epi, a, p, nrb, st);
    case 8: return launch_ct<8, MT, 4, 3>(epi, a, p, nrb, st);
    default: return false;
  }
}

}  // namespace

// Tiles per workgroup (nw) and K split: the least traffic of the busiest CU,
// its workgroups' weights and activations (every k-step 1 KB a tile and 2 KB a
// row block) and the split's partial outputs, written and read back, which count
// sixteenfold (they come after the last product, and a consumer waits for them:
// QKV 3 tiles x 2 splits 10.3 us, 6 x 4 11.0, 3 unsplit 15.1; down 4 x 4 18.5 and 5.2 for
// the RMSNorm that adds its partials, 8 x 8 19.0 and 6.9).  On the
// 8B shape at 16 rows it takes 6 tiles for gate/up, 3 x 2 splits for QKV and 4 x
// 4 for down, each the fastest of those measured.  EPI_RESID: one tile, no split.
GemmPlan plan_gemm_rows(int ntiles, int KS, int M, int epi, int n_cu, int max_split) {
  GemmPlan p;
  p.rows = 1;
  p.MT = M <= 16 ? 1 : 2;
  p.WPT = 1;
  p.mgroups = 1;
  p.kcm = 1;
  p.pgrid = 0;
  p.ksplit = 1;
  p.nw = 1;
  p.groups = ntiles;
  if (epi == EPI_RESID) return p;
  double best = 1e300;
  for (int ct : {1, 2, 3, 4, 6, 8}) {
    if (epi == EPI_SWIGLU && ct % 2) continue;
    const int groups = (ntiles + ct - 1) / ct;
    for (int ks = 1; ks <= (epi == EPI_STORE ? std::min(max_split, 8) : 1); ++ks) {
      const int spw = (KS + ks - 1) / ks;
      if (ks > 1 && ((ks - 1) * spw >= KS || spw < 16)) continue;  // an empty or a very short split
      const long wgs = (long)groups * ks;
      const double part = ks > 1 ? 16 * 2.0 * ks * (double)M * ntiles * 16 * 4 / 1024.0 / n_cu : 0.0;
      const double cost = (double)((wgs + n_cu - 1) / n_cu) * spw * (ct + 2 * p.MT) + part;
      if (cost < best * 0.999) {
        best = cost;
        p.nw = ct;
        p.groups = groups;
        p.ksplit = ks;
      }
    }
  }
  return p;
}

bool launch_gemm_rows(int epi, const GemmArgs &a, const GemmPlan &p, hipStream_t st) {
  // whole k-steps, one or two row blocks, planes for the input (and the output where it is planes)
  if (a.K != a.KS * 32 || a.M <= 0 || a.M > 16 * p.MT || p.MT > 2 || !a.xf || a.X) return false;
  if (epi != EPI_STORE && (!a.yf || a.N % 32)) return false;
  if (epi == EPI_SWIGLU && (!a.rs_ssq || a.rs_ng <= 0 || a.rs_d <= 0)) return false;
  if (epi == EPI_RESID && (!a.res_in || !a.res_out || !a.res_ssq || !a.res_gain || a.ldy % 4 || a.N != a.ntiles * 16))
    return false;
  const int nrb = (a.M + 15) / 16;
  return p.MT == 1 ? launch_mt<1>(epi, a, p, nrb, st) : launch_mt<2>(epi, a, p, nrb, st);
}

}  // namespace dk
