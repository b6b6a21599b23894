// Matrix-core GEMM for wide activations (more than 32 rows: batched drafting,
// the training forward over many rows, the table build at model creation):
//   Y[m][n] = sum_k X[m][k] * W[n][k]      (X fp32 [M][K], W [N][K] bf16)
// with the packed weight tiles of the skinny kernel and the same hi + lo bf16
// split of the activations, so both kernels compute to the same precision.
//
// The activations are split once per projection, by the kernel that produces
// them (the RMSNorms, the attention merge, gate/up's own epilogue) or, where
// that leaves fp32 rows, by split_frag_kernel, into two bf16 planes, hi and lo, stored in MFMA fragment order: fragment (row block
// rb, k-step s) is 1 KB, lane l = 16 g + r holding the 8 k values
// 32 s + 8 g .. + 7 of row 16 rb + r.  A fragment is then one coalesced 1 KB
// wave load, exactly like a packed weight fragment, and no arithmetic is left
// between the loads and the products.
//
// A workgroup of 4 waves owns CT weight tiles (16 CT output columns) and 4 TM
// row blocks (64 TM rows); wave w multiplies all CT tiles by row blocks
// TM w .. TM w + TM - 1, hi and lo.  One wave per SIMD, so a wave may hold up to
// 512 registers: the sums, and two iterations (four k-steps) of activation
// fragments, which only this wave uses and which come straight from memory.  The
// weight fragments, used by all four waves, pass through LDS.  The loop takes two
// k-steps an iteration with one barrier, placed between its two halves: the
// fragments of iteration i + 1 are written into the third of three LDS buffers at
// the start of iteration i, so no wave waits for another at an iteration's edge,
// and the weights of iteration i + 3 and the activations of i + 2 are in flight.
//
// What bounds it (gate/up of the 8B shape, 201 MB of weights, K 4096; the old
// kernel, 128 columns x 256 rows with one k-step of prefetch, in brackets, its
// 5 us of activation split included): 64 rows 43 us [107], 128 rows 56 us [108],
// 256 rows 91 us [112], 512 rows 155 us [194]; the weights' floor is 31 us.  From
// 256 rows on it is the chip's power: on random bf16 data a registers-only loop
// of these products reaches 1.8 PFLOP/s (2.3 on zeros), this loop without its
// loads 1.65, and the core clock reads 1.7 to 2.0 GHz while it runs, so every byte
// moved costs time even where it is hidden.  That is why the tile is as large
// as the shape allows: 12 or 13 tiles x 256 rows read 0.23 KB per block product,
// 6 x 256 read 0.40.  Measured and not kept: two groups of four waves splitting K
// (equal or slower by 3%), loads spread between the products (4 to 8% slower),
// three or four iterations in flight (equal), 32x32x16 products (8% slower on
// random data, from the clock).
#include "common.h"
#include "kernels.h"
#include "mfma.h"

#include <algorithm>
#include <type_traits>

namespace dk {

namespace {

constexpr int kWideThreads = 256;
constexpr int kWideBuffers = 3;

DEVI float silu_w(float x) { return x / (1.f + expf(-x)); }

// One thread per (row block, k-step, lane): 8 values of one row, split.
__global__ __launch_bounds__(256) void split_frag_kernel(const float *__restrict__ X, int ldx, int M, int KS,
                                                         u32x4 *__restrict__ Xf, int nrb) {
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (size_t)nrb * KS * 64) return;
  const int lane = (int)(idx & 63);
  const size_t rs = idx >> 6;
  const int s = (int)(rs % KS), rb = (int)(rs / KS);
  const int m = rb * 16 + (lane & 15), k0 = s * 32 + (lane >> 4) * 8;
  float f[8];
  if (m < M) {
    const float4 *p = (const float4 *)(X + (size_t)m * ldx + k0);
    const float4 a = p[0], b = p[1];
    f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w;
    f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) f[e] = 0.f;
  }
  bf16x8 hi, lo;
  split8(f, hi, lo);
  Xf[((size_t)rb * KS + s) * 64 + lane] = __builtin_bit_cast(u32x4, hi);
  Xf[(((size_t)nrb + rb) * KS + s) * 64 + lane] = __builtin_bit_cast(u32x4, lo);
}

// Workgroup order (a 1-D grid, workgroup L on XCD L % 8): the workgroups of
// one (column group, K split) pair u = 8 c + x, one per row group mz, are
// L = 8 (c mgroups + mz) + x: they share L % 8 and are dispatched 8 apart, so the second
// row group finds the weight tiles in its XCD's L2 instead of reading them again.
struct WideMap {
  int groups, ksplit, mgroups;
};
DEVI bool wide_coords(const WideMap &mp, int L, int &grp, int &ky, int &mz) {
  const int x = L & 7, r = L >> 3;
  const int c = r / mp.mgroups;
  mz = r % mp.mgroups;
  const int u = c * 8 + x;
  grp = u % mp.groups;
  ky = u / mp.groups;
  return ky < mp.ksplit;
}

template <int CT, int TM, int EPI>
__global__ __launch_bounds__(kWideThreads) __attribute__((amdgpu_waves_per_eu(1, 1))) void gemm_wide_kernel(
    GemmArgs a, int nrb, WideMap mp) {
  static_assert(EPI != EPI_SWIGLU || CT % 2 == 0, "(gate, up) pairs stay in one workgroup");
  constexpr int WF = 2 * CT;           // weight fragments of an iteration (two k-steps)
  constexpr int WPW = (WF + 3) / 4;    // of them staged by each wave (the last wave may repeat the last one)
  constexpr int RA = TM >= 3 ? 2 : 3;  // weight fragments read from LDS ahead of their products
  constexpr int RING = RA + 1;
  // Splits of a few iterations end soon after their last load: a descriptor
  // without records past the end fetches nothing there (1 us of 12 to 16 on the
  // QKV, O and down shapes at 64 rows).  On long ranges with large tiles plain
  // loads of the last step again are faster (LM head, 13 tiles: 957 against 1011 us).
  constexpr bool kSkipPastEnd = CT <= 10;
  __shared__ u32x4 lds[kWideBuffers * WF][64];

  int grp, ky, mz;
  if (!wide_coords(mp, (int)blockIdx.x, grp, ky, mz)) return;  // past the last pair (workgroup-uniform)
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // the K range in iterations c0 .. c1 - 1 of two k-steps; kend: past its last k-step
  const int KS = a.KS, nch = (KS + 1) / 2;
  const int cps = (nch + a.ksplit - 1) / a.ksplit;
  const int c0 = min(nch, ky * cps), c1 = min(nch, c0 + cps);
  const int nit = c1 - c0, kend = min(KS, 2 * c1);

  // this wave's weight fragments f = WPW * wave + q (tile f % CT, step f / CT of
  // an iteration) and its row blocks in the two planes.  Tiles and blocks past
  // the end are clamped: they only feed outputs that are never stored.
  const u32x4 *wsrc[WPW];
#pragma unroll
  for (int q = 0; q < WPW; ++q) {
    const int f = min(WPW * wave + q, WF - 1);
    const int t = min(grp * CT + f % CT, a.ntiles - 1);
    wsrc[q] = (const u32x4 *)a.P + (size_t)(a.tile0 + t) * KS * 64;
  }
  const u32x4 *xsrc[2 * TM];
#pragma unroll
  for (int f = 0; f < 2 * TM; ++f) {
    const int rb = min((mz * 4 + wave) * TM + f % TM, nrb - 1);
    xsrc[f] = (const u32x4 *)a.xf + ((size_t)(f / TM) * nrb + rb) * KS * 64;
  }

  floatx4 acc[CT][TM];
#pragma unroll
  for (int i = 0; i < CT; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  // fragment s of a tile or row block (KS KB from p); past the end nothing, or the last one again
  auto frag = [&](const u32x4 *p, int s, auto stream) {
    constexpr bool kStream = decltype(stream)::value;
    if constexpr (kSkipPastEnd) {
      const bool in = s < kend;
      const __amdgpu_buffer_rsrc_t r =
          __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, in ? KS * 1024 : 0, 0x00020000);
      const int so = in ? s * 1024 : 0;
      return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, lane * 16, so, kStream ? 2 : 0));
    } else {
      const u32x4 *q = p + (size_t)min(s, kend - 1) * 64 + lane;
      return kStream ? __builtin_nontemporal_load(q) : *q;
    }
  };

  // weights of iterations i + 1 and i + 2 (slot: parity), activations of iterations i and i + 1
  u32x4 wr[2][WPW], xr[2][2][2 * TM], wf[RING];
  auto issue_w = [&](int d, int i) {
#pragma unroll
    for (int q = 0; q < WPW; ++q)
      wr[d][q] = frag(wsrc[q], 2 * (c0 + i) + min(WPW * wave + q, WF - 1) / CT, std::true_type{});
  };
  auto issue_x = [&](int d, int u, int i) {
#pragma unroll
    for (int f = 0; f < 2 * TM; ++f) xr[d][u][f] = frag(xsrc[f], 2 * (c0 + i) + u, std::false_type{});
  };
  auto stage = [&](int d, int b) {
#pragma unroll
    for (int q = 0; q < WPW; ++q) lds[b * WF + min(WPW * wave + q, WF - 1)][lane] = wr[d][q];
  };

  if (nit > 0) {
    // the prologue's loads go out in order (no reordering across the
    // scheduling barriers), so that the loop's waits leave the later ones in flight
    issue_w(0, 0);
    __builtin_amdgcn_sched_barrier(0);
    issue_w(1, 1);
    __builtin_amdgcn_sched_barrier(0);
    issue_x(0, 0, 0);
    issue_x(0, 1, 0);
    __builtin_amdgcn_sched_barrier(0);
    stage(0, 0);
    issue_w(0, 2);
    __builtin_amdgcn_sched_barrier(0);
    issue_x(1, 0, 1);
    issue_x(1, 1, 1);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < RA; ++t) wf[t] = lds[t][lane];
    int b = 0;
    // Iteration i (parity d): writes the weights of iteration i + 1 to the next
    // LDS buffer, multiplies its own out of buffer b and refills the registers
    // it has used.  The next buffer was last read in iteration i - 2, which
    // every wave had left at the barrier of iteration i - 1.  kFull: both
    // k-steps exist and loads are due.
    auto iter = [&](int i, auto par, auto full) {
      constexpr int d = decltype(par)::value;
      constexpr bool kFull = decltype(full)::value;
      const int bn = b == kWideBuffers - 1 ? 0 : b + 1;
      const int nst = kFull || 2 * (c0 + i) + 1 < KS ? 2 : 1;
      stage(d ^ 1, bn);
      if (kFull) issue_w(d ^ 1, i + 3);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if (u < nst) {
#pragma unroll
          for (int c = 0; c < CT; ++c) {
            const int t = u * CT + c;
            if (t + RA < WF) wf[(t + RA) % RING] = lds[b * WF + t + RA][lane];
            __builtin_amdgcn_sched_barrier(0);
            const bf16x8 w = __builtin_bit_cast(bf16x8, wf[t % RING]);
#pragma unroll
            for (int j = 0; j < 2 * TM; ++j)  // hi of every row block, then lo
              acc[c][j % TM] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, __builtin_bit_cast(bf16x8, xr[d][u][j]),
                                                                      acc[c][j % TM], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        if (kFull) issue_x(d, u, i + 2);
        __builtin_amdgcn_sched_barrier(0);
        if (u == 0) __syncthreads();
      }
#pragma unroll
      for (int t = 0; t < RA; ++t) wf[t] = lds[bn * WF + t][lane];
      b = bn;
    };
    constexpr std::integral_constant<int, 0> even{};
    constexpr std::integral_constant<int, 1> odd{};
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    // pairs of whole iterations without a branch (its waits are then exact),
    // then the at most two that are left, whose loads are all in flight
    const int nfull = min(c1, KS / 2) - c0;
    int i = 0;
    for (; i + 2 <= nfull; i += 2) {
      iter(i, even, yes);
      iter(i + 1, odd, yes);
    }
    if (i < nit) iter(i, even, no);
    if (i + 1 < nit) iter(i + 1, odd, no);
  }

  float *Y = a.Y + (size_t)ky * a.ysplit;
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    const int tile = grp * CT + c;
    if (EPI == EPI_SWIGLU) {
      // packed tiles come in (gate, up) pairs; tile parity equals c's parity
      if ((c & 1) || tile + 1 >= a.ntiles) continue;
      const int col = (tile / 2) * 16 + 4 * (lane >> 4);
#pragma unroll
      for (int j = 0; j < TM; ++j) {
        const int m = ((mz * 4 + wave) * TM + j) * 16 + (lane & 15);
        if (m >= a.M) continue;
        float o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = silu_w(acc[c][j][e]) * acc[c + (c + 1 < CT ? 1 : 0)][j][e];
        // rounded to fp32 before the split: the last product is not to be fused into its subtraction
#pragma unroll
        for (int e = 0; e < 4; ++e) __asm__("" : "+v"(o[e]));
        // the next projection's fragment planes: 8 bytes of the lane's 16 (N is a multiple of 32)
        const int KSo = a.N / 32;
        const size_t at =
            (((size_t)(m >> 4) * KSo + (col >> 5)) * 64 + 16 * ((col >> 3) & 3) + (m & 15)) * 2 + ((col >> 2) & 1);
        const float o8[8] = {o[0], o[1], o[2], o[3], 0.f, 0.f, 0.f, 0.f};
        bf16x8 hi, lo;
        split8(o8, hi, lo);
        const u32x4 hu = __builtin_bit_cast(u32x4, hi), lu = __builtin_bit_cast(u32x4, lo);
        uint2 *pf = (uint2 *)a.yf;
        pf[at] = make_uint2(hu[0], hu[1]);
        pf[(size_t)nrb * KSo * 128 + at] = make_uint2(lu[0], lu[1]);
      }
    } else {
      if (tile >= a.ntiles) continue;
      const int n = tile * 16 + 4 * (lane >> 4);
#pragma unroll
      for (int j = 0; j < TM; ++j) {
        const int m = ((mz * 4 + wave) * TM + j) * 16 + (lane & 15);
        if (m >= a.M) continue;
        float *y = Y + (size_t)m * a.ldy + n;
        if (n + 4 <= a.N && (a.ldy & 3) == 0) {
          *(floatx4 *)y = acc[c][j];
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (n + e < a.N) y[e] = acc[c][j][e];
        }
      }
    }
  }
}

template <int CT, int TM>
void launch_tile(int epi, const GemmArgs &a, const GemmPlan &p, int nrb, hipStream_t st) {
  const WideMap mp{p.groups, p.ksplit, p.mgroups};
  const long pairs = (long)p.groups * p.ksplit;
  const dim3 grid((unsigned)((pairs + 7) / 8 * 8 * p.mgroups));
  if constexpr (CT % 2 == 0) {
    if (epi == EPI_SWIGLU) {
      hipLaunchKernelGGL((gemm_wide_kernel<CT, TM, EPI_SWIGLU>), grid, dim3(kWideThreads), 0, st, a, nrb, mp);
      return;
    }
  }
  hipLaunchKernelGGL((gemm_wide_kernel<CT, TM, EPI_STORE>), grid, dim3(kWideThreads), 0, st, a, nrb, mp);
}

template <int CT>
bool launch_cols(int epi, const GemmArgs &a, const GemmPlan &p, int nrb, hipStream_t st) {
  switch (p.MT) {
    case 1: launch_tile<CT, 1>(epi, a, p, nrb, st); return true;
    case 2: launch_tile<CT, 2>(epi, a, p, nrb, st); return true;
    case 3: launch_tile<CT, 3>(epi, a, p, nrb, st); return true;
    case 4: launch_tile<CT, 4>(epi, a, p, nrb, st); return true;
    default: return false;
  }
}

constexpr int kWideCols[] = {4, 6, 8, 10, 12, 13};  // weight tiles per workgroup

}  // namespace

// Cost of the busiest CU in core cycles, fitted to the gate/up shape at
// 64 .. 512 rows and the tiles 6 x 1, 6 x 2, 6 x 4, 12 x 2 and 12 x 4 (measured
// 1076, 1542, 2680, 2790 and 4463 cycles an iteration): an iteration costs its products
// (64 per tile and row block) plus 400 plus 11 per KB loaded; a workgroup
// about 6000 to fill and drain; a K split its partial outputs, written and read
// back.
namespace {
constexpr double kStageCycles = 6000.0;
double iter_cycles(int ct, int tm) { return 64.0 * ct * tm + 400.0 + 11.0 * (2 * ct + 16 * tm); }
double part_cycles(int ks, int M, int ntiles, int n_cu) { return 2.0 * ks * (double)M * ntiles * 16 * 4 / n_cu / 10.0; }
}  // namespace

// A split saves at most the last round of workgroups, and costs its partials: above
// this many rows those of two splits cost more than a round of the largest tile (a tenth
// more, for what the comparison below lets pass).
int gemm_wide_split_rows(int ntiles, int KS, int n_cu) {
  const double round = (KS + 1) / 2 * iter_cycles(13, 4) + kStageCycles;
  return (int)std::min(1e9, 1.1 * round / part_cycles(2, 1, ntiles, n_cu));
}

// The tile (nw: weight tiles, MT: row blocks of a wave) and the K split of least cost.
// SwiGLU, nonlinear in the sum, is never split.
GemmPlan plan_gemm_wide(int ntiles, int KS, int M, int epi, int n_cu, int max_split) {
  GemmPlan p;
  p.wide = 1;
  p.WPT = 1;
  p.kcm = 1;
  p.pgrid = 0;
  const int nrb = (M + 15) / 16, nch = (KS + 1) / 2;
  const int splits = epi == EPI_STORE && M <= gemm_wide_split_rows(ntiles, KS, n_cu) ? max_split : 1;
  double best = 1e300;
  for (int tm = 1; tm <= 4; ++tm) {
    const int mg = (nrb + 4 * tm - 1) / (4 * tm);
    for (int ct : kWideCols) {
      if (epi == EPI_SWIGLU && ct % 2) continue;
      const int groups = (ntiles + ct - 1) / ct;
      const double iter = iter_cycles(ct, tm);
      for (int ks = 1; ks <= splits; ++ks) {
        const int cps = (nch + ks - 1) / ks;
        if (ks > 1 && ((ks - 1) * cps >= nch || cps < 4)) continue;  // an empty or a very short split
        const long wgs = (long)groups * mg * ks;
        const double rounds = (double)((wgs + n_cu - 1) / n_cu);
        const double part = ks > 1 ? part_cycles(ks, M, ntiles, n_cu) : 0.0;
        const double cost = rounds * (cps * iter + kStageCycles) + part;
        if (cost < best * 0.999) {
          best = cost;
          p.nw = ct;
          p.MT = tm;
          p.groups = groups;
          p.mgroups = mg;
          p.ksplit = ks;
        }
      }
    }
  }
  return p;
}

size_t gemm_wide_scratch_bytes(int M, int K) {
  const size_t nrb = (size_t)(M + 15) / 16, KS = (size_t)(K + 31) / 32;
  return 2 * nrb * KS * 1024;
}

bool launch_gemm_wide(int epi, const GemmArgs &a, const GemmPlan &p, hipStream_t st) {
  // the activation loads assume whole k-steps (K = 32 KS) and at least one row;
  // the model's config checks guarantee both for every projection
  if (a.K != a.KS * 32 || a.M <= 0 || (a.X && a.ldx < a.K) || !a.xf) return false;
  if ((epi == EPI_SWIGLU) != (a.yf != nullptr) || (a.yf && a.N % 32)) return false;
  const int nrb = (a.M + 15) / 16;
  const size_t items = (size_t)nrb * a.KS * 64;
  if (a.X)  // not split by its producer
    hipLaunchKernelGGL(split_frag_kernel, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, st, a.X, a.ldx, a.M,
                       a.KS, (u32x4 *)a.xf, nrb);
  switch (p.nw) {
    case 4: return launch_cols<4>(epi, a, p, nrb, st);
    case 6: return launch_cols<6>(epi, a, p, nrb, st);
    case 8: return launch_cols<8>(epi, a, p, nrb, st);
    case 10: return launch_cols<10>(epi, a, p, nrb, st);
    case 12: return launch_cols<12>(epi, a, p, nrb, st);
    case 13: return launch_cols<13>(epi, a, p, nrb, st);
    default: return false;
  }
}

}  // namespace dk
