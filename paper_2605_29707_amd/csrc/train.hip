// Teacher-forced training forward of the Domino head and its loss (Sec. 4.2).
//
// With ground-truth tokens fed to the causal encoder the rollout no longer
// waits on an argmax, so everything after the state recurrence is batched
// over positions:
//   u      u = SiLU(P + Y) for every row (P = W1[:, :d] H from the LM-head
//          pass, Y = W1[:, d:] S from one small GEMM over all states), once,
//          as matrix-core fragments (hi/lo split as in the rollout);
//   ce     L_final = L_base + W2 u for all bs*(B-1) rows at once: W2 streams
//          from HBM once (tile-packed, kept in registers), L_base once, and the
//          corrected logits never leave the chip.  Each workgroup leaves, per
//          row, the (max, sum exp) pair of its vocabulary slice for the base and
//          the final logits, and the workgroup holding the label writes the
//          label's two logits.  A workgroup walks the rows 16 at a time with the
//          next 16's operands in flight and one barrier each.  240 rows of
//          151936 logits: 165 us while every workgroup formed every u itself,
//          loaded after each barrier and used expf; now 153, against 35 us for
//          the bytes (W2 and L_base) and 17 for the products.
//   ce_row a wave per row merges the pairs (CE = log-sum-exp - label logit);
//   loss   one wave: the position-weighted means (weights exp(-k / gamma), k = 0
//          for the first draft position) and the curriculum mix
//          (1 - lambda) L_final + lambda L_base, in a fixed order
//          (deterministic).  As one workgroup for all rows the two took 80 us
//          at 240 rows, now 7 and 5.
#include "common.h"
#include "kernels.h"
#include "mfma.h"

namespace dk {

constexpr int kCeWaves = 8;
constexpr int ce_tpw(int KS) { return KS <= 8 ? 5 : 2; }  // W2 tiles per wave (fragments stay in registers)

// (m, s) <- merge of two (max, sum exp(x - max)) pairs
DEVI void lse_merge(float &m, float &s, float m2, float s2) {
  const float mn = fmaxf(m, m2);
  if (mn == -INFINITY) {
    m = mn;
    s = 0.f;
    return;
  }
  s = s * expf(m - mn) + s2 * expf(m2 - mn);
  m = mn;
}

// u = SiLU(P + Y) as B fragments: [row tile][KS][64][XF], rows past the end a copy of the last one
template <typename WT, int KS>
__global__ __launch_bounds__(256) void train_u_kernel(TrainArgs t) {
  constexpr int EPL = Frag<WT>::EPL, KSTEP = Frag<WT>::KSTEP, XF = XStage<WT>::XF;
  const int it = blockIdx.x * 256 + threadIdx.x;
  if (it >= (t.Mr + 15) / 16 * KS * 64) return;
  const int l = it & 63, s = (it >> 6) % KS, row = min((it >> 6) / KS * 16 + (l & 15), t.Mr - 1);
  const int k0 = s * KSTEP + (l >> 4) * EPL;
  const float *py = t.Y + (size_t)row * t.r + k0;
  const float *pp = t.P + (size_t)row * t.ldp + k0;
  float4 u[EPL / 4];
#pragma unroll
  for (int e = 0; e < EPL / 4; ++e) {
    const float4 a = *(const float4 *)(py + 4 * e), b = *(const float4 *)(pp + 4 * e);
    float4 x = make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
    x.x = x.x / (1.f + expf(-x.x));
    x.y = x.y / (1.f + expf(-x.y));
    x.z = x.z / (1.f + expf(-x.z));
    x.w = x.w / (1.f + expf(-x.w));
    u[e] = x;
  }
  XStage<WT>::put((u32x4 *)t.uf + (size_t)it * XF, u);
}

constexpr float kLog2e = 1.4426950408889634f;

template <typename WT, int KS>
__global__ __launch_bounds__(kCeWaves * 64) void train_ce_kernel(TrainArgs t) {
  constexpr int XF = XStage<WT>::XF;
  constexpr int kTPW = ce_tpw(KS);
  constexpr int kUV = KS * XF / kCeWaves;  // U fragments each wave stages per row tile
  static_assert(KS * XF % kCeWaves == 0, "U fragments must divide over the waves");
  const int V = t.V, Mr = t.Mr;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, cc = lane & 15;
  const int NT = (V + 15) / 16, nrt = (Mr + 15) / 16;
  __shared__ u32x4 us[2][KS * 64 * XF];        // U tile as B fragments
  __shared__ float4 red[2][kCeWaves][16];      // per-wave (mb, sb, mf, sf) of each row
  // L_base of the tile in work, a lane's own values: parked here because the
  // registers hold this wave's W2 fragments and the next tile's loads
  __shared__ float4 lbs[kCeWaves][kTPW][64];

  int tiles[kTPW];
#pragma unroll
  for (int q = 0; q < kTPW; ++q) tiles[q] = (blockIdx.x * kCeWaves + wave) * kTPW + q;
  // this wave's W2 fragments, loaded once and reused for every row tile
  const u32x4 *w2p = (const u32x4 *)t.w2p;
  u32x4 wf[kTPW][KS];
#pragma unroll
  for (int q = 0; q < kTPW; ++q) {
    const int tc = min(tiles[q], NT - 1);
#pragma unroll
    for (int s = 0; s < KS; ++s) wf[q][s] = w2p[((size_t)tc * KS + s) * 64 + lane];
  }
  // The next row tile's operands: its U fragments (element tid + 512 q of the
  // tile) and L_base of this lane's row and the four vocabulary ids of each
  // weight tile (rows are padded to whole tiles: the float4 stays inside the row)
  const u32x4 *uf = (const u32x4 *)t.uf;
  u32x4 ur[kUV];
  float4 lb[kTPW];
  int label = 0;
  auto load = [&](int rt) {
    rt = min(rt, nrt - 1);
#pragma unroll
    for (int q = 0; q < kUV; ++q) ur[q] = uf[(size_t)rt * KS * 64 * XF + q * kCeWaves * 64 + tid];
    const int rowc = min(16 * rt + cc, Mr - 1);
#pragma unroll
    for (int q = 0; q < kTPW; ++q)
      lb[q] = *(const float4 *)(t.Lbase + (size_t)rowc * t.ldl + min(tiles[q], NT - 1) * 16 + 4 * g);
    label = t.labels[rowc];
  };
  // merge of the waves' pairs of row tile rt: eight lanes a row
  auto merge = [&](int rt) {
    if (wave >= 2) return;
    const int m = tid >> 3;
    float4 p = red[rt & 1][tid & 7][m];
#pragma unroll
    for (int o = 1; o <= 4; o <<= 1) {
      const float x = __shfl_xor(p.x, o, 64), y = __shfl_xor(p.y, o, 64);
      const float z = __shfl_xor(p.z, o, 64), w = __shfl_xor(p.w, o, 64);
      lse_merge(p.x, p.y, x, y);
      lse_merge(p.z, p.w, z, w);
    }
    if ((tid & 7) == 0 && 16 * rt + m < Mr)
      *(float4 *)(t.part + ((size_t)(16 * rt + m) * gridDim.x + blockIdx.x) * 4) = p;
  };

  load(0);
  for (int rt = 0; rt < nrt; ++rt) {
    u32x4 *ub = us[rt & 1];
#pragma unroll
    for (int q = 0; q < kUV; ++q) ub[q * kCeWaves * 64 + tid] = ur[q];
#pragma unroll
    for (int q = 0; q < kTPW; ++q) lbs[wave][q][lane] = lb[q];
    const int row = 16 * rt + cc, lab = label;
    // one barrier a tile: U of this one is staged, every wave has left the
    // products of the last one (whose buffer the next one takes) and its pairs
    // are in red
    __syncthreads();
    load(rt + 1);
    if (rt > 0) merge(rt - 1);

    // k-step major: each staged U fragment is read from LDS once for all tiles
    floatx4 acc[kTPW][1];
#pragma unroll
    for (int q = 0; q < kTPW; ++q) acc[q][0] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      u32x4 xf[XF];
#pragma unroll
      for (int f = 0; f < XF; ++f) xf[f] = ub[((size_t)s * 64 + lane) * XF + f];
#pragma unroll
      for (int q = 0; q < kTPW; ++q) Mac2<WT, 1>::step(wf[q][s], xf, acc[q]);
    }

    // lane (g, cc) holds vocabulary ids 16 tile + 4 g + e of row m0 + cc:
    // stores, the label's logits and the maximum first, then the sums (of
    // 2^(x log2 e - m log2 e): one multiply-add and one instruction a term)
    float mb = -INFINITY, mf = -INFINITY;
#pragma unroll
    for (int q = 0; q < kTPW; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int n = tiles[q] * 16 + 4 * g + e;
        const bool ok = row < Mr && n < V;
        const float base = (&lbs[wave][q][lane].x)[e];
        const float fin = base + acc[q][0][e];
        if (t.final_logits && ok) t.final_logits[(size_t)row * V + n] = fin;
        if (ok && n == lab) {
          t.lab[row] = base;
          t.lab[Mr + row] = fin;
        }
        mb = fmaxf(mb, ok ? order_val(base) : -INFINITY);
        acc[q][0][e] = ok ? order_val(fin) : -INFINITY;
        mf = fmaxf(mf, acc[q][0][e]);
      }
    // a slice with no finite value (maximum -inf) keeps its sum at 0; one of +inf is NaN, as inf - inf
    const float rb = mb == -INFINITY ? 0.f : mb * kLog2e, rf = mf == -INFINITY ? 0.f : mf * kLog2e;
    float sb = 0.f, sf = 0.f;
#pragma unroll
    for (int q = 0; q < kTPW; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool ok = row < Mr && tiles[q] * 16 + 4 * g + e < V;
        const float base = ok ? order_val((&lbs[wave][q][lane].x)[e]) : -INFINITY;
        sb += __builtin_amdgcn_exp2f(fmaf(base, kLog2e, -rb));
        sf += __builtin_amdgcn_exp2f(fmaf(acc[q][0][e], kLog2e, -rf));
      }
    // the four lanes of a row; the waves one tile later
#pragma unroll
    for (int o = 16; o <= 32; o <<= 1) {
      const float mb2 = __shfl_xor(mb, o, 64), sb2 = __shfl_xor(sb, o, 64);
      const float mf2 = __shfl_xor(mf, o, 64), sf2 = __shfl_xor(sf, o, 64);
      lse_merge(mb, sb, mb2, sb2);
      lse_merge(mf, sf, mf2, sf2);
    }
    if (g == 0) red[rt & 1][wave][cc] = make_float4(mb, sb, mf, sf);
  }
  __syncthreads();
  merge(nrt - 1);
}

// A wave per row merges the workgroups' pairs (CE = log-sum-exp - label logit).
constexpr int kLoadsPerLane = 8;
__global__ __launch_bounds__(256) void train_ce_row_kernel(TrainArgs t, int GC) {
  const int lane = threadIdx.x & 63, row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= t.Mr) return;
  // the label and its two logits first, so their round trip overlaps the pairs'
  const int label = t.labels[row];
  const float lb = order_val(t.lab[row]), lf = order_val(t.lab[t.Mr + row]);
  float mb = -INFINITY, s_b = 0.f, mf = -INFINITY, s_f = 0.f;
  // kLoadsPerLane pairs per lane in flight together (clamped index, masked
  // after): a load per merge would pay one memory round trip each
  const float4 *pr = (const float4 *)t.part + (size_t)row * GC;
  for (int c0 = 0; c0 < GC; c0 += 64 * kLoadsPerLane) {
    float4 p[kLoadsPerLane];
#pragma unroll
    for (int q = 0; q < kLoadsPerLane; ++q) p[q] = pr[min(c0 + q * 64 + lane, GC - 1)];
#pragma unroll
    for (int q = 0; q < kLoadsPerLane; ++q)
      if (c0 + q * 64 + lane < GC) {
        lse_merge(mb, s_b, p[q].x, p[q].y);
        lse_merge(mf, s_f, p[q].z, p[q].w);
      }
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const float mb2 = __shfl_xor(mb, o, 64), sb2 = __shfl_xor(s_b, o, 64);
    const float mf2 = __shfl_xor(mf, o, 64), sf2 = __shfl_xor(s_f, o, 64);
    lse_merge(mb, s_b, mb2, sb2);
    lse_merge(mf, s_f, mf2, sf2);
  }
  if (lane == 0) {
    const bool ok = label >= 0 && label < t.V;
    if (!ok) raise_error(t.err, DEV_BAD_TOKEN);
    t.ce[row] = ok ? mb + logf(s_b) - lb : NAN;
    t.ce[t.Mr + row] = ok ? mf + logf(s_f) - lf : NAN;
  }
}

// One wave: the position-weighted means and the curriculum mix; lane l takes
// rows l, l + 64, ... and the lanes are added in a fixed order (deterministic).
__global__ __launch_bounds__(64) void train_loss_kernel(TrainArgs t) {
  __shared__ double wk[64];
  const int lane = threadIdx.x;
  if (lane < t.depth) wk[lane] = exp(-(double)lane / (double)t.gamma);  // depth <= 63
  __syncthreads();
  double tb = 0.0, tf = 0.0;
  for (int row = lane; row < t.Mr; row += 64) {
    tb += wk[row % t.depth] * (double)t.ce[row];
    tf += wk[row % t.depth] * (double)t.ce[t.Mr + row];
  }
  for (int o = 32; o >= 1; o >>= 1) {
    tb += __shfl_xor(tb, o, 64);
    tf += __shfl_xor(tf, o, 64);
  }
  if (lane == 0) {
    double wsum = 0.0;
    for (int k = 0; k < t.depth; ++k) wsum += wk[k];
    const double n = wsum * (double)(t.Mr / t.depth);
    const double lb = tb / n, lf = tf / n;
    t.loss[0] = (float)((1.0 - (double)t.lambda) * lf + (double)t.lambda * lb);
    t.loss[1] = (float)lb;
    t.loss[2] = (float)lf;
  }
}

template <typename WT, int KS>
static void launch_ce_t(const TrainArgs &t, int GC, hipStream_t st) {
  const int items = (t.Mr + 15) / 16 * KS * 64;
  hipLaunchKernelGGL((train_u_kernel<WT, KS>), dim3((items + 255) / 256), dim3(256), 0, st, t);
  hipLaunchKernelGGL((train_ce_kernel<WT, KS>), dim3(GC), dim3(kCeWaves * 64), 0, st, t);
}

int train_ce_grid(int V, int r, bool bf16) {
  const int KS = r / kstep_of(bf16);
  const int rows = kCeWaves * ce_tpw(KS) * 16;
  return (V + rows - 1) / rows;
}

hipError_t launch_train_loss(const TrainArgs &t, bool bf16, hipStream_t st) {
  const int KS = t.r / kstep_of(bf16);
  const int GC = train_ce_grid(t.V, t.r, bf16);
  if (bf16) {
    if (KS == 8) launch_ce_t<bf16_t, 8>(t, GC, st);
    else return hipErrorInvalidValue;
  } else {
    if (KS == 16) launch_ce_t<float, 16>(t, GC, st);
    else if (KS == 8) launch_ce_t<float, 8>(t, GC, st);
    else return hipErrorInvalidValue;
  }
  hipLaunchKernelGGL(train_ce_row_kernel, dim3((t.Mr + 3) / 4), dim3(256), 0, st, t, GC);
  hipLaunchKernelGGL(train_loss_kernel, dim3(1), dim3(64), 0, st, t);
  return hipGetLastError();
}

}  // namespace dk
