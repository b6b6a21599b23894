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
//          corrected logits never leave the chip.  Each wave leaves, per
//          row, the (max, sum exp) pair of its vocabulary slice for the base and
//          the final logits, and the wave holding the label writes the
//          label's two logits.  A workgroup walks the rows 16 at a time with the
//          next 16's operands loaded during the products and one barrier each.  240
//          rows of 151936 logits: 165 us while every workgroup formed every u itself,
//          loaded after each barrier and used expf, 120 while the waves' pairs
//          were merged through LDS, 102 while the L_base values in flight were structs,
//          which the compiler kept in private memory and so waited for at once; now 94, against
//          35 us for the bytes (W2 and L_base) and 17 for the products.  Two waves a
//          SIMD, 256 registers each, are not quite enough: one of the five L_base
//          fragments and some addresses spill (32 bytes of scratch a lane), and its store waits for
//          the loads, so that only the products hide them and the exponentials do not.
//   ce_row a workgroup per row merges the pairs (CE = log-sum-exp - label logit);
//   loss   one wave: the position-weighted means (weights exp(-k / gamma), k = 0
//          for the first draft position) and the curriculum mix
//          (1 - lambda) L_final + lambda L_base, in a fixed order
//          (deterministic).  As one workgroup for all rows the two took 80 us
//          at 240 rows, now 8 and 5.
#include <type_traits>

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

// FINAL: the corrected logits are also written out
template <typename WT, int KS, bool FINAL>
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
  // L_base of the tile in work, a lane's own values: parked here because the
  // registers hold this wave's W2 fragments and the next tile's loads
  __shared__ floatx4 lbs[kCeWaves][kTPW][64];

  int tiles[kTPW];
#pragma unroll
  for (int q = 0; q < kTPW; ++q) tiles[q] = (blockIdx.x * kCeWaves + wave) * kTPW + q;
  // this wave's W2 fragments, loaded once and reused for every row tile: the
  // last of five tiles in LDS, because with all of them in registers values of the
  // products spill, and a spill's reload waits for every load issued before it, the next
  // rows' operands included (153 us instead of 120)
  constexpr int kReg = kTPW > 4 ? 4 : kTPW;
  extern __shared__ __align__(16) unsigned char smem[];
  u32x4 *w2s = (u32x4 *)smem + (size_t)wave * KS * 64 + lane;  // [s * 64], kTPW > kReg
  const u32x4 *w2p = (const u32x4 *)t.w2p;
  u32x4 wf[kReg][KS];
#pragma unroll
  for (int q = 0; q < kTPW; ++q) {
    const int tc = min(tiles[q], NT - 1);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const u32x4 w = w2p[((size_t)tc * KS + s) * 64 + lane];
      if (q < kReg) wf[q < kReg ? q : 0][s] = w;
      else w2s[s * 64] = w;
    }
  }
  // The next row tile's operands: its U fragments (element tid + 512 q of the
  // tile) and L_base of this lane's row and the four vocabulary ids of each
  // weight tile (rows are padded to whole tiles: the float4 stays inside the row)
  const u32x4 *uf = (const u32x4 *)t.uf;
  u32x4 ur[kUV];
  floatx4 lb[kTPW];
  int label = 0;
  auto load = [&](int rt) {
    rt = min(rt, nrt - 1);
#pragma unroll
    for (int q = 0; q < kUV; ++q) ur[q] = uf[(size_t)rt * KS * 64 * XF + q * kCeWaves * 64 + tid];
    const int rowc = min(16 * rt + cc, Mr - 1);
#pragma unroll
    for (int q = 0; q < kTPW; ++q)
      lb[q] = *(const floatx4 *)(t.Lbase + (size_t)rowc * t.ldl + min(tiles[q], NT - 1) * 16 + 4 * g);
    label = t.labels[rowc];
  };
  load(0);
  for (int rt = 0; rt < nrt; ++rt) {
    u32x4 *ub = us[rt & 1];
#pragma unroll
    for (int q = 0; q < kUV; ++q) ub[q * kCeWaves * 64 + tid] = ur[q];
#pragma unroll
    for (int q = 0; q < kTPW; ++q) lbs[wave][q][lane] = lb[q];
    const int row = 16 * rt + cc, lab = label;
    // one barrier a tile: U of this one is staged, and every wave has left the
    // products of the last one, whose buffer the next one takes
    __syncthreads();
    load(rt + 1);

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
      for (int q = 0; q < kTPW; ++q) {
        const u32x4 w = q < kReg ? wf[q < kReg ? q : 0][s] : w2s[s * 64];
        Mac2<WT, 1>::step(w, xf, acc[q]);
      }
    }

    // lane (g, cc) holds vocabulary ids 16 tile + 4 g + e of row 16 rt + cc: the
    // label's logits (by selection, one branch at the end) and the maximum first,
    // then the sums (the difference first, so that the largest term is 1 exactly
    // and a row of the type's lowest value stays finite).  Ids past V are tested only in a wave that has some;
    // rows past the end only feed pairs that are never stored.
    float mb = -INFINITY, mf = -INFINITY, sb = 0.f, sf = 0.f;
    float lab_b = 0.f, lab_f = 0.f;
    auto reduce = [&](auto masked) {
      constexpr bool kMasked = decltype(masked)::value;
#pragma unroll
      for (int q = 0; q < kTPW; ++q) {
        const floatx4 l4 = lbs[wave][q][lane];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int n = tiles[q] * 16 + 4 * g + e;
          const bool ok = !kMasked || n < V;
          const float base = l4[e];
          const float fin = base + acc[q][0][e];
          if (FINAL && ok && row < Mr) t.final_logits[(size_t)row * V + n] = fin;
          lab_b = n == lab ? base : lab_b;
          lab_f = n == lab ? fin : lab_f;
          mb = fmaxf(mb, ok ? base : -INFINITY);  // (a NaN drops out: it counts as -inf)
          acc[q][0][e] = ok ? order_val(fin) : -INFINITY;
          mf = fmaxf(mf, acc[q][0][e]);
        }
      }
      // the row's maximum over its four lanes, so that their sums add
#pragma unroll
      for (int o = 16; o <= 32; o <<= 1) {
        mb = fmaxf(mb, __shfl_xor(mb, o, 64));
        mf = fmaxf(mf, __shfl_xor(mf, o, 64));
      }
      // a slice with no finite value (maximum -inf) keeps its sum at 0; one of +inf is NaN, as inf - inf
      const float rb = mb == -INFINITY ? 0.f : mb, rf = mf == -INFINITY ? 0.f : mf;
#pragma unroll
      for (int q = 0; q < kTPW; ++q) {
        const floatx4 l4 = lbs[wave][q][lane];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool ok = !kMasked || tiles[q] * 16 + 4 * g + e < V;
          const float base = ok ? order_val(l4[e]) : -INFINITY;
          sb += __builtin_amdgcn_exp2f((base - rb) * kLog2e);
          sf += __builtin_amdgcn_exp2f((acc[q][0][e] - rf) * kLog2e);
        }
      }
    };
    if ((tiles[kTPW - 1] + 1) * 16 <= V) reduce(std::false_type{});  // wave-uniform
    else reduce(std::true_type{});
    const int lt = lab - tiles[0] * 16;  // (the tiles are consecutive)
    if (row < Mr && lab < V && lt >= 0 && lt < kTPW * 16 && ((lt >> 2) & 3) == g) {
      t.lab[row] = lab_b;
      t.lab[Mr + row] = lab_f;
    }
#pragma unroll
    for (int o = 16; o <= 32; o <<= 1) {
      sb += __shfl_xor(sb, o, 64);
      sf += __shfl_xor(sf, o, 64);
    }
    if (g == 0 && row < Mr)
      *(float4 *)(t.part + (((size_t)row * gridDim.x + blockIdx.x) * kCeWaves + wave) * 4) =
          make_float4(mb, sb, mf, sf);
  }
}

// A workgroup per row merges the waves' pairs (CE = log-sum-exp - label logit):
// 1904 of them at 151936 logits and 238 workgroups, two rounds of loads a lane.
constexpr int kLoadsPerLane = 4;
__global__ __launch_bounds__(256) void train_ce_row_kernel(TrainArgs t, int npair) {
  __shared__ float4 red[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, row = blockIdx.x;
  // the label and its two logits first, so their round trip overlaps the pairs'
  const int label = t.labels[row];
  const float lb = order_val(t.lab[row]), lf = order_val(t.lab[t.Mr + row]);
  float mb = -INFINITY, s_b = 0.f, mf = -INFINITY, s_f = 0.f;
  // kLoadsPerLane pairs per lane in flight together (clamped index, masked
  // after): a load per merge would pay one memory round trip each
  const float4 *pr = (const float4 *)t.part + (size_t)row * npair;
  for (int c0 = wave * 64 + lane; c0 < npair; c0 += 256 * kLoadsPerLane) {
    float4 p[kLoadsPerLane];
#pragma unroll
    for (int q = 0; q < kLoadsPerLane; ++q) p[q] = pr[min(c0 + q * 256, npair - 1)];
#pragma unroll
    for (int q = 0; q < kLoadsPerLane; ++q)
      if (c0 + q * 256 < npair) {
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
  if (lane == 0) red[wave] = make_float4(mb, s_b, mf, s_f);
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) {
      lse_merge(mb, s_b, red[w].x, red[w].y);
      lse_merge(mf, s_f, red[w].z, red[w].w);
    }
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
  constexpr size_t lds = ce_tpw(KS) > 4 ? (size_t)kCeWaves * KS * 1024 : 0;  // the fifth tiles
  auto go = [&](auto kernel) {
    (void)hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(kernel, dim3(GC), dim3(kCeWaves * 64), lds, st, t);
  };
  if (t.final_logits) go(train_ce_kernel<WT, KS, true>);
  else go(train_ce_kernel<WT, KS, false>);
}

size_t train_part_bytes(int Mr, int V, int r, bool bf16) {
  return (size_t)Mr * train_ce_grid(V, r, bf16) * kCeWaves * 16;
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
  hipLaunchKernelGGL(train_ce_row_kernel, dim3(t.Mr), dim3(256), 0, st, t, GC * kCeWaves);
  hipLaunchKernelGGL(train_loss_kernel, dim3(1), dim3(64), 0, st, t);
  return hipGetLastError();
}

}  // namespace dk
