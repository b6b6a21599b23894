// Domino-head rollout (Sec. 4.1.2 causal encoder and low-rank correction,
// Fig. 3 sequential rollout), as short kernels per draft position j:
//
//   gru    y_{j-1} = top-1 of position j-1 (the best of the logits kernel's
//          keys; the anchor for j = 1; a forced token when
//          teacher forcing), then S_{j-1} = GRU(E[y_{j-1}], S_{j-2}) for a
//          slice of the d_s state indices per workgroup.  The input half of
//          the gates, E[y] W_ih^T, is a row of the table G = E W_ih^T built at
//          model creation, so a step gathers 3*d_s values instead of streaming
//          W_ih.
//   u      u = SiLU(W1[:, :d] H_j + W1[:, d:] S_{j-1}) (the H half comes from
//          the LM-head GEMM), and W_hh S_{j-1} for the next position's gates.
//   logits L_j = L_base_j + W2 u over a vocabulary slice per workgroup, and an
//          atomic max of its top-1 into the position's key.  With beta > 1 the
//          corrected logits also replace L_base_j in memory: only the top-1 is
//          on the chain from position to position, the other ranks are selected
//          for all positions at once after the loop.
// A kernel boundary is the cheapest grid-wide handshake on this device (about
// 1.6 us against about 4 us for a 256-workgroup spin barrier), so the
// rollout is 3(B-1) launches and the final selection rather than one persistent
// kernel (which up to eight batch rows run, below); the top-1
// of each position is a 64-bit atomic max, so no launch merges lists inside
// the loop.
#include <mutex>

#include "common.h"
#include "kernels.h"
#include "mfma.h"
#include "philox.h"

namespace dk {

// Insert (v, id) into a sorted list (best first) by bubbling.
template <int L>
DEVI void list_insert(float (&lv)[L], int (&li)[L], float v, int id) {
#pragma unroll
  for (int q = 0; q < L; ++q) {
    if (better(v, id, lv[q], li[q])) {
      const float tv = lv[q];
      const int ti = li[q];
      lv[q] = v;
      li[q] = id;
      v = tv;
      id = ti;
    }
  }
}

// Extract the wave's top-beta from per-lane sorted lists: lane k (< beta)
// receives the k-th best in (mv, mi); other lanes get (-inf, INT_MAX).
DEVI void wave_extract(float (&lv)[8], int (&li)[8], int beta, float &mv, int &mi) {
  const int lane = threadIdx.x & 63;
  mv = -INFINITY;
  mi = INT_MAX;
  for (int k = 0; k < beta; ++k) {
    float bv = lv[0];
    int bi = li[0];
    wave_best(bv, bi);
    if (lane == k) {
      mv = bv;
      mi = bi;
    }
    if (li[0] == bi && bi != INT_MAX) {  // ids are unique: exactly one owner advances
#pragma unroll
      for (int q = 0; q < 7; ++q) {
        lv[q] = lv[q + 1];
        li[q] = li[q + 1];
      }
      lv[7] = -INFINITY;
      li[7] = INT_MAX;
    }
  }
}

// Wave-level top-beta of the candidates c in [c0, c1) produced by get(c);
// lane k (< beta) ends with the k-th best in (mv, mi).
template <typename Get>
DEVI void wave_select(Get get, int c0, int c1, int beta, float &mv, int &mi) {
  const int lane = threadIdx.x & 63;
  if (beta == 1) {  // a running best is enough
    float bv = -INFINITY;
    int bi = INT_MAX;
    for (int c = c0 + lane; c < c1; c += 64) {
      float v;
      int id;
      get(c, v, id);
      v = order_val(v);
      if (id != INT_MAX && better(v, id, bv, bi)) {
        bv = v;
        bi = id;
      }
    }
    wave_best(bv, bi);
    mv = lane == 0 ? bv : -INFINITY;
    mi = lane == 0 ? bi : INT_MAX;
    return;
  }
  float lv[8];
  int li[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    lv[q] = -INFINITY;
    li[q] = INT_MAX;
  }
  for (int c = c0 + lane; c < c1; c += 64) {
    float v;
    int id;
    get(c, v, id);
    if (id == INT_MAX) continue;
    list_insert(lv, li, order_val(v), id);
  }
  wave_extract(lv, li, beta, mv, mi);
}

// wave_select over candidates in global memory: each lane loads its
// candidates 8 at a time, all loads of a batch in flight together.
DEVI void wave_select_mem(const float *__restrict__ pv, const int32_t *__restrict__ pi, int cnt, int beta,
                          float &mv, int &mi) {
  const int lane = threadIdx.x & 63;
  float lv[8];
  int li[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    lv[q] = -INFINITY;
    li[q] = INT_MAX;
  }
  for (int c0 = 0; c0 < cnt; c0 += 8 * 64) {
    float v[8];
    int id[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int c = c0 + u * 64 + lane;
      const int cc = c < cnt ? c : cnt - 1;
      v[u] = pv[cc];
      id[u] = c < cnt ? pi[cc] : INT_MAX;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (id[u] != INT_MAX) list_insert(lv, li, order_val(v[u]), id[u]);
  }
  wave_extract(lv, li, beta, mv, mi);
}

DEVI float sigm(float x) { return 1.f / (1.f + expf(-x)); }
// The GRU's new state (1 - z) n + z h, written as n + z (h - n) with one
// explicit fused multiply-add: left to the compiler, the two products of the
// plain form get contracted differently from one kernel instantiation to the
// next, and the instantiations would disagree in the last bit.
DEVI float gru_mix(float z, float n, float h) { return fmaf(z, h - n, n); }

constexpr int kBestSlots = 8;  // atomic targets per (position, row), spread to cut contention

template <typename WT>
DEVI void unpack16(const u32x4 &w, float *f);
template <>
DEVI void unpack16<bf16_t>(const u32x4 &w, float *f) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    f[2 * q] = __uint_as_float(w[q] << 16);
    f[2 * q + 1] = __uint_as_float(w[q] & 0xffff0000u);
  }
}
template <>
DEVI void unpack16<float>(const u32x4 &w, float *f) {
#pragma unroll
  for (int q = 0; q < 4; ++q) f[q] = __uint_as_float(w[q]);
}

// ---------------------------------------------------------------------------
// state (batches up to kFusedBatch; replaces gru + u): every workgroup forms
// the whole S_{j-1} itself from the gathered input gates G[y_{j-1}], the
// hidden gates W_hh S_{j-2} that the previous position left in ghbuf, and
// S_{j-2}; its waves then take rows of the stacked matrix [W1[:, d:]; W_hh]
// against S_{j-1}.  The first r rows give u_j = SiLU(P_j + W1[:, d:] S_{j-1}),
// the other 3 d_s rows the hidden gates of position j+1, so the elementwise
// update is the only step repeated per workgroup and no launch sits between
// the state and u.  Weight rows are loaded before the state is formed.
// ---------------------------------------------------------------------------
constexpr int kFusedBatch = kHeadFusedBatch;
constexpr int kStateWaves = 8;
constexpr int kStateMaxGrid = 256;

template <typename WT>
__global__ __launch_bounds__(kStateWaves * 64) void head_state_kernel(HeadArgs h, int j) {
  constexpr int EPL = 16 / sizeof(WT);
  const Dims &D = h.D;
  const int bs = D.bs, ds = D.ds, r = D.r, d = D.d, depth = D.B - 1, V = D.V;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  extern __shared__ __align__(16) float sl[];  // S_{j-1} [bs][ds]
  __shared__ int ys[kFusedBatch];
  const int nchunk = ds / EPL;  // <= 256
  const int nrows = r + (j < depth ? 3 * ds : 0);
  const int rbeg = h.skip_u ? r : 0;  // skip_u: only the W_hh rows (u is formed later, batched)
  const int nw = gridDim.x * kStateWaves;
  const int w0 = blockIdx.x * kStateWaves + wave;
  const WT *w1 = (const WT *)h.w1, *whh = (const WT *)h.w_hh;

  // ---- the sources of y_{j-1} first (every thread, clamped batch row, so no
  // branch holds the later loads back), then this wave's weight rows
  const int bq = min(tid, bs - 1);
  const int anc = h.anchor[bq];
  unsigned long long keys[kBestSlots];
  {
    const unsigned long long *bk = h.best + ((size_t)(j > 1 ? j - 2 : 0) * bs + bq) * kBestSlots;
#pragma unroll
    for (int q = 0; q < kBestSlots; ++q) keys[q] = bk[q];
  }
  // two rows per wave per round (rows w0 + k*nw); the first round's loads go out now
  u32x4 w[2][4];
  auto load_rows = [&](int base) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int row = min(base + q * nw, nrows - 1);
      const WT *p = row < r ? w1 + (size_t)row * (d + ds) + d : whh + (size_t)(row - r) * ds;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int ch = min(lane + 64 * c, nchunk - 1);
        w[q][c] = *(const u32x4 *)(p + (size_t)ch * EPL);
      }
    }
  };
  load_rows(rbeg + w0);

  // ---- y_{j-1}: the anchor, a forced token, or the decoded best key of position j-1
  if (tid < bs) {
    int y;
    if (j == 1) y = clamp_token(anc, V, h.err);
    else if (h.forced) y = clamp_token(h.forced[(size_t)tid * depth + (j - 2)], V, h.err);  // teacher forcing
    else {
      unsigned long long key = keys[0];
#pragma unroll
      for (int q = 1; q < kBestSlots; ++q) key = keys[q] > key ? keys[q] : key;
      y = decode_best_id(key, V);
    }
    ys[tid] = y;
  }
  __syncthreads();

  // ---- S_{j-1} = GRU(x = E[y_{j-1}], S_{j-2}), four state indices per item.
  // G holds E W_ih^T + b_ih; the stored gates hold W_hh S_{j-2} + b_hh (at j = 1,
  // S = 0: the gates are b_hh).  Every load is unconditional (the position-1
  // values are selected after), so none waits behind a branch.
  const float *ghp = h.ghbuf + (size_t)((j - 1) & 1) * bs * 3 * ds;  // W_hh S_{j-2} + b_hh
  const float *sprev = h.hbuf + (size_t)(j & 1) * bs * ds;            // S_{j-2}
  float *scur = h.hbuf + (size_t)((j - 1) & 1) * bs * ds;             // S_{j-1}
  for (int it = tid; it < bs * ds / 4; it += kStateWaves * 64) {
    const int b = it / (ds / 4), i = (it % (ds / 4)) * 4;
    const float *gy = h.gtab + (size_t)ys[b] * 3 * ds;
    float gi[3][4], gh[3][4], hold[4];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const float4 a = *(const float4 *)(gy + q * ds + i);
      const float4 c = *(const float4 *)(ghp + (size_t)b * 3 * ds + q * ds + i);
      const float4 c0 = *(const float4 *)(h.bhh + q * ds + i);
      gi[q][0] = a.x; gi[q][1] = a.y; gi[q][2] = a.z; gi[q][3] = a.w;
      gh[q][0] = j > 1 ? c.x : c0.x; gh[q][1] = j > 1 ? c.y : c0.y;
      gh[q][2] = j > 1 ? c.z : c0.z; gh[q][3] = j > 1 ? c.w : c0.w;
    }
    {
      const float4 c = *(const float4 *)(sprev + (size_t)b * ds + i);
      hold[0] = j > 1 ? c.x : 0.f; hold[1] = j > 1 ? c.y : 0.f;
      hold[2] = j > 1 ? c.z : 0.f; hold[3] = j > 1 ? c.w : 0.f;
    }
    float out[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float rg = sigm(gi[0][e] + gh[0][e]);
      const float zg = sigm(gi[1][e] + gh[1][e]);
      const float ng = tanhf(fmaf(rg, gh[2][e], gi[2][e]));
      out[e] = gru_mix(zg, ng, hold[e]);
    }
    const float4 o = make_float4(out[0], out[1], out[2], out[3]);
    *(float4 *)(sl + (size_t)b * ds + i) = o;
    if (blockIdx.x == 0) {
      *(float4 *)(scur + (size_t)b * ds + i) = o;
      if (h.states) *(float4 *)(h.states + ((size_t)b * depth + (j - 1)) * ds + i) = o;
    }
  }
  __syncthreads();

  // ---- rows of [W1[:, d:]; W_hh] against S_{j-1}
  float *ghn = h.ghbuf + (size_t)(j & 1) * bs * 3 * ds;  // W_hh S_{j-1}
  for (int base = rbeg + w0; base < nrows; base += 2 * nw) {
    if (base != rbeg + w0) load_rows(base);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int row = base + q * nw;
      if (row >= nrows) continue;  // wave-uniform
      float wf[4][EPL];
#pragma unroll
      for (int c = 0; c < 4; ++c) unpack16<WT>(w[q][c], wf[c]);
      for (int b = 0; b < bs; ++b) {
        const float *sb = sl + (size_t)b * ds;
        float acc = 0.f;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const int ch = lane + 64 * c;
          if (ch < nchunk) {
#pragma unroll
            for (int e = 0; e < EPL; e += 4) {
              const float4 t = *(const float4 *)(sb + (size_t)ch * EPL + e);
              acc = fmaf(wf[c][e], t.x, acc);
              acc = fmaf(wf[c][e + 1], t.y, acc);
              acc = fmaf(wf[c][e + 2], t.z, acc);
              acc = fmaf(wf[c][e + 3], t.w, acc);
            }
          }
        }
        acc = wave_sum(acc);
        if (lane == 0) {
          if (row < r) {
            const float x = h.P[((size_t)b * depth + (j - 1)) * h.ldp + row] + acc;
            h.ubuf[(size_t)b * h.u_ld + (size_t)(j - 1) * h.u_pos + row] = x / (1.f + expf(-x));
          } else {
            ghn[(size_t)b * 3 * ds + (row - r)] = acc + h.bhh[row - r];
          }
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Batches above kFusedBatch: the elementwise GRU update and the state's two
// products are a launch each.  (Two K-split GEMMs and two elementwise launches
// to add their partials took 24 us a position at 32 rows, 20 at 16; the two
// launches take 13 and 11.)
// ---------------------------------------------------------------------------
// S_j = GRU(G[y_{j-1}], S_{j-1}), one workgroup row per batch row
__global__ __launch_bounds__(256) void head_gru_elem_kernel(HeadArgs h, int j) {
  const Dims &D = h.D;
  const int bs = D.bs, ds = D.ds, depth = D.B - 1, V = D.V;
  const int b = blockIdx.y, i = blockIdx.x * 256 + threadIdx.x;
  // the hidden gates W_hh S_{j-1} + b_hh (S_0 = 0: b_hh alone at j = 1), loaded beside the keys
  float gh[3];
  const float *ghp = j > 1 ? h.ghbuf + ((size_t)((j - 1) & 1) * bs + b) * 3 * ds : h.bhh;
#pragma unroll
  for (int q = 0; q < 3; ++q) gh[q] = ghp[q * ds + min(i, ds - 1)];
  __shared__ int ysh;
  if (threadIdx.x == 0) {  // y_{j-1}: the anchor, a forced token, or the decoded best key of position j-1
    int y;
    if (j == 1) y = clamp_token(h.anchor[b], V, h.err);
    else if (h.forced) y = clamp_token(h.forced[(size_t)b * depth + (j - 2)], V, h.err);
    else {
      const unsigned long long *bk = h.best + ((size_t)(j - 2) * bs + b) * kBestSlots;
      unsigned long long key = bk[0];
#pragma unroll
      for (int q = 1; q < kBestSlots; ++q) key = bk[q] > key ? bk[q] : key;
      y = decode_best_id(key, V);
    }
    ysh = y;
  }
  __syncthreads();
  if (i >= ds) return;
  const float *hprev = h.hbuf + (size_t)((j - 1) & 1) * bs * ds;
  float *hnext = h.hbuf + (size_t)(j & 1) * bs * ds;
  const float *gy = h.gtab + (size_t)ysh * 3 * ds;  // b_ih is in G
  const float rg = sigm(gy[i] + gh[0]), zg = sigm(gy[ds + i] + gh[1]);
  const float ng = tanhf(fmaf(rg, gh[2], gy[2 * ds + i]));
  const float hold = j > 1 ? hprev[(size_t)b * ds + i] : 0.f;
  const float hn = gru_mix(zg, ng, hold);
  hnext[(size_t)b * ds + i] = hn;
  if (h.states) h.states[((size_t)b * depth + (j - 1)) * ds + i] = hn;
}

// One 16-row tile of [W1[:, d:]; W_hh] times S_j for every batch row: the first
// nu workgroups give u_j = SiLU(W1[:, :d] H_j + W1[:, d:] S_j), the others the
// hidden gates W_hh S_j + b_hh of the next position.  Its 8 waves split K
// (consecutive k-steps of the packed tiles); each loads its own states straight
// into fragments, and the partial sums meet in LDS, added in wave order.
// Latency-bound: every load of a wave is in flight at once.
constexpr int kRowWaves = 8;
template <typename WT, int MT>
__global__ __launch_bounds__(kRowWaves * 64) void head_rows_kernel(HeadArgs h, int j, int nu) {
  constexpr int EPL = Frag<WT>::EPL, KSTEP = Frag<WT>::KSTEP, XF = XStage<WT>::XF;
  constexpr int kU = 4;  // k-steps in flight
  const Dims &D = h.D;
  const int bs = D.bs, ds = D.ds, r = D.r, depth = D.B - 1;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, cc = lane & 15;
  const bool is_u = (int)blockIdx.x < nu;  // workgroup-uniform
  const int tile = is_u ? blockIdx.x : blockIdx.x - nu;
  const int KS = is_u ? h.w1s_KS : h.whh_KS;  // equal: both are over d_s
  const u32x4 *P = (const u32x4 *)(is_u ? h.w1s_p : h.whh_p) + (size_t)tile * KS * 64 + lane;
  const float *S = h.hbuf + (size_t)(j & 1) * bs * ds;
  const int per = (KS + kRowWaves - 1) / kRowWaves, s0 = wave * per, s1 = min(KS, s0 + per);
  floatx4 acc[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) acc[mt] = floatx4{0.f, 0.f, 0.f, 0.f};
  for (int s = s0; s < s1; s += kU) {
    u32x4 w[kU];
    float4 x[kU][MT][EPL / 4];
#pragma unroll
    for (int q = 0; q < kU; ++q) {
      const int sc = min(s + q, s1 - 1);
      w[q] = P[(size_t)sc * 64];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const float *src = S + (size_t)min(mt * 16 + cc, bs - 1) * ds + sc * KSTEP + g * EPL;
#pragma unroll
        for (int e = 0; e < EPL / 4; ++e) x[q][mt][e] = *(const float4 *)(src + 4 * e);
      }
    }
#pragma unroll
    for (int q = 0; q < kU; ++q)
      if (s + q < s1) {
        u32x4 xf[MT * XF];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) XStage<WT>::put(xf + mt * XF, x[q][mt]);
        Mac2<WT, MT>::step(w[q], xf, acc);
      }
  }
  __shared__ floatx4 red[kRowWaves][MT][64];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) red[wave][mt][lane] = acc[mt];
  __syncthreads();
  if (wave >= MT) return;
  const int bb = wave * 16 + cc;  // wave mt finishes batch rows 16 mt ..
  floatx4 t = red[0][wave][lane];
#pragma unroll
  for (int w = 1; w < kRowWaves; ++w) t += red[w][wave][lane];
  if (bb >= bs) return;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int row = tile * 16 + 4 * g + e;
    if (is_u) {
      if (row >= r) continue;
      const float x = h.P[((size_t)bb * depth + (j - 1)) * h.ldp + row] + t[e];
      h.ubuf[(size_t)bb * h.u_ld + (size_t)(j - 1) * h.u_pos + row] = x / (1.f + expf(-x));
    } else if (row < 3 * ds) {
      h.ghbuf[((size_t)(j & 1) * bs + bb) * 3 * ds + row] = t[e] + h.bhh[row];
    }
  }
}

// ---------------------------------------------------------------------------
// logits: matrix-core W2 tiles times the staged u (batch rows as the 16
// columns of the B operand, hi/lo split for bf16), added onto L_base, then each
// workgroup's top-1 per batch row.  A workgroup covers ROWS vocabulary
// rows (8 waves x kTPW tiles of 16).  (With the top-beta of beta > 1 selected
// here, a position took 44 us at 32 rows and beta 4, half of it the selection;
// now 31 us, and 47 once for the selection.)
// ---------------------------------------------------------------------------
constexpr int kLogitWaves = 8;
// W2 tiles per wave: five, so that the grid fits the GPU in one round at the
// Qwen3 vocabulary (238 workgroups); one where the vocabulary is so small that
// even then most CUs get no workgroup
constexpr int logit_tpw(int KS, int MT) { return KS == 8 ? 5 : (MT == 1 ? 5 : (MT == 2 ? 3 : 1)); }
constexpr int kSmallVocabTiles = 256 * kLogitWaves;

template <typename WT, int KS, int MT, int kTPW>
__global__ __launch_bounds__(kLogitWaves * 64) void head_logits_kernel(HeadArgs h, int j) {
  constexpr int EPL = Frag<WT>::EPL, KSTEP = Frag<WT>::KSTEP, XF = XStage<WT>::XF;
  const Dims &D = h.D;
  const int bs = D.bs, V = D.V, depth = D.B - 1;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 4, cc = lane & 15;
  const int NT = (V + 15) / 16;
  extern __shared__ __align__(16) unsigned char smem[];
  u32x4 *us = (u32x4 *)smem;                                      // [KS][MT][64][XF]

  // u_j first (a few L2-resident values), so the matrix-core work can follow
  // the W2 stream as its fragments arrive
  constexpr int kUIt = (KS * MT * 64 + kLogitWaves * 64 - 1) / (kLogitWaves * 64);
  float4 uv[kUIt][EPL / 4];
#pragma unroll
  for (int q = 0; q < kUIt; ++q) {
    const int it = min(tid + q * kLogitWaves * 64, KS * MT * 64 - 1);
    const int l = it & 63, mt = (it >> 6) % MT, s = (it >> 6) / MT;
    const int bb = mt * 16 + (l & 15);
    const int k0 = s * KSTEP + (l >> 4) * EPL;
    // unconditional loads at a clamped row: a guarded load becomes a branch
    // whose join drains every outstanding load, holding back the W2 stream
    // issued below.  Columns of padding rows (bb >= bs) only reach output
    // columns that are never read, so their values do not matter.
    const float *src = h.ubuf + (size_t)min(bb, bs - 1) * h.u_ld + (size_t)(j - 1) * h.u_pos + k0;
#pragma unroll
    for (int e = 0; e < EPL / 4; ++e) uv[q][e] = *(const float4 *)(src + 4 * e);
  }
  // then the L_base values the products are added onto (rows are padded to whole
  // tiles, ldl >= 16 * NT, so a tile's four values load as one float4, the layout
  // of the sums; entries past V are masked below), then the W2 fragments of its tiles
  int tiles[kTPW];
#pragma unroll
  for (int q = 0; q < kTPW; ++q) tiles[q] = (blockIdx.x * kLogitWaves + wave) * kTPW + q;
  floatx4 acc[kTPW][MT];
#pragma unroll
  for (int q = 0; q < kTPW; ++q)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int bb = mt * 16 + cc;
      const int t = tiles[q] < NT ? tiles[q] : NT - 1;
      // clamped row, unconditional (lanes of padding rows are never read)
      acc[q][mt] =
          *(const floatx4 *)(h.Lbase + ((size_t)min(bb, bs - 1) * depth + (j - 1)) * h.ldl + t * 16 + 4 * g);
    }
  // W2 fragments: kRing tiles in flight (8 waves then keep 192 KB or more per CU on
  // the way, several times what the latency needs), later tiles into the
  // registers of the finished ones
  constexpr int kRing = KS == 8 ? (kTPW < 3 ? kTPW : 3) : (kTPW < 2 ? kTPW : 2);
  const u32x4 *w2p = (const u32x4 *)h.w2p;
  u32x4 wf[kRing][KS];
  auto load_tile = [&](int q) {
    const int t = tiles[q] < NT ? tiles[q] : NT - 1;
#pragma unroll
    for (int s = 0; s < KS; ++s) wf[q % kRing][s] = w2p[((size_t)t * KS + s) * 64 + lane];
  };
#pragma unroll
  for (int q = 0; q < kRing; ++q) load_tile(q);
  // u staged as matrix-core B fragments
#pragma unroll
  for (int q = 0; q < kUIt; ++q) {
    const int it = tid + q * kLogitWaves * 64;
    if (it < KS * MT * 64) XStage<WT>::put(us + (size_t)it * XF, uv[q]);
  }
  __syncthreads();

  // tile-major, in the order the fragments were requested: tile q's products
  // start as soon as its fragments arrive, overlapping the rest of the stream
#pragma unroll
  for (int q = 0; q < kTPW; ++q) {
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      u32x4 xf[MT * XF];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int f = 0; f < XF; ++f) xf[mt * XF + f] = us[((size_t)(s * MT + mt) * 64 + lane) * XF + f];
      Mac2<WT, MT>::step(wf[q % kRing][s], xf, acc[q]);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (q + kRing < kTPW) load_tile(q + kRing);
    __builtin_amdgcn_sched_barrier(0);
  }

  // corrected logits of this workgroup's rows: lane (g, cc) holds rows
  // 16 t + 4 g + e of batch row mt * 16 + cc
  if (h.lout) {  // beta > 1: for the selection after the loop (whole tiles: the padding keeps its zeros)
#pragma unroll
    for (int q = 0; q < kTPW; ++q)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const int bb = mt * 16 + cc;
        if (bb < bs && tiles[q] < NT)
          *(floatx4 *)(h.lout + ((size_t)bb * depth + (j - 1)) * h.ldl + tiles[q] * 16 + 4 * g) = acc[q][mt];
      }
  }
  {
    // top-1 without staging: a running best per batch row in registers, the
    // four lanes of a row combined by shuffles, then one entry per (wave, row).
    // With sampling the key is L / T + Gumbel noise of (row, position, id): the
    // maximum is a draw from softmax(L / T); raw carries the chosen L.
    __shared__ float best_v[kLogitWaves][64], best_r[kLogitWaves][64];
    __shared__ int best_i[kLogitWaves][64];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int bb = mt * 16 + cc;
      float bv = -INFINITY, br = 0.f;
      int bi = INT_MAX;
#pragma unroll
      for (int q = 0; q < kTPW; ++q) {
        Philox4 noise = {{0u, 0u, 0u, 0u}};
        if (h.sample && bb < bs) noise = rng_block(h.seed_lo, h.seed_hi, RNG_DRAFT, bb, j, tiles[q] * 4 + g);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int n = tiles[q] * 16 + 4 * g + e;
          const float val = acc[q][mt][e];
          if (bb < bs && n < V) {
            if (h.final_logits) h.final_logits[((size_t)bb * depth + (j - 1)) * V + n] = val;
            const float key = h.sample ? val * h.inv_temp + rng_gumbel(noise.x[e]) : val;
            const float ov = order_val(key);
            if (better(ov, n, bv, bi)) {
              bv = ov;
              bi = n;
              br = val;
            }
          }
        }
      }
#pragma unroll
      for (int o = 16; o <= 32; o <<= 1) {
        const float ov = __shfl_xor(bv, o, 64);
        const int oi = __shfl_xor(bi, o, 64);
        const float orw = __shfl_xor(br, o, 64);
        if (better(ov, oi, bv, bi)) {
          bv = ov;
          bi = oi;
          br = orw;
        }
      }
      if (g == 0) {
        best_v[wave][bb] = bv;
        best_i[wave][bb] = bi;
        best_r[wave][bb] = br;
      }
    }
    __syncthreads();
    for (int bb = tid; bb < bs; bb += kLogitWaves * 64) {
      float v = best_v[0][bb], raw = best_r[0][bb];
      int id = best_i[0][bb];
#pragma unroll
      for (int w = 1; w < kLogitWaves; ++w)
        if (better(best_v[w][bb], best_i[w][bb], v, id)) {
          v = best_v[w][bb];
          id = best_i[w][bb];
          raw = best_r[w][bb];
        }
      if (!h.lout) {  // branch 1: one entry a workgroup for the final merge
        const size_t o = ((size_t)(j - 1) * bs + bb) * h.GC + blockIdx.x;
        h.pval[o] = v;
        h.pid[o] = id;
        if (h.sample) h.praw[o] = raw;
      }
      if (id != INT_MAX)
        atomicMax(&h.best[((size_t)(j - 1) * bs + bb) * kBestSlots + (blockIdx.x % kBestSlots)], encode_best(v, id));
    }
  }
}

// Maximum over the wave by lane rotations within rows and four lane reads
DEVI float wave_max_dpp(float v) {
  v = fmaxf(v, row_ror<8>(v));
  v = fmaxf(v, row_ror<4>(v));
  v = fmaxf(v, row_ror<2>(v));
  v = fmaxf(v, row_ror<1>(v));
  float r = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 0));
#pragma unroll
  for (int k = 1; k < 4; ++k) r = fmaxf(r, __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 16 * k)));
  return r;
}

// The top-beta (1 < beta <= L) of every position's corrected logits, after the
// rollout: a wave per kTopWave values of one row, 64 a lane in registers.  The
// beta-th largest of the 64 lane maxima bounds the wave's beta-th best from
// below, so only the few values from there on (about beta of 4096) are
// inserted, one by one, into a sorted list that every lane keeps alike; the bound
// follows the list's last entry.  Four values share a test.  Bound by reading
// the logits (292 MB at 32 rows, 45 us; the whole selection 47, 92 with a
// test and eight list entries for each value).
constexpr int kTopWave = 4096;
template <int L>
__global__ __launch_bounds__(256) void head_topb_kernel(HeadArgs h, int nchunk) {
  const int V = h.D.V, beta = h.beta, depth = h.D.B - 1, bs = h.D.bs;
  const int lane = threadIdx.x & 63;
  const int c = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int j = blockIdx.y, b = blockIdx.z;
  if (c >= nchunk) return;  // (whole waves; no barrier below)
  const float *row = h.Lbase + ((size_t)b * depth + j) * h.ldl;
  constexpr int NQ = kTopWave / 256;
  float4 x[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {  // rows are padded to whole tiles of 16: a float4 that starts inside ends inside
    const int id = c * kTopWave + q * 256 + 4 * lane;
    x[q] = __builtin_bit_cast(float4, __builtin_nontemporal_load((const floatx4 *)(row + min(id, (V - 1) / 4 * 4))));
  }
  if ((c + 1) * kTopWave > V) {  // wave-uniform: ids past V become NaN, which nothing below takes
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (c * kTopWave + q * 256 + 4 * lane + e >= V) (&x[q].x)[e] = NAN;
  }
  float m4[NQ], m = -INFINITY;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    m4[q] = fmaxf(fmaxf(x[q].x, x[q].y), fmaxf(x[q].z, x[q].w));  // a NaN drops out
    m = fmaxf(m, m4[q]);
  }
  float t = -INFINITY;
  for (int k = 0; k < beta; ++k) {  // the beta-th largest lane maximum (equal ones leave together: the bound is only lower)
    t = wave_max_dpp(m);
    if (m == t) m = -INFINITY;
  }
  float lv[L];
  int li[L];
#pragma unroll
  for (int k = 0; k < L; ++k) {
    lv[k] = -INFINITY;
    li[k] = INT_MAX;
  }
  float wv = t;  // what a value has to beat: the bound, then the list's entry of rank beta
  int wi = INT_MAX;
  // A bound of -inf admits every value: NaN (as -inf) too, below V
  const bool low = t == -INFINITY;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    if (!low && !__any(m4[q] >= wv)) continue;
    const int id = c * kTopWave + q * 256 + 4 * lane;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float v = order_val((&x[q].x)[e]);
      unsigned long long mk = __ballot(id + e < V && better(v, id + e, wv, wi));
      while (mk) {  // wave-uniform
        const int l = __ffsll(mk) - 1;
        mk &= mk - 1;
        const float cv = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
        const int ci = c * kTopWave + q * 256 + 4 * l + e;
        if (!better(cv, ci, wv, wi)) continue;
        list_insert<L>(lv, li, cv, ci);
        float ev = lv[0];
        int ei = li[0];
#pragma unroll
        for (int k = 1; k < L; ++k)
          if (k < beta) {
            ev = lv[k];
            ei = li[k];
          }
        if (ei != INT_MAX) {  // the list has beta entries
          wv = ev;
          wi = ei;
        }
      }
    }
  }
  if (lane == 0) {
    const size_t o = (((size_t)j * bs + b) * nchunk + c) * beta;
#pragma unroll
    for (int k = 0; k < L; ++k)
      if (k < beta) {
        h.pval[o + k] = lv[k];
        h.pid[o + k] = li[k];
      }
  }
}

// Merge the nlist top-beta lists of one (position, batch row) after the
// rollout (branch 1: a workgroup's top-1 each); one wave per (j, b).
__global__ __launch_bounds__(64) void head_merge_kernel(HeadArgs h, int nlist) {
  const int j = blockIdx.x, b = blockIdx.y;
  const int bs = h.D.bs, depth = h.D.B - 1, beta = h.beta;
  const int lane = threadIdx.x;
  const size_t base = ((size_t)j * bs + b) * nlist * beta;
  if (h.sample) {  // branch 1: the largest key wins; its raw logit is the reported value
    float bv = -INFINITY, br = 0.f;
    int bi = INT_MAX;
    for (int c = lane; c < nlist; c += 64) {
      const float v = order_val(h.pval[base + c]);
      const int id = h.pid[base + c];
      const float raw = h.praw[base + c];
      if (id != INT_MAX && better(v, id, bv, bi)) {
        bv = v;
        bi = id;
        br = raw;
      }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      const float ov = __shfl_xor(bv, o, 64);
      const int oi = __shfl_xor(bi, o, 64);
      const float orw = __shfl_xor(br, o, 64);
      if (better(ov, oi, bv, bi)) {
        bv = ov;
        bi = oi;
        br = orw;
      }
    }
    if (lane == 0) {
      h.topk_ids[(size_t)b * depth + j] = bi;
      h.topk_vals[(size_t)b * depth + j] = br;
    }
    return;
  }
  float mv;
  int mi;
  wave_select_mem(h.pval + base, h.pid + base, nlist * beta, beta, mv, mi);
  if (lane < beta) {
    h.topk_ids[((size_t)b * depth + j) * beta + lane] = mi;
    h.topk_vals[((size_t)b * depth + j) * beta + lane] = mv;
  }
}

// ---------------------------------------------------------------------------
// Persistent rollout (bf16 weights, r = 256, up to eight batch rows, greedy or
// sampled): one launch of at most one workgroup per CU runs all B-1 positions
// (134 us at one row of the Qwen3 vocabulary, 294 at four, which took 412 as two
// launches of two rows).  Each workgroup keeps its slice of W2 for the whole rollout (kPersTiles tiles per wave, the last one in
// LDS, the rest in registers: 77.8 MB over 238 workgroups) and its rows of [W1[:, d:]; W_hh] in LDS, so W2 leaves HBM once
// per step instead of once per position.  Bound by the serial chain of a
// position: the state's update, two exchanges between all workgroups and the
// logits.  The rows of a batch are columns of the same products (u's high and
// low parts, 2 x 8 of the tile's 16) and words of the same 64-byte exchange line,
// polled by as many waves, so that eight rows cost one row's traffic; what grows
// with the rows (about 4 us a position and row) is the state's update, which every
// workgroup makes for itself rather than pay a third exchange.
//
// Workgroups exchange data through tagged 64-bit slots in the workspace
// header (zeroed at every step), written with device-scope atomic stores and
// polled with device-scope atomic loads by a wave per batch row; a slot is ready when its
// top bits carry the position's tag, so a poll both waits and delivers:
//   u slot [k][b]   (j << 32) | bits of u_j[k], written by the owner of row k
//   key slot [g][b] (j << 50) | value(32) << 18 | (2^18 - 1 - id): workgroup
//                   g's top-1 for position j; the maximum over g is the argmax
//                   under (value desc, id asc)
// The hidden gates W_hh S for the next position go out as plain device-scope
// stores while other waves wait for u; each thread waits for its own stores
// before its workgroup publishes its key, so "all key slots ready" also means
// "all gates stored".
// Waits are bounded: a timeout sets DEV_BARRIER_TIMEOUT and the abort flag,
// and every workgroup leaves; the kernel always ends.  Workgroup 0 writes the
// drafted token and its value of every position (no merge kernel; at beta > 1 the
// selection from the corrected logits follows, as after the launch loop).
// ---------------------------------------------------------------------------
constexpr int kPersWaves = 8, kPersTiles = 5, kPersKS = 8, kPersRegTiles = kPersTiles - 1;
constexpr int kPersMaxBatch = kSlotStride;  // batch rows: a word of an exchange line each
static_assert(kPersMaxBatch <= kPersWaves && 2 * kPersMaxBatch <= 16, "a polling wave and two tile columns per row");
constexpr int kKeyIdBits = 18;
// 64-lane loads of 16 bytes that bring a wave's tiles of L_base for BS rows
constexpr int pers_lb_loads(int BS) { return (kPersTiles * BS * 4 + 63) / 64; }

DEVI unsigned long long ld_slot(const unsigned long long *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
DEVI void st_slot(unsigned long long *p, unsigned long long v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
DEVI unsigned long long pack_key50(float v, int id) {
  uint32_t u = __float_as_uint(order_val(v));
  u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return ((unsigned long long)u << kKeyIdBits) | (unsigned long long)((1 << kKeyIdBits) - 1 - id);
}
DEVI int key50_id(unsigned long long k) { return (1 << kKeyIdBits) - 1 - (int)(k & ((1ull << kKeyIdBits) - 1)); }

// The first BS waves poll `n` <= 256 lines (kSlotStride words apart, word b batch
// row b's) until each word carries `tag` (top bits from `shift`): lane l of wave
// w holds units e = (4 w + q) 64 + l in x[q], line e / BS, word e % BS (past the
// last line or row: a copy).  Returns false on timeout (`limit` polls made, none
// complete) or when another workgroup has aborted.
template <int BS>
DEVI bool poll_tagged(const unsigned long long *slots, int n, int bs, int wave, unsigned long long tag, int shift,
                      unsigned *abort_flag, int32_t *err, unsigned limit, unsigned long long (&x)[4]) {
  const int lane = threadIdx.x & 63;
  unsigned polls = 0;
  while (true) {
    if (polls++ >= limit) {  // this wait gives up: every workgroup is told to leave
      if (lane == 0) {
        __hip_atomic_store(abort_flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        raise_error(err, DEV_BARRIER_TIMEOUT);
      }
      return false;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int e = (4 * wave + q) * 64 + lane;
      x[q] = ld_slot(slots + (size_t)min(e / BS, n - 1) * kSlotStride + (BS == 1 ? 0 : min(e % BS, bs - 1)));
    }
    bool ready = true;
#pragma unroll
    for (int q = 0; q < 4; ++q) ready = ready && (x[q] >> shift) == tag;
    if (__all(ready)) return true;
    if ((polls & 63) == 0 && __hip_atomic_load(abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return false;
  }
}

// BS: the largest batch the instantiation serves (1, 2, 4 or 8; arrays sized by it);
// DBG: the final logits are also written out (h.final_logits, h.lout);
// SAMPLE: temperature sampling, the selection key is L / T + Gumbel noise
// (Philox stream RNG_DRAFT, as in the launch-pair rollout) and the reported
// value is the chosen token's raw logit
template <int BS, bool DBG, bool SAMPLE>
__global__ __launch_bounds__(kPersWaves * 64) void head_persist_kernel(HeadArgs h, int nr) {
  using WT = bf16_t;
  constexpr int EPL = 8, KSTEP = 32;
  const Dims &D = h.D;
  const int bs = D.bs, ds = D.ds, r = D.r, d = D.d, depth = D.B - 1, V = D.V;
  // the wave index is uniform in a wave: held in a scalar register, so the
  // per-wave offsets below cost no vector registers (the resident W2 tiles
  // take 128 of the 256)
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, cc = lane & 15;
  const int G = gridDim.x, NT = (V + 15) / 16;
  const int nchunk = ds / EPL;  // 16-byte chunks of a row (<= 256 by the config check)
  const int nrows_all = r + 3 * ds;
  extern __shared__ __align__(16) unsigned char smem[];
  u32x4 *rows = (u32x4 *)smem;                          // [nr][nchunk] rows of [W1s; W_hh]
  float *S = (float *)(rows + (size_t)nr * nchunk);     // [bs][ds] the state
  u32x4 *us = (u32x4 *)(S + (size_t)bs * ds);           // [KS][64] u as B fragments
  u32x4 *w2s = us + kPersKS * 64;                       // [waves][KS][64] each wave's last W2 tile
  constexpr int NI = pers_lb_loads(BS);
  float4 *lbs = (float4 *)(w2s + kPersWaves * kPersKS * 64);  // [waves][NI * 64] L_base, see below
  const int nu = (r + G - 1) / G;                              // u rows per workgroup: k < nu (R < r)
  float *P_s = (float *)(lbs + kPersWaves * NI * 64);  // [depth][bs][nu] W1[:, :d] H at the u rows
  // each lane's best of its tiles, value, id and raw logit by [row group g][batch
  // row]: over the wave's own part of lbs, once its values are used
  auto best_at = [&](int w, int field, int gg, int b) { return (float *)(lbs + w * NI * 64) + (field * 4 + gg) * BS + b; };
  __shared__ unsigned long long s_key[BS][BS];  // polling wave's best key of each batch row
  __shared__ int ys[BS], s_ok[BS];
  auto all_ok = [&] {
    int ok = 1;
#pragma unroll
    for (int w = 0; w < BS; ++w) ok &= s_ok[w];
    return ok != 0;
  };
  auto key_of = [&](int b) {
    unsigned long long k = s_key[0][b];
#pragma unroll
    for (int w = 1; w < BS; ++w) k = s_key[w][b] > k ? s_key[w][b] : k;
    return k;
  };
  const WT *w1 = (const WT *)h.w1, *whh = (const WT *)h.w_hh;
  const int tile0 = (blockIdx.x * kPersWaves + wave) * kPersTiles;  // this wave's tiles tile0 + q

  // ---- resident operands, loaded once: W2 tiles, rows, b_ih
  u32x4 wf[kPersRegTiles][kPersKS];
  {
    const u32x4 *w2p = (const u32x4 *)h.w2p;
#pragma unroll
    for (int q = 0; q < kPersTiles; ++q) {
      const int t = min(tile0 + q, NT - 1);
#pragma unroll
      for (int s = 0; s < kPersKS; ++s) {
        const u32x4 v = w2p[((size_t)t * kPersKS + s) * 64 + lane];
        if (q < kPersRegTiles) wf[q < kPersRegTiles ? q : 0][s] = v;
        else w2s[((size_t)wave * kPersKS + s) * 64 + lane] = v;
      }
    }
  }
  for (int e = tid; e < nr * nchunk; e += kPersWaves * 64) {
    const int k = e / nchunk, ch = e % nchunk;
    const int R = min(blockIdx.x + k * G, nrows_all - 1);
    const WT *src = R < r ? w1 + (size_t)R * (d + ds) + d : whh + (size_t)(R - r) * ds;
    rows[e] = *(const u32x4 *)(src + (size_t)ch * EPL);
  }
  for (int e = tid; e < bs * ds; e += kPersWaves * 64) S[e] = 0.f;
  // the u fragments' unused columns stay zero for the whole launch
  for (int e = tid; e < kPersKS * 64; e += kPersWaves * 64) us[e] = u32x4{0u, 0u, 0u, 0u};
  for (int e = tid; e < depth * bs * nu; e += kPersWaves * 64) {
    const int k = e % nu, b = (e / nu) % bs, jj = e / (nu * bs);
    const int R = min(blockIdx.x + k * G, r - 1);
    P_s[e] = h.P[((size_t)b * depth + jj) * h.ldp + R];
  }
  __syncthreads();

  // state items: two indices of one batch row each, so that all eight waves
  // share the GRU's transcendental arithmetic (one item per thread at one
  // batch row and d_s = 1024)
  constexpr int GE = 2, GU = BS < 2 ? BS : 2;
  const int nit = bs * ds / GE;
  for (int j = 1; j <= depth; ++j) {
    // the thread index, opaque to the compiler once per position: addresses
    // derived from it are recomputed here (a few instructions) instead of being
    // hoisted out of the loop, where they would not fit the registers the
    // resident W2 tiles leave and would be reloaded from scratch every position
    int tj = threadIdx.x;
    __asm__ volatile("" : "+v"(tj));
    const int lane_j = tj & 63, cc_j = lane_j & 15;
    // ---- y_{j-1}: anchor, forced token, or the argmax the previous wait delivered
    if (tj < bs) {
      int y;
      if (j == 1) y = clamp_token(h.anchor[tj], V, h.err);
      else if (h.forced) y = clamp_token(h.forced[(size_t)tj * depth + (j - 2)], V, h.err);
      else y = min(max(key50_id(key_of(tj)), 0), V - 1);
      ys[tj] = y;
    }
    __syncthreads();
    // L_base of this wave's tiles, straight from memory into LDS (no registers
    // held): 16 bytes for (tile q, row b, group g) at (q BS + b) 4 + g.
    // Issued after the barrier above, whose wait would otherwise take in its whole
    // latency, and alongside the GRU's loads: the barrier after the GRU finds
    // both complete.
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int e = i * 64 + lane_j;
      const int t = min(tile0 + min(e / (4 * BS), kPersTiles - 1), NT - 1), bb = min((e >> 2) % BS, bs - 1);
      __builtin_amdgcn_global_load_lds(
          (const void *)(h.Lbase + ((size_t)bb * depth + (j - 1)) * h.ldl + t * 16 + 4 * (e & 3)),
          (void __attribute__((address_space(3))) *)(lbs + ((size_t)wave * NI + i) * 64), 16, 0, 0);
    }
    // ---- S_{j-1} = GRU(E[y_{j-1}], S_{j-2}) in place
    for (int it0 = tid; it0 < nit; it0 += kPersWaves * 64 * GU) {
      // W_hh S_{j-2} + b_hh (stored by the previous position's row owners) and
      // the G rows of GU items, loaded together (past the last one: a copy)
      float2 gh[GU][3], gi[GU][3];
#pragma unroll
      for (int u = 0; u < GU; ++u) {
        const int it = min(it0 + u * kPersWaves * 64, nit - 1);
        const int b = it / (ds / GE), i = (it % (ds / GE)) * GE;
        const float *gb = h.ghbuf + (size_t)((j - 1) & 1) * bs * 3 * ds + (size_t)b * 3 * ds + i;
        const float *gy = h.gtab + (size_t)ys[b] * 3 * ds + i;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          // (8-byte aligned: i and d_s are even)
          const float2 c0 = *(const float2 *)(h.bhh + q * ds + i);  // the gates at j = 1 (S = 0)
          const float2 v = __builtin_bit_cast(float2, ld_slot((const unsigned long long *)(gb + q * ds)));
          gh[u][q] = j > 1 ? v : c0;
          gi[u][q] = *(const float2 *)(gy + q * ds);
        }
      }
#pragma unroll
      for (int u = 0; u < GU; ++u) {
        const int it = it0 + u * kPersWaves * 64;
        if (GU > 1 && it >= nit) break;
        const int b = it / (ds / GE), i = (it % (ds / GE)) * GE;
        float2 s2 = *(const float2 *)(S + (size_t)b * ds + i);
        const float hold[GE] = {s2.x, s2.y};
        float out[GE];
#pragma unroll
        for (int e = 0; e < GE; ++e) {
          auto at = [&](const float2 &v) { return e == 0 ? v.x : v.y; };
          const float rg = sigm(at(gi[u][0]) + at(gh[u][0])), zg = sigm(at(gi[u][1]) + at(gh[u][1]));
          const float ng = tanhf(fmaf(rg, at(gh[u][2]), at(gi[u][2])));
          out[e] = gru_mix(zg, ng, hold[e]);
        }
        s2 = make_float2(out[0], out[1]);
        *(float2 *)(S + (size_t)b * ds + i) = s2;
        if (blockIdx.x == 0 && h.states) *(float2 *)(h.states + ((size_t)b * depth + (j - 1)) * ds + i) = s2;
      }
    }
    __syncthreads();
    // ---- this workgroup's u rows against S_{j-1} into the tagged u slots
    for (int it = wave; it < nu * bs; it += kPersWaves) {
      const int k = it / bs, b = it % bs;
      const int R = blockIdx.x + k * G;
      if (R >= r) continue;  // wave-uniform
      float acc = 0.f;
      for (int c = 0; c < 4; ++c) {
        const int ch = lane + 64 * c;
        if (ch >= nchunk) break;
        float wfl[EPL];
        unpack16<WT>(rows[(size_t)k * nchunk + ch], wfl);
        const float *sb = S + (size_t)b * ds + (size_t)ch * EPL;
        const float4 s0 = *(const float4 *)sb, s1 = *(const float4 *)(sb + 4);
        acc = fmaf(wfl[0], s0.x, acc);
        acc = fmaf(wfl[1], s0.y, acc);
        acc = fmaf(wfl[2], s0.z, acc);
        acc = fmaf(wfl[3], s0.w, acc);
        acc = fmaf(wfl[4], s1.x, acc);
        acc = fmaf(wfl[5], s1.y, acc);
        acc = fmaf(wfl[6], s1.z, acc);
        acc = fmaf(wfl[7], s1.w, acc);
      }
      acc = wave_sum_dpp(acc);
      if (lane == 0) {
        const float x = P_s[((size_t)(j - 1) * bs + b) * nu + k] + acc;
        const float u = x / (1.f + expf(-x));
        st_slot(h.uslot + (size_t)R * kSlotStride + b, ((unsigned long long)j << 32) | __float_as_uint(u));
      }
    }
    // ---- gates of the next position, W_hh S_{j-1} + b_hh (plain device-scope
    // stores), by the waves that do not wait for u (all of them first where
    // every wave will); the stores are waited for before this workgroup publishes its top-1, so "every key slot of position
    // j ready" also means "every gate of position j + 1 stored"
    constexpr int W0 = BS < kPersWaves ? BS : 0;
    if (wave >= W0 && j < depth) {
      float *gh_out = h.ghbuf + (size_t)(j & 1) * bs * 3 * ds;
      for (int k = wave - W0; k < nr; k += kPersWaves - W0) {
        const int R = blockIdx.x + k * G;
        if (R < r || R >= nrows_all) continue;  // wave-uniform
        float accb[BS];
#pragma unroll
        for (int b = 0; b < BS; ++b) accb[b] = 0.f;
        for (int c = 0; c < 4; ++c) {
          const int ch = lane + 64 * c;
          if (ch >= nchunk) break;
          float wfl[EPL];
          unpack16<WT>(rows[(size_t)k * nchunk + ch], wfl);
#pragma unroll
          for (int b = 0; b < BS; ++b) {
            if (b >= bs) break;
            const float *sb = S + (size_t)b * ds + (size_t)ch * EPL;
            const float4 s0 = *(const float4 *)sb, s1 = *(const float4 *)(sb + 4);
            accb[b] = fmaf(wfl[0], s0.x, accb[b]);
            accb[b] = fmaf(wfl[1], s0.y, accb[b]);
            accb[b] = fmaf(wfl[2], s0.z, accb[b]);
            accb[b] = fmaf(wfl[3], s0.w, accb[b]);
            accb[b] = fmaf(wfl[4], s1.x, accb[b]);
            accb[b] = fmaf(wfl[5], s1.y, accb[b]);
            accb[b] = fmaf(wfl[6], s1.z, accb[b]);
            accb[b] = fmaf(wfl[7], s1.w, accb[b]);
          }
        }
        const float bias = h.bhh[R - r];
#pragma unroll
        for (int b = 0; b < BS; ++b) {
          if (b >= bs) break;
          const float acc = wave_sum_dpp(accb[b]);
          if (lane == 0) st_coherent(gh_out + (size_t)b * 3 * ds + (R - r), acc + bias);
        }
      }
    }
    // ---- wait for u (the slots deliver the values)
    if (wave < BS) {
      unsigned long long w[4];
      const bool ok = poll_tagged<BS>(h.uslot, r, bs, wave, (unsigned long long)j, 32, h.abort_flag, h.err, h.poll_limit, w);
      // u goes straight into the B fragments of the logits product: element
      // (b, k) sits at k-step k / 32, lane 16 ((k / 8) mod 4) + column, slot k mod 8,
      // where column b holds the bf16 high part of batch row b's u and column
      // BS + b its low part (u - hi).  One product per tile and k-step then
      // carries both; the two columns are summed after the k loop.
      unsigned short *us16 = (unsigned short *)us;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int e = (4 * wave + q) * 64 + lane_j, k = e / BS, b = e % BS;  // r = 256 lines: 4 units a lane
        if (BS <= 2 || b < bs) {
          const float u = __uint_as_float((uint32_t)(w[q] & 0xffffffffu));
          const __bf16 hi = (__bf16)u, lo = (__bf16)(u - (float)hi);
          const int at = ((k >> 5) * 64 + ((k >> 3) & 3) * 16 + b) * 8 + (k & 7);
          us16[at] = __builtin_bit_cast(unsigned short, hi);
          us16[at + BS * 8] = __builtin_bit_cast(unsigned short, lo);
        }
      }
      if (lane == 0) s_ok[wave] = ok;
    }
    __syncthreads();
    if (!all_ok()) return;
    // ---- logits: u as B fragments against the resident W2
    floatx4 acc[kPersTiles];
#pragma unroll
    for (int q = 0; q < kPersTiles; ++q) acc[q] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < kPersKS; ++s) {
      const bf16x8 xb = __builtin_bit_cast(bf16x8, us[(size_t)s * 64 + lane]);
#pragma unroll
      for (int q = 0; q < kPersRegTiles; ++q)
        acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wf[q][s]), xb, acc[q], 0, 0, 0);
      acc[kPersRegTiles] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
          __builtin_bit_cast(bf16x8, w2s[((size_t)wave * kPersKS + s) * 64 + lane]), xb, acc[kPersRegTiles], 0, 0, 0);
    }
    // lane (g, cc) holds vocabulary ids 16 (tile0 + q) + 4 g + e: column cc < bs
    // adds the low-part column of lane cc + BS (a row shift within 16 lanes).
    // Each tile's four corrected logits are formed, written (DBG) and folded
    // into the running best before the next tile's, so only one tile's values
    // are live at a time.
    const bool rowok = cc < bs;
    {
      // ids grow along (q, e) within a lane, so a strict comparison keeps the
      // smallest id of equal keys; ids past V occur only in the last workgroup
      float bv = -INFINITY, br = 0.f;
      int bi = (tile0 * 16 + 4 * g) < V ? tile0 * 16 + 4 * g : INT_MAX;
      const bool full = (tile0 + kPersTiles) * 16 <= V;
      const size_t orow = (size_t)min(cc, bs - 1) * depth + (j - 1);
#pragma unroll
      for (int q = 0; q < kPersTiles; ++q) {
        const float4 l4 = lbs[wave * NI * 64 + (q * BS + (cc & (BS - 1))) * 4 + g];
        const float lv[4] = {l4.x, l4.y, l4.z, l4.w};
        float val[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int a = __float_as_int(acc[q][e]);
          const int lo = __builtin_amdgcn_update_dpp(0, a, 0x100 + BS, 0xf, 0xf, false);  // lane + BS
          val[e] = lv[e] + (acc[q][e] + __int_as_float(lo));
        }
        // beta > 1: in the place of L_base, which only this wave reads, for the
        // selection after the rollout (whole tiles: the padding keeps its zeros)
        if (DBG && rowok && h.lout && tile0 + q < NT)
          *(float4 *)(h.lout + orow * h.ldl + (tile0 + q) * 16 + 4 * g) = make_float4(val[0], val[1], val[2], val[3]);
        if (DBG && rowok && h.final_logits) {  // output of sampled drafting, debug output otherwise
          float *fl = h.final_logits + orow * V;
          const int n = (tile0 + q) * 16 + 4 * g;
          if ((V & 3) == 0 && n + 4 <= V) {  // rows start 16-byte aligned: four ids per store
            *(float4 *)(fl + n) = make_float4(val[0], val[1], val[2], val[3]);
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (n + e < V) fl[n + e] = val[e];
          }
        }
        Philox4 noise = {{0u, 0u, 0u, 0u}};
        if (SAMPLE) noise = rng_block(h.seed_lo, h.seed_hi, RNG_DRAFT, cc, j, (tile0 + q) * 4 + g);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int n = (tile0 + q) * 16 + 4 * g + e;
          const float key = SAMPLE ? val[e] * h.inv_temp + rng_gumbel(noise.x[e]) : val[e];
          const float ov = (full || n < V) ? order_val(key) : -INFINITY;
          const bool take = ov > bv;
          bv = take ? ov : bv;
          bi = take ? n : bi;
          if (SAMPLE) br = take ? val[e] : br;
        }
      }
      // every lane's best goes to LDS as it is (no cross-row exchange here):
      // the merge below takes 32 candidates per batch row
      __asm__ volatile("" ::: "memory");  // the wave's L_base values are read before they are written over
      if (cc < BS) {
        *best_at(wave, 0, g, cc) = bv;
        *best_at(wave, 1, g, cc) = __int_as_float(bi);
        if (SAMPLE) *best_at(wave, 2, g, cc) = br;
      }
    }
    __builtin_amdgcn_s_waitcnt(0);  // this thread's gate stores are done
    __syncthreads();                // ... and every thread's
    if (wave < (BS + 1) / 2) {
      // wave w merges the 32 candidates (8 waves x 4 row groups) of batch rows
      // 2 w and 2 w + 1, 32 lanes each: rotations within each 16-lane row, then
      // across the two rows of a batch row
      const int bb = 2 * wave + (lane_j >> 5), c = lane_j & 31;
      const bool have = bb < bs;
      const int bc = min(bb, BS - 1);
      float v = have ? *best_at(c >> 2, 0, c & 3, bc) : -INFINITY;
      float raw = (SAMPLE && have) ? *best_at(c >> 2, 2, c & 3, bc) : 0.f;
      int id = have ? __float_as_int(*best_at(c >> 2, 1, c & 3, bc)) : INT_MAX;
      auto step = [&](float ov, int oi, float orw) {
        const bool take = better(ov, oi, v, id);
        v = take ? ov : v;
        id = take ? oi : id;
        if (SAMPLE) raw = take ? orw : raw;
      };
      step(row_ror<8>(v), row_ror<8>(id), SAMPLE ? row_ror<8>(raw) : 0.f);
      step(row_ror<4>(v), row_ror<4>(id), SAMPLE ? row_ror<4>(raw) : 0.f);
      step(row_ror<2>(v), row_ror<2>(id), SAMPLE ? row_ror<2>(raw) : 0.f);
      step(row_ror<1>(v), row_ror<1>(id), SAMPLE ? row_ror<1>(raw) : 0.f);
      // the odd rows take the best of the row before them (DPP row_bcast:15:
      // lane 15 of rows 0 and 2 to every lane of rows 1 and 3), so lanes 16 and
      // 48 hold the workgroup's best of the wave's two batch rows
      step(__int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), 0x142, 0xa, 0xf, false)),
           __builtin_amdgcn_update_dpp(id, id, 0x142, 0xa, 0xf, false),
           SAMPLE ? __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(raw), __float_as_int(raw), 0x142, 0xa, 0xf, false))
                  : 0.f);
      if (c == 16 && have) {
        if (SAMPLE) {  // the raw logit goes out before the key that announces it
          st_coherent(h.praw + ((size_t)(j - 1) * bs + bb) * h.GC + blockIdx.x, raw);
          __builtin_amdgcn_s_waitcnt(0);
        }
        // an empty slice (no valid id) publishes the smallest key
        const unsigned long long key = id == INT_MAX ? 0ull : pack_key50(v, id);
        st_slot(h.kslot + (size_t)blockIdx.x * kSlotStride + bb, ((unsigned long long)j << 50) | key);
      }
    }
    // ---- wait for every workgroup's top-1: the maximum key is y_j.  Also the
    // guard that no workgroup writes the next position's slots while another
    // still polls this position's, so it runs with forced tokens as well.
    // Workgroup 0 reports (y_j, its value) for every position, the last included.
    if (j < depth || blockIdx.x == 0) {
      if (wave < BS) {
        unsigned long long w[4];
        const bool ok = poll_tagged<BS>(h.kslot, G, bs, wave, (unsigned long long)j, 50, h.abort_flag, h.err, h.poll_limit, w);
        unsigned long long best = 0;  // of batch row lane % BS, in lines of this wave
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const unsigned long long k = w[q] & ((1ull << 50) - 1);
          best = k > best ? k : best;
        }
        if (BS == 1) {
          best = wave_max_u64(best);
        } else {
#pragma unroll
          for (int o = 32; o >= BS; o >>= 1) {
            const unsigned long long k = __shfl_xor(best, o, 64);
            best = k > best ? k : best;
          }
        }
        if (lane < BS) s_key[wave][lane] = best;
        if (lane == 0) s_ok[wave] = ok;
      }
      __syncthreads();
      if (!all_ok()) return;
      if (blockIdx.x == 0 && tid < bs && !h.lout) {
        const unsigned long long best = key_of(tid);
        const uint32_t u = (uint32_t)(best >> kKeyIdBits);
        h.topk_ids[(size_t)tid * depth + (j - 1)] = key50_id(best);
        if (!SAMPLE)
          h.topk_vals[(size_t)tid * depth + (j - 1)] = __uint_as_float((u & 0x80000000u) ? (u ^ 0x80000000u) : ~u);
      }
    }
  }
  if (SAMPLE && blockIdx.x == 0) {  // reported values: the drafted tokens' raw logits, from their owners
    __syncthreads();                // (the ids were stored by this workgroup's first threads)
    for (int e = tid; e < depth * bs; e += kPersWaves * 64) {
      const int b = e / depth, jj = e % depth;
      const int id = __hip_atomic_load(h.topk_ids + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const int owner = min(max(id, 0), V - 1) / (16 * kPersWaves * kPersTiles);
      h.topk_vals[e] = ld_coherent(h.praw + ((size_t)jj * bs + b) * h.GC + owner);
    }
  }
}

// Its workgroups, and so best-key slots in use per batch row (never more than
// the GC the workspace has, whose workgroups hold at most as many tiles)
static int persist_groups(const Dims &D) {
  return ((D.V + 15) / 16 + kPersWaves * kPersTiles - 1) / (kPersWaves * kPersTiles);
}

template <int BS>
static const void *persist_fn(bool dbg, bool smp) {
  if (dbg) return smp ? (const void *)head_persist_kernel<BS, true, true> : (const void *)head_persist_kernel<BS, true, false>;
  return smp ? (const void *)head_persist_kernel<BS, false, true> : (const void *)head_persist_kernel<BS, false, false>;
}

// Checks the shapes and the device, and picks the instantiation and its LDS size.
static bool persist_plan(const HeadArgs &h, int n_cu, const void **fn, size_t *lds_out, int *nr_out) {
  const Dims &D = h.D;
  if (!D.bf16 || D.r != kPersKS * 32 || D.bs < 1 || D.bs > kPersMaxBatch || (h.beta > 1 && h.sample) || D.ds % 32 || D.ds > 256 * 8 ||
      D.V >= (1 << kKeyIdBits) || D.B > 64 || !h.uslot || !h.kslot || !h.abort_flag || (h.sample && !h.praw))
    return false;
  const int G = persist_groups(D);
  if (G > h.GC || G > n_cu || G > D.r) return false;  // (the polls cover r = 256 lines)
  const int nr = (D.r + 3 * D.ds + G - 1) / G, BS = D.bs <= 2 ? D.bs : (D.bs <= 4 ? 4 : 8);
  const size_t lds = (size_t)nr * (D.ds / 8) * 16 + sizeof(float) * (size_t)D.bs * D.ds +
                     sizeof(u32x4) * kPersKS * 64 + sizeof(u32x4) * kPersWaves * kPersKS * 64 +
                     sizeof(float4) * kPersWaves * pers_lb_loads(BS) * 64 +
                     sizeof(float) * (size_t)(D.B - 1) * D.bs * ((D.r + G - 1) / G);
  if (lds > 160 * 1024) return false;
  const bool dbg = h.final_logits || h.lout, smp = h.sample != 0;
  *fn = BS == 1 ? persist_fn<1>(dbg, smp) : (BS == 2 ? persist_fn<2>(dbg, smp) : (BS == 4 ? persist_fn<4>(dbg, smp) : persist_fn<8>(dbg, smp)));
  if (hipFuncSetAttribute(*fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  // Every workgroup waits for all others, so the grid must be resident at once:
  // one workgroup per CU at most (its LDS share allows no second), G <= CUs.  An
  // ordinary launch is used (a cooperative one cost ~60 us per step in
  // queue synchronisation); it gets the whole device once the previous kernel
  // on the stream has drained.  Should other work hold CUs, the waits are
  // bounded and end in DEV_BARRIER_TIMEOUT rather than a hang.
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, *fn, kPersWaves * 64, lds) != hipSuccess || per_cu < 1) {
    (void)hipGetLastError();
    return false;
  }
  *lds_out = lds;
  *nr_out = nr;
  return true;
}

// Two persistent launches of different streams must not share the device: each
// could hold CUs that the other's missing workgroups need.  So those of one device
// are ordered by an event: every launch first waits for the last one.  Stream handles are
// not compared: hipStreamPerThread is one handle for a stream of each thread, and a
// destroyed stream's handle may come back (a wait for the stream's own last event costs
// nothing measurable: 822.7 and 822.8 us a step of the Qwen3-8B shape).  Where the
// order cannot be had (`ok` is false), the rollout goes launch by launch, which needs none.
// A captured launch cannot be ordered from here: its graph runs later, and two graphs may
// run at once.  So a capture takes the persistent launch only where programs have had it in their
// graphs all along, at up to kPersCapturedBatch rows and one candidate a position
// (their owner keeps such graphs apart); other steps are captured launch by launch, which
// replays beside anything.
constexpr int kPersCapturedBatch = 4;
namespace {
struct PersistOrder {
  struct Device {
    std::mutex m;
    hipEvent_t done = nullptr;
    bool any = false;   // `done` has been recorded
    bool lost = false;  // a launch went out without its record: nothing can wait for it any more
  };
  static constexpr int kDevices = 64;
  static Device *device() {
    static Device *d = new Device[kDevices];  // (never freed: a stream may outlive static destructors)
    int id = 0;
    if (hipGetDevice(&id) != hipSuccess || id < 0 || id >= kDevices) return nullptr;
    return d + id;
  }
  Device *d = nullptr;
  hipStream_t st;
  std::unique_lock<std::mutex> lock;
  bool captured = false, ok = false;
  explicit PersistOrder(hipStream_t s) : st(s) {
    ok = begin();
    if (!ok) (void)hipGetLastError();
  }
  bool begin() {
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cs) != hipSuccess) return false;
    captured = cs != hipStreamCaptureStatusNone;
    if (captured) return true;
    d = device();
    if (!d) return false;
    lock = std::unique_lock<std::mutex>(d->m);
    if (d->lost) return false;
    if (!d->done && hipEventCreateWithFlags(&d->done, hipEventDisableTiming | hipEventDisableSystemFence) != hipSuccess) {
      d->done = nullptr;
      return false;
    }
    return !d->any || hipStreamWaitEvent(st, d->done, 0) == hipSuccess;
  }
  void launched() {
    if (!d) return;
    d->any = true;
    if (hipEventRecord(d->done, st) == hipSuccess) return;
    (void)hipGetLastError();
    d->lost = true;
  }
};
}  // namespace

// beta > 1: the lists of every position's corrected logits (h.lout); their merge, or
// at branch 1 that of the workgroups' top-1
static void launch_select(const HeadArgs &h, hipStream_t st) {
  const Dims &D = h.D;
  const int depth = D.B - 1;
  int nlist = h.GC;
  if (h.beta > 1) {
    nlist = (D.V + kTopWave - 1) / kTopWave;  // (at most GC: the lists fit the workspace)
    const dim3 grid((nlist + 3) / 4, depth, D.bs);
    if (h.beta <= 2) hipLaunchKernelGGL(head_topb_kernel<2>, grid, dim3(256), 0, st, h, nlist);
    else if (h.beta <= 4) hipLaunchKernelGGL(head_topb_kernel<4>, grid, dim3(256), 0, st, h, nlist);
    else hipLaunchKernelGGL(head_topb_kernel<8>, grid, dim3(256), 0, st, h, nlist);
  }
  hipLaunchKernelGGL(head_merge_kernel, dim3(depth, D.bs), dim3(64), 0, st, h, nlist);
}

bool launch_head_persistent(const HeadArgs &h, int n_cu, hipStream_t st) {
  // Up to eight batch rows, as many as an exchange line has words.  A drafting
  // step of the 4B shape with 256 tokens of context, persistent against launch
  // by launch: 715 and 935 us at 2 rows, 926 and 1057 at 4, 1088 and 1205 at 5,
  // 1214 and 1273 at 8 (sampled 1294 and 1315; four candidates a position 639 and
  // 863 at 1 row, 951 and 1076 at 4, 1229 and 1296 at 8): the gap closes with the rows.
  const void *fn;
  size_t lds;
  int nr;
  HeadArgs a = h;
  a.lout = h.beta > 1 ? const_cast<float *>(h.Lbase) : nullptr;
  if (!persist_plan(a, n_cu, &fn, &lds, &nr)) return false;
  void *args[] = {&a, &nr};
  PersistOrder order(st);
  if (!order.ok || (order.captured && (h.D.bs > kPersCapturedBatch || h.beta > 1))) return false;
  if (hipLaunchKernel(fn, dim3(persist_groups(a.D)), dim3(kPersWaves * 64), args, lds, st) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  order.launched();
  if (a.lout) launch_select(a, st);
  return true;
}

static int logits_mt(const Dims &D) { return D.bs <= 16 ? 1 : (D.bs <= 32 ? 2 : 4); }
static int logits_tiles(const Dims &D) {  // W2 tiles per wave
  const int KS = D.r / (D.bf16 ? 32 : 16);
  return (D.V + 15) / 16 <= kSmallVocabTiles ? 1 : logit_tpw(KS, logits_mt(D));
}
int head_logits_grid(const Dims &D) {
  const int rows = kLogitWaves * logits_tiles(D) * 16;
  return (D.V + rows - 1) / rows;
}

// u of position j (nu tiles) and the next position's hidden gates (ng tiles) from S_j
template <typename WT>
static void launch_rows(const HeadArgs &h, int j, int nu, int ng, hipStream_t st) {
  if (nu + ng <= 0) return;
  const dim3 grid(nu + ng), block(kRowWaves * 64);
  if (h.D.bs <= 16) hipLaunchKernelGGL((head_rows_kernel<WT, 1>), grid, block, 0, st, h, j, nu);
  else if (h.D.bs <= 32) hipLaunchKernelGGL((head_rows_kernel<WT, 2>), grid, block, 0, st, h, j, nu);
  else hipLaunchKernelGGL((head_rows_kernel<WT, 4>), grid, block, 0, st, h, j, nu);
}

// One position's state (and u, unless skip_u)
template <typename WT>
static void launch_state(const HeadArgs &h, int j, hipStream_t st) {
  const Dims &D = h.D;
  if (D.bs <= kFusedBatch) {
    const size_t slds = sizeof(float) * (size_t)D.bs * D.ds;
    const int rows = (h.skip_u ? 0 : D.r) + 3 * D.ds;
    const int gs = min((rows + 2 * kStateWaves - 1) / (2 * kStateWaves), kStateMaxGrid);
    hipLaunchKernelGGL(head_state_kernel<WT>, dim3(gs), dim3(kStateWaves * 64), slds, st, h, j);
    return;
  }
  hipLaunchKernelGGL(head_gru_elem_kernel, dim3((D.ds + 255) / 256, D.bs), dim3(256), 0, st, h, j);
  launch_rows<WT>(h, j, h.skip_u ? 0 : h.w1s_NT, j < D.B - 1 ? h.whh_NT : 0, st);  // the last S has no successor
}
template <typename WT>
static void prepare_state(const HeadArgs &h) {
  if (h.D.bs <= kFusedBatch)
    (void)hipFuncSetAttribute((const void *)head_state_kernel<WT>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)(sizeof(float) * (size_t)h.D.bs * h.D.ds));
}

template <typename WT, int KS, int MT, int TPW>
static void launch_loop(HeadArgs h, hipStream_t st) {
  const Dims &D = h.D;
  const int depth = D.B - 1;
  constexpr size_t lds = sizeof(u32x4) * KS * MT * 64 * XStage<WT>::XF;
  static_assert(lds + 8192 <= 160 * 1024, "logits LDS (u fragments and 6 KB of static LDS)");
  auto logits = head_logits_kernel<WT, KS, MT, TPW>;
  (void)hipFuncSetAttribute((const void *)logits, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  prepare_state<WT>(h);
  h.lout = h.beta > 1 ? const_cast<float *>(h.Lbase) : nullptr;
  for (int j = 1; j <= depth; ++j) {
    launch_state<WT>(h, j, st);
    hipLaunchKernelGGL(logits, dim3(h.GC), dim3(kLogitWaves * 64), lds, st, h, j);
  }
  launch_select(h, st);
}

template <typename WT>
static void launch_states_t(const HeadArgs &h, hipStream_t st) {
  prepare_state<WT>(h);
  for (int j = 1; j <= h.D.B - 1; ++j) launch_state<WT>(h, j, st);
}

hipError_t launch_head_states(const HeadArgs &h, hipStream_t st) {
  if (!h.forced) return hipErrorInvalidValue;
  if (h.D.bf16) launch_states_t<bf16_t>(h, st);
  else launch_states_t<float>(h, st);
  return hipGetLastError();
}

template <typename WT, int KS, int MT>
static void launch_tpw(const HeadArgs &h, hipStream_t st) {
  constexpr int T = logit_tpw(KS, MT);
  if (logits_tiles(h.D) == T) launch_loop<WT, KS, MT, T>(h, st);
  else if constexpr (T != 1) launch_loop<WT, KS, MT, 1>(h, st);
}
template <typename WT, int KS>
static void launch_mt(const HeadArgs &h, hipStream_t st) {
  const int MT = logits_mt(h.D);
  if (MT == 1) launch_tpw<WT, KS, 1>(h, st);
  else if (MT == 2) launch_tpw<WT, KS, 2>(h, st);
  else launch_tpw<WT, KS, 4>(h, st);
}

hipError_t launch_head(const HeadArgs &h, hipStream_t st) {
  const bool bf = h.D.bf16;
  const int KS = h.D.r / (bf ? 32 : 16);
  if (bf) {
    if (KS == 8) launch_mt<bf16_t, 8>(h, st);
    else return hipErrorInvalidValue;
  } else {
    if (KS == 16) launch_mt<float, 16>(h, st);
    else if (KS == 8) launch_mt<float, 8>(h, st);
    else return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace dk

namespace dk {
int head_best_slots() { return kBestSlots; }
}  // namespace dk
