// Draft-tree construction and greedy acceptance (Sec. 3.1: the longest valid
// prefix plus the target's bonus token).  Integer / compare work only; every
// argmax uses the total order (value desc, id asc) with NaN as -inf, so the
// results are exact and independent of reduction order.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace dk {

// One workgroup per batch row.
__global__ __launch_bounds__(256) void build_tree_kernel(int depth, int beta,
                                                         const int32_t *__restrict__ topk,
                                                         const int32_t *__restrict__ anchor,
                                                         const int32_t *__restrict__ ctx_lens,
                                                         int32_t *tok, int32_t *par, int32_t *dep,
                                                         int32_t *pos, uint8_t *mask) {
  const int b = blockIdx.x;
  const int nn = 1 + depth * beta;
  const int n = ctx_lens[b];
  for (int i = threadIdx.x; i < nn; i += blockDim.x) {
    int t, p, d;
    if (i == 0) {
      t = anchor[b];
      p = -1;
      d = 0;
    } else {
      d = (i - 1) / beta + 1;
      const int rho = (i - 1) % beta;
      t = topk[((size_t)b * depth + (d - 1)) * beta + rho];
      p = d == 1 ? 0 : 1 + (d - 2) * beta;
    }
    tok[(size_t)b * nn + i] = t;
    par[(size_t)b * nn + i] = p;
    dep[(size_t)b * nn + i] = d;
    pos[(size_t)b * nn + i] = n + d;
  }
  if (!mask) return;
  for (int e = threadIdx.x; e < nn * nn; e += blockDim.x) {
    const int i = e / nn, k = e % nn;
    // ancestors of i: i itself, then the spine nodes of depths dep(i)-1 .. 1, then the root
    uint8_t m = 0;
    if (k == i || k == 0) {
      m = 1;
    } else if (i > 0) {
      const int di = (i - 1) / beta + 1;
      const int dk = (k - 1) / beta + 1;
      const bool spine = ((k - 1) % beta) == 0;
      m = (spine && dk < di) ? 1 : 0;
    }
    mask[((size_t)b * nn + i) * nn + k] = m;
  }
}

void launch_build_tree(int bs, int depth, int beta, const int32_t *topk, const int32_t *anchor,
                       const int32_t *ctx_lens, int32_t *tok, int32_t *par, int32_t *dep,
                       int32_t *pos, uint8_t *mask, hipStream_t st) {
  hipLaunchKernelGGL(build_tree_kernel, dim3(bs), dim3(256), 0, st, depth, beta, topk, anchor, ctx_lens,
                     tok, par, dep, pos, mask);
}

// ---------------------------------------------------------------------------
// acceptance: two launches.  (1) the argmax of the rows of nodes that have
// children (the walk can only continue from those), split into vocabulary
// chunks; (2) one workgroup per batch row checks the tree and walks it from
// the root.  When the walk stops on a node without children (a leaf of a
// tree, or the end of a fully accepted chain) the bonus token is that row's
// argmax, which the walk's workgroup scans itself: one row, and only then.
// workspace: [err:int32][pad to 256 B][partials: 64-bit best keys bs*nn*nchunk]
// 32 rows x 61 nodes (15 with children) x 151936 bf16 logits: 146 MB of rows and, where
// the walk ends on a leaf, 0.3 MB more a batch row.  40 us while a workgroup took 8 neighbouring
// node rows (two of them with children) and 43 us for a walk that scanned the leaf
// with 256 threads; now 29 us and 12.
// ---------------------------------------------------------------------------
constexpr int ACH = 4096;  // vocabulary elements per argmax chunk

static size_t acc_part_off() { return 256; }
size_t accept_ws_bytes(int bs, int nn, int V) {
  const int nch = (V + ACH - 1) / ACH;
  return acc_part_off() + (size_t)bs * nn * nch * 8;
}

template <typename LT>
DEVI float ld_logit(const LT *p);
template <>
DEVI float ld_logit<float>(const float *p) {
  return *p;
}
template <>
DEVI float ld_logit<bf16_t>(const bf16_t *p) {
  return to_f32(*p);
}

// 16 bytes of logits as values: 8 bf16 or 4 fp32
template <typename LT>
struct LVec;
template <>
struct LVec<bf16_t> {
  static constexpr int N = 8;
  DEVI static float get(const u32x4 &x, int e) {
    const uint32_t w = x[e >> 1];
    return __uint_as_float((e & 1) ? (w & 0xffff0000u) : (w << 16));
  }
};
template <>
struct LVec<float> {
  static constexpr int N = 4;
  DEVI static float get(const u32x4 &x, int e) { return __uint_as_float(x[e]); }
};

// Best (value, id) of the values of NV 16-byte loads of one row, as the 64-bit
// key of the whole wave: the maximum first (NaN drops out of fmaxf, so it counts
// as -inf), then the smallest id holding it.  Load q holds ids id0 + q * step ..;
// ids from v1 on do not count (unsigned: loads reach past the largest int vocabulary).
template <typename LT, int NV>
DEVI unsigned long long wave_best_key(const u32x4 (&x)[NV], uint32_t id0, uint32_t step, uint32_t v1) {
  constexpr int N = LVec<LT>::N;
  float m[NV], t = -INFINITY;
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    m[q] = -INFINITY;
    const uint32_t id = id0 + q * step;
    if (id + N <= v1) {
#pragma unroll
      for (int e = 0; e < N; ++e) m[q] = fmaxf(m[q], LVec<LT>::get(x[q], e));
    }
    t = fmaxf(t, m[q]);
  }
  const float wm = wave_max(t);
  uint32_t best = INT_MAX;
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    const uint32_t id = id0 + q * step;
    if (id + N <= v1 && m[q] == wm) {
#pragma unroll
      for (int e = N - 1; e >= 0; --e)
        if (order_val(LVec<LT>::get(x[q], e)) == wm) best = min(best, id + (uint32_t)e);
    }
  }
  // (+ 0: a zero's sign is no difference)
  return wave_max_u64(best == INT_MAX ? 0ull : encode_best(wm + 0.f, (int)best));
}
// the same of single values (rows that are not whole 16-byte loads): ids grow
// within a thread, so a strict comparison keeps the smallest id of equal values
template <int NV>
DEVI unsigned long long wave_best_key(const float (&x)[NV], uint32_t id0, uint32_t step, uint32_t v1) {
  float bv = -INFINITY;
  uint32_t bi = id0 < v1 ? id0 : INT_MAX;
#pragma unroll
  for (int q = 0; q < NV; ++q)
    if (id0 + q * step < v1 && x[q] > bv) {  // (a NaN is no more than -inf)
      bv = x[q];
      bi = id0 + q * step;
    }
  return wave_max_u64(bi == INT_MAX ? 0ull : encode_best(bv + 0.f, (int)bi));
}

// Partial argmax over one vocabulary chunk of the rows of nodes that have
// children (the walk scans another row itself if it ends there).  Every
// workgroup lists those rows of its batch row (a few loads that hit the L2) and
// takes entries y, y + gridDim.y, ... of the list, two rows in flight: the
// work is split by rows that are read, wherever they lie among the leaves.
// kVals = 0: every value comes from 16-byte loads (rows are 16-byte aligned when V is
// a multiple of 8 (bf16) or 4 (fp32)); otherwise one value per load, kVals a
// thread (1 where a row has no more than 256).  The first workgroup also clears the
// error word (only the walk, a later launch, raises errors).
//
// Many small rows are bound by the workgroups in flight, so the registers are held
// to 64 (eight workgroups a CU; 16 single values take 100: five), and a workgroup with one
// row loads no second one: chains of 128 rows x 4000 fp32 logits 11.8 us with 80
// registers and two rows always, 7.0 now.  Single values are compared in one pass, not two
// as vectors are: 32 rows x 50257 bf16 logits 22.1 and 13.3 us.
constexpr int kWalkMaxNodes = 1024;

template <typename LT, int kVals>
__global__ __launch_bounds__(256, kVals > 1 ? 4 : 8) void argmax_partial_kernel(int nn, int V, const LT *__restrict__ logits,
                                                             const int32_t *__restrict__ par,
                                                             unsigned long long *__restrict__ part, int32_t *err) {
  constexpr int EV = LVec<LT>::N, VPT = ACH / EV / 256;  // 16-byte loads per thread and row
  const int ch = blockIdx.x, b = blockIdx.z;
  const int nch = gridDim.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if ((ch | blockIdx.y | b) == 0 && tid == 0) *err = 0;
  __shared__ unsigned char s_has[kWalkMaxNodes];
  __shared__ int s_list[kWalkMaxNodes], s_n;
  __shared__ unsigned long long s_key[2][4];
  for (int c = tid; c < nn; c += blockDim.x) s_has[c] = 0;
  __syncthreads();
  for (int c = 1 + tid; c < nn; c += blockDim.x) {  // children come after their parent
    const int p = par[(size_t)b * nn + c];
    if (p >= 0 && p < c) s_has[p] = 1;
  }
  __syncthreads();
  if (wave == 0) {  // the list, in node order
    int n = 0;
    for (int c0 = 0; c0 < nn; c0 += 64) {
      const bool has = c0 + lane < nn && s_has[c0 + lane];
      const unsigned long long mk = __ballot(has);
      if (has) s_list[n + __popcll(mk & ((1ull << lane) - 1))] = c0 + lane;
      n += __popcll(mk);
    }
    if (lane == 0) s_n = n;
  }
  __syncthreads();
  const int n = s_n, ys = gridDim.y;
  const int v0 = ch * ACH, v1 = min(V, v0 + ACH);
  auto finish = [&](int k, int slot, unsigned long long key) {  // list entry k: the four waves' keys
    if (lane == 0) s_key[slot][wave] = key;
    __syncthreads();
    if (tid == 0) {
      unsigned long long o = s_key[slot][0];
#pragma unroll
      for (int w = 1; w < 4; ++w) o = s_key[slot][w] > o ? s_key[slot][w] : o;
      part[((size_t)b * nn + s_list[k]) * nch + ch] = o;
    }
  };
  // entries k, k + ys, ...: the next row's loads go out before this one's
  // values are used; a workgroup with one row loads no other
  auto rows = [&](auto &x, auto load, auto key) {
    int k = blockIdx.y;
    if (k >= n) return;  // uniform
    load(x[0], k);
    if (k + ys >= n) {
      finish(k, 0, key(x[0]));
      return;
    }
    for (; k < n; k += 2 * ys) {  // clamped within the list: every load valid
      load(x[1], k + ys);
      finish(k, 0, key(x[0]));
      load(x[0], k + 2 * ys);
      if (k + ys < n) finish(k + ys, 1, key(x[1]));
    }
  };
  auto row = [&](int k) { return logits + ((size_t)b * nn + s_list[min(k, n - 1)]) * V; };
  if constexpr (kVals == 0) {
    u32x4 x[2][VPT];
    const int id0 = v0 + tid * EV;
    auto load = [&](u32x4 (&y)[VPT], int k) {
      const LT *r = row(k);
#pragma unroll
      for (int q = 0; q < VPT; ++q) y[q] = __builtin_nontemporal_load((const u32x4 *)(r + min(id0 + q * 256 * EV, V - EV)));
    };
    rows(x, load, [&](const u32x4 (&y)[VPT]) { return wave_best_key<LT>(y, id0, 256 * EV, v1); });
  } else {
    LT x[2][kVals];
    auto load = [&](LT (&y)[kVals], int k) {
      const LT *r = row(k);
#pragma unroll
      for (int q = 0; q < kVals; ++q) y[q] = r[min(v0 + tid + q * 256, v1 - 1)];
    };
    rows(x, load, [&](const LT (&y)[kVals]) {
      float f[kVals];
#pragma unroll
      for (int q = 0; q < kVals; ++q) f[q] = to_f32(y[q]);
      return wave_best_key(f, v0 + tid, 256, v1);
    });
  }
}

// The walk of one batch row.  Every table the walk needs is formed in
// parallel first, with all of its memory reads in flight together: which nodes
// have children (the rows argmax_partial_kernel took), each such node's argmax
// R from its chunk partials (a wave per node, four nodes per pass), and the
// first child of each node whose token is that R.  The walk from the root is
// then a chase through LDS.  Only if it stops on a node without children (a
// leaf of a tree, or the end of a fully accepted chain) is that row's argmax
// needed, which the workgroup scans itself: with 8 waves, and 16 where the row is longer
// than one and a half passes of 8 (120 KB in 16-byte loads).  16 waves against 8 for one
// chain: 9.5 and 7.3 us at 32000 bf16 logits, 11.9 and 11.8 at 128256 (a tree 10.9 and
// 12.3); for 512 chains of 100 logits 11.8 and 7.5.
constexpr int kWalkLoads = 10;  // in flight a thread
template <typename LT, int kWalkThreads>
__global__ __launch_bounds__(kWalkThreads) void accept_walk_kernel(int nn, int V, int B,
                                                                   const int32_t *__restrict__ tok,
                                                                   const int32_t *__restrict__ par,
                                                                   const unsigned long long *__restrict__ part,
                                                                   const LT *__restrict__ logits, int32_t *acc_len,
                                                                   int32_t *acc_nodes, int32_t *out_tok,
                                                                   int32_t *err) {
  constexpr int kWaves = kWalkThreads / 64;
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nch = (V + ACH - 1) / ACH;
  __shared__ unsigned long long s_key[kWaves];
  __shared__ int s_R[kWalkMaxNodes], s_next[kWalkMaxNodes];
  __shared__ unsigned char s_kid[kWalkMaxNodes];
  const int32_t *pr = par + (size_t)b * nn, *tk = tok + (size_t)b * nn;
  for (int c = tid; c < nn; c += blockDim.x) {
    s_kid[c] = 0;
    s_next[c] = INT_MAX;
  }
  __syncthreads();
  // the tree: node 0 is the root, every other node's parent comes before it
  for (int c = tid; c < nn; c += blockDim.x) {
    const int p = pr[c];
    if (!((c == 0) ? (p == -1) : (p >= 0 && p < c))) raise_error(err, DEV_BAD_TREE);
    if (c > 0 && p >= 0 && p < c) s_kid[p] = 1;
  }
  __syncthreads();
  // R of every node with children: wave w takes nodes w + 16 q (+ 64 per pass),
  // lanes over the vocabulary chunks
  for (int c0 = wave; c0 < nn; c0 += 4 * kWaves) {
    unsigned long long best[4] = {0ull, 0ull, 0ull, 0ull};
    for (int k0 = 0; k0 < nch; k0 += 64) {
      unsigned long long x[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {  // clamped: every load valid, all in flight together
        const int c = min(c0 + kWaves * q, nn - 1), k = min(k0 + lane, nch - 1);
        x[q] = part[((size_t)b * nn + c) * nch + k];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) best[q] = x[q] > best[q] ? x[q] : best[q];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const unsigned long long o = wave_max_u64(best[q]);
      const int c = c0 + kWaves * q;  // (a row without children has no partials: its R is never used)
      if (lane == 0 && c < nn) s_R[c] = s_kid[c] ? decode_best_id(o, V) : -1;
    }
  }
  __syncthreads();
  // each node's child carrying R (children have distinct tokens; the first one)
  for (int c = 1 + tid; c < nn; c += blockDim.x) {
    const int p = pr[c];
    if (p >= 0 && p < c && tk[c] == s_R[p]) atomicMin(&s_next[p], c);
  }
  __syncthreads();
  // the walk (every thread follows it)
  int cur = 0, a = 0, R = 0;
  bool leaf = false;
  while (true) {
    if (!s_kid[cur]) {
      leaf = true;
      break;
    }
    R = s_R[cur];
    if (a >= B - 1) break;  // walk bound
    const int nx = s_next[cur];
    if (nx == INT_MAX || nx <= cur) break;
    if (tid == 0) {
      acc_nodes[(size_t)b * (B - 1) + a] = nx;
      out_tok[(size_t)b * B + a] = R;
    }
    ++a;
    cur = nx;
  }
  if (leaf) {  // the bonus token: the argmax of this row, scanned here
    const LT *row = logits + ((size_t)b * nn + cur) * V;
    constexpr int EV = LVec<LT>::N, U = kWalkLoads;
    unsigned long long best = 0ull;
    if (V % EV == 0) {  // 16-byte rows: U loads of EV values per thread in flight
      for (uint32_t g0 = 0; g0 < (uint32_t)V; g0 += kWalkThreads * U * EV) {
        u32x4 x[U];
        const uint32_t id0 = g0 + tid * EV;
#pragma unroll
        for (int q = 0; q < U; ++q) x[q] = *(const u32x4 *)(row + min(id0 + q * kWalkThreads * EV, (uint32_t)(V - EV)));
        const unsigned long long o = wave_best_key<LT>(x, id0, kWalkThreads * EV, V);
        best = o > best ? o : best;
      }
    } else {
      for (uint32_t g0 = 0; g0 < (uint32_t)V; g0 += kWalkThreads * U) {
        float x[U];
        const uint32_t id0 = g0 + tid;
#pragma unroll
        for (int q = 0; q < U; ++q) x[q] = ld_logit<LT>(row + min(id0 + q * kWalkThreads, (uint32_t)(V - 1)));
        const unsigned long long o = wave_best_key(x, id0, kWalkThreads, V);
        best = o > best ? o : best;
      }
    }
    if (lane == 0) s_key[wave] = best;
    __syncthreads();
    for (int w = 0; w < kWaves; ++w) best = s_key[w] > best ? s_key[w] : best;
    R = decode_best_id(best, V);
  }
  if (tid == 0) {
    acc_len[b] = a;
    out_tok[(size_t)b * B + a] = R;
  }
  for (int q = a + 1 + tid; q < B; q += blockDim.x) out_tok[(size_t)b * B + q] = -1;
  for (int q = a + tid; q < B - 1; q += blockDim.x) acc_nodes[(size_t)b * (B - 1) + q] = -1;
}

size_t accept_part_entries(int bs, int nn, int V) { return (size_t)bs * nn * ((V + ACH - 1) / ACH); }

void launch_accept(int bs, int nn, int V, int B, const int32_t *tok, const int32_t *par,
                   const void *logits, bool bf16, int32_t *acc_len, int32_t *acc_nodes,
                   int32_t *out_tok, void *ws, hipStream_t st) {
  unsigned char *w = (unsigned char *)ws;
  launch_accept_parts(bs, nn, V, B, tok, par, logits, bf16, acc_len, acc_nodes, out_tok, w + acc_part_off(),
                      (int32_t *)w, st);
}

void launch_accept_parts(int bs, int nn, int V, int B, const int32_t *tok, const int32_t *par,
                         const void *logits, bool bf16, int32_t *acc_len, int32_t *acc_nodes,
                         int32_t *out_tok, void *part, int32_t *err, hipStream_t st) {
  const int nch = (V + ACH - 1) / ACH;
  // as many workgroups as the chip holds (8 a CU, 5 of those with 16 single values a thread):
  // a row each while there are few, several each for large batches.  Where one a chunk
  // and batch row are more than that, two, of half the rows each, while the last
  // round weighs (64 rows x 151936 bf16 logits 65 us with one, 56 with two; 300 x
  // 100000 158 and 161).  Not for fp32 rows in 16-byte loads (102 and 114).
  const bool wide = V % (bf16 ? 8 : 4) == 0;
  const long fit = 256L * (wide || V <= 256 ? 8 : 5), one = (long)nch * bs;
  const int ys = (int)std::min((long)nn, one <= fit ? fit / one : one <= 3 * fit && (bf16 || !wide) ? 2L : 1L);
  const dim3 grid(nch, ys, bs);
  auto go = [&](auto *lg) {
    using LT = std::remove_cv_t<std::remove_pointer_t<decltype(lg)>>;
    unsigned long long *p = (unsigned long long *)part;
    auto argmax = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, nn, V, lg, par, p, err); };
    if (wide) argmax(argmax_partial_kernel<LT, 0>);
    else if (V <= 256) argmax(argmax_partial_kernel<LT, 1>);
    else argmax(argmax_partial_kernel<LT, ACH / 256>);
    auto walk = [&](auto kernel, int threads) {
      hipLaunchKernelGGL(kernel, dim3(bs), dim3(threads), 0, st, nn, V, B, tok, par, (const unsigned long long *)p, lg,
                         acc_len, acc_nodes, out_tok, err);
    };
    if (2L * V <= 3L * 512 * kWalkLoads * (wide ? LVec<LT>::N : 1)) walk(accept_walk_kernel<LT, 512>, 512);
    else walk(accept_walk_kernel<LT, 1024>, 1024);
  };
  if (bf16) go((const bf16_t *)logits);
  else go((const float *)logits);
}

}  // namespace dk
