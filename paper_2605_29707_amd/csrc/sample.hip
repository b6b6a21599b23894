// Speculative-sampling verification of a drafted chain at temperature T
// (Sec. 3.1: the standard speculative verification rule; Fig. 3: draft tokens
// sampled from the final logits).  For batch row b and depth j = 1..B-1 the
// draft token x_j was drawn from q_j = softmax(draft_j / T); the target's
// distribution there is p_j = softmax(target_{j-1} / T) (target row m follows
// node m).  x_j is accepted iff u_j q_j(x_j) < p_j(x_j), i.e. with probability
// min(1, p_j / q_j), u_j the acceptance uniform of (b, j).  At the first
// rejection j the bonus token is a draw from max(0, p_j - q_j); if all B-1 are
// accepted it is a draw from p_B.  Draws use the Philox streams of philox.h
// and the Gumbel-max form.
//
// Three launches: per (row, vocabulary chunk) log-sum-exp partials of every
// target and draft row; per (batch row, chunk) the acceptance decisions, formed
// by every workgroup for itself (15 ratios from a few KB of partials in the L2,
// cheaper than a launch), and the chunk's best bonus candidate at the depth where
// the row stops; one wave per batch row for the bonus token.  8 rows of
// 151936 bf16 and fp32 logits: 34 us for the partials with single loads, 72 for
// the candidates of every possible depth, 26 for a walk of one depth after
// another and 5 for clearing the error word; now 17 + 23 + 5.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "philox.h"

namespace dk {

constexpr int kVsChunk = 4096;  // vocabulary ids per workgroup
constexpr int kVsThreads = 256;
constexpr int kVsPer = kVsChunk / kVsThreads;  // 16 ids per thread, 4 groups of 4

template <typename LT>
DEVI float ld_logit(const LT *p, size_t i);
template <>
DEVI float ld_logit<float>(const float *p, size_t i) { return p[i]; }
template <>
DEVI float ld_logit<bf16_t>(const bf16_t *p, size_t i) { return to_f32(p[i]); }

// block-wide max / sum over kVsThreads threads
DEVI float block_max(float v, float *red) {
  v = wave_max(v);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) red[wave] = v;
  __syncthreads();
  float r = red[0];
#pragma unroll
  for (int w = 1; w < kVsThreads / 64; ++w) r = fmaxf(r, red[w]);
  __syncthreads();
  return r;
}
DEVI float block_sum(float v, float *red) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) red[wave] = v;
  __syncthreads();
  float r = 0.f;
#pragma unroll
  for (int w = 0; w < kVsThreads / 64; ++w) r += red[w];
  __syncthreads();
  return r;
}

// Row r of the 2B-1 softmax rows of batch row b: r < B the target row r,
// r >= B the draft row of depth r - B + 1.
template <typename LT>
DEVI float row_logit(const LT *target, const float *draft, int b, int r, int B, int V, int v) {
  return r < B ? ld_logit<LT>(target, ((size_t)b * B + r) * V + v)
               : draft[((size_t)b * (B - 1) + (r - B)) * V + v];
}

// 16 bytes of logits as values: 8 bf16 or 4 fp32
template <typename LT>
struct VsVec;
template <>
struct VsVec<bf16_t> {
  static constexpr int N = 8;
  DEVI static float get(const u32x4 &x, int e) {
    const uint32_t w = x[e >> 1];
    return __uint_as_float((e & 1) ? (w & 0xffff0000u) : (w << 16));
  }
};
template <>
struct VsVec<float> {
  static constexpr int N = 4;
  DEVI static float get(const u32x4 &x, int e) { return __uint_as_float(x[e]); }
};

constexpr float kVsLog2e = 1.4426950408889634f;

// kVsPer values of a row's chunk c, this thread's; -inf past the end.  WIDE:
// 16-byte loads (whole vectors: V a multiple of VsVec<LT>::N, aligned rows).
template <typename LT, bool WIDE>
DEVI void load_chunk(const LT *row, int c, int V, float (&z)[kVsPer]) {
  constexpr int N = VsVec<LT>::N;
  if constexpr (WIDE) {
    u32x4 x[kVsPer / N];
#pragma unroll
    for (int q = 0; q < kVsPer / N; ++q)  // unconditional loads at clamped ids, masked afterwards
      x[q] = *(const u32x4 *)(row + min(c * kVsChunk + (q * kVsThreads + (int)threadIdx.x) * N, V - N));
#pragma unroll
    for (int q = 0; q < kVsPer / N; ++q) {
      const bool in = c * kVsChunk + (q * kVsThreads + (int)threadIdx.x) * N < V;
#pragma unroll
      for (int e = 0; e < N; ++e) z[q * N + e] = in ? VsVec<LT>::get(x[q], e) : -INFINITY;
    }
  } else {
#pragma unroll
    for (int q = 0; q < kVsPer; ++q) {
      const int v = c * kVsChunk + q * kVsThreads + threadIdx.x;
      const float raw = ld_logit<LT>(row, min(v, V - 1));
      z[q] = v < V ? raw : -INFINITY;
    }
  }
}

// (1) max and sum of exp over one vocabulary chunk of one row (NaN as -inf).
// Bound by the logits' bytes: 16-byte loads and one exp2 instruction a value,
// of the difference to the maximum first, since a chunk may hold nothing but a
// mask of the type's lowest value, whose multiple is infinite.  The first
// workgroup clears the error word (the next launch raises errors).
template <typename LT, bool WIDE>
__global__ __launch_bounds__(kVsThreads) void vs_lse_partial_kernel(const LT *__restrict__ target,
                                                                    const float *__restrict__ draft, int B, int V,
                                                                    float inv_t, int nch, float2 *__restrict__ part,
                                                                    int32_t *err) {
  const int c = blockIdx.x, r = blockIdx.y, b = blockIdx.z;
  if ((c | r | b) == 0 && threadIdx.x == 0) *err = 0;
  __shared__ float red[kVsThreads / 64];
  float z[kVsPer];
  if (r < B) load_chunk<LT, WIDE>(target + ((size_t)b * B + r) * V, c, V, z);  // workgroup-uniform
  else load_chunk<float, WIDE>(draft + ((size_t)b * (B - 1) + (r - B)) * V, c, V, z);
  float m = -INFINITY;
#pragma unroll
  for (int q = 0; q < kVsPer; ++q) {
    z[q] = order_val(z[q] * inv_t);
    m = fmaxf(m, z[q]);
  }
  m = block_max(m, red);
  const float ref = m == -INFINITY ? 0.f : m;  // (every term is then 0)
  float s = 0.f;
#pragma unroll
  for (int q = 0; q < kVsPer; ++q) s += __builtin_amdgcn_exp2f((z[q] - ref) * kVsLog2e);
  s = block_sum(s, red);
  if (threadIdx.x == 0) part[((size_t)b * (2 * B - 1) + r) * nch + c] = make_float2(m, s);
}

// log-sum-exp of one row from its chunk partials (one wave; lanes over chunks)
DEVI float row_lse(const float2 *__restrict__ part, int nch) {
  const int lane = threadIdx.x & 63;
  float m = -INFINITY;
  for (int c = lane; c < nch; c += 64) m = fmaxf(m, part[c].x);
  m = wave_max(m);
  float s = 0.f;
  for (int c = lane; c < nch; c += 64) {
    const float2 t = part[c];
    s += t.x == -INFINITY ? 0.f : t.y * expf(t.x - m);
  }
  s = wave_sum(s);
  return m + logf(s);
}

// (2) The row's acceptance decisions (wave w: depths w + 1, w + 5, ...), then
// the best bonus candidate of chunk c at its stop depth.  The workgroup of
// chunk 0 writes the accepted tokens and `stop` (1 .. B) for the last launch.
template <typename LT>
__global__ __launch_bounds__(kVsThreads) void vs_bonus_partial_kernel(
    const int32_t *__restrict__ node_token, const LT *__restrict__ target, const float *__restrict__ draft, int B,
    int V, float inv_t, int nch, const float2 *__restrict__ part, uint32_t seed_lo, uint32_t seed_hi,
    unsigned long long *__restrict__ bkey, int32_t *__restrict__ stops, int32_t *__restrict__ accept_len,
    int32_t *__restrict__ accepted_nodes, int32_t *__restrict__ out_tokens, int32_t *err) {
  const int c = blockIdx.x, b = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  __shared__ float s_lse[2][64];  // of target row j - 1 and draft row j - 1, by depth j (B <= 64)
  __shared__ unsigned char s_no[64];
  __shared__ unsigned long long red[kVsThreads / 64];
  const float2 *prow = part + (size_t)b * (2 * B - 1) * nch;
  for (int j = 1 + wave; j <= B; j += kVsThreads / 64) {
    const float lt = row_lse(prow + (size_t)(j - 1) * nch, nch);
    const float ld = j < B ? row_lse(prow + (size_t)(B + j - 1) * nch, nch) : 0.f;
    if (lane == 0) {
      s_lse[0][j - 1] = lt;
      s_lse[1][j - 1] = ld;
      bool no = true;  // depth B: every draft accepted, nothing more to accept
      if (j < B) {
        const int x = node_token[(size_t)b * B + j];
        if (x >= 0 && x < V) {
          const float p =
              expf(order_val(ld_logit<LT>(target, ((size_t)b * B + (j - 1)) * V + x) * inv_t) - lt);
          const float q = expf(order_val(draft[((size_t)b * (B - 1) + (j - 1)) * V + x] * inv_t) - ld);
          const float u = rng_uniform(rng_block(seed_lo, seed_hi, RNG_ACCEPT, b, j, 0).x[0]);
          no = !(u * q < p);
        }
      }
      s_no[j - 1] = no;
    }
  }
  __syncthreads();
  int stop = 1;  // the first depth that is not accepted
  while (!s_no[stop - 1]) ++stop;  // ends at B
  const int a = stop - 1;
  if (c == 0) {
    for (int i = tid; i < B; i += kVsThreads) {
      const int x = i + 1 < B ? node_token[(size_t)b * B + i + 1] : 0;
      if (i < B - 1) accepted_nodes[(size_t)b * (B - 1) + i] = i < a ? i + 1 : -1;
      if (i != a) out_tokens[(size_t)b * B + i] = i < a ? x : -1;  // place a is the last launch's
      if (i == a && i + 1 < B && (x < 0 || x >= V)) raise_error(err, DEV_BAD_TOKEN);
    }
    if (tid == 0) {
      accept_len[b] = a;
      stops[b] = stop;
    }
  }
  const float lt = s_lse[0][stop - 1], ld = s_lse[1][stop - 1];
  const int j = stop;
  float bv = -INFINITY;
  int bi = INT_MAX;
  // all loads first, at clamped ids (masked afterwards), so none waits on another
  float tl[kVsPer], dl[kVsPer];
  const int jd = j < B ? j - 1 : B - 2;  // the last depth has no draft row (its q is 0)
#pragma unroll
  for (int q = 0; q < kVsPer; ++q) {
    const int v = min(c * kVsChunk + ((q / 4) * kVsThreads + tid) * 4 + (q % 4), V - 1);
    tl[q] = row_logit<LT>(target, draft, b, j - 1, B, V, v);
    dl[q] = draft[((size_t)b * (B - 1) + jd) * V + v];
  }
#pragma unroll
  for (int grp = 0; grp < kVsPer / 4; ++grp) {
    const int v0 = c * kVsChunk + (grp * kVsThreads + tid) * 4;  // four consecutive ids
    const Philox4 noise = rng_block(seed_lo, seed_hi, RNG_BONUS, b, j, v0 / 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int v = v0 + e;
      const float p = expf(order_val(tl[grp * 4 + e] * inv_t) - lt);
      const float q = j < B ? expf(order_val(dl[grp * 4 + e] * inv_t) - ld) : 0.f;
      const float w = v < V ? fmaxf(p - q, 0.f) : 0.f;
      if (w > 0.f) {
        const float key = logf(w) + rng_gumbel(noise.x[e]);
        if (better(key, v, bv, bi)) {
          bv = key;
          bi = v;
        }
      }
    }
  }
  wave_best(bv, bi);
  if (lane == 0) red[wave] = bi == INT_MAX ? 0ull : encode_best(bv, bi);
  __syncthreads();
  if (tid == 0) {
    unsigned long long k = red[0];
#pragma unroll
    for (int w = 1; w < kVsThreads / 64; ++w) k = red[w] > k ? red[w] : k;
    bkey[(size_t)b * nch + c] = k;
  }
}

// (3) the bonus token: the best candidate over the chunks, one wave per batch row
__global__ __launch_bounds__(64) void vs_bonus_kernel(int B, int V, int nch,
                                                      const unsigned long long *__restrict__ bkey,
                                                      const int32_t *__restrict__ stops,
                                                      int32_t *__restrict__ out_tokens) {
  const int b = blockIdx.x, lane = threadIdx.x;
  const int a = stops[b] - 1;
  unsigned long long k = 0ull;
  for (int c = lane; c < nch; c += 64) {
    const unsigned long long t = bkey[(size_t)b * nch + c];
    k = t > k ? t : k;
  }
  k = wave_max_u64(k);
  if (lane == 0) out_tokens[(size_t)b * B + a] = k ? decode_best_id(k, V) : 0;
}

int vs_nchunks(int V) { return (V + kVsChunk - 1) / kVsChunk; }

// [error word, padded to 256][log-sum-exp partials][best keys bs * nch][stop depths bs]
size_t vs_ws_bytes(int bs, int B, int V) {
  const size_t nch = vs_nchunks(V);
  return 256 + (((size_t)bs * (2 * B - 1) * nch * sizeof(float2) + 255) & ~(size_t)255) + (size_t)bs * nch * 8 +
         (size_t)bs * 4;
}

void launch_verify_sample(int bs, int B, int V, const int32_t *node_token, const void *target, bool bf16,
                          const float *draft, float temperature, uint64_t seed, int32_t *accept_len,
                          int32_t *accepted_nodes, int32_t *out_tokens, void *ws, hipStream_t st) {
  const int nch = vs_nchunks(V);
  int32_t *err = (int32_t *)ws;
  float2 *part = (float2 *)((char *)ws + 256);
  unsigned long long *bkey =
      (unsigned long long *)((char *)part + (((size_t)bs * (2 * B - 1) * nch * sizeof(float2) + 255) & ~(size_t)255));
  int32_t *stops = (int32_t *)(bkey + (size_t)bs * nch);
  const float inv_t = 1.0f / temperature;
  const uint32_t slo = (uint32_t)seed, shi = (uint32_t)(seed >> 32);
  auto go = [&](auto *t) {
    using LT = std::remove_cv_t<std::remove_pointer_t<decltype(t)>>;
    // 16-byte loads where every row of both tensors is whole, aligned vectors
    const bool wide = V % VsVec<LT>::N == 0 && V % VsVec<float>::N == 0 && ((uintptr_t)t & 15) == 0 &&
                      ((uintptr_t)draft & 15) == 0;
    const dim3 grid(nch, 2 * B - 1, bs), block(kVsThreads);
    if (wide)
      hipLaunchKernelGGL((vs_lse_partial_kernel<LT, true>), grid, block, 0, st, t, draft, B, V, inv_t, nch, part, err);
    else
      hipLaunchKernelGGL((vs_lse_partial_kernel<LT, false>), grid, block, 0, st, t, draft, B, V, inv_t, nch, part,
                         err);
    hipLaunchKernelGGL(vs_bonus_partial_kernel<LT>, dim3(nch, bs), block, 0, st, node_token, t, draft, B, V, inv_t,
                       nch, part, slo, shi, bkey, stops, accept_len, accepted_nodes, out_tokens, err);
  };
  if (bf16) go((const bf16_t *)target);
  else go((const float *)target);
  hipLaunchKernelGGL(vs_bonus_kernel, dim3(bs), dim3(64), 0, st, B, V, nch, bkey, stops, out_tokens);
}

// Philox words for explicit counters (tests and callers that need the same draws)
__global__ void philox_words_kernel(const uint32_t *__restrict__ ctr, uint32_t k0, uint32_t k1, uint32_t *__restrict__ out,
                                    int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const Philox4 r = philox4x32_10(ctr[4 * i], ctr[4 * i + 1], ctr[4 * i + 2], ctr[4 * i + 3], k0, k1);
#pragma unroll
  for (int e = 0; e < 4; ++e) out[4 * i + e] = r.x[e];
}

void launch_philox_words(const uint32_t *ctr, uint64_t key, uint32_t *out, int n, hipStream_t st) {
  if (n <= 0) return;
  hipLaunchKernelGGL(philox_words_kernel, dim3((n + 255) / 256), dim3(256), 0, st, ctr, (uint32_t)key,
                     (uint32_t)(key >> 32), out, n);
}

}  // namespace dk
