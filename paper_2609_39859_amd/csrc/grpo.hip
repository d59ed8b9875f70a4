// ForkGRPO objective and JustGRPO-Fast position selection (Fork-dLLM paper,
// Section 3.2).
//
// Objective: for each prompt (group g of G rollouts) the advantages
// A_i = (r_i - mean_g) / std_g (std with divisor G; a group with std 0 is
// skipped), the ratios rho_e = exp(log q_new - log q_old) of the rollout's
// fallback-step entries e, the clipped terms min(rho A, clip(rho, 1-eps,
// 1+eps) A), their mean over each rollout's entries, the mean over the
// group's rollouts, and finally the mean over the groups not skipped.  One
// workgroup per group; every sum is a fixed-order reduction, so results are
// bit-reproducible.  The likelihoods themselves come from the teacher-forced
// LM head (gemm_stats target kernels + merge).
//
// Selection: per rollout, the k positions of highest entropy (equal values
// in increasing position): a binary search over the entropies' bits for the
// k-th highest, its counts by ballots.
#include "fork_kernels.h"

#include <math.h>

namespace fork {
namespace {

constexpr int kBatchThreads = 256;

__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
  return x;
}

// Sum over a workgroup of kWaves waves in a fixed order: wave sums, then every
// thread adds them.
template <int kWaves>
__device__ __forceinline__ float block_sum(float x, float* red) {
  x = wave_sum(x);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) red[w] = x;
  __syncthreads();
  float s = 0.f;
#pragma unroll
  for (int k = 0; k < kWaves; ++k) s += red[k];
  __syncthreads();
  return s;
}

// One workgroup of kWaves waves per group, one wave per rollout at a time.  The
// launch is bound by its chain of dependent loads and reductions, so a
// rollout's offsets and first 64 entries are loaded before the advantages,
// which need two reductions over the workgroup, are known.
template <int kWaves>
__global__ __launch_bounds__(64 * kWaves) void grpo_group_kernel(
    int G, int n, const float* __restrict__ rewards, const int32_t* __restrict__ offsets,
    const float* __restrict__ lp_new, const float* __restrict__ lp_old, float eps,
    float* __restrict__ adv, float* __restrict__ ratio, float* __restrict__ term,
    float* __restrict__ rollout_obj, float* __restrict__ group_obj,
    uint8_t* __restrict__ skipped) {
  __shared__ float red[kWaves];
  __shared__ float2 first[kWaves];  // sum of the rewards, whether they differ
  __shared__ float ro[kMaxGroupSize];
  const int g = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const float* r = rewards + (size_t)g * G;

  // the wave's first rollout: offsets and first 64 entries, in flight while
  // the rewards are reduced
  int n0 = 0, n1 = 0;
  float d0 = 0.f;
  if (w < G) {
    const size_t i = (size_t)g * G + w;
    n0 = min(max(offsets[i], 0), n);
    n1 = min(max(offsets[i + 1], n0), n);
    if (n0 + lane < n1) d0 = lp_new[n0 + lane] - lp_old[n0 + lane];
  }
  // Equal rewards have std 0 whatever the rounding of their sum: the mean of 9
  // or of 512 times 0.1 in binary32 is not 0.1.
  float s = 0.f;
  bool equal = true;
  const float r0 = r[0];
  for (int j = tid; j < G; j += 64 * kWaves) {
    s += r[j];
    equal &= r[j] == r0;
  }
  s = wave_sum(s);
  const unsigned long long unequal = __ballot(!equal);
  if (lane == 0) first[w] = make_float2(s, unequal ? 1.f : 0.f);
  __syncthreads();
  float sum = 0.f, any = 0.f;
#pragma unroll
  for (int k = 0; k < kWaves; ++k) {
    const float2 f = first[k];
    sum += f.x;
    any += f.y;
  }
  const float mean = sum / (float)G;
  float q = 0.f;
  for (int j = tid; j < G; j += 64 * kWaves) q += (r[j] - mean) * (r[j] - mean);
  const float sd = sqrtf(block_sum<kWaves>(q, red) / (float)G);
  const bool skip = !(sd > 0.f) || any == 0.f;

  // one wave per rollout, lanes over its entries
  for (int j = w; j < G; j += kWaves) {
    const size_t i = (size_t)g * G + j;
    const float A = skip ? 0.f : (r[j] - mean) / sd;
    if (j != w) {
      n0 = min(max(offsets[i], 0), n);
      n1 = min(max(offsets[i + 1], n0), n);
    }
    float acc = 0.f;
    for (int e = n0 + lane; e < n1; e += 64) {
      const float rho = expf(j == w && e < n0 + 64 ? d0 : lp_new[e] - lp_old[e]);
      const float clipped = fminf(fmaxf(rho, 1.f - eps), 1.f + eps);
      const float tm = fminf(rho * A, clipped * A);
      if (ratio) ratio[e] = rho;
      if (term) term[e] = tm;
      acc += tm;
    }
    acc = wave_sum(acc);
    const float obj = n1 > n0 ? acc / (float)(n1 - n0) : 0.f;
    if (lane == 0) {
      ro[j] = obj;
      if (adv) adv[i] = A;
      if (rollout_obj) rollout_obj[i] = obj;
    }
  }
  __syncthreads();
  float t = 0.f;
  for (int j = tid; j < G; j += 64 * kWaves) t += ro[j];
  const float gsum = block_sum<kWaves>(t, red);
  if (tid == 0) {
    group_obj[g] = skip ? 0.f : gsum / (float)G;
    skipped[g] = skip ? 1 : 0;
  }
}

__global__ __launch_bounds__(kBatchThreads) void grpo_batch_kernel(
    int n_groups, const float* __restrict__ group_obj, const uint8_t* __restrict__ skipped,
    float* __restrict__ J) {
  __shared__ float red[kBatchThreads / 64];
  float s = 0.f, c = 0.f;
  for (int g = threadIdx.x; g < n_groups; g += kBatchThreads)
    if (!skipped[g]) {
      s += group_obj[g];
      c += 1.f;
    }
  const float total = block_sum<kBatchThreads / 64>(s, red);
  const float kept = block_sum<kBatchThreads / 64>(c, red);
  if (threadIdx.x == 0) J[0] = kept > 0.f ? total / kept : 0.f;
}

// The k positions of highest entropy of a rollout, one workgroup of kWaves
// waves per rollout, wave w holding positions [w * 64 N, (w + 1) * 64 N) with
// N per lane.  Entropies become unsigned keys of the same order (+0 and -0
// the same key, 0 for a NaN and past the end), and the k-th highest key is
// built bit by bit from the top: bit b stays set if at least k keys are
// >= the trial value; a trial with exactly k ends the search.  Keys equal to
// the k-th are taken in increasing position.  A NaN is ordered before nothing
// and nothing is ordered before it: it is selected whenever k > 0, and does
// not count towards k.
// Counting a trial is one compare and one bit count per 64 positions, 32
// trials at most, where comparing every position with every other took Lg per
// position: 256 rollouts x 256 positions 8.8 -> 3.9 us, 342 x 495 30 -> 6.3 us,
// 66 x 1387 210 -> 7.6 us, 64 x 16384 25.9 ms -> 22 us.
template <int kWaves, int N>
__global__ __launch_bounds__(64 * kWaves) void top_entropy_kernel(
    int Lg, int k, const float* __restrict__ entropy, uint8_t* __restrict__ sel) {
  __shared__ int cnt[2][kWaves];
  const int lane = threadIdx.x & 63;
  const int w = threadIdx.x >> 6;
  const size_t base = (size_t)blockIdx.x * Lg;
  const int p0 = w * 64 * N + lane;
  uint32_t key[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int p = p0 + 64 * i;
    const float h = p < Lg ? entropy[base + p] + 0.0f : __int_as_float(0x7fc00000);
    const uint32_t b = __float_as_uint(h);
    key[i] = h != h ? 0u : (b & 0x80000000u ? ~b : b | 0x80000000u);
  }
  int parity = 0;
  // keys >= t over the workgroup
  auto count = [&](uint32_t t) {
    int c = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) c += __popcll(__ballot(key[i] >= t));
    if (kWaves == 1) return c;
    if (lane == 0) cnt[parity][w] = c;
    __syncthreads();
    c = 0;
#pragma unroll
    for (int v = 0; v < kWaves; ++v) c += cnt[parity][v];
    parity ^= 1;
    return __builtin_amdgcn_readfirstlane(c);
  };
  uint32_t t = 1;  // every key that counts
  bool all = count(t) <= k, exact = all;
  if (!all) {
    t = 0;
    for (int b = 31; b >= 0 && !exact; --b) {
      const uint32_t trial = t | 1u << b;
      const int c = count(trial);
      if (c >= k) t = trial;
      exact = c == k;
    }
  }
  // keys above t are selected; of the keys equal to t all (exact) or the first
  // `left` in position order
  int left = 0;
  if (!exact) {
    left = k - count(t + 1);
    int before = 0;  // equal keys of the lower waves
    int mine = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) mine += __popcll(__ballot(key[i] == t));
    if (kWaves > 1) {
      if (lane == 0) cnt[parity][w] = mine;
      __syncthreads();
      for (int v = 0; v < w; ++v) before += cnt[parity][v];
    }
    left -= before;
  }
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int p = p0 + 64 * i;
    const bool equal = key[i] == t;
    const unsigned long long eq = __ballot(equal);
    const bool take = key[i] > t || key[i] == 0u ||
                      (equal && (exact || (int)__popcll(eq & ((1ull << lane) - 1ull)) < left));
    left -= (int)__popcll(eq);  // may fall below 0: __popcll is unsigned
    if (p < Lg) sel[base + p] = k > 0 && take ? 1 : 0;
  }
}

}  // namespace

hipError_t launch_grpo_objective(int n_groups, int G, int n, const float* rewards,
                                 const int32_t* offsets, const float* lp_new,
                                 const float* lp_old, float eps, float* adv, float* ratio,
                                 float* term, float* rollout_obj, float* group_obj,
                                 uint8_t* skipped, float* J, hipStream_t stream) {
#define FORK_GROUPS(WAVES)                                                                     \
  hipLaunchKernelGGL(grpo_group_kernel<WAVES>, dim3((unsigned)n_groups), dim3(64 * WAVES), 0, \
                     stream, G, n, rewards, offsets, lp_new, lp_old, eps, adv, ratio, term,    \
                     rollout_obj, group_obj, skipped)
  // Sixteen waves pay while the groups run at once (two such workgroups per CU,
  // 512 in all) and have rollouts for more than four: 16 groups x 16 rollouts x
  // 15 entries 6.2 -> 4.9 us, 64 x 64 x 100 21 -> 10.  Past that the idle waves
  // and the larger reductions cost more (4096 x 16 x 15: 25.5 -> 44.8 us), with
  // 128 rollouts or more from about 2048 groups on (x 300 x 15: 1024 groups 1.4
  // times as fast as four waves, 4096 0.97 times).
  if (n_groups > 0) {
    if (G > 4 && n_groups <= (G >= 128 ? 2048 : 512))
      FORK_GROUPS(16);
    else
      FORK_GROUPS(4);
  }
#undef FORK_GROUPS
  hipLaunchKernelGGL(grpo_batch_kernel, dim3(1), dim3(kBatchThreads), 0, stream, n_groups,
                     group_obj, skipped, J);
  return hipGetLastError();
}

static_assert(kMaxTopEntropyLen == 64 * 16 * 16, "the largest selection workgroup");

hipError_t launch_top_entropy(int R, int Lg, int k, const float* entropy, uint8_t* sel,
                              hipStream_t stream) {
  // a launch holds fewer than 2^32 work-items: more rollouts go in further ones
#define FORK_TOP(WAVES, N)                                                                    \
  for (int r0 = 0; r0 < R;) {                                                                 \
    const int most = (int)(((1LL << 32) - 1) / (64 * WAVES));                                 \
    const int n = R - r0 < most ? R - r0 : most;                                              \
    hipLaunchKernelGGL((top_entropy_kernel<WAVES, N>), dim3((unsigned)n), dim3(64 * WAVES),   \
                       0, stream, Lg, k, entropy + (size_t)r0 * Lg, sel + (size_t)r0 * Lg);   \
    const hipError_t e = hipGetLastError();                                                   \
    if (e != hipSuccess) return e;                                                            \
    r0 += n;                                                                                  \
  }
  // one wave while a lane holds at most 8 keys (no barrier per trial)
  if (Lg <= 64)
    FORK_TOP(1, 1)
  else if (Lg <= 128)
    FORK_TOP(1, 2)
  else if (Lg <= 256)
    FORK_TOP(1, 4)
  else if (Lg <= 512)
    FORK_TOP(1, 8)
  else if (Lg <= 2048)
    FORK_TOP(4, 8)
  else
    FORK_TOP(16, 16)
#undef FORK_TOP
  return hipSuccess;
}

}  // namespace fork
