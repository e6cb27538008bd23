// Reward post-processing ahead of GAE (appendix "Reward Weights": game time
// weighting, team spirit, zero sum; Table "Hyperparameters": rewards are
// normalised by a running estimate of their standard deviation).
//
// The ten heroes of a game are ten adjacent segments of the [L, S] layout,
// so one thread owns one (step, game): it reads 10 shaped rewards, 10
// outcomes and the game time (84 bytes, 8-byte loads; a wave reads 64
// consecutive games) and forms the ten processed rewards z in registers.
// (Staging the 10-wide rows through LDS for 16-byte coalesced loads measured
// slower: the block-wide barriers serialise the tiles.)
// The normalisation needs the variance of every z before any output can be
// written, hence two launches (short calls are bound by their number: L = 256,
// 13 games, 30.6 us with GAE and the cut when a third launch merged the
// summaries, 27.0 without it):
//  1. reward_stats: z per (step, game); per-block (count, mean, M2) in fp64,
//     merged in a fixed order; also keeps the running summary as it was;
//  2. reward_apply: every block merges the block summaries into that running
//     summary, in the same fixed order (at most 24 KB from L2: 9.1 us at L = 256,
//     1152 games, against 4.0 + 7.2 as two launches), and recomputes z
//     (cheaper than a round trip of z through HBM: the same 84 bytes are read
//     either way) for r = z / sqrt(var + eps); block 0 writes the new running
//     summary.
// 20.8 bytes move per (step, segment) against 12.4 that the operation needs
// at least (inputs once, output once): the inputs are read twice.
#include "common.h"

namespace o5 {

constexpr int kHeroes = 10;       // two teams of five
constexpr int kRwThreads = 256;
constexpr int kRwMaxBlocks = 1024;

struct Summary {
  double n, mean, m2;  // count, mean, sum of squared deviations
};

// Pairwise merge of two summaries of disjoint sets (Chan, Golub, LeVeque).
__device__ __forceinline__ Summary merge(const Summary& a, const Summary& b) {
  const double n = a.n + b.n;
  if (n == 0.0) return a;
  const double d = b.mean - a.mean;
  return {n, a.mean + d * (b.n / n), a.m2 + b.m2 + d * d * (a.n * b.n / n)};
}

struct RewardConsts {
  float tau;
  float log2_base_per_minute;  // log2(decay_base) / decay_minutes
};

// The ten processed rewards z of one (step, game) from its raw rewards rho
// (time weight already applied, outcome added).
__device__ __forceinline__ void mix_game(const float (&rho)[kHeroes], float tau, float (&z)[kHeroes]) {
  const float ma = 0.2f * (rho[0] + rho[1] + rho[2] + rho[3] + rho[4]);
  const float mb = 0.2f * (rho[5] + rho[6] + rho[7] + rho[8] + rho[9]);
  const float keep = 1.0f - tau;
  // team spirit mixes in the own team's mean; zero sum takes the enemies'
  // mean (team spirit leaves a team's mean unchanged)
  const float off_a = tau * ma - mb, off_b = tau * mb - ma;
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    z[k] = keep * rho[k] + off_a;
    z[5 + k] = keep * rho[5 + k] + off_b;
  }
}

// The ten processed rewards of game g at step t (item i = t * G + g), read
// with 8-byte loads (a wave covers 64 consecutive games, 2.5 KB per array).
__device__ __forceinline__ void shape_game(const float* __restrict__ shaped, const float* __restrict__ outcome,
                                           const float* __restrict__ game_time, size_t i, const RewardConsts& c,
                                           float (&z)[kHeroes]) {
  const float w = exp2f(c.log2_base_per_minute * game_time[i]);
  const float2* s2 = reinterpret_cast<const float2*>(shaped + i * kHeroes);
  float rho[kHeroes];
#pragma unroll
  for (int k = 0; k < kHeroes / 2; ++k) {
    const float2 v = s2[k];
    rho[2 * k] = v.x * w;
    rho[2 * k + 1] = v.y * w;
  }
  if (outcome) {
    const float2* o2 = reinterpret_cast<const float2*>(outcome + i * kHeroes);
#pragma unroll
    for (int k = 0; k < kHeroes / 2; ++k) {
      const float2 v = o2[k];
      rho[2 * k] += v.x;
      rho[2 * k + 1] += v.y;
    }
  }
  mix_game(rho, c.tau, z);
}

// One sum over the block's threads, the same in every thread: a butterfly in
// each wave, then the wave sums in order.  A fixed order, so the result is the
// same from call to call.
__device__ double block_sum(double v, double* lds) {
#pragma unroll
  for (int w = 32; w > 0; w >>= 1) v += __shfl_xor(v, w, 64);
  if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = lds[0];
#pragma unroll
  for (int k = 1; k < kRwThreads / 64; ++k) s += lds[k];
  __syncthreads();
  return s;
}

// The union of KP summaries per thread (in every thread): mean = sum n_i m_i /
// n, M2 = sum (M2_i + n_i (m_i - mean)^2), the same moments that pairwise
// merges give, with one division instead of two at each of eight serial levels
// (reward_stats at 13 games: 4.0 us against 4.8).
template <int KP>
__device__ Summary block_merge(const Summary (&s)[KP], double* lds) {
  double n = 0.0, nm = 0.0, m2 = 0.0;
#pragma unroll
  for (int k = 0; k < KP; ++k) {
    n += s[k].n;
    nm += s[k].n * s[k].mean;
  }
  n = block_sum(n, lds);
  const double mean = block_sum(nm, lds) / n;
#pragma unroll
  for (int k = 0; k < KP; ++k) {
    const double d = s[k].mean - mean;
    m2 += s[k].m2 + s[k].n * d * d;
  }
  return Summary{n, mean, block_sum(m2, lds)};
}

__global__ void __launch_bounds__(kRwThreads) reward_stats(size_t items, const float* __restrict__ shaped,
                                                           const float* __restrict__ outcome,
                                                           const float* __restrict__ game_time, RewardConsts c,
                                                           Summary* __restrict__ part,
                                                           const double* __restrict__ stats,
                                                           double* __restrict__ before) {
  __shared__ double lds[kRwThreads / 64];
  Summary s{0.0, 0.0, 0.0};
  if (blockIdx.x == 0 && threadIdx.x < 3) before[threadIdx.x] = stats[threadIdx.x];
  for (size_t i = static_cast<size_t>(blockIdx.x) * kRwThreads + threadIdx.x; i < items;
       i += static_cast<size_t>(gridDim.x) * kRwThreads) {
    float z[kHeroes];
    shape_game(shaped, outcome, game_time, i, c, z);
    double sum = 0.0;
#pragma unroll
    for (int k = 0; k < kHeroes; ++k) sum += z[k];
    const double m = sum / kHeroes;
    double q = 0.0;
#pragma unroll
    for (int k = 0; k < kHeroes; ++k) {
      const double d = z[k] - m;
      q += d * d;
    }
    const Summary g{static_cast<double>(kHeroes), m, q};
    s = s.n == 0.0 ? g : merge(s, g);
  }
  const Summary b = block_merge({s}, lds);
  if (threadIdx.x == 0) part[blockIdx.x] = b;
}

__global__ void __launch_bounds__(kRwThreads) reward_apply(size_t items, const float* __restrict__ shaped,
                                                           const float* __restrict__ outcome,
                                                           const float* __restrict__ game_time, RewardConsts c,
                                                           int nparts, const Summary* __restrict__ part,
                                                           const double* __restrict__ before,
                                                           double* __restrict__ stats, float eps,
                                                           float* __restrict__ r) {
  constexpr int kPer = kRwMaxBlocks / kRwThreads;
  __shared__ double lds[kRwThreads / 64];
  Summary p[kPer];
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int i = threadIdx.x + q * kRwThreads;
    p[q] = i < nparts ? part[i] : Summary{0.0, 0.0, 0.0};
  }
  const Summary run = merge(Summary{before[0], before[1], before[2]}, block_merge(p, lds));
  const float k = static_cast<float>(1.0 / sqrt(run.m2 / run.n + static_cast<double>(eps)));
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    stats[0] = run.n;
    stats[1] = run.mean;
    stats[2] = run.m2;
  }
  for (size_t i = static_cast<size_t>(blockIdx.x) * kRwThreads + threadIdx.x; i < items;
       i += static_cast<size_t>(gridDim.x) * kRwThreads) {
    float z[kHeroes];
    shape_game(shaped, outcome, game_time, i, c, z);
    float2* r2 = reinterpret_cast<float2*>(r + i * kHeroes);
#pragma unroll
    for (int q = 0; q < kHeroes / 2; ++q) r2[q] = make_float2(z[2 * q] * k, z[2 * q + 1] * k);
  }
}

struct RewardWs {
  size_t part, before, total;
  int blocks;
};

static RewardWs reward_ws(int L, int G) {
  RewardWs w;
  const size_t items = static_cast<size_t>(L) * G;
  w.blocks = static_cast<int>(std::min<size_t>((items + kRwThreads - 1) / kRwThreads, kRwMaxBlocks));
  w.part = 0;
  w.before = align_up(static_cast<size_t>(w.blocks) * sizeof(Summary));
  w.total = w.before + align_up(3 * sizeof(double));
  return w;
}

}  // namespace o5

using namespace o5;

static int check_reward_shape(const char* fn, int L, int G) {
  O5_CHECK(L >= 1 && G >= 1, O5_E_SHAPE, "%s: L=%d and G=%d must be >= 1", fn, L, G);
  O5_CHECK(static_cast<long long>(L) * G < (1ll << 31) && static_cast<long long>(L) * G * kHeroes < (1ll << 31),
           O5_E_SHAPE, "%s: L*G*10 must stay below 2^31", fn);
  return O5_OK;
}

extern "C" size_t o5_reward_process_workspace_bytes(int L, int G) {
  if (check_reward_shape("o5_reward_process_workspace_bytes", L, G) != O5_OK) return 0;
  return reward_ws(L, G).total;
}

extern "C" int o5_reward_process(int L, int G, const float* shaped, const float* outcome, const float* game_time,
                                 o5_reward_hp hp, double* stats, float* r, void* ws, size_t ws_bytes,
                                 void* stream) {
  {
    const int st = check_reward_shape("o5_reward_process", L, G);
    if (st != O5_OK) return st;
  }
  O5_CHECK(hp.tau >= 0.0f && hp.tau <= 1.0f, O5_E_ARG, "o5_reward_process: tau=%g must lie in [0, 1]", hp.tau);
  O5_CHECK(hp.decay_base > 0.0f && hp.decay_base <= 1.0f && hp.decay_minutes > 0.0f && hp.eps > 0.0f, O5_E_ARG,
           "o5_reward_process: need 0 < decay_base <= 1, decay_minutes > 0 and eps > 0");
  O5_PTR(shaped, "shaped");
  O5_OPT_PTR(outcome, "outcome");
  O5_PTR(game_time, "game_time");
  O5_PTR(stats, "stats");
  O5_PTR(r, "r");
  const RewardWs w = reward_ws(L, G);
  O5_CHECK(ws != nullptr && ws_bytes >= w.total, O5_E_WORKSPACE,
           "o5_reward_process: workspace needs %zu bytes, got %zu", w.total,
           ws ? ws_bytes : static_cast<size_t>(0));
  O5_CHECK(aligned16(ws), O5_E_ALIGN, "o5_reward_process: 'ws' is not 16-byte aligned");
  RewardConsts c;
  c.tau = hp.tau;
  c.log2_base_per_minute = static_cast<float>(std::log2(static_cast<double>(hp.decay_base)) / hp.decay_minutes);
  const size_t items = static_cast<size_t>(L) * G;
  char* wsb = static_cast<char*>(ws);
  Summary* part = reinterpret_cast<Summary*>(wsb + w.part);
  double* before = reinterpret_cast<double*>(wsb + w.before);
  hipStream_t s = as_stream(stream);
  ktimer_begin(kSiteReward, s);
  hipLaunchKernelGGL(reward_stats, dim3(w.blocks), dim3(kRwThreads), 0, s, items, shaped, outcome, game_time, c,
                     part, stats, before);
  hipLaunchKernelGGL(reward_apply, dim3(w.blocks), dim3(kRwThreads), 0, s, items, shaped, outcome, game_time, c,
                     w.blocks, part, before, stats, hp.eps, r);
  ktimer_end(kSiteReward, s);
  return check_launch("o5_reward_process");
}
