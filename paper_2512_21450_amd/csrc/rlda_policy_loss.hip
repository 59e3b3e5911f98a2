// Scoring, group advantage estimation and the clipped policy loss (Eq. 6 of the paper; Sec. 3.2.2
// scoring, advantage-estimation and policy-update stages).  Element-wise work over [B] and [B, T]
// arrays with deterministic reductions: per-thread partial sums in a fixed order, a fixed tree
// inside the workgroup, and a fold of the per-sequence sums in fp64 by the last workgroup to end or by a further kernel.
//
// rl_group_advantage: one workgroup per prompt.  The group's mean and deviations are taken in
// fp64: with fp32 a group whose samples all earned the same reward can get a mean one ulp off and,
// after division by (std + eps), advantages of several percent out of pure rounding.
//
// rl_policy_loss: one workgroup per sequence streams its valid tokens once (HBM-bound: 2 to 4
// input arrays and one output array of 4 bytes per token).
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/rl_policy_loss.h"
#include "rlda_arrive.h"

namespace {

constexpr int NT = 256;

// fixed-order tree over the workgroup; every thread returns the total
template <typename T>
__device__ __forceinline__ T block_sum(T v, T* sh) {
  const int tid = threadIdx.x;
  __syncthreads();                                          // sh may still be read from a previous call
  sh[tid] = v;
  __syncthreads();
#pragma unroll
  for (int s = NT / 2; s > 0; s >>= 1) {
    if (tid < s) sh[tid] += sh[tid + s];
    __syncthreads();
  }
  return sh[0];
}

struct AdvParams {
  const float* metrics; const float* weights; float* rewards; float* adv;
  int P, G, M, mode, unbiased;
  float eps;
};

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {                // fixed butterfly, in every lane
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// N: threads of a prompt's workgroup.  What bounds a call is one chain of round trips and barriers: groups of up to 64 samples,
// which is all that rollouts use, are one wavefront's, whose two sums need no barrier (18 of them with 256 threads); it adds in
// the order of block_sum, so the bits are the same.  us, advantages and loss from Python, 256 threads / 64: 512 prompts x 8 of 4096
// tokens 54.1 / 53.0, 512 x 16 of 700 30.4 / 29.5, 350 x 16 of 2000 30.3 / 29.3; below 4096 sequences the host's launches are waited for.
template <int N>
__global__ void __launch_bounds__(N) group_advantage_kernel(const AdvParams A) {
  constexpr int K = N == 64 ? 1 : 4;                        // samples of a thread: G <= K * N
  __shared__ double sh[N == 64 ? 1 : N];
  const auto sum_of = [&](double v) {
    if constexpr (N == 64) return wave_sum(v);
    else return block_sum<double>(v, sh);
  };
  const int p = blockIdx.x, tid = threadIdx.x;
  const size_t B = (size_t)A.P * A.G;
  float r[K];
  double s = 0.0;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int g = tid + k * N;
    r[k] = 0.f;
    if (g < A.G) {
      const size_t b = (size_t)p * A.G + g;
      float acc = 0.f;
      for (int m = 0; m < A.M; ++m) acc = fmaf(A.weights[m], A.metrics[(size_t)m * B + b], acc);
      r[k] = acc;
      if (A.rewards) A.rewards[b] = acc;
      s += (double)acc;
    }
  }
  const double sum = sum_of(s), mean = sum / A.G;
  double q = 0.0;
#pragma unroll
  for (int k = 0; k < K; ++k)
    if (tid + k * N < A.G) { const double d = (double)r[k] - mean; q += d * d; }
  const double ss = sum_of(q);
  const int div = A.unbiased ? A.G - 1 : A.G;
  const double sd = div > 0 ? sqrt(ss / div) : 0.0;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int g = tid + k * N;
    if (g >= A.G) continue;
    const double d = (double)r[k] - mean;
    double a;
    if (A.mode == RL_ADV_GROUP_CENTER) a = d;
    else if (A.mode == RL_ADV_LEAVE_ONE_OUT) a = A.G > 1 ? (double)r[k] - (sum - (double)r[k]) / (A.G - 1) : 0.0;
    else a = d / (sd + (double)A.eps);
    A.adv[(size_t)p * A.G + g] = (float)a;
  }
}

struct LossParams {
  const float* lp; const float* old; const float* adv; const float* kl; const float* ent;
  const int32_t* lens;
  float* grad; float* stats;
  long long* counts;                                        // [2] valid tokens, sequences with tokens (first 256 workspace bytes)
  uint64_t* part;                                           // [B][4] per-sequence sums in pairs of floats; behind them a group's counter
  uint64_t* groups_done;                                    // a counter (behind the counts)
  uint64_t call;                                            // its number
  int B, T, form, agg;
  int64_t stride;
  float lo, hi, beta_kl, beta_ent;
};

__device__ __forceinline__ int clamp_len(int v, int T) { return v < 0 ? 0 : (v > T ? T : v); }

// The two kernels around the token pass run in one workgroup each, so their time is a chain of round trips: as many
// threads as a workgroup holds, several independent loads in flight per thread, sums over a wavefront by shuffles (one
// barrier) instead of a tree through LDS (eight).  4096 sequences: count 7.3 -> 3.3 us, reduction 14.7 -> 5.3 us.
constexpr int NB = 1024, NBW = NB / 64;

// batch totals the token weights need: valid tokens, sequences with tokens (one workgroup)
__global__ void __launch_bounds__(NB) policy_count_kernel(const LossParams L) {
  __shared__ long long sh[2][NBW];
  const int tid = threadIdx.x;
  long long a = 0, c = 0;
  for (int b0 = tid; b0 < L.B; b0 += 8 * NB) {
    int n[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) n[k] = b0 + k * NB < L.B ? L.lens[b0 + k * NB] : 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int m = clamp_len(n[k], L.T);
      a += m; c += m > 0;
    }
  }
  a = wave_sum(a); c = wave_sum(c);
  if ((tid & 63) == 0) { sh[0][tid >> 6] = a; sh[1][tid >> 6] = c; }
  __syncthreads();
  if (tid < 2) {
    long long t = 0;
#pragma unroll
    for (int k = 0; k < NBW; ++k) t += sh[tid][k];
    L.counts[tid] = t;
  }
}

// one sequence's sums into the batch's, in fp64
__device__ __forceinline__ void add_sequence(const LossParams& L, int n, float2 x, float2 y, float2 z, double wt, long long n_seq, double (&acc)[6]) {
  if (n == 0) return;
  const double wa = L.agg == RL_AGG_SEQ_MEAN ? 1.0 / ((double)n * (double)n_seq) : wt;
  acc[0] += wa * x.x; acc[1] += wa * x.y; acc[2] += wa * y.x;
  acc[3] += wt * y.y; acc[4] += wt * z.x; acc[5] += wt * z.y;
}

// by one wavefront; t: lane k < 6 holds the k-th sum
__device__ __forceinline__ void write_stats(const LossParams& L, double t, long long n_tok) {
  const int lane = threadIdx.x;
  if (lane < 6) L.stats[lane + 1] = (float)t;
  const double kl = __shfl(t, 1, 64), ent = __shfl(t, 2, 64);
  if (lane == 0) {
    L.stats[0] = (float)(-t + (double)L.beta_kl * kl - (double)L.beta_ent * ent);
    L.stats[7] = (float)n_tok;
  }
}

// per-sequence sums -> batch statistics, in fp64 and in a fixed order: a thread's sequences in turn, the lanes of a
// wavefront by a butterfly, the wavefronts in order
__global__ void __launch_bounds__(NB) policy_loss_reduce_kernel(const LossParams L) {
  __shared__ double sh[6][NBW];
  const int tid = threadIdx.x;
  const long long n_tok = L.counts[0], n_seq = L.counts[1];
  const double wt = n_tok > 0 ? 1.0 / (double)n_tok : 0.0;
  double acc[6] = {0, 0, 0, 0, 0, 0};
  constexpr int U = 4;
  for (int b0 = tid; b0 < L.B; b0 += U * NB) {
    int len[U];
    float4 p[U];
    float2 q[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int b = min(b0 + k * NB, L.B - 1);
      len[k] = b0 + k * NB < L.B ? L.lens[b] : 0;
      p[k] = *reinterpret_cast<const float4*>(L.part + (size_t)b * 4);
      q[k] = *reinterpret_cast<const float2*>(L.part + (size_t)b * 4 + 2);
    }
#pragma unroll
    for (int k = 0; k < U; ++k)
      add_sequence(L, clamp_len(len[k], L.T), make_float2(p[k].x, p[k].y), make_float2(p[k].z, p[k].w), q[k], wt, n_seq, acc);
  }
#pragma unroll
  for (int k = 0; k < 6; ++k) acc[k] = wave_sum(acc[k]);
  if ((tid & 63) == 0) {
#pragma unroll
    for (int k = 0; k < 6; ++k) sh[k][tid >> 6] = acc[k];
  }
  __syncthreads();
  if (tid < 64) {
    double t = 0.0;
    if (tid < 6) {
#pragma unroll
      for (int k = 0; k < NBW; ++k) t += sh[tid][k];
    }
    write_stats(L, t, n_tok);
  }
}

// the k-th sum over a wavefront, in lane k
__device__ __forceinline__ double sums_by_lane(double (&acc)[6]) {
  double t = 0.0;
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    const double v = wave_sum(acc[k]);
    if ((int)threadIdx.x == k) t = v;
  }
  return t;
}

// The same inside the token pass, by the first wavefront of each workgroup (the others are gone): sequences meet in groups of
// GROUP, the last group is up to twice as large; the last of a group adds the group's, one or two to a lane, and leaves six
// doubles where nothing else is kept; the last group's adds the groups'.  What is left for others and read of it goes past the
// caches of one die.
constexpr int GROUP = 64, MAX_GROUPS = 64;
__device__ __forceinline__ int n_groups(const LossParams& L) { return max(1, L.B / GROUP); }
__device__ __forceinline__ void reduce_groups(const LossParams& L, int g, uint64_t seen, long long n_tok, long long n_seq) {
  const int lane = threadIdx.x, n = n_groups(L), first = g * GROUP, size = g == n - 1 ? L.B - first : GROUP;
  const double wt = n_tok > 0 ? 1.0 / (double)n_tok : 0.0;
  int last = 0;
  if (lane == 0) last = rlda::arrive(L.part + (size_t)first * 4 + 3, L.call, seen, size);
  if (!__shfl(last, 0, 64)) return;
  double acc[6] = {0, 0, 0, 0, 0, 0};
  for (int i = lane; i < size; i += 64) {
    const uint64_t* const at = L.part + (size_t)(first + i) * 4;
    const float2 x = rlda::get(at), y = rlda::get(at + 1), z = rlda::get(at + 2);
    add_sequence(L, clamp_len(L.lens[first + i], L.T), x, y, z, wt, n_seq, acc);
  }
  double t = sums_by_lane(acc);
  if (n > 1) {
    if (lane < 6)
      __hip_atomic_store(L.part + (size_t)(first + 1 + lane) * 4 + 3, (uint64_t)__double_as_longlong(t), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    rlda::stores_done();
    last = 0;
    if (lane == 0) last = rlda::arrive(L.groups_done, L.call, rlda::claim(L.groups_done, L.call), n);
    if (!__shfl(last, 0, 64)) return;
#pragma unroll
    for (int k = 0; k < 6; ++k) acc[k] = 0;
    if (lane < n) {
      const uint64_t* const at = L.part + ((size_t)lane * GROUP + 1) * 4 + 3;
#pragma unroll
      for (int k = 0; k < 6; ++k)
        acc[k] = __longlong_as_double((long long)__hip_atomic_load(at + k * 4, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    }
    t = sums_by_lane(acc);
  }
  write_stats(L, t, n_tok);
}

// per-token arithmetic; accumulates into sums[6] = (term, kl, entropy, flat-branch count, rho, old - new)
__device__ __forceinline__ float token_term(const LossParams& L, float lp, float old, float kl, float ent, float A,
                                            float w, float (&sums)[6]) {
  const float rho = expf(lp - old);
  const float ra = rho * A;
  float term;
  bool flat;
  if (L.form == RL_PG_AS_PRINTED) {
    flat = rho > L.hi;
    term = fminf(rho, L.hi) * A;
  } else {
    const float ca = fminf(fmaxf(rho, L.lo), L.hi) * A;
    flat = !(ra <= ca);                                     // inside the range both products are equal: not flat
    term = fminf(ra, ca);
  }
  sums[0] += term; sums[1] += kl; sums[2] += ent; sums[3] += flat ? 1.f : 0.f; sums[4] += rho; sums[5] += old - lp;
  return flat ? 0.f : -w * ra;
}

// Token pass, one workgroup per sequence.  COUNT: every workgroup adds up all lengths itself before its first token, which
// saves the launch of policy_count_kernel in front of it (1.5 us on the device and one of the host's).  That reads 4 bytes per
// pair of sequences, so it pays up to COUNT_MAX of them only; one launch / two, advantages and loss together, captured, us:
// 8 sequences 10.9 / 13.2, 128 11.5 / 13.6, 1024 14.0 / 16.4; 2048 19.3 / 19.7, 4096 27.1 / 24.2, 8192 48.4 / 33.7.
// (Workgroups that stay and take several sequences in turn read less, but longer ones hold them up: 4096 x 4096 tokens
// 51 us against 48.)  Four tokens per thread and step: one 16-byte load per array, which the hardware wants aligned to 4
// bytes only, so rows of any length take it (8192 x 999 tokens 35.2 -> 33.7 us, one by one before), and single elements at a
// row's end.  A thread adds its tokens in increasing t, the 64 lanes of a wavefront are folded by a fixed butterfly and the
// four wavefronts in order, so the sums do not depend on anything but the data.
constexpr int COUNT_MAX = 1024;
// ONE: the first wavefront of the last workgroup to end reduces (reduce_groups), which saves the launch behind.  A workgroup's other
// wavefronts end before it waits, so that the next workgroup finds most of its place free; while all 256 threads waited and one
// workgroup added up everything, it paid up to 2048 sequences only (4096, captured: 20.4 with a launch / 22.9).  us, advantages and
// loss from Python, a launch / so: 512 prompts x 8 of 4096 tokens 52.7 / 50.5, of 1000 24.3 / 22.6, 200 x 16 of 3000 32.5 / 30.8; beyond
// ONE_MAX the queue of workgroups pays for each: 350 x 16 of 2000 29.4 / 29.5, 512 x 16 of 700 29.5 / 29.4, of 80 27.9 / 28.6.
// Few sequences, two or three launches / one or two: 8 20.5 / 18.2, 1024 21.9 / 19.3, 2048 24.9 / 22.2.
// Captured, a launch / so: 17 x 3972 tokens 14.0 / 11.4, 1024 x 512 14.5 / 12.7, 4095 x 500 22.2 / 21.4, 4096 x 4096 58.4 / 55.2.  The line lies at what 64
// groups hold, one to a lane.
constexpr int ONE_MAX = GROUP * MAX_GROUPS;
static_assert(COUNT_MAX <= ONE_MAX && 2 * GROUP - 1 <= rlda::MAX_ARRIVALS && MAX_GROUPS <= 64, "a counter, and a wavefront, hold no more");
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef f32x4 f32x4u __attribute__((aligned(4)));

template <bool COUNT, bool ONE>
__global__ void __launch_bounds__(NT) policy_loss_kernel(const LossParams L) {
  static_assert(!COUNT || ONE, "the kernel behind the token pass reads the counts that policy_count_kernel leaves");
  __shared__ float shf[NT / 64][6];
  const int tid = threadIdx.x;
  long long n_tok, n_seq;
  // This sequence's length, asked for with the batch's: behind them it is a round trip more (us, captured with the advantages, behind / with
  // them: 8 x 8 x 290 tokens 9.1 / 8.85, 4000 x 700 22.0 / 21.6; the other way 848 x 87 12.8 / 13.2).
  int own;
  if (COUNT) {
    __shared__ long long sh[2][NT / 64];
    static_assert(COUNT_MAX % NT == 0, "a thread's sequences");
    constexpr int U = COUNT_MAX / NT;                     // all of them, asked for at once
    long long a = 0;
    int c = 0, n[U];
#pragma unroll
    for (int k = 0; k < U; ++k) n[k] = tid + k * NT < L.B ? L.lens[tid + k * NT] : 0;
    own = L.lens[blockIdx.x];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int m = clamp_len(n[k], L.T);
      a += m; c += m > 0;
    }
    a = wave_sum(a); c = wave_sum(c);
    if ((tid & 63) == 0) { sh[0][tid >> 6] = a; sh[1][tid >> 6] = c; }
    __syncthreads();
    n_tok = (sh[0][0] + sh[0][1]) + (sh[0][2] + sh[0][3]);
    n_seq = (sh[1][0] + sh[1][1]) + (sh[1][2] + sh[1][3]);
  } else {
    own = L.lens[blockIdx.x];
    n_tok = L.counts[0]; n_seq = L.counts[1];
  }
  const int b = blockIdx.x;
  const int met = min(b / GROUP, n_groups(L) - 1);        // the group it meets in
  uint64_t seen = 0;
  if (ONE && tid == 0) seen = rlda::claim(L.part + (size_t)met * GROUP * 4 + 3, L.call);
  const unsigned len = clamp_len(own, L.T);
  float w = 0.f;                                          // weight of one of this sequence's tokens in the aggregate
  if (len > 0) w = L.agg == RL_AGG_SEQ_MEAN ? (float)(1.0 / ((double)len * (double)n_seq)) : (float)(1.0 / (double)n_tok);
  const float A = L.adv[b];
  const size_t row = (size_t)b * L.stride;
  float sums[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const unsigned T = L.T;                                 // unsigned: the last step of a row of nearly 2^31 tokens ends behind them
  for (unsigned t = 4 * tid; t < T; t += 4 * NT) {
    f32x4 g = {0.f, 0.f, 0.f, 0.f};
    if (t + 4 <= T) {                                     // the four tokens exist as memory; some may be padding
      if (t < len) {
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        const f32x4 lp = *reinterpret_cast<const f32x4u*>(L.lp + row + t), old = *reinterpret_cast<const f32x4u*>(L.old + row + t);
        const f32x4 kl = L.kl ? *reinterpret_cast<const f32x4u*>(L.kl + row + t) : zero;
        const f32x4 en = L.ent ? *reinterpret_cast<const f32x4u*>(L.ent + row + t) : zero;
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (t + k < len) g[k] = token_term(L, lp[k], old[k], kl[k], en[k], A, w, sums);
      }
      if (L.grad) *reinterpret_cast<f32x4u*>(L.grad + row + t) = g;
    } else {
      for (unsigned k = t; k < T; ++k) {
        float gk = 0.f;
        if (k < len)
          gk = token_term(L, L.lp[row + k], L.old[row + k], L.kl ? L.kl[row + k] : 0.f, L.ent ? L.ent[row + k] : 0.f, A, w, sums);
        if (L.grad) L.grad[row + k] = gk;
      }
    }
  }
#pragma unroll
  for (int k = 0; k < 6; ++k) sums[k] = wave_sum(sums[k]);
  if ((tid & 63) == 0) {
#pragma unroll
    for (int k = 0; k < 6; ++k) shf[tid >> 6][k] = sums[k];
  }
  __syncthreads();
  if constexpr (!ONE) {
    if (tid < 6) reinterpret_cast<float*>(L.part)[(size_t)b * 8 + tid] = ((shf[0][tid] + shf[1][tid]) + shf[2][tid]) + shf[3][tid];
    return;
  }
  if (tid >= 64) return;
  if (tid < 3) {
    const auto sum = [&](int k) { return ((shf[0][k] + shf[1][k]) + shf[2][k]) + shf[3][k]; };
    rlda::put(L.part + (size_t)b * 4 + tid, sum(2 * tid), sum(2 * tid + 1));
  }
  rlda::stores_done();
  reduce_groups(L, met, seen, n_tok, n_seq);
}

int check(const rl_policy_loss_desc* d) {
  if (!d) return -1;
  if (d->struct_size != sizeof(rl_policy_loss_desc)) return -4;
  if (d->B < 0 || d->T < 0) return -1;
  if (!(d->clip_low >= 0.f) || !(d->clip_high >= 0.f)) return -1;
  if (d->form != RL_PG_PPO_CLIP && d->form != RL_PG_AS_PRINTED) return -2;
  if (d->agg != RL_AGG_TOKEN_MEAN && d->agg != RL_AGG_SEQ_MEAN) return -2;
  if (d->row_stride < d->T) return -2;
  return 0;
}

}  // namespace

extern "C" {

int rl_group_advantage(const rl_group_advantage_desc* d, void* hip_stream) {
  if (!d) return -1;
  if (d->struct_size != sizeof(rl_group_advantage_desc)) return -4;
  if (d->P < 0 || d->G < 0 || !(d->eps >= 0.f)) return -1;
  if (d->mode != RL_ADV_GROUP_NORM && d->mode != RL_ADV_GROUP_CENTER && d->mode != RL_ADV_LEAVE_ONE_OUT) return -2;
  if (d->G > 4 * NT || d->n_metrics < 1 || d->n_metrics > 64) return -2;
  if (d->P == 0 || d->G == 0) return 0;
  if (!d->metrics || !d->weights || !d->advantages) return -1;
  const AdvParams A{d->metrics, d->weights, d->rewards, d->advantages, d->P, d->G, d->n_metrics, d->mode,
                    d->unbiased, d->eps};
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  if (d->G <= 64) hipLaunchKernelGGL(group_advantage_kernel<64>, dim3(d->P), dim3(64), 0, st, A);
  else            hipLaunchKernelGGL(group_advantage_kernel<NT>, dim3(d->P), dim3(NT), 0, st, A);
  return hipGetLastError() == hipSuccess ? 0 : -5;
}

size_t rl_policy_loss_workspace_bytes(const rl_policy_loss_desc* d) {
  if (check(d) != 0) return 0;
  return 256 + (size_t)d->B * 8 * sizeof(float);
}

int rl_policy_loss(const rl_policy_loss_desc* d, void* hip_stream) {
  const int rc = check(d);
  if (rc != 0) return rc;
  if (!d->stats) return -1;
  if (d->B > 0 && (!d->advantages || !d->lens)) return -1;
  if (d->B > 0 && d->T > 0 && (!d->logprob || !d->old_logprob)) return -1;
  const size_t need = rl_policy_loss_workspace_bytes(d);
  if (need > 0 && (!d->workspace || d->workspace_bytes < need)) return -3;
  if (need > 0 && (reinterpret_cast<uintptr_t>(d->workspace) & 255u)) return -3;
  LossParams L;
  L.lp = d->logprob; L.old = d->old_logprob; L.adv = d->advantages; L.kl = d->kl; L.ent = d->entropy;
  L.lens = d->lens; L.grad = d->grad_logprob; L.stats = d->stats;
  L.counts = static_cast<long long*>(d->workspace);
  L.groups_done = reinterpret_cast<uint64_t*>(L.counts + 2);
  L.part = reinterpret_cast<uint64_t*>(static_cast<char*>(d->workspace) + 256);
  L.B = d->B; L.T = d->T; L.form = d->form; L.agg = d->agg; L.stride = d->row_stride;
  L.lo = 1.f - d->clip_low; L.hi = 1.f + d->clip_high; L.beta_kl = d->beta_kl; L.beta_ent = d->beta_ent;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  const bool own = d->B > 0 && d->B <= COUNT_MAX;           // the token pass counts for itself
  const bool one = d->B > 0 && d->B <= ONE_MAX;             // and reduces
  L.call = one ? rlda::next_call() : 0;
  if (!own) {
    hipLaunchKernelGGL(policy_count_kernel, dim3(1), dim3(NB), 0, st, L);
    if (hipGetLastError() != hipSuccess) return -5;
  }
  if (d->B > 0) {
    const dim3 grid(d->B);
    if (own)      hipLaunchKernelGGL((policy_loss_kernel<true, true>), grid, dim3(NT), 0, st, L);
    else if (one) hipLaunchKernelGGL((policy_loss_kernel<false, true>), grid, dim3(NT), 0, st, L);
    else          hipLaunchKernelGGL((policy_loss_kernel<false, false>), grid, dim3(NT), 0, st, L);
    if (hipGetLastError() != hipSuccess) return -5;
  }
  if (one) return 0;
  hipLaunchKernelGGL(policy_loss_reduce_kernel, dim3(1), dim3(NB), 0, st, L);
  return hipGetLastError() == hipSuccess ? 0 : -5;
}

}  // extern "C"
