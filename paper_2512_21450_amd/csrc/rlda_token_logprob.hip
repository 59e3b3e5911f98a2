// Per-token policy statistics from vocabulary logits: log-prob of the sampled token, entropy,
// KL to a reference policy (Sec. 2.2 of the paper: importance ratio r_t, entropy bonus,
// KL-to-reference; Omega and L^PG of Eq. 6).
//
// HBM-bound streaming reduction.  A row is cut into S contiguous splits (S chosen on the host
// so that the grid fills the chip); workgroup (split, row) streams its part with 16-byte
// nontemporal loads and keeps, per thread, an online-softmax state
//   m, s = sum e^(a-m), t = sum e^(a-m) a          for a = logits * inv_temperature
//   mr, sr = sum e^(b-mr), u = sum e^(a-m) b       for b = ref_logits * inv_temperature
// which is merged over the wavefront (xor shuffles), the workgroup (LDS) and, when S > 1, the
// splits (one wavefront per row: of the row's last workgroup to end, or of a second kernel).  Then
//   lse = m + ln s, entropy = lse - t/s, kl = (t - u)/s - lse + (mr + ln sr).
// All merges have a fixed order, so results do not change from call to call.
//
// The inner loop is close to the vector-ALU limit at HBM speed (bf16: ~12 issue slots per
// logit are available at 6.5 TB/s, the exponential alone takes 4), so the state is kept in
// base 2 (a, b pre-multiplied by inv_temperature * log2 e: the hardware exponential is 2^x) and
// masked logits (-inf) are clamped to -1e30, which makes 0 * a finite without a branch and
// cannot overflow a sum.
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/rl_token_logprob.h"
#include "rlda_arrive.h"

namespace {

// threads per workgroup: 256 when there are thousands of workgroups, 1024 when there is about one
// per compute unit (a decode step's few hundred rows), so that either way the chip is full
constexpr int UNR = 4;             // independent 16-byte loads in flight per thread
constexpr int MAX_SPLITS = 64;     // one lane per split in the final merge

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

struct Params {
  const char* logits; const char* ref; const int32_t* ids;
  float* logprob; float* lse; float* entropy; float* ref_logprob; float* kl;
  float* part;                     // [n_rows][slots][6]
  int slots;                       // per row: S, one launch: and one more
  uint64_t call;                   // one launch: the call's number
  long long stride;                // elements
  int V, S, chunk;                 // chunk: elements per split, multiple of the vector width
  float k2;                        // inv_temperature * log2(e): logits -> base-2 exponents
};

constexpr float LN2 = 0.69314718055994531f;
constexpr float MASKED = -1e30f;        // stands for a logit of -inf inside the reductions

struct Acc { float m, s, t, mr, sr, u; };

__device__ __forceinline__ Acc acc_empty() { return Acc{-INFINITY, 0.f, 0.f, -INFINITY, 0.f, 0.f}; }

__device__ __forceinline__ float rescale(float m_old, float m_new) {      // 2^(m_old - m_new), 0 for an empty side
  return m_old == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_old - m_new);
}

template <bool REF>
__device__ __forceinline__ Acc acc_merge(const Acc& x, const Acc& y) {
  Acc r;
  r.m = fmaxf(x.m, y.m);
  const float cx = rescale(x.m, r.m), cy = rescale(y.m, r.m);
  r.s = x.s * cx + y.s * cy;
  r.t = x.t * cx + y.t * cy;
  r.u = x.u * cx + y.u * cy;
  r.mr = -INFINITY; r.sr = 0.f;
  if (REF) {
    r.mr = fmaxf(x.mr, y.mr);
    r.sr = x.sr * rescale(x.mr, r.mr) + y.sr * rescale(y.mr, r.mr);
  }
  return r;
}

template <bool REF>
__device__ __forceinline__ Acc acc_shfl_xor(const Acc& a, int mask) {
  Acc r;
  r.m = __shfl_xor(a.m, mask, 64); r.s = __shfl_xor(a.s, mask, 64); r.t = __shfl_xor(a.t, mask, 64);
  r.mr = -INFINITY; r.sr = 0.f; r.u = 0.f;
  if (REF) { r.mr = __shfl_xor(a.mr, mask, 64); r.sr = __shfl_xor(a.sr, mask, 64); r.u = __shfl_xor(a.u, mask, 64); }
  return r;
}

template <typename T> struct Elem;
template <> struct Elem<float> {
  static constexpr int VN = 4;
  __device__ static void unpack(const u32x4& v, float (&f)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) f[i] = __uint_as_float(v[i]);
  }
  __device__ static float one(const char* p, long long i) { return reinterpret_cast<const float*>(p)[i]; }
};
template <> struct Elem<uint16_t> {
  static constexpr int VN = 8;
  __device__ static void unpack(const u32x4& v, float (&f)[8]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f[2 * i] = __uint_as_float(v[i] << 16);
      f[2 * i + 1] = __uint_as_float(v[i] & 0xffff0000u);
    }
  }
  __device__ static float one(const char* p, long long i) {
    return __uint_as_float((uint32_t)reinterpret_cast<const uint16_t*>(p)[i] << 16);
  }
};

// N values of the row (and of the reference row), already in base-2 units and >= MASKED, into the
// thread's state.  Next to a live logit a masked one gives e = 2^(MASKED - m) = 0 and adds 0 * MASKED = 0; a state
// that has seen masked logits only (m = MASKED) is wiped by the rescale when the first live one arrives.
template <bool REF, int N>
__device__ __forceinline__ void absorb(Acc& A, const float (&a)[N], const float (&b)[N]) {
  float cm = a[0];
#pragma unroll
  for (int i = 1; i < N; ++i) cm = fmaxf(cm, a[i]);
  const float mn = fmaxf(A.m, cm);
  const float c = rescale(A.m, mn);
  float s = A.s * c, t = A.t * c, u = A.u * c;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const float e = __builtin_amdgcn_exp2f(a[i] - mn);
    s += e;
    t = fmaf(e, a[i], t);
    if (REF) u = fmaf(e, b[i], u);
  }
  A.m = mn; A.s = s; A.t = t; A.u = u;
  if (REF) {
    float cr = b[0];
#pragma unroll
    for (int i = 1; i < N; ++i) cr = fmaxf(cr, b[i]);
    const float mrn = fmaxf(A.mr, cr);
    float sr = A.sr * rescale(A.mr, mrn);
#pragma unroll
    for (int i = 0; i < N; ++i) sr += __builtin_amdgcn_exp2f(b[i] - mrn);
    A.mr = mrn; A.sr = sr;
  }
}

// State (base-2 units) -> outputs (natural units).  a_y, b_y: the sampled token's scaled logits.
template <bool REF>
__device__ __forceinline__ void finish_row(const Params& P, long long row, const Acc& A, float a_y, float b_y, int y) {
  const bool dead = A.m <= MASKED;                           // every logit masked: no distribution
  const float lse2 = A.m + __log2f(A.s);
  const float mean_a = A.t / A.s;                           // sum_i p_i a_i
  const float lse = dead ? -INFINITY : lse2 * LN2;
  if (P.lse) P.lse[row] = lse;
  if (P.entropy) P.entropy[row] = dead ? NAN : (lse2 - mean_a) * LN2;
  // !(x > MASKED): masked, also when the sampled token's logit is NaN (read as masked like every NaN logit)
  if (P.logprob) P.logprob[row] = y < 0 ? 0.f : (y >= P.V ? NAN : (!(a_y > MASKED) ? -INFINITY : (a_y - lse2) * LN2));
  if (REF) {
    const float lse_r2 = A.mr + __log2f(A.sr);
    float mean_b = A.u / A.s;                               // sum_i p_i b_i; a masked reference logit under p > 0
    if (mean_b < -1e6f) mean_b = -INFINITY;                 // drags it towards MASKED: the KL is infinite
    if (P.kl) P.kl[row] = dead ? NAN : (mean_a - mean_b - lse2 + lse_r2) * LN2;
    if (P.ref_logprob)
      P.ref_logprob[row] = y < 0 ? 0.f : (y >= P.V ? NAN : (!(b_y > MASKED) ? -INFINITY : (b_y - lse_r2) * LN2));
  }
}

// lane i of a wavefront has split i, merged in a fixed butterfly order
template <typename T, bool REF>
__device__ __forceinline__ void merge_row(const Params& P, long long row, Acc A, int lane) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) A = acc_merge<REF>(A, acc_shfl_xor<REF>(A, o));
  if (lane == 0) {
    const char* za = P.logits + (size_t)row * P.stride * sizeof(T);
    const char* zb = REF ? P.ref + (size_t)row * P.stride * sizeof(T) : nullptr;
    const int y = P.ids[row];
    const bool ok = y >= 0 && y < P.V;
    finish_row<REF>(P, row, A, ok ? Elem<T>::one(za, y) * P.k2 : 0.f,
                    REF && ok ? Elem<T>::one(zb, y) * P.k2 : 0.f, y);
  }
}

// ONE: the last of a row's workgroups to end merges what they left, its counter stands behind their states.
// workgroup row * S + split: partial state of elements [split * chunk, min(V, (split + 1) * chunk)) of a row
template <typename T, bool REF, int NT, bool ONE = false>
__global__ void __launch_bounds__(NT) token_partial_kernel(const Params P) {
  constexpr int VN = Elem<T>::VN;
  __shared__ Acc red[NT / 64];
  __shared__ bool last;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const long long row = blockIdx.x / P.S;
  const int split = blockIdx.x % P.S;
  const char* za = P.logits + (size_t)row * P.stride * sizeof(T);
  const char* zb = REF ? P.ref + (size_t)row * P.stride * sizeof(T) : nullptr;
  const int c0 = split * P.chunk, c1 = min(P.V, c0 + P.chunk);
  const int v0 = c0 / VN, v1 = max(c1, c0) / VN;           // whole vectors [v0, v1)
  uint64_t* const slots = reinterpret_cast<uint64_t*>(P.part) + (size_t)row * P.slots * 3;
  uint64_t* const counter = slots + P.S * 3;
  uint64_t seen = 0;
  if (ONE && tid == 0) seen = rlda::claim(counter, P.call);
  Acc A = acc_empty();
  for (int v = v0 + tid; v < v1; v += NT * UNR) {
    u32x4 ra[UNR], rb[UNR];
#pragma unroll
    for (int k = 0; k < UNR; ++k) {
      const int vk = v + k * NT;
      if (vk < v1) {                                        // past the end: no load, the slot is not used
        ra[k] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(za) + vk);
        if (REF) rb[k] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(zb) + vk);
      }
    }
#pragma unroll
    for (int k = 0; k < UNR; ++k) {
      if (v + k * NT < v1) {
        float a[VN], b[VN];
        Elem<T>::unpack(ra[k], a);
        if (REF) Elem<T>::unpack(rb[k], b);
#pragma unroll
        for (int i = 0; i < VN; ++i) {
          a[i] = fmaxf(a[i] * P.k2, MASKED);
          b[i] = REF ? fmaxf(b[i] * P.k2, MASKED) : 0.f;
        }
        absorb<REF, VN>(A, a, b);
      }
    }
  }
  // the row's last V % VN elements, one per thread, belong to the split that holds them
  const int tail0 = v1 * VN;
  if (c1 == P.V && c1 > c0 && tail0 + tid < c1) {
    float a[1] = {fmaxf(Elem<T>::one(za, tail0 + tid) * P.k2, MASKED)};
    float b[1] = {REF ? fmaxf(Elem<T>::one(zb, tail0 + tid) * P.k2, MASKED) : 0.f};
    absorb<REF, 1>(A, a, b);
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) A = acc_merge<REF>(A, acc_shfl_xor<REF>(A, o));
  if (lane == 0) red[wv] = A;
  __syncthreads();
  if (tid == 0) {
    Acc R = red[0];
#pragma unroll
    for (int k = 1; k < NT / 64; ++k) R = acc_merge<REF>(R, red[k]);
    if (ONE) {
      uint64_t* const o = slots + split * 3;
      rlda::put(o, R.m, R.s);
      rlda::put(o + 1, R.t, R.mr);
      if (REF) rlda::put(o + 2, R.sr, R.u);
      rlda::stores_done();
      last = rlda::arrive(counter, P.call, seen, P.S);
    } else if (P.S == 1) {
      const int y = P.ids[row];
      const bool ok = y >= 0 && y < P.V;
      finish_row<REF>(P, row, R, ok ? Elem<T>::one(za, y) * P.k2 : 0.f,
                      REF && ok ? Elem<T>::one(zb, y) * P.k2 : 0.f, y);
    } else {
      float* o = P.part + ((size_t)row * P.S + split) * 6;
      o[0] = R.m; o[1] = R.s; o[2] = R.t; o[3] = R.mr; o[4] = R.sr; o[5] = R.u;
    }
  }
  if constexpr (ONE) {
    __syncthreads();
    if (!last || wv > 0) return;
    Acc W = acc_empty();
    if (lane < P.S) {
      const uint64_t* const o = slots + lane * 3;
      const float2 a = rlda::get(o), b = rlda::get(o + 1), c = REF ? rlda::get(o + 2) : make_float2(0.f, 0.f);
      W = Acc{a.x, a.y, b.x, b.y, c.x, c.y};
    }
    merge_row<T, REF>(P, row, W, lane);
  }
}

// one wavefront per row
template <typename T, bool REF>
__global__ void __launch_bounds__(64) token_final_kernel(const Params P) {
  const long long row = blockIdx.x;
  const int lane = threadIdx.x;
  Acc A = acc_empty();
  if (lane < P.S) {
    const float* o = P.part + ((size_t)row * P.S + lane) * 6;
    A = Acc{o[0], o[1], o[2], o[3], o[4], o[5]};
  }
  merge_row<T, REF>(P, row, A, lane);
}

int check(const rl_token_logprob_desc* d) {
  if (!d) return -1;
  if (d->struct_size != sizeof(rl_token_logprob_desc)) return -4;
  if (d->n_rows < 0 || d->vocab < 1 || d->row_stride < 0) return -1;
  if (!(d->inv_temperature > 0.f) || d->inv_temperature > 3.0e38f) return -1;   // masked (-inf) logits must stay -inf after scaling
  if (d->dtype != 0 && d->dtype != 1) return -2;
  const int vn = d->dtype == 0 ? 4 : 8;
  if (d->row_stride < d->vocab || d->row_stride % vn != 0) return -2;
  if (d->n_rows > ((long long)1 << 31) / MAX_SPLITS - 1) return -2;   // rows * splits is the grid size
  if (d->vocab > (1 << 30)) return -2;
  return 0;
}

// Splits per row.  What bounds a call of few rows is the dependent rounds of loads of a thread (256 threads take 16 KB of a row
// a round); the merge of the splits costs 1 to 2 us.  us, captured and merged by a launch of its own, inputs changing, rows x logits; with a
// reference: [R].
//   * Fewer than 64 rows: at least 12 splits, and three workgroups of 256 threads a compute unit, down to 8 KB of a row each;
//     where 64 splits, the merge's limit, still leave more than 32 KB, workgroups of 1024 threads.  12 splits / as many as the
//     compute units want of 1024 threads and 8192 logits and more / this:
//       16 x 32000 bf16 [R] 7.5 / 9.7 / 7.5    16 x 151936 bf16 [R] 10.0 / 10.6 / 9.4   48 x 151936 bf16 [R] 14.4 / 17.5 / 13.4
//       1 x 256000 bf16 [R] 10.9 / 9.1 / 7.0   8 x 151936 fp32 8.6 / 7.6 / 6.5          4 x 1000000 fp32 25.8 / 9.1 / 9.1
//   * 64 to 191 rows: 12, down to 4096 logits each.  The same columns (the third as the first):
//       100 x 32000 bf16 [R] 10.4 / 13.2       150 x 151936 fp32 20.3 / 25.3            191 x 256000 bf16 [R] 40.0 / 48.3
//   * Fewer than 16384 logits, and about one row a compute unit: none, 16 wavefronts take a row (two workgroups of 256 threads
//     / none: 48 x 9000 bf16 6.8 / 5.4, 191 x 9000 fp32 [R] 10.3 / 8.5).
//   * A little over one or two rows a compute unit, most compute units would wait for those with one row more.  What that
//     costs grows with a row's bytes, what splits cost with the rows; none / 4 / 8 splits:
//       257 x 32000 bf16 [R] 16.1 / 14.4 / 14.7    257 x 32000 bf16 9.3 / 9.7 / 10.4       300 x 60000 fp32 [R] 34.0 / 29.7 / 29.8
//       300 x 151936 bf16 [R] 51.4 / 40.2 / 40.0   352 x 65536 bf16 15.3 / 15.4 / 16.2     352 x 60000 fp32 19.8 / 20.3 / 19.1
//       400 x 65536 bf16 16.1 / 16.9 / 18.1        448 x 151936 bf16 [R] 54.6 / 51.5 / 53.5   448 x 151936 fp32 44.9 / 46.5 / 46.8
//       513 x 65536 bf16 [R] 36.4 / 32.3 / 34.5    576 x 151936 bf16 41.6 / 36.1 / 36.2    576 x 151936 fp32 56.0 / 59.0 / 57.2
//       600 x 65536 fp32 [R] 55.7 / 54.3 / 53.2    640 x 65536 bf16 22.1 / 22.5 / 24.3     640 x 256000 bf16 [R] 130.5 / 108.3 / 110.9
// The numbers of rows are those of 256 compute units; on a part of a device the calls run, with other waits.
constexpr int64_t PER_SPLIT = 6 * sizeof(float);
constexpr long long KB = 1024, ROUNDS = 32 * KB;             // what 256 threads read in two rounds
int clamp_splits(long long s, long long by_size) {
  s = s < by_size ? s : by_size;
  s = s < MAX_SPLITS ? s : MAX_SPLITS;
  return s < 1 ? 1 : (int)s;
}
long long row_bytes(const rl_token_logprob_desc* d) { return (long long)d->vocab * (d->dtype == 0 ? 4 : 2); }
int splits_for(const rl_token_logprob_desc* d) {
  const long long n = d->n_rows, row = row_bytes(d), all = d->ref_logits ? 2 * row : row;
  const bool f32 = d->dtype == 0, ref = d->ref_logits != nullptr;
  if (n <= 0 || d->vocab < 16384) return 1;
  if (n < 64) return clamp_splits((767 + n) / n > 12 ? (767 + n) / n : 12, row / (8 * KB));
  if (n < 192) return clamp_splits(12, d->vocab / 4096);
  if (n > 256 && n <= 448) {
    const bool pays = n <= 320 ? all >= (ref ? 72 : 96) * KB : n <= 352 ? all >= (f32 ? 160 : 120) * KB
                    : n <= 376 ? all >= 256 * KB : !f32 && all >= 500 * KB;
    const bool eight = n <= 400 && (f32 || row >= 384 * KB || (ref && row >= 128 * KB));
    return pays ? (eight ? 8 : 4) : 1;
  }
  if (n > 512 && n <= 640) {
    if (f32) return ref && row >= (n <= 600 ? 256 : 512) * KB ? 8 : 1;
    return row >= (n <= 600 ? 128 : 192) * KB ? (row >= 384 * KB ? 8 : 4) : 1;
  }
  return 1;
}
// What a caller with less workspace gets, never more splits than the above: as many as give every compute unit a workgroup of
// 1024 threads, of 8192 logits and more, for fewer than 192 rows; else none.
int splits_with_less(const rl_token_logprob_desc* d) {
  if (d->n_rows <= 0 || d->n_rows >= 192) return 1;
  return clamp_splits((256 + d->n_rows - 1) / d->n_rows, d->vocab / 8192);
}
// The last workgroup of a row merges its splits where a call is so short that the host's second launch (4.4 us) is most of what it
// waits for; the counter takes one split's place, which long calls pay more for than the launch they save.  (By the logits alone, so that
// what does not depend on a reference keeps its bits without one.)  us, calls one after the other from Python (captured), two launches / one:
//   16 x 32000 bf16 16.5 (5.6) / 14.0 (5.2)      48 x 151936 bf16 [R] 18.9 (12.8) / 16.7 (12.5)   150 x 50001 fp32 [R] 19.7 (16.2) / 17.2 (15.8)
//   257 x 32000 bf16 [R] 19.9 (13.7) / 17.2 (13.4)   100 x 151936 fp32 [R] 25.3 (24.9) / 25.9 (25.8)   448 x 151936 bf16 [R] 52.6 / 56.7
//   1 x 151936 fp32 [R] 18.7 / 16.3
// Beyond MEET splits so many workgroups meet at a counter that a captured call, which waits for no host, loses: it gets the second
// kernel.  Captured, the counter / the second kernel, 1 and 12 rows: 151936 fp32 (63 splits) 5.6 / 5.0 and 7.1 / 6.8, [R] 7.0 / 6.5 and
// 9.6 / 9.1, 256000 bf16 (61) 5.7 / 5.4 and 7.4 / 7.1; but 151936 bf16 (36) 5.5 / 5.1 and 6.3 / 6.5, 8 rows 5.9 / 6.3.  (A split less is
// a round of loads more for a few: 24 x 256000 bf16 captured 8.4 with 32 splits, 8.7 so.)
constexpr long long ONE_LAUNCH = 48 * 1000 * KB;             // bytes of logits
constexpr int MEET = 48;
bool captured(hipStream_t st) {
  hipStreamCaptureStatus s = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &s) != hipSuccess) { (void)hipGetLastError(); return false; }
  return s == hipStreamCaptureStatusActive;
}
size_t bytes_for(const rl_token_logprob_desc* d, int S) { return S == 1 ? 0 : (size_t)d->n_rows * S * PER_SPLIT; }

thread_local hipError_t g_last = hipSuccess;

}  // namespace

extern "C" {

size_t rl_token_logprob_workspace_bytes(const rl_token_logprob_desc* d) {
  if (check(d) != 0) return 0;
  return bytes_for(d, splits_for(d));
}

int rl_token_logprob(const rl_token_logprob_desc* d, void* hip_stream) {
  const int rc = check(d);
  if (rc != 0) return rc;
  if (d->n_rows == 0) return 0;
  if (!d->logits || !d->token_ids) return -1;
  if (!d->ref_logits && (d->kl || d->ref_logprob)) return -1;
  if ((reinterpret_cast<uintptr_t>(d->logits) & 15u) || (reinterpret_cast<uintptr_t>(d->ref_logits) & 15u)) return -2;
  auto fits = [&](int splits) {
    const size_t need = bytes_for(d, splits);
    return need == 0 || (d->workspace && d->workspace_bytes >= need && !(reinterpret_cast<uintptr_t>(d->workspace) & 255u));
  };
  int S = splits_for(d);
  const bool less = !fits(S);
  if (less) S = splits_with_less(d);
  if (!fits(S)) return -3;
  const int vn = d->dtype == 0 ? 4 : 8;
  Params P{};
  P.logits = static_cast<const char*>(d->logits); P.ref = static_cast<const char*>(d->ref_logits);
  P.ids = d->token_ids;
  P.logprob = d->logprob; P.lse = d->lse; P.entropy = d->entropy; P.ref_logprob = d->ref_logprob; P.kl = d->kl;
  P.part = static_cast<float*>(d->workspace);
  const bool ref = d->ref_logits != nullptr;
  P.stride = d->row_stride; P.V = d->vocab; P.slots = S;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  bool one = S > 2 && row_bytes(d) * d->n_rows <= ONE_LAUNCH;
  if (one) {
    P.call = rlda::next_call();
    one = S <= MEET || !captured(st);
    --S;                                                    // the last slot is the counter's; captured or not, the bits are the same
  }
  P.S = S;
  const int per = (d->vocab + S - 1) / S;
  P.chunk = (per + vn - 1) / vn * vn;
  P.k2 = d->inv_temperature * 1.4426950408889634f;
  const dim3 grid((unsigned)(d->n_rows * S)), fin((unsigned)d->n_rows);
  // few workgroups, each with more than two rounds of loads for 256 threads (or none to share a row with): 16 wavefronts
  const bool wide = d->n_rows * S <= 512 && (S == 1 || less || row_bytes(d) / S > ROUNDS);
#define RLTL_LAUNCH(T)                                                                                      \
  do {                                                                                                      \
    if (one) {                                                                                              \
      if (wide && ref) hipLaunchKernelGGL((token_partial_kernel<T, true, 1024, true>), grid, dim3(1024), 0, st, P);   \
      else if (wide)   hipLaunchKernelGGL((token_partial_kernel<T, false, 1024, true>), grid, dim3(1024), 0, st, P);  \
      else if (ref)    hipLaunchKernelGGL((token_partial_kernel<T, true, 256, true>), grid, dim3(256), 0, st, P);     \
      else             hipLaunchKernelGGL((token_partial_kernel<T, false, 256, true>), grid, dim3(256), 0, st, P);    \
      break;                                                                                                \
    }                                                                                                       \
    if (wide) {                                                                                             \
      if (ref) hipLaunchKernelGGL((token_partial_kernel<T, true, 1024>), grid, dim3(1024), 0, st, P);       \
      else     hipLaunchKernelGGL((token_partial_kernel<T, false, 1024>), grid, dim3(1024), 0, st, P);      \
    } else {                                                                                                \
      if (ref) hipLaunchKernelGGL((token_partial_kernel<T, true, 256>), grid, dim3(256), 0, st, P);         \
      else     hipLaunchKernelGGL((token_partial_kernel<T, false, 256>), grid, dim3(256), 0, st, P);        \
    }                                                                                                       \
    if (S > 1) {                                                                                            \
      if (ref) hipLaunchKernelGGL((token_final_kernel<T, true>), fin, dim3(64), 0, st, P);                  \
      else     hipLaunchKernelGGL((token_final_kernel<T, false>), fin, dim3(64), 0, st, P);                 \
    }                                                                                                       \
  } while (0)
  if (d->dtype == 0) RLTL_LAUNCH(float); else RLTL_LAUNCH(uint16_t);
#undef RLTL_LAUNCH
  g_last = hipGetLastError();
  return g_last == hipSuccess ? 0 : -5;
}

}  // extern "C"
