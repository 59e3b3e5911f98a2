// Decode-step state transition for one attention layer (Sec. 3.1 of the paper, item (3):
// s' = (s, a)): rotary embedding of the new token's q and k (RoFormer rotation in the rotate-half
// pairing, three position components over sections of the frequency index), append of the rotated
// key and the value to the sequence's suffix store (contiguous or paged), length count.
//
// One workgroup per sequence.  The d/2 angles of a sequence are shared by all heads: they are
// evaluated once, in fp64 (64 or fewer evaluations per sequence; an fp32 product pos * inv_freq
// would already be off by 2e-3 rad at position 32k), rounded to fp32 and kept in LDS.  The rest is
// a few KB of element-wise work.  What bounds the kernel is how many round trips to memory follow each
// other, so a thread takes 16 bytes of either half of a head (a sequence's 28 + 4 heads of 128 bf16 are
// one pass of the workgroup) and requests them, its values and the lengths before the angles are
// evaluated.  Eight dependent passes of one element each took 6.5-7.3 us for 128 such sequences; now 3.1-4.0
// (a captured decode step of append, attention and combine 48.4 -> 44.5).  Buffers that are not aligned
// to 16 bytes take one element at a time, and so do heads so few that a thread has one or two elements anyway.
// Stores may hold e4m3 bytes: the appended rows are then divided by the KV head's factor and
// rounded to the nearest e4m3 value with integer operations (ties to even, saturating).
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/rl_kv_append.h"

namespace {

struct Params {
  char* q; const char* k_new; const char* v_new;
  const int32_t* pos; const float* inv_freq;
  char* ks; char* vs; const int32_t* table; int32_t* lens; const uint8_t* active;
  int B, Hq, Hkv, d, Ls_cap, page_shift, max_pages, n_pages;
  int s0, s1;                      // frequency indices below s0: temporal; below s0 + s1: height; else width
  const float* kscale; const float* vscale;   // e4m3 stores: per-KV-head factors, or null
};

template <typename T> struct Elt;
template <> struct Elt<float> {
  __device__ static float ld(const char* p, size_t i) { return reinterpret_cast<const float*>(p)[i]; }
  __device__ static void st(char* p, size_t i, float v) { reinterpret_cast<float*>(p)[i] = v; }
};
template <> struct Elt<uint16_t> {
  __device__ static float ld(const char* p, size_t i) {
    return __uint_as_float((uint32_t)reinterpret_cast<const uint16_t*>(p)[i] << 16);
  }
  __device__ static void st(char* p, size_t i, float v) {          // round to nearest even (finite values)
    const uint32_t u = __float_as_uint(v);
    reinterpret_cast<uint16_t*>(p)[i] = (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
  }
};

// fp32 -> e4m3 byte (1 sign, 4 exponent bits with bias 7, 3 mantissa bits, subnormals, no infinity):
// nearest value, ties to the even code, |y| > 448 -> 448, NaN -> 0x7f.
__device__ __forceinline__ uint8_t f32_to_e4m3(float y) {
  const uint32_t sign = (__float_as_uint(y) >> 24) & 0x80u;
  float a = fabsf(y);
  if (!(a == a)) return (uint8_t)(sign | 0x7Fu);
  a = fminf(a, 448.f);
  uint32_t code;
  if (a < 0.015625f) {                                      // below 2^-6 the grid is 2^-9; 8 steps reach the first normal
    code = (uint32_t)__float2int_rn(a * 512.f);
  } else {
    uint32_t b = __float_as_uint(a);
    b += 0x7FFFFu + ((b >> 20) & 1u);                       // nearest even at 3 mantissa bits; a carry moves the exponent
    code = (b >> 20) - (120u << 3);                         // exponent bias 127 -> 7
  }
  return (uint8_t)(sign | code);
}

// One rotated pair.  The products are rounded as written here (one fused, one not), so that every kernel gives the same bits.
__device__ __forceinline__ float rot_lo(float lo, float hi, float c, float s) { return __builtin_fmaf(lo, c, -__fmul_rn(hi, s)); }
__device__ __forceinline__ float rot_hi(float lo, float hi, float c, float s) { return __builtin_fmaf(hi, c, __fmul_rn(lo, s)); }

// how a rotated key element / a value element reaches the store
template <typename T, bool F8> struct Store {
  __device__ static void put(char* p, size_t i, float v, float) { Elt<T>::st(p, i, v); }
};
template <typename T> struct Store<T, true> {
  __device__ static void put(char* p, size_t i, float v, float factor) {
    reinterpret_cast<uint8_t*>(p)[i] = f32_to_e4m3(__fdiv_rn(v, factor));
  }
};

template <typename T, bool F8>
__global__ void __launch_bounds__(256) kv_append_rope_kernel(const Params P) {
  __shared__ float cs[64], sn[64];
  const int b = blockIdx.x, tid = threadIdx.x, half = P.d >> 1;
  if (tid < half) {
    const int comp = tid < P.s0 ? 0 : (tid < P.s0 + P.s1 ? 1 : 2);
    const double ang = (double)P.pos[(size_t)comp * P.B + b] * (double)P.inv_freq[tid];
    double s, c;
    sincos(ang, &s, &c);
    cs[tid] = (float)c; sn[tid] = (float)s;
  }
  // destination row of this sequence, if it takes one
  const int n = P.lens[b];
  const bool live = !P.active || P.active[b] != 0;
  const bool room = live && n >= 0 && n < P.Ls_cap;
  size_t row = 0;                                           // first element of row n, KV head 0; heads are `hstride` apart
  size_t hstride = 0;
  if (room) {
    if (P.table) {
      const int ps = 1 << P.page_shift;
      const int pg = min(max(P.table[(size_t)b * P.max_pages + (n >> P.page_shift)], 0), P.n_pages - 1);
      row = (((size_t)pg * P.Hkv) * ps + (n & (ps - 1))) * P.d;
      hstride = (size_t)ps * P.d;
    } else {
      row = (((size_t)b * P.Hkv) * P.Ls_cap + n) * P.d;
      hstride = (size_t)P.Ls_cap * P.d;
    }
  }
  __syncthreads();
  // q (in place) and k_new (to the store): one thread per (head, pair)
  const int pairs = (P.Hq + P.Hkv) * half;
  for (int idx = tid; idx < pairs; idx += 256) {
    const int head = idx / half, i = idx - head * half;
    const float c = cs[i], s = sn[i];
    if (head < P.Hq) {
      const size_t o = ((size_t)b * P.Hq + head) * P.d + i;
      const float lo = Elt<T>::ld(P.q, o), hi = Elt<T>::ld(P.q, o + half);
      Elt<T>::st(P.q, o, rot_lo(lo, hi, c, s));
      Elt<T>::st(P.q, o + half, rot_hi(lo, hi, c, s));
    } else if (room) {
      const int j = head - P.Hq;
      const size_t o = ((size_t)b * P.Hkv + j) * P.d + i;
      const float lo = Elt<T>::ld(P.k_new, o), hi = Elt<T>::ld(P.k_new, o + half);
      const size_t dst = row + j * hstride + i;
      const float f = F8 && P.kscale ? P.kscale[j] : 1.f;
      Store<T, F8>::put(P.ks, dst, rot_lo(lo, hi, c, s), f);
      Store<T, F8>::put(P.ks, dst + half, rot_hi(lo, hi, c, s), f);
    }
  }
  if (room) {
    for (int idx = tid; idx < P.Hkv * P.d; idx += 256) {    // the value row: a copy, or quantised
      const int j = idx / P.d, i = idx - j * P.d;
      const size_t src = ((size_t)b * P.Hkv + j) * P.d + i, dst = row + j * hstride + i;
      if (F8) Store<T, F8>::put(P.vs, dst, Elt<T>::ld(P.v_new, src), P.vscale ? P.vscale[j] : 1.f);
      else    reinterpret_cast<T*>(P.vs)[dst] = reinterpret_cast<const T*>(P.v_new)[src];
    }
    if (tid == 0) P.lens[b] = n + 1;                        // every thread read n before the barrier above
  }
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <typename T> struct Chunk;                         // 16 bytes of a row
template <> struct Chunk<float> {
  static constexpr int N = 4;
  __device__ static float get(const u32x4& c, int i) { return __uint_as_float(c[i]); }
  __device__ static void set(u32x4& c, int i, float v) { c[i] = __float_as_uint(v); }
};
template <> struct Chunk<uint16_t> {
  static constexpr int N = 8;
  __device__ static float get(const u32x4& c, int i) { return __uint_as_float(i & 1 ? c[i >> 1] & 0xFFFF0000u : c[i >> 1] << 16); }
  __device__ static void set(u32x4& c, int i, float v) {
    uint16_t h;
    Elt<uint16_t>::st(reinterpret_cast<char*>(&h), 0, v);
    c[i >> 1] = i & 1 ? (c[i >> 1] & 0xFFFFu) | (uint32_t)h << 16 : h;
  }
};

// a chunk of rotated keys or values into the store at element i
template <typename T, bool F8>
__device__ __forceinline__ void put_chunk(char* p, size_t i, const float (&v)[Chunk<T>::N], float factor) {
  if constexpr (F8) {
    uint32_t w[Chunk<T>::N / 4];
#pragma unroll
    for (int k = 0; k < Chunk<T>::N / 4; ++k) {
      w[k] = 0;
#pragma unroll
      for (int x = 0; x < 4; ++x) w[k] |= (uint32_t)f32_to_e4m3(__fdiv_rn(v[4 * k + x], factor)) << (8 * x);
    }
    *reinterpret_cast<uint2*>(p + i) = make_uint2(w[0], w[1]);
  } else {
    u32x4 c;
#pragma unroll
    for (int x = 0; x < Chunk<T>::N; ++x) Chunk<T>::set(c, x, v[x]);
    *reinterpret_cast<u32x4*>(p + i * sizeof(T)) = c;
  }
}

template <typename T, bool F8>
__global__ void __launch_bounds__(256) kv_append_rope_vec_kernel(const Params P) {
  constexpr int N = Chunk<T>::N;
  __shared__ __attribute__((aligned(16))) float cs[64], sn[64];
  const int b = blockIdx.x, tid = threadIdx.x, half = P.d >> 1, per_half = half / N;
  const int chunks = (P.Hq + P.Hkv) * per_half, vchunks = P.Hkv * 2 * per_half;
  auto rope_src = [&](int idx) {                            // the head's lower half; the upper one is `half` elements on
    const int head = idx / per_half, i = (idx - head * per_half) * N;
    return head < P.Hq ? P.q + (((size_t)b * P.Hq + head) * P.d + i) * sizeof(T)
                       : P.k_new + (((size_t)b * P.Hkv + head - P.Hq) * P.d + i) * sizeof(T);
  };
  const char* const vsrc = P.v_new + (size_t)b * P.Hkv * P.d * sizeof(T);
  u32x4 lo = {0, 0, 0, 0}, hi = {0, 0, 0, 0}, val = {0, 0, 0, 0};
  if (tid < chunks) {
    const char* const p = rope_src(tid);
    lo = *reinterpret_cast<const u32x4*>(p);
    hi = *reinterpret_cast<const u32x4*>(p + half * sizeof(T));
  }
  if (tid < vchunks) val = *reinterpret_cast<const u32x4*>(vsrc + (size_t)tid * 16);
  const int n = P.lens[b];
  const bool live = !P.active || P.active[b] != 0;
  if (tid < half) {
    const int comp = tid < P.s0 ? 0 : (tid < P.s0 + P.s1 ? 1 : 2);
    const double ang = (double)P.pos[(size_t)comp * P.B + b] * (double)P.inv_freq[tid];
    double s, c;
    sincos(ang, &s, &c);
    cs[tid] = (float)c; sn[tid] = (float)s;
  }
  const bool room = live && n >= 0 && n < P.Ls_cap;
  size_t row = 0, hstride = 0;                              // as above
  if (room) {
    if (P.table) {
      const int ps = 1 << P.page_shift;
      const int pg = min(max(P.table[(size_t)b * P.max_pages + (n >> P.page_shift)], 0), P.n_pages - 1);
      row = (((size_t)pg * P.Hkv) * ps + (n & (ps - 1))) * P.d;
      hstride = (size_t)ps * P.d;
    } else {
      row = (((size_t)b * P.Hkv) * P.Ls_cap + n) * P.d;
      hstride = (size_t)P.Ls_cap * P.d;
    }
  }
  __syncthreads();
  for (int idx = tid; idx < chunks; idx += 256) {
    const int head = idx / per_half, i = (idx - head * per_half) * N;
    if (idx != tid) {
      const char* const p = rope_src(idx);
      lo = *reinterpret_cast<const u32x4*>(p);
      hi = *reinterpret_cast<const u32x4*>(p + half * sizeof(T));
    }
    float a[N], z[N];
#pragma unroll
    for (int x = 0; x < N; ++x) {
      const float c = cs[i + x], s = sn[i + x], l = Chunk<T>::get(lo, x), h = Chunk<T>::get(hi, x);
      a[x] = rot_lo(l, h, c, s);
      z[x] = rot_hi(l, h, c, s);
    }
    if (head < P.Hq) {
      const size_t o = ((size_t)b * P.Hq + head) * P.d + i;
      put_chunk<T, false>(P.q, o, a, 1.f);
      put_chunk<T, false>(P.q, o + half, z, 1.f);
    } else if (room) {
      const int j = head - P.Hq;
      const size_t dst = row + j * hstride + i;
      const float f = F8 && P.kscale ? P.kscale[j] : 1.f;
      put_chunk<T, F8>(P.ks, dst, a, f);
      put_chunk<T, F8>(P.ks, dst + half, z, f);
    }
  }
  if (room) {
    for (int idx = tid; idx < vchunks; idx += 256) {
      const int j = idx / (2 * per_half), i = (idx - j * 2 * per_half) * N;
      const size_t dst = row + j * hstride + i;
      if (idx != tid) val = *reinterpret_cast<const u32x4*>(vsrc + (size_t)idx * 16);
      if constexpr (F8) {
        float v[N];
#pragma unroll
        for (int x = 0; x < N; ++x) v[x] = Chunk<T>::get(val, x);
        put_chunk<T, true>(P.vs, dst, v, P.vscale ? P.vscale[j] : 1.f);
      } else {
        *reinterpret_cast<u32x4*>(P.vs + dst * sizeof(T)) = val;
      }
    }
    if (tid == 0) P.lens[b] = n + 1;                        // every thread read n before the barrier above
  }
}

}  // namespace

extern "C" int rl_kv_append_rope(const rl_kv_append_desc* d, void* hip_stream) {
  if (!d) return -1;
  if (d->struct_size != sizeof(rl_kv_append_desc)) return -4;
  if (d->B < 0 || d->Hq <= 0 || d->Hkv <= 0 || d->d <= 0) return -1;
  if (d->dtype != 0 && d->dtype != 1 && d->dtype != 2) return -2;
  if (d->d != 64 && d->d != 128) return -2;
  if (d->sections[0] < 0 || d->sections[1] < 0 || d->sections[2] < 0 ||
      d->sections[0] + d->sections[1] + d->sections[2] != d->d / 2) return -2;
  const bool paged = d->block_table != nullptr;
  int cap = d->Ls_cap, shift = 0;
  if (paged) {
    if (d->page_size <= 0 || d->max_pages < 0 || d->n_pages < 1) return -1;
    if (d->page_size < 32 || (d->page_size & (d->page_size - 1))) return -2;
    if ((int64_t)d->max_pages * d->page_size > (int64_t)1 << 30) return -2;
    cap = d->max_pages * d->page_size;
    shift = __builtin_ctz((unsigned)d->page_size);
  } else if (cap < 0) {
    return -1;
  }
  if (d->B == 0) return 0;
  if (!d->q || !d->k_new || !d->v_new || !d->positions || !d->inv_freq || !d->suffix_lens) return -1;
  if (cap > 0 && (!d->k_store || !d->v_store)) return -1;
  Params P;
  P.q = static_cast<char*>(d->q); P.k_new = static_cast<const char*>(d->k_new); P.v_new = static_cast<const char*>(d->v_new);
  P.pos = d->positions; P.inv_freq = d->inv_freq;
  P.ks = static_cast<char*>(d->k_store); P.vs = static_cast<char*>(d->v_store);
  P.table = d->block_table; P.lens = d->suffix_lens; P.active = d->seq_active;
  P.B = d->B; P.Hq = d->Hq; P.Hkv = d->Hkv; P.d = d->d; P.Ls_cap = cap;
  P.page_shift = shift; P.max_pages = d->max_pages; P.n_pages = d->n_pages;
  P.s0 = d->sections[0]; P.s1 = d->sections[1];
  P.kscale = d->dtype == 2 ? d->k_scale : nullptr; P.vscale = d->dtype == 2 ? d->v_scale : nullptr;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  // 16 bytes at a time where every row starts on such a line (d is a multiple of 64, so the bases decide) and there is
  // enough to do: a thread with 16 bytes rounds 8 or 16 e4m3 values one after the other, where few heads leave other
  // threads without work.  us, 16 bytes / one element at a time, sequences x heads of 128 (64) columns:
  //   e4m3  128 x 3/1 6.0 / 3.6, 128 x 8/2 4.55 / 4.27, 128 x 28/4 (64) 4.7 / 4.5, 256 x 16/2 4.6 / 4.9, 128 x 8/8 5.5 / 6.1,
  //         4096 x 4/1 (64) 12.5 / 7.4, 2048 x 12/2 8.3 / 8.3, 2048 x 16/2 8.0 / 9.1
  //   bf16  64 x 2/2 (64) 3.34 / 3.21, 128 x 3/1 3.36 / 3.40, 128 x 4/4 3.3 / 3.9;   fp32  64 x 2/2 (64) 3.22 / 3.28
  const int64_t elements = (int64_t)(d->Hq + d->Hkv) * (d->d / 2) + (int64_t)d->Hkv * d->d;   // rotations and values
  static constexpr int64_t few[3] = {0, 256, 1280};
  const uintptr_t bases = (uintptr_t)P.q | (uintptr_t)P.k_new | (uintptr_t)P.v_new | (uintptr_t)P.ks | (uintptr_t)P.vs;
  typedef void (*kern_t)(const Params);
  static constexpr kern_t kerns[2][3] = {
      {kv_append_rope_kernel<float, false>, kv_append_rope_kernel<uint16_t, false>, kv_append_rope_kernel<uint16_t, true>},
      {kv_append_rope_vec_kernel<float, false>, kv_append_rope_vec_kernel<uint16_t, false>, kv_append_rope_vec_kernel<uint16_t, true>}};
  hipLaunchKernelGGL(kerns[bases % 16 == 0 && elements > few[d->dtype]][d->dtype], dim3(d->B), dim3(256), 0, st, P);
  return hipGetLastError() == hipSuccess ? 0 : -5;
}
