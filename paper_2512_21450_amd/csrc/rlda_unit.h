// Decode attention with one workgroup per unit: all keys of one (sequence, KV head) against its Hq/Hkv query rows,
// one launch; few units of many keys are shared by several workgroups each (SPLIT), if there is a workspace that no other call
// uses meanwhile (plans of RLDA_ALGO_SHARED, RLDA_ALGO_AUTO_SCRATCH).  Two uses:
//   * most of what the shared-prefix kernels do not take (fp32 stores, d = 64, wider head ratios, scales that are
//     not positive, pages under 32 rows), but for few rows over few keys, which the simple kernel runs faster
//     (unit_pays).  Weights enter the value contraction with 24 bits (EXACT below);
//   * batches so small that two dependent launches cost more than reading the prefix once per sequence
//     (unit_preferred).  Weights then have 16 bits (the shared-prefix kernels: 8) where 8 or 4 wavefronts share a
//     unit of two segments, or 8 one of a tree, and 24 in the forms with fewer.
//
// The NW = 8, 4, 2 or 1 wavefronts of a workgroup (unit_grid says how many) take the unit's 32-key tiles in turn
// (tile t goes to wavefront t % NW) and keep an online-softmax state each; the states meet in LDS at the end.  Tiles
// are numbered segment by segment (shared levels, then the own suffix), so the order of additions depends on the
// lengths and NW only.
//
// What bounds it: the round trips before the first product, and the 30 or so bytes a clock that a compute unit takes in (32
// to 128 units grow by 1.7 us per 8 tiles of 128 bf16 columns, 128 KB, and by 0.95 per 8 of 64).  A wavefront has the next tile on the way in registers while it computes on the present one,
// which goes through its private part of LDS.  (K straight into the registers of the matrix operand, 16 rows to an
// instruction, saved that trip but took the address unit four times as long as whole rows do: 1.05 us per 64 KB and
// compute unit.)  So the start is what counts for units of few tiles: the lengths are asked for first, then q and, where
// the first segment's capacity has room for a whole tile, the wavefront's first K tile, before the lengths are known (a
// tile that turns out shorter is loaded again: 512 units whose first segment is empty pay 0.3-0.7 us for it; asking for V as
// well gained 0.2 us more and cost those 1.0-1.7); the second tile is asked for before the first has landed; the place in
// the grid is found without divisions.  From the second tile on the next K and the next V are asked for apart, each as soon
// as its registers are free: both at once, after both had landed, cost units of many tiles up to 1.5 us of 16.  (fp32 of 64
// columns alone is faster with both at once and one copy of the step for the tiles from the second on, where a tile's rows lie
// together: 16 units of 30 and up to 3000 keys 28.7 apart / 27.6, on pages of 32 29.3 / 27.7, 16 of 309 and 1905 26.5 / 25.6, 64
// of 300 and 500 13.2 / 13.2; but on pages of 16 49.2 / 50.1, fp32 of 128 columns 26.3 / 27.4.)  A finished
// sequence's flag is looked at before anything of it is asked for (no measurable cost: 16 units of live sequences 5.43 / 5.38).
// Calls captured back to back, without all of this / so, us: 64 units x 256 keys, bf16, 64 columns 5.38 / 4.48, 128 columns
// 6.5 / 5.8, fp32 of 64 8.4 / 7.6; x 512 keys 6.4 / 5.4, 8.7 / 7.5, 11.9 / 11.2; e4m3 of 128 columns x 512 keys 8.3 / 7.3; 448
// units of up to 1864 keys, e4m3, 64 columns 20.2 / 18.4; 512 units of 452 and up to 1024 keys, bf16, 64 columns 19.1 / 18.0, on
// pages of 64 19.5 / 18.4, half finished 16.3 / 14.2; 512 units of 256 and up to 512, bf16, 128 columns, pages of 32, half
// finished 14.7 / 14.0 (with K and V at once 15.5).
// Samples of one prompt sit on one die, side by side in dispatch order, so that the prefix a group shares comes from
// memory once and from that die's L2 for the other samples.
//
// Units that are fewer than half the compute units and long are shared by up to 16 workgroups (split_rule): the wavefronts of
// all of them take the tiles in turn, every workgroup merges its own in LDS and leaves rows, maxima and sums in the workspace, and
// the one that arrives last (rlda_arrive.h) merges those, in order, so that the sum does not depend on who that is.  It costs about
// a microsecond, four dependent round trips; what it saves is the rounds of tiles behind one another (2.9 us each in fp32 of 64
// columns, 1.7 in bf16 of 128, 0.95 of 64).  How many take part follows from the lengths, on the device: short sequences in long
// buffers stay with one workgroup, the others end at once.  One workgroup / split, us, buffers full: 32 units of 1087 keys fp32
// 17.1 / 9.6, of 4064 46.7 / 18.4, 2 of 2048 25.0 / 7.7; bf16 of 64 columns 32 of 4000 18.4 / 11.5, 64 of 2048 11.8 / 10.7, 2 of
// 1024 6.8 / 6.1; e4m3 of 64 64 of 4000 19.5 / 12.1; bf16 of 128 32 of 1024 11.0 / 8.2, 8 of 2000 15.6 / 7.7.
//
// Tile math as in the shared-prefix kernels: S^T = K Q^T, so that a lane's accumulators (one query row, 4 keys per
// 16-key half) are the operand of O^T += V^T P^T.  A weight is split into two bf16 pieces (16 bits), EXACT: three (24),
// each contracted with V on the matrix cores; fp32 stores use the fp32 matrix instruction.
#pragma once

#include "rlda_arrive.h"
#include "rlda_internal.h"
#include "rlda_sched.h"

#include <float.h>
#include <math.h>

#include <mutex>
#include <type_traits>

namespace rlda {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr int MAX_SEG = RLDA_MAX_TREE_LEVELS + 1;
constexpr int MAX_UNIT_SPLITS = 16;
// keys shared by `group` consecutive sequences: stores [n, Hkv, cap, d], lens [n]
struct Segment { const char* k; const char* v; const int32_t* lens; int group, cap; FastDiv div; };   // div: by group

struct UnitParams {
  const char* q;
  float* out; float* lse;
  Segment seg[MAX_SEG];            // shared levels, then the own suffix (group 1), at index n_seg - 1
  int n_seg;
  int B, G, Hq, Hkv, r, RB;        // r = Hq / Hkv query rows in RB blocks of 16
  FastDiv div_per, div_RB, div_Hkv;   // quotients by G * RB, RB and Hkv
  int groups8;                     // (prompt, KV head) groups (SPLIT: times splits) rounded up to the dies, 0: units in plain order
  float scale, c, c_lo;            // and |scale| * log2(e) with what its rounding left; 1 and 0 when the scale is 0
  uint32_t qsign, qmask;           // q bits: & qmask (0 when the scale is 0), ^ qsign (for a negative factor), per 16-bit half or word
  const int32_t* table;            // paged suffix: [B, max_pages] page ids, else null
  int page_shift, max_pages, n_pages;
  const uint8_t* active;
  const float* kscale; const float* vscale;
  // units that several workgroups share (SPLIT): how many at most, from how many tiles on, what the grid counts first
  // (groups where groups8 is set, else units), the call's number, and in the workspace a counter per unit and, per workgroup and
  // row, the maximum with the weights' sum and the values against it
  int splits, min_tiles, n_first;
  FastDiv div_first;
  uint64_t call;
  uint64_t* arrived; uint64_t* part_ml; uint64_t* part_o;
};

enum Kind { KV_BF16, KV_F8, KV_F32 };

__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
#define RLDA_LDS(T, p) ((__attribute__((address_space(3))) T*)(p))
// max without the quieting of operands that fmaxf needs (no score is NaN here, or the result is NaN either way)
__device__ __forceinline__ float max_raw(float a, float b) {
  uint32_t inf = 0x7f800000u;
  asm("" : "+s"(inf));
  return __builtin_amdgcn_fmed3f(a, b, __uint_as_float(inf));
}
// maximum over the four lanes (l, l ^ 16, l ^ 32, l ^ 48) that share a query row
__device__ __forceinline__ float row_max(float t) {
  typedef unsigned int u32p __attribute__((ext_vector_type(2)));
  const u32p a = __builtin_amdgcn_permlane16_swap(__float_as_uint(t), __float_as_uint(t), false, false);
  t = max_raw(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const u32p b = __builtin_amdgcn_permlane32_swap(__float_as_uint(t), __float_as_uint(t), false, false);
  return max_raw(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ u32x2 e4m3x4_to_bf16(uint32_t w) {            // exact
  const bf16x2 lo = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, false);
  const bf16x2 hi = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, true);
  return u32x2{*reinterpret_cast<const uint32_t*>(&lo), *reinterpret_cast<const uint32_t*>(&hi)};
}
__device__ __forceinline__ void e4m3x16_to_bf16(const u32x4& w, u32x4& lo, u32x4& hi) {
  const u32x2 a = e4m3x4_to_bf16(w[0]), b = e4m3x4_to_bf16(w[1]), c = e4m3x4_to_bf16(w[2]), d = e4m3x4_to_bf16(w[3]);
  lo = u32x4{a[0], a[1], b[0], b[1]};
  hi = u32x4{c[0], c[1], d[0], d[1]};
}
__device__ __forceinline__ bf16x8 as_bf16x8(const u32x4& v) { return *reinterpret_cast<const bf16x8*>(&v); }

// Layout of one store type and head dimension.
template <int KIND, int D>
struct Lay {
  static constexpr int EB = KIND == KV_F32 ? 4 : (KIND == KV_F8 ? 1 : 2);   // bytes per stored element
  static constexpr int ROWB = D * EB;                  // a K/V row in the store
  static constexpr int LB = KIND == KV_F32 ? 4 : 2;    // bytes per element in LDS (e4m3 is widened on the way)
  static constexpr int LROWB = D * LB;
  static constexpr int TILE = TK * LROWB;              // one K or V tile in LDS
  static constexpr int NF = LROWB / 64;                // 16-byte fragments per lane of a row of q or K
  static constexpr int CPR = ROWB / 16;                // 16-byte chunks of a store row
  static constexpr int RPI = 64 / CPR;                 // tile rows per load instruction
  static constexpr int NL = TK / RPI;                  // load instructions per tile
  // xor pattern of the 16-byte chunks of K row `row` in LDS: a wavefront reads one chunk of 16 rows
  __device__ static __forceinline__ int kswz(int row) { return LROWB == 128 ? (row >> 1) & 7 : row & 15; }
  // the same for V: the transposing reads take 4 rows x 2 adjacent chunks
  // per 16 lanes, the fp32 reads 4 rows (4 apart) x 64 bytes per wavefront; either then touches every bank once
  __device__ static __forceinline__ int vswz(int row) {
    if (KIND == KV_F32) return ((row >> 2) & 3) << 2;
    return D == 128 ? (row & 7) << 1 : ((row >> 1) & 3) << 1;
  }
};

// Columns 4 ch .. 4 ch + 3 of a row: its values against the maximum M, L the sum of their weights; vfac 0: there is no key.  Returns
// whether one of them is not finite where the weights are.  (As a closure of the kernel this cost fp32 of 64 columns 64 register
// moves in the loop over the tiles and 0.1 us of 5.)
template <int D>
__device__ __forceinline__ bool write_row(const UnitParams& P, size_t orow, int ch, float vfac, float kabs, float M, float L, f32x4 acc) {
  acc *= vfac != 0.f ? vfac / L : 0.f;
  *reinterpret_cast<f32x4*>(P.out + orow * D + 4 * ch) = acc;
  if (P.lse && ch == 0) {
    const float f = fabsf(P.scale) * kabs, f_lo = f <= FLT_MAX ? fmaf(fabsf(P.scale), kabs, -f) : 0.f;
    const float log_l = __builtin_amdgcn_logf(L) * 0.69314718055994531f;
    P.lse[orow] = L > 0.f ? fmaf(M, f, fmaf(M, f_lo, log_l)) : -INFINITY;   // no key, or none that is a number
  }
  return L < INFINITY && !(fabsf(acc[0]) + fabsf(acc[1]) + fabsf(acc[2]) + fabsf(acc[3]) < INFINITY);
}

// NSEG: segments per sequence (2, or MAX_SEG for a tree); ROWS: pages of fewer rows than a tile, every row is looked up
// SPLIT: up to P.splits workgroups share a unit, wavefront for wavefront as if they were one; the last to end merges what they left
template <int KIND, int D, bool EXACT, int NW, int NSEG, bool ROWS, bool SPLIT>
__global__ void __launch_bounds__(64 * NW, KIND == KV_F32 && D == 128 ? 1 : 2) unit_kernel(const UnitParams P) {
  using L_ = Lay<KIND, D>;
  constexpr int CT = D / 16;                           // 16-column tiles of O
  constexpr int QE = KIND == KV_F32 ? 4 : 2;           // bytes per q element
  constexpr int NQ = L_::NF;                           // 16-byte q fragments per lane
  extern __shared__ __attribute__((aligned(16))) char lds[];
  __shared__ float wm[NW][16], wl[NW][16];
  const int tid = threadIdx.x, lane = tid & 63, wv = uni(tid >> 6), m16 = lane & 15, g = lane >> 4;

  // ---- which unit: sequence b, KV head j, row block rb
  int b, j, rb, split = 0;
  if (P.groups8 > 0) {
    const int xcd = blockIdx.x & 7, s = blockIdx.x >> 3, per = P.G * P.RB;
    const int round = fast_div(s, P.div_per), in = s - round * per;
    int grp = round * 8 + xcd;
    if constexpr (SPLIT) {                             // a group's samples meet in the same keys: what a die holds is one part of it
      split = fast_div(grp, P.div_first);
      grp -= split * P.n_first;
      if (split >= P.splits) return;
    }
    const int p = fast_div(grp, P.div_Hkv), own = fast_div(in, P.div_RB);
    j = grp - p * P.Hkv; b = p * P.G + own; rb = in - own * P.RB;
    if (!SPLIT && b >= P.B) return;                    // groups are rounded up to the eight dies
  } else {
    int at = blockIdx.x;
    if constexpr (SPLIT) {
      split = fast_div(at, P.div_first);
      at -= split * P.n_first;
    }
    const int u = fast_div(at, P.div_RB);
    rb = at - u * P.RB; b = fast_div(u, P.div_Hkv); j = u - b * P.Hkv;
  }
  const int nr = min(16, P.r - 16 * rb), h0 = j * P.r + 16 * rb;

  // ---- the segments: where they start, and their lengths, which are on their way while q and the first K tile are asked for
  size_t at[NSEG];
  int len[NSEG], first[NSEG], T = 0;
  const int act = P.active ? P.active[b] : 1;
#pragma unroll
  for (int s = 0; s < NSEG; ++s) {
    len[s] = 0; at[s] = 0;
    if (NSEG == 2 || s < P.n_seg) {
      const int owner = fast_div(b, P.seg[s].div);
      at[s] = ((size_t)owner * P.Hkv + j) * P.seg[s].cap * L_::ROWB;
      len[s] = P.seg[s].lens[owner];
    }
  }

  struct Tile { const char* k; const char* v; int n0, last; };            // n0: 0, or (ROWS, suffix) the tile's first key + 1
  auto tile_of = [&](int t) {
    Tile x{nullptr, nullptr, 0, 0};
#pragma unroll
    for (int s = 0; s < NSEG; ++s) {
      const bool own = NSEG == 2 ? s == 1 : s == P.n_seg - 1;
      if ((NSEG == 2 || s < P.n_seg) && t >= first[s] && len[s] > 0) {
        const int n0 = (t - first[s]) * TK;
        size_t off = at[s] + (size_t)n0 * L_::ROWB;
        x.last = min(TK, len[s] - n0) - 1;
        x.n0 = 0;
        if (own && P.table) {
          if constexpr (ROWS) {
            off = 0; x.n0 = n0 + 1;
          } else {                                     // a tile lies in one page
            const int pg = uni(clampi(P.table[(size_t)b * P.max_pages + (n0 >> P.page_shift)], 0, P.n_pages - 1));
            off = ((((size_t)pg * P.Hkv + j) << P.page_shift) + (n0 & ((1 << P.page_shift) - 1))) * L_::ROWB;
          }
        }
        x.k = P.seg[s].k + off;
        x.v = P.seg[s].v + off;
      }
    }
    return x;
  };
  // address of byte `byte` of tile row `i`; rows past the length re-read the last real row
  auto row_at = [&](const Tile& x, const char* base, int i, int byte) -> const char* {
    const int n = min(i, x.last);
    if constexpr (ROWS) {
      if (x.n0 > 0) {
        const int key = x.n0 - 1 + n;
        const int pg = clampi(P.table[(size_t)b * P.max_pages + (key >> P.page_shift)], 0, P.n_pages - 1);
        return base + ((((size_t)pg * P.Hkv + j) << P.page_shift) + (key & ((1 << P.page_shift) - 1))) * L_::ROWB + byte;
      }
    }
    return base + (uint32_t)(n * L_::ROWB + byte);     // uniform base, 32-bit offset
  };

  char* const kst = lds + wv * 2 * L_::TILE;           // this wavefront's K tile and V tile in LDS
  char* const vst = kst + L_::TILE;
  const int lrow = lane / L_::CPR, chunk = lane % L_::CPR;
  u32x4 kr[L_::NL], vr[L_::NL];
  // (inlined always: called, the registers of a tile whose rows are looked up would lie in scratch memory)
  auto load = [&](const Tile& x, const char* base, u32x4 (&r)[L_::NL]) __attribute__((always_inline)) {   // every instruction takes whole rows
#pragma unroll
    for (int i = 0; i < L_::NL; ++i) r[i] = *reinterpret_cast<const u32x4*>(row_at(x, base, L_::RPI * i + lrow, 16 * chunk));
  };
  auto store = [&](char* st, const u32x4 (&r)[L_::NL], auto swz) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < L_::NL; ++i) {
      const int row = L_::RPI * i + lrow;
      char* const dst = st + row * L_::LROWB;
      if constexpr (KIND == KV_F8) {
        u32x4 a, d;
        e4m3x16_to_bf16(r[i], a, d);
        *RLDA_LDS(u32x4, dst + (((2 * chunk) ^ swz(row)) << 4)) = a;
        *RLDA_LDS(u32x4, dst + (((2 * chunk + 1) ^ swz(row)) << 4)) = d;
      } else {
        *RLDA_LDS(u32x4, dst + ((chunk ^ swz(row)) << 4)) = r[i];
      }
    }
  };

  if (act == 0) {                                      // finished: nothing of it is read
    if (SPLIT && split > 0) return;
    for (int it = tid; it < nr * (D / 4); it += 64 * NW) {
      const int row = it / (D / 4), ch = it % (D / 4);
      const size_t orow = (size_t)b * P.Hq + h0 + row;
      *reinterpret_cast<f32x4*>(P.out + orow * D + 4 * ch) = f32x4{0.f, 0.f, 0.f, 0.f};
      if (P.lse && ch == 0) P.lse[orow] = -INFINITY;
    }
    return;
  }

  // ---- what needs no length: q, and the wavefront's first K tile where the first segment has room for all of it
  u32x4 qr[NQ], ka[L_::NL], va[L_::NL];
  const char* qp = P.q + ((size_t)b * P.Hq + h0 + min(m16, nr - 1)) * D * QE;
#pragma unroll
  for (int i = 0; i < NQ; ++i) qr[i] = *reinterpret_cast<const u32x4*>(qp + 64 * i + 16 * g);   // chunk 4 i + g, as K
  const int w0 = SPLIT ? split * NW + wv : wv;         // the wavefront's first tile
  const bool early = (w0 + 1) * TK <= P.seg[0].cap && (NSEG == 2 || P.n_seg > 1);
  if (early) {
    const size_t off = at[0] + (size_t)w0 * TK * L_::ROWB;
    const Tile guess{P.seg[0].k + off, P.seg[0].v + off, 0, TK - 1};
    load(guess, guess.k, ka);
  }

  // ---- tiles of the segments
#pragma unroll
  for (int s = 0; s < NSEG; ++s) {
    first[s] = T;
    if (NSEG == 2 || s < P.n_seg) {
      len[s] = clampi(len[s], 0, P.seg[s].cap);
      T += ceil_div(len[s], TK);
    }
  }
  int parts = 1;                                       // workgroups that share this unit
  if constexpr (SPLIT) {
    if (T >= P.min_tiles) parts = min(P.splits, ceil_div(T, NW));
    if (split >= parts) return;
  }
  uint64_t* const counter = SPLIT ? P.arrived + ((size_t)b * P.Hkv + j) * P.RB + rb : nullptr;
  uint64_t seen = 0;
  if (SPLIT && parts > 1 && tid == 0) seen = claim(counter, P.call);
  const int stride = SPLIT ? NW * parts : NW;          // from one tile of a wavefront to its next

  // The factor of the exponents meets differences of products only, so that the size of the scores costs a weight
  // nothing, and is kept positive and finite (a difference of 0 or -inf times it has to stay).  EXACT: what its rounding
  // left, the same for all keys, would show in lse; that part is positive too, for the same reason.
  const float ks = KIND == KV_F8 && P.kscale ? P.kscale[j] : 1.f, kabs = fabsf(ks);
  float c = P.c * kabs, c_lo = fmaf(P.c, kabs, -c) + P.c_lo * kabs;
  if (c < FLT_MIN) { c = FLT_MIN; c_lo = 0.f; }
  if (c > FLT_MAX) { c = FLT_MAX; c_lo = 0.f; }
  if (EXACT) {
    const float below = __uint_as_float(__float_as_uint(c) - 1);
    if (!(c_lo > 0.f) && c > FLT_MIN) { c_lo += c - below; c = below; }
    c_lo = max_raw(c_lo, FLT_MIN);
  }
  const float vfac = KIND == KV_F8 && P.vscale ? P.vscale[j] : 1.f;

  f32x4 O[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) O[ct] = f32x4{0.f, 0.f, 0.f, 0.f};
  // m: a product q . k, not yet times the scale; finite from the start, because products may be -inf (infinite keys, or an
  // overflow) and -inf less itself is not a number
  float m = -FLT_MAX, l = 0.f;

  // the tile whose K is in LDS, its first `nvalid` keys; `values` brings V there, once the weights are known
  auto step = [&](int nvalid, auto values) {
    // ---- scores of this lane's row (m16) for keys 4 g + x and 16 + 4 g + x
    // (fp32: two sums each, half as long a chain of roundings and of waits)
    f32x4 s0{0.f, 0.f, 0.f, 0.f}, s1{0.f, 0.f, 0.f, 0.f}, s2{0.f, 0.f, 0.f, 0.f}, s3{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < L_::NF; ++i) {
      const int off = m16 * L_::LROWB + (((4 * i + g) ^ L_::kswz(m16)) << 4);     // the pattern repeats after 16 rows
      const u32x4 k0 = *RLDA_LDS(const u32x4, kst + off), k1 = *RLDA_LDS(const u32x4, kst + off + 16 * L_::LROWB);
      if constexpr (KIND != KV_F32) {
        s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(k0), as_bf16x8(qr[i]), s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(k1), as_bf16x8(qr[i]), s1, 0, 0, 0);
      } else {
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          f32x4& a = i & 1 ? s2 : s0;
          f32x4& d = i & 1 ? s3 : s1;
          a = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(k0[x]), __uint_as_float(qr[i][x]), a, 0, 0, 0);
          d = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(k1[x]), __uint_as_float(qr[i][x]), d, 0, 0, 0);
        }
      }
    }
    if constexpr (KIND == KV_F32) { s0 += s2; s1 += s3; }

    // ---- online softmax in base 2; a row's reference maximum moves only when a tile exceeds it by a factor of 2^8
    // in the weights (fp32 holds the larger sums without loss)
    float sv[8];
#pragma unroll
    for (int x = 0; x < 4; ++x) { sv[x] = s0[x]; sv[4 + x] = s1[x]; }
    if (nvalid < TK)                                   // (uniform)
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        sv[x] = 4 * g + x < nvalid ? s0[x] : -INFINITY;
        sv[4 + x] = 16 + 4 * g + x < nvalid ? s1[x] : -INFINITY;
      }
    float tm = max_raw(max_raw(max_raw(sv[0], sv[1]), max_raw(sv[2], sv[3])),
                       max_raw(max_raw(sv[4], sv[5]), max_raw(sv[6], sv[7])));
    tm = row_max(tm);
    const float mn = max_raw(m, tm);
    if (__any((mn - m) * c > 8.f || m == -FLT_MAX)) {  // or a wavefront's first tile
      const float al = __builtin_amdgcn_exp2f((m - mn) * c);
      l *= al;
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) O[ct] *= al;
      m = mn;
    }
    float p[8];
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      const float dx = sv[x] - m, e = dx * c;
      p[x] = __builtin_amdgcn_exp2f(EXACT ? fmaf(dx, c_lo, e) : e);
    }
    l += ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));

    values();

    // ---- O^T += V^T P^T
    if constexpr (KIND == KV_F32) {
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const int row = 4 * g + x;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          const int off = (((4 * ct + (m16 >> 2)) ^ L_::vswz(row)) << 4) + 4 * (m16 & 3);
          const float v0 = *RLDA_LDS(const float, vst + row * L_::LROWB + off);
          const float v1 = *RLDA_LDS(const float, vst + (row + 16) * L_::LROWB + off);   // the pattern repeats after 16 rows
          O[ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(v0, p[x], O[ct], 0, 0, 0);
          O[ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(v1, p[4 + x], O[ct], 0, 0, 0);
        }
      }
    } else {
      constexpr int NP = EXACT ? 3 : 2;                // bf16 pieces of a weight
      bf16x8 pb[NP];
      float rest[8];
#pragma unroll
      for (int x = 0; x < 8; ++x) rest[x] = p[x];
#pragma unroll
      for (int k = 0; k < NP; ++k)
#pragma unroll
        for (int x = 0; x < 8; x += 2) {
          const bf16x2 pr = __builtin_convertvector(f32x2{rest[x], rest[x + 1]}, bf16x2);
          pb[k][x] = pr[0]; pb[k][x + 1] = pr[1];
          if (k + 1 < NP) {                            // exact: what the piece leaves has fewer bits
            rest[x] -= static_cast<float>(pr[0]);
            rest[x + 1] -= static_cast<float>(pr[1]);
          }
        }
      // a 16-lane group addresses rows 4 g .. 4 g + 3, columns 16 ct .. 16 ct + 15, and a lane receives its column of them
      const int vrow = 4 * g + (m16 >> 2);
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        const int off = (((2 * ct + ((m16 & 3) >> 1)) ^ L_::vswz(vrow)) << 4) + ((m16 & 1) << 3);
        union { s16x4 h[2]; bf16x8 v; } vt;
        vt.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(RLDA_LDS(s16x4, vst + vrow * L_::LROWB + off));
        vt.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(RLDA_LDS(s16x4, vst + (vrow + 16) * L_::LROWB + off));
#pragma unroll
        for (int k = NP - 1; k >= 0; --k) O[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt.v, pb[k], O[ct], 0, 0, 0);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");   // LDS serves a wavefront in order: the stage may be rewritten
    __builtin_amdgcn_wave_barrier();
  };
  if (w0 < T) {
    const Tile cur = tile_of(w0);
    if (!(early && (w0 + 1) * TK <= len[0])) load(cur, cur.k, ka);
    load(cur, cur.v, va);
    const uint32_t qm = m16 < nr ? P.qmask : 0u;
    const uint32_t qs = m16 < nr && (P.scale < 0.f) != (ks < 0.f) ? P.qsign : 0u;
    Tile nxt = cur;
    // the second tile is asked for before the first has landed; in branches of their own, so that the wait for the first
    // counts the loads that follow it
    if (w0 + stride < T) {
      nxt = tile_of(w0 + stride);
      load(nxt, nxt.k, kr); load(nxt, nxt.v, vr);
      store(kst, ka, L_::kswz);
      store(vst, va, L_::vswz);
    } else {
      store(kst, ka, L_::kswz);
      store(vst, va, L_::vswz);
    }
#pragma unroll
    for (int i = 0; i < NQ; ++i) qr[i] = (qr[i] & qm) ^ qs;
    auto staged = [] {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
    };
    staged();
    step(cur.last + 1, [] {});
    // The next K is asked for before the scores and the next V before the values, as soon as its registers are free.  The last
    // tile is a copy of its own: the waits of the others then count exactly the loads that follow.
    auto turn = [&](auto more, int t) {                // more: tile t + stride follows
      constexpr bool MORE = decltype(more)::value;
      const int nvalid = nxt.last + 1;
      store(kst, kr, L_::kswz);
      if constexpr (MORE) { nxt = tile_of(t + stride); load(nxt, nxt.k, kr); }
      staged();
      step(nvalid, [&] {
        store(vst, vr, L_::vswz);
        if constexpr (MORE) load(nxt, nxt.v, vr);
        staged();
      });
    };
    int t = w0 + stride;
    if constexpr (KIND == KV_F32 && D == 64 && !ROWS) {   // both at once, see above
      for (; t < T; t += stride) {
        const int nvalid = nxt.last + 1;
        store(kst, kr, L_::kswz);
        store(vst, vr, L_::vswz);
        if (t + stride < T) { nxt = tile_of(t + stride); load(nxt, nxt.k, kr); load(nxt, nxt.v, vr); }
        staged();
        step(nvalid, [] {});
      }
    } else {
      for (; t + stride < T; t += stride) turn(std::true_type{}, t);
      if (t < T) turn(std::false_type{}, t);
    }
  }

  // ---- merge: every wavefront leaves its rows (O against its own maximum) in its stages, from the K stage on
  l += __shfl_xor(l, 16, 64); l += __shfl_xor(l, 32, 64);
  constexpr int OC = D / 4;                            // 16-byte chunks of an O row
  constexpr int OROWB = D * 4;
  constexpr int OSTRIDE = 2 * L_::TILE;
  static_assert(16 * OROWB <= OSTRIDE, "a wavefront's O rows fit its stage");
  if (m16 < nr) {
    char* o = lds + wv * OSTRIDE + m16 * OROWB;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) *RLDA_LDS(f32x4, o + (((4 * ct + g) ^ m16) << 4)) = O[ct];
  }
  if (g == 0) { wm[wv][m16] = m; wl[wv][m16] = l; }
  __syncthreads();
  bool odd = false;                                    // a column that is not finite where the row's weights are
  for (int it = tid; it < nr * OC; it += 64 * NW) {
    const int row = it / OC, ch = it % OC;
    float M = wm[0][row];                              // a wavefront without a tile: the lowest maximum, and zeros
#pragma unroll
    for (int w = 1; w < NW; ++w) M = fmaxf(M, wm[w][row]);
    float L = 0.f;
    f32x4 acc{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float a = __builtin_amdgcn_exp2f((wm[w][row] - M) * c);
      L = fmaf(a, wl[w][row], L);
      const f32x4 o = *RLDA_LDS(const f32x4, lds + w * OSTRIDE + row * OROWB + ((ch ^ row) << 4));
#pragma unroll
      for (int x = 0; x < 4; ++x) acc[x] = fmaf(a, o[x], acc[x]);
    }
    const size_t orow = (size_t)b * P.Hq + h0 + row;
    if (SPLIT && parts > 1) {
      const size_t at_row = (size_t)split * P.B * P.Hq + orow;
      put(P.part_o + at_row * (D / 2) + 2 * ch, acc[0], acc[1]);
      put(P.part_o + at_row * (D / 2) + 2 * ch + 1, acc[2], acc[3]);
      if (ch == 0) put(P.part_ml + at_row, M, L);
      continue;
    }
    odd = write_row<D>(P, orow, ch, T > 0 ? vfac : 0.f, kabs, M, L, acc) || odd;
  }
  if constexpr (SPLIT) {
    if (parts > 1) {
      __shared__ bool last;
      stores_done();
      __syncthreads();
      if (tid == 0) last = arrive(counter, P.call, seen, parts);
      __syncthreads();
      if (!last) return;
      for (int it = tid; it < nr * OC; it += 64 * NW) {
        const int row = it / OC, ch = it % OC;
        const size_t orow = (size_t)b * P.Hq + h0 + row, step_ml = (size_t)P.B * P.Hq;
        const uint64_t* const ml = P.part_ml + orow;
        const uint64_t* const o = P.part_o + orow * (D / 2) + 2 * ch;
        float M = -FLT_MAX, L = 0.f;
        f32x4 acc{0.f, 0.f, 0.f, 0.f};
        constexpr int U = 8;                           // parts asked for at once
        for (int k0 = 0; k0 < parts; k0 += U) {
          float2 mlv[U], oa[U], ob[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const size_t k = min(k0 + u, parts - 1) * step_ml;
            mlv[u] = get(ml + k);
            oa[u] = get(o + k * (D / 2));
            ob[u] = get(o + k * (D / 2) + 1);
          }
          float Mn = M;
#pragma unroll
          for (int u = 0; u < U; ++u) Mn = fmaxf(Mn, mlv[u].x);
          const float resc = __builtin_amdgcn_exp2f((M - Mn) * c);
          L *= resc; acc *= resc;
          M = Mn;
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (k0 + u < parts) {
              const float a = __builtin_amdgcn_exp2f((mlv[u].x - M) * c);
              L = fmaf(a, mlv[u].y, L);
              acc[0] = fmaf(a, oa[u].x, acc[0]); acc[1] = fmaf(a, oa[u].y, acc[1]);
              acc[2] = fmaf(a, ob[u].x, acc[2]); acc[3] = fmaf(a, ob[u].y, acc[3]);
            }
        }
        odd = write_row<D>(P, orow, ch, vfac, kabs, M, L, acc) || odd;
      }
    }
  }
  // An infinite value gives an infinite result; but split weights leave pieces of 0 or below zero, and rows past the
  // length repeat the last one at weight 0, and either makes it NaN.  Such columns are the sum of what is not finite.
  // (In a loop of its own, which reads the arguments again: inside the one above, or with what the tiles used kept for it,
  // it cost 0.3 us of 9 without being entered.)
  if constexpr (KIND != KV_F8) {                       // e4m3 has no infinity
    if (!odd) return;
    typedef const __attribute__((address_space(4))) UnitParams* args_t;
    args_t A = (args_t)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(A));
    for (int it = tid; it < nr * OC; it += 64 * NW) {
      const int row = it / OC, ch = it % OC;
      float L = 0.f;
      if (SPLIT && parts > 1) {
        for (int k = 0; k < parts; ++k) L += get(A->part_ml + (size_t)k * A->B * A->Hq + (size_t)b * A->Hq + h0 + row).y;
      } else {
        for (int w = 0; w < NW; ++w) L += wl[w][row];
      }
      if (!(L < INFINITY)) continue;                   // a score that is not a number: the row is none
      f32x4 sum{0.f, 0.f, 0.f, 0.f};
      for (int s = 0; s < A->n_seg; ++s) {
        const int owner = b / A->seg[s].group, cap = A->seg[s].cap, n_keys = clampi(A->seg[s].lens[owner], 0, cap);
        for (int n = 0; n < n_keys; ++n) {
          size_t at = ((size_t)owner * A->Hkv + j) * cap + n;
          if (A->table && s == A->n_seg - 1) {
            const int pg = clampi(A->table[(size_t)b * A->max_pages + (n >> A->page_shift)], 0, A->n_pages - 1);
            at = (((size_t)pg * A->Hkv + j) << A->page_shift) + (n & ((1 << A->page_shift) - 1));
          }
          const char* const src = A->seg[s].v + at * L_::ROWB + 4 * ch * L_::EB;
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const float v = KIND == KV_F32 ? reinterpret_cast<const float*>(src)[k]
                                           : __uint_as_float((uint32_t)reinterpret_cast<const uint16_t*>(src)[k] << 16);
            if (!(fabsf(v) < INFINITY)) sum[k] += v;
          }
        }
      }
      float* const o = P.out + ((size_t)b * P.Hq + h0 + row) * D + 4 * ch;
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (sum[k] != 0.f) o[k] = sum[k];
    }
  }
}

template <int KIND, int D, bool EXACT, int NW, int NSEG = 2, bool ROWS = false, bool SPLIT = false>
hipError_t launch(const UnitParams& P, int64_t blocks, hipStream_t stream) {
  constexpr int lds = NW * 2 * Lay<KIND, D>::TILE;
  // once per device: more than 64 KB of LDS in total needs an opt-in
  static std::mutex mu;
  static bool done[64] = {};
  if (lds + 4096 > 65536) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lock(mu);
    if (dev < 0 || dev >= 64 || !done[dev]) {
      e = hipFuncSetAttribute(reinterpret_cast<const void*>(unit_kernel<KIND, D, EXACT, NW, NSEG, ROWS, SPLIT>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, lds);
      if (e != hipSuccess) return e;
      if (dev >= 0 && dev < 64) done[dev] = true;
    }
  }
  hipLaunchKernelGGL((unit_kernel<KIND, D, EXACT, NW, NSEG, ROWS, SPLIT>), dim3((unsigned)blocks), dim3(64 * NW), lds, stream, P);
  return hipGetLastError();
}

// two fp32 tiles of 128 columns take half a SIMD's registers
constexpr int wide_waves(bool f32, int d) { return f32 && d == 128 ? 4 : 8; }

// pages of fewer rows than a tile: every row is looked up
bool row_lookup(const Problem& pb) { return pb.block_table && pb.page_shift < 5; }
int64_t shared_cap(const Problem& pb) {
  int64_t n = pb.Lp_cap;
  for (int l = 0; l < pb.n_levels; ++l) n += pb.levels[l].cap;
  return n;
}

// Grid of a problem (n_sequences > 0).
struct UnitGrid {
  int groups8;                     // as in UnitParams
  int64_t blocks;
  int nw;                          // wavefronts of a workgroup
  int splits, min_tiles;           // workgroups of a unit at most, and the tiles from which on it gets more than one
};

// What a unit shared by several workgroups leaves in the workspace: a counter, and per workgroup and row the values, their
// maximum and the weights' sum.
size_t split_counters(const Problem& pb) {             // rounded up so that what follows starts on 256 bytes
  return ((size_t)n_sequences(pb) * pb.Hkv * ceil_div(pb.Hq / pb.Hkv, 16) + 31) & ~(size_t)31;
}
size_t split_bytes(const Problem& pb, int splits) {
  return split_counters(pb) * 8 + (size_t)splits * n_sequences(pb) * pb.Hq * (8 + (size_t)pb.d * 4);
}

// (group, part) pairs that a die takes, or 0: fewer than two of them, plain order, so that neighbours spread over the dies
int64_t die_groups(const Problem& pb, int splits) {
  const int64_t n = n_sequences(pb) / max_group(pb) * pb.Hkv * splits;
  return n >= 16 && max_group(pb) > 1 ? (n + 7) / 8 : 0;
}
int64_t unit_blocks(const Problem& pb, int splits) {
  const int64_t rb = ceil_div(pb.Hq / pb.Hkv, 16), g8 = die_groups(pb, splits);
  return g8 > 0 ? g8 * 8 * max_group(pb) * rb : n_sequences(pb) * pb.Hkv * rb * splits;
}
int full_tiles(const Problem& pb) {                    // of a sequence that fills its buffers (up to the largest int)
  const auto of = [](int cap) { return cap / TK + (cap % TK != 0); };
  int n = of(pb.Ls_cap) + of(pb.Lp_cap);
  for (int l = 0; l < pb.n_levels; ++l) n += of(pb.levels[l].cap);
  return n;
}

struct Split { int splits, nw, min_tiles; };
// How many workgroups share a unit at most: as many as the compute units hold, up to 16, and more than one from `min_tiles` of the unit's
// real tiles on, if the buffers hold half as many again: workgroups that find nothing to do cost 0.3 to 0.7 us (80 units of e4m3, 128
// columns, capacities 520 + 24, half full 6.9 / 7.3).  Eight wavefronts each, as one workgroup has; but where the buffers hold 32 tiles at most and there is a compute unit for
// every four of them, workgroups of four, so that each wavefront has one tile and more compute units share them.  Both where a round
// of tiles costs enough: not in 16-bit stores of 64 columns.  us, one workgroup / eight wavefronts each / four each:
//   fp32, 64 columns, 512 keys: 2 units 9.6 / 7.7 / 6.8, 64 10.9 / 9.2 / 8.3; 1024 keys: 2 14.8 / 8.3 / 6.9, 64 16.6 / 11.9 / 12.2
//   bf16, 128 columns, 512 keys: 32 7.2 / 7.1 / 6.8, half full 6.0 / 7.1 / 6.5 (so not below 800 keys; fp32 400); 1024 keys: 2 9.9 / 7.0 / 6.4, 64 11.5 / 10.8 / 11.5
//   bf16, 64 columns, 512 keys: 32 5.3 / 6.2 / 6.1; 1024 keys: 32 6.9 / 6.6 / 6.9
// With two workgroups to a unit (86 to 128 of them on 256 compute units) the saving is half of that and the memory is nearly busy: from
// more tiles on only (128 units, one / two: fp32 512 keys 11.1 / 9.8, 384 8.1 / 8.1; bf16 of 128 columns 1024 11.8 / 12.5, 1088 11.1 /
// 10.4, 2048 18.7 / 17.4; bf16 of 64 1024 8.2 / 9.1, 2112 10.6 / 9.5), and not where the sequences' own keys are most of a call in bf16
// of 64 columns (64 + 2048 keys 13.6 / 15.2, half full 9.4 / 10.7; e4m3 12.9 / 12.3).  Where buffers are far from full there may be next
// to nothing in it (64 units of 1100 + up to 256 keys in four parts 13.8 / 13.6).  200 drawn calls of fp32 and 64 columns: 1.80 times as
// fast full, 1.67 with lengths spread, the least 1.03 and 0.98.  More than half as many units as compute units
// gain nothing (256 units of 1088 to 4000 keys: 2 to 15 % slower).  Nor do parts that no compute unit is free for: a die takes whole
// (group, part) pairs, and where their number is no multiple of eight some would get a second round of workgroups (e4m3, 10 prompts of
// 5 samples, 3888 + 2760 keys: five parts, 35 workgroups on a die, 27.4, four 20.8; bf16, 3000 + 2000 keys 27.7 / 20.3).
Split split_rule(const Problem& pb, int pairs) {
  const int64_t units = n_sequences(pb) * pb.Hkv * ceil_div(pb.Hq / pb.Hkv, 16);
  const bool f32 = pb.dtype == RLDA_F32, wide = pb.d == 128;
  Split s{1, 0, 0};
  if (2 * units > pairs || units < 1 || (pb.paged && pb.page_shift < 5)) return s;   // (a query brings no table)
  const int tiles = full_tiles(pb), n = pairs / (int)units, most = n < MAX_UNIT_SPLITS ? n : MAX_UNIT_SPLITS;
  if (tiles > (f32 ? 12 : 24) && tiles <= 32 && (f32 || wide) && ceil_div(tiles, 4) <= n) {
    s.nw = 4;
    s.min_tiles = 5;
  } else {
    s.nw = wide_waves(f32, pb.d);
    s.min_tiles = f32 ? (n > 2 ? 9 : 14) : wide ? (n > 2 ? 17 : 41) : (n > 2 ? 25 : 57);
    if (n == 2 && pb.dtype == RLDA_BF16 && !wide && units * pb.Ls_cap > (int64_t)512 * pairs) return s;
  }
  if (2 * tiles >= 3 * s.min_tiles) s.splits = most < ceil_div(tiles, s.nw) ? most : ceil_div(tiles, s.nw);
  const int held = (160 << 10) / (s.nw * 2 * TK * pb.d * (f32 ? 4 : 2));   // workgroups in the LDS of a compute unit
  while (s.splits > 1 && unit_blocks(pb, s.splits) > (int64_t)held * pairs) --s.splits;
  return s;
}

// How many wavefronts a unit gets.  Eight while every workgroup has a compute unit to itself (128 units x 964 keys: 11.7 us,
// 12.7 with four).  When workgroups queue, what counts is how many units are on their way at once: a workgroup holds the
// LDS of all its wavefronts from the first length it reads to the last row it writes, so the more of them there are and
// the shorter they are, the fewer wavefronts each may take.  Measured, us with 8 / 4 / 2 / 1 wavefronts:
//   fp32, 64 columns    512 units x 1024 keys     42 / 38 / 50 / 61     1024 x 64     19 / 14 / 10.6 / 9.8
//                      4096 x 64                   68 / 41 / 28 / 24     4096 x 1024  280 / 253 / 265 / 283
//   bf16, 64 columns   1024 x 256                14.3 / 12.0 / 12.5 / 13.2       16384 x 32   104 / 56 / 36 / 29
//   fp32, 128 columns   512 x 256                   - / 25 / 23 / 31     4096 x 64      - / 108 / 62 / 49
//   small batches (two bf16 pieces), 1024 x 128  19.8 / 14.8 / 12.6 / 13.1        8192 x 64    137 / 85 / 66 / 66
//   pages of 16 rows, bf16, 128 columns  320 x 1000  38 / 44 / - / -     512 x 1000  44 / 40 / - / -   1024 x 64 34 / 21 / 13 / 14
//                                        256 x 1024  26 / 39 / 62 / 108  4096 x 256   223 / 134 / 134 / 117
UnitGrid unit_grid(const Problem& pb, int pairs, bool exact, Split sp) {
  const int64_t keys = shared_cap(pb) + pb.Ls_cap;
  UnitGrid u{};
  u.splits = sp.splits;
  u.groups8 = (int)die_groups(pb, sp.splits);
  u.blocks = unit_blocks(pb, sp.splits);
  if (sp.splits > 1) {
    u.nw = sp.nw; u.min_tiles = sp.min_tiles;
    return u;
  }
  const bool f32 = pb.dtype == RLDA_F32, many = u.blocks > 4 * (int64_t)pairs;
  // workgroups of four wavefronts that the compute units' LDS holds (tiles of 64 16-bit columns are half as large), and a
  // quarter more, which follow as soon as short units end: 528 units of up to 182 keys 9.5 us with four, 10.0 with two
  const int64_t fit = (pb.d == 64 && !f32 ? 4 : 2) * (int64_t)pairs * 5 / 4;
  // rows looked up one by one make a long chain, worth more wavefronts than the queue costs a little longer
  if (u.blocks <= pairs || (row_lookup(pb) && keys >= 512 && 2 * u.blocks <= 3 * (int64_t)pairs)) {
    u.nw = wide_waves(f32, pb.d);
  } else if (row_lookup(pb) || pb.n_levels > 1) {
    u.nw = many ? 1 : (u.blocks > 2 * (int64_t)pairs || (f32 && pb.d == 128) ? 2 : 4);
  } else if (f32 && pb.d == 128) {
    u.nw = u.blocks > fit && keys <= 256 ? 1 : 2;
  } else if (u.blocks <= fit || (exact && (keys >= 512 || (keys >= 256 && u.blocks <= 8 * (int64_t)pairs)))) {
    u.nw = 4;
  } else {
    u.nw = u.blocks > 2 * fit && (!exact || keys <= 128) ? 1 : 2;
  }
  return u;
}
UnitGrid unit_grid(const Problem& pb, int pairs, bool exact) {
  Split sp = split_rule(pb, pairs);
  while (sp.splits > 1 && (!pb.workspace || (reinterpret_cast<uintptr_t>(pb.workspace) & 255u) || split_bytes(pb, sp.splits) > pb.workspace_bytes))
    --sp.splits;                                       // a caller with less workspace than asked for, or none
  return unit_grid(pb, pairs, exact, sp);
}

// The form of one store type and head dimension: pages of fewer rows than a tile, a tree, or two segments.  The fewer
// wavefronts share a unit's tiles, the fewer of a row's large weights are a tile's own maximum, which is 1 and needs no
// bits: few wavefronts keep all 24 of the others (16 bits: 1.7e-6 of out against 64 bits, 1.1e-6 with one tile a wavefront).
template <int KIND, int D, bool EXACT>
hipError_t launch_form(const UnitParams& P, int nw, int64_t blocks, hipStream_t stream) {
  constexpr int WIDE = wide_waves(KIND == KV_F32, D);
  if (P.splits > 1) {
    if constexpr (KIND == KV_BF16 && D == 128 && !EXACT)
      if (P.n_seg != 2) return nw == 4 ? launch<KIND, D, true, 4, MAX_SEG, false, true>(P, blocks, stream)
                                       : launch<KIND, D, EXACT, WIDE, MAX_SEG, false, true>(P, blocks, stream);
    return nw == 4 ? launch<KIND, D, EXACT, 4, 2, false, true>(P, blocks, stream)
                   : launch<KIND, D, EXACT, WIDE, 2, false, true>(P, blocks, stream);
  }
  if constexpr (EXACT)                                        // the shared-prefix path refuses small pages, so only here
    if (P.table && P.page_shift < 5) {
      if (nw == 1) return launch<KIND, D, EXACT, 1, 2, true>(P, blocks, stream);
      if (nw == 2) return launch<KIND, D, EXACT, 2, 2, true>(P, blocks, stream);
      if (nw == 4) return launch<KIND, D, EXACT, 4, 2, true>(P, blocks, stream);
      return launch<KIND, D, EXACT, WIDE, 2, true>(P, blocks, stream);
    }
  if constexpr (KIND == KV_BF16 && D == 128 && !EXACT)        // what a tree holds
    if (P.n_seg != 2) {
      if (nw == 1) return launch<KIND, D, true, 1, MAX_SEG>(P, blocks, stream);
      if (nw == 2) return launch<KIND, D, true, 2, MAX_SEG>(P, blocks, stream);
      if (nw == 4) return launch<KIND, D, true, 4, MAX_SEG>(P, blocks, stream);
      return launch<KIND, D, EXACT, WIDE, MAX_SEG>(P, blocks, stream);
    }
  if (nw == 1) return launch<KIND, D, true, 1>(P, blocks, stream);
  if (nw == 2) return launch<KIND, D, true, 2>(P, blocks, stream);
  return nw == 4 ? launch<KIND, D, EXACT, 4>(P, blocks, stream) : launch<KIND, D, EXACT, WIDE>(P, blocks, stream);
}

}  // namespace

// stores, q and outputs start on 16 bytes (the loads are that wide), lengths fit the 32-bit tile arithmetic, and the
// launch its limit of 2^32 threads (the simple kernel spends 64 threads on a row and takes the calls beyond)
bool unit_supported(const Problem& pb, int pairs) {
  if (!(pb.scale - pb.scale == 0.f)) return false;                     // an infinite or NaN factor: the simple kernel's result
  uintptr_t a = reinterpret_cast<uintptr_t>(pb.q) | reinterpret_cast<uintptr_t>(pb.out) |
                reinterpret_cast<uintptr_t>(pb.k_suffix) | reinterpret_cast<uintptr_t>(pb.v_suffix);
  int64_t cap = pb.Ls_cap;
  if (pb.n_levels > 0) {
    for (int l = 0; l < pb.n_levels; ++l) {
      a |= reinterpret_cast<uintptr_t>(pb.levels[l].k) | reinterpret_cast<uintptr_t>(pb.levels[l].v);
      cap += pb.levels[l].cap;
    }
  } else {
    a |= reinterpret_cast<uintptr_t>(pb.k_prefix) | reinterpret_cast<uintptr_t>(pb.v_prefix);
    cap += pb.Lp_cap;
  }
  if ((a & 15u) || cap > (int64_t)1 << 30) return false;
  if (n_sequences(pb) * pb.Hkv * ceil_div(pb.Hq / pb.Hkv, 16) < (int64_t)1 << 20) return true;   // 512 threads each, rounded up, and splits
  for (bool exact : {false, true}) {
    const UnitGrid u = unit_grid(pb, pairs, exact);
    if (u.blocks * 64 * u.nw >= (int64_t)1 << 32) return false;
  }
  return true;
}

// Where one wavefront per query head is faster than one workgroup per KV head, among what the shared-prefix path does not
// take: few rows that share a KV head over few keys, so that little is shared and the tiles are mostly padding, and fp32
// tiles whose rows are looked up one by one.  The line is drawn over r * (keys + 10), with r the heads per KV head and
// the keys as capacities; measured, us unit / simple kernel, units x keys:
//   fp32, 64 columns    r 1: 64 x 16 5.8 / 5.4, 64 x 24 5.7 / 6.5, 512 x 32 7.4 / 5.9, 1024 x 100 13.1 / 14.2,
//                            4096 x 100 34 / 31, 4096 x 128 41 / 42;   r 2: 4096 x 24 21.0 / 20.1, 4096 x 48 22 / 26
//   fp32, 128 columns   r 1: 64 x 32 7.8 / 7.0, 512 x 64 11 / 12, 1024 x 100 21 / 19, 4096 x 128 85 / 80, 4096 x 300 177 / 187;
//                       r 2: 4096 x 24 41 / 34, 4096 x 48 43 / 49;     r 4: 4096 x 1 43 / 36, 4096 x 16 42 / 49
//   bf16, r 1           64 columns: 1024 x 4 5.9 / 6.8, 4096 x 16 10.2 / 8.1, 4096 x 48 11.1 / 12.2;
//                       128: 4096 x 48 18.2 / 17.1, 4096 x 100 29 / 32
//   pages of 16 rows    bf16, 128 columns: r 1: 1024 x 64 13 / 12, 1024 x 256 25 / 28, 4096 x 1024 429 / 319;
//                       r 2: 4096 x 64 29 / 37;                        bf16, 64 columns: as without pages
//                       fp32, 64: r 1: 1024 x 256 29 / 26, 4096 x 1024 474 / 307;    r 4: 256 x 32 7.9 / 6.7, 4096 x 32 31 / 37
//                       fp32, 128: r 1: 1024 x 1024 385 / 199;  r 2: 4096 x 256 389 / 250;  r 4: 4096 x 64 115 / 119
// e4m3 bytes cost the simple kernel's vector ALU too much at any size.
bool unit_pays(const Problem& pb, int pairs) {
  if (pb.dtype == RLDA_BF16_KV8 || n_sequences(pb) == 0) return true;
  const int64_t r = pb.Hq / pb.Hkv, keys = shared_cap(pb) + pb.Ls_cap, units = n_sequences(pb) * pb.Hkv;
  const bool f32 = pb.dtype == RLDA_F32, wide = pb.d == 128;
  const bool queue = units > pairs, many = units > 4 * (int64_t)pairs;
  constexpr int64_t never = INT64_MAX;
  int64_t line = 0;
  if (row_lookup(pb) && f32 && wide) {
    line = !queue ? 100 : (r <= 2 ? never : 200);
  } else if (row_lookup(pb) && f32) {
    line = queue && r == 1 ? (many ? never : 400) : 170;
  } else if (row_lookup(pb) && wide) {
    line = r == 1 ? (many ? never : 100) : 60;
  } else if (f32) {
    line = !queue ? (wide ? 45 : 30) : (r > 1 ? 70 : (wide && units > 2 * (int64_t)pairs ? 150 : (many ? 115 : 60)));
  } else if (many && r == 1) {
    line = wide ? 70 : 50;
  }
  return r * (keys + 10) > line;
}

// Where one launch beats the shared-prefix path's two.  The lengths live on the device, so the line is drawn on the
// capacities; shorter sequences favour the single launch further.  Full buffers, us (256 pairs):
//   * here about 4 + 0.87 per 1000 tiles walked, shared ones once per sequence, or 2.6 per 1000 tiles that come from memory (e4m3
//     1.4), if that is more; places that workgroups leave empty cost as if they walked too;
//   * over there about 12 + 2.5 per 1000 tiles that come from memory (e4m3 1.4), and 1 to 2 less where a group has 16 rows or fewer.
// So the single launch wins unless long prefixes are shared by many.  P x G x Hkv, prefix + suffix keys, here / over there, bf16 with 4
// rows per KV head:
//   1 x 1 x 4   3500 + 500   8.2 / 14.8      2 x 16 x 1   500 + 3500  15.7 / 20.7     8 x 8 x 1  1200 + 1200 13.7 / 18.3
//   8 x 8 x 1   3500 + 500  14.0 / 15.9      32 x 4 x 1  3500 + 500   21.1 / 26.0     3 x 8 x 4  3500 + 500  19.4 / 18.9
//   8 x 16 x 1  3500 + 500  20.1 / 18.2      8 x 16 x 1  1200 + 1200  19.2 / 25.0     16 x 16 x 1 3500 + 500 32.0 / 26.1
//   32 x 4 x 1   500 + 3500 45.4 / 47.2      32 x 8 x 1  2048 + 256   20.2 / 22.8     32 x 16 x 1 600 + 600  34.5 / 39.0
// with 1 row 8 x 16 x 1 2048 + 256 14.5 / 13.3, with 8 32 x 8 x 1 2048 + 256 20.5 / 25.5; e4m3 32 x 8 x 1 64 + 2000 23.7 / 32.3, 64 x 8 x 1
// 49.1 / 51.6, 16 x 16 x 1 2048 + 256 18.7 / 16.4, 3500 + 500 29.1 / 19.7.  Beyond 20 000 tiles (e4m3 32 768) units differ in length too
// much: half full, 64 x 8 x 1 64 + 2000 59 / 51.  Groups of 16 rows or fewer, which share little and are read at the memory's rate either
// way, stay at 16 384.
// And a wavefront's own chain of tiles has to be short, which the other path cuts as it needs: up to 8 tiles in bf16 where units are
// shared or a group has 16 rows or fewer, 10 else; 12 in e4m3, 14 where a group has more than 64 rows, which cost the other path row
// parts; 7 where workgroups queue.  Beyond, lengths that differ and a queue's last round decide: 13 x 5 x 4 348 + 2030 (18.8 tiles) 78.8 /
// 54.9, half full 38.4 / 35.3; 9 x 16 x 2 991 + 1284 55.6 / 42.4; 66 x 5 x 1 44 + 1936 half full 45.8 / 36.4; 19 x 4 x 2 2241 + 2017 39.0 /
// 30.8; e4m3 33 x 5 x 8 386 + 330 44.4 / 35.5.  Of 1009 drawn points that the two lines above take, full and with lengths spread up to
// that: 688 within these too are 1.25 and 1.29 times as fast here in the geometric mean, one less than 0.97 times by the sum of both (128
// units of 1870 + 377, in two parts each, 18.3 / 16.7 full and 13.7 / 16.2 so); the 321 beyond 1.02 and 1.03, 92 of them slower.
// Trees of several levels cost the other path more: 146 drawn ones 1.42 and 1.50, none below 0.99.
// Units of hardly any key, which wait for nothing but their turn: 16384 x (16 + 16) 58 / 70, 65536 x (1 + 1)
// 163 / 149.  Stores of up to 2048 suffix rows and 3600 in all, prefix rows counted three times, are always taken up to 16 384 tiles: the
// other path is up to twice as slow there with many short units.  Units of more than 8960 keys stay over there: one launch is quicker
// for a few of them only (1 of 12 000 keys 12.7 / 14.5, 8 of 9500 13.4 / 14.0, 32 of 10 240 19.9 / 19.9, 64 of 9500 27.5 / 23.5, 64 of
// 18 000 42.5 / 27.7).  So do trees of several levels over stores of more than 2048 suffix rows, although 84 drawn ones would be 1.24 times
// as fast in one launch: a tree call has no algo field, and this is how tests take it to the shared-prefix kernels.
bool unit_preferred(const Problem& pb, int pairs) {
  const int64_t units = n_sequences(pb) * pb.Hkv, keys = shared_cap(pb) + pb.Ls_cap;
  const bool f8 = pb.dtype == RLDA_BF16_KV8, few = max_group(pb) * (pb.Hq / pb.Hkv) <= 16;
  if (pb.Ls_cap <= 2048 && 3 * shared_cap(pb) + pb.Ls_cap <= 3600 && units <= (int64_t)64 * pairs && units * keys <= (int64_t)2048 * pairs)
    return unit_supported(pb, pairs);
  if (units == 0) return false;                        // nothing runs; and what follows divides by units
  if (keys > 8960 || (pb.n_levels > 1 && pb.Ls_cap > 2048) || units > (int64_t)64 * pairs) return false;
  if (units * keys > (f8 ? 4096 : few ? 2048 : 2560) * (int64_t)pairs || !unit_supported(pb, pairs)) return false;
  int64_t read = units * pb.Ls_cap + (int64_t)pb.P * pb.Hkv * pb.Lp_cap;                  // keys that come from memory
  for (int l = 0; l < pb.n_levels; ++l) read += (int64_t)pb.levels[l].n_seg * pb.Hkv * pb.levels[l].cap;
  // places that the workgroups leave empty cost as if they walked too
  const Split sp = split_rule(pb, pairs);
  const int64_t blocks = units * sp.splits, places = units > pairs ? 2 * (int64_t)pairs : pairs;
  const int64_t walked = blocks < places ? units * keys * places / blocks : units * keys;
  if (4 * walked > (int64_t)(few ? 4 * 560 : 4 * 864) * pairs + (f8 ? 6 : 11) * read) return false;
  if (pb.n_levels > 1) return true;
  // the tiles that a wavefront walks one after the other
  const UnitGrid g = unit_grid(pb, pairs, false, sp);
  const int64_t rows = max_group(pb) * (pb.Hq / pb.Hkv);
  const int most = g.blocks * g.nw > (int64_t)8 * pairs ? 7 : f8 ? (rows > 64 ? 14 : 12) : few || g.splits > 1 ? 8 : 10;
  return full_tiles(pb) <= most * g.nw * g.splits;
}

size_t unit_workspace_bytes(const Problem& pb) {
  const int splits = split_rule(pb, N_CU).splits;
  return splits > 1 ? split_bytes(pb, splits) : 0;
}

hipError_t launch_unit(const Problem& pb, bool exact, int pairs, hipStream_t stream) {
  UnitParams P{};
  P.q = static_cast<const char*>(pb.q); P.out = pb.out; P.lse = pb.lse;
  int n = 0;
  if (pb.n_levels > 0) {
    for (; n < pb.n_levels; ++n) {
      const Problem::Level& lv = pb.levels[n];
      P.seg[n] = Segment{static_cast<const char*>(lv.k), static_cast<const char*>(lv.v), lv.lens, lv.group, lv.cap,
                         make_fastdiv(lv.group)};
    }
  } else {
    P.seg[n++] = Segment{static_cast<const char*>(pb.k_prefix), static_cast<const char*>(pb.v_prefix), pb.prefix_lens, pb.G, pb.Lp_cap,
                         make_fastdiv(pb.G)};
  }
  P.seg[n++] = Segment{static_cast<const char*>(pb.k_suffix), static_cast<const char*>(pb.v_suffix), pb.suffix_lens, 1, pb.Ls_cap,
                       make_fastdiv(1)};
  P.n_seg = n;
  P.B = (int)n_sequences(pb); P.G = max_group(pb); P.Hq = pb.Hq; P.Hkv = pb.Hkv;
  P.r = pb.Hq / pb.Hkv; P.RB = ceil_div(P.r, 16);
  P.div_per = make_fastdiv(P.G * P.RB); P.div_RB = make_fastdiv(P.RB); P.div_Hkv = make_fastdiv(P.Hkv);
  P.scale = pb.scale;
  const double c = pb.scale == 0.f ? 1.0 : fabs((double)pb.scale) * 1.4426950408889634;
  P.c = (float)c; P.c_lo = P.c <= FLT_MAX ? (float)(c - (double)P.c) : 0.f;
  P.qmask = pb.scale == 0.f ? 0u : 0xffffffffu;
  P.qsign = pb.dtype == RLDA_F32 ? 0x80000000u : 0x80008000u;
  P.table = pb.block_table; P.page_shift = pb.page_shift; P.max_pages = pb.max_pages; P.n_pages = pb.n_pages;
  P.active = pb.seq_active; P.kscale = pb.k_scale; P.vscale = pb.v_scale;
  if (P.B == 0) return hipSuccess;
  const UnitGrid grid = unit_grid(pb, pairs, exact);
  P.groups8 = grid.groups8;
  P.splits = grid.splits; P.min_tiles = grid.min_tiles;
  if (grid.splits > 1) {
    const size_t rows = (size_t)P.B * P.Hq;
    const int first = grid.groups8 > 0 ? P.B / P.G * P.Hkv : P.B * P.Hkv * P.RB;
    P.n_first = first; P.div_first = make_fastdiv(first);
    P.call = next_call();
    P.arrived = static_cast<uint64_t*>(pb.workspace);
    P.part_ml = P.arrived + split_counters(pb);
    P.part_o = P.part_ml + rows * grid.splits;
  }
  const int64_t blocks = grid.blocks;
  const int nw = grid.nw;
  if (pb.dtype == RLDA_F32)
    return pb.d == 64 ? launch_form<KV_F32, 64, true>(P, nw, blocks, stream) : launch_form<KV_F32, 128, true>(P, nw, blocks, stream);
  if (pb.dtype == RLDA_BF16_KV8) {
    if (pb.d == 64) return launch_form<KV_F8, 64, true>(P, nw, blocks, stream);
    return exact ? launch_form<KV_F8, 128, true>(P, nw, blocks, stream) : launch_form<KV_F8, 128, false>(P, nw, blocks, stream);
  }
  if (pb.d == 64) return launch_form<KV_BF16, 64, true>(P, nw, blocks, stream);
  return exact ? launch_form<KV_BF16, 128, true>(P, nw, blocks, stream) : launch_form<KV_BF16, 128, false>(P, nw, blocks, stream);
}

}  // namespace rlda
