// vit_decoder_row.h -- FP32 decoder of four blocks a wave, for many blocks, on
// gfx950: device templates, instantiated per constraint length (3 <= k <= 6) in
// vit_kernels_row_k*.hip, rates 1/2 and 1/3, for codes whose generators tap
// both ends.
//
// The arithmetic is that of vit_decoder.h, operation by operation and slot by
// slot (rotating slots, sign-folded metrics, the same fma, compare and med3), so
// that every metric and decision is the same, bit for bit.  What differs:
//
//  * A row of 16 lanes decodes a block: slot bits 0..3 are its lanes (xor 1, 2,
//    7, 8: DPP), bits 4.. the register.  No permlane swaps (3.6 ns each, two of
//    K=7's six phases), and at k <= 6 no idle lanes.
//  * A stage selects between the tags of the two ancestors (a DPP select by the
//    compare's mask) instead of shifting a decision bit into a word: after a
//    period of P = k-1 stages a slot's tag is its ancestor's index at the
//    period's start, as in vit_decoder_int.h, and the traceback (devm::trace_tile,
//    one lane per block) reads LDS once per period.
//  * Blocks of different lengths share a wave: all end at the last stage of the
//    last body, and a block is set to its start metrics at its first stage.
//  * Branch metrics as there: a table per row of the 2^beta sums of T stages,
//    one ds_bpermute per slot and stage.
//
// What bounds it: issue and the crossbar; a stage of K=5 takes a wave alone
// 42 ns, and 17 with four on a SIMD, for four blocks (one block a wave took 11.5
// each).  Measured, us, one / four blocks a wave, 2^24 FP32 bits, L = 512:
// K=3 r1/2 199 / 82, K=4 r1/2 200 / 84, K=5 r1/2 205 / 78, K=5 r1/3 205 / 95,
// K=6 r1/2 210 / 121, K=6 r1/3 226 / 127.
#pragma once

#include "vit_decoder_mx.h"
#include "vit_internal.h"

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace vit {
namespace devr {

using devm::gin_t;
using devm::gout_t;
using devm::Blk;

constexpr int largest_divisor(int n, int cap) {
  int best = 1;
  for (int d = 1; d <= cap; ++d)
    if (n % d == 0) best = d;
  return best;
}

template <int K, int BETA>
struct ShapeR {
  static constexpr int P = K - 1, S = 1 << P, R = S > 16 ? S / 16 : 1;
  static constexpr int NB = 4;                       // blocks per wave
  static constexpr int NG = 32 / P, BODY = P * NG;   // as the other decoders' bodies
  static constexpr int NCODE = 1 << BETA;
  static constexpr int T = largest_divisor(BODY, 16 / NCODE);  // stages of a row's metric table
  static constexpr int NT = BODY / T;
  static constexpr int AHEAD = largest_divisor(NT, 12 / BETA);  // tables' LLRs on the way
  static constexpr int NR = 0;                       // bodies with survivors in registers
  static constexpr int REGION = S * NB;              // dwords of a body's survivor words in LDS
};

// One stage of one register whose partner is in another lane: partner and own
// candidate, compare (odd predecessor wins), the better metric, and the
// winner's tag (k: lanes whose own predecessor is the even one).  Every DPP
// read comes two instructions or more after the write of its register.
#define VITR_LANE(DPPSTR, SN)                                       \
  asm volatile("v_fma_f32 %[B], " SN "%[s], %[o], -%[x]\n\t"        \
               "v_fmac_f32_dpp %[x], %[o], " SN "%[s] " DPPSTR "\n\t" \
               "v_cmp_gt_f32 vcc, %[x], %[B]\n\t"                   \
               "v_med3_f32 %[o], %[x], %[B], %[c]\n\t"              \
               "s_xor_b64 vcc, vcc, %[k]\n\t"                       \
               "v_cndmask_b32_dpp %[t], %[t], %[t], vcc " DPPSTR    \
               : [o] "+v"(o), [x] "+v"(x), [t] "+v"(t), [B] "=&v"(B) \
               : [s] "v"(s), [c] "v"(c), [k] "s"(k)                 \
               : "vcc", "scc")
// Registers a (own predecessor even) and b (odd) of one lane.
#define VITR_PAIR(SA, SB)                                               \
  asm volatile("v_fma_f32 %[Ba], " SA "%[s], %[oa], -%[xa]\n\t"         \
               "v_fma_f32 %[xa], " SA "%[s], %[ob], %[xa]\n\t"          \
               "v_fma_f32 %[Bb], " SB "%[s], %[ob], -%[xb]\n\t"         \
               "v_fma_f32 %[xb], " SB "%[s], %[oa], %[xb]\n\t"          \
               "v_cmp_gt_f32 %[pa], %[xa], %[Ba]\n\t"                   \
               "v_cmp_gt_f32 %[pb], %[xb], %[Bb]\n\t"                   \
               "v_med3_f32 %[oa], %[xa], %[Ba], %[ca]\n\t"              \
               "v_med3_f32 %[ob], %[xb], %[Bb], %[cb]\n\t"              \
               "v_cndmask_b32 %[Ba], %[ta], %[tb], %[pa]\n\t"           \
               "v_cndmask_b32 %[tb], %[ta], %[tb], %[pb]"               \
               : [oa] "+v"(oa), [ob] "+v"(ob), [xa] "+v"(xa), [xb] "+v"(xb), [tb] "+v"(tb), \
                 [Ba] "=&v"(Ba), [Bb] "=&v"(Bb), [pa] "=&s"(pa), [pb] "=&s"(pb) \
               : [s] "v"(s), [ta] "v"(ta), [ca] "v"(INFINITY), [cb] "v"(-INFINITY))

template <int Q, bool NEG>
__device__ __forceinline__ void acs_lane(float &o, float x, uint32_t &t, float s, float c, uint64_t k) {
  float B;
#define VITR_SIGN(DPPSTR) if constexpr (NEG) VITR_LANE(DPPSTR, "-"); else VITR_LANE(DPPSTR, "")
  if constexpr (Q == 0) { VITR_SIGN("quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf"); }
  else if constexpr (Q == 1) { VITR_SIGN("quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf"); }
  else if constexpr (Q == 2) { VITR_SIGN("row_half_mirror row_mask:0xf bank_mask:0xf"); }
  else { VITR_SIGN("row_ror:8 row_mask:0xf bank_mask:0xf"); }
#undef VITR_SIGN
}
template <bool NA, bool NB>
__device__ __forceinline__ void acs_pair(float &oa, float &ob, float xa, float xb, uint32_t &ta, uint32_t &tb, float s) {
  float Ba, Bb;
  uint64_t pa, pb;
  if constexpr (NA && NB) VITR_PAIR("-", "-");
  else if constexpr (NA) VITR_PAIR("-", "");
  else if constexpr (NB) VITR_PAIR("", "-");
  else VITR_PAIR("", "");
  ta = __builtin_bit_cast(uint32_t, Ba);
}
#undef VITR_LANE
#undef VITR_PAIR

// Lane within a row -> slot bits 0..3.
__host__ __device__ constexpr int row_slot(int l) { return (l & 15) ^ (((l >> 2) & 1) ? 3 : 0); }
// Lanes whose slot bit q is 0.
constexpr uint64_t even_lanes(int q) {
  uint64_t m = 0;
  for (int l = 0; l < 64; ++l)
    if (((row_slot(l) >> q) & 1) == 0) m |= (uint64_t)1 << l;
  return m;
}

template <int K, int BETA>
struct DecoderR {
  using Sh = ShapeR<K, BETA>;
  static constexpr int P = Sh::P, S = Sh::S, R = Sh::R, NB = Sh::NB, T = Sh::T, NT = Sh::NT, BODY = Sh::BODY, NCODE = Sh::NCODE;
  static constexpr int QL = P < 4 ? P : 4;  // lane phases

  // per-lane constants
  int addr[P][R];     // byte address within a stage's table of the partner branch's metric
  float sgn[P];       // sign convention product for register 0
  float cmed[QL];     // +inf (keep the max) / -inf
  float bsign[BETA];  // signs of this lane's output pattern in the table
  int tl;             // stage of this lane's table entry
  int lane, slot0;

  // per-wave state
  float o[R], xn[R];
  uint32_t t[R], dec[R];
  int table;
  uint32_t raw[Sh::AHEAD][BETA];
  gin_t llr;          // of the row's block: the window's first LLR
  int off0, end;      // byte offset from there of this lane's stage of the timeline's first table; of the last stage
  int start;          // the row's block: the timeline stage at which it starts, 2 t + (in state 0)
  uint32_t *lds;
  int body, keep, decoded;

  __device__ __forceinline__ static uint32_t rotl_p(uint32_t x, int r) {
    return ((x << r) | (x >> ((P - r) % P))) & (uint32_t)(S - 1);
  }
  // sign factor that register r adds to the lane sign of phase q
  static constexpr bool reg_neg(int q, int r) { return ((((r << 4) >> q) ^ ((r << 4) >> ((q + P - 1) % P))) & 1) != 0; }

  __device__ __forceinline__ void setup(const uint32_t *gen) {
    lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    slot0 = row_slot(lane) & (S - 1);
    tl = (lane & 15) >> BETA;
    const int pat = lane & (NCODE - 1);
#pragma unroll
    for (int b = 0; b < BETA; ++b) bsign[b] = ((pat >> b) & 1) ? -1.0f : 1.0f;
#pragma unroll
    for (int q = 0; q < P; ++q) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const uint32_t st = (uint32_t)((r << 4) | slot0);
        int c = 0;
#pragma unroll
        for (int b = 0; b < BETA; ++b)
          c |= (__builtin_popcount(rotl_p(gen[b] & (uint32_t)(S - 1), q) & st) & 1) << b;
        addr[q][r] = ((lane & 48) | (c ^ (NCODE - 1))) << 2;
      }
      const int bq = (slot0 >> q) & 1, bqm = (slot0 >> ((q + P - 1) % P)) & 1;
      sgn[q] = (bq ^ bqm) ? -1.0f : 1.0f;
      if (q < QL) cmed[q] = bq ? -INFINITY : INFINITY;
    }
  }
  __device__ __forceinline__ uint32_t own_tag(int r) const { return (uint32_t)((S - 1) - slot0 - (r << 4)); }

  // LLRs of the table's stage of this lane, clamped into the window.
  template <int TILE>
  __device__ __forceinline__ void load(int bd) {
    int at = off0 + (bd * BODY + TILE * T) * (4 * BETA);
    at = at < end ? at : end;
    at = at > 0 ? at : 0;
    const __attribute__((address_space(1))) uint32_t *p = (const __attribute__((address_space(1))) uint32_t *)(llr + at);
#pragma unroll
    for (int b = 0; b < BETA; ++b) raw[TILE % Sh::AHEAD][b] = p[b];
  }
  // The table of tile TILE, its registers loaded anew; eq. (2) summed in order,
  // each fma with a factor +-1 rounding like the add.
  template <int TILE>
  __device__ __forceinline__ void take(int bd) {
    const uint32_t(&w)[BETA] = raw[TILE % Sh::AHEAD];
    float d = __builtin_bit_cast(float, w[0]) * bsign[0];
#pragma unroll
    for (int b = 1; b < BETA; ++b) d = __builtin_fmaf(bsign[b], __builtin_bit_cast(float, w[b]), d);
    table = __builtin_bit_cast(int, d);
    load<(TILE + Sh::AHEAD) % NT>(bd + (TILE + Sh::AHEAD) / NT);
  }
  template <int G>
  __device__ __forceinline__ void fetch() {
#pragma unroll
    for (int r = 0; r < R; ++r)
      xn[r] = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(addr[G % P][r] + (G % T) * NCODE * 4, table));
  }
  // (keeps the addresses out of loop-invariant code motion, so that the stage
  // stays in the fetch's offset field)
  __device__ __forceinline__ void refresh() {
#pragma unroll
    for (int q = 0; q < P; ++q)
#pragma unroll
      for (int r = 0; r < R; ++r) asm volatile("" : "+v"(addr[q][r]));
  }

  template <int I, int TILE>
  __device__ __forceinline__ void load_ahead() {
    if constexpr (I < Sh::AHEAD) {
      load<(TILE + I) % NT>((TILE + I) / NT);
      load_ahead<I + 1, TILE>();
    }
  }
  // The first body is entered at offset G.
  template <int G>
  __device__ __forceinline__ void enter() {
    load_ahead<0, G / T>();
    take<G / T>(0);
    fetch<G>();
  }

  // Rows whose block starts at this stage: its start metrics (as vit_decoder.h's).
  template <int G>
  __device__ __forceinline__ void set_starts(int at) {
    constexpr int qm1 = (G + P - 1) % P;
    const bool now = (start >> 1) == at;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int slot = (r << 4) | slot0;
      const float far = ((slot >> qm1) & 1) ? INFINITY : -INFINITY;
      o[r] = now ? ((start & 1) && slot != 0 ? far : 0.0f) : o[r];
      t[r] = now ? own_tag(r) : t[r];
    }
    asm volatile("s_nop 1");  // (the stage reads them by DPP)
  }

  template <int G, bool GUARD>
  __device__ __forceinline__ void step(int from = -1) {
    constexpr int q = G % P;
    if constexpr (GUARD) {
      if (G == from) enter<G>();
      const int at = body * BODY + G;
      if (__builtin_amdgcn_ballot_w64((start >> 1) == at)) set_starts<G>(at);
    }
    float x[R];
#pragma unroll
    for (int r = 0; r < R; ++r) x[r] = xn[r];
    if constexpr (G % T == T - 1) take<(G / T + 1) % NT>(body + (G / T + 1) / NT);
    fetch<(G + 1) % BODY>();
    if constexpr (q < 4) {
      uint64_t k = even_lanes(q);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (reg_neg(q, r)) acs_lane<q, true>(o[r], x[r], t[r], sgn[q], cmed[q < QL ? q : 0], k);
        else acs_lane<q, false>(o[r], x[r], t[r], sgn[q], cmed[q < QL ? q : 0], k);
      }
    } else {
      constexpr int bit = 1 << (q < 4 ? 0 : q - 4);
#pragma unroll
      for (int a = 0; a < R; ++a) {
        if (a & bit) continue;
        const int b = (a | bit) & (R - 1);
        const bool na = reg_neg(q, a), nb = reg_neg(q, b);
        if (na && nb) acs_pair<true, true>(o[a], o[b], x[a], x[b], t[a], t[b], sgn[q]);
        else if (na) acs_pair<true, false>(o[a], o[b], x[a], x[b], t[a], t[b], sgn[q]);
        else if (nb) acs_pair<false, true>(o[a], o[b], x[a], x[b], t[a], t[b], sgn[q]);
        else acs_pair<false, false>(o[a], o[b], x[a], x[b], t[a], t[b], sgn[q]);
      }
    }
    if constexpr (q == P - 1) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        dec[r] = __builtin_amdgcn_alignbit(t[r], dec[r], P);
        t[r] = own_tag(r);
      }
    }
    if constexpr (G == BODY - 1) {
      if (body >= keep) store_words(body - keep, dec);
    }
  }

  // Survivor words: [slot's complement][tau].
  __device__ __forceinline__ void store_words(int region, const uint32_t (&d)[R]) {
    uint32_t *w = lds + region * Sh::REGION + (((S - 1) & 15) - slot0 % 16) * NB + (lane >> 4);
#pragma unroll
    for (int r = 0; r < R; ++r) w[(R - 1 - r) * 16 * NB] = d[r];
  }
  __device__ __forceinline__ int decoded_at(int n) const { return decoded + n * NB; }
  __device__ __forceinline__ int last_at(int bodies) const { return decoded + bodies * NB; }
  __device__ __forceinline__ static int word_at(uint32_t uc, int tau) { return (int)uc * NB + tau; }

  // Lane tau: the complement of block tau's best state (largest metric, lowest
  // state) at the end of a body, where slot j holds state j.
  __device__ __forceinline__ uint32_t best() const {
    float sig[R], m = -INFINITY;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int slot = (r << 4) | slot0;
      sig[r] = ((slot >> (P - 1)) & 1) ? -o[r] : o[r];
      m = __builtin_fmaxf(m, sig[r]);
    }
#pragma unroll
    for (int x = 1; x < 16; x <<= 1)
      m = __builtin_fmaxf(m, __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute((lane ^ x) << 2, __builtin_bit_cast(int, m))));
    int lab = 0x7fffffff;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int cand = sig[r] == m ? (r << 4) | slot0 : 0x7fffffff;
      lab = cand < lab ? cand : lab;
    }
#pragma unroll
    for (int x = 1; x < 16; x <<= 1) {
      const int other = __builtin_amdgcn_ds_bpermute((lane ^ x) << 2, lab);
      lab = other < lab ? other : lab;
    }
    return (uint32_t)(S - 1) & ~(uint32_t)__builtin_amdgcn_ds_bpermute((lane & 3) << 6, lab);
  }
};

#define VITR_G1(NN, M)                                          \
  if constexpr ((NN) < (M)) {                                   \
    if ((NN) >= from) D.template step<(NN), true>(first);        \
  }

// Decode four blocks; lane tau < 4 describes block tau (lanes above: any block
// again), before the recursion and again after it.
template <int K, int BETA, class Describe>
__device__ __forceinline__ void decode_rows(DecoderR<K, BETA> &D, Describe describe) {
  using Sh = ShapeR<K, BETA>;
  constexpr int BODY = Sh::BODY, R = Sh::R;
  Blk bk = describe();
  const int most = devm::wave_max_all(bk.M);
  const int r = (BODY - most % BODY) % BODY;
  const int nbody = (most + r) / BODY;
  const int begin = nbody * BODY - bk.M;
  const int grp_lo = -devm::wave_max_all(-(begin + bk.core)) / BODY;  // the first body with a core bit's decision
  D.keep = grp_lo;
  D.decoded = (nbody - grp_lo) * Sh::REGION;
  {
    const int row = (D.lane >> 4) << 2;
    const uint64_t p = (uint64_t)bk.llr;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute(row, (int)(uint32_t)p);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute(row, (int)(uint32_t)(p >> 32));
    D.llr = (gin_t)(((uint64_t)hi << 32) | lo);
    const int M = __builtin_amdgcn_ds_bpermute(row, bk.M);
    D.off0 = (M - nbody * BODY + D.tl) * (4 * BETA);
    D.end = (M - 1) * (4 * BETA);
    D.start = __builtin_amdgcn_ds_bpermute(row, 2 * begin + (bk.known ? 1 : 0));
  }
#pragma unroll
  for (int x = 0; x < R; ++x) {
    D.o[x] = 0.0f;
    D.t[x] = D.own_tag(x);
    D.dec[x] = 0u;
  }
  const int starts_in = (D.start >> 1) / BODY;
  D.body = 0;
  while (D.body < nbody) {  // one body in which blocks start (as in the first), and those up to the next such
    const int from = D.body == 0 ? r : 0, first = D.body == 0 ? r : -1;
    D.refresh();
    VITM_X32(VITR_G1, BODY)
    for (++D.body; D.body < nbody && !__builtin_amdgcn_ballot_w64(starts_in == D.body); ++D.body) {
      D.refresh();
      VITM_X32(VITM_U1, BODY)
    }
  }
  devm::lds_phase();
  bk = describe();
  const uint32_t uc = D.best();
  devm::trace_tile(D, bk, uc, nbody, grp_lo);
}

// Stream kernel: wave w decodes blocks 4 w .. 4 w + 3, then those 4 x (waves of
// the grid) further on; blocks past the last are the last again, not written.
template <int K, int BETA>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4, 8))) void vit_blocked_row_kernel(DecodeArgs a) {
  extern __shared__ uint32_t vit_ldsr[];
  DecoderR<K, BETA> D;
  D.setup(a.gen);
  D.lds = vit_ldsr;
  const int64_t tiles = (a.nblocks + 3) / 4;
  for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    decode_rows(D, [&] {
      int tau = D.lane & 3;
      asm volatile("" : "+v"(tau));  // (computed anew at each call)
      const int64_t want = tile * 4 + tau;
      const int64_t blk = want < a.nblocks ? want : a.nblocks - 1;
      const int64_t cs = blk * a.L;
      const int64_t ce = (cs + a.L < a.n) ? cs + a.L : a.n;
      const int64_t s = (cs - a.v1 > 0) ? cs - a.v1 : 0;
      const int64_t e = (ce + a.v2 < a.N) ? ce + a.v2 : a.N;
      Blk b;
      b.llr = (const uint8_t *)a.llr + s * (4 * BETA);
      b.out = a.out + (cs >> 3);
      b.before = 0;
      b.M = (int)(e - s);
      b.core = (int)(cs - s);
      b.ncore = (int)(ce - cs);
      b.known = s == 0;
      b.zero = a.terminated && e == a.N;
      b.emit = want < a.nblocks;
      return b;
    });
  }
}

// Batch kernel: the code's items (longest first), four at a time.
template <int K, int BETA>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4, 8))) void vit_batch_row_kernel(BatchArgs a) {
  extern __shared__ uint32_t vit_ldsr[];
  const int nitems = __builtin_amdgcn_readfirstlane(a.header[kMaxCodes + a.code_index]);
  const int tiles = (nitems + 3) / 4;
  if ((int)blockIdx.x >= tiles) return;
  DecoderR<K, BETA> D;
  D.setup(a.gen);
  D.lds = vit_ldsr;
  const WorkItem *items = a.items + a.header[2 * kMaxCodes + a.code_index];
  for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    decode_rows(D, [&] {
      int tau = D.lane & 3;
      asm volatile("" : "+v"(tau));  // (loaded anew at each call)
      const int want = tile * 4 + tau;
      const WorkItem it = items[want < nitems ? want : nitems - 1];
      Blk b;
      b.llr = (const uint8_t *)a.llr + it.llr_off + (int64_t)it.s * (4 * BETA);
      b.out = a.out + it.out_off + (it.cs >> 3);
      b.before = 0;
      b.M = it.e - it.s;
      b.core = it.cs - it.s;
      b.ncore = it.ce - it.cs;
      b.known = (it.flags & 1) != 0;
      b.zero = (it.flags & 2) != 0;
      b.emit = want < nitems;
      return b;
    });
  }
}
#undef VITR_G1

}  // namespace devr

// FP32 kernel instances for (K, beta) of four blocks a wave, taking DecodeArgs or BatchArgs.
template <int K>
void *pick_kernel_row_k(int beta, bool batch) {
  switch (beta) {
    case 2: return batch ? (void *)devr::vit_batch_row_kernel<K, 2> : (void *)devr::vit_blocked_row_kernel<K, 2>;
    case 3: return batch ? (void *)devr::vit_batch_row_kernel<K, 3> : (void *)devr::vit_blocked_row_kernel<K, 3>;
  }
  return nullptr;
}

void *pick_kernel_row_k3(int beta, bool batch);
void *pick_kernel_row_k4(int beta, bool batch);
void *pick_kernel_row_k5(int beta, bool batch);
void *pick_kernel_row_k6(int beta, bool batch);

}  // namespace vit
