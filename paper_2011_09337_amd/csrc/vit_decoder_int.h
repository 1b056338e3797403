// vit_decoder_int.h -- integer decoder for int8 and hard-decision inputs on
// gfx950: device templates, instantiated per constraint length in
// vit_kernels_int_k*.hip.
//
// One wave decodes one block, in the rotating-slot layout of vit_decoder.h
// (slot j holds state rotr^m(j) after m stages; the two predecessors of a
// butterfly differ in slot bit q = m mod (k-1); slot bits 0..5 are lane xors
// 1, 2, 7, 8, 16, 32, higher bits are registers).  Integer metrics allow a
// shorter recursion than the FP32 one:
//
//  * Ancestor tags.  A metric register holds metric * 2^P + tag (P = k-1).  At
//    the start of each period of P stages the tag is the complement of the
//    slot's own index; from then on the survivor's tag travels with its
//    metric, so that after P stages it names the slot the path came from: P
//    decisions at once, with no compare, no decision bit and no select.
//    max() also keeps the tie rule: at phase q the two candidates of a slot
//    come from ancestors that agree in the index bits of the phases after q
//    and differ in bit q, where the even predecessor's complement is the
//    larger.
//  * A stage is P = o + x, Q = o - x and o = max(P, Q of the partner), the
//    exchange fused into the max as a DPP read (permlane swaps for lane xors
//    16 and 32; plain registers above): 3 instructions and 8 issue cycles
//    against 5 and 18 for the fp32 recursion (which the integer inputs ran
//    before), and a period's end adds two (shift the tag into the survivor
//    word, put the slot's own tag back).
//  * The traceback takes one v_readlane per period instead of one per stage.
//
// What bounds it: with few waves the latency of a stage (1000 stages of K=7 in
// one wave: 40.9 us in the fp32 recursion, 24.8 here); with the chip full the
// branch-metric fetch: a CU's crossbar answers a ds_bpermute every 5.7 cycles,
// one per 23 cycles and SIMD, and a stage of K=7 takes 25 (2^24 bits, L = 512,
// v = 35: 246 us before, 198 here; K=9, 2^22 bits, L = 256: 261 and 236).
// Branch metrics by v_dot4 on LLRs from scalar loads instead of the crossbar
// measured 205 and 197 us there, but half as slow again where waves are few
// (the scalar cache's misses then show).
//  * The best final state is one wave-wide max: after the last period's reset
//    the tag is the complement of the state's index, so the largest register
//    is the best metric with the lowest index.
//
// Ranges: |metric| <= stages * 128 beta, and 160 KiB of LDS hold at most
// 20480 stages for k <= 7, 10240 for k = 8 and 5120 for k = 9: with the tag
// every register stays below 2^30.  States other than 0 at a known start begin
// 2^14 below state 0, more than the spread (k-1) * 2 * 128 * beta <= 2^13 of
// the reachable ones.
#pragma once

#include "vit_internal.h"

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace vit {
namespace devi {

constexpr int largest_even_split_divisor(int n, int cap) {
  int best = 1;
  for (int d = 1; d <= cap; ++d)
    if (n % d == 0 && (n / d) % 2 == 0) best = d;
  return best;
}

template <int K, int BETA>
struct ShapeI {
  static constexpr int P = K - 1;
  static constexpr int S = 1 << P;
  static constexpr int REGS = S > 64 ? S / 64 : 1;
  static constexpr int NCODE = 1 << BETA;
  static constexpr int NG = 32 / P;          // periods per survivor word
  static constexpr int BODY = P * NG;
  static constexpr int T = largest_even_split_divisor(BODY, 64 / NCODE);  // stages per branch-metric tile
};

// The partner's value across slot bit Q (Q < 6).
template <int Q>
__device__ __forceinline__ int exchange(int v) {
  if constexpr (Q == 0) return __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, true);        // quad_perm [1,0,3,2]
  else if constexpr (Q == 1) return __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, true);   // quad_perm [2,3,0,1]
  else if constexpr (Q == 2) return __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, true);  // row_half_mirror
  else if constexpr (Q == 3) return __builtin_amdgcn_update_dpp(0, v, 0x128, 0xF, 0xF, true);  // row_ror:8
  else if constexpr (Q == 4) {
    asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %0" : "+v"(v));
    return v;
  } else {
    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %0" : "+v"(v));
    return v;
  }
}

__device__ __forceinline__ int max_i(int a, int b) { return __builtin_elementwise_max(a, b); }

__device__ __forceinline__ int wave_max(int v) {
  v = max_i(v, exchange<0>(v));
  v = max_i(v, exchange<1>(v));
  v = max_i(v, exchange<2>(v));
  v = max_i(v, exchange<3>(v));
  v = max_i(v, exchange<4>(v));
  return max_i(v, exchange<5>(v));
}

// Hard decisions: byte 0 (coded bit 0) -> +1, any other value -> -1.
__device__ __forceinline__ uint32_t hard_to_pm1(uint32_t w) {
  uint32_t t = w | ((w >> 4) & 0x0F0F0F0Fu);
  t |= (t >> 2) & 0x33333333u;
  t |= (t >> 1) & 0x55555555u;
  return 0x01010101u + (t & 0x01010101u) * 0xFEu;
}

// STD: every generator taps the newest input, so that the two branches that
// leave a state carry opposite metrics.  IN: VIT_LLR_I8 or VIT_LLR_HARD.
template <int K, int BETA, bool STD, int IN>
struct DecoderI {
  using Sh = ShapeI<K, BETA>;
  static constexpr int P = Sh::P, S = Sh::S, REGS = Sh::REGS, NCODE = Sh::NCODE, BODY = Sh::BODY, T = Sh::T;
  static constexpr int kUnreached = -(1 << 14);  // start metric of states other than 0 at a known start
  // Stages between a branch metric's fetch and its use (one and two measure
  // alike with the chip full, where the crossbar's rate counts).
  static constexpr int AHEAD = 2;
  static_assert(BODY % AHEAD == 0 && AHEAD <= T, "fetch distance");

  // per-lane constants
  int addr[P][REGS];   // byte offset, within a stage's table entries, of the branch that stays in this slot
  int qflip;           // xor of that offset for the branch that leaves for the partner's slot
  int tag[REGS];       // complement of the slot's index
  uint32_t ssign;      // byte b: +1 or -1, the sign of LLR b in this lane's table pattern
  int lane, slot0, tl;

  // per-block state
  int o[REGS];
  uint32_t dec[REGS];
  int xq[AHEAD][REGS], yq[AHEAD][REGS];  // branch metrics of the next AHEAD stages
  int table;
  uint32_t nxt[2];     // LLR bytes of this lane's stage in the next two tiles
  const uint8_t *llr;
  int tile_stage0, s_lo, s_hi;
  uint32_t *lds;
  int body;

  __device__ __forceinline__ static uint32_t rotl_p(uint32_t x, int r) {
    return ((x << r) | (x >> ((P - r) % P))) & (uint32_t)(S - 1);
  }

  // Output bit b of the branch that stays in slot st at phase q is the parity
  // of st with the generator's low P bits rotated left by q, the newest-input
  // tap added at bit q (the predecessor's low bit is the input of the branch).
  __device__ __forceinline__ int own_addr(const uint32_t *gen, int q, int reg) const {
    const uint32_t st = (uint32_t)(((reg << 6) | slot0) & (S - 1));
    int c = 0;
#pragma unroll
    for (int b = 0; b < BETA; ++b) {
      const uint32_t m = rotl_p(gen[b] & (uint32_t)(S - 1), q) ^ (((gen[b] >> P) & 1u) << q);
      c |= (__builtin_popcount(m & st) & 1) << b;
    }
    return c << 2;
  }

  __device__ __forceinline__ void setup(const uint32_t *gen) {
    lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    slot0 = lane ^ (((lane >> 2) & 1) ? 3 : 0);  // inverse of the lane xor map
    tl = lane / NCODE;
    const int pat = lane % NCODE;
    ssign = 0;
#pragma unroll
    for (int b = 0; b < BETA; ++b) ssign |= (((pat >> b) & 1) ? 0xFFu : 0x01u) << (8 * b);
    qflip = 0;
#pragma unroll
    for (int b = 0; b < BETA; ++b) qflip |= (int)((gen[b] >> P) & 1u) << (b + 2);
#pragma unroll
    for (int q = 0; q < P; ++q)
#pragma unroll
      for (int reg = 0; reg < REGS; ++reg) addr[q][reg] = own_addr(gen, q, reg);
#pragma unroll
    for (int reg = 0; reg < REGS; ++reg) tag[reg] = (S - 1) ^ (((reg << 6) | slot0) & (S - 1));
  }

  // LLR bytes of this lane's stage in tile tau, the stage clamped into the
  // block (every lane reads inside it).
  __device__ __forceinline__ uint32_t tile_word(int tau) const {
    int stc = tile_stage0 + tau * T;
    stc = __builtin_elementwise_max(__builtin_elementwise_min(stc, s_hi), s_lo);
    const uint8_t *p = llr + (uint32_t)stc * (uint32_t)BETA;
    uint32_t w = 0;
    if constexpr (BETA == 4) {
      __builtin_memcpy(&w, p, 4);
    } else {
      uint16_t h;
      __builtin_memcpy(&h, p, 2);
      w = h;
      if constexpr (BETA == 3) w |= (uint32_t)p[2] << 16;
    }
    return w;
  }

  // eq. (2) for this lane's pattern, scaled past the tag.
  __device__ __forceinline__ void build_table(uint32_t w) {
    if constexpr (IN == VIT_LLR_HARD) w = hard_to_pm1(w);
    table = __builtin_amdgcn_sdot4((int)w, (int)ssign, 0, false) << P;
  }

  // Keep the addresses out of loop-invariant code motion, so that each fetch
  // keeps its tile offset in the instruction's offset field.
  __device__ __forceinline__ void refresh_addresses() {
#pragma unroll
    for (int q = 0; q < P; ++q)
#pragma unroll
      for (int reg = 0; reg < REGS; ++reg) asm volatile("" : "+v"(addr[q][reg]));
  }

  template <int G>
  __device__ __forceinline__ void fetch_step() {
    constexpr int q = G % P, off = (G % T) * NCODE * 4, at = G % AHEAD;
#pragma unroll
    for (int reg = 0; reg < REGS; ++reg) {
      xq[at][reg] = __builtin_amdgcn_ds_bpermute(addr[q][reg] + off, table);
      if constexpr (!STD) yq[at][reg] = __builtin_amdgcn_ds_bpermute((addr[q][reg] ^ qflip) + off, table);
    }
  }

  // Pipeline prologue for the entry step r: the branch metrics of the first
  // AHEAD stages, the table of the last of them, and the LLRs of the two
  // tiles after that one.
  __device__ __forceinline__ void start(const uint32_t *gen, int r) {
    int tau = r / T;
    const uint32_t n0 = tile_word(tau);
    uint32_t n1 = tile_word(tau + 1), n2 = tile_word(tau + 2);
    build_table(n0);
    int x[AHEAD][REGS], y[AHEAD][REGS];
#pragma unroll
    for (int d = 0; d < AHEAD; ++d) {
      const int g = r + d;
      if (d > 0 && g % T == 0) {
        ++tau;
        build_table(n1);
        n1 = n2;
        n2 = tile_word(tau + 2);
      }
      const int off = (g % T) * NCODE * 4;
#pragma unroll
      for (int reg = 0; reg < REGS; ++reg) {
        const int a = own_addr(gen, g % P, reg);
        x[d][reg] = __builtin_amdgcn_ds_bpermute(a + off, table);
        y[d][reg] = STD ? 0 : __builtin_amdgcn_ds_bpermute((a ^ qflip) + off, table);
      }
    }
    nxt[0] = (tau & 1) ? n1 : n2;  // tile tau lives in buffer tau % 2
    nxt[1] = (tau & 1) ? n2 : n1;
#pragma unroll
    for (int d = 0; d < AHEAD; ++d)  // stage g lives in place g % AHEAD
#pragma unroll
      for (int reg = 0; reg < REGS; ++reg) {
        xq[d][reg] = (r & 1) ? x[d ^ 1][reg] : x[d][reg];
        yq[d][reg] = (r & 1) ? y[d ^ 1][reg] : y[d][reg];
      }
  }

  // One trellis stage at body offset G: its branch metrics were fetched AHEAD
  // stages ago.  A tile's table is built when its first stage is fetched, and
  // the LLRs of the tile after the next are loaded into the buffer it leaves.
  template <int G>
  __device__ __forceinline__ void step() {
    constexpr int q = G % P, at = G % AHEAD, ahead = G + AHEAD;
    int x[REGS], y[REGS];
#pragma unroll
    for (int reg = 0; reg < REGS; ++reg) {
      x[reg] = xq[at][reg];
      y[reg] = STD ? -x[reg] : yq[at][reg];
    }
    if constexpr (ahead % T == 0) {
      constexpr int buf = (ahead / T) % 2;
      build_table(nxt[buf]);
      nxt[buf] = tile_word(body * (BODY / T) + ahead / T + 2);
    }
    fetch_step<ahead % BODY>();
    int own[REGS], out[REGS];
#pragma unroll
    for (int reg = 0; reg < REGS; ++reg) {
      own[reg] = o[reg] + x[reg];
      out[reg] = o[reg] + y[reg];
    }
#pragma unroll
    for (int reg = 0; reg < REGS; ++reg) {
      if constexpr (q < 6) o[reg] = max_i(own[reg], exchange<(q < 6 ? q : 0)>(out[reg]));
      else o[reg] = max_i(own[reg], out[reg ^ (1 << (q - 6 < 0 ? 0 : q - 6))]);
    }
    if constexpr (q == P - 1) {
#pragma unroll
      for (int reg = 0; reg < REGS; ++reg) {
        dec[reg] = __builtin_amdgcn_alignbit((uint32_t)o[reg], dec[reg], P);  // newest period at the top
        o[reg] = (o[reg] & -S) | tag[reg];
      }
    }
    if constexpr (G == BODY - 1) {
      // at the complement of the slot's index, where the traceback looks
#pragma unroll
      for (int reg = 0; reg < REGS; ++reg)
        lds[(body * REGS + (tag[reg] >> 6)) * 64 + (S < 64 ? (63 ^ slot0) : (tag[reg] & 63))] = dec[reg];
    }
  }
};

template <int REGS>
__device__ __forceinline__ uint32_t select_reg(const uint32_t (&v)[REGS], uint32_t rsel) {
  typedef uint32_t vec_t __attribute__((ext_vector_type(REGS)));
  vec_t t;
#pragma unroll
  for (int i = 0; i < REGS; ++i) t[i] = v[i];
  return t[rsel & (REGS - 1)];
}

// The first body of a block runs its steps from the entry offset r on.
#define VITI_G1(NN, M) \
  if constexpr ((NN) < (M)) { \
    if ((NN) >= r) D.template step<(NN)>(); \
  }
#define VITI_U1(NN, M) \
  if constexpr ((NN) < (M)) D.template step<(NN)>();
#define VITI_X8(X, B, M)                                                                 \
  X(B + 0, M) X(B + 1, M) X(B + 2, M) X(B + 3, M) X(B + 4, M) X(B + 5, M) X(B + 6, M)   \
  X(B + 7, M)
#define VITI_X32(X, M) VITI_X8(X, 0, M) VITI_X8(X, 8, M) VITI_X8(X, 16, M) VITI_X8(X, 24, M)

// Decode one block (Sec. III), as decode_block of vit_decoder.h: stages [s, e)
// of a frame, core bits [cs, ce).  The caller guarantees (e - s) * beta <
// 2^31 and cs a multiple of 8.
template <int K, int BETA, bool STD, int IN>
__device__ __forceinline__ void decode_block_int(DecoderI<K, BETA, STD, IN> &D, const uint8_t *llr, uint8_t *out,
                                                 int64_t s, int64_t e, int64_t cs, int64_t ce, bool start_known,
                                                 bool end_zero, const uint32_t *gen) {
  using Sh = ShapeI<K, BETA>;
  constexpr int P = Sh::P, S = Sh::S, REGS = Sh::REGS, NG = Sh::NG, BODY = Sh::BODY;
  const int M = (int)(e - s);
  const int r = (BODY - M % BODY) % BODY;  // entry offset: the block's last stage is the body's last
  const int nbody = (M + r) / BODY;
  const int stage_base = (int)s - r;
  D.llr = llr;
  D.tile_stage0 = stage_base + D.tl;
  D.s_lo = (int)s;
  D.s_hi = (int)e - 1;
#pragma unroll
  for (int reg = 0; reg < REGS; ++reg) {
    const bool far = start_known && D.tag[reg] != S - 1;  // slot 0 is state 0 at any phase
    D.o[reg] = (far ? D.kUnreached * S : 0) + D.tag[reg];
    D.dec[reg] = 0u;
  }
  D.start(gen, r);
  D.body = 0;
  D.refresh_addresses();
  VITI_X32(VITI_G1, BODY)
  for (D.body = 1; D.body < nbody; ++D.body) {
    D.refresh_addresses();
    VITI_X32(VITI_U1, BODY)
  }

  // ---- traceback start, as the complement of the slot's index: state 0 at a
  // terminated end, else the best state
  uint32_t uc = S - 1;
  if (!end_zero) {
    int m = D.o[0];
#pragma unroll
    for (int reg = 1; reg < REGS; ++reg) m = max_i(m, D.o[reg]);
    uc = (uint32_t)__builtin_amdgcn_readfirstlane(wave_max(m)) & (uint32_t)(S - 1);
  }
  const uint32_t lam_start = uc ^ (uint32_t)(S - 1);

  // ---- traceback: one step per period, from the last body down to the one
  // with the first core bit.  The slot index after a period holds the
  // decisions of its P stages, the input bits of P stages earlier (as in
  // vit_decoder.h): the body's decoded word replaces its first survivor word.
  // The next body's survivor words are read while this body's chain runs.
  const int grp_lo = ((int)(cs - s) + r) / BODY;
  __builtin_amdgcn_s_setprio(1);
  uint32_t nv[REGS];
#pragma unroll
  for (int rr = 0; rr < REGS; ++rr) nv[rr] = D.lds[((nbody - 1) * REGS + rr) * 64 + D.lane];
  for (int grp = nbody - 1; grp >= grp_lo; --grp) {
    uint32_t dv[REGS];
    const int below = grp > 0 ? grp - 1 : 0;
#pragma unroll
    for (int rr = 0; rr < REGS; ++rr) {
      dv[rr] = nv[rr];
      nv[rr] = D.lds[(below * REGS + rr) * 64 + D.lane];
    }
    uint32_t acc = 0;
#pragma unroll
    for (int g = NG - 1; g >= 0; --g) {
      uint32_t w;
      if constexpr (REGS > 1) w = __builtin_amdgcn_readlane(select_reg<REGS>(dv, uc >> 6), (int)(uc & 63u));
      else w = __builtin_amdgcn_readlane(dv[0], (int)uc + (S < 64 ? 64 - S : 0));
      uc = (w >> (32 - BODY + g * P)) & (uint32_t)(S - 1);
      acc |= uc << (g * P);
    }
    D.lds[grp * REGS * 64] = ~acc;  // every lane writes the same word
  }
  __builtin_amdgcn_s_setprio(0);

  // ---- output: lane-parallel assembly of the core bits [cs, ce) into bytes:
  // bit t is stream bit (t - stage_base) + k - 1 of the decoded words, with
  // the start slot's k - 1 bits behind the last.
  {
    const int64_t b_lo = cs >> 3, b_hi = (ce - 1) >> 3;
    constexpr uint32_t body_mask = BODY == 32 ? 0xffffffffu : ((1u << (BODY % 32)) - 1u);
    for (int64_t B = b_lo + D.lane; B <= b_hi; B += 64) {
      const int gbit = (int)(8 * B - stage_base) + P;
      const int wa = gbit / BODY, sh = gbit - wa * BODY;
      auto word = [&](int i) -> uint64_t {
        if (i < nbody) return D.lds[i * REGS * 64] & body_mask;
        return i == nbody ? lam_start : 0u;
      };
      const uint64_t cat = word(wa) | (word(wa + 1) << BODY);
      uint32_t byte = (uint32_t)(cat >> sh) & 0xffu;
      const int64_t nvalid = ce - 8 * B;
      if (nvalid < 8) byte &= (1u << nvalid) - 1u;
      out[B] = (uint8_t)byte;
    }
  }
}

// Blocks are dealt to waves as in the FP32 stream kernel: with more blocks
// than waves each XCD gets a contiguous range.
template <int K, int BETA, bool STD, int IN>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(K <= 7 ? 8 : 1, 8))) void vit_blocked_int_kernel(DecodeArgs a, int lds_words_per_wave) {
  extern __shared__ uint32_t vit_ldsi[];
  DecoderI<K, BETA, STD, IN> D;
  D.setup(a.gen);
  const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int wpb = (int)(blockDim.x >> 6);
  D.lds = vit_ldsi + (size_t)wid * lds_words_per_wave;
  const int64_t nwaves = (int64_t)gridDim.x * wpb;
  int64_t first, stride, last;
  if ((gridDim.x & 7) == 0 && a.nblocks >= nwaves) {
    const int xcd = blockIdx.x & 7;
    const int64_t wx = (int64_t)(blockIdx.x >> 3) * wpb + wid;
    const int64_t per = (a.nblocks + 7) / 8;
    first = (int64_t)xcd * per + wx;
    last = (int64_t)(xcd + 1) * per;
    if (last > a.nblocks) last = a.nblocks;
    stride = nwaves / 8;
  } else {
    first = (int64_t)blockIdx.x * wpb + wid;
    last = a.nblocks;
    stride = nwaves;
  }
  for (int64_t blk = first; blk < last; blk += stride) {
    const int64_t cs = blk * a.L;
    const int64_t ce = (cs + a.L < a.n) ? cs + a.L : a.n;
    const int64_t s = (cs - a.v1 > 0) ? cs - a.v1 : 0;
    const int64_t e = (ce + a.v2 < a.N) ? ce + a.v2 : a.N;
    decode_block_int(D, (const uint8_t *)a.llr, a.out, s, e, cs, ce, s == 0, a.terminated && (e == a.N), a.gen);
  }
}

// Batched decode: the code's items (sorted by cost) with a static stride, as
// vit_batch_kernel of vit_decoder.h.
template <int K, int BETA, bool STD, int IN>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(K <= 7 ? 8 : 1, 8))) void vit_batch_int_kernel(BatchArgs a, int lds_words_per_wave) {
  extern __shared__ uint32_t vit_ldsi[];
  const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int wpb = (int)(blockDim.x >> 6);
  const int nitems = __builtin_amdgcn_readfirstlane(a.header[kMaxCodes + a.code_index]);
  if ((int)blockIdx.x * wpb + wid >= nitems) return;  // waves without an item leave before any setup
  DecoderI<K, BETA, STD, IN> D;
  D.setup(a.gen);
  D.lds = vit_ldsi + (size_t)wid * lds_words_per_wave;
  const WorkItem *items = a.items + a.header[2 * kMaxCodes + a.code_index];
  const int nwaves = (int)gridDim.x * wpb;
  for (int idx = (int)blockIdx.x * wpb + wid; idx < nitems; idx += nwaves) {
    const WorkItem it = items[idx];
    decode_block_int(D, (const uint8_t *)a.llr + it.llr_off, a.out + it.out_off, it.s, it.e, it.cs, it.ce,
                     (it.flags & 1) != 0, (it.flags & 2) != 0, a.gen);
  }
}

#undef VITI_G1
#undef VITI_U1
#undef VITI_X8
#undef VITI_X32

}  // namespace devi

// Kernel instances for (K, beta, newest-input taps in every generator, input
// kind VIT_LLR_I8 / VIT_LLR_HARD): a KernelFn, or a BatchKernelFn.
template <int K>
void *pick_kernel_int_k(int beta, bool top, int in, bool batch) {
  auto pick = [&](auto bt, auto tp) -> void * {
    constexpr int B = decltype(bt)::value;
    constexpr bool TOP = decltype(tp)::value;
    if (batch)
      return in == VIT_LLR_HARD ? (void *)devi::vit_batch_int_kernel<K, B, TOP, VIT_LLR_HARD>
                                : (void *)devi::vit_batch_int_kernel<K, B, TOP, VIT_LLR_I8>;
    return in == VIT_LLR_HARD ? (void *)devi::vit_blocked_int_kernel<K, B, TOP, VIT_LLR_HARD>
                              : (void *)devi::vit_blocked_int_kernel<K, B, TOP, VIT_LLR_I8>;
  };
  auto by_top = [&](auto bt) { return top ? pick(bt, std::true_type{}) : pick(bt, std::false_type{}); };
  switch (beta) {
    case 2: return by_top(std::integral_constant<int, 2>{});
    case 3: return by_top(std::integral_constant<int, 3>{});
    case 4: return by_top(std::integral_constant<int, 4>{});
  }
  return nullptr;
}

void *pick_kernel_int_k3(int beta, bool top, int in, bool batch);
void *pick_kernel_int_k4(int beta, bool top, int in, bool batch);
void *pick_kernel_int_k5(int beta, bool top, int in, bool batch);
void *pick_kernel_int_k6(int beta, bool top, int in, bool batch);
void *pick_kernel_int_k7(int beta, bool top, int in, bool batch);
void *pick_kernel_int_k8(int beta, bool top, int in, bool batch);
void *pick_kernel_int_k9(int beta, bool top, int in, bool batch);

}  // namespace vit
