// vit_decoder_mx.h -- integer decoder on the matrix cores, for int8 and
// hard-decision inputs with many blocks, on gfx950: device templates,
// instantiated per constraint length (3 <= k <= 9) in vit_kernels_mx_k*.hip.
//
// The recursion is that of vit_decoder_int.h (rotating slots, metrics that
// carry their ancestor's tag in the low P = k-1 bits, o = max(o + x, partner's
// o - x)).  Here one wave decodes NB blocks at once, and both additions of a
// stage are matrix instructions with the metrics as the accumulator.  Two
// layouts:
//
//   16 registers (k = 6..9, NB = 32, 16, 8, 4: 1024 slots a wave)
//     v_mfma_*_16x16x4 (4 blocks): D[b][row, col] = A_b[row, :] . B_b[:, col] + C
//   4 registers ("quad", k = 3..7, NB = 64, 32, 16, 8, 4: 256 slots a wave)
//     v_mfma_i32_4x4x4 (16 blocks)
//
//  * A is a stage's LLRs (the four products are the code's outputs), B the
//    signs of each slot's branch times 2^P: one instruction adds the branch
//    that stays in the slot, another the branch that leaves for the partner's
//    slot.  What is left for the vector unit is one max per slot and stage, and
//    two instructions per period for the tags: 4 issue cycles per 64 slots
//    instead of 8 and a crossbar fetch.  The 16x16x4 form (32 cycles) runs beside
//    the vector work of the SIMD's other wave; the 4x4x4 form (8 cycles, a
//    quarter of the slots) holds the vector unit up, but a wave needs a quarter of
//    the blocks and of the survivor space.
//  * 16 registers: slot bits 0..3 are the lanes of a row of 16 (col: lane xors 1,
//    2, 7, 8, which DPP reads inside the max); bits 4, 5 are the instruction's
//    blocks b and bits 6, 7 the register within a row quad: partners in
//    registers, no exchange at all.  The other row, quad and b indices number the
//    blocks (tau).  A row that carries slot bits (k = 8, 9) puts their branch
//    signs on its LLRs.
//  * 4 registers: the lane's low P bits are the slot, its other bits and the
//    register number the blocks.  Bits 4, 5 exchange by a permlane swap of the
//    two candidates: the lanes of that bit hold them the other way round (their B
//    signs are swapped), so that one swap brings both of a slot together.
//  * All instruction blocks that belong to the same tau take their A from one of
//    them (CBSZ, ABID), so each lane holds another dword of its row's LLRs: one
//    load a lane brings 64 bytes of each row at k = 7 in the 4-register layout,
//    and 16 in the other.
//  * k <= 7: int8 LLRs straight from memory, 32-bit integer sums.  k = 8, 9
//    need 2^P > 64, more than a byte's sign factor: fp16 operands (a byte and a
//    power of two, both exact), fp32 sums kept as 2^23 + 2^22 + integer, whose
//    bits count like the integer's (the tags and the max work on the bits); the
//    metrics are taken back towards 0 every RENORM stages, so that each sum is
//    the exact integer.
//  * Blocks of different lengths share a wave: all end at the last stage of
//    the last body; a block is set to its start metrics at its first stage (only
//    the bodies in which some block starts look for it: a short last block of a
//    stream made its whole wave half as slow again when all earlier ones did).
//  * Survivor words as in vit_decoder_int.h: those of a block's first 8 (or 16)
//    traced bodies in 128 (or 64) registers of their own, the others in LDS,
//    [slot][tau].  The traceback runs one lane per block, one dependent LDS read
//    per period.
//
// What bounds it.  16 registers: a wave alone on a SIMD takes 95 ns per stage
// (k = 7, 16 blocks: the two matrix instructions one after the other, their
// latency, then 16 max); two waves overlap the one's matrix with the other's
// vector work, 147 ns for both; registers and LDS hold no third.  4 registers:
// alone 44 ns per stage (4 blocks: the chain of instruction latencies), four
// waves 92 for all: 7 ns of matrix and 14 of vector work each.  Measured, one-block
// kernel / 16 / 4 registers, us: K=7 r1/2, 2^24 int8 bits, v = 35: L = 256
// 210 / 84 / 113, L = 512 (LDS holds one 16-register wave a SIMD; without the
// survivor registers two a CU and 212 us) 199 / 121 / 107; K=7 r1/2, 2^22 bits,
// L = 512 59 / 60 / 39; K=9 r1/2, 2^22 bits, L = 256, v = 64 236 / 94 / -;
// K=5 r1/2, 2^24 bits, L = 256 204 / - / 34 (16 registers: 48); K=3 r1/2 the
// same 201 / - / 31.  With a row's LLRs loaded by periods in every lane (up to
// 15 registers, unaligned) instead of by broadcast: K=7 r1/3, L = 512 123 in 16
// registers and 242 in 4 (now 134 and 107); K=9, L = 256 104 (now 94).
#pragma once

#include "vit_decoder_int.h"
#include "vit_internal.h"

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace vit {
namespace devm {

using devi::hard_to_pm1;
using devi::max_i;

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));

// Bodies whose survivors a wave keeps in registers of its own: 128 of them in
// the 16-register layout, 64 in the 4-register one.
constexpr int kept_bodies(bool quad) { return quad ? 16 : 8; }
// Dwords of a body's survivor words in LDS.
constexpr int region_words(bool quad) { return quad ? 256 : 1024; }

template <int K, int BETA, bool QUAD>
struct ShapeM {
  static constexpr int P = K - 1;
  static constexpr int S = 1 << P;
  static constexpr int R = QUAD ? 4 : 16;                           // metric registers
  static constexpr int BB = QUAD ? 0 : P - 4 < 2 ? P - 4 : 2;       // slot bits in b
  static constexpr int IB = QUAD ? 0 : P - 4 - BB;                  // slot bits in the quad's register
  static constexpr int NB = QUAD ? 256 >> P : 64 >> (BB + IB);      // blocks per wave
  static constexpr int NCLS = QUAD ? 4 : NB / 4;                    // blocks per lane
  static constexpr int NG = 32 / P;                 // periods per body
  static constexpr int BODY = P * NG;
  // LLRs: a dword holds SPD stages, one load DPL dwords of every row, one per
  // instruction block, which the instruction takes by broadcast (CBSZ, ABID).
  static constexpr int SPD = BETA == 2 ? 2 : 1;
  static constexpr int CBSZ = QUAD ? P - 2 : BB, DPL = 1 << CBSZ;
  static constexpr int SPL = SPD * DPL;             // stages of a load
  static constexpr int NL = (BODY + SPL - 1) / SPL; // loads of a body
  static constexpr int AHEAD = !QUAD && P > 6 && NL % 4 == 0 ? 4 : NL < 16 ? NL : 16;  // loads between one and its use (registers; divides NL)
  static constexpr bool F16 = !QUAD && P > 6;
  static constexpr int NR = kept_bodies(QUAD);
  static constexpr int REGION = region_words(QUAD);
  // Stages between two renormalisations of the fp32 sums, whole periods: the
  // spread 2^8 P beta + 1, and 2^7 beta a stage, stay below 2^22 / 2^P.
  static constexpr int kRoom = ((1 << 22) >> P) - 1 - 256 * P * BETA;
  static constexpr int RENORM = kRoom / (128 * BETA) >= BODY ? BODY : kRoom / (128 * BETA) >= 2 * P ? 2 * P : P;
  static_assert(!F16 || kRoom >= 128 * BETA * RENORM, "fp32 sums leave their binade");
  // A block that starts in state 0 n < P stages before its sums are taken back:
  // its other states, 2^8 P beta + 1 below at the start, may have come down 2^7
  // beta a stage and the reference up as much, and they come down further until
  // every state is reached, P - n stages on (15873 of 16384 for k = 9, rate 1/4).
  static_assert(!F16 || kRoom >= 128 * BETA * (2 * P - 1) + 1, "fp32 sums leave their binade after a start");
};

typedef const __attribute__((address_space(1))) uint8_t *gin_t;
typedef __attribute__((address_space(1))) uint8_t *gout_t;
typedef uint32_t una32 __attribute__((aligned(1)));
typedef const __attribute__((address_space(1))) una32 *gword_t;

// What lane tau knows of block tau.
struct Blk {
  const uint8_t *llr;  // the window's first LLR
  uint8_t *out;        // the byte of the core's first bit
  int before;          // LLR bytes of the frame before the window (at most 2^20 counted)
  int M;               // stages of the window
  int core, ncore;     // first core bit within the window, core bits
  bool known, zero, emit;  // starts in state 0; ends in state 0; its bytes are written
};

// Survivor words of the first kept bodies: v128..v255, 16 registers a body,
// moved by asm that names them.  The kernels are compiled for 128 vector
// registers (amdgpu_num_vgpr: the compiler cannot allocate the others) and
// claim all 256 by naming v255 once as overwritten.  (As C++ values the words
// are copied at every branch, and spill.)
#define VITM_KEEP16(N0, N1, N2, N3, N4, N5, N6, N7, N8, N9, N10, N11, N12, N13, N14, N15)                            \
  asm volatile("v_mov_b32 v" #N0 ", %0\n\tv_mov_b32 v" #N1 ", %1\n\tv_mov_b32 v" #N2 ", %2\n\tv_mov_b32 v" #N3        \
               ", %3\n\tv_mov_b32 v" #N4 ", %4\n\tv_mov_b32 v" #N5 ", %5\n\tv_mov_b32 v" #N6 ", %6\n\tv_mov_b32 v" #N7 \
               ", %7\n\tv_mov_b32 v" #N8 ", %8\n\tv_mov_b32 v" #N9 ", %9\n\tv_mov_b32 v" #N10 ", %10\n\tv_mov_b32 v"    \
               #N11 ", %11\n\tv_mov_b32 v" #N12 ", %12\n\tv_mov_b32 v" #N13 ", %13\n\tv_mov_b32 v" #N14              \
               ", %14\n\tv_mov_b32 v" #N15 ", %15" ::"v"(d[0]), "v"(d[1]), "v"(d[2]), "v"(d[3]), "v"(d[4]),         \
               "v"(d[5]), "v"(d[6]), "v"(d[7]), "v"(d[8]), "v"(d[9]), "v"(d[10]), "v"(d[11]), "v"(d[12]),          \
               "v"(d[13]), "v"(d[14]), "v"(d[15]))
#define VITM_KEPT16(N0, N1, N2, N3, N4, N5, N6, N7, N8, N9, N10, N11, N12, N13, N14, N15)                            \
  asm volatile("v_mov_b32 %0, v" #N0 "\n\tv_mov_b32 %1, v" #N1 "\n\tv_mov_b32 %2, v" #N2 "\n\tv_mov_b32 %3, v" #N3   \
               "\n\tv_mov_b32 %4, v" #N4 "\n\tv_mov_b32 %5, v" #N5 "\n\tv_mov_b32 %6, v" #N6 "\n\tv_mov_b32 %7, v" #N7 \
               "\n\tv_mov_b32 %8, v" #N8 "\n\tv_mov_b32 %9, v" #N9 "\n\tv_mov_b32 %10, v" #N10                      \
               "\n\tv_mov_b32 %11, v" #N11 "\n\tv_mov_b32 %12, v" #N12 "\n\tv_mov_b32 %13, v" #N13                  \
               "\n\tv_mov_b32 %14, v" #N14 "\n\tv_mov_b32 %15, v" #N15                                             \
               : "=&v"(d[0]), "=&v"(d[1]), "=&v"(d[2]), "=&v"(d[3]), "=&v"(d[4]), "=&v"(d[5]), "=&v"(d[6]),           \
                 "=&v"(d[7]), "=&v"(d[8]), "=&v"(d[9]), "=&v"(d[10]), "=&v"(d[11]), "=&v"(d[12]), "=&v"(d[13]),       \
                 "=&v"(d[14]), "=&v"(d[15]))
#define VITM_BODIES(OP)                                                                               \
  switch (n) {                                                                                        \
    case 0: OP(128, 129, 130, 131, 132, 133, 134, 135, 136, 137, 138, 139, 140, 141, 142, 143); break;\
    case 1: OP(144, 145, 146, 147, 148, 149, 150, 151, 152, 153, 154, 155, 156, 157, 158, 159); break;\
    case 2: OP(160, 161, 162, 163, 164, 165, 166, 167, 168, 169, 170, 171, 172, 173, 174, 175); break;\
    case 3: OP(176, 177, 178, 179, 180, 181, 182, 183, 184, 185, 186, 187, 188, 189, 190, 191); break;\
    case 4: OP(192, 193, 194, 195, 196, 197, 198, 199, 200, 201, 202, 203, 204, 205, 206, 207); break;\
    case 5: OP(208, 209, 210, 211, 212, 213, 214, 215, 216, 217, 218, 219, 220, 221, 222, 223); break;\
    case 6: OP(224, 225, 226, 227, 228, 229, 230, 231, 232, 233, 234, 235, 236, 237, 238, 239); break;\
    default: OP(240, 241, 242, 243, 244, 245, 246, 247, 248, 249, 250, 251, 252, 253, 254, 255); break;\
  }
__device__ __forceinline__ void keep_words(int n, const uint32_t (&d)[16]) { VITM_BODIES(VITM_KEEP16) }
__device__ __forceinline__ void kept_words(int n, uint32_t (&d)[16]) { VITM_BODIES(VITM_KEPT16) }

// The same for the 4-register layout: v64..v127, compiled for 64.
#define VITM_KEEP4(N0, N1, N2, N3)                                                                        \
  asm volatile("v_mov_b32 v" #N0 ", %0\n\tv_mov_b32 v" #N1 ", %1\n\tv_mov_b32 v" #N2 ", %2\n\tv_mov_b32 v" #N3 ", %3" \
               ::"v"(d[0]), "v"(d[1]), "v"(d[2]), "v"(d[3]))
#define VITM_KEPT4(N0, N1, N2, N3)                                                                        \
  asm volatile("v_mov_b32 %0, v" #N0 "\n\tv_mov_b32 %1, v" #N1 "\n\tv_mov_b32 %2, v" #N2 "\n\tv_mov_b32 %3, v" #N3   \
               : "=&v"(d[0]), "=&v"(d[1]), "=&v"(d[2]), "=&v"(d[3]))
#define VITM_BODIES4(OP)                    \
  switch (n) {                              \
    case 0: OP(64, 65, 66, 67); break;      \
    case 1: OP(68, 69, 70, 71); break;      \
    case 2: OP(72, 73, 74, 75); break;      \
    case 3: OP(76, 77, 78, 79); break;      \
    case 4: OP(80, 81, 82, 83); break;      \
    case 5: OP(84, 85, 86, 87); break;      \
    case 6: OP(88, 89, 90, 91); break;      \
    case 7: OP(92, 93, 94, 95); break;      \
    case 8: OP(96, 97, 98, 99); break;      \
    case 9: OP(100, 101, 102, 103); break;  \
    case 10: OP(104, 105, 106, 107); break; \
    case 11: OP(108, 109, 110, 111); break; \
    case 12: OP(112, 113, 114, 115); break; \
    case 13: OP(116, 117, 118, 119); break; \
    case 14: OP(120, 121, 122, 123); break; \
    default: OP(124, 125, 126, 127); break; \
  }
__device__ __forceinline__ void keep_words(int n, const uint32_t (&d)[4]) { VITM_BODIES4(VITM_KEEP4) }
__device__ __forceinline__ void kept_words(int n, uint32_t (&d)[4]) { VITM_BODIES4(VITM_KEPT4) }

// IN: VIT_LLR_I8 or VIT_LLR_HARD.
template <int K, int BETA, int IN, bool QUAD>
struct DecoderM {
  using Sh = ShapeM<K, BETA, QUAD>;
  static constexpr int P = Sh::P, S = Sh::S, BB = Sh::BB, IB = Sh::IB, NB = Sh::NB, NCLS = Sh::NCLS, NG = Sh::NG,
                       BODY = Sh::BODY, R = Sh::R;
  static constexpr bool F16 = Sh::F16;
  static constexpr int kZero = F16 ? 0x4B400000 : 0;  // bits of metric 0 with tag 0
  // a state that a known start cannot reach begins below every reachable one
  static constexpr int kUnreached = -(256 * P * BETA + 1);

  // per-lane constants
  uint32_t stay[P][F16 ? (BETA + 1) / 2 : 1];  // B: +-2^P per output (bytes, or pairs of fp16): the branch that stays (QUAD,
                                               // q = 4, 5: in lanes of bit q, the one that leaves)
  uint32_t newest[F16 ? (BETA + 1) / 2 : 1];   // xor of that for the branch that leaves for the partner's slot (uniform)
  uint32_t rowsign[F16 ? (BETA + 1) / 2 : 1];  // F16: bits 15 - x and 31 - x: sign of this lane's LLRs in half x of the loads
  int tag[R / 4];             // own tags, per b, of the quad's register whose slot bits are 0
  int lane;
  uint32_t nothing;           // 0, unknown to the compiler (uniform): a copy that it must make where it stands

  // per-wave state
  typename std::conditional<QUAD, i32x4, i32x16>::type o;
  uint32_t dec[R];
  uint32_t raw[Sh::AHEAD];    // the loads ahead: this lane's row and dword
  uint32_t cur[Sh::SPD][F16 && BETA > 2 ? 2 : 1];  // the load in use, as A operands
  gin_t llr;                  // of the block of this lane's A row: the window's first LLR
  int off0;                   // byte offset from there of this lane's dword of timeline stage 0
  int before, end;            // lowest / highest offset of a dword that lies in the frame's window
  int start;                  // lane tau: the timeline stage at which block tau starts, 2 t + (in state 0)
  uint32_t *lds;
  int body, keep;             // bodies from `keep` on are traced, and kept
  int decoded;                // QUAD: place of the decoded words in LDS

  __device__ __forceinline__ static uint32_t rotl_p(uint32_t x, int r) {
    return ((x << r) | (x >> ((P - r) % P))) & (uint32_t)(S - 1);
  }
  // Slot bits in lane l: those of a row of 16, or (QUAD) up to all six.
  __device__ __forceinline__ static int lane_slot(int l) {
    return ((QUAD ? l : l & 15) ^ (((l >> 2) & 1) ? 3 : 0)) & (S - 1);
  }
  // Block of lane l's register r of the metrics, and of lane l's A row.
  __device__ __forceinline__ static int tau_of(int l, int r) {
    if constexpr (QUAD) return ((l >> P) << 2) | r;
    return ((((r >> 2) >> BB) << 4) | ((l >> 4) << 2) | (r & 3)) >> IB;
  }
  __device__ __forceinline__ static int tau_a(int l) {
    if constexpr (QUAD) return ((l >> P) << 2) | (l & 3);
    return ((((l >> 4) >> BB) << 4) | (l & 15)) >> IB;
  }
  // Which of a load's dwords lane l holds.
  __device__ __forceinline__ static int dword_of(int l) { return (l >> (QUAD ? 2 : 4)) & (Sh::DPL - 1); }
  // Register's share of the slot index, and of the lane's blocks.
  static constexpr int reg_slot(int r) { return (((r >> 2) & ((1 << BB) - 1)) << 4) | ((r & ((1 << IB) - 1)) << 6); }
  static constexpr int reg_class(int r) { return QUAD ? r : ((((r >> 2) >> BB) << 2) | (r & 3)) >> IB; }
  static constexpr int class_reg(int c) {
    for (int r = 0; r < R; ++r)
      if (reg_class(r) == c) return r;
    return 0;
  }

  // Parity pattern (bit b) of slot bits st in the branch that stays, phase q.
  __device__ __forceinline__ static uint32_t pattern(const uint32_t *gen, int q, uint32_t st) {
    uint32_t c = 0;
#pragma unroll
    for (int b = 0; b < BETA; ++b) {
      const uint32_t m = rotl_p(gen[b] & (uint32_t)(S - 1), q) ^ (((gen[b] >> P) & 1u) << q);
      c |= (uint32_t)(__builtin_popcount(m & st) & 1) << b;
    }
    return c;
  }
  // Word w of a stage's B operand for sign pattern c.
  __device__ __forceinline__ static uint32_t signs(uint32_t c, int w) {
    uint32_t v = 0;
    if constexpr (F16) {
      constexpr uint32_t one = (uint32_t)(15 + P) << 10;  // fp16 2^P
#pragma unroll
      for (int b = 2 * w; b < BETA && b < 2 * w + 2; ++b)
        v |= (one | (((c >> b) & 1) ? 0x8000u : 0u)) << (16 * (b - 2 * w));
    } else {
#pragma unroll
      for (int b = 0; b < BETA; ++b) v |= (((c >> b) & 1) ? 0x100u - S : (uint32_t)S) << (8 * b + (BETA == 3 ? 8 : 0));
    }
    return v;
  }

  __device__ __forceinline__ void setup(const uint32_t *gen) {
    lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    nothing = 0;
    asm volatile("" : "+s"(nothing));
    constexpr int W = F16 ? (BETA + 1) / 2 : 1;
    uint32_t top = 0;
#pragma unroll
    for (int b = 0; b < BETA; ++b) top |= ((gen[b] >> P) & 1u) << b;
    const uint32_t st = (uint32_t)(lane_slot(lane) | (((lane >> 4) & ((1 << BB) - 1)) << 4));
    const uint32_t row = (uint32_t)(lane & ((1 << IB) - 1)) << 6;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      newest[w] = signs(0, w) ^ signs(top, w);
      rowsign[w] = 0;
    }
#pragma unroll
    for (int q = 0; q < P; ++q) {
      uint32_t c = pattern(gen, q, st);
      if (QUAD && q >= 4) c ^= (lane >> q) & 1 ? top : 0u;
#pragma unroll
      for (int w = 0; w < W; ++w) stay[q][w] = signs(c, w);
    }
    if constexpr (F16) {
#pragma unroll
      for (int x = 0; x < Sh::NL * Sh::SPD; ++x) {
        const int t = (x / Sh::SPD) * Sh::SPL + dword_of(lane) * Sh::SPD + x % Sh::SPD;
        const uint32_t s = pattern(gen, t % P, row);
#pragma unroll
        for (int w = 0; w < W; ++w) rowsign[w] |= (((s >> (2 * w)) & 1) << (15 - x)) | (((s >> (2 * w + 1)) & 1) << (31 - x));
      }
    }
#pragma unroll
    for (int b = 0; b < R / 4; ++b) tag[b] = (S - 1) ^ (lane_slot(lane) | reg_slot(4 * b));
  }
  __device__ __forceinline__ int own_tag(int r) const { return tag[r >> 2] - (reg_slot(r) & ~63); }

  // ---- LLRs.  beta = 2: two stages a dword; 3: a stage's three bytes end the
  // dword; 4: a stage.  A dword ends with its last stage's last LLR, so that
  // none reaches past the window; dwords before the frame or past the window
  // are clamped (no stage of the block's uses them).
  __device__ __forceinline__ int offset(int l, int bd) const { return off0 + (bd * BODY + l * Sh::SPL) * BETA; }
  template <int L>
  __device__ __forceinline__ void load(int bd) {
    int at = offset(L, bd);
    at = at < end ? at : end;
    at = at > before ? at : before;
    raw[L % Sh::AHEAD] = *(gword_t)(llr + at);
  }
  // Load L's dwords as A operands; its register is free for a later one.
  // START: of a body in which blocks start; a dword that straddles the frame's
  // first byte was read from that byte on.
  template <int L, bool START>
  __device__ __forceinline__ void take() {
    uint32_t w = raw[L % Sh::AHEAD];
    if constexpr (START && BETA != 4) {
      const int at = offset(L, body), c = at > before ? at : before;
      w <<= (8 * (c - at)) & 31;
    }
    if constexpr (IN == VIT_LLR_HARD) w = hard_to_pm1(w);
    if constexpr (F16) {
#pragma unroll
      for (int h = 0; h < Sh::SPD; ++h) to_f16(w, h, L * Sh::SPD + h);
    } else {
      cur[0][0] = w ^ nothing;
      if constexpr (Sh::SPD == 2) cur[Sh::SPD - 1][0] = cur[0][0] >> 16;
    }
  }
  // fp16 values of half h's LLR bytes, exact: 0x6400 | (byte + 128) is 1152
  // more than the byte; the row's signs on top.
  __device__ __forceinline__ void to_f16(uint32_t w, int h, int x) {
    asm volatile("" : "+s"(x));  // (keeps the signs out of loop-invariant code motion)
    const uint32_t sel = BETA == 3 ? 0x0C020C01u : h ? 0x0C030C02u : 0x0C010C00u;
    const uint32_t v = __builtin_amdgcn_perm(0u, w, sel) ^ 0x64806480u;
    const f16x2 lo = __builtin_bit_cast(f16x2, v) - (f16x2){(_Float16)1152.0f, (_Float16)1152.0f};
    cur[h][0] = __builtin_bit_cast(uint32_t, lo) ^ ((rowsign[0] << x) & 0x80008000u);
    if constexpr (BETA > 2) {
      constexpr uint32_t sel2 = BETA > 3 ? 0x0C030C02u : 0x0C0C0C03u, off = BETA > 3 ? 0x64806480u : 0x00006480u;
      const uint32_t g = __builtin_amdgcn_perm(0u, w, sel2) ^ off;
      const f16x2 hi = __builtin_bit_cast(f16x2, g) - (f16x2){(_Float16)1152.0f, (_Float16)(BETA > 3 ? 1152.0f : 0.0f)};
      cur[h][F16 && BETA > 2 ? 1 : 0] =
          __builtin_bit_cast(uint32_t, hi) ^ ((rowsign[F16 && BETA > 2 ? 1 : 0] << x) & 0x80008000u);
    }
  }
  __device__ __forceinline__ static f16x4 pair(uint32_t lo, uint32_t hi) {
    return __builtin_bit_cast(f16x4, ((uint64_t)hi << 32) | lo);
  }

  // Blocks that start at timeline stage t: their start metrics.  (Rare: kept
  // out of loop-invariant code motion, which would hold its values in
  // registers through every body.)
  __device__ __forceinline__ void set_starts(int t) {
    int packed = start, from = lane;
    asm volatile("" : "+v"(packed), "+v"(from));
#pragma unroll
    for (int c = 0; c < NCLS; ++c) {
      const int st = __builtin_amdgcn_ds_bpermute(tau_of(from, class_reg(c)) << 2, packed);
      const bool now = (st >> 1) == t;
      const int far = (st & 1) ? kUnreached * S : 0;          // slots other than 0
      const int far0 = lane_slot(from) ? far : 0;             // registers whose share of the slot is 0
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (reg_class(r) != c) continue;
        o[r] = now ? kZero + own_tag(r) + (reg_slot(r) ? far : far0) : o[r];
      }
    }
  }

  // One trellis stage at body offset G.
  template <int G, bool GUARD>
  __device__ __forceinline__ void step() {
    constexpr int q = G % P, load_of = G / Sh::SPL, dword = G % Sh::SPL / Sh::SPD, half = G % Sh::SPD;
    if constexpr (GUARD) {
      const int t = body * BODY + G;
      if (__builtin_amdgcn_ballot_w64((start >> 1) == t)) set_starts(t);
    }
    if constexpr (G % Sh::SPL == 0) {
      take<load_of, GUARD>();
      constexpr int next = (load_of + Sh::AHEAD) % Sh::NL, later = (load_of + Sh::AHEAD) / Sh::NL;
      load<next>(body + later);
    }
    const uint32_t(&w)[F16 && BETA > 2 ? 2 : 1] = cur[half];
    uint32_t flip[F16 && BETA > 2 ? 2 : 1];
#pragma unroll
    for (uint32_t x = 0; x < sizeof(flip) / 4; ++x) {
      flip[x] = newest[x];
      if constexpr (F16) asm volatile("" : "+s"(flip[x]));  // (keeps the products out of loop-invariant code motion)
    }
    decltype(o) out;
    if constexpr (!QUAD) __builtin_amdgcn_s_setprio(1);
    if constexpr (QUAD) {
      out = __builtin_amdgcn_mfma_i32_4x4x4i8((int)w[0], (int)(stay[q][0] ^ flip[0]), o, Sh::CBSZ, dword, 0);
      o = __builtin_amdgcn_mfma_i32_4x4x4i8((int)w[0], (int)stay[q][0], o, Sh::CBSZ, dword, 0);
    } else if constexpr (F16) {
      const f32x16 c = __builtin_bit_cast(f32x16, o);
      constexpr int h = BETA > 2 ? 1 : 0;
      const f16x4 a = pair(w[0], h ? w[h] : 0u);
      const f16x4 leave = pair(stay[q][0] ^ flip[0], h ? stay[q][h] ^ flip[h] : 0u);
      out = __builtin_bit_cast(i32x16, __builtin_amdgcn_mfma_f32_16x16x4f16(a, leave, c, Sh::CBSZ, dword, 0));
      o = __builtin_bit_cast(i32x16, __builtin_amdgcn_mfma_f32_16x16x4f16(a, pair(stay[q][0], h ? stay[q][h] : 0u), c,
                                                                          Sh::CBSZ, dword, 0));
    } else {
      out = __builtin_amdgcn_mfma_i32_16x16x4i8((int)w[0], (int)(stay[q][0] ^ flip[0]), o, Sh::CBSZ, dword, 0);
      o = __builtin_amdgcn_mfma_i32_16x16x4i8((int)w[0], (int)stay[q][0], o, Sh::CBSZ, dword, 0);
    }
    if constexpr (!QUAD) __builtin_amdgcn_s_setprio(0);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if constexpr (q < 4) {
        o[r] = max_i(o[r], devi::exchange<q < 4 ? q : 0>(out[r]));
      } else if constexpr (QUAD) {
        // stay in the lower lanes and leave in the upper ones of o, the others in out: the swap brings a slot's
        // two candidates together
        const auto v = q == 4 ? __builtin_amdgcn_permlane16_swap((uint32_t)o[r], (uint32_t)out[r], false, false)
                              : __builtin_amdgcn_permlane32_swap((uint32_t)o[r], (uint32_t)out[r], false, false);
        o[r] = max_i((int)v[0], (int)v[1]);
      } else {
        o[r] = max_i(o[r], out[r ^ (q < 6 ? 4 << (q < 4 ? 0 : q - 4) : 1 << (q < 6 ? 0 : q - 6))]);
      }
    }
    if constexpr (q == P - 1) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        dec[r] = __builtin_amdgcn_alignbit((uint32_t)o[r], dec[r], P);
        o[r] = ((o[r] & -S) | tag[r >> 2]) - (reg_slot(r) & ~63);
      }
    }
    if constexpr (F16 && (G + 1) % Sh::RENORM == 0) {
      // less the metric of slot 0 (state 0, always reachable): lane 0 of the
      // row, register i of b = 0
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int ref = o[i & ~((1 << IB) - 1)];
        const int d = (__builtin_amdgcn_update_dpp(0, ref, 0x150, 0xF, 0xF, true) & -S) - kZero;  // row_newbcast:0
#pragma unroll
        for (int b = 3; b >= 0; --b) {
          if ((i & ((1 << IB) - 1)) != 0 || b != 0) o[4 * b + i] -= d;
        }
        if (((i + 1) & ((1 << IB) - 1)) == 0) o[i & ~((1 << IB) - 1)] -= d;  // the reference last
      }
    }
    if constexpr (G == BODY - 1) {
      const int at = body - keep;
      if (at >= Sh::NR) {
        store_words(at - Sh::NR, dec);
      } else {
        keep_words(at, dec);
      }
    }
  }

  // A body's survivor words to LDS: [slot's complement][tau], the quad's
  // registers together.
  __device__ __forceinline__ void store_words(int region, const uint32_t (&d)[R]) {
    if constexpr (QUAD) {
      const u32x4 v = {d[0], d[1], d[2], d[3]};
      *(u32x4 *)(lds + region * Sh::REGION + tag[0] * NB + ((lane >> P) << 2)) = v;
      return;
    }
    const int pos = ((15 - lane_slot(lane)) << 4) | ((lane >> 4) << 2);
#pragma unroll
    for (int b = 0; b < R / 4; ++b) {
      // b's slot bits complemented, its block bits as they are
      constexpr int sb = (1 << BB) - 1;
      const int row = (b & ~sb) | (sb - (b & sb));
      u32x4 v;
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i ^ ((1 << IB) - 1)] = d[4 * b + i];
      *(u32x4 *)(lds + region * Sh::REGION + row * 256 + pos) = v;
    }
  }
  // Where the blocks' decoded words of kept body n go: after the survivors, or
  // (where LDS limits the waves) over the survivors of a region that has been
  // traced: the register bodies use region 0 in turn, so they and body NR leave
  // theirs in region 1.
  __device__ __forceinline__ int decoded_at(int n) const {
    if constexpr (QUAD) return decoded + n * NB;
    return n > Sh::NR ? (n - Sh::NR) * Sh::REGION : Sh::REGION + 128 + (Sh::NR - n) * 64;
  }
  __device__ __forceinline__ int last_at(int bodies) const { return QUAD ? decoded + bodies * NB : Sh::REGION + 64; }
  static_assert(QUAD || 128 + (Sh::NR + 1) * 64 <= Sh::REGION, "decoded words of the register bodies");

  // Dword within a body's survivors of block tau's word for complement uc.
  __device__ __forceinline__ static int word_at(uint32_t uc, int tau) {
    if constexpr (QUAD) return (int)uc * NB + tau;
    int at = ((tau >> 4) << (8 + BB)) + (int)((uc & ((16u << BB) - 1u)) << 4) + ((tau & 15) << IB);
    if constexpr (IB) at += (int)(uc >> (4 + BB));
    return at;
  }
};

#define VITM_G1(NN, M)                                     \
  if constexpr ((NN) < (M)) {                              \
    if ((NN) >= from) D.template step<(NN), true>();          \
  }
#define VITM_U1(NN, M) \
  if constexpr ((NN) < (M)) D.template step<(NN), false>();
#define VITM_X8(X, B, M)                                                                 \
  X(B + 0, M) X(B + 1, M) X(B + 2, M) X(B + 3, M) X(B + 4, M) X(B + 5, M) X(B + 6, M)   \
  X(B + 7, M)
#define VITM_X32(X, M) VITM_X8(X, 0, M) VITM_X8(X, 8, M) VITM_X8(X, 16, M) VITM_X8(X, 24, M)

__device__ __forceinline__ int wave_max_all(int v) { return __builtin_amdgcn_readfirstlane(devi::wave_max(v)); }

__device__ __forceinline__ void lds_phase() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The loads ahead of an entry at offset r of the first body; one that is entered
// past its first stage is taken here.
template <int L, class D>
__device__ __forceinline__ void first_loads(D &d, int r) {
  using Sh = typename D::Sh;
  if constexpr (L < Sh::NL) {
    constexpr int first = L * Sh::SPL, past = first + Sh::SPL < Sh::BODY ? first + Sh::SPL : Sh::BODY;
    constexpr int next = (L + Sh::AHEAD) % Sh::NL, later = (L + Sh::AHEAD) / Sh::NL;
    if (L < Sh::AHEAD && r < past) d.template load<L>(0);
    if (r >= past) d.template load<next>(later);
    if (first < r && r < past) {
      d.template take<L, true>();
      d.template load<next>(later);
    }
    first_loads<L + 1>(d, r);
  }
}

// From the survivors to the decoded bytes: uc is lane tau's block's best state's
// complement.
template <class D_>
__device__ __forceinline__ void trace_tile(D_ &D, const Blk &bk, uint32_t uc, int nbody, int grp_lo) {
  using Sh = typename D_::Sh;
  constexpr int P = Sh::P, S = Sh::S, NB = Sh::NB, NG = Sh::NG, BODY = Sh::BODY, R = Sh::R;
  const int lane = D.lane, kept = nbody - grp_lo;
  const int gcore = nbody * BODY - bk.M + bk.core;
  if (bk.zero) uc = S - 1;
  const uint32_t lam_start = uc ^ (uint32_t)(S - 1);
  for (int grp = kept - 1; grp >= 0; --grp) {
    int region = grp - Sh::NR;
    if constexpr (Sh::NR > 0) {
      if (region < 0) {
        region = 0;
        uint32_t d[R];
        kept_words(grp, d);
        D.store_words(0, d);
        lds_phase();
      }
    }
    if (lane < NB) {
      const uint32_t *w = D.lds + region * Sh::REGION;
      uint32_t acc = 0;
#pragma unroll
      for (int g = NG - 1; g >= 0; --g) {
        uc = (w[D.word_at(uc, lane)] >> (32 - BODY + g * P)) & (uint32_t)(S - 1);
        acc |= uc << (g * P);
      }
      D.lds[D.decoded_at(grp) + lane] = ~acc;
    }
    lds_phase();
  }
  if (lane < NB) D.lds[D.last_at(kept) + lane] = lam_start;  // (region 1 has been traced)
  lds_phase();
  lds_phase();

  // ---- output: 64 / NB lanes per block, a dword each where it is whole
  {
    constexpr int LPT = 64 / NB;
    const int tau = lane / LPT, from = tau << 2;
    const int gc = __builtin_amdgcn_ds_bpermute(from, gcore) + P - grp_lo * BODY;
    const int emit = __builtin_amdgcn_ds_bpermute(from, (int)bk.emit);
    const int ncore = emit ? __builtin_amdgcn_ds_bpermute(from, bk.ncore) : 0;
    const uint64_t p = (uint64_t)bk.out;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)(uint32_t)p);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)(uint32_t)(p >> 32));
    const gout_t out = (gout_t)(((uint64_t)hi << 32) | lo);
    constexpr uint32_t body_mask = BODY == 32 ? 0xffffffffu : ((1u << (BODY % 32)) - 1u);
    for (int bit = (lane % LPT) * 32; bit < ncore; bit += 32 * LPT) {
      const int at = gc + bit;
      const int wa = at / BODY, sh = at - wa * BODY;
      auto word = [&](int i) -> uint64_t {
        if (i < kept) return D.lds[D.decoded_at(i) + tau] & body_mask;
        return i == kept ? D.lds[D.last_at(kept) + tau] : 0u;
      };
      uint64_t cat = word(wa) | (word(wa + 1) << BODY);
      if constexpr (BODY < 32) cat |= word(wa + 2) << (2 * BODY);
      uint32_t v = (uint32_t)(cat >> sh);
      const int left = ncore - bit;
      if (left >= 32) {
        *(__attribute__((address_space(1))) una32 *)(out + (bit >> 3)) = v;
      } else {
        v &= (1u << left) - 1u;
        for (int j = 0; j < left; j += 8) out[(bit + j) >> 3] = (uint8_t)(v >> j);
      }
    }
  }
  lds_phase();
}

// Decode NB blocks; lane tau < NB describes block tau (lanes above: any block
// again).  The caller guarantees windows that lie in memory from `before` bytes
// ahead on and, with those bytes, hold at least four.
// `describe` is called before the recursion and again after it, which costs
// less than holding its result in registers.
template <int K, int BETA, int IN, bool QUAD, class Describe>
__device__ __forceinline__ void decode_tile(DecoderM<K, BETA, IN, QUAD> &D, Describe describe) {
  Blk bk = describe();
  using Sh = ShapeM<K, BETA, QUAD>;
  constexpr int P = Sh::P, S = Sh::S, NCLS = Sh::NCLS, BODY = Sh::BODY, R = Sh::R;
  const int lane = D.lane;
  const int most = wave_max_all(bk.M);
  const int r = (BODY - most % BODY) % BODY;
  const int nbody = (most + r) / BODY;
  const int begin = nbody * BODY - bk.M;
  D.start = 2 * begin + (bk.known ? 1 : 0);
  const int grp_lo = -wave_max_all(-(begin + bk.core)) / BODY;  // the first body with a core bit's decision
  D.keep = grp_lo;
  const int kept = nbody - grp_lo;
  D.decoded = (kept - Sh::NR > 1 ? kept - Sh::NR : 1) * Sh::REGION;
  {
    const int from = D.tau_a(lane) << 2;
    const uint64_t p = (uint64_t)bk.llr;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)(uint32_t)p);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)(uint32_t)(p >> 32));
    D.llr = (gin_t)(((uint64_t)hi << 32) | lo);
    const int M = __builtin_amdgcn_ds_bpermute(from, bk.M);
    D.off0 = (M - nbody * BODY + D.dword_of(lane) * Sh::SPD) * BETA - (BETA == 3 ? 1 : 0);
    D.before = -__builtin_amdgcn_ds_bpermute(from, bk.before);
    D.end = M * BETA - 4;
  }
#pragma unroll
  for (int x = 0; x < R; ++x) {
    D.o[x] = D.kZero + D.own_tag(x);
    D.dec[x] = 0u;
  }
  D.body = 0;
  first_loads<0>(D, r);
  const int starts_in = begin / BODY;
  while (D.body < nbody) {  // one body in which blocks start (as in the first), and those up to the next such
    const int from = D.body == 0 ? r : 0;
    VITM_X32(VITM_G1, BODY)
    for (++D.body; D.body < nbody && !__builtin_amdgcn_ballot_w64(starts_in == D.body); ++D.body) {
      VITM_X32(VITM_U1, BODY)
    }
  }
  lds_phase();
  bk = describe();

  // ---- traceback starts: block tau's best state (largest metric, largest
  // complement) to lane tau
  uint32_t uc = S - 1;
#pragma unroll
  for (int c = 0; c < NCLS; ++c) {
    int m = INT32_MIN;
#pragma unroll
    for (int x = 0; x < R; ++x)
      if (D.reg_class(x) == c) m = max_i(m, D.o[x]);
    m = max_i(m, devi::exchange<0>(m));
    m = max_i(m, devi::exchange<1>(m));
    if constexpr (P > 2) m = max_i(m, devi::exchange<2>(m));
    if constexpr (P > 3) m = max_i(m, devi::exchange<3>(m));
    if constexpr (QUAD && P > 4) m = max_i(m, devi::exchange<4>(m));
    if constexpr (QUAD && P > 5) m = max_i(m, devi::exchange<5>(m));
    // to lane tau, if class c is its block's: any lane that holds the block
    constexpr int kQ = 2 - Sh::IB;  // bits of tau below the row quad
    const int at = QUAD ? ((lane >> 2) << P) & 63 : ((lane >> kQ) & 3) << 4;
    const int got = __builtin_amdgcn_ds_bpermute(at << 2, m);
    const int mine = QUAD ? lane & 3 : ((lane >> (kQ + 2)) << kQ) | (lane & ((1 << kQ) - 1));
    uc = mine == c ? (uint32_t)got & (uint32_t)(S - 1) : uc;
  }
  trace_tile(D, bk, uc, nbody, grp_lo);
}

// Stream kernel: wave w decodes blocks [NB w, NB w + NB), then those NB x
// (waves of the grid) further on; blocks past the last are the last again, not
// written.
template <int K, int BETA, int IN, bool QUAD>
__device__ __forceinline__ void blocked_mx(const DecodeArgs &a) {
  using Sh = ShapeM<K, BETA, QUAD>;
  extern __shared__ uint32_t vit_ldsm[];
  DecoderM<K, BETA, IN, QUAD> D;
  D.setup(a.gen);
  D.lds = vit_ldsm;
  const int64_t tiles = (a.nblocks + Sh::NB - 1) / Sh::NB;
  for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    decode_tile(D, [&] {
      int tau = D.lane & (Sh::NB - 1);
      asm volatile("" : "+v"(tau));  // (computed anew at each call)
      const int64_t want = tile * Sh::NB + tau;
      const int64_t blk = want < a.nblocks ? want : a.nblocks - 1;
      const int64_t cs = blk * a.L;
      const int64_t ce = (cs + a.L < a.n) ? cs + a.L : a.n;
      const int64_t s = (cs - a.v1 > 0) ? cs - a.v1 : 0;
      const int64_t e = (ce + a.v2 < a.N) ? ce + a.v2 : a.N;
      Blk b;
      b.llr = (const uint8_t *)a.llr + s * BETA;
      b.out = a.out + (cs >> 3);
      b.before = (int)(s < (1 << 18) ? s * BETA : 1 << 20);
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

// Batch kernel: the code's items (longest first), NB at a time.
template <int K, int BETA, int IN, bool QUAD>
__device__ __forceinline__ void batch_mx(const BatchArgs &a) {
  using Sh = ShapeM<K, BETA, QUAD>;
  extern __shared__ uint32_t vit_ldsm[];
  const int nitems = __builtin_amdgcn_readfirstlane(a.header[kMaxCodes + a.code_index]);
  const int tiles = (nitems + Sh::NB - 1) / Sh::NB;
  if ((int)blockIdx.x >= tiles) return;
  DecoderM<K, BETA, IN, QUAD> D;
  D.setup(a.gen);
  D.lds = vit_ldsm;
  const WorkItem *items = a.items + a.header[2 * kMaxCodes + a.code_index];
  for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    decode_tile(D, [&] {
      int tau = D.lane & (Sh::NB - 1);
      asm volatile("" : "+v"(tau));  // (loaded anew at each call)
      const int want = tile * Sh::NB + tau;
      const WorkItem it = items[want < nitems ? want : nitems - 1];
      Blk b;
      b.llr = (const uint8_t *)a.llr + it.llr_off + (int64_t)it.s * BETA;
      b.out = a.out + it.out_off + (it.cs >> 3);
      b.before = it.s < (1 << 18) ? it.s * BETA : 1 << 20;
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

// Compiled for 128 vector registers and claiming 256, or for 64 and claiming
// 128 (amdgpu_num_vgpr counts in pairs here).
#define VITM_WIDE __global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 8), amdgpu_num_vgpr(64))) void
#define VITM_NARROW __global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4, 8), amdgpu_num_vgpr(32))) void
template <int K, int BETA, int IN>
VITM_WIDE vit_blocked_mx_kernel(DecodeArgs a) {
  asm volatile("" ::: "v255");
  blocked_mx<K, BETA, IN, false>(a);
}
template <int K, int BETA, int IN>
VITM_WIDE vit_batch_mx_kernel(BatchArgs a) {
  asm volatile("" ::: "v255");
  batch_mx<K, BETA, IN, false>(a);
}
template <int K, int BETA, int IN>
VITM_NARROW vit_blocked_quad_kernel(DecodeArgs a) {
  asm volatile("" ::: "v127");
  blocked_mx<K, BETA, IN, true>(a);
}
template <int K, int BETA, int IN>
VITM_NARROW vit_batch_quad_kernel(BatchArgs a) {
  asm volatile("" ::: "v127");
  batch_mx<K, BETA, IN, true>(a);
}

}  // namespace devm

// Kernel instances for (K, beta, input kind VIT_LLR_I8 / VIT_LLR_HARD), taking
// DecodeArgs, or BatchArgs: the 16-register layout (k = 6..9) or the
// 4-register one (k = 3..7).
template <int K, int BETA>
void *pick_kernel_mx_kb(int in, bool batch, bool quad) {
  const bool hard = in == VIT_LLR_HARD;
  if constexpr (K <= 7) {
    if (quad && batch)
      return hard ? (void *)devm::vit_batch_quad_kernel<K, BETA, VIT_LLR_HARD> : (void *)devm::vit_batch_quad_kernel<K, BETA, VIT_LLR_I8>;
    if (quad)
      return hard ? (void *)devm::vit_blocked_quad_kernel<K, BETA, VIT_LLR_HARD> : (void *)devm::vit_blocked_quad_kernel<K, BETA, VIT_LLR_I8>;
  }
  if constexpr (K >= 6) {
    if (!quad && batch)
      return hard ? (void *)devm::vit_batch_mx_kernel<K, BETA, VIT_LLR_HARD> : (void *)devm::vit_batch_mx_kernel<K, BETA, VIT_LLR_I8>;
    if (!quad)
      return hard ? (void *)devm::vit_blocked_mx_kernel<K, BETA, VIT_LLR_HARD> : (void *)devm::vit_blocked_mx_kernel<K, BETA, VIT_LLR_I8>;
  }
  return nullptr;
}
template <int K>
void *pick_kernel_mx_k(int beta, int in, bool batch, bool quad) {
  switch (beta) {
    case 2: return pick_kernel_mx_kb<K, 2>(in, batch, quad);
    case 3: return pick_kernel_mx_kb<K, 3>(in, batch, quad);
    case 4: return pick_kernel_mx_kb<K, 4>(in, batch, quad);
  }
  return nullptr;
}

void *pick_kernel_mx_k3(int beta, int in, bool batch, bool quad);
void *pick_kernel_mx_k4(int beta, int in, bool batch, bool quad);
void *pick_kernel_mx_k5(int beta, int in, bool batch, bool quad);
void *pick_kernel_mx_k6(int beta, int in, bool batch, bool quad);
void *pick_kernel_mx_k7(int beta, int in, bool batch, bool quad);
void *pick_kernel_mx_k8(int beta, int in, bool batch, bool quad);
void *pick_kernel_mx_k9(int beta, int in, bool batch, bool quad);

}  // namespace vit
