// vit_launch.hip -- host side of the blocked decoder: kernel selection,
// occupancy-based grid size, LDS sizing and launch.
#include "vit_decoder.h"
#include "vit_decoder16.h"
#include "vit_decoder_int.h"
#include "vit_decoder_mx.h"
#include "vit_decoder_row.h"
#include "vit_shapes.h"

#include <utility>

namespace vit {
namespace {


// Every generator taps the newest input (bit k-1).
bool taps_newest(int k, int beta, const uint32_t *gen) {
  bool t = true;
  for (int b = 0; b < beta; ++b) t = t && ((gen[b] >> (k - 1)) & 1u);
  return t;
}

// Every generator taps both ends of the register.
bool taps_both_ends(int k, int beta, const uint32_t *gen) {
  bool t = taps_newest(k, beta, gen);
  for (int b = 0; b < beta; ++b) t = t && (gen[b] & 1u);
  return t;
}

void *pick_kernel_int(int k, int beta, const uint32_t *gen, int in, bool batch) {
  const bool top = taps_newest(k, beta, gen);
  switch (k) {
    case 3: return pick_kernel_int_k3(beta, top, in, batch);
    case 4: return pick_kernel_int_k4(beta, top, in, batch);
    case 5: return pick_kernel_int_k5(beta, top, in, batch);
    case 6: return pick_kernel_int_k6(beta, top, in, batch);
    case 7: return pick_kernel_int_k7(beta, top, in, batch);
    case 8: return pick_kernel_int_k8(beta, top, in, batch);
    case 9: return pick_kernel_int_k9(beta, top, in, batch);
  }
  return nullptr;
}

void *pick_kernel_mx(int k, int beta, int in, bool batch, bool quad) {
  switch (k) {
    case 3: return pick_kernel_mx_k3(beta, in, batch, quad);
    case 4: return pick_kernel_mx_k4(beta, in, batch, quad);
    case 5: return pick_kernel_mx_k5(beta, in, batch, quad);
    case 6: return pick_kernel_mx_k6(beta, in, batch, quad);
    case 7: return pick_kernel_mx_k7(beta, in, batch, quad);
    case 8: return pick_kernel_mx_k8(beta, in, batch, quad);
    case 9: return pick_kernel_mx_k9(beta, in, batch, quad);
  }
  return nullptr;
}

KernelFn pick_kernel(int k, int beta, bool stdc, int in, bool sub) {
  switch (k) {
    case 3: return sub ? pick_kernel_sub_k3(beta, stdc, in) : pick_kernel_k3(beta, stdc, in);
    case 4: return sub ? pick_kernel_sub_k4(beta, stdc, in) : pick_kernel_k4(beta, stdc, in);
    case 5: return sub ? pick_kernel_sub_k5(beta, stdc, in) : pick_kernel_k5(beta, stdc, in);
    case 6: return sub ? pick_kernel_sub_k6(beta, stdc, in) : pick_kernel_k6(beta, stdc, in);
    case 7: return sub ? pick_kernel_sub_k7(beta, stdc, in) : pick_kernel_k7(beta, stdc, in);
    case 8: return sub ? pick_kernel_sub_k8(beta, stdc, in) : pick_kernel_k8(beta, stdc, in);
    case 9: return sub ? pick_kernel_sub_k9(beta, stdc, in) : pick_kernel_k9(beta, stdc, in);
  }
  return nullptr;
}

int body_len(int k) {
  const int P = k - 1;
  return P * (32 / P);
}

void *pick_kernel16(int k, int beta, int in, bool batch) {
  switch (k) {
    case 3: return pick_kernel16_k3(beta, in, batch);
    case 4: return pick_kernel16_k4(beta, in, batch);
    case 5: return pick_kernel16_k5(beta, in, batch);
    case 6: return pick_kernel16_k6(beta, in, batch);
    case 7: return pick_kernel16_k7(beta, in, batch);
    case 8: return pick_kernel16_k8(beta, in, batch);
    case 9: return pick_kernel16_k9(beta, in, batch);
  }
  return nullptr;
}

struct DeviceInfo {
  int dev = -1;
  int num_cu = 0;
  int max_lds = 0;
};
thread_local DeviceInfo t_dev;

}  // namespace

int64_t lds_bytes_per_block(int k, int beta, int64_t max_block_stages) {
  if (k < 3 || k > 9 || beta < 2 || beta > 4) return 0;
  const int64_t body = body_len(k);
  const int64_t regs = (k > 7) ? (1 << (k - 1)) / 64 : 1;
  const int64_t bodies = (max_block_stages + body - 1) / body;  // block + entry offset fill whole bodies
  return bodies * regs * 64 * 4;
}

int64_t lds16_bytes_per_wave(int k, int beta, int64_t max_block_stages) {
  if (k < 3 || k > 9 || beta < 2 || beta > 4) return 0;
  const int64_t body = dev16::body16(k - 1);
  const int64_t regs = (k > 7) ? (1 << (k - 1)) / 64 : 1;
  const int64_t bodies = (max_block_stages + body - 1) / body;
  return bodies * regs * 64 * 4;
}

bool fp32_integer_exact(int beta, int64_t max_block_stages) {
  return max_block_stages * 128 * beta < ((int64_t)1 << 24);
}

namespace {

hipError_t device_info() {
  int dev = 0;
  hipError_t err = hipGetDevice(&dev);
  if (err != hipSuccess) return err;
  if (t_dev.dev != dev) {
    err = hipDeviceGetAttribute(&t_dev.num_cu, hipDeviceAttributeMultiprocessorCount, dev);
    if (err != hipSuccess) return err;
    err = hipDeviceGetAttribute(&t_dev.max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
    if (err != hipSuccess) return err;
    t_dev.dev = dev;
  }
  return hipSuccess;
}

void *pick_kernel_row(int k, int beta, bool batch) {
  switch (k) {
    case 3: return pick_kernel_row_k3(beta, batch);
    case 4: return pick_kernel_row_k4(beta, batch);
    case 5: return pick_kernel_row_k5(beta, batch);
    case 6: return pick_kernel_row_k6(beta, batch);
  }
  return nullptr;
}

// Resolve the integer metric width for a decode of blocks of at most
// max_block_stages stages: the 16-bit kernels where asked for, the 32-bit
// integer kernels where asked for or (auto) where their bound and the one-block
// kernel's survivor storage allow, else (auto) the 16-bit kernels where two
// blocks' survivors fit a workgroup's LDS.  Auto prefers 32 bits, which measured
// faster (8192 int8 frames of three codes 0.36 ms, with 16-bit
// metrics 1.00).  -1 = no kernel (why is set).
int resolve_metric(int k, int beta, int in, int metric_bits, int64_t max_block_stages, const char **why) {
  if (in == VIT_LLR_F32) return 0;
  const bool fits16 = lds16_bytes_per_wave(k, beta, max_block_stages) <= t_dev.max_lds;
  const bool fits32 = lds_bytes_per_block(k, beta, max_block_stages) <= t_dev.max_lds &&
                      fp32_integer_exact(beta, max_block_stages);
  if (metric_bits == kMetric16 || (metric_bits == kMetricAuto && !fits32 && fits16)) {
    if (!fits16) *why = "the 16-bit metric kernel's survivor storage for two blocks exceeds the per-workgroup LDS";
    return fits16 ? kMetric16 : -1;
  }
  if (!fits32) {
    *why = lds_bytes_per_block(k, beta, max_block_stages) > t_dev.max_lds
               ? "one block's survivor storage exceeds the per-workgroup LDS"
               : "int8 block too long for exact integers in fp32 (use 16-bit metrics)";
    return -1;
  }
  return kMetric32;
}

// The 16-bit metric stream kernel: one wave per pair of blocks.
hipError_t launch_blocked16(const DecodeArgs &a, hipStream_t stream, int *unsupported, const char **why) {
  void *fn = pick_kernel16(a.k, a.beta, a.llr_type, false);
  if (!fn) {
    *unsupported = 1;
    *why = "no 16-bit metric kernel instance for this (k, beta)";
    return hipSuccess;
  }
  const int64_t lds_wave = lds16_bytes_per_wave(a.k, a.beta, a.max_block_stages);
  int wpb = (2 * lds_wave <= t_dev.max_lds) ? 2 : 1;
  int occ = 0;
  hipError_t err = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, fn, 64 * wpb, (size_t)lds_wave * wpb);
  if (err != hipSuccess) return err;
  if (occ < 1) occ = 1;
  // same rule as the one-block-per-wave kernels (launch_blocked), in pairs
  const bool persistent = a.max_block_stages >= 1000 || occ <= 4;
  if (!persistent) wpb = 1;
  const size_t lds = (size_t)lds_wave * wpb;
  const int64_t npairs = (a.nblocks + 1) / 2;
  const int64_t need = (npairs + wpb - 1) / wpb;
  int64_t grid = need;
  if (persistent) {
    grid = (int64_t)occ * t_dev.num_cu;
    if (grid >= need) grid = need;
    else grid = grid / 8 * 8;
  }
  if (grid < 1) grid = 1;
  if (lds > 65536) {
    err = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (err != hipSuccess) return err;
  }
  DecodeArgs args = a;
  int words = (int)(lds_wave / 4);
  void *kargs[] = {&args, &words};
  err = hipLaunchKernel(fn, dim3((unsigned)grid), dim3(64 * wpb), kargs, lds, stream);
  if (err != hipSuccess) return err;
  return hipGetLastError();
}

// ---- the matrix-core kernels (vit_decoder_mx.h)

// Two layouts: 16 metric registers a wave (k = 6..9), or 4 (quad, k = 3..7).
bool mx_takes(int k, bool quad) { return quad ? k <= 7 : k >= 6; }
int mx_blocks(int k, bool quad) { return 1 << ((quad ? 9 : 11) - k); }  // per wave

// LDS of a wave whose blocks are traced over `traced` stages (from the first
// core bit to the window's end): survivors of the bodies beyond those in
// registers, and (quad) the decoded words.
int64_t mx_lds_bytes(int k, int64_t traced, bool quad) {
  const int64_t body = body_len(k);
  const int64_t bodies = (traced + body - 1) / body;
  const int64_t regions = bodies - devm::kept_bodies(quad);
  if (!quad) return (regions > 2 ? regions : 2) * 4 * devm::region_words(false);
  return 4 * ((regions > 1 ? regions : 1) * devm::region_words(true) + (bodies + 1) * mx_blocks(k, true));
}

// Waves a CU holds: two per SIMD by registers (quad: four), fewer by LDS (in
// units of 1280 bytes).
int mx_waves_per_cu(int64_t lds, int max_lds, bool quad) {
  const int64_t unit = (lds + 1279) / 1280 * 1280;
  const int64_t by_lds = max_lds / unit, most = quad ? 16 : 8;
  return (int)(by_lds < most ? by_lds : most);
}

// Time per stage (nanoseconds) of the three integer kernels for `blocks`
// blocks, measured with the chip full and with one wave on a SIMD; a block's
// stages are the same for all, so the least is the fastest.  Measured around
// the lines between them (us, one-block kernel / 16 registers / 4 registers):
// K=7 r1/2, L = 256, 1024 blocks 11 / 34 / 19, 4096 20 / 34 / 20,
// 16384 58 / 39 / 36, 65536 210 / 84 / 113; K=7, L = 512 (here LDS holds four
// waves of the 16-register kernel a CU), 8192 blocks 59 / 60 / 39,
// 32768 199 / 121 / 107; K=7, L = 1024, 16384 blocks 223 / 407 / 168;
// K=6, L = 256, 4096 blocks 20 / 35 / 19, 65536 209 / 49 / 60; K=5, L = 256,
// 4096 blocks 20 / - / 18, 65536 204 / - / 34; K=3, L = 256, 4096 blocks
// 22 / - / 24, 16384 58 / - / 25; K=9, L = 256, 1024 blocks 26 / 38 / -,
// 4096 66 / 48 / -, 16384 237 / 94 / -.  Over eight lengths (64 to 2048) and
// thirteen sizes of eight codes the choice took 0.2 % more than the best in the
// mean, and more than 10 % at eight: K=3, 4 and 7 r1/3 with 2900 to 4096 long
// blocks (to 15 %), K=6 at L = 320, 2^24 bits (13 %), K=7 at L = 64, 4096 blocks
// (18 %), K=8 at L = 512, 4096 blocks (13 %), K=9 at L = 768, 1366 blocks (14 %).
//
// One block a wave: one wave's latency, and 10.6 for each further 64 states on
// a SIMD; in rounds where LDS (lds: a block's) holds fewer than four waves a SIMD.
double one_block_ns(int k, int64_t blocks, int64_t simds, int64_t lds, int max_lds) {
  const double regs = k > 7 ? 1 << (k - 7) : 1;
  const double latency = k <= 7 ? 24.0 : k == 8 ? 30.0 : 70.0;
  const double waves = (double)((blocks + simds - 1) / simds);
  const double fit = (double)(max_lds / ((lds + 1279) / 1280 * 1280)) / 4;
  if (fit < 4 && waves > fit) return waves / fit * (latency + 10.6 * regs * (fit > 1 ? fit - 1 : 0));
  return latency + 10.6 * regs * (waves - 1);
}
// 16 registers: a second wave on a SIMD costs half as much again (some get one
// before every SIMD has its first); as many as fit at a time, whole rounds of
// persistent waves where that is at most one a SIMD (mx_grid).
double mx_ns(int k, int64_t blocks, int64_t simds, int per_cu) {
  const int64_t slots = per_cu * simds / 4;
  const int64_t tiles = (blocks + mx_blocks(k, false) - 1) / mx_blocks(k, false);
  const double wave = k == 6 ? 106.0 : k == 7 ? 95.0 : k == 8 ? 100.0 : 115.0;
  if (per_cu <= 4) return (double)((tiles + slots - 1) / slots) * wave;
  const double share = tiles > simds ? 1.55 * wave : tiles > simds / 2 ? 1.3 * wave : wave;
  return tiles > slots ? (double)tiles / (double)slots * share : share;
}
// 4 registers: each further wave on a SIMD 15 more, in rounds of as many as fit.
double quad_ns(int k, int64_t blocks, int64_t simds, int per_cu) {
  const double lone = k == 3 ? 68.0 : k == 4 ? 58.0 : 49.0;
  const int64_t tiles = (blocks + mx_blocks(k, true) - 1) / mx_blocks(k, true), slots = per_cu * simds / 4;
  const int64_t full = (tiles - 1) / slots;
  if (per_cu < 4) return lone * (double)(full + 1);
  const double waves = (double)(tiles - full * slots) / (double)simds;
  return (double)full * (lone + 15 * (per_cu / 4.0 - 1)) + lone + (waves > 1 ? 15 * (waves - 1) : 0);
}

// Workgroups (of one wave): one per tile, refilled by the dispatcher, where
// several waves share a SIMD; where LDS allows at most one per SIMD, that many
// persistent waves (K=7, L = 512, 2^24 bits, 16 registers: 117 us against 149,
// the dispatcher's refills landing two on one SIMD).
unsigned mx_grid(int k, int64_t blocks, int64_t lds, int num_cu, int max_lds, bool quad) {
  const int64_t tiles = (blocks + mx_blocks(k, quad) - 1) / mx_blocks(k, quad);
  const int per_cu = mx_waves_per_cu(lds, max_lds, quad);
  const int64_t slots = (int64_t)per_cu * num_cu;
  return (unsigned)(per_cu <= 4 && tiles > slots ? slots : tiles);
}

hipError_t launch_blocked_mx(const DecodeArgs &a, int64_t lds, bool quad, hipStream_t stream) {
  void *fn = pick_kernel_mx(a.k, a.beta, a.llr_type, false, quad);
  if (lds > 65536) {
    const hipError_t err = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (err != hipSuccess) return err;
  }
  DecodeArgs args = a;
  void *kargs[] = {&args};
  const unsigned grid = mx_grid(a.k, a.nblocks, lds, t_dev.num_cu, t_dev.max_lds, quad);
  const hipError_t err = hipLaunchKernel(fn, dim3(grid), dim3(64), kargs, (size_t)lds, stream);
  if (err != hipSuccess) return err;
  return hipGetLastError();
}

// ---- the FP32 kernels of four blocks a wave (vit_decoder_row.h)

// (rate 1/4 builds a table per stage and spills: K=4 507 us against 347 at
// 2^24 bits, L = 64; K=7's four phases across lanes cost what its two permlane
// phases do: 245 us against 254 at L = 256, and 320 against 238 at L = 512)
bool row_takes(int k, int beta, const uint32_t *gen) { return k <= 6 && beta <= 3 && taps_both_ends(k, beta, gen); }

// LDS of a wave: the survivors of four blocks, and the decoded words.
int64_t row_lds_bytes(int k, int64_t traced) {
  const int64_t body = body_len(k), bodies = (traced + body - 1) / body;
  return 16 * ((bodies << (k - 1)) + bodies + 1);
}

// Whether `blocks` FP32 blocks take less time four a wave, by the time per
// stage (nanoseconds) of both, measured with one wave on a SIMD and with the
// chip full.  One block a wave: 30, and 10.5 for each further on a SIMD.  Four:
// 44 (k = 5, rate 1/2), 56 or 62 (k = 6), and 13 (20) for each further wave, as
// many as registers (four a SIMD) and LDS hold at a time.  Measured (us, one /
// four a wave): K=5 r1/2, L = 256, 4096 blocks 22 / 18, 16384 63 / 27, 65536
// 214 / 82; K=5, L = 512, 2048 blocks 23 / 28, 4096 37 / 29; K=6 r1/2, L = 256,
// 4096 blocks 23 / 25, 8192 36 / 28, 65536 221 / 130; K=6 r1/3, L = 512, 32768
// blocks 226 / 129; K=3 r1/2, L = 256, 3104 blocks 21 / 21, 65536 204 / 83.  Over
// the lengths and sizes above the choice took at most 6 % more than the better one
// but for K=6 r1/3 at L = 2048, 4096 blocks (208 / 147).
bool row_is_faster(int k, int beta, int64_t blocks, int64_t lds, int num_cu, int max_lds) {
  const int64_t unit = (lds + 1279) / 1280 * 1280, by_lds = max_lds / unit;
  const double fit = by_lds < 16 ? (double)by_lds / 4 : 4.0;
  if (fit < 0.5) return false;
  const int64_t simds = 4 * (int64_t)num_cu, tiles = (blocks + 3) / 4;
  const double one = 30.0 + 10.5 * (double)((blocks - 1) / simds);
  const double lone = k == 6 ? 62.0 : k == 5 && beta == 2 ? 44.0 : 56.0, more = k == 6 ? 20.0 : 13.0;
  const double waves = (double)((tiles + simds - 1) / simds);
  const double four = waves <= fit ? lone + more * (waves - 1) : waves / fit * (lone + more * (fit > 1 ? fit - 1 : 0));
  return four < one;
}
unsigned row_grid(int64_t blocks) { return (unsigned)((blocks + 3) / 4); }

hipError_t launch_blocked_row(const DecodeArgs &a, int64_t lds, hipStream_t stream) {
  void *fn = pick_kernel_row(a.k, a.beta, false);
  if (lds > 65536) {
    const hipError_t err = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (err != hipSuccess) return err;
  }
  DecodeArgs args = a;
  void *kargs[] = {&args};
  const hipError_t err = hipLaunchKernel(fn, dim3(row_grid(a.nblocks)), dim3(64), kargs, (size_t)lds, stream);
  if (err != hipSuccess) return err;
  return hipGetLastError();
}

// ---- the choice between them

// LDS bytes of a wave of each kernel for blocks of at most max_block_stages
// stages, `traced` of them from the first core bit on; 0 where that kernel
// cannot take them.
struct Layouts {
  int64_t one, mx, quad, row;
};
Layouts layouts(int k, int beta, const uint32_t *gen, int in, int64_t max_block_stages, int64_t traced, int max_lds) {
  auto fits = [&](int64_t lds) { return lds <= max_lds ? lds : 0; };
  Layouts l = {fits(lds_bytes_per_block(k, beta, max_block_stages)), 0, 0, 0};
  // (a shape that one block a wave cannot hold is refused, whatever the others could)
  if (!l.one || traced <= 0) return l;
  if (in == VIT_LLR_F32) {
    if (row_takes(k, beta, gen)) l.row = fits(row_lds_bytes(k, traced));
  } else {
    if (mx_takes(k, false)) l.mx = fits(mx_lds_bytes(k, traced, false));
    if (mx_takes(k, true)) l.quad = fits(mx_lds_bytes(k, traced, true));
  }
  return l;
}

// The kernel that takes the least time for `blocks` blocks.
int choose_kernel(int k, int beta, const Layouts &l, int64_t blocks, int num_cu, int max_lds) {
  if (blocks < 2) return VIT_KERNEL_ONE_BLOCK;
  if (l.row && row_is_faster(k, beta, blocks, l.row, num_cu, max_lds)) return VIT_KERNEL_ROW;
  const int64_t simds = 4 * (int64_t)num_cu;
  int best = VIT_KERNEL_ONE_BLOCK;
  double ns = l.mx || l.quad ? one_block_ns(k, blocks, simds, l.one, max_lds) : 0;
  for (const bool quad : {false, true}) {
    const int64_t lds = quad ? l.quad : l.mx;
    if (!lds) continue;
    const int per_cu = mx_waves_per_cu(lds, max_lds, quad);
    if (per_cu < 1) continue;
    const double t = quad ? quad_ns(k, blocks, simds, per_cu) : mx_ns(k, blocks, simds, per_cu);
    if (t < ns) {
      ns = t;
      best = quad ? VIT_KERNEL_MX4 : VIT_KERNEL_MX16;
    }
  }
  return best;
}

}  // namespace

int kernel_for(int k, int beta, const uint32_t *gen, int in, int64_t blocks, int64_t max_block_stages, int64_t traced,
               int num_cu, int max_lds) {
  const Layouts l = layouts(k, beta, gen, in, max_block_stages, traced, max_lds);
  if (!l.one || (in != VIT_LLR_F32 && !fp32_integer_exact(beta, max_block_stages))) return -1;
  return choose_kernel(k, beta, l, blocks, num_cu, max_lds);
}

hipError_t launch_blocked(const DecodeArgs &a, hipStream_t stream, int *unsupported, const char **why) {
  *unsupported = 0;
  {
    const hipError_t err = device_info();
    if (err != hipSuccess) return err;
  }
  const Layouts l = layouts(a.k, a.beta, a.gen, a.llr_type, a.max_block_stages, a.sub_bits == 0 ? a.L + a.v2 : 0, t_dev.max_lds);
  if (a.llr_type != VIT_LLR_F32 && a.sub_bits == 0) {
    const int m = resolve_metric(a.k, a.beta, a.llr_type, a.metric_bits, a.max_block_stages, why);
    if (m < 0) {
      *unsupported = 1;
      return hipSuccess;
    }
    if (m == kMetric16) return launch_blocked16(a, stream, unsupported, why);
  } else if (a.llr_type != VIT_LLR_F32) {
    // subframe traceback: the exact-in-fp32 integer kernels only
    if (a.metric_bits == kMetric16) {
      *unsupported = 1;
      *why = "subframe traceback runs with 32-bit metrics only";
      return hipSuccess;
    }
    if (!fp32_integer_exact(a.beta, a.max_block_stages)) {
      *unsupported = 1;
      *why = "int8 block too long for exact integers in fp32";
      return hipSuccess;
    }
  }
  switch (choose_kernel(a.k, a.beta, l, a.nblocks, t_dev.num_cu, t_dev.max_lds)) {
    case VIT_KERNEL_MX16: return launch_blocked_mx(a, l.mx, false, stream);
    case VIT_KERNEL_MX4: return launch_blocked_mx(a, l.quad, true, stream);
    case VIT_KERNEL_ROW: return launch_blocked_row(a, l.row, stream);
  }
  const void *fn = a.llr_type != VIT_LLR_F32 && a.sub_bits == 0
                       ? pick_kernel_int(a.k, a.beta, a.gen, a.llr_type, false)
                       : reinterpret_cast<const void *>(pick_kernel(a.k, a.beta, taps_both_ends(a.k, a.beta, a.gen),
                                                                    a.llr_type, a.sub_bits > 0));
  if (!fn) {
    *unsupported = 1;
    *why = "no kernel instance for this (k, beta)";
    return hipSuccess;
  }
  hipError_t err;
  // the parallel traceback keeps one decoded byte per core bit after the survivors
  const int64_t lds_wave = lds_bytes_per_block(a.k, a.beta, a.max_block_stages) +
                           (a.sub_bits > 0 ? (a.L + 3) / 4 * 4 : 0);
  if (lds_wave > t_dev.max_lds) {
    *unsupported = 1;
    *why = "one block's survivor storage exceeds the per-workgroup LDS";
    return hipSuccess;
  }
  // Grid: one block per wave, the hardware dispatcher refilling a CU as soon
  // as a workgroup ends, except for long blocks or low occupancy, where
  // persistent waves that loop over blocks are faster.  Measured on 2^24-bit
  // streams: one block per wave is 5-15% faster for K=7 up to L = 896 and
  // K=9 up to L = 448; persistent waves are 5-16% faster from about 1000
  // stages per block (K=5..7, L = 1024, 2048) and at 4 or fewer two-wave
  // workgroups per CU (K=9, L = 512).  Persistent waves run two per
  // workgroup where their survivor storage fits (8-25% faster than one);
  // one block per wave runs one wave per workgroup (K=7 r1/2 at L = 512:
  // 64.0 against 62.2 Gb/s; -2% to +5% for the other codes and lengths).
  int wpb = (2 * lds_wave <= t_dev.max_lds) ? 2 : 1;
  int occ = 0;
  err = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, fn, 64 * wpb,
                                                     (size_t)lds_wave * wpb);
  if (err != hipSuccess) return err;
  if (occ < 1) occ = 1;
  const bool persistent = a.max_block_stages >= 1000 || occ <= 4;
  if (!persistent) wpb = 1;
  const size_t lds = (size_t)lds_wave * wpb;
  const int64_t need = (a.nblocks + wpb - 1) / wpb;
  int64_t grid = need;
  if (persistent) {
    grid = (int64_t)occ * t_dev.num_cu;
    if (grid >= need) grid = need;
    else grid = grid / 8 * 8;
  }
  if (grid < 1) grid = 1;
  if (lds > 65536) {
    err = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)lds);
    if (err != hipSuccess) return err;
  }
  DecodeArgs args = a;
  int words = (int)(lds_wave / 4);
  void *kargs[] = {&args, &words};
  err = hipLaunchKernel(fn, dim3((unsigned)grid), dim3(64 * wpb), kargs, lds,
                        stream);
  if (err != hipSuccess) return err;
  return hipGetLastError();
}

unsigned batch_launch_grid(const BatchLaunch &bl, int64_t count, int64_t max_block_stages, int num_cu) {
  const int64_t units = (count + bl.items_per_wave - 1) / bl.items_per_wave;
  return batch_grid(units, (int)(bl.block / 64), max_block_stages, bl.grid, num_cu);
}

BatchGrid batch_grid_for(const BatchLaunch &bl, int64_t count, int64_t max_block_stages, bool whole_words) {
  const Layouts l = {(int64_t)bl.lds_words_per_wave * 4, whole_words ? (int64_t)bl.mx_lds[0] : 0,
                     whole_words ? (int64_t)bl.mx_lds[1] : 0, (int64_t)bl.row_lds};
  const int which = choose_kernel(bl.k, bl.beta, l, count, bl.num_cu, bl.max_lds);
  if (which == VIT_KERNEL_ROW) return {bl.row_fn, row_grid(count), 64, bl.row_lds};
  if (which != VIT_KERNEL_ONE_BLOCK) {
    const bool quad = which == VIT_KERNEL_MX4;
    return {bl.mx_fn[quad], mx_grid(bl.k, count, (int64_t)bl.mx_lds[quad], bl.num_cu, bl.max_lds, quad), 64, bl.mx_lds[quad]};
  }
  return {bl.fn, batch_launch_grid(bl, count, max_block_stages, bl.num_cu), bl.block, bl.lds};
}

hipError_t plan_batch_launch(int k, int beta, const uint32_t *gen, int in, int metric_bits, int64_t max_block_stages,
                             int64_t traced, int wpb, BatchLaunch *bl, int *unsupported, const char **why) {
  *unsupported = 0;
  {
    const hipError_t err = device_info();
    if (err != hipSuccess) return err;
  }
  bl->k = k;
  bl->beta = beta;
  bl->num_cu = t_dev.num_cu;
  bl->max_lds = t_dev.max_lds;
  bl->row_fn = nullptr;
  bl->row_lds = 0;
  for (const bool quad : {false, true}) {
    bl->mx_fn[quad] = nullptr;
    bl->mx_lds[quad] = 0;
  }
  const int metric = resolve_metric(k, beta, in, metric_bits, max_block_stages, why);
  if (metric < 0) {
    *unsupported = 1;
    return hipSuccess;
  }
  if (metric == kMetric16) {
    void *fn16 = pick_kernel16(k, beta, in, true);
    if (!fn16) {
      *unsupported = 1;
      *why = "no 16-bit metric batch kernel instance for this (k, beta)";
      return hipSuccess;
    }
    const int64_t lds_wave = lds16_bytes_per_wave(k, beta, max_block_stages);
    const size_t lds = (size_t)lds_wave * wpb;
    if ((int64_t)lds > t_dev.max_lds) {
      *unsupported = 1;
      *why = "the workgroup's survivor storage exceeds the per-workgroup LDS";
      return hipSuccess;
    }
    hipError_t err;
    if (lds > 65536) {
      err = hipFuncSetAttribute(fn16, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (err != hipSuccess) return err;
    }
    int occ = 0;
    err = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, fn16, 64 * wpb, lds);
    if (err != hipSuccess) return err;
    if (occ < 1) occ = 1;
    bl->fn = fn16;
    bl->grid = (unsigned)(occ * t_dev.num_cu);
    bl->block = (unsigned)(64 * wpb);
    bl->lds = lds;
    bl->lds_words_per_wave = (int)(lds_wave / 4);
    bl->items_per_wave = 2;
    bl->metric_bits = kMetric16;
    return hipSuccess;
  }
  const void *fn = nullptr;
  const bool stdc = taps_both_ends(k, beta, gen);
  if (in != VIT_LLR_F32) fn = pick_kernel_int(k, beta, gen, in, true);
  else switch (k) {
    case 3: fn = reinterpret_cast<const void *>(pick_batch_kernel_k3(beta, stdc)); break;
    case 4: fn = reinterpret_cast<const void *>(pick_batch_kernel_k4(beta, stdc)); break;
    case 5: fn = reinterpret_cast<const void *>(pick_batch_kernel_k5(beta, stdc)); break;
    case 6: fn = reinterpret_cast<const void *>(pick_batch_kernel_k6(beta, stdc)); break;
    case 7: fn = reinterpret_cast<const void *>(pick_batch_kernel_k7(beta, stdc)); break;
    case 8: fn = reinterpret_cast<const void *>(pick_batch_kernel_k8(beta, stdc)); break;
    case 9: fn = reinterpret_cast<const void *>(pick_batch_kernel_k9(beta, stdc)); break;
  }
  if (!fn) {
    *unsupported = 1;
    *why = "no batch kernel instance for this (k, beta)";
    return hipSuccess;
  }
  hipError_t err;
  const int64_t lds_wave = lds_bytes_per_block(k, beta, max_block_stages);
  const size_t lds = (size_t)lds_wave * wpb;
  if ((int64_t)lds > t_dev.max_lds) {
    *unsupported = 1;
    *why = "a block's survivor storage exceeds the per-workgroup LDS";
    return hipSuccess;
  }
  if (lds > 65536) {
    err = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)lds);
    if (err != hipSuccess) return err;
  }
  int occ = 0;
  err = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, fn, 64 * wpb, lds);
  if (err != hipSuccess) return err;
  if (occ < 1) occ = 1;
  bl->fn = fn;
  bl->grid = (unsigned)(occ * t_dev.num_cu);
  bl->block = (unsigned)(64 * wpb);
  bl->lds = lds;
  bl->lds_words_per_wave = (int)(lds_wave / 4);
  bl->items_per_wave = 1;
  bl->metric_bits = metric;
  const Layouts l = layouts(k, beta, gen, in, max_block_stages, traced, t_dev.max_lds);
  if (l.row) bl->row_fn = pick_kernel_row(k, beta, true);
  bl->row_lds = (size_t)l.row;
  for (const bool quad : {false, true}) {
    bl->mx_lds[quad] = (size_t)(quad ? l.quad : l.mx);
    if (bl->mx_lds[quad]) bl->mx_fn[quad] = pick_kernel_mx(k, beta, in, true, quad);
  }
  for (const auto &[other, need] : {std::pair{bl->row_fn, bl->row_lds}, std::pair{bl->mx_fn[0], bl->mx_lds[0]},
                                    std::pair{bl->mx_fn[1], bl->mx_lds[1]}}) {
    if (need <= 65536) continue;
    err = hipFuncSetAttribute(other, hipFuncAttributeMaxDynamicSharedMemorySize, (int)need);
    if (err != hipSuccess) return err;
  }
  return hipSuccess;
}

}  // namespace vit
