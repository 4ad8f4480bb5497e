// 3x3 stride-1 convolution of 64 to 64 channels on wide images, with the 2x2 stride-2 max-pool that alone reads it.
//
// VGG-16's second layer, 224 x 224: wider than a patch of consecutive pixels can be, so the tile kernel fetched every pixel nine
// times (388 us at batch 64), wrote 411 MB and the pooling launch read them back (87 us).  Here a workgroup of eight waves walks blocks of 16 x 16
// pixels: the patch under the next block comes into LDS by direct loads (pixels outside the image as zeros, so no tap is masked) while this
// one is multiplied, a wave holds the weights of 32 output channels as operands for life (six taps in registers, three in LDS), and the pool
// is taken between the lanes of the accumulators' layout, so that a quarter of the output leaves.  217 to 240 us for both launches (233 alone, 1.02 PFLOP/s).  Bound: a block takes
// 4.4 to 4.9 us, of which the matrix instructions need 1.9: the phases (addresses, multiply, pool) do not overlap, as the waves meet at every block.
// Tried: pooling the rounded values with shuffles 270 us; masks from divisions per load 222.
//
// The order of the sums is the tile kernel's (tap after tap, 16 channels per instruction), so are the bits.
#include <hip/hip_runtime.h>

#include "fi_device.h"
#include "fi_internal.h"

namespace fi {
namespace {

constexpr int PW = 18, PPIX = 18 * 18, PLOADS = (PPIX + 7) / 8;   // pixels of a patch: 16 x 16 and one on every side; load instructions for them
constexpr int PBYTES = PLOADS * 1024;
constexpr int REGS = 6;   // taps whose weights stay in registers (24 fragments of four); those of the others are read from LDS

__global__ void __launch_bounds__(512, 2) conv_pool_kernel(KArgs a) {
  // two patches, and the weights read from LDS: ONE array (with several, the compiler tells them apart and makes every operand read wait
  // for the direct loads into the other patch)
  constexpr int LATE = 2 * (9 - REGS) * 4096;
  __shared__ __attribute__((aligned(1024))) uint8_t smem[2 * PBYTES + LATE];
  int p, bid;
  if (!find_problem_at(a, xcd_contiguous((int)blockIdx.x, (int)gridDim.x), p, bid)) return;
  const Desc d = a.d[p];
  const int batch = a.batch[p];
  // d.H x d.W (= the convolution's output) in blocks of 16 x 16; the stored tensor is d.Ho x d.Wo
  const int bw = (d.W + 15) / 16, bh = (d.H + 15) / 16, T = batch * bh * bw, groups = a.first_block[p + 1] - a.first_block[p];
  const int t0 = (int)((int64_t)T * bid / groups), t1 = (int)((int64_t)T * (bid + 1) / groups);
  const int tid = threadIdx.x, lane = tid & 63, r31 = lane & 31, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wp = wave >> 1, wn = wave & 1;   // four rows of pixels, 32 of the channels
  const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(a.abase + d.x_off, 0, (int)((int64_t)batch * d.H * d.W * 128), 0x00020000);

  // the weights of this wave's 32 output channels, as operands: they stay
  bf16x8 w[REGS][4];
  uint8_t* const late = smem + 2 * PBYTES + wn * (9 - REGS) * 4096 + lane * 16;
  {
    const bf16_t* const wp0 = reinterpret_cast<const bf16_t*>(a.wbase + d.w_off) + (int64_t)(wn * 32 + r31) * d.Kp + half * 8;
#pragma unroll
    for (int tap = 0; tap < 9; ++tap)
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        const bf16x8 v = *reinterpret_cast<const bf16x8*>(wp0 + tap * 64 + kk * 16);
        if (tap < REGS) w[tap < REGS ? tap : 0][kk] = v;
        else if (wp == 0) *reinterpret_cast<bf16x8*>(late + ((tap - REGS) * 4 + kk) * 1024) = v;
      }
  }
  const bool g1 = (lane & 1) != 0, g2 = (lane & 16) != 0;   // the run of four channels that this lane finishes (below)
  const int run = wn * 32 + (g2 ? 16 : 0) + (g1 ? 8 : 0) + 4 * half;
  const float4 bias = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(a.wbase + d.b_off) + run);
  const Activation<false> act(d.act);

  // A load instruction brings 8 pixels of 128 bytes, lane l's 16 bytes to l * 16: the pieces of a pixel are permuted at the source
  // (piece ^ column / 2 % 8: the sixteen pixels of a row read from sixteen places of 16 bytes, all banks, and a tap's row is an offset).  Pixels outside the image, and past the patch, are written as zeros.
  const int lrow = lane >> 3;
  constexpr int NL = (PLOADS + 7) / 8;
  int rel[NL], at_yx[NL];   // this lane's piece of a load relative to the block's origin (bytes), and its row and column in the patch
#pragma unroll
  for (int u = 0; u < NL; ++u) {
    const int px = (wave + u * 8) * 8 + lrow, py = px / PW, col = px - py * PW;
    rel[u] = (((py - 1) * d.W + col - 1) * 64 + ((lane & 7) ^ ((col >> 1) & 7)) * 8) * 2;
    at_yx[u] = px < PPIX ? ((py - 1) & 0xFFFF) | ((col - 1) << 16) : 0x7FFF;   // (past the patch: a row below any image)
  }
  const int n0 = t0 / (bh * bw), r0 = t0 - n0 * bh * bw;
  int fn = n0, fy = r0 / bw * 16, fx = r0 % bw * 16, left = t1 - t0;   // the block to fetch: image, origin; blocks left
  auto fetch = [&](int buf) {
    const uint32_t origin = (uint32_t)(((fn * d.H + fy) * d.W + fx) * 128), dead = left > 0 ? 0u : OOB;
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      const int i = wave + u * 8;
      if (i >= PLOADS) break;
      const bool ok = (unsigned)(fy + (int16_t)at_yx[u]) < (unsigned)d.H && (unsigned)(fx + (at_yx[u] >> 16)) < (unsigned)d.W;
      load_lds<16>(xres, smem + buf * PBYTES + i * 1024, (ok ? origin + (uint32_t)rel[u] : OOB) | dead);
    }
    --left;
    fx += 16;
    if (fx >= d.W) { fx = 0; fy += 16; }
    if (fy >= d.H) { fy = 0; ++fn; }
  };
  if (t0 >= t1) return;
  fetch(0);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
  for (int tap = 0; tap < REGS; ++tap)   // (used here, so that the compiler's own wait for them stands before the loop and not in it)
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) asm volatile("" : "+v"(w[tap][kk]));

  const __amdgpu_buffer_rsrc_t yres = __builtin_amdgcn_make_buffer_rsrc(
      a.abase + d.y_off, 0, (int)((((int64_t)batch * d.Ho * d.Wo - 1) * d.ys + 64) * 2), 0x00020000);
  // operand addresses of the first row of pixels for the three columns of taps; rows are constant offsets
  int at[3][4];
#pragma unroll
  for (int ks = 0; ks < 3; ++ks)
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const int col = (r31 & 15) + ks;
      at[ks][kk] = ((wp * 4 + (r31 >> 4)) * PW + col) * 128 + (((2 * kk + half) ^ ((col >> 1) & 7)) << 4);
    }
  int n = n0, by = r0 / bw * 8, bx = r0 % bw * 8, buf = 0;
  for (int t = t0; t < t1; ++t, buf ^= 1) {
    // this wave's share of the patch is in LDS (the two stores of the block before may still be on their way), and it has read the other
    // buffer to the end; behind the barrier that holds for all eight
    asm volatile("s_waitcnt vmcnt(2) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    fetch(buf ^ 1);
    asm volatile("" ::: "memory");   // (the count above holds if the block's two stores come behind)
    __builtin_amdgcn_sched_barrier(0);
    f32x16 acc[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][e] = 0.0f;
    const uint8_t* const P = smem + buf * PBYTES;
#pragma unroll
    for (int tap = 0; tap < 9; ++tap)
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        const bf16x8 wf = tap < REGS ? w[tap < REGS ? tap : 0][kk] : *reinterpret_cast<const bf16x8*>(late + ((tap - REGS) * 4 + kk) * 1024);
        bf16x8 af[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) af[i] = *reinterpret_cast<const bf16x8*>(P + at[tap % 3][kk] + (2 * i + tap / 3) * PW * 128);
#pragma unroll
        for (int i = 0; i < 2; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf, af[i], acc[i], 0, 0, 0);
      }
    // A lane holds, for pixel (row r31 / 16, column r31 % 16), four runs of four consecutive channels; the pixels of a 2 x 2 window are the
    // lanes that differ in bits 0 and 4.  The maximum is taken of the bare sums (adding the bias, identity / ReLU / ReLU6 and the rounding keep
    // the order), then each of the window's lanes finishes and stores one run.
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const float q = acc[i][e];
        const float v = fmaxf(q, __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(q), 0xB1, 0xF, 0xF, true)));   // (lane ^ 1)
        const auto rows = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);         // (lane ^ 16)
        acc[i][e] = fmaxf(__uint_as_float(rows[0]), __uint_as_float(rows[1]));
      }
      const float b4[4] = {bias.x, bias.y, bias.z, bias.w};
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float lo = g1 ? acc[i][4 + e] : acc[i][e], hi = g1 ? acc[i][12 + e] : acc[i][8 + e];
        v[e] = (g2 ? hi : lo) + b4[e];
      }
      act.apply(v);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = fmaxf(v[e], -INFINITY);   // (a window of NaN: as in the pooling kernel)
      const u32x2 out = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
      const int y = by + wp * 2 + i, x = bx + ((lane & 15) >> 1);   // (of the pooled image)
      const uint32_t off = y < d.Ho && x < d.Wo ? (uint32_t)((((n * d.Ho + y) * d.Wo + x) * d.ys + run) * 2) : OOB;
      __builtin_amdgcn_raw_buffer_store_b64(out, yres, off, 0, 0);
    }
    bx += 8;
    if (2 * bx >= d.W) { bx = 0; by += 8; }
    if (2 * by >= d.H) { by = 0; ++n; }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (the fetch after the last block writes zeros: not into another workgroup's LDS)
}

}  // namespace

int launch_pool(const Launch& L, const KArgs& args, void* stream, const std::vector<Desc>& hd) {
  if (L.n < 1 || L.n > FI_MAX_GROUP || L.wdtype != FI_BF16 || L.adtype != FI_BF16) return (int)hipErrorInvalidValue;
  KArgs a = args;
  int64_t blocks = 0, share[FI_MAX_GROUP], groups[FI_MAX_GROUP];
  for (int i = 0; i < L.n; ++i) {
    const Desc& t = hd[(size_t)(L.first_desc + i)];
    a.d[i] = t;
    const int64_t b = a.batch[i];
    if (b < 0 || t.Cp != 64 || t.xs != 64 || t.Co != 64 || t.Cop != 64 || t.k != 3 || t.kw != 3 || t.stride != 1 || t.pad != 1 || t.pad_w != 1 || t.Kp != 576 || t.ext ||
        t.out_f32 || t.r_off != kNone || t.act > FI_ACT_RELU6 || t.Ho != t.H / 2 || t.Wo != t.W / 2 || t.Ho < 1 || t.Wo < 1 || t.ys % 4 ||
        b * t.H * t.W * 128 >= (1ll << 31) || b * t.Ho * t.Wo * t.ys * 2 >= (1ll << 31))
      return (int)hipErrorInvalidValue;
    share[i] = b * ((t.H + 15) / 16) * ((t.W + 15) / 16);
  }
  share_workgroups(share, share, L.n, 256, groups);
  for (int i = 0; i < L.n; ++i) {
    a.first_block[i] = (int32_t)blocks;
    blocks += groups[i];
  }
  if (blocks == 0) return (int)hipSuccess;
  for (int i = L.n; i <= FI_MAX_GROUP; ++i) a.first_block[i] = (int32_t)blocks;
  hipLaunchKernelGGL(conv_pool_kernel, dim3((unsigned)blocks), dim3(512), 0, static_cast<hipStream_t>(stream), a);
  return (int)hipGetLastError();
}

}  // namespace fi
