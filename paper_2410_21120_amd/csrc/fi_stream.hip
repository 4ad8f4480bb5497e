// Pointwise convolutions of many rows and a short reduction: rows stream through waves that never meet.
//
// Such a layer is bound by HBM: each row is read once, each output row written once, and the weights (at most 128 columns x 384
// elements) stay on chip.  The tile kernel of fi_kernels.hip gives a workgroup one 128-row tile, whose life is a prologue, one to
// six reduction tiles with two barriers each and one tile of loads in flight, and an epilogue: 2.0 to 3.4 TB/s.  Here eight waves share
// the weights in LDS (one workgroup per compute unit, loaded once) and each takes blocks of 32 rows on its own: a lane loads
// the 16-byte pieces that the matrix instruction wants of it straight into registers, the whole next block requested piece by piece
// while this one is multiplied (up to 128 KB in flight per compute unit), no barrier after the start.  The end of a block breaks into that: loads return
// in order, so the loads of a residual (fp32 rows make them without one too, out of range) wait for the next block's rows, one after the other; and
// as a store is one of two kinds by a branch, the first multiply of a block waits for its rows as if no store had been issued behind them.  Outputs turn through a 4 KB patch of the wave's own, so
// that whole cache lines leave: 16-byte pieces straight from the accumulators' layout, 32 bytes of a row at a time, written past the
// cache cost 166 us where the tile took 69 (112 x 112, fp32 rows, 16 -> 64 channels).
//
// Measured alone, tile kernel -> this one (us): DenseNet-121, four members at batch 32, 56 x 56, affine and ReLU on the way in, 64 / 128 /
// 192 / 256 -> 128 channels 54 / 67 / 79 / 103 -> 32 / 42 / 53 / 79 (3.9 to 4.9 TB/s; a copy reaches 5.2); MobileNetV3-Large, fp32 rows,
// two members at batch 32, 112 x 112, 16 -> 16 60 -> 29, 16 -> 64 64 -> 46, 56 x 56, 24 -> 72 36 -> 27.
// Wider outputs would read every row once per 128 columns, at different times: 256 -> 256 channels, 56 x 56, 69.6 -> 124.6 us, so they keep the tile.
//
// The order of the sums (ascending channels, 16 per instruction, from zero; for fp32 rows the small halves first) and the epilogue's operations are the
// tile kernel's, so the bits are the same whichever kernel a launch takes.
#include <hip/hip_runtime.h>

#include "fi_device.h"
#include "fi_internal.h"

namespace fi {
namespace {

constexpr int SW = STREAM_WAVES;

// max(x * scale + shift, 0) of eight channels: product and sum rounded separately, one rounding to bf16 (the depthwise kernel's operations).
__device__ __forceinline__ bf16x8 affine_relu(u32x4 x, const u32x4 (&scale)[2], const u32x4 (&shift)[2]) {
  u32x4 h;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float s0 = __uint_as_float(scale[e >> 1][(2 * e) & 3]), s1 = __uint_as_float(scale[e >> 1][(2 * e + 1) & 3]);
    const float b0 = __uint_as_float(shift[e >> 1][(2 * e) & 3]), b1 = __uint_as_float(shift[e >> 1][(2 * e + 1) & 3]);
    h[e] = pack_bf16x2(fmaxf(__fadd_rn(__fmul_rn(__uint_as_float(x[e] << 16), s0), b0), 0.0f),
                       fmaxf(__fadd_rn(__fmul_rn(__uint_as_float(x[e] & 0xFFFF0000u), s1), b1), 0.0f));
  }
  return __builtin_bit_cast(bf16x8, h);
}

// Whether the output is written past the cache: from the tile kernel's size on, which counts two bytes an element for fp32 rows as well (52 MB
// of them, 4 x 160 x 160 x 128, made the mean behind them take 400 us where it takes 256), and only rows that are whole lines of 128 bytes. Of the others
// every line leaves in pieces: 40 -> 120 channels, bf16, 16384 blocks of 32 rows 65 us past the cache, 35 through it (43 on the tile), 32768 blocks of
// fp32 rows, 96 -> 40 179 and 127 (121), 24 -> 72 183 and 93 (123).
__device__ __forceinline__ bool past_the_cache(const Desc& d, int M, int es) {
  return (int64_t)M * d.Cop * 2 > (int64_t)STREAM_OUT_BYTES && (((uint64_t)d.Cop * es | (uint64_t)d.ys * es | d.y_off) & 127) == 0;
}

// A lane holds, for pixel (lane & 31) of 32, runs of four consecutive channels: bias, residual, activation, the one rounding.  A bf16 line of the patch
// is two blocks of columns: with an odd NB the half of the last one that nothing wrote is not stored, as there Cop <= n0 + NB * 32.
template <bool WIDE, int NB>
__device__ __forceinline__ void finish_rows(const Desc& d, const f32x16 (&acc)[NB], int row0, int n0, int lane, const float* bias, uint8_t* patch, const Activation<false>& act,
                                            const __amdgpu_buffer_rsrc_t rres, bool has_res, const __amdgpu_buffer_rsrc_t yres, bool stream_out) {
  constexpr int AE = WIDE ? 4 : 2;
  const int r31 = lane & 31, half = lane >> 5, lrow = lane >> 3, bsw = (r31 >> 1) & 7;
  const bool hardswish = d.act == FI_ACT_HARDSWISH;
  const int m = row0 + r31;
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    float v[16];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int cl = j * 32 + 8 * g + 4 * half;
      const float4 b = *reinterpret_cast<const float4*>(bias + cl);
      v[4 * g] = acc[j][4 * g] + b.x; v[4 * g + 1] = acc[j][4 * g + 1] + b.y; v[4 * g + 2] = acc[j][4 * g + 2] + b.z; v[4 * g + 3] = acc[j][4 * g + 3] + b.w;
    }
    if (WIDE || has_res) {   // (fp32 rows: no residual adds +0.0, as on the tiles)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int c = n0 + j * 32 + 8 * g + 4 * half;
        const uint32_t off = c < d.Cop ? (uint32_t)((m * d.Cop + c) * AE) : OOB;
        if constexpr (WIDE) {
          const u32x4 r = __builtin_amdgcn_raw_buffer_load_b128(rres, off, 0, 0);
#pragma unroll
          for (int e = 0; e < 4; ++e) v[4 * g + e] += __uint_as_float(r[e]);
        } else {
          const u32x2 r = __builtin_amdgcn_raw_buffer_load_b64(rres, off, 0, 0);
#pragma unroll
          for (int e = 0; e < 4; ++e) v[4 * g + e] += __uint_as_float((e & 1) ? r[e >> 1] & 0xFFFF0000u : r[e >> 1] << 16);
        }
      }
    }
    if (hardswish) {
#pragma unroll
      for (int e = 0; e < 16; ++e) v[e] = act_hardswish(v[e]);
    } else {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float q[4] = {v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
        act.apply(q);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[4 * g + e] = q[e];
      }
    }
    // Through a patch of the wave's own (32 rows of 128 bytes), so that whole cache lines leave.
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      if constexpr (WIDE) {
        *reinterpret_cast<float4*>(patch + r31 * 128 + (((2 * g + half) ^ bsw) << 4)) = make_float4(v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]);
      } else {
        const u32x2 pk = {pack_bf16x2(v[4 * g], v[4 * g + 1]), pack_bf16x2(v[4 * g + 2], v[4 * g + 3])};
        *reinterpret_cast<u32x2*>(patch + r31 * 128 + ((((j & 1) * 4 + g) ^ bsw) << 4) + 8 * half) = pk;
      }
    }
    if (!WIDE && (j & 1) == 0 && j + 1 < NB) continue;   // (bf16: two blocks of columns make a line)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");   // the wave's own LDS writes precede its reads
    const int c = n0 + (WIDE ? j * 32 + (lane & 7) * 4 : j / 2 * 64 + (lane & 7) * 8);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = i * 8 + lrow;
      const u32x4 o = *reinterpret_cast<const u32x4*>(patch + r * 128 + (((lane & 7) ^ ((r >> 1) & 7)) << 4));
      const uint32_t off = c < d.Cop ? (uint32_t)(((row0 + r) * d.ys + c) * AE) : OOB;
      if (stream_out) __builtin_amdgcn_raw_buffer_store_b128(o, yres, off, 0, 2);
      else __builtin_amdgcn_raw_buffer_store_b128(o, yres, off, 0, 0);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

// WIDE: fp32-stored activations, multiplied as hi + lo bf16 halves.  PRE: 1 = per-channel affine and ReLU on the way in.
// PRE 2 (not a pointwise convolution): 3x3 over the four-channel staged input, the first layer of the mobile families.  A row's 36 elements
// are gathered tap by tap (8 or 16 bytes) from the pixels around it, which neighbouring rows share in the vector cache.  MobileNetV3-Large, fp32
// rows, 112 x 112 x 16, two members at batch 32: 80 us on the tile kernel, 37 here.
// NB: 32-column blocks of a workgroup's weights.  NCH: 128-byte pieces of a row (64 bf16 or 32 fp32 elements).
template <bool WIDE, int PRE, int NB, int NCH>
__global__ void __launch_bounds__(SW * 64, 2) conv_stream_kernel(KArgs a) {
  constexpr int AE = WIDE ? 4 : 2, CE = 128 / AE;   // elements of a piece
  constexpr int ST = CE / 16;                       // 16-element steps of a piece
  constexpr int V = WIDE ? 2 : 1;                   // 16-byte vectors per lane and step
  constexpr int BN = NB * 32;
  constexpr int KW = (NCH * CE + 63) / 64;          // 64-element pieces of a weight row
  constexpr int W_BYTES = KW * BN * 128, KP = KW * 64;
  __shared__ __attribute__((aligned(1024))) uint8_t smem[W_BYTES + SW * 4096 + BN * 4 + (PRE == 1 ? KP * 8 : 0)];
  static_assert(sizeof(smem) <= 160 * 1024, "LDS of a compute unit");
  float* const bias_s = reinterpret_cast<float*>(smem + W_BYTES + SW * 4096);
  float* const shift_s = bias_s + BN;
  float* const scale_s = shift_s + KP;

  int p, bid;
  if (!find_problem_at(a, xcd_contiguous((int)blockIdx.x, (int)gridDim.x), p, bid)) return;
  const Desc d = a.d[p];
  const int batch = a.batch[p];
  const int M = batch * d.Ho * d.Wo, T = (M + 31) >> 5;
  const int groups = a.first_block[p + 1] - a.first_block[p];
  const int t0 = (int)((int64_t)T * bid / groups), t1 = (int)((int64_t)T * (bid + 1) / groups);   // this workgroup's blocks of 32 rows
  const int tid = threadIdx.x, lane = tid & 63, r31 = lane & 31, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(
      a.abase + d.x_off, 0, M > 0 ? (int)((PRE == 2 ? (int64_t)batch * d.H * d.W * 4 : ((int64_t)M - 1) * d.xs + d.Cp) * AE) : 0, 0x00020000);
  const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(a.wbase + d.w_off), 0, (int)((int64_t)d.Co * d.Kp * 2), 0x00020000);

  u32x4 av[NCH][ST][V];   // a block of rows, requested one block ahead
  int t = t0 + wave;
  uint32_t row = (uint32_t)((t * 32 + r31) * d.xs * AE + half * 8 * AE);
  // PRE 2: where the block of rows to request has its windows (the first tap's row, column and byte offset)
  int ih0 = 0, iw0 = 0;
  auto window = [&](int block) {
    const int m = block * 32 + r31, mm = m < M ? m : 0;
    const int q1 = fast_div(mm, d.Wo, 1.0f / (float)d.Wo), n = fast_div(q1, d.Ho, 1.0f / (float)d.Ho);
    ih0 = m < M ? (q1 - n * d.Ho) * d.stride - d.pad : -(1 << 20);   // (rows past M read as zero)
    iw0 = (mm - q1 * d.Wo) * d.stride - d.pad_w;
    row = (uint32_t)(((n * d.H + ih0) * d.W + iw0) * 4 * AE);
  };
  if constexpr (PRE == 2) window(t);
  auto request = [&](int c, uint32_t at) {
    if constexpr (PRE == 2) {
#pragma unroll
      for (int s = 0; s < ST; ++s)
#pragma unroll
        for (int v = 0; v < 2; ++v) {   // this lane's two taps of the step: 4 (c ST + s) + 2 half + v
          const int tap0 = 4 * (c * ST + s) + v, tap1 = tap0 + 2;
          const int r = half ? tap1 / 3 : tap0 / 3, q = half ? tap1 % 3 : tap0 % 3;
          const bool ok = r < 3 && (unsigned)(ih0 + r) < (unsigned)d.H && (unsigned)(iw0 + q) < (unsigned)d.W;
          const uint32_t off = ok ? (row + (uint32_t)((r * d.W + q) * 4 * AE)) | (at & OOB) : OOB;
          if constexpr (WIDE) {
            av[c][s][v % V] = __builtin_amdgcn_raw_buffer_load_b128(xres, off, 0, 0);
          } else {
            const u32x2 px = __builtin_amdgcn_raw_buffer_load_b64(xres, off, 0, 0);
            av[c][s][0][2 * v] = px[0];
            av[c][s][0][2 * v + 1] = px[1];
          }
        }
      return;
    }
#pragma unroll
    for (int s = 0; s < ST; ++s) {
      const uint32_t off = c * CE + s * 16 + half * 8 < d.Cp ? at + (uint32_t)((c * CE + s * 16) * AE) : OOB;
#pragma unroll
      for (int v = 0; v < V; ++v) av[c][s][v] = __builtin_amdgcn_raw_buffer_load_b128(xres, off + 16 * v, 0, 0);
    }
  };

  // weights: 8 rows of 128 bytes per instruction, the 16-byte pieces of a row permuted at the source (piece ^ row / 2 % 8: sixteen rows read from
  // sixteen places of 16 bytes, all banks)
  const int lrow = lane >> 3;
  for (int i = wave; i < KW * (BN / 8); i += SW) {
    const int kc = i / (BN / 8), r = i % (BN / 8) * 8 + lrow;
    const int k = kc * 64 + ((lane & 7) ^ ((r >> 1) & 7)) * 8;
    load_lds<16>(wres, smem + i * 1024, k < d.Kp ? (uint32_t)(r * d.Kp + k) * 2 : OOB);   // (rows past Co lie past the buffer's end)
  }
  for (int i = tid; i < BN; i += SW * 64) bias_s[i] = i < d.Cop ? reinterpret_cast<const float*>(a.wbase + d.b_off)[i] : 0.0f;
  if constexpr (PRE == 1)
    for (int i = tid; i < KP; i += SW * 64) {
      scale_s[i] = i < d.Cp ? bf2f(reinterpret_cast<const bf16_t*>(a.wbase + d.pw_off)[i]) : 0.0f;
      shift_s[i] = i < d.Cp ? reinterpret_cast<const float*>(a.wbase + d.pb_off)[i] : 0.0f;
    }
  {
    const uint32_t live = t < t1 ? PRE == 2 ? 0u : row : OOB;
#pragma unroll
    for (int c = 0; c < NCH; ++c) request(c, live);
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  __syncthreads();

  const bool has_res = d.r_off != kNone, stream_out = past_the_cache(d, M, AE);
  const __amdgpu_buffer_rsrc_t rres = __builtin_amdgcn_make_buffer_rsrc(
      a.abase + (has_res ? d.r_off : 0), 0, has_res ? (int)((int64_t)M * d.Cop * AE) : 0, 0x00020000);
  const __amdgpu_buffer_rsrc_t yres = __builtin_amdgcn_make_buffer_rsrc(
      a.abase + d.y_off, 0, M > 0 ? (int)((((int64_t)M - 1) * d.ys + d.Cop) * AE) : 0, 0x00020000);
  const uint32_t next = (uint32_t)(SW * 32) * (uint32_t)d.xs * AE;
  const int bsw = (r31 >> 1) & 7;
  uint8_t* const patch = smem + W_BYTES + wave * 4096;
  const Activation<false> act(d.act);
  constexpr bool RESIDENT = !PRE && NCH * ST * NB * 4 <= 32;   // a weight fragment is 4 registers: few of them stay there for the life of the workgroup
  int fresh = 0;
  for (; t < t1; t += SW) {
    if constexpr (!RESIDENT) asm volatile("" : "+v"(fresh));   // (zero: keeps the reads of weights, bias and scale in the loop, where there are registers for them)
    f32x16 acc[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[j][e] = 0.0f;
    if constexpr (PRE == 2) window(t + SW);
    else row += next;
    const uint32_t live = t + SW < t1 ? PRE == 2 ? 0u : row : OOB;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
#pragma unroll
      for (int s = 0; s < ST; ++s) {
        const int k = c * CE + s * 16;   // (this lane: elements k + 8 half .. + 7)
        bf16x8 hi, lo;
        if constexpr (WIDE) {
          u32x4 h, l;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float x0 = __uint_as_float(av[c][s][e >> 1][(2 * e) & 3]), x1 = __uint_as_float(av[c][s][e >> 1][(2 * e + 1) & 3]);
            const uint32_t h0 = f2bf(x0), h1 = f2bf(x1);
            h[e] = h0 | (h1 << 16);
            l[e] = pack_bf16x2(x0 - __uint_as_float(h0 << 16), x1 - __uint_as_float(h1 << 16));
          }
          hi = __builtin_bit_cast(bf16x8, h);
          lo = __builtin_bit_cast(bf16x8, l);
        } else if constexpr (PRE == 1) {
          const u32x4* const sc = reinterpret_cast<const u32x4*>(scale_s + k + 8 * half + fresh);
          const u32x4* const sh = reinterpret_cast<const u32x4*>(shift_s + k + 8 * half + fresh);
          const u32x4 scale[2] = {sc[0], sc[1]}, shift[2] = {sh[0], sh[1]};
          hi = affine_relu(av[c][s][0], scale, shift);
        } else {
          hi = __builtin_bit_cast(bf16x8, av[c][s][0]);
        }
        const uint8_t* const W = smem + (k >> 6) * (BN * 128) + r31 * 128 + fresh + ((((k & 63) / 8 + half) ^ bsw) << 4);
        bf16x8 bfr[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j) bfr[j] = *reinterpret_cast<const bf16x8*>(W + j * 32 * 128);
        if constexpr (WIDE)   // small terms first
#pragma unroll
          for (int j = 0; j < NB; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[j], lo, acc[j], 0, 0, 0);
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[j], hi, acc[j], 0, 0, 0);
      }
      request(c, live);   // the same piece of the next block
      __builtin_amdgcn_sched_barrier(0);
    }
    finish_rows<WIDE, NB>(d, acc, t * 32, 0, lane, bias_s + fresh, patch, act, rres, has_res, yres, stream_out);
  }
}

// The same, for rows of any length behind an affine stage with ReLU (DenseNet's layers beyond 384 channels, or of too few rows to pay for resident
// weights): four waves, a block of 32 rows each, the weights of 64 channels at a time through a ring of three stages in LDS (one barrier per
// 64 channels), the rows four pieces ahead in registers (three for the first of every four: a row may end after
// any piece, so the compiler's wait there counts as if the piece before had been the last), scale and shift as tables in LDS, read before the barrier.  A piece
// takes 0.9 us, that wait included, for 32 KB from L2.  DenseNet-121, four members at batch 32, 14 x 14, 288 / 480 / 672 / 960 -> 128 channels: 19.1 / 23.8 / 27.2 / 33.3 us on the
// 128x64 tile, 16.0 / 19.2 / 20.8 / 25.4 here.
constexpr int LW = LONG_WAVES, LK = LONG_K;   // (the tables of the longest row leave room for two workgroups per compute unit)

__global__ void __launch_bounds__(LW * 64, 2) conv_long_kernel(KArgs a) {
  constexpr int NB = 4, BN = 128, NS = 3, STAGE = BN * 128, D = 4;   // columns; stages of the weights' ring; pieces of a row in registers
  constexpr int AT_PATCH = NS * STAGE, AT_BIAS = AT_PATCH + LW * 4096, AT_SHIFT = AT_BIAS + BN * 4, AT_SCALE = AT_SHIFT + LK * 4;
  __shared__ __attribute__((aligned(1024))) uint8_t smem[AT_SCALE + LK * 4];   // (one array: operand reads must not wait for the direct loads)
  static_assert(sizeof(smem) <= 80 * 1024, "two workgroups per compute unit");
  float* const bias_s = reinterpret_cast<float*>(smem + AT_BIAS);
  float* const shift_s = reinterpret_cast<float*>(smem + AT_SHIFT);
  float* const scale_s = reinterpret_cast<float*>(smem + AT_SCALE);

  int p, bid;
  if (!find_problem_at(a, xcd_contiguous((int)blockIdx.x, (int)gridDim.x), p, bid)) return;
  const Desc d = a.d[p];
  const int M = a.batch[p] * d.Ho * d.Wo, slabs = (d.Cop + BN - 1) / BN;
  const int tid = threadIdx.x, lane = tid & 63, r31 = lane & 31, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n0 = bid % slabs * BN, row0 = bid / slabs * (LW * 32) + wave * 32;
  const int pieces = (d.Cp + 63) >> 6;
  const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(
      a.abase + d.x_off, 0, M > 0 ? (int)((((int64_t)M - 1) * d.xs + d.Cp) * 2) : 0, 0x00020000);
  const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(a.wbase + d.w_off), 0, (int)((int64_t)d.Co * d.Kp * 2), 0x00020000);

  for (int i = tid; i < pieces * 64; i += LW * 64) {
    scale_s[i] = i < d.Cp ? bf2f(reinterpret_cast<const bf16_t*>(a.wbase + d.pw_off)[i]) : 0.0f;
    shift_s[i] = i < d.Cp ? reinterpret_cast<const float*>(a.wbase + d.pb_off)[i] : 0.0f;
  }
  if (tid < BN) bias_s[tid] = n0 + tid < d.Cop ? reinterpret_cast<const float*>(a.wbase + d.b_off)[n0 + tid] : 0.0f;

  u32x4 av[D][4];
  const uint32_t row = (uint32_t)((row0 + r31) * d.xs + half * 8) * 2;   // (rows past M lie past the buffer's end)
  auto request = [&](int u, int c) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
      av[u][s] = __builtin_amdgcn_raw_buffer_load_b128(xres, c * 64 + s * 16 + half * 8 < d.Cp ? row + (uint32_t)(c * 128 + s * 32) : OOB, 0, 0);
  };
  // weights: 8 rows of 128 bytes per instruction, pieces of 16 bytes permuted at the source (piece ^ row / 2 % 8)
  const int lrow = lane >> 3, piece = (lane & 7) ^ ((4 * wave + (lrow >> 1)) & 7);
  const uint32_t w_row = (uint32_t)((n0 + wave * 8 + lrow) * d.Kp + piece * 8) * 2, w_step = (uint32_t)(LW * 8) * (uint32_t)d.Kp * 2;   // (rows past Co: past the end)
  auto weights = [&](int c, int stage) {
    const uint32_t dead = c * 64 + piece * 8 < d.Kp ? 0u : OOB;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      load_lds<16>(wres, smem + stage * STAGE + (wave + LW * i) * 1024, (w_row + w_step * i + (uint32_t)(c * 128)) | dead);
  };
  // The loop's count of outstanding loads holds if the weights stand before the rows, and its waits are short if the rows come piece by piece: the
  // compiler must not mix them (with the pieces mixed, 4x DenseNet-121 at batch 32 2613 -> 2628 us).
  weights(0, 0);
  weights(1, 1);
#pragma unroll
  for (int u = 0; u < D; ++u) {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    request(u, u);
  }

  f32x16 acc[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[j][e] = 0.0f;
  const int bsw = (r31 >> 1) & 7;
  int stage = 0;
  for (int c0 = 0; c0 < pieces; c0 += D) {
#pragma unroll
    for (int u = 0; u < D; ++u) {
      const int c = c0 + u;
      if (c >= pieces) break;
      u32x4 scale[4][2], shift[4][2];   // (native vectors: of a float4 the compiler believes that it may be what a direct load brings, and waits for all of them)
      if (c == 0) __syncthreads();   // (the tables are complete)
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          scale[s][h] = *reinterpret_cast<const u32x4*>(smem + AT_SCALE + (c * 64 + s * 16 + 8 * half + 4 * h) * 4);
          shift[s][h] = *reinterpret_cast<const u32x4*>(smem + AT_SHIFT + (c * 64 + s * 16 + 8 * half + 4 * h) * 4);
        }
      // this wave's share of the piece's weights is in LDS (requested behind them: at least two pieces of rows and one of weights; past the last
      // piece the requests are out of range, so that they are always as many), and it has read the stage before to the end
      asm volatile("s_waitcnt vmcnt(12) lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      const int into = stage == 0 ? NS - 1 : stage - 1;   // the stage that the piece before had
      weights(c + 2, into);
      __builtin_amdgcn_sched_barrier(0);
      const uint8_t* const S = smem + stage * STAGE + r31 * 128;
      stage = stage == NS - 1 ? 0 : stage + 1;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const bf16x8 x = affine_relu(av[u][s], scale[s], shift[s]);
#pragma unroll
        for (int j = 0; j < NB; ++j)
          acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(S + j * 4096 + (((2 * s + half) ^ bsw) << 4)), x, acc[j], 0, 0, 0);
      }
      request(u, c + D);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (nothing lands in LDS any more)
  const bool has_res = d.r_off != kNone, stream_out = past_the_cache(d, M, 2);
  const __amdgpu_buffer_rsrc_t rres = __builtin_amdgcn_make_buffer_rsrc(
      a.abase + (has_res ? d.r_off : 0), 0, has_res ? (int)((int64_t)M * d.Cop * 2) : 0, 0x00020000);
  const __amdgpu_buffer_rsrc_t yres = __builtin_amdgcn_make_buffer_rsrc(
      a.abase + d.y_off, 0, M > 0 ? (int)((((int64_t)M - 1) * d.ys + d.Cop) * 2) : 0, 0x00020000);
  finish_rows<false, NB>(d, acc, row0, n0, lane, bias_s, smem + AT_PATCH + wave * 4096, Activation<false>(d.act), rres, has_res, yres, stream_out);
}

template <bool WIDE, int PRE, int NB, int NCH>
int go_stream(int blocks, const KArgs& a, hipStream_t s) {
  if (blocks <= 0) return (int)hipSuccess;
  hipLaunchKernelGGL((conv_stream_kernel<WIDE, PRE, NB, NCH>), dim3((unsigned)blocks), dim3(SW * 64), 0, s, a);
  return (int)hipGetLastError();
}

}  // namespace

int launch_long(const Launch& L, const KArgs& args, void* stream) {
  KArgs a = args;
  int64_t blocks = 0;
  for (int i = 0; i < L.n; ++i) {
    a.first_block[i] = (int32_t)blocks;
    blocks += ((int64_t)a.batch[i] * a.d[i].Ho * a.d[i].Wo + LW * 32 - 1) / (LW * 32) * ((a.d[i].Cop + 127) / 128);
  }
  for (int i = L.n; i <= FI_MAX_GROUP; ++i) a.first_block[i] = (int32_t)blocks;
  if (blocks <= 0) return (int)hipSuccess;
  hipLaunchKernelGGL(conv_long_kernel, dim3((unsigned)blocks), dim3(LW * 64), 0, static_cast<hipStream_t>(stream), a);
  return (int)hipGetLastError();
}

int launch_stream(const Launch& L, const KArgs& args, int nb, int nch, void* stream) {
  KArgs a = args;
  hipStream_t s = static_cast<hipStream_t>(stream);
  int64_t blocks = 0, rows[FI_MAX_GROUP], most[FI_MAX_GROUP], groups[FI_MAX_GROUP];
  for (int i = 0; i < L.n; ++i) {
    rows[i] = ((int64_t)a.batch[i] * a.d[i].Ho * a.d[i].Wo + 31) / 32;
    most[i] = (rows[i] + SW - 1) / SW;
  }
  share_workgroups(rows, most, L.n, 256, groups);
  for (int i = 0; i < L.n; ++i) {
    if (a.d[i].Cop > nb * 32) return (int)hipErrorInvalidValue;   // (a workgroup holds the weights of all columns)
    a.first_block[i] = (int32_t)blocks;
    blocks += groups[i];
  }
  for (int i = L.n; i <= FI_MAX_GROUP; ++i) a.first_block[i] = (int32_t)blocks;
  const int n = (int)blocks;
  const bool wide = L.adtype != FI_BF16;
  const int pre = a.d[0].Cp == 4 ? 2 : a.d[0].pre_kind;
#define FI_TAKE(WIDE, PRE, NB, NCH) if (wide == (WIDE) && pre == (PRE) && nb == (NB) && nch == (NCH)) return go_stream<WIDE, PRE, NB, NCH>(n, a, s);
  FI_STREAM_FORMS(FI_TAKE)
#undef FI_TAKE
  return (int)hipErrorInvalidValue;
}

}  // namespace fi
