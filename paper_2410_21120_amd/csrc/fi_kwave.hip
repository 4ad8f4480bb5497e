// Implicit-GEMM convolution / FC whose waves share the reduction instead of the tile.
//
// The tile kernel of fi_kernels.hip gives its four waves a quarter of the tile each and walks the reduction with two
// workgroup barriers per 64 elements, one tile of loads in flight.  A problem of few tiles and a long reduction (one
// workgroup per compute unit) then runs at one memory latency per step, whatever the arithmetic.  Here every wave owns
// the WHOLE tile and every NW-th step of the reduction: it has LDS buffers of its own, so the loop has no barrier, the
// waves' loads are in flight side by side (NW steps at a time), and the NW partial sums meet in LDS at the end, in wave
// order, where bias, residual, activation and rounding follow.  No partial sum leaves the workgroup and no second
// launch adds them up.
//
// A step is 128 bytes of a row (64 bf16 or 32 fp32 elements).  Rows come into LDS by direct global -> LDS loads (no
// staging registers, no LDS-write instructions): eight lanes fetch one row's 128 contiguous bytes, and lane l's 16
// bytes land at l * 16, so the 16-byte pieces of a row are permuted at the source (piece ^ row % 8), which spreads the
// operand reads (32 rows, one piece each) over the banks (0.42 conflict cycles per active LDS cycle are left on DenseNet-121's
// layers).  Out-of-range offsets write zeros: that is the padding, the rows past M, the channels past Co and the
// reduction's tail.
//
// fp32 models multiply with v_mfma_f32_32x32x2_f32 (fp32 products, fp32 sums): a 16-byte piece is four reduction
// elements of both operands, multiplied in four instructions.  Bound: the fp32 matrix rate (157 TFLOP/s, a sixteenth of
// bf16), which asks so little of LDS and L1 that a wave may own a whole 64 x 64 tile.  Measured, ResNet-18 in fp32 at
// batch 4: the 56 x 56 x 64 3x3 layers 20 us each (46 TFLOP/s), the pass 18.2 ms -> 0.40 ms against one thread per
// output element, whose serial sums also gave way to four or eight shorter ones (closer to the exact value).
//
// bf16 problems take eight waves and tiles of 32 x 32, or of 64 x 64 (128 KB of LDS, one workgroup per compute unit) where a launch
// fills the chip: half the operand bytes per product.  The eight partial sums of an element are the same ones in either
// tile.  512 -> 512, 3x3, 7 x 7, batch 16, eight members: 87.5 -> 70.8 us.
#include <hip/hip_runtime.h>

#include "fi_device.h"
#include "fi_internal.h"

namespace fi {

// Finishes four consecutive channels [o, o + 4) of an fp32 output pixel m from their sums.
__device__ __forceinline__ void finish_f32(const KArgs& a, const Desc& d, int p, int m, int o, float4 sum) {
  if (__builtin_expect(__builtin_isnan((sum.x + sum.y) + (sum.z + sum.w)) && (d.pad | d.pad_w) != 0, 0)) {
    // A tap outside the image reads zero here, and zero times a weight that is not finite is no zero: such a sum is
    // taken again over the taps inside the image only.
    int again_p = p;
    asm volatile("" : "+s"(again_p));   // (the descriptor is read again: its fields take no registers before)
    const Desc& e = a.d[again_p];
    const int g = m / e.Wo, n = g / e.Ho;
#pragma unroll 1
    for (int t = 0; t < 4; ++t) {
      const float v = t == 0 ? sum.x : t == 1 ? sum.y : t == 2 ? sum.z : sum.w;
      if (!__builtin_isnan(v) || o + t >= e.Co) continue;
      const float again = conv_element<true>(a, e, n, g - n * e.Ho, m - g * e.Wo, o + t);
      sum.x = t == 0 ? again : sum.x; sum.y = t == 1 ? again : sum.y; sum.z = t == 2 ? again : sum.z; sum.w = t == 3 ? again : sum.w;
    }
  }
  if (d.Cop % 4 == 0) {
    finish_row4<float>(a, d, p, m, o, sum);
    return;
  }
  // fp32 rows of any channel count: no vector of four is aligned
  const float s[4] = {sum.x, sum.y, sum.z, sum.w};
  for (int t = 0; t < 4 && o + t < d.Co; ++t) {
    float v = s[t] + reinterpret_cast<const float*>(a.wbase + d.b_off)[o + t];
    if (d.r_off != kNone) v += reinterpret_cast<const float*>(a.abase + d.r_off)[(int64_t)m * d.Cop + o + t];
    v = activate(v, d.act);
    if (d.ext) static_cast<float*>(a.ext_out[p])[(int64_t)m * d.Co + o + t] = v;
    else reinterpret_cast<float*>(a.abase + d.y_off)[(int64_t)m * d.Cop + o + t] = v;
  }
}

// F32: fp32 weights and activations.  SCALAR: a channel stride that four does not divide (an RGB input): rows are not
// 16-byte aligned and a piece may span two filter taps, so every element is fetched by itself (4-byte loads, no swizzle).
template <bool F32, bool SCALAR, int MI, int NI, int NW>
__global__ void __launch_bounds__(NW * 64) conv_kwave_kernel(KArgs a) {
  static_assert(F32 || !SCALAR, "bf16 tensors have channel strides that eight divides");
  using TA = typename std::conditional<F32, float, bf16_t>::type;
  constexpr int ES = (int)sizeof(TA);
  constexpr int TK = 128 / ES;                 // reduction elements per step
  constexpr int BM = 32 * MI, BN = 32 * NI;
  constexpr int WAVE_LDS = (BM + BN) * 128;
  constexpr int EPS = BN + 4;                  // fp32 row stride of a partial tile
  constexpr int SMEM = NW * WAVE_LDS;
  static_assert(NW * 32 * EPS * 4 <= SMEM, "the partial sums of 32 rows fit in the operand buffers");
  __shared__ __attribute__((aligned(1024))) uint8_t smem[SMEM];

  int p, bid;
  if (!find_problem_at(a, xcd_contiguous((int)blockIdx.x, (int)gridDim.x), p, bid)) return;
  const Desc d = a.d[p];
  const int batch = a.batch[p];
  const int M = batch * d.Ho * d.Wo;
  // Neighbouring workgroups (one XCD, one L2) share the larger operand: the rows of a column tile where a bf16 problem's weights
  // are larger than its input, the columns of a row tile otherwise.
  // 2048 -> 2048 pointwise, 125 rows, eight members 32.6 -> 26.9 us, 512 -> 1024, 3x3, 100 rows, two members 17.4 -> 13.4.
  const int tiles_m = (M + BM - 1) / BM;
  const bool by_column = !F32 && (int64_t)d.Co * d.Kp > (int64_t)batch * d.H * d.W * d.Cp;
  const int along = by_column ? tiles_m : d.tiles_n;
  const int outer = bid / along, inner = bid - outer * along;
  const int m0 = (by_column ? inner : outer) * BM, n0 = (by_column ? outer : inner) * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(
      a.abase + d.x_off, 0, (int)((int64_t)batch * d.H * d.W * d.Cp * ES), 0x00020000);
  const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(a.wbase + d.w_off), 0, (int)((int64_t)d.Co * d.Kp * ES), 0x00020000);

  // what this lane fetches of a step: rows lrow + RPI * i, element kv (the same in every row)
  constexpr int RPI = SCALAR ? 2 : 8;          // rows per load instruction
  constexpr int AI = BM / RPI, BI = BN / RPI;
  const int lrow = SCALAR ? lane >> 5 : lane >> 3;
  const int kv = SCALAR ? lane & 31 : ((lane & 7) ^ (lane >> 3)) * (16 / ES);
  const float inv_wo = 1.0f / (float)d.Wo, inv_ho = 1.0f / (float)d.Ho, inv_cp = 1.0f / (float)d.Cp, inv_kw = 1.0f / (float)d.kw;
  int a_row[AI], a_rc[AI];                     // byte offset of the row's window origin; filter rows / columns inside the image
#pragma unroll
  for (int i = 0; i < AI; ++i) {
    const int m = m0 + lrow + RPI * i;
    const bool ok = m < M;
    const int mm = ok ? m : 0;   // (rows past M read as zero)
    const int t = fast_div(mm, d.Wo, inv_wo);
    const int q = mm - t * d.Wo;
    const int n = fast_div(t, d.Ho, inv_ho);
    const int pp = t - n * d.Ho;
    const int ih0 = pp * d.stride - d.pad, iw0 = q * d.stride - d.pad_w;
    a_row[i] = ((n * d.H + ih0) * d.W + iw0) * d.Cp * ES;
    int rc = (int)(taps_inside(ih0, d.k, d.H) | (taps_inside(iw0, d.kw, d.W) << 16));
    asm volatile("" : "+v"(rc));   // (computed for every row: a select, not a branch per row)
    a_rc[i] = ok ? rc : 0;
  }
  const uint32_t b_row = (uint32_t)(n0 + lrow) * (uint32_t)d.Kp * ES;   // rows past Co lie past the buffer's end
  const uint32_t b_step = (uint32_t)RPI * (uint32_t)d.Kp * ES;
  const int K = d.k * d.kw * d.Cp;
  const int steps = (K + TK - 1) / TK;

  uint8_t* const As = smem + wave * WAVE_LDS;
  uint8_t* const Bs = As + BM * 128;
  auto fetch = [&](int step) {
    const int k = step * TK + kv;
    const int rs = fast_div(k, d.Cp, inv_cp);
    const int kr = fast_div(rs, d.kw, inv_kw);
    const int ks = rs - kr * d.kw;
    const uint32_t tvar = (uint32_t)(((kr * d.W + ks) * d.Cp + (k - rs * d.Cp)) * ES);
    const uint32_t dead = k < K ? 0u : OOB;    // past the reduction (a weight row's next elements belong to the next row)
    const uint32_t tap_r = k < K ? (uint32_t)kr : 0u, tap_c = k < K ? 16u + (uint32_t)ks : 16u;
#pragma unroll
    for (int i = 0; i < AI; ++i) {
      const bool ok = (((uint32_t)a_rc[i] >> tap_r) & ((uint32_t)a_rc[i] >> tap_c) & 1) != 0;
      const uint32_t off = (ok ? (uint32_t)a_row[i] + tvar : OOB) | dead;
      load_lds<SCALAR ? 4 : 16>(xres, As + i * RPI * 128, off);
    }
#pragma unroll
    for (int i = 0; i < BI; ++i)
      load_lds<SCALAR ? 4 : 16>(wres, Bs + i * RPI * 128, (b_row + b_step * i + (uint32_t)(k * ES)) | dead);
  };

  f32x16 acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

  const int r31 = lane & 31, half = lane >> 5;
  if (wave < steps) fetch(wave);
  for (int step = wave; step < steps; step += NW) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's step is in its LDS buffers
    u32x4 af[4][MI], bf[4][NI];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int piece = 2 * j + half;
      const int at = r31 * 128 + ((SCALAR ? piece : piece ^ (r31 & 7)) << 4);
#pragma unroll
      for (int i = 0; i < MI; ++i) af[j][i] = *reinterpret_cast<const u32x4*>(As + i * 32 * 128 + at);
#pragma unroll
      for (int i = 0; i < NI; ++i) bf[j][i] = *reinterpret_cast<const u32x4*>(Bs + i * 32 * 128 + at);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // every operand is in registers: the buffers may be overwritten
    if (step + NW < steps) fetch(step + NW);            // in flight while this step is multiplied
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int n = 0; n < NI; ++n) {
          if constexpr (F32) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              acc[i][n] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(bf[j][n][e]), __uint_as_float(af[j][i][e]), acc[i][n], 0, 0, 0);
          } else {
            acc[i][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, bf[j][n]), __builtin_bit_cast(bf16x8, af[j][i]), acc[i][n], 0, 0, 0);
          }
        }
  }

  // The weights were the first operand: a lane holds, for pixel (lane & 31), four runs of four consecutive channels.
  float* const part = reinterpret_cast<float*>(smem);
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    __syncthreads();   // the operand buffers (or the previous rows' partial sums) are no longer read
#pragma unroll
    for (int n = 0; n < NI; ++n)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<float4*>(&part[(wave * 32 + r31) * EPS + n * 32 + 8 * g + 4 * half]) =
            make_float4(acc[i][n][4 * g], acc[i][n][4 * g + 1], acc[i][n][4 * g + 2], acc[i][n][4 * g + 3]);
    __syncthreads();
    for (int u = tid; u < 32 * (BN / 4); u += NW * 64) {
      const int row = u / (BN / 4), c = (u % (BN / 4)) * 4;
      const int m = m0 + i * 32 + row, o = n0 + c;
      if (m >= M || o >= d.Cop) continue;
      float4 sum = *reinterpret_cast<const float4*>(&part[row * EPS + c]);
#pragma unroll
      for (int w = 1; w < NW; ++w) {
        const float4 v = *reinterpret_cast<const float4*>(&part[(w * 32 + row) * EPS + c]);
        sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w;
      }
      if constexpr (F32) finish_f32(a, d, p, m, o, sum);
      else finish_row4<TA>(a, d, p, m, o, sum);
    }
  }
}

// fp32 convolutions of one to three channels (the first layer of an unconverted model): a thread owns four pixels x eight output
// channels, in vector arithmetic.  The kernel above fetches such rows element by element (a channel stride that four does not divide), 64
// loads of 4 bytes per lane and step: 112 x 112 x 64, 7x7 stride 2, batch 4 67 us at 14 TFLOP/s.  Here a workgroup owns 16 x 16 pixels x 32
// channels, with the input patch under them and the weights, [tap][channel][output], in LDS: one round of loads, then a
// wave reads an input value for 8 products and the eight weights as two broadcasts for 32: 37 us for that layer.  Bound: the LDS reads and
// their latency, 0.4 us per tap.  (Without the patch, a tap's pixels requested one tap ahead, every tap waits for memory: 57 us.)  A filter row's products (three at
// least) are summed first, then the rows: short serial sums, as close to the exact value as the sums shared among waves above or the element kernel's.  (One
// product a row would be rounded twice: distance from 64 bits 5.5e-8 -> 6.2e-8 of 7x1, one channel; rows that are too long for this stay with the kernel above.)
template <int C>
__global__ void __launch_bounds__(256) conv_rgb_kernel(KArgs a) {
  extern __shared__ __attribute__((aligned(16))) float lds[];   // weights [k * kw * C][32], patch [PH][PW * C]
  int p, bid;   // (neighbouring rows on one die, as in the kernel above: the layer behind reads an image from its own die's cache: 8 x 112 x 112 x 32, the mean behind it 108 -> 54 us)
  if (!find_problem_at(a, xcd_contiguous((int)blockIdx.x, (int)gridDim.x), p, bid)) return;
  const Desc d = a.d[p];
  const int slabs = (d.Co + 31) / 32, bw = (d.Wo + 15) / 16, bh = (d.Ho + 15) / 16;
  const int n0 = bid % slabs * 32;
  bid /= slabs;
  const int q0 = bid % bw * 16, p0 = bid / bw % bh * 16, n = bid / bw / bh;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int K = d.k * d.kw * C, pitch = (15 * d.stride + d.kw) * C, rows = 15 * d.stride + d.k;
  float* const patch = lds + K * 32;
  {
    // eight loads of a thread at a time, the first of each kind requested together: one memory latency, not one per element
    const float* const w = reinterpret_cast<const float*>(a.wbase + d.w_off);
    const int ih0 = p0 * d.stride - d.pad, iw0 = q0 * d.stride - d.pad_w;
    const float* const x = reinterpret_cast<const float*>(a.abase + d.x_off) + (int64_t)n * d.H * d.W * C;
    const float inv_pitch = 1.0f / (float)pitch, inv_k = 1.0f / (float)K;
    const int lo = -iw0 * C, hi = (d.W - iw0) * C;   // the elements of a patch row that are inside the image
    const int nw = K * 32, nx = rows * pitch;
    for (int u0 = tid; u0 < nw || u0 < nx; u0 += 8 * 256) {
      float wv[8], xv[8];
      int to[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int u = u0 + t * 256, o = fast_div(u, K, inv_k), k = u - o * K;
        to[t] = k * 32 + o;
        wv[t] = u < nw && n0 + o < d.Co ? w[(int64_t)(n0 + o) * d.Kp + k] : 0.0f;
      }
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int u = u0 + t * 256, r = fast_div(u, pitch, inv_pitch), c = u - r * pitch;
        const bool ok = u < nx && (unsigned)(ih0 + r) < (unsigned)d.H && c >= lo && c < hi;
        xv[t] = ok ? x[((int64_t)(ih0 + r) * d.W + iw0) * C + c] : 0.0f;
      }
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int u = u0 + t * 256;
        if (u < nw) lds[to[t]] = wv[t];
        if (u < nx) patch[u] = xv[t];
      }
    }
  }
  __syncthreads();
  const int g0 = wave * 8;
  if (n0 + g0 >= d.Cop) return;
  // pixels: column lane & 15, rows (lane >> 4) + 4 i
  const float* xp[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) xp[i] = patch + ((lane >> 4) + 4 * i) * d.stride * pitch + (lane & 15) * d.stride * C;
  float acc[4][8], row[4][8];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int o = 0; o < 8; ++o) acc[i][o] = 0.0f;
  const float* wt = lds + g0;
  int held = 0;   // products in `row` (of three channels a filter row has enough by itself)
  for (int r = 0; r < d.k; ++r) {
    if (C > 2 || held == 0)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int o = 0; o < 8; ++o) row[i][o] = 0.0f;
#pragma unroll 3
    for (int s = 0; s < d.kw * C; s += C) {
#pragma unroll
      for (int c = 0; c < C; ++c) {
        const float4 w0 = *reinterpret_cast<const float4*>(wt + c * 32), w1 = *reinterpret_cast<const float4*>(wt + c * 32 + 4);
        const float wv[8] = {w0.x, w0.y, w0.z, w0.w, w1.x, w1.y, w1.z, w1.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float v = xp[i][s + c];
#pragma unroll
          for (int o = 0; o < 8; ++o) row[i][o] = __builtin_fmaf(v, wv[o], row[i][o]);
        }
      }
      wt += C * 32;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) xp[i] += pitch;
    if constexpr (C <= 2) {
      held += d.kw * C;
      if (held < 3 && r + 1 < d.k) continue;
      held = 0;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int o = 0; o < 8; ++o) acc[i][o] += row[i][o];
  }
  const int q = q0 + (lane & 15), o = n0 + g0;
  // The common case is finished from registers; an element in doubt (NaN beside padding), a residual, the caller's buffer or rows of any
  // channel count take the general way.
  bool plain = d.r_off == kNone && !d.ext && d.Cop % 8 == 0;
  float4 b0 = make_float4(0, 0, 0, 0), b1 = b0;
  if (plain) {
    b0 = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(a.wbase + d.b_off) + o);
    b1 = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(a.wbase + d.b_off) + o + 4);
    float sum = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int t = 0; t < 8; ++t) sum += acc[i][t];
    plain = !__builtin_isnan(sum);
  }
  if (plain) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float bias[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
#pragma unroll
      for (int t = 0; t < 8; ++t) acc[i][t] += bias[t];
      activate_n<8>(acc[i], d.act);
      const int pp = p0 + (lane >> 4) + 4 * i;
      if (pp < d.Ho && q < d.Wo) {
        float* const y = reinterpret_cast<float*>(a.abase + d.y_off) + ((int64_t)(n * d.Ho + pp) * d.Wo + q) * d.Cop + o;
        *reinterpret_cast<float4*>(y) = make_float4(acc[i][0], acc[i][1], acc[i][2], acc[i][3]);
        *reinterpret_cast<float4*>(y + 4) = make_float4(acc[i][4], acc[i][5], acc[i][6], acc[i][7]);
      }
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int pp = p0 + (lane >> 4) + 4 * i;
    if (pp >= d.Ho || q >= d.Wo) continue;
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (o + 4 * h < d.Cop)
        finish_f32(a, d, p, (n * d.Ho + pp) * d.Wo + q, o + 4 * h, make_float4(acc[i][4 * h], acc[i][4 * h + 1], acc[i][4 * h + 2], acc[i][4 * h + 3]));
  }
}

template <typename F>
static int go_kwave(F kernel, int blocks, int waves, const KArgs& a, hipStream_t s) {
  if (blocks <= 0) return (int)hipSuccess;
  hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3((unsigned)(waves * 64)), 0, s, a);
  return (int)hipGetLastError();
}

int launch_kwave(const Launch& L, const KArgs& args, void* stream, const std::vector<Desc>& hd) {
  const bool f32 = L.wdtype == FI_F32;
  if (L.n < 1 || L.n > FI_MAX_GROUP || (f32 ? L.adtype != FI_F32 : L.adtype != FI_BF16)) return (int)hipErrorInvalidValue;
  const bool scalar = (L.tile & KW_SCALAR) != 0;
  const bool rgb = (L.tile & KW_RGB) != 0;
  const int tile = L.tile & ~(KW_SCALAR | KW_RGB);
  if (tile >= KW_NTILES || (scalar && !f32) || (rgb && !scalar)) return (int)hipErrorInvalidValue;
  const int side = kwave_side(tile), es = f32 ? 4 : 2;
  KArgs a = args;
  int64_t blocks = 0;
  int lds = 0;
  for (int i = 0; i < L.n; ++i) {
    const Desc& t = hd[(size_t)(L.first_desc + i)];
    a.d[i] = t;
    const int b = a.batch[i];
    // 32-bit byte offsets, indices decoded with exact float arithmetic, 16-byte pieces inside one filter tap, no input stage
    if (b < 0 || t.xs != t.Cp || t.pre_kind != 0 || t.gin > 0 || t.splits != 1 || t.k < 1 || t.k > 15 || t.kw < 1 || t.kw > 15 ||
        (!scalar && t.Cp % (16 / es)) || (!f32 && t.Cop % 8) || (f32 && t.ys != t.Cop) || t.tiles_n != (t.Co + side - 1) / side ||
        !kwave_fits(b, t.H, t.W, t.Cp, t.Ho, t.Wo, t.Co, t.k * t.kw, t.Kp, es))
      return (int)hipErrorInvalidValue;
    a.first_block[i] = (int32_t)blocks;
    if (rgb) {   // 16 x 16 pixels x 32 channels
      const int64_t bytes = rgb_lds(t.k, t.kw, t.stride, t.Cp);
      if (t.Cp != a.d[0].Cp || t.Cp > 3 || t.C != t.Cp || bytes > KW_RGB_LDS) return (int)hipErrorInvalidValue;
      lds = bytes > lds ? (int)bytes : lds;
      blocks += (int64_t)b * ((t.Ho + 15) / 16) * ((t.Wo + 15) / 16) * ((t.Co + 31) / 32);
    } else {
      blocks += ((int64_t)b * t.Ho * t.Wo + side - 1) / side * t.tiles_n;
    }
    if (blocks > 0x7FFFFFFF) return (int)hipErrorInvalidConfiguration;
  }
  for (int i = L.n; i <= FI_MAX_GROUP; ++i) a.first_block[i] = (int32_t)blocks;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int nb = (int)blocks;
  if (rgb) {
    if (nb <= 0) return (int)hipSuccess;
    if (a.d[0].Cp == 1) hipLaunchKernelGGL(conv_rgb_kernel<1>, dim3((unsigned)nb), dim3(256), lds, s, a);
    else if (a.d[0].Cp == 2) hipLaunchKernelGGL(conv_rgb_kernel<2>, dim3((unsigned)nb), dim3(256), lds, s, a);
    else hipLaunchKernelGGL(conv_rgb_kernel<3>, dim3((unsigned)nb), dim3(256), lds, s, a);
    return (int)hipGetLastError();
  }
#define FI_KWAVE_CASE(F32, SCALAR, T, MI, NW) \
  if (f32 == (F32) && scalar == (SCALAR) && tile == (T)) return go_kwave(conv_kwave_kernel<F32, SCALAR, MI, MI, NW>, nb, NW, a, s);
  FI_KWAVE_CASE(true, false, KW_64x4, 2, 4)
  FI_KWAVE_CASE(true, false, KW_32x8, 1, 8)
  FI_KWAVE_CASE(true, true, KW_64x4, 2, 4)
  FI_KWAVE_CASE(true, true, KW_32x8, 1, 8)
  FI_KWAVE_CASE(false, false, KW_32x8, 1, 8)
  FI_KWAVE_CASE(false, false, KW_64x8, 2, 8)
#undef FI_KWAVE_CASE
  return (int)hipErrorInvalidValue;
}

}  // namespace fi
