// 3x3 stride-1 convolution (padding 1) whose nine filter taps are read from one input patch in LDS.
//
// The tile kernel of fi_kernels.hip fetches its input rows once per tap: nine times the tile's pixels, and the weights
// once per 256 rows: about 10 TB/s arrive at the compute units (tile sizes over times, whether through registers or by direct loads, and
// whatever the order of the walk).  Counted at the L2, VGG-16 at batch 64: 42 M requests for the 224 x 224 x 64 layer, which is
// wider than a patch and stays on the tile kernel, 6.3 M for a launch of the 512 x 128 patch.
// Here a workgroup owns BM consecutive output pixels.  With stride 1 their inputs, for every tap, are the BM + 2 W + 2
// consecutive pixels around them, one contiguous run of memory per 64 channels: they come into LDS once, by direct
// global -> LDS loads, and the tap only moves the row a lane reads (pixels outside the image read a row of zeros).
// The weights of one tap (BN rows x 64 channels) follow through a ring of three stages, two of them in flight.
// Per 64 channels a 256 x 64 tile then fetches 47 + 72 KB (56 pixels wide) instead of 9 x 40.
//
// Tiles: two workgroups of 256 rows share a compute unit's LDS (80 KB each; one loads its patch while the other
// multiplies), up to 91 pixels of width.  512 x 128 is one workgroup of eight waves per compute unit and fetches least
// (80 + 144 KB per 64 channels of 56-pixel rows, where the 256 x 128 tile moved 864 KB for the same work): matrix-bound
// layers.  Measured alone, before and after: DenseNet's 56 x 56, 128 -> 32 layers of four members at batch 32 107 -> 58 us
// (bound: LDS reads, 2.2 TB/s of HBM traffic), ResNeXt-101's 56 x 56 x 256 layers of two members 100 -> 75 us,
// VGG-16 at batch 64 28 x 28 x 512 289 -> 224 us (1.06 PFLOP/s), 56 x 56 x 256 265 -> 243 us (0.97 PFLOP/s; the patch of
// the next 64 channels is not yet loaded while these are multiplied, and 784 workgroups are 3.06 rounds).
//
// The order of the sums (64 channels, in them tap after tap, 16 elements per instruction) is the tile kernel's, so the
// bits are the same whichever kernel a launch takes.
#include <hip/hip_runtime.h>

#include "fi_device.h"
#include "fi_internal.h"

namespace fi {
namespace {

// NW waves, each owns 64 rows of the tile.  PX: pixels the patch holds.  DIAG: a grouped convolution with groups of at
// most 32 channels: of a tap's 64 x 64 weights only the two 32 x 32 blocks on the diagonal are other than zero.
template <int TILE, bool DIAG>
__global__ void __launch_bounds__(patch_bm(TILE)) conv_patch_kernel(KArgs a) {
  constexpr int BM = patch_bm(TILE), BN = patch_bn(TILE), PX = patch_pixels(TILE);
  constexpr int NW = BM / 64, MI = 2, NI = BN / 32;
  constexpr int STAGE_B = BN * 128;
  constexpr int LPB = BN / 8 / NW;             // weight loads per wave and tap (8 rows each)
  static_assert(BN / 8 % NW == 0 && (!DIAG || BN == 64), "whole loads per wave");
  constexpr int SMEM = PX * 128 + 3 * STAGE_B;
  static_assert(SMEM <= 160 * 1024, "LDS of a compute unit");
  constexpr int EPS = BN + 4;                  // fp32 row stride of a wave's epilogue patch
  static_assert(NW * 32 * EPS * 4 <= SMEM, "the epilogue patches fit");
  __shared__ __attribute__((aligned(1024))) uint8_t smem[SMEM];

  int p, bid;
  if (!find_problem_at(a, xcd_contiguous((int)blockIdx.x, (int)gridDim.x), p, bid)) return;
  const Desc d = a.d[p];
  const int batch = a.batch[p];
  const int W = d.W, Cp = d.Cp, npix = batch * d.H * W;   // stride 1, padding 1: as many outputs as inputs
  const int m0 = (bid / d.tiles_n) * BM, n0 = (bid % d.tiles_n) * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(a.abase + d.x_off, 0, (int)((int64_t)npix * Cp * 2), 0x00020000);
  const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(a.wbase + d.w_off), 0, (int)((int64_t)d.Co * d.Kp * 2), 0x00020000);

  // A load instruction brings 8 rows of 128 bytes; lane l's 16 bytes land at l * 16, so the pieces of a row are permuted
  // at the source (piece ^ row / 2 % 8): sixteen neighbouring rows, which an operand read takes at once, lie in sixteen different
  // places of 16 bytes, all banks.  (With piece ^ row % 8, eight places: 0.47 to 0.49 conflict cycles per active LDS cycle on VGG-16 at batch 64 and
  // DenseNet-121; now 0.03 to 0.14 and half the active cycles, DenseNet's 56 x 56 layers 58.5 -> 55.9 us, the matrix-bound ones unchanged: waves wait
  // 34 to 37 % of their cycles.)
  const int lrow = lane >> 3, piece = (lane & 7) ^ ((4 * wave + (lrow >> 1)) & 7);   // (a wave's loads are an even number of eight rows apart)
  const int c_lo = d.gin > 0 ? n0 : 0;         // a grouped convolution's columns read the channels of the same index
  const int nchunks = d.gin > 0 ? 1 : Cp >> 6;
  const int T = nchunks * 9;
  const int g0 = m0 - W - 1;                   // first pixel of the patch
  const int nload = (BM + 2 * W + 2 + 7) >> 3; // instructions that bring the patch (the host checks that 8 nload <= PX - 8)
  uint8_t* const ring = smem + PX * 128;
  uint32_t w_row[LPB];
#pragma unroll
  for (int i = 0; i < LPB; ++i) {
    int o = n0 + (wave + i * NW) * 8 + lrow;
    o = o < d.Co ? o : d.Co - 1;               // rows past Co are computed and discarded
    w_row[i] = (uint32_t)(o * d.Kp + c_lo + piece * 8) * 2;
  }
  int fetched = 0, f_tap = 0, f_off = 0, f_stage = 0;   // next tap to fetch: number, tap of its chunk, byte offset in a weight row, stage
  auto fetch_b = [&]() {
    const uint32_t dead = fetched < T ? 0u : OOB;
#pragma unroll
    for (int i = 0; i < LPB; ++i)
      load_lds<16>(wres, ring + f_stage * STAGE_B + (wave + i * NW) * 1024, (w_row[i] + (uint32_t)f_off) | dead);
    ++fetched;
    f_stage = f_stage == 2 ? 0 : f_stage + 1;
    const bool wrap = ++f_tap == 9;
    f_off += wrap ? 128 - 8 * Cp * 2 : Cp * 2;
    f_tap = wrap ? 0 : f_tap;
  };
  auto fetch_a = [&](int chunk) {
    const int c_off = (c_lo + chunk * 64 + piece * 8) * 2;
    for (int i = wave; i < nload; i += NW) {
      const int g = g0 + i * 8 + lrow;
      const uint32_t off = (g >= 0 && g < npix) ? (uint32_t)(g * Cp * 2 + c_off) : OOB;
      load_lds<16>(xres, smem + i * 1024, off);
    }
  };
  fetch_b();
  fetch_b();
  fetch_a(0);

  // the rows this lane reads: row r of the tile sees, for tap (kr, ks), patch pixel r + kr W + ks
  const int r31 = lane & 31, half = lane >> 5;
  uint32_t okr[MI], okc[MI];
  {
    const float inv_w = 1.0f / (float)W, inv_h = 1.0f / (float)d.H;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int m = m0 + wave * 64 + i * 32 + r31;
      const int mm = m < npix ? m : 0;
      const int t = fast_div(mm, W, inv_w);
      const int q = mm - t * W;
      const int pp = t - fast_div(t, d.H, inv_h) * d.H;
      okr[i] = m < npix ? taps_inside(pp - 1, 3, d.H) : 0u;
      okc[i] = taps_inside(q - 1, 3, W);
    }
  }
  if (tid < 8) *reinterpret_cast<uint4*>(smem + (PX - 1) * 128 + tid * 16) = make_uint4(0, 0, 0, 0);   // the row of zeros

  f32x16 acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

  int tap = 0, kr = 0, ks = 0, chunk = 0, stage = 0;
  for (int t = 0; t < T; ++t) {
    if (tap == 0) {
      if (t > 0) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();          // nobody reads the patch of the previous 64 channels any more
        asm volatile("" ::: "memory");
        fetch_a(chunk);
      }
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    } else {
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(LPB) : "memory");   // this wave's share of the tap's weights is in LDS
    }
    __builtin_amdgcn_s_barrier();              // everybody's is, and the stage before is free
    asm volatile("" ::: "memory");
    fetch_b();
    const uint8_t* at[MI];
    int sw[MI];
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int px = wave * 64 + i * 32 + r31 + kr * W + ks;
      const bool ok = ((okr[i] >> kr) & (okc[i] >> ks) & 1) != 0;
      at[i] = smem + (ok ? px : PX - 1) * 128;
      sw[i] = (((px >> 1) & 7) ^ half) << 4;
    }
    const uint8_t* const Bs = ring + stage * STAGE_B + r31 * 128;
    const int bsw = (((r31 >> 1) & 7) ^ half) << 4;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      bf16x8 af[MI], bfr[NI];
#pragma unroll
      for (int i = 0; i < MI; ++i) af[i] = *reinterpret_cast<const bf16x8*>(at[i] + (sw[i] ^ (kk << 5)));
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        if (DIAG && j != kk / 2) continue;
        bfr[j] = *reinterpret_cast<const bf16x8*>(Bs + j * 32 * 128 + (bsw ^ (kk << 5)));
      }
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) {
          if (DIAG && j != kk / 2) continue;
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[j], af[i], acc[i][j], 0, 0, 0);
        }
    }
    stage = stage == 2 ? 0 : stage + 1;
    const bool wrap = ++ks == 3;
    ks = wrap ? 0 : ks;
    kr += wrap ? 1 : 0;
    if (++tap == 9) { tap = 0; kr = 0; ++chunk; }
  }
  // nothing may land in, or be read from, the stages once the epilogue writes there
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  __syncthreads();

  // Every wave turns its rows through a patch of its own, 32 at a time: 8 consecutive channels per lane, bias, residual,
  // activation, the one rounding, 16-byte stores.
  float* const ep = reinterpret_cast<float*>(smem) + wave * 32 * EPS;
  constexpr int CPR = BN / 8, CH = 32 * CPR / 64, RSTEP = 64 / CPR;
  const int cc = (lane % CPR) * 8, lr0 = lane / CPR, o = n0 + cc;
  const bool col_ok = o < d.Cop, has_res = d.r_off != kNone, stream_out = (int64_t)npix * d.Cop * 2 > (int64_t)STREAM_OUT_BYTES;
  const uint32_t col_dead = col_ok ? 0u : OOB;
  const __amdgpu_buffer_rsrc_t rres = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(a.abase + (has_res ? d.r_off : 0)), 0, has_res ? (int)((int64_t)npix * d.Cop * 2) : 0, 0x00020000);
  const __amdgpu_buffer_rsrc_t yres = __builtin_amdgcn_make_buffer_rsrc(
      a.abase + d.y_off, 0, npix > 0 ? (int)((((int64_t)npix - 1) * d.ys + d.Cop) * 2) : 0, 0x00020000);
  // without a residual the loads return zero and the addend becomes -0.0, which leaves every value as it is
  uint32_t res_and = has_res ? 0xFFFFFFFFu : 0u, res_or = has_res ? 0u : 0x80008000u;
  asm volatile("" : "+v"(res_and), "+v"(res_or));
  const float* const bias = reinterpret_cast<const float*>(a.wbase + d.b_off) + (col_ok ? o : 0);
  const float4 b0 = *reinterpret_cast<const float4*>(bias), b1 = *reinterpret_cast<const float4*>(bias + 4);
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    const int mb = m0 + wave * 64 + i * 32;
    u32x4 rq[CH];
#pragma unroll
    for (int ch = 0; ch < CH; ++ch)
      rq[ch] = __builtin_amdgcn_raw_buffer_load_b128(rres, (uint32_t)(((mb + lr0 + ch * RSTEP) * d.Cop + o) * 2) | col_dead, 0, 0);
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<float4*>(&ep[r31 * EPS + j * 32 + 8 * g + 4 * half]) =
            make_float4(acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");   // the wave's own LDS writes precede its reads
    float v[CH][8];
#pragma unroll
    for (int ch = 0; ch < CH; ++ch) {
      const float4 v0 = *reinterpret_cast<const float4*>(&ep[(lr0 + ch * RSTEP) * EPS + cc]);
      const float4 v1 = *reinterpret_cast<const float4*>(&ep[(lr0 + ch * RSTEP) * EPS + cc + 4]);
      v[ch][0] = v0.x + b0.x; v[ch][1] = v0.y + b0.y; v[ch][2] = v0.z + b0.z; v[ch][3] = v0.w + b0.w;
      v[ch][4] = v1.x + b1.x; v[ch][5] = v1.y + b1.y; v[ch][6] = v1.z + b1.z; v[ch][7] = v1.w + b1.w;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t r = (rq[ch][e] & res_and) | res_or;
        v[ch][2 * e] += __uint_as_float(r << 16);
        v[ch][2 * e + 1] += __uint_as_float(r & 0xFFFF0000u);
      }
    }
    activate_n<CH * 8>(&v[0][0], d.act);
#pragma unroll
    for (int ch = 0; ch < CH; ++ch) {
      u32x4 pk;
#pragma unroll
      for (int e = 0; e < 4; ++e) pk[e] = pack_bf16x2(v[ch][2 * e], v[ch][2 * e + 1]);
      const uint32_t off = (uint32_t)(((mb + lr0 + ch * RSTEP) * d.ys + o) * 2) | col_dead;
      if (stream_out) __builtin_amdgcn_raw_buffer_store_b128(pk, yres, off, 0, 2);   // (far larger than the last-level cache: past it)
      else __builtin_amdgcn_raw_buffer_store_b128(pk, yres, off, 0, 0);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");   // reads done before the next rows' writes
  }
}

template <int TILE, bool DIAG>
int go_patch(int blocks, const KArgs& a, hipStream_t s) {
  if (blocks <= 0) return (int)hipSuccess;
  hipLaunchKernelGGL((conv_patch_kernel<TILE, DIAG>), dim3((unsigned)blocks), dim3((unsigned)patch_bm(TILE)), 0, s, a);
  return (int)hipGetLastError();
}

}  // namespace

int launch_patch(const Launch& L, const KArgs& args, void* stream, const std::vector<Desc>& hd) {
  if (L.n < 1 || L.n > FI_MAX_GROUP || L.wdtype != FI_BF16 || L.adtype != FI_BF16 || L.tile < 0 || L.tile >= PT_NTILES) return (int)hipErrorInvalidValue;
  const bool diag = L.tile == PT_256x64_DIAG || L.tile == PT_512x64_DIAG;
  const int bm = patch_bm(L.tile), bn = patch_bn(L.tile);
  KArgs a = args;
  int64_t blocks = 0;
  for (int i = 0; i < L.n; ++i) {
    const Desc& t = hd[(size_t)(L.first_desc + i)];
    a.d[i] = t;
    const int64_t m = (int64_t)a.batch[i] * t.H * t.W;
    if (a.batch[i] < 0 || t.k != 3 || t.kw != 3 || t.stride != 1 || t.pad != 1 || t.pad_w != 1 || t.Ho != t.H || t.Wo != t.W || t.Cp % 64 ||
        t.xs != t.Cp || t.Kp != 9 * t.Cp || t.Co != t.Cop || t.Co % 8 || t.ext || t.out_f32 || t.pre_kind != 0 || t.splits != 1 ||
        t.tiles_n != (t.Co + bn - 1) / bn || !patch_fits(L.tile, t.W) || m >= (1 << 24) || m * t.Cp * 2 >= (1ll << 31) ||
        (int64_t)t.Co * t.Kp * 2 >= (1ll << 31) || (m + 512) * (t.ys > t.Cop ? t.ys : t.Cop) * 2 >= (1ll << 31))
      return (int)hipErrorInvalidValue;
    // groups: a 64-column tile reads the 64 channels of the same index
    if (t.gin > 0 ? (bn != 64 || t.gin != t.gout || 64 % t.gin || t.Co % 64 || t.Co != t.Cp || (diag && t.gin > 32)) : diag) return (int)hipErrorInvalidValue;
    a.first_block[i] = (int32_t)blocks;
    blocks += (m + bm - 1) / bm * t.tiles_n;
    if (blocks > 0x7FFFFFFF) return (int)hipErrorInvalidConfiguration;
  }
  for (int i = L.n; i <= FI_MAX_GROUP; ++i) a.first_block[i] = (int32_t)blocks;
  hipStream_t s = static_cast<hipStream_t>(stream);
  switch (L.tile) {
    case PT_256x32: return go_patch<PT_256x32, false>((int)blocks, a, s);
    case PT_256x64: return go_patch<PT_256x64, false>((int)blocks, a, s);
    case PT_256x64_DIAG: return go_patch<PT_256x64_DIAG, true>((int)blocks, a, s);
    case PT_512x64_DIAG: return go_patch<PT_512x64_DIAG, true>((int)blocks, a, s);
    case PT_512x128: return go_patch<PT_512x128, false>((int)blocks, a, s);
  }
  return (int)hipErrorInvalidValue;
}

}  // namespace fi
