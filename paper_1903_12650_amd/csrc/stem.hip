// The 3-channel 7x7 / stride 2 stem in bf16, forward, from the padded 4-channel image (appendix log: 64 filters, no bias).
//
// A filter row of an output pixel is 8 input pixels x 4 channels = 64 consecutive bytes, 16 bytes further on for the next
// output pixel: so an MFMA operand fragment (32 pixels x 8 values) is read straight from the image rows in LDS, lane after
// lane 16 bytes apart, and nothing is gathered or unfolded.  A workgroup takes two output rows of an image at a time -- the
// nine input rows behind them are one contiguous block of memory, brought in by LDS-destination loads while the rows before
// are multiplied -- and keeps all the weights (up to 64 channels x 7 rows x 32 values) in registers, a wave per 32 pixels.
// Against the general implicit GEMM (64x64 tiles: half of what it loaded were the same 32 KB of weights again in every
// workgroup): with the padding pass 53 -> 36 us at batch 40, 307 -> 175
// at batch 256 (the output alone is 79 us at copy rate); evaluation at batch 256 4.80 -> 4.63 ms.
#include <algorithm>
#include <mutex>

#include "common.h"
#include "conv_internal.h"
#include "step_internal.h"

namespace rn50 {

constexpr int kStemSteps = 14;              // k steps of 16: seven filter rows x 32 values
constexpr int kStemRowBytes = 128 + 16;     // a pixel's row in the output staging buffer
constexpr int kStemStage = 32 * kStemRowBytes;

struct StemArgs {
  const void* xp;      // [N][Hp][pitch bytes]
  const uint16_t* w;   // [Cout][7][7][3]
  uint16_t* y;         // [N*P*Q][Cout]
  int y_through;       // writes_through of its bytes
  uint32_t xp_bytes;
  int Cout, Hp, pitch, P, Q;
  int rows;            // output rows per tile, 1 or 2 (a divisor of P)
  int patch;           // bytes of a tile's input rows
  int patch_lds;       // rounded up to whole load passes
  int tiles, per_wg;   // tiles in all, consecutive tiles per workgroup
  int M;
  FastDiv div_tpi;     // by the tiles of an image
  float* partial;      // batch-norm sums, one row per workgroup (as IgemmArgs::partial), or null
  int partial_wide;    // as doubles (bn_self_finalizes)
  // inference-mode batch norm in the output stage (AFF)
  const float *gamma, *beta, *mean, *var;
  float eps;
  int relu;
};

template <bool AFF, bool THROUGH>
__global__ __launch_bounds__(256, 2) void stem_fwd_kernel(const StemArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ double sums[4][2][64];                 // per wave: sums of the values and of their squares
  __shared__ __align__(16) float prm[AFF ? 128 : 4];  // scale, bias
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
  unsigned char* const stage = smem + 2 * a.patch_lds + wave * kStemStage;
  const OutTensor<uint16_t, THROUGH> out(a.y, a.y_through);
  const int tile0 = blockIdx.x * a.per_wg, tile1 = min(tile0 + a.per_wg, a.tiles);

  // The weights as [channel][row][tap][4 channels] in LDS (over the image buffers, which are not in use yet), then this
  // lane's fragments of them: channel l32 (+ 32), values 8 * half .. of every k step.
  for (int i = tid; i < 64 * 56; i += 256) {
    const int k = i / 56, rs = i - k * 56, r = rs >> 3, s = rs & 7;
    uint32_t lo = 0, hi = 0;
    if (k < a.Cout && s < 7) {
      const uint16_t* p = a.w + ((k * 7 + r) * 7 + s) * 3;
      lo = p[0] | static_cast<uint32_t>(p[1]) << 16;
      hi = p[2];
    }
    *reinterpret_cast<uint2*>(smem + i * 8) = make_uint2(lo, hi);
  }
  if (AFF && tid < 64) {
    const int c = min(tid, a.Cout - 1);
    float sc, bi;
    bn_coeffs(a.gamma[c], a.beta[c], a.mean[c], static_cast<float>(1.0 / sqrt(static_cast<double>(a.var[c]) + static_cast<double>(a.eps))), &sc, &bi);
    prm[tid] = sc; prm[64 + tid] = bi;
  }
  __syncthreads();
  Vec16 fw[2][kStemSteps];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int ks = 0; ks < kStemSteps; ++ks)
      fw[i][ks].u = *reinterpret_cast<const uint4*>(smem + (i * 32 + l32) * 448 + ks * 32 + half * 16);
  __syncthreads();

  const rsrc_words rs = make_rsrc_words(a.xp, a.xp_bytes);
  typedef __attribute__((address_space(3))) unsigned char* lds_byte_ptr;
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(
      static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_byte_ptr)smem)) + static_cast<uint32_t>(wave) * 1024u);
  auto load_patch = [&](int t, int buf) __attribute__((always_inline)) {
    const int tpi = a.P / a.rows;
    const int n = static_cast<int>(fdiv(static_cast<uint32_t>(t), a.div_tpi)), tr = t - n * tpi;
    const uint32_t at = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>((n * a.Hp + 2 * tr * a.rows) * a.pitch));
    for (int off = 0; off < a.patch; off += 4096) {
      const int mine = off + tid * 16;
      buffer_load16_to_lds(rs, lds0 + static_cast<uint32_t>(buf * a.patch_lds + off), mine < a.patch ? static_cast<uint32_t>(mine) : kOob, at);
    }
  };

  const int npix = a.rows * a.Q, nblk = (npix + 31) >> 5;
  const int op = lane & 7, orow = lane >> 3;      // output stage: 16-byte piece and row of a pass
  const bool col_ok = op * 8 < a.Cout;
  // Sums of what is stored, about zero, in double: a lane adds up to some 200 pixels at batch 256.  (In float about the wave's
  // first pixel 1 / std was 6.3 units in the last place off at batch 256, and 160 where images have a mean of 5 and that pixel
  // lies at the border; the general kernel's tiles: 1.0 and 1.9; this: 0.5.  A square of a bf16 value is exact in double.  It
  // costs 30.1 -> 32.0 us at batch 40, 133.6 -> 138.1 at batch 256.)
  double s1[8], s2[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) s1[j] = s2[j] = 0.0;
  if (tile0 < tile1) load_patch(tile0, 0);
  for (int t = tile0; t < tile1; ++t) {
    wait_loads_then_barrier<0>();                  // tile t has landed; everybody is done with tile t - 1
    if (t + 1 < tile1) load_patch(t + 1, (t + 1 - tile0) & 1);
    const unsigned char* img = smem + ((t - tile0) & 1) * a.patch_lds;
    const int64_t m0 = static_cast<int64_t>(t) * npix;
    for (int blk = wave; blk < nblk; blk += 4) {
      const int px = blk * 32 + l32, pc = px < npix ? px : npix - 1;
      const int row = pc >= a.Q ? 1 : 0, q = pc - row * a.Q;
      const unsigned char* src = img + 2 * row * a.pitch + q * 16 + half * 16;
      Vec16 fx[kStemSteps];
#pragma unroll
      for (int ks = 0; ks < kStemSteps; ++ks) fx[ks].u = *reinterpret_cast<const uint4*>(src + (ks >> 1) * a.pitch + (ks & 1) * 32);
      f32x16 acc[2];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;
#pragma unroll
      for (int ks = 0; ks < kStemSteps; ++ks)
#pragma unroll
        for (int i = 0; i < 2; ++i)
          acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(&fw[i][ks]),
                                                           *reinterpret_cast<const bf16x8*>(&fx[ks]), acc[i], 0, 0, 0);
      // acc[i][v]: channel i*32 + (v/4)*8 + half*4 + v%4 of pixel l32.  Rows of the block are staged in this wave's own buffer.
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int col = i * 32 + g * 8 + half * 4;
          float4 v = make_float4(acc[i][g * 4], acc[i][g * 4 + 1], acc[i][g * 4 + 2], acc[i][g * 4 + 3]);
          if constexpr (AFF) {
            const float4 sc = *reinterpret_cast<const float4*>(prm + col), bi = *reinterpret_cast<const float4*>(prm + 64 + col);
            v = make_float4(bn_affine(v.x, sc.x, bi.x), bn_affine(v.y, sc.y, bi.y), bn_affine(v.z, sc.z, bi.z), bn_affine(v.w, sc.w, bi.w));
            if (a.relu) v = make_float4(fmaxf(v.x, 0.f), fmaxf(v.y, 0.f), fmaxf(v.z, 0.f), fmaxf(v.w, 0.f));
          }
          *reinterpret_cast<uint2*>(stage + l32 * kStemRowBytes + col * 2) = make_uint2(float2_to_bf16x2_bits(v.x, v.y), float2_to_bf16x2_bits(v.z, v.w));
        }
      Vec16 o[4];
#pragma unroll
      for (int p = 0; p < 4; ++p) o[p].u = *reinterpret_cast<const uint4*>(stage + (orow + p * 8) * kStemRowBytes + op * 16);
      const int live = min(32, npix - blk * 32);
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const int r = orow + p * 8;
        if (r < live && col_ok) {
          out.store((m0 + blk * 32 + r) * a.Cout + op * 8, o[p]);
          if (!AFF && a.partial) {
            float f[8];
            Elem<uint16_t>::unpack(o[p], f);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              const double d = static_cast<double>(f[j]);
              s1[j] += d;
              s2[j] = fma(d, d, s2[j]);
            }
          }
        }
      }
    }
  }
  if (AFF || a.partial == nullptr) return;
  // The sums of the workgroup's pixels: eight row groups of a wave by shuffles, then the four waves in order.
#pragma unroll
  for (int off = 8; off < 64; off <<= 1)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      s1[j] += __shfl_xor(s1[j], off, 64);
      s2[j] += __shfl_xor(s2[j], off, 64);
    }
  if (orow == 0) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      sums[wave][0][op * 8 + j] = s1[j];
      sums[wave][1][op * 8 + j] = s2[j];
    }
  }
  __syncthreads();
  if (tid < a.Cout) {
    const double t1 = ((sums[0][0][tid] + sums[1][0][tid]) + sums[2][0][tid]) + sums[3][0][tid];
    const double t2 = ((sums[0][1][tid] + sums[1][1][tid]) + sums[2][1][tid]) + sums[3][1][tid];
    const int64_t at = bn_sums_at(blockIdx.x, tid, gridDim.x);
    if (a.partial_wide) {
      reinterpret_cast<double2*>(a.partial)[at] = make_double2(t1, t2);
    } else {  // moved to their mean, rounded to float, as shift
      const double n = static_cast<double>((tile1 - tile0) * npix);
      const float k = static_cast<float>(t1 / n);
      const double kd = static_cast<double>(k);
      reinterpret_cast<BnTileRow*>(a.partial)[at] = BnTileRow{k, static_cast<float>(t1 - n * kd), static_cast<float>(t2 - kd * (2.0 * t1 - n * kd))};
    }
  }
}

// Tiles of a launch; rows = 0: the shape does not run this kernel (float, more than 64 channels, images so small that a
// tile is less than 64 pixels or so large that two tiles' input rows exceed what two workgroups per compute unit leave).
struct StemPlan {
  int rows, tiles, per_wg, grid, patch, patch_lds;
};
static StemPlan stem_plan(const rn50_conv_desc* d) {
  StemPlan p{};
  if (!is_stem(d) || d->dtype != RN50_BF16 || d->Cout > 64) return p;
  const StemGeom g = stem_geom(d);
  const int P = out_dim(d->H, 3, 7, 2), Q = out_dim(d->W, 3, 7, 2);
  const int rows = P % 2 == 0 ? 2 : 1;
  p.patch = (2 * rows + 5) * g.Wp * 8;
  p.patch_lds = static_cast<int>(align_up(p.patch, 4096));
  if (rows * Q < 64 || 2 * p.patch_lds > 56 * 1024) return p;
  p.rows = rows;
  p.tiles = d->N * (P / rows);
  p.per_wg = static_cast<int>(ceil_div(p.tiles, 512));  // two workgroups per compute unit, all at once
  p.grid = static_cast<int>(ceil_div(p.tiles, p.per_wg));
  return p;
}
PartialRows stem_partial_rows(const rn50_conv_desc* d) {
  const StemPlan p = stem_plan(d);
  return p.rows ? PartialRows{p.per_wg * p.rows * out_dim(d->W, 3, 7, 2), p.grid} : PartialRows{0, 0};
}
bool stem_fwd_run(const rn50_conv_desc* d, const void* xp, const void* w, void* y, float* bn_partial, hipStream_t s,
                  const BnAffine* affine) {
  const StemPlan p = stem_plan(d);
  if (!p.rows) return false;
  const StemGeom g = stem_geom(d);
  StemArgs a{};
  a.xp = xp; a.w = static_cast<const uint16_t*>(w); a.y = static_cast<uint16_t*>(y);
  a.Cout = d->Cout; a.Hp = g.Hp; a.pitch = g.Wp * 8;
  a.P = out_dim(d->H, 3, 7, 2); a.Q = out_dim(d->W, 3, 7, 2);
  a.M = d->N * a.P * a.Q;
  a.y_through = writes_through(static_cast<int64_t>(a.M) * d->Cout * 2, kConvThroughBytes);
  a.xp_bytes = static_cast<uint32_t>(static_cast<size_t>(d->N) * g.Hp * a.pitch);
  a.rows = p.rows; a.patch = p.patch; a.patch_lds = p.patch_lds; a.tiles = p.tiles; a.per_wg = p.per_wg;
  a.div_tpi = make_fastdiv(a.P / a.rows);
  a.partial = bn_partial; a.partial_wide = bn_self_finalizes(p.grid, false);
  const int lds = std::max(2 * p.patch_lds + 4 * kStemStage, 64 * 448);
  static std::once_flag once;
  std::call_once(once, [] {
    allow_big_lds(stem_fwd_kernel<false, false>, 76 * 1024);
    allow_big_lds(stem_fwd_kernel<false, true>, 76 * 1024);
    allow_big_lds(stem_fwd_kernel<true, false>, 76 * 1024);
    allow_big_lds(stem_fwd_kernel<true, true>, 76 * 1024);
  });
  if (affine) {
    a.gamma = affine->gamma; a.beta = affine->beta; a.mean = affine->mean; a.var = affine->var;
    a.eps = affine->eps; a.relu = affine->relu;
    if (a.y_through) RN50_LAUNCH("conv_fwd", (stem_fwd_kernel<true, true>), dim3(p.grid), dim3(256), lds, s, a);
    else RN50_LAUNCH("conv_fwd", (stem_fwd_kernel<true, false>), dim3(p.grid), dim3(256), lds, s, a);
  } else {
    if (a.y_through) RN50_LAUNCH("conv_fwd", (stem_fwd_kernel<false, true>), dim3(p.grid), dim3(256), lds, s, a);
    else RN50_LAUNCH("conv_fwd", (stem_fwd_kernel<false, false>), dim3(p.grid), dim3(256), lds, s, a);
  }
  return true;
}

}  // namespace rn50
