// Weight gradient of a convolution: the GEMM whose reduction runs over the output pixels,
//     dw[ko][k] = sum_m dy[m][ko] * A[m][k],   k = tap * Cg + c,  A[m][k] = x at the pixel that tap reads for m,
// on the gfx950 matrix cores (v_mfma_f32_32x32x16_bf16 / v_mfma_f32_32x32x2_f32, float accumulation).
//
// Both operands have the reduction index as their slow index in memory, so tiles are copied to LDS untransposed and the
// bf16 fragments are fetched with the gfx950 transposing LDS read (ds_read_b64_tr_b16); the reduction is split over
// workgroups and finished by a fixed-order sum (bitwise reproducible).
#include <stdlib.h>

#include <algorithm>
#include <mutex>

#include "common.h"
#include "conv_internal.h"
#include "step_internal.h"

namespace rn50 {

struct WgradArgs {
  const void* x;   // gathered activation tensor [N][H][W] pixels of PS elements
  const void* dy;  // [M][Cout]
  float* out;      // dw [Cout][Ktot], or split partials
  int out_through;  // through_bytes of their bytes
  uint32_t x_bytes, dy_bytes;
  int M, Cout, Ktot;
  int H, W, P, Q, PS, Cg, R, S, stride, pad;
  int ctiles;          // column tiles
  int tiles_per_split; // column tiles * output-channel tiles
  int rows_per_split;  // multiple of the K chunk
  int64_t split_stride;
  FastDiv divQ, divP, div_Cg, div_S;
  // gathered: from a pixel to the one BKM further on.  The input row and column advance by step_h and step_w, the byte offset by
  // step_off; where the output column wraps, by -wrap_w, and one row (stride) and row_off bytes more; where the row wraps, by -wrap_h
  // and img_off.
  int step_h, step_w, step_off, wrap_w, row_off, wrap_h, img_off;
  FastDiv div_tps, div_ctiles;  // the tile decode's divisors
  // BNIN kernels (1x1, stride 1): x is the INPUT of a BN+ReLU layer whose output is the convolution's input;
  // relu(x*scale + bias) is applied to the x tile in LDS (as in igemm_kernel).  Null: x is used as is.
  const float *in_gamma, *in_beta, *in_mean, *in_rstd;
  // wgrad3x3_kernel: the padded pixel index space, Gpad = N * (H + 1) * (W + 1) positions (step_*: in it, step_off in pixels)
  int Gpad;
  FastDiv div_img, div_w1;  // by (H + 1) * (W + 1) and by W + 1
};

template <typename T> struct WgradCfg;
template <> struct WgradCfg<uint16_t> {
  static constexpr int BKM = 64;
  static __device__ __forceinline__ void mma(const Vec16& a, const Vec16& b, f32x16& acc) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(&a), *reinterpret_cast<const bf16x8*>(&b), acc, 0, 0, 0);
  }
};
template <> struct WgradCfg<float> {
  static constexpr int BKM = 32;
  static __device__ __forceinline__ void mma(const Vec16& a, const Vec16& b, f32x16& acc) {
#pragma unroll
    for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.f[j], b.f[j], acc, 0, 0, 0);
  }
};

// One workgroup: the BMO x BC tile (output channels x columns of k) of one split of the pixel range.  2 x 2 waves; per
// 64-row (32 in float) chunk of pixels the dy and x rows go straight into LDS (a ring of chunk buffers, one barrier per
// chunk, as in igemm_kernel) and are read back transposed.
// k = tap * Cg + c is one flat index: every lane fetches 16 bytes of columns and these lie in one tap (Cg is a multiple of
// the vector), so each lane has a tap of its own, a tile may span taps, and only the last tile of a filter is ragged.  (With
// tiles inside one tap, the 64 "channels" of the stem's filter-row pairs held it to 64x64 tiles, four readers of every dy.)
// What bounds the main loop: the transposing reads deliver 70 / 129 bytes per clock and compute unit with 4 / 8 waves on
// it, and a 64-pixel chunk of a 128x128 tile reads 64 KB of fragments for 512 clocks of MFMAs.  So a compute unit should
// hold two workgroups: the ring is two buffers deep (64 KB) where the tile is 128x128, three otherwise, and the plan below
// makes about two workgroups per compute unit where every one of them still has a long enough reduction.
template <typename T, int BMO, int BC, int NSTAGE, bool LIN, bool BNIN>
__global__ __launch_bounds__(256) void wgrad_kernel(const WgradArgs a) {
  static_assert(!BNIN || LIN, "the input-side BN goes with 1x1 stride-1 layers");
  constexpr int V = 16 / sizeof(T);
  constexpr int BKM = WgradCfg<T>::BKM;
  constexpr int KSTEP = sizeof(T) == 2 ? 16 : 8;
  constexpr int RA = BMO * sizeof(T), RB = BC * sizeof(T);  // row bytes of the two tiles
  constexpr int LA = RA / 16, LB = RB / 16;                  // lanes (16-byte pieces) per row
  constexpr int NA = BKM * LA / 256, NB = BKM * LB / 256;    // load instructions per thread and chunk
  constexpr int NL = NA + NB;
  constexpr int STAGE = BKM * (RA + RB);
  constexpr int TM = BMO / 64, TN = BC / 64;  // 2x2 waves
  static_assert(NA >= 1 && NB >= 1 && 256 % LA == 0 && 256 % LB == 0, "tile shape");
  extern __shared__ __align__(16) unsigned char smem[];

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int wm = wave & 1, wn = wave >> 1;
  // Logical id = (split, output-channel tile, column tile), the last fastest.  All tiles of one
  // split read the same rows of x and dy, so the renumbering keeps them on one XCD and in its L2.
  const int lid = xcd_remap(blockIdx.x, gridDim.x);
  const int split = static_cast<int>(fdiv(static_cast<uint32_t>(lid), a.div_tps)), tile = lid - split * a.tiles_per_split;
  const int ko_tile = static_cast<int>(fdiv(static_cast<uint32_t>(tile), a.div_ctiles));
  const int k0 = (tile - ko_tile * a.ctiles) * BC, ko0 = ko_tile * BMO;
  const int row_begin = split * a.rows_per_split;
  const int row_end = min(row_begin + a.rows_per_split, a.M);
  const rsrc_words rsX = make_rsrc_words(a.x, a.x_bytes), rsD = make_rsrc_words(a.dy, a.dy_bytes);

  // this thread's rows of a chunk and the 16-byte piece of them it fetches (the slot's permuted partner)
  const int rowa = tid / LA, rowb = tid / LB;
  const int pa = (tid % LA) ^ wgrad_swz<T, RA>(rowa), pb = (tid % LB) ^ wgrad_swz<T, RB>(rowb);
  const bool a_col_ok = ko0 + pa * V < a.Cout;
  const int kb = k0 + pb * V;  // this thread's first column of k
  const bool b_col_ok = kb < a.Ktot;
  // byte offsets of this thread's first rows at m = row_begin; later chunks add a scalar offset
  uint32_t a_off[NA], b_off[NB];
#pragma unroll
  for (int i = 0; i < NA; ++i)
    a_off[i] = a_col_ok ? static_cast<uint32_t>((row_begin + rowa + i * (256 / LA)) * a.Cout + ko0 + pa * V) * sizeof(T) : kOob;
  // gathered: input row, column and byte offset of the pixels that this thread's rows of the load cursor's chunk read, and the
  // limits beyond which column and row wrap (the output column Q and row P, as the tap sees them).  They are kept and advanced by a
  // chunk, at most one wrap each way: two divisions per row and chunk were as many cycles as the chunk's products (3x3 256 -> 256 at 14x14,
  // batch 256, 75.3 -> 69.6 us, the stem 195 -> 178; 23 shapes at batch 256 1945 -> 1912).
  int ih[LIN ? 1 : NB], iw[LIN ? 1 : NB], lim_h = 0, lim_w = 0;
  if constexpr (LIN) {
#pragma unroll
    for (int i = 0; i < NB; ++i)
      b_off[i] = b_col_ok ? static_cast<uint32_t>((row_begin + rowb + i * (256 / LB)) * a.PS + kb) * sizeof(T) : kOob;
  } else {
    const int tap = static_cast<int>(fdiv(static_cast<uint32_t>(kb), a.div_Cg));
    const int r = static_cast<int>(fdiv(static_cast<uint32_t>(tap), a.div_S));
    const int tc = kb - tap * a.Cg, tr = r - a.pad, ts = tap - r * a.S - a.pad;
    lim_h = a.wrap_h + tr;
    lim_w = a.wrap_w + ts;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const uint32_t mm = static_cast<uint32_t>(row_begin + rowb + i * (256 / LB));
      const uint32_t t = fdiv(mm, a.divQ), n = fdiv(t, a.divP);
      ih[i] = static_cast<int>(t - n * a.P) * a.stride + tr;
      iw[i] = static_cast<int>(mm - t * a.Q) * a.stride + ts;
      b_off[i] = static_cast<uint32_t>(((static_cast<int>(n) * a.H + ih[i]) * a.W + iw[i]) * a.PS + tc) * sizeof(T);
    }
  }

  typedef __attribute__((address_space(3))) unsigned char* lds_byte_ptr;
  const uint32_t wave_dst = __builtin_amdgcn_readfirstlane(
      static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_byte_ptr)smem)) + static_cast<uint32_t>(wave) * 1024u);
  int cur = 0;  // chunk index of the load cursor
  // Rows past row_end load zeros (no memory access): the last chunk of a split needs no special case.
  auto load_chunk = [&](int stage) __attribute__((always_inline)) {
    const int m_base = row_begin + cur * BKM;
    const int left = row_end - m_base;  // rows of this chunk that belong to the split
    const uint32_t sa = wave_dst + static_cast<uint32_t>(stage) * STAGE, sb = sa + BKM * RA;
    const uint32_t soA = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(cur) * static_cast<uint32_t>(BKM * a.Cout) * sizeof(T));
#pragma unroll
    for (int i = 0; i < NA; ++i)
      buffer_load16_to_lds(rsD, sa + i * 4096, (rowa + i * (256 / LA) < left) ? a_off[i] : kOob, soA);
    if constexpr (LIN) {
      const uint32_t soB = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(cur) * static_cast<uint32_t>(BKM * a.PS) * sizeof(T));
#pragma unroll
      for (int i = 0; i < NB; ++i)
        buffer_load16_to_lds(rsX, sb + i * 4096, (rowb + i * (256 / LB) < left) ? b_off[i] : kOob, soB);
    } else {
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const bool ok = b_col_ok && rowb + i * (256 / LB) < left && static_cast<unsigned>(ih[i]) < static_cast<unsigned>(a.H) &&
                        static_cast<unsigned>(iw[i]) < static_cast<unsigned>(a.W);
        buffer_load16_to_lds(rsX, sb + i * 4096, ok ? b_off[i] : kOob, 0u);
        iw[i] += a.step_w;
        const bool cw = iw[i] >= lim_w;
        iw[i] -= cw ? a.wrap_w : 0;
        ih[i] += a.step_h + (cw ? a.stride : 0);
        const bool ch = ih[i] >= lim_h;
        ih[i] -= ch ? a.wrap_h : 0;
        b_off[i] += static_cast<uint32_t>(a.step_off + (cw ? a.row_off : 0) + (ch ? a.img_off : 0));
      }
    }
    ++cur;
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  int fa_base[TM], fb_base[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) fa_base[i] = wgrad_frag_base<T, RA>(lane, wm * (BMO / 2) + i * 32);
#pragma unroll
  for (int j = 0; j < TN; ++j) fb_base[j] = BKM * RA + wgrad_frag_base<T, RB>(lane, wn * (BC / 2) + j * 32);
  const int nchunks = (row_end - row_begin + BKM - 1) / BKM;
  constexpr int KK = BKM / KSTEP;
  constexpr int AHEAD = (TM + TN <= 3) ? KK : 1;  // k steps whose fragments are read before the first MFMA
  auto compute = [&](int stage, auto&& next) __attribute__((always_inline)) {
    const unsigned char* st = smem + stage * STAGE;
    Vec16 fa[KK][TM], fb[KK][TN];
    auto read_frags = [&](int kk) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[kk][i] = wgrad_read_frag<T, RA>(st, fa_base[i], kk);
#pragma unroll
      for (int j = 0; j < TN; ++j) fb[kk][j] = wgrad_read_frag<T, RB>(st, fb_base[j], kk);
    };
#pragma unroll
    for (int kk = 0; kk < AHEAD; ++kk) read_frags(kk);
    __builtin_amdgcn_sched_barrier(0);
    next();  // (the next loads go out behind the first fragment reads, not in front: float at batch 8 499 -> 481 us, bf16 the same)
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      if (kk + AHEAD < KK) {
        read_frags(kk + AHEAD);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) WgradCfg<T>::mma(fa[kk][i], fb[kk][j], acc[i][j]);  // D[ko][c]
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // BNIN: this thread's piece of every x row is the same 16 bytes of channels for the whole launch
  float in_scale[BNIN ? V : 1], in_bias[BNIN ? V : 1];
  if constexpr (BNIN) {
#pragma unroll
    for (int j = 0; j < V; ++j) {
      const int c = min(kb + j, a.Cg - 1);
      bn_coeffs(a.in_gamma[c], a.in_beta[c], a.in_mean[c], a.in_rstd[c], &in_scale[j], &in_bias[j]);
    }
  }
  // the ring of igemm_kernel: loads NSTAGE-1 chunks ahead, one barrier per chunk
#pragma unroll
  for (int c = 0; c < NSTAGE - 1; ++c)
    if (c < nchunks) load_chunk(c);
  int stage = 0;
  for (int kc = 0; kc < nchunks; ++kc) {
    ring_wait<NSTAGE, NL>(nchunks - 1 - kc);
    auto next = [&]() __attribute__((always_inline)) { if (kc + NSTAGE - 1 < nchunks) load_chunk(stage >= 1 ? stage - 1 : NSTAGE - 1); };
    if constexpr (BNIN) {
      next();
      // every thread transforms, in place, the x vectors of chunk kc that its own loads brought.  Rows past the
      // split's end (loaded as zeros) become relu(bias); their dy rows are zeros, so they add nothing.
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        uint4* p = reinterpret_cast<uint4*>(smem + stage * STAGE + BKM * RA + i * 4096 + tid * 16);
        Vec16 v;
        v.u = *p;
        *p = bn_relu_vector<T>(v, in_scale, in_bias).u;
      }
      lds_writes_then_barrier();
      compute(stage, [] {});
    } else {
      compute(stage, next);
    }
    stage = stage == NSTAGE - 1 ? 0 : stage + 1;
  }

  // acc[i][j][v]: ko = i*32 + (v/4)*8 + (lane/32)*4 + v%4, k = j*32 + lane%32
  if (a.out_through != 0 && ko0 + BMO <= a.Cout && k0 + BC <= a.Ktot) {
    // a whole tile, written through: one offset per block and lane, the rows of the block by a scalar
    const __amdgpu_buffer_rsrc_t r = make_rsrc(a.out, a.out_through);
    const uint32_t base = static_cast<uint32_t>(split * a.split_stride), pitch = static_cast<uint32_t>(a.Ktot) * 4u;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const uint32_t off = (base + static_cast<uint32_t>((ko0 + wm * (BMO / 2) + i * 32 + (lane >> 5) * 4) * a.Ktot + k0 + wn * (BC / 2) + j * 32 + (lane & 31))) * 4u;
#pragma unroll
        for (int v = 0; v < 16; ++v)
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[i][j][v]), r, static_cast<int>(off),
                                                static_cast<int>(static_cast<uint32_t>((v >> 2) * 8 + (v & 3)) * pitch), kSystemScope);
      }
    return;
  }
  float* out = a.out + static_cast<int64_t>(split) * a.split_stride;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int k = k0 + wn * (BC / 2) + j * 32 + (lane & 31);
      if (k >= a.Ktot) continue;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int ko = ko0 + wm * (BMO / 2) + i * 32 + (v >> 2) * 8 + (lane >> 5) * 4 + (v & 3);
        if (ko < a.Cout) out[static_cast<int64_t>(ko) * a.Ktot + k] = acc[i][j][v];
      }
    }
}

// Weight gradient of a 3x3 / stride 1 / padding 1 layer of at most 64 channels each way, bf16, all nine taps in one workgroup.
// The reduction index is a PADDED pixel position: every image row gets one more column and every image one more
// row, whose dy and x are zero (never stored: the loads of those positions carry an out-of-range offset and
// write zeros).  In that index space tap (r, s) of position k reads x at k + (r-1)(W+1) + (s-1), a constant shift,
// and every tap that falls off the image lands on a zero position -- so there is nothing to mask: per chunk of 64
// positions the workgroup brings one dy tile [64][64 output channels] and one x run [64 + 2W + 4][64 input
// channels] into LDS and multiplies the dy tile with nine row-shifted windows of the run (transposing reads, the
// slot permutation follows the shifted row) into nine 64x64 accumulator tiles.  Against one gathered tile per tap
// that is 9x fewer dy loads and 9 / (1 + (2W+4)/64) fewer x loads; the reduction grows by (1+1/H)(1+1/W).
// NBX: load passes (32 rows each) of the run; NSTAGE: chunk buffers in the ring (as in wgrad_kernel).
template <int NBX, int NSTAGE>
__global__ __launch_bounds__(256) void wgrad3x3_kernel(const WgradArgs a) {
  typedef uint16_t T;
  constexpr int V = 8, BKM = 64, RBY = 128, KK = 4;
  constexpr int NA = 2, NL = NA + NBX;
  constexpr int STAGE = BKM * RBY + NBX * 4096;
  extern __shared__ __align__(16) unsigned char smem[];

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int wm = wave & 1, wn = wave >> 1;
  const int split = xcd_remap(blockIdx.x, gridDim.x);  // neighbours share the run's border rows
  const int row_begin = split * a.rows_per_split;
  const int row_end = min(row_begin + a.rows_per_split, a.Gpad);
  const rsrc_words rsX = make_rsrc_words(a.x, a.x_bytes), rsD = make_rsrc_words(a.dy, a.dy_bytes);

  const int row = tid >> 3;                                  // this thread's row in every 32-row load pass
  const int pc = (tid & 7) ^ wgrad_swz<T, RBY>(row);        // the 16-byte piece of its rows it fetches
  const bool a_col_ok = pc * V < a.Cout, b_col_ok = pc * V < a.Cg;
  const int W1 = a.W + 1, IMG = (a.H + 1) * W1;
  // A padded position: its column and row (W and H: padding), its pixel, what it is itself.  Decoded once and then moved on by a chunk of
  // 64, at most one wrap each way (WgradArgs::step_*; a row's padding takes a column back, an image's a row).  (Eight positions divided out
  // per chunk were 1450 cycles beside 1152 of products: 64 -> 64 at 56x56, batch 256 98.5 -> 89.8 us, 40 32.1 -> 30.0.)
  struct Position {
    int x, y, pix, g;
  };
  auto position = [&](int g) __attribute__((always_inline)) {  // (g > -IMG: the first run starts in front of the first image)
    const uint32_t gg = static_cast<uint32_t>(g + IMG), n = fdiv(gg, a.div_img), rem = gg - n * static_cast<uint32_t>(IMG);
    const uint32_t y = fdiv(rem, a.div_w1);
    Position p;
    p.y = static_cast<int>(y);
    p.x = static_cast<int>(rem) - p.y * W1;
    p.pix = ((static_cast<int>(n) - 1) * a.H + p.y) * a.W + p.x;
    p.g = g;
    return p;
  };
  auto advance = [&](Position& p) __attribute__((always_inline)) {
    p.x += a.step_w;
    const bool cx = p.x >= W1;
    p.x -= cx ? W1 : 0;
    p.y += a.step_h + (cx ? 1 : 0);
    const bool cy = p.y > a.H;
    p.y -= cy ? a.H + 1 : 0;
    p.pix += a.step_off - (cx ? 1 : 0) - (cy ? a.W : 0);
    p.g += BKM;
  };
  auto real = [&](const Position& p, int end) __attribute__((always_inline)) { return p.g >= 0 && p.g < end && p.y < a.H && p.x < a.W; };
  typedef __attribute__((address_space(3))) unsigned char* lds_byte_ptr;
  const uint32_t wave_dst = __builtin_amdgcn_readfirstlane(
      static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_byte_ptr)smem)) + static_cast<uint32_t>(wave) * 1024u);
  // This thread's rows of a chunk: two of dy (positions of this split only, the others belong to other workgroups) and NBX of the run of
  // x, which starts W + 2 positions before the chunk.  They lie 32 apart, so the next chunk's run has this one's rows from the third on
  // first, and two new ones.
  Position pd[NA], px[2];
  uint32_t off_d[NA], off_x[NBX];
  auto offset_d = [&](const Position& p) __attribute__((always_inline)) {
    return real(p, row_end) && a_col_ok ? static_cast<uint32_t>(p.pix * a.Cout + pc * V) * 2u : kOob;
  };
  auto offset_x = [&](const Position& p) __attribute__((always_inline)) {
    return real(p, a.Gpad) && b_col_ok ? static_cast<uint32_t>(p.pix * a.PS + pc * V) * 2u : kOob;
  };
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    pd[i] = position(row_begin + row + 32 * i);
    off_d[i] = offset_d(pd[i]);
  }
#pragma unroll
  for (int i = 0; i < NBX; ++i) {
    const Position p = position(row_begin - (a.W + 2) + row + 32 * i);
    off_x[i] = offset_x(p);
    if (i >= NBX - 2) px[i - (NBX - 2)] = p;
  }
  auto load_chunk = [&](int stage) __attribute__((always_inline)) {
    const uint32_t sa = wave_dst + static_cast<uint32_t>(stage) * STAGE, sb = sa + BKM * RBY;
#pragma unroll
    for (int i = 0; i < NA; ++i) buffer_load16_to_lds(rsD, sa + i * 4096, off_d[i], 0u);
#pragma unroll
    for (int i = 0; i < NBX; ++i) buffer_load16_to_lds(rsX, sb + i * 4096, off_x[i], 0u);
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      advance(pd[i]);
      off_d[i] = offset_d(pd[i]);
    }
#pragma unroll
    for (int i = 0; i + 2 < NBX; ++i) off_x[i] = off_x[i + 2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      advance(px[i]);
      off_x[NBX - 2 + i] = offset_x(px[i]);
    }
  };

  f32x16 acc[9];
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;

  // Fragment addresses.  dy: as in wgrad_kernel.  x: the same transposing read r*(W+1) + s rows further down the
  // run; the slot permutation of a row depends on bit 1 of the row, so it is taken from the shifted row (the
  // reads' +4 and +16*kk rows leave that bit alone).
  const int fa_base = wgrad_frag_base<T, RBY>(lane, wm * 32);
  int fb_base[9];
  {
    const int g4 = lane >> 4, t = lane & 15;
    const int krow = 8 * (g4 >> 1) + (t >> 2);
    const int cb = 2 * (wn * 32 + 16 * (g4 & 1) + 4 * (t & 3));
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      const int kr = krow + (tap / 3) * W1 + (tap % 3);
      fb_base[tap] = BKM * RBY + kr * RBY + (((cb >> 4) ^ wgrad_swz<T, RBY>(kr)) << 4) + (cb & 15);
    }
  }
  const int nchunks = (row_end - row_begin + BKM - 1) / BKM;
  auto compute = [&](int stage) __attribute__((always_inline)) {
    const unsigned char* st = smem + stage * STAGE;
    Vec16 fa[KK], fb[2][KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) fa[kk] = wgrad_read_frag<T, RBY>(st, fa_base, kk);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) fb[0][kk] = wgrad_read_frag<T, RBY>(st, fb_base[0], kk);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      if (tap + 1 < 9) {
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) fb[(tap + 1) & 1][kk] = wgrad_read_frag<T, RBY>(st, fb_base[tap + 1], kk);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) WgradCfg<T>::mma(fa[kk], fb[tap & 1][kk], acc[tap]);  // D[ko][c]
      __builtin_amdgcn_sched_barrier(0);
    }
  };
#pragma unroll
  for (int c = 0; c < NSTAGE - 1; ++c)
    if (c < nchunks) load_chunk(c);
  int stage = 0;
  for (int kc = 0; kc < nchunks; ++kc) {
    ring_wait<NSTAGE, NL>(nchunks - 1 - kc);
    if (kc + NSTAGE - 1 < nchunks) load_chunk(stage >= 1 ? stage - 1 : NSTAGE - 1);
    compute(stage);
    stage = stage == NSTAGE - 1 ? 0 : stage + 1;
  }

  // acc[tap][v]: ko = (v/4)*8 + (lane/32)*4 + v%4, c = lane%32 of this wave's 32x32 block
  const int c = wn * 32 + (lane & 31);
  if (a.out_through != 0 && a.Cout == 64 && a.Cg == 64) {  // (as in wgrad_kernel)
    const __amdgpu_buffer_rsrc_t r = make_rsrc(a.out, a.out_through);
    const uint32_t off = (static_cast<uint32_t>(split * a.split_stride) + static_cast<uint32_t>((wm * 32 + (lane >> 5) * 4) * a.Ktot + c)) * 4u;
#pragma unroll
    for (int tap = 0; tap < 9; ++tap)
#pragma unroll
      for (int v = 0; v < 16; ++v)
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[tap][v]), r, static_cast<int>(off),
                                              static_cast<int>(static_cast<uint32_t>(((v >> 2) * 8 + (v & 3)) * a.Ktot + tap * a.Cg) * 4u), kSystemScope);
    return;
  }
  float* out = a.out + static_cast<int64_t>(split) * a.split_stride;
  if (c < a.Cg) {
#pragma unroll
    for (int tap = 0; tap < 9; ++tap)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int ko = wm * 32 + (v >> 2) * 8 + (lane >> 5) * 4 + (v & 3);
        if (ko < a.Cout) out[static_cast<int64_t>(ko) * a.Ktot + tap * a.Cg + c] = acc[tap][v];
      }
  }
}

// ------------------------------------------------------------------ sum of the splits
// dw[i] = sum_s partial[s][i].  A workgroup owns 16 float4 outputs; its sixteen groups of 16 threads each sum every
// sixteenth split (ascending) and the sixteen sums are added in order: a fixed order.
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* __restrict__ partial, int splits, int64_t n,
                                                            float* __restrict__ out) {
  __shared__ float4 red[16][16];
  const int lane = threadIdx.x & 15, grp = threadIdx.x >> 4;
  const int64_t i = (static_cast<int64_t>(blockIdx.x) * 16 + lane) * 4;  // (n is a multiple of 4)
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  if (i < n) {
#pragma unroll 8
    for (int k = grp; k < splits; k += 16) {
      const float4 v = *reinterpret_cast<const float4*>(partial + k * n + i);
      s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
  }
  red[grp][lane] = s;
  __syncthreads();
  if (grp == 0 && i < n) {
    float4 r = red[0][lane];
#pragma unroll
    for (int g = 1; g < 16; ++g) {
      const float4 v = red[g][lane];
      r.x += v.x; r.y += v.y; r.z += v.z; r.w += v.w;
    }
    *reinterpret_cast<float4*>(out + i) = r;
  }
}

// dw [K][7][7][3] <- dwp [K][8][8][4]
__global__ __launch_bounds__(256) void stem_unpad_dw_kernel(const float* __restrict__ dwp, float* __restrict__ dw, int K) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= K * 147) return;
  const int c = i % 3, s = (i / 3) % 7, r = (i / 21) % 7, k = i / 147;
  dw[i] = dwp[((k * 8 + r) * 8 + s) * 4 + c];
}

// ------------------------------------------------------------------------------ host side
struct WgradPlan {
  int bmo, bc, ctiles, splits, rows_per_split;
};
// Tile shape and number of reduction splits: the cheapest of the four tiles x about 256, 512 or 768 workgroups by an
// estimate of the launch's microseconds.  A small tile loads more bytes per flop; a large one gives few tiles, so it needs
// many splits to fill the chip, and every split costs a full-size partial result written and read again -- which of the two
// is dearer moves with the pixel count, the channel counts and the filter (the 7x7 layers at batch 40: 64x64 tiles and no
// split 12.8 us, 128x128 tiles 22 us; the 14x14 3x3 layer at batch 256: 128x128 tiles 74 us, 64x64 tiles 110 us).
// The estimate: workgroups fill the compute units in rounds of `slots` each; a chunk of n workgroups on one compute unit
// takes the longer of one's latency (lat) and n times the tile's share of the LDS and load rates (thr), both dearer where
// pixels are gathered; `ends` is prologue and result stores; splits add the reduction launch and the partials' traffic.
// Constants fitted to ResNet-50's 23 shapes x 12 plans at batch 12 to 256 (bf16) and 2 to 24 (float), when a chunk's pixels were still
// divided out; since they are advanced from chunk to chunk the plan it takes is within 0 to 5 % of the best of the twelve, summed over the
// shapes, 6 % at batch 90 and in float at batch 4 (profiles/wgrad_plan_sweep.txt: 480 against 467 us at batch 40, 805 against 757 at 90, 1755 against
// 1713 at 256, float at batch 8 510 against 502).  Against the fixed rule before it (128-wide tiles, 192 or 384 workgroups), when it was fitted: 23 shapes at
// batch 40 640 -> 565 us call by call, at batch 256 2343 -> 2000, float at batch 8 830 -> 531.
struct WgradCost {
  float thr[3], lat[3], ends[3];  // us; tile area 64x64, 128x64, 128x128
  float thr_gather, lat_gather, reduce, partial_us_per_mb;
};
static const WgradCost kWgradCostBf16 = {{.20f, .30f, .48f}, {.35f, .47f, .64f}, {.5f, 1.f, 1.45f}, 1.04f, 1.45f, 4.7f, .28f};
static const WgradCost kWgradCostF32 = {{.18f, .28f, .55f}, {.45f, .87f, 1.42f}, {.5f, 1.f, .8f}, 2.76f, 1.47f, 1.8f, .71f};
static WgradPlan plan_wgrad(const WgradArgs& a, int dtype) {
  const int bkm = dtype == RN50_BF16 ? 64 : 32, min_chunks = 4;
  const WgradCost& c = dtype == RN50_BF16 ? kWgradCostBf16 : kWgradCostF32;
  const bool gather = !(a.R == 1 && a.S == 1 && a.stride == 1 && a.pad == 0);
  const double dw_mb = static_cast<double>(a.Cout) * a.Ktot * 4e-6;
  const int64_t cap = a.M / (min_chunks * bkm) > 1 ? a.M / (min_chunks * bkm) : 1;
  WgradPlan best{};
  double best_us = 0.0;
  for (int t = 0; t < 4; ++t) {
    const int bmo = t & 1 ? 128 : 64, bc = t & 2 ? 128 : 64, area = (t & 1) + (t >> 1);
    if ((bmo > 64 && a.Cout <= 64) || (bc > 64 && a.Ktot <= 64)) continue;
    const int64_t ctiles = ceil_div(a.Ktot, bc), tiles = ctiles * ceil_div(a.Cout, bmo);
    int t_lo = 256, t_hi = 768;
#ifdef RN50_TUNING  // tuning builds only: RN50_WGRAD_TARGETS=lowest,highest workgroup target
    if (const char* e = getenv("RN50_WGRAD_TARGETS")) sscanf(e, "%d,%d", &t_lo, &t_hi);
#endif
    for (int target = t_lo; target <= t_hi; target += 256) {
      int64_t sp = (target + tiles / 2) / tiles;
      sp = sp < 1 ? 1 : (sp > cap ? cap : sp);
      const int64_t rps = ceil_div(ceil_div(a.M, sp), bkm) * bkm;
      const int splits = static_cast<int>(ceil_div(a.M, rps));
      const int64_t grid = tiles * splits, chunks = rps / bkm;
      const int slots = area == 0 ? 3 : 2;
      auto round_us = [&](int64_t n) {
        const double one = c.lat[area] * (gather ? c.lat_gather : 1.f), all = n * c.thr[area] * (gather ? c.thr_gather : 1.f);
        return chunks * (one > all ? one : all) + n * c.ends[area];
      };
      const int64_t full = grid / (256 * slots), rem = grid % (256 * slots);
      double us = full * round_us(slots) + (rem ? round_us(ceil_div(rem, 256)) : 0.0);
      if (splits > 1) us += c.reduce + splits * dw_mb * c.partial_us_per_mb;
      if (best.splits == 0 || us < best_us) {
        best_us = us;
        best = WgradPlan{bmo, bc, static_cast<int>(ctiles), splits, static_cast<int>(rps)};
      }
    }
  }
  return best;
}

template <typename T, int BMO, int BC>
static void launch_wgrad_cfg(const WgradArgs& a, dim3 grid, hipStream_t s) {
  constexpr int NSTAGE = BMO == 128 && BC == 128 ? 2 : 3;
  constexpr int lds = NSTAGE * WgradCfg<T>::BKM * (BMO + BC) * static_cast<int>(sizeof(T));
  static std::once_flag once;
  std::call_once(once, [] {
    allow_big_lds(wgrad_kernel<T, BMO, BC, NSTAGE, true, true>, lds);
    allow_big_lds(wgrad_kernel<T, BMO, BC, NSTAGE, true, false>, lds);
    allow_big_lds(wgrad_kernel<T, BMO, BC, NSTAGE, false, false>, lds);
  });
  const bool linear = a.R == 1 && a.S == 1 && a.stride == 1 && a.pad == 0;
  if (a.in_gamma) RN50_LAUNCH("conv_wgrad", (wgrad_kernel<T, BMO, BC, NSTAGE, true, true>), grid, dim3(256), lds, s, a);
  else if (linear) RN50_LAUNCH("conv_wgrad", (wgrad_kernel<T, BMO, BC, NSTAGE, true, false>), grid, dim3(256), lds, s, a);
  else RN50_LAUNCH("conv_wgrad", (wgrad_kernel<T, BMO, BC, NSTAGE, false, false>), grid, dim3(256), lds, s, a);
}

static WgradArgs wgrad_args(const rn50_conv_desc* d, const void* x, const void* dy) {
  WgradArgs a{};
  a.x = x; a.dy = dy;
  a.Cout = d->Cout;
  if (is_stem(d)) {
    // the padded image: filter rows of 8 taps x 4 channels = 32 consecutive elements; eight rows (one of
    // zeros) make k
    const StemGeom g = stem_geom(d);
    a.P = out_dim(d->H, 3, 7, 2); a.Q = out_dim(d->W, 3, 7, 2);
    a.Ktot = kStemK;
    a.H = g.Hp; a.W = g.Wp; a.PS = 4; a.Cg = 32; a.S = 1; a.stride = 2; a.pad = 0;
    a.R = 8;
    a.x_bytes = static_cast<uint32_t>(static_cast<size_t>(d->N) * g.Hp * g.Wp * 4 * esize(d->dtype));
  } else {
    a.P = out_dim(d->H, d->pad, d->R, d->stride); a.Q = out_dim(d->W, d->pad, d->S, d->stride);
    a.Ktot = d->R * d->S * d->Cin;
    a.H = d->H; a.W = d->W; a.PS = d->Cin; a.Cg = d->Cin; a.R = d->R; a.S = d->S; a.stride = d->stride; a.pad = d->pad;
    a.x_bytes = static_cast<uint32_t>(static_cast<size_t>(d->N) * d->H * d->W * d->Cin * esize(d->dtype));
  }
  a.M = d->N * a.P * a.Q;
  a.dy_bytes = static_cast<uint32_t>(static_cast<size_t>(a.M) * d->Cout * esize(d->dtype));
  a.split_stride = static_cast<int64_t>(a.Cout) * a.Ktot;
  return a;
}
// 3x3, stride 1, padding 1 layers of at most 64 channels each way in bf16 (one 64x64 tile per tap; wider layers do better on wgrad_kernel's
// 128-wide tiles), of an image width whose run of 2W + 68 rows fits six load passes, from kNineTapPositions padded positions on: the nine-tap
// kernel (wgrad3x3_kernel).  With fewer, its workgroups are too few or too short: there one tile per tap, in splits of kShortSplitRows rows,
// whose float sums are no longer than the nine-tap kernel's.  64 -> 64, us, nine taps / per tap / per tap as plan_wgrad would split it, and their
// errors against 64 bits in 1e-7: 56x56 at batch 4 22.0 / 11.8 / 11.8 (1.31 / 1.09 / 1.09), 12 23.8 / 16.0 / 15.8 (1.37 / 1.33 / 1.46), 24 26.8 / 24.2 /
// 20.3, 40 28.7 / 30.5 / 27.1 (1.40 / 1.38 / 1.77), 90 46.2 / - / 45.8 (1.75 / - / 2.80), 256 83 / - / 97; 28x28 at batch 70 28 / 21 / 18 (1.34 / 1.34 / 1.63).
// In the step short splits gain at batch 12 (2.398 -> 2.386 ms), not at 24 and 33, and lose at 40 (4.165 -> 4.187); splits as plan_wgrad
// would take them gain up to batch 64 (4.165 -> 4.146 at 40), but their sums are less exact than the nine-tap kernel's.
// Plan: the padded pixel range split to give about 384 workgroups, each at least 8 chunks long.
constexpr int64_t kNineTapPositions = 1 << 16;
constexpr int kShortSplitRows = 512;
struct Wgrad3x3Plan {
  int nbx;  // load passes of the x run: 3, 4 or 6; 0: the layer does not run this kernel
  int splits, rows_per_split, gpad;
};
static Wgrad3x3Plan plan_wgrad3x3(const rn50_conv_desc* d, bool* fewer) {  // fewer: such a layer, with fewer positions
  Wgrad3x3Plan p{};
  *fewer = false;
  if (d->dtype != RN50_BF16 || d->R != 3 || d->S != 3 || d->stride != 1 || d->pad != 1) return p;
  if (d->Cin > 64 || d->Cout > 64) return p;
  const int need = static_cast<int>(ceil_div(2 * d->W + 68, 32));
  if (need > 6) return p;
  const int64_t gpad = static_cast<int64_t>(d->N) * (d->H + 1) * (d->W + 1);
  *fewer = gpad < kNineTapPositions;
  if (*fewer || gpad >= (1ll << 31) - 64) return p;
  p.nbx = need <= 3 ? 3 : (need == 4 ? 4 : 6);
  p.gpad = static_cast<int>(gpad);
  constexpr int target = 384, min_chunks = 8;
  const int64_t sp = std::min<int64_t>(target, gpad / (min_chunks * 64));
  const int64_t rps = ceil_div(ceil_div(gpad, sp), 64) * 64;
  p.rows_per_split = static_cast<int>(rps);
  p.splits = static_cast<int>(ceil_div(gpad, rps));
  return p;
}
static WgradPlan short_splits(WgradPlan p, const WgradArgs& a) {
  if (p.rows_per_split <= kShortSplitRows) return p;
  return WgradPlan{64, 64, static_cast<int>(ceil_div(a.Ktot, 64)), static_cast<int>(ceil_div(a.M, kShortSplitRows)), kShortSplitRows};
}
template <int NBX, int NSTAGE>
static void launch_wgrad3x3_ring(const WgradArgs& a, dim3 grid, hipStream_t s) {
  constexpr int lds = NSTAGE * (64 * 128 + NBX * 4096);
  static std::once_flag once;
  std::call_once(once, [] { allow_big_lds(wgrad3x3_kernel<NBX, NSTAGE>, lds); });
  RN50_LAUNCH("conv_wgrad", (wgrad3x3_kernel<NBX, NSTAGE>), grid, dim3(256), lds, s, a);
}
template <int NBX>
static void launch_wgrad3x3_nbx(const WgradArgs& a, dim3 grid, hipStream_t s) {
  // three chunk buffers where the workgroups on a compute unit, two at most, have the LDS for them, else two
  if constexpr (2 * 3 * (64 * 128 + NBX * 4096) > 156 * 1024) {
    if (grid.x > 256) return launch_wgrad3x3_ring<NBX, 2>(a, grid, s);
  }
  launch_wgrad3x3_ring<NBX, 3>(a, grid, s);
}
static void launch_wgrad3x3(WgradArgs a, const Wgrad3x3Plan& p, int H, hipStream_t s) {
  a.rows_per_split = p.rows_per_split;
  a.Gpad = p.gpad;
  const int img = (H + 1) * (a.W + 1), in_img = 64 % img;  // 64 positions: whole images, rows and columns
  a.step_h = in_img / (a.W + 1);
  a.step_w = in_img % (a.W + 1);
  a.step_off = (64 / img * H + a.step_h) * a.W + a.step_w;
  a.div_img = make_fastdiv(img);
  a.div_w1 = make_fastdiv(a.W + 1);
  const dim3 grid(static_cast<unsigned>(p.splits));
  if (p.nbx == 3) launch_wgrad3x3_nbx<3>(a, grid, s);
  else if (p.nbx == 4) launch_wgrad3x3_nbx<4>(a, grid, s);
  else launch_wgrad3x3_nbx<6>(a, grid, s);
}

size_t wgrad_partial_bytes(const rn50_conv_desc* d) {
  const size_t dw_elems = static_cast<size_t>(d->Cout) * (is_stem(d) ? kStemK : d->R * d->S * d->Cin);
  bool fewer;
  const Wgrad3x3Plan p9 = plan_wgrad3x3(d, &fewer);
  const WgradArgs a = wgrad_args(d, nullptr, nullptr);
  const WgradPlan p = plan_wgrad(a, d->dtype);
  const int splits = std::max(p9.nbx ? p9.splits : 1, fewer ? short_splits(p, a).splits : p.splits);
  size_t b = splits > 1 ? align_up(dw_elems * splits * sizeof(float), 256) : 0;
  if (is_stem(d)) b += align_up(dw_elems * sizeof(float), 256);  // padded dw
  return b;
}

// Weight gradient; for the stem x must be the padded input.  scratch: wgrad_partial_bytes(d).
void wgrad_run(const rn50_conv_desc* d, const void* x_or_xp, const void* dy, float* dw, void* scratch, hipStream_t s,
               const BnIn* in) {
  WgradArgs a = wgrad_args(d, x_or_xp, dy);
  if (in) { a.in_gamma = in->gamma; a.in_beta = in->beta; a.in_mean = in->mean; a.in_rstd = in->rstd; }
  float* partial = static_cast<float*>(scratch);
  float* target = dw;
  const bool stem = is_stem(d);
  if (stem) {
    target = partial;
    partial += align_up(static_cast<size_t>(d->Cout) * kStemK * sizeof(float), 256) / sizeof(float);
  }
  int splits;
  bool fewer;
  if (const Wgrad3x3Plan p9 = plan_wgrad3x3(d, &fewer); p9.nbx) {
    splits = p9.splits;
    a.out = splits > 1 ? partial : target;
    a.out_through = through_bytes(4 * splits * a.split_stride);
    launch_wgrad3x3(a, p9, d->H, s);
  } else {
    WgradPlan p = plan_wgrad(a, d->dtype);
    if (fewer) p = short_splits(p, a);
    splits = p.splits;
    a.out = splits > 1 ? partial : target;
    a.out_through = through_bytes(4 * splits * a.split_stride);
    a.ctiles = p.ctiles;
    a.rows_per_split = p.rows_per_split;
    a.tiles_per_split = p.ctiles * static_cast<int>(ceil_div(a.Cout, p.bmo));
    a.divQ = make_fastdiv(a.Q);
    a.divP = make_fastdiv(a.P);
    a.div_Cg = make_fastdiv(a.Cg);
    a.div_S = make_fastdiv(a.S);
    const int es = esize(d->dtype), bkm = d->dtype == RN50_BF16 ? WgradCfg<uint16_t>::BKM : WgradCfg<float>::BKM;
    const int img = a.P * a.Q, in_img = bkm % img;  // BKM pixels: whole images, rows and columns
    a.step_h = in_img / a.Q * a.stride;
    a.step_w = in_img % a.Q * a.stride;
    a.step_off = ((bkm / img * a.H + a.step_h) * a.W + a.step_w) * a.PS * es;
    a.wrap_w = a.Q * a.stride;
    a.row_off = (a.stride * a.W - a.wrap_w) * a.PS * es;
    a.wrap_h = a.P * a.stride;
    a.img_off = (a.H - a.wrap_h) * a.W * a.PS * es;
    a.div_tps = make_fastdiv(a.tiles_per_split);
    a.div_ctiles = make_fastdiv(a.ctiles);
    const dim3 grid(static_cast<unsigned>(a.tiles_per_split) * p.splits);
#define RN50_WGRAD_TILE(BMO, BC)                                                        \
  if (p.bmo == BMO && p.bc == BC) {                                                     \
    if (d->dtype == RN50_BF16) launch_wgrad_cfg<uint16_t, BMO, BC>(a, grid, s);         \
    else launch_wgrad_cfg<float, BMO, BC>(a, grid, s);                                  \
  }
    RN50_WGRAD_TILE(128, 128) RN50_WGRAD_TILE(128, 64) RN50_WGRAD_TILE(64, 128) RN50_WGRAD_TILE(64, 64)
#undef RN50_WGRAD_TILE
  }
  if (splits > 1) {
    const int64_t n = a.split_stride;
    RN50_LAUNCH("splitk_reduce", splitk_reduce_kernel, dim3(static_cast<unsigned>(ceil_div(n, 64))), dim3(256), 0, s, partial, splits, n, target);
  }
  if (stem)
    RN50_LAUNCH("stem_unpad", stem_unpad_dw_kernel, dim3(ceil_div(d->Cout * 147, 256)), dim3(256), 0, s, target, dw, d->Cout);
}

}  // namespace rn50
