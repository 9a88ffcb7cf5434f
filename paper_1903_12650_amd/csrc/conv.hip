// Convolution forward and data gradient as implicit GEMMs on
// the gfx950 matrix cores (v_mfma_f32_32x32x16_bf16 for bf16 storage,
// v_mfma_f32_32x32x2_f32 for float storage; float accumulation in both).
//
// Forward and data gradient share one kernel, igemm_kernel:
//     C[m][n] = sum_k A[m][k] * B[n][k]
// where row m is an output pixel, A is gathered on the fly from the NHWC
// activation tensor (k = tap*Cg + channel, 128 contiguous bytes per tap and row,
// zero outside the image), and B is the weight matrix with K contiguous
// (the KRSC weights as they are; in the data gradient K runs over the output channels, the
// weights' slow index, so its B tiles are [K][columns] and its fragments transposing LDS reads,
// as in the weight gradient: no transposed copy of the weights is made).
// 256 threads = 4 waves; both operands go straight into LDS (one
// barrier per 128-byte K chunk); each wave owns 32x32 MFMA tiles fed by 16-byte
// LDS reads; the MFMA is issued with the weight fragment as its first operand
// so that every lane ends up with 4 consecutive output channels of one pixel,
// which the epilogue packs, stages through LDS and stores as full rows.
//
// (The weight gradient is in wgrad.hip, the bf16 stem's forward pass in stem.hip.)
//
// The output stage of igemm_kernel can also take the per-channel sums of the
// batch norm that consumes the output (forward: sum and sum of squares about a
// shift of the tile's own, or about zero in double; data gradient: sum(g), sum(g*xhat) of the BN layer below, with an
// optional second gradient branch added before the one rounding), so that no
// separate pass re-reads the tensor.  Stride-2 data gradients process the output
// pixels in four parity classes, each looping over its own taps only.
#include <stdlib.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "common.h"
#include "conv_internal.h"
#include "step_internal.h"

namespace rn50 {

// ----------------------------------------------------------- small utilities
template <typename T> struct Mma;
template <> struct Mma<uint16_t> {  // bf16: one 32x32x16 MFMA per 16-byte fragment pair
  static __device__ __forceinline__ void run(const Vec16& a, const Vec16& b, f32x16& acc) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(&a),
                                                  *reinterpret_cast<const bf16x8*>(&b), acc, 0, 0, 0);
  }
};
template <> struct Mma<float> {  // float: four 32x32x2 MFMAs (k pairs {j, 4+j} of the 8 in flight)
  static __device__ __forceinline__ void run(const Vec16& a, const Vec16& b, f32x16& acc) {
#pragma unroll
    for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.f[j], b.f[j], acc, 0, 0, 0);
  }
};

// ------------------------------------------------- forward / dgrad implicit GEMM
struct IgemmArgs {
  const void* act;  // gathered activation tensor [N][H][W] pixels of PS elements
  const void* wgt;  // B: [Ncols][Ktot]
  void* out;        // C: [M][Ncols]
  int out_through;  // writes_through of its bytes
  uint32_t act_bytes, wgt_bytes;
  int M, Ncols, Ktot;
  int H, W;         // spatial size of the gathered tensor
  int P, Q;         // spatial size of the output pixel grid (M = N*P*Q)
  int PS;           // pixel stride of the gathered tensor, in elements
  int Cg;           // channels per tap
  int R, S, stride, pad;
  int cpt;          // 128-byte chunks per tap
  int ntn;          // number of column tiles
  int pair;         // stem in bf16: a 128-byte chunk holds two filter rows (pieces 0-3: row 2r, 4-7: row 2r+1)
  int nimg;         // images (M = nimg*P*Q)
  // Divisions of the tile / pixel decode by exact multiply-shift (an integer division costs a wave some 40
  // instructions, and every workgroup starts with several of them).  div_w / div_h: by the width / height of
  // the row tiles' pixel grid -- [1] for the odd parity class of a stride-2 data gradient.
  int mtiles;       // row tiles (grid = mtiles * ntn)
  FastDiv div_ntn, div_w[2], div_h[2];
  int mode;         // host side only: forward, data gradient, evaluation; selects the MODE template argument with `partial`
  // Optional batch-norm sums over the rows of each output tile, taken from the rounded values that are
  // stored (null: none), one row per tile row (bn_sums_at).  Forward: float sums of the values and of their squares about
  // the tile's first row.  Data gradient: sum(g), sum(g * xhat) with g the output
  // gradient masked by the ReLU of the BN layer whose conv output is bn_x [M][Ncols], xhat its
  // normalized input.
  float* partial;
  int partial_wide;  // forward: as doubles (bn_self_finalizes)
  unsigned long long* slots;  // (or null) one word per column, made empty for the pass that adds the sums up (BnShare)
  const void* bn_x;
  const float *bn_gamma, *bn_beta, *bn_mean, *bn_rstd;
  // Data gradient with sums only.  addend [M][Ncols] (or null): a second gradient branch, added to the
  // product in float before the one rounding to the storage type (the stored output is the sum).
  // bn_zmask (or null): the BN layer's recorded ReLU decision bits, one byte per 16-byte vector of its
  // output; without them the decision is recomputed from bn_x.
  // addend_mask (or null): the addend is the output gradient of a residual-add layer that is still
  // unmasked; it counts only where that layer's recorded ReLU bit is set (same byte layout as bn_zmask).
  const void* addend;
  const uint8_t* bn_zmask;
  const uint8_t* addend_mask;
  // The addend holds the pixels with even row and column only, [nimg][ceil(P/2)][ceil(Q/2)][Ncols]; it is zero elsewhere (the data
  // gradient of a 1x1 / stride 2 convolution; 1x1 / stride 1 launches, without addend_mask).
  int addend_even;
  // A 1x1 / stride 2 data gradient without sums: the tiles are those of the parity class that has the tap, and each of their
  // pixels stores the zeros of the other three classes' pixels beside it, in front of the main loop.  (Three of four workgroups
  // that only stored zeros had a tile's LDS and a tile's prologue each: 56x56 256 <- 512 at batch 40 29.9 -> 20.0 us, 223 -> 144 at
  // batch 256, 28x28 512 <- 1024 25.6 -> 17.2, 118 -> 103; with the zeros behind the products 23.6, 139, 17.7, 102.)
  int fill;
  // Forward, 1x1 / stride 1 only (BNIN kernels): the gathered tensor is the INPUT of a BN+ReLU layer, whose
  // relu(x*scale + bias) is applied to every operand vector once it sits in LDS (null: the tensor is used as is).
  // in_lds: byte offset of the per-channel coefficient table behind the ring (host side: lds bytes without it).
  const float *in_gamma, *in_beta, *in_mean, *in_rstd;
  int in_lds;
  // Forward with an inference-mode batch norm in the output stage (MODE 2): the output is
  // [relu](product * scale + bias [+ addend]), scale = bn_gamma / sqrt(aff_var + aff_eps), bias = bn_beta - bn_mean * scale,
  // from the float accumulators and rounded once; addend [M][Ncols] (or null) is the residual.
  const float* aff_var;
  float aff_eps;
  int aff_relu;
};

// MODE 0: forward gather  ih = p*stride - pad + r.
// MODE 1: data gradient with the batch-norm sums of the layer below.  MODE 3: without, a kernel of its own: in one for both, launches without sums
// held the registers of the sums' operands, a workgroup less per compute unit (bf16 128x128 224 registers, alone 128: 256 <- 64 at 56x56, batch 256
// 113 -> 92 us; 22 shapes, operands from memory, batch 256 3512 -> 3428 us, 40 709 -> 702; float at batch 24 2677 -> 2600).
// Their gather is  ih = (p + pad - r)/stride when divisible (stride 1 or 2).  With stride 2
// an output pixel only receives the taps r = (p + pad) mod 2, s = (q + pad) mod 2 (mod 2), so the pixels
// are processed in four parity classes (p mod 2, q mod 2): a row tile holds pixels of one class and loops
// over that class's taps only (a quarter of the taps on average, none for three classes of a 1x1 filter:
// IgemmArgs::fill).
// MODE 2: the forward gather with an inference-mode batch norm (+ residual, + ReLU) applied to the accumulators: an
// evaluation pass needs no statistics of the tensor it produces, so the separate pass that read y and wrote z (two
// thirds of the bytes of a 1x1 layer with its neighbours in HBM, and a third of the pass's time at batch 256) is gone.
// LIN: compiled for a 1x1 filter with stride 1 and no padding (output row m is pixel m of the gathered
// tensor): no pixel decode, no tap cursor, no bounds checks -- these layers have the shortest reductions
// of the network, and a workgroup's instruction count outside the main loop is what bounds them.
//
// Tile BM x BN, WM x WN waves (4 or 8), each wave a (BM/WM) x (BN/WN) tile of 32x32 MFMA blocks.  A 128-byte
// K chunk of the tile is (BM + BN) rows of 128 bytes in LDS, filled by buffer loads that write LDS directly
// (8 lanes per row, 8 rows per wave instruction) into a ring of three chunk buffers: the loads of chunk k+2 are
// issued when chunk k starts, one barrier per chunk.  Within a row the eight 16-byte pieces are stored
// permuted, piece p of row r in slot p ^ ((r >> 1) & 7): the MFMA fragment reads (lane = row, 16 bytes of one
// piece) then touch every bank once per 16 lanes.  What bounds the main loop per compute unit, measured:
// 16-byte vector loads deliver ~60 B/clk, 16-byte LDS reads ~220 B/clk, one 32x32x16 MFMA per SIMD every 32
// clocks.  A 32x32 wave tile reads 2 KB of fragments per MFMA (LDS-bound at half the MFMA rate), a 64x64
// wave tile 1 KB; a 64x64 workgroup tile loads 16 KB per 128 MFMA-clocks (load-bound at half the MFMA rate),
// a 128x128 tile 32 KB per 512.  Hence the largest tile that still gives every compute unit work is chosen
// per layer shape (igemm_tile below).
// Chunk buffers in the ring: three (loads two chunks ahead), or two where three would leave room for only one
// four-wave workgroup per compute unit (160 KB of LDS): two workgroups hide each other's barriers and latencies.
template <int BM, int BN, int NW>
constexpr int igemm_ring() {
  return (NW == 4 && 3 * (BM + BN) * 128 > 80 * 1024) ? 2 : 3;
}
// DEEP: the 128x128 tile of the evaluation pass and of the float forward pass, whose three whole buffers would leave a compute unit one workgroup, has
// three for A and two for B: 80 KB, two workgroups to the byte (so these kernels have no static LDS; MODE 2's coefficients lie behind the output
// tile).  A comes from memory, B, the weights, from the L2: with both one chunk ahead a chunk took as long as A's loads, 1.2 us.  Evaluation at batch
// 256 4.40 -> 4.28 ms, 64 1.331 -> 1.297; float forward, 23 shapes at batch 24 1308 -> 1287 us.  Not the data gradients: beside the weight gradients they
// leave them no LDS (step at batch 256 19.14 -> 19.18 ms when it was tried).
template <typename T, int BM, int BN, int WM, int WN, int MODE, bool BNIN, bool HALO>
constexpr bool igemm_deep_a() {
  return BM == 128 && BN == 128 && WM * WN == 4 && (MODE == 2 || (MODE == 0 && sizeof(T) == 4)) && !BNIN && !HALO;
}
// LEAN: the same tile's training forward in bf16 has two buffers for A and one for B, 48 KB: three workgroups per compute unit (at most 168 registers; no
// static LDS).  What these layers are short of is not depth but another workgroup: a workgroup's products and its output stage, which
// writes most of the bytes, take as long as each other and two workgroups do not keep them side by side (256 -> 1024 at 14x14, batch 256: 29 us without the
// output stage, 24 without the products, 58 together).  B, from the L2, is requested behind the barrier that ends its last reading, a wait that
// the other two workgroups cover.  With sums, from memory, DEEP -> LEAN at batch 256: 256 -> 1024 at 14x14 57.8 -> 50.7 us, 128 -> 512 at 28x28 92.7 -> 80.3,
// 512 -> 256 at 28x28 82.7 -> 76.8, 1024 -> 512 at 14x14 70.5 -> 64.6; step 18540 -> 18440.  Not the evaluation pass (160 registers and more, with a
// residual 69 KB: two workgroups; 4180 -> 4240 us) and not float (an output tile of 68 KB).
template <typename T, int BM, int BN, int WM, int WN, int MODE, bool BNIN, bool HALO>
constexpr bool igemm_lean_b() {
  return BM == 128 && BN == 128 && WM * WN == 4 && MODE == 0 && sizeof(T) == 2 && !BNIN && !HALO;
}
// PAIRED: the 128x128 tile's halo loop.  Its two runs and two weight tiles (three everywhere else) are at most 80 KB up to images 31 wide, so
// two workgroups share a compute unit (no static LDS; the output stage's coefficients lie behind its tile; at most 256 registers, in both types).  A step takes a pair as long as
// the 256x128 tile's one workgroup (0.75 to 0.85 us, 0.46 of it products), but a rest of the grid that gives each unit a single workgroup
// takes little more than half a round, where the taller tile takes a whole one, and the two cover each other's prologue and output stage
// (5 us of a round): see igemm_halo_tile.
template <int BM, int BN, int WM, int WN>
constexpr bool igemm_halo_paired() { return BM == 128 && BN == 128 && WM * WN == 4; }
template <int BM, int BN>
constexpr int igemm_out_tile() { return BM * (BN * 4 + 16); }  // the output tile in float, with its pitch
// KS (launched with WM = WN = 1): the four waves of a workgroup split K instead of the tile.  Every wave computes the whole
// BM x BN tile over a quarter of the chunks, with a ring of its own that it fills and reads without any barrier; at the end
// the four partial tiles are added in wave order through LDS.  For grids that leave compute units idle or give each a single
// workgroup: there a chunk costs the latency of its loads (0.35 us per chunk in the shared ring, whose depth is bounded
// by LDS), and four independent rings take four of these latencies at a time; the wave tile is also the whole tile, so
// fragments are read from LDS once (64x64: half the bytes per MFMA of four 32x32 waves).  Buffers per wave:
template <int BM, int BN, bool BNIN>
constexpr int igemm_ks_ring() {
  return BNIN || BM + BN > 96 ? 2 : (BM + BN > 64 ? 3 : 4);
}
// The halo loop by filter rows (TAPS = 3, below): steps by which the weights of a row are requested ahead.  One row where two
// workgroups share a compute unit (the LDS for more is the other one's), and in float, whose products take longer than a load; three
// where a workgroup has it alone in bf16 (512 -> 512 at 7x7, batch 40: 16.6 us, with one row 21.6; float at batch 8 34.6 with three, 31.5
// with one).
template <typename T, bool KS>
constexpr int igemm_row_ahead() { return KS && sizeof(T) == 2 ? 3 : 1; }
//
// Data gradient (MODE 1 and 3): the B tile of a chunk is BK output channels (K) x BN input channels of the weights as they lie
// in memory, filled and read like wgrad_kernel's tiles (transposing reads in bf16).  A transposing read delivers fewer
// bytes per clock than a plain one, but the tile is the smaller half of the fragment traffic and was never what bounds
// these layers: per layer at batch 40 7.5 to 33 us against 8.9 to 34 with a transposed copy (whole network 794 against
// 854 us, 3884 against 3926 at batch 256), and the copy itself -- 4 to 5 us per conv_dgrad call, 57 us per step on the
// side stream -- is gone (the 22 shapes at batch 40, call by call: 562 -> 465 us).
//
// HALO: compiled for a 3x3 filter with stride 1 and padding 1 (output pixel m reads input pixels m + dy*W + dx,
// dy, dx in -1..1, of the same flat pixel index space).  The nine taps of a tile then read one contiguous run of
// BM + 2W + 2 input pixels: that run is brought into LDS once per 128-byte channel chunk (instead of a gathered
// BM-row tile per tap: nine times the operand traffic), and the fragment reads of tap (dy, dx) start dy*W + dx rows
// further down in it.  Taps that fall off the image (or into the neighbouring image of the run) are zeroed in
// the fragment registers, by a per-lane bit mask computed once.  The weights go through a ring of three
// BN-row tiles, two taps ahead; the next chunk's run is loaded one pass per tap while the
// current one is in use, so that every step issues the same number of loads (the load waits count them).  (PAIRED: two weight
// tiles, one tap ahead, and a step with or without a pass of the next run behind them.)
//
// TAPS: taps between two barriers, 1 or 3 (0: no halo).  With small tiles a tap is a few MFMAs per wave between a barrier, the
// fragment reads' latency and the issue of the next loads; three taps, a filter row, share these.  By rows run
//  - the tiles of grids of at most 256 of 64x64, whose four waves split K (KS): every wave multiplies the whole tile with one 32-byte
//    quarter of every chunk, so a fragment is read from LDS once, weights and run are loaded once per workgroup (own rings gathered
//    nine times the run), and the weights come three rows ahead;
//  - the 64x64 tile of 2x2 waves as long as two workgroups per compute unit hold the grid (512) and their LDS fits.
// Forward, tap by tap -> by rows, us: bf16 256 -> 256 at 14x14, batch 40 15.7 -> 14.3 (2x2 waves), 16 13.0 -> 10.0, 8 9.5 -> 7.7, 4 9.0 -> 7.4;
// 512 -> 512 at 7x7, batch 40 20.9 -> 16.6, 16 14.8 -> 12.2, 4 13.8 -> 11.2; 64 -> 64 at 56x56, batch 4 8.1 -> 5.4; float 256 -> 256 at 14x14,
// batch 8 35.7 -> 25.4, 512 -> 512 at 7x7, batch 16 65 -> 48.  Data gradients alike.  At more than 512 tiles the third workgroup on a compute
// unit is worth more (512 -> 512 at 7x7, batch 90, 552 tiles: 32.2 us, by rows 37.7).
template <typename T, int BM, int BN, int WM, int WN, int MODE, bool LIN, bool BNIN, int TAPS, bool THROUGH>
__global__ __launch_bounds__(WM * WN == 1 ? 256 : 64 * WM * WN) void igemm_kernel(const IgemmArgs a) {
  static_assert(!BNIN || (LIN && MODE == 0), "the input-side BN is compiled for the linear forward kernel only");
  constexpr bool HALO = TAPS > 0;
  static_assert(!HALO || (!LIN && !BNIN), "the halo main loop is a kernel of its own");
  constexpr bool DG = MODE == 1 || MODE == 3, FWD = !DG, AFF = MODE == 2, DGS = MODE == 1, DGP = MODE == 3;
  constexpr bool KS = WM * WN == 1;
  constexpr bool OWN = KS && !HALO;             // every wave has chunks and a ring of its own (halo: they share run and weights)
  constexpr int NW = KS ? 4 : WM * WN, NT = 64 * NW;
  constexpr int LT = OWN ? 64 : NT;              // threads that fill a chunk buffer together
  constexpr int V = 16 / sizeof(T);
  constexpr int BK = 128 / sizeof(T);
  constexpr int RPL = LT / 8;                   // tile rows covered by one load pass
  constexpr int RA = BM / RPL, RB = BN / RPL;  // load passes (= load instructions per thread and chunk)
  constexpr int NL = RA + RB;
  constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
  constexpr int STAGE = (BM + BN) * 128;
  constexpr bool DEEP = igemm_deep_a<T, BM, BN, WM, WN, MODE, BNIN, HALO>();
  constexpr bool LEAN = igemm_lean_b<T, BM, BN, WM, WN, MODE, BNIN, HALO>();
  constexpr bool PAIRED = HALO && igemm_halo_paired<BM, BN, WM, WN>();
  constexpr int NSTAGE = OWN ? igemm_ks_ring<BM, BN, BNIN>() : igemm_ring<BM, BN, WM * WN>();
  constexpr int CP = BN * sizeof(T) + 16;  // epilogue pitch
  static_assert((NW == 4 || NW == 8) && TM >= 1 && TN >= 1 && RA >= 1 && RB >= 1, "tile shape");
  static_assert(BM % RPL == 0 && BN % RPL == 0, "every load pass covers whole rows of the tile");
  constexpr int CPW = BN * 4 + 16;         // pitch of a float output tile (bf16 data gradient with an addend)
  // (the launch sizes the dynamic LDS as the larger of the ring and what the output stage stores in it)
  extern __shared__ __align__(16) unsigned char smem[];

  request_kernel_args<sizeof(IgemmArgs)>();
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int lt = OWN ? lane : tid, slot = lt & 7, lrow = lt >> 3;
  const int piece0 = slot ^ ((lrow >> 1) & 7);  // the 16-byte piece of its rows' chunk this thread fetches
  // (KS: passes are 8 rows apart, which moves bit 2 of the permutation from one to the next)
  auto piece_of = [&](int i) __attribute__((always_inline)) { return OWN ? piece0 ^ ((i & 1) << 2) : piece0; };
  const int wm = KS ? 0 : wave % WM, wn = KS ? 0 : wave / WM;
  const int bid = xcd_remap(blockIdx.x, gridDim.x);
  const int mt = static_cast<int>(fdiv(static_cast<uint32_t>(bid), a.div_ntn)), nt = bid - mt * a.ntn;
  const int n0 = nt * BN;
  const rsrc_words rsA = make_rsrc_words(a.act, a.act_bytes), rsB = make_rsrc_words(a.wgt, a.wgt_bytes);
  if (!AFF && a.slots != nullptr && mt == 0 && tid < BN && n0 + tid < a.Ncols) a.slots[n0 + tid] = kBnSlotEmpty;

  // Rows of this tile: pixels m0.. of the whole output grid, or of one parity class of it.
  const bool classes = !LIN && !HALO && DG && a.stride == 2;
  __shared__ int pix_s[BM];  // classes only: output pixel index of every tile row
  // Data gradient with batch-norm sums: the per-channel coefficients of this tile's columns, fetched by one
  // thread per column while the main loop runs (every thread loading its own copies costs the texture path
  // as much as two chunks of the main loop).
  // (MODE 2: the same for the inference-mode affine step.)
  float* prm_s;
  if constexpr (DEEP || PAIRED) {
    prm_s = reinterpret_cast<float*>(smem + igemm_out_tile<BM, BN>());
  } else {
    __shared__ __align__(16) float prm_static[DGS ? 4 * BN : (AFF ? 2 * BN : 4)];
    prm_s = prm_static;
  }
  float pg = 0.f, pb = 0.f, pm = 0.f, pr = 0.f;
  if ((AFF || DGS) && tid < BN) {
    const int c = min(n0 + tid, a.Ncols - 1);
    pg = a.bn_gamma[c]; pb = a.bn_beta[c]; pm = a.bn_mean[c]; pr = AFF ? a.aff_var[c] : a.bn_rstd[c];
  }
  int ph = 0, pw = 0, Hc = a.P, Wc = a.Q, Mc = a.M, m0 = mt * BM;
  int r0 = 0, s0 = 0, tstep = 1;
  if (classes) {
    // the four classes of one pixel range are neighbours in the tile order: they read the same rows of
    // the incoming gradient, and every XCD gets its share of the classes that have taps.  An XCD hands its workgroups to its
    // 32 compute units in turn, so in one fixed order a compute unit would have tiles of one class only, four taps or one; the
    // order changes every 32 workgroups, each second time to the opposite one (two tiles of a compute unit have five or four
    // taps together).  3x3 / 2 data gradients, 128 -> 128 at 56x56 and 256 -> 256 at 28x28: batch 40 24.1 -> 22.1 and 19.5 -> 18.2
    // us, float at batch 8 41.0 -> 33.9 and 42.6 -> 35.7, batch 256 157 -> 148 and 108 -> 107 (turned by one class each time
    // 22.6 and 18.6, 34.4 and 35.9, 144 and 109).
    const int turn = (mt >> 2) * a.ntn >> 3;
    const bool fill = DGP && a.fill;
    const int cls = fill ? 0 : (mt & 3) ^ ((turn & 1) * 3) ^ ((turn >> 1) & 1);
    m0 = (fill ? mt : mt >> 2) * BM;
    ph = cls >> 1; pw = cls & 1;
    Hc = (a.P - ph + 1) >> 1; Wc = (a.Q - pw + 1) >> 1;
    Mc = a.nimg * Hc * Wc;
    r0 = (ph + a.pad) & 1; s0 = (pw + a.pad) & 1; tstep = 2;
  }
  const int nr = r0 < a.R ? (a.R - r0 + tstep - 1) >> (tstep - 1) : 0, ns = s0 < a.S ? (a.S - s0 + tstep - 1) >> (tstep - 1) : 0;
  FastDiv dvw, dvh;  // selected field by field, by value
  dvw.mul = pw ? +a.div_w[1].mul : +a.div_w[0].mul; dvw.sh1 = pw ? +a.div_w[1].sh1 : +a.div_w[0].sh1; dvw.sh2 = pw ? +a.div_w[1].sh2 : +a.div_w[0].sh2;
  dvh.mul = ph ? +a.div_h[1].mul : +a.div_h[0].mul; dvh.sh1 = ph ? +a.div_h[1].sh1 : +a.div_h[0].sh1; dvh.sh2 = ph ? +a.div_h[1].sh2 : +a.div_h[0].sh2;

  // per-thread rows of the A tile: decode the output pixel once
  int a_h0[RA], a_w0[RA], a_base[RA];
#pragma unroll
  for (int i = 0; i < RA; ++i) {
    const int m = m0 + lrow + RPL * i;
    const bool ok = m < Mc;
    const int mm = ok ? m : 0;
    if constexpr (LIN) {  // no pixel decode: "image" base mm, coordinates (0, 0)
      a_base[i] = mm;
      a_h0[i] = ok ? 0 : -(1 << 20);
      a_w0[i] = 0;
      continue;
    }
    const int t = static_cast<int>(fdiv(static_cast<uint32_t>(mm), dvw));
    int q = mm - t * Wc;
    const int n = static_cast<int>(fdiv(static_cast<uint32_t>(t), dvh));
    int p = t - n * Hc;
    if (classes) {
      p = 2 * p + ph; q = 2 * q + pw;
      // (fill: with whether there is a pixel to the right, below; pixel numbers are below 2^28)
      if (slot == 0) pix_s[lrow + RPL * i] = ok ? ((n * a.P + p) * a.Q + q) | (q + 1 < a.Q ? 1 << 29 : 0) | (p + 1 < a.P ? 1 << 30 : 0) : 0;
    }
    a_base[i] = n * a.H * a.W;
    // a row beyond the last gets coordinates that fail every bounds check below
    a_h0[i] = ok ? (FWD ? p * a.stride - a.pad : p + a.pad) : -(1 << 20);
    a_w0[i] = FWD ? q * a.stride - a.pad : q + a.pad;
  }
  // What the output stage reads besides the tile: the BN layer's input, the second branch, recorded ReLU bits.  EARLY: requested
  // here, in front of everything the main loop loads (the hand-placed load waits count in order, and these are the oldest), so
  // that it is there when the last product is: workgroups of an earlier round are not enough to cover the 2 us these loads take from memory.
  // Step at batch 12 2395 -> 2375 us, 40 4161 -> 4134, 64 5852 -> 5809 (all against the 128x128 tile alone, which had given 4271 -> 4190 and at
  // batch 256 19024 -> 18840).  The operands take 20 to 90 registers through the main loop; from three chunks on LDS allows no more workgroups per
  // compute unit than are left (two of 128 rows, three of 64x64), with one or two chunks it is one or two workgroups less, and still the faster form
  // (256 <- 64 at 56x56 with a second branch, batch 256 257 -> 235 us).  Not the paired 128x128 tiles (three data gradients at 28x28, batch 256
  // 250 -> 325 us) and tiles of more than eight rows a thread (float, 128 columns or 256 rows), which it would leave a single workgroup.  These request the
  // operands in front of the rows that use them, eight rows at a time: with all sixteen at once they needed more than 256 registers, a single
  // workgroup too (22 float data gradients at batch 24, with sums / with a second branch 2895 / 3050 -> 2820 / 2975 us; 128 <- 128 3x3 / 2 at 56x56
  // 120 -> 92).
  constexpr int PPR = BN * sizeof(T) / 16;  // 16-byte pieces per output row
  constexpr int RPP = NT / PPR;             // rows per pass
  constexpr int NPASS = BM / RPP;
  constexpr bool EARLY = KS || AFF || (!PAIRED && NPASS <= 8);
  constexpr int GROUP = EARLY ? NPASS : std::min(NPASS, 8);  // rows whose operands are requested together
  static_assert(NPASS % GROUP == 0, "whole groups of rows");
  const int op = tid % PPR, orow = tid / PPR;
  const int n = n0 + op * V;
  const bool col_ok = n < a.Ncols;
  Vec16 xv[DGS ? NPASS : 1], av[DGS || AFF ? NPASS : 1];
  uint32_t zb[DGS ? NPASS : 1], ab[DGS ? NPASS : 1];
  auto pixel = [&](int row) __attribute__((always_inline)) { return pix_s[row] & ((1 << 29) - 1); };
  auto load_output_operands = [&](int first) __attribute__((always_inline)) {
    if (AFF && a.addend == nullptr) return;
    const T* add = static_cast<const T*>(a.addend);
    const int nc = col_ok ? n : 0;
    auto pixel_of = [&](int pass) __attribute__((always_inline)) {
      const int row = orow + pass * RPP;
      return classes ? pixel(row) : min(m0 + row, a.M - 1);  // rows past the last read a valid pixel
    };
    // (one loop per operand: a test of a pointer per row is a branch per row, and no load passes a branch; byte offsets are 31-bit)
    const int last = first + GROUP;
    uint32_t at[NPASS];
#pragma unroll
    for (int pass = first; pass < last; ++pass) at[pass] = static_cast<uint32_t>(pixel_of(pass)) * static_cast<uint32_t>(a.Ncols) + nc;
    if constexpr (DGS) {
#pragma unroll
      for (int pass = first; pass < last; ++pass) xv[pass] = load16(static_cast<const T*>(a.bn_x) + at[pass]);
      if (a.bn_zmask) {
#pragma unroll
        for (int pass = first; pass < last; ++pass) zb[pass] = a.bn_zmask[at[pass] / V];
      }
      if (a.addend_mask) {
#pragma unroll
        for (int pass = first; pass < last; ++pass) ab[pass] = a.addend_mask[at[pass] / V];
      } else {
#pragma unroll
        for (int pass = first; pass < last; ++pass) ab[pass] = 0xffu;
      }
    }
    if constexpr (DGS && LIN) {
      if (add && a.addend_even) {
#pragma unroll
        for (int pass = first; pass < last; ++pass) {
          const int px = pixel_of(pass);
          const uint32_t t = fdiv(static_cast<uint32_t>(px), a.div_w[0]), w = static_cast<uint32_t>(px) - t * a.Q;
          const uint32_t img = fdiv(t, a.div_h[0]), h = t - img * a.P;
          const int64_t e = (static_cast<int64_t>(img) * ((a.P + 1) >> 1) + (h >> 1)) * ((a.Q + 1) >> 1) + (w >> 1);
          av[pass].u = make_uint4(0, 0, 0, 0);
          if (((h | w) & 1) == 0) av[pass] = load16_stream(add + e * a.Ncols + nc);
        }
        return;
      }
    }
    if (add) {
#pragma unroll
      for (int pass = first; pass < last; ++pass) av[pass] = load16_stream(add + at[pass]);  // (its last reader)
    }
  };
  if constexpr ((DGS || AFF) && EARLY) {
    if (classes) __syncthreads();  // (pix_s)
    load_output_operands(0);
  }
  if (DGP && !LIN && !HALO && a.fill) {  // (stores in front of the loads only make the hand-placed waits stricter)
    __syncthreads();
#pragma unroll
    for (int pass = 0; pass < NPASS; ++pass) {
      const int row = orow + pass * RPP;
      if (m0 + row < Mc && col_ok) {
        const bool right = pix_s[row] & (1 << 29), below = pix_s[row] & (1 << 30);
        Vec16 zero;
        zero.u = make_uint4(0, 0, 0, 0);
        const OutTensor<T, THROUGH> out(static_cast<T*>(a.out), a.out_through);
        const int64_t at = static_cast<int64_t>(pixel(row)) * a.Ncols + n, next_row = static_cast<int64_t>(a.Q) * a.Ncols;
        if (right) out.store(at + a.Ncols, zero);
        if (below) out.store(at + next_row, zero);
        if (right && below) out.store(at + next_row + a.Ncols, zero);
      }
    }
  }
  // The B tile: BN rows (output columns) of one 128-byte chunk of K each, or (data gradient) BK rows (K) of BN columns.
  constexpr int BRB = BN * static_cast<int>(sizeof(T)), LB = BRB / 16;  // data gradient: bytes and 16-byte pieces per tile row
  const int b_krow = DG ? lt / LB : 0;                                 // ... this thread's tile row in load pass 0
  const int k_pitch = a.R * a.S * a.Ncols;                              // ... elements from one K row of the weights to the next
  uint32_t b_row[RB];
#pragma unroll
  for (int i = 0; i < RB; ++i) {
    if constexpr (DG) {
      const int col = n0 + ((lt % LB) ^ wgrad_swz<T, BRB>(b_krow + (LT / LB) * i)) * V;
      b_row[i] = col < a.Ncols ? static_cast<uint32_t>((b_krow + (LT / LB) * i) * k_pitch + col) * sizeof(T) : kOob;
    } else {
      const int n = n0 + lrow + RPL * i;
      b_row[i] = n < a.Ncols ? static_cast<uint32_t>(n * a.Ktot + piece_of(i) * V) * sizeof(T) : kOob;
    }
  }
  // byte offset of (tap, chunk cc) in the weights, and whether load pass i brings anything (cval: the forward pass's answer)
  auto b_at = [&](int tap, int cc) __attribute__((always_inline)) {
    return DG ? static_cast<uint32_t>(cc * BK * k_pitch + tap * a.Ncols) * static_cast<uint32_t>(sizeof(T))
              : static_cast<uint32_t>(tap * a.Cg) * static_cast<uint32_t>(sizeof(T)) + static_cast<uint32_t>(cc) * 128u;
  };
  auto b_live = [&](int i, int cc, bool cval) __attribute__((always_inline)) {
    return DG ? (a.Cg % BK == 0 || cc * BK + b_krow + (LT / LB) * i < a.Cg) : cval;
  };

  // Load cursor: tap (r,s), chunk cc within the tap.  Per tap, the byte offset of every row's pixel (or
  // kOob); within a tap successive chunks only differ by a scalar offset.
  const int allchunks = nr * ns * a.cpt;
  int cur_r = r0, cur_s = s0, cur_cc = 0, cur = 0;
  int nchunks = allchunks, first_chunk = 0;  // this wave's (KS) or the workgroup's range of chunks
  if constexpr (OWN) {
    const int w = __builtin_amdgcn_readfirstlane(wave);
    first_chunk = (allchunks * w) >> 2;
    nchunks = ((allchunks * (w + 1)) >> 2) - first_chunk;
    if (LIN) {
      cur_cc = first_chunk;
    } else if (nchunks > 0) {
      const int tap = first_chunk / a.cpt;
      cur_cc = first_chunk - tap * a.cpt;
      cur_r = r0 + tstep * (tap / ns);
      cur_s = s0 + tstep * (tap % ns);
    }
  }
  uint32_t a_off[RA];
  int b_tap = cur_r * a.S + cur_s;
  const bool ragged = (a.Cg % BK) != 0;
  auto tap_setup = [&]() __attribute__((always_inline)) {
    if constexpr (LIN) {
#pragma unroll
      for (int i = 0; i < RA; ++i)
        a_off[i] = a_h0[i] < 0 ? kOob : static_cast<uint32_t>(a_base[i] * a.PS + piece_of(i) * V) * sizeof(T);
      return;
    }
#pragma unroll
    for (int i = 0; i < RA; ++i) {
      const int piece = piece_of(i);
      int ih, iw;
      bool ok = true;
      if (FWD) {
        ih = a_h0[i] + (a.pair ? 2 * cur_r + (piece >> 2) : cur_r);
        iw = a_w0[i] + cur_s;
      } else {
        const int th = a_h0[i] - cur_r, tw = a_w0[i] - cur_s;
        const int msk = a.stride - 1;  // stride is 1 or 2
        ok = th >= 0 && tw >= 0 && ((th | tw) & msk) == 0;
        ih = th >> msk;
        iw = tw >> msk;
      }
      ok = ok && static_cast<unsigned>(ih) < static_cast<unsigned>(a.H) &&
           static_cast<unsigned>(iw) < static_cast<unsigned>(a.W);
      const int pc = (FWD && a.pair) ? (piece & 3) : piece;
      a_off[i] = ok ? static_cast<uint32_t>((a_base[i] + ih * a.W + iw) * a.PS + pc * V) * sizeof(T) : kOob;
    }
  };
  // One chunk into one ring buffer: every wave fills its 8 rows of each load pass (1 KB per instruction).
  typedef __attribute__((address_space(3))) unsigned char* lds_byte_ptr;
  const uint32_t wave_dst = __builtin_amdgcn_readfirstlane(
      static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_byte_ptr)smem)) + static_cast<uint32_t>(wave) * (OWN ? NSTAGE * STAGE : 1024u));
  // A's part moves the cursor on and leaves what B's part of the same chunk needs: B's may follow one chunk later (DEEP).
  uint32_t sob = 0;
  int b_cc = 0;
  auto load_a = [&](uint32_t sa) __attribute__((always_inline)) {
    const uint32_t so = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(cur_cc) * 128u);
    auto cval = [&](int i) __attribute__((always_inline)) { return !ragged || (cur_cc * BK + piece_of(i) * V < a.Cg); };
    ++cur;
    b_cc = cur_cc;
    sob = __builtin_amdgcn_readfirstlane(b_at(b_tap, cur_cc));
#pragma unroll
    for (int i = 0; i < RA; ++i) buffer_load16_to_lds(rsA, sa + i * (RPL * 128), cval(i) ? a_off[i] : kOob, so);
    // advance the cursor
    if constexpr (LIN) {
      ++cur_cc;
    } else if (++cur_cc == a.cpt) {
      cur_cc = 0;
      cur_s += tstep;
      if (cur_s >= a.S) {
        cur_s = s0;
        cur_r += tstep;
      }
      b_tap = cur_r * a.S + cur_s;
      if (cur < nchunks) tap_setup();  // (nothing is loaded past the last chunk)
    }
  };
  auto load_b = [&](uint32_t sb, int cc, uint32_t so) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < RB; ++i)
      buffer_load16_to_lds(rsB, sb + i * (RPL * 128), b_live(i, cc, !ragged || (cc * BK + piece_of(i) * V < a.Cg)) ? b_row[i] : kOob, so);
  };
  auto load_chunk = [&](int stage) __attribute__((always_inline)) {
    const uint32_t sa = wave_dst + static_cast<uint32_t>(stage) * STAGE;
    load_a(sa);
    load_b(sa + BM * 128, b_cc, sob);
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  // Fragment of a 32-row block for k step kk: row = lane % 32, piece 2*kk + lane/32, in its permuted slot
  // (the block starts at a multiple of 32 rows, so the permutation depends on the lane alone).
  int frag_off[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk)
    frag_off[kk] = (lane & 31) * 128 + (((2 * kk + (lane >> 5)) ^ ((lane >> 1) & 7)) << 4);
  // The fragment reads run ahead of the MFMAs that use them -- a whole chunk ahead for the small wave tiles
  // (one MFMA per k step is far shorter than an LDS read's latency), one k step ahead for 64x64 wave tiles --
  // so a wave pays the LDS latency once per chunk, not once per k step.
  int bt_base[TN];  // data gradient: the transposing reads of the [K][columns] tile
#pragma unroll
  for (int j = 0; j < TN; ++j) bt_base[j] = DG ? wgrad_frag_base<T, BRB>(lane, wn * (BN / WN) + j * 32) : 0;
  constexpr int AHEAD = (TM + TN <= 3) ? 4 : 1;  // k steps whose fragments are in registers before the first MFMA
  // `next` issues the loads that go out behind the first fragment reads.
  auto compute = [&](const unsigned char* tile_a, const unsigned char* tile_b, auto&& next) __attribute__((always_inline)) {
    const unsigned char* sa = tile_a + wm * (BM / WM) * 128;
    const unsigned char* sb = tile_b + (DG ? 0 : wn * (BN / WN) * 128);
    Vec16 fa[4][TM], fb[4][TN];
    auto read_frags = [&](int kk) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[kk][i].u = *reinterpret_cast<const uint4*>(sa + i * 32 * 128 + frag_off[kk]);
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        if constexpr (DG) fb[kk][j] = wgrad_read_frag<T, BRB>(sb, bt_base[j], kk);
        else fb[kk][j].u = *reinterpret_cast<const uint4*>(sb + j * 32 * 128 + frag_off[kk]);
      }
    };
#pragma unroll
    for (int kk = 0; kk < AHEAD; ++kk) read_frags(kk);
    __builtin_amdgcn_sched_barrier(0);  // (the instruction scheduler would sink every read to its first use)
    next();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      if (kk + AHEAD < 4) {
        read_frags(kk + AHEAD);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) Mma<T>::run(fb[kk][j], fa[kk][i], acc[i][j]);  // D'[n][m]
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // Ring of NSTAGE chunk buffers, loads NSTAGE-1 chunks ahead.  At the top of iteration kc this wave waits for
  // its own loads of chunk kc (those of the later chunks may still be in flight), then the barrier: behind it
  // every wave's part of chunk kc is in LDS and every wave is done reading chunk kc-1, whose buffer the loads
  // of chunk kc+NSTAGE-1 issued next will overwrite.
  if constexpr (HALO) {
    constexpr int NSB = 3;                       // weight tiles in the ring
    const int Wd = a.W;
    const int NA = (BM + 2 * Wd + 2 + RPL - 1) / RPL;  // load passes of one run (with another chunk to load: the host checked NA <= 8)
    const uint32_t run_bytes = static_cast<uint32_t>(NA) * (RPL * 128);
    const int cpt = a.cpt;
    const uint32_t b_base = (cpt > 1 ? 2u : 1u) * run_bytes;  // two runs when there is a next chunk to prefetch
    const uint32_t dump = b_base + NSB * BN * 128;          // where the loads that only keep the count go (zeros)
    const uint32_t lds0 = wave_dst;                           // LDS address of smem + this wave's 1 KB share of a pass
    const int q0 = m0 - Wd - 1 + lrow;                        // input pixel of this thread's row in pass 0 of a run
    const int piece = piece0;
    // (the addresses are uniform; in the loop of filter rows the compiler does not see it)
    auto uniform = [](uint32_t v) __attribute__((always_inline)) { return TAPS == 3 ? static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(v)) : v; };
    auto load_run_pass = [&](int j, int cc, int buf) __attribute__((always_inline)) {
      const int q = q0 + RPL * j;
      const bool ok = static_cast<unsigned>(q) < static_cast<unsigned>(a.M) && (!ragged || cc * BK + piece * V < a.Cg);
      const uint32_t off = ok ? static_cast<uint32_t>(q * a.PS + piece * V) * sizeof(T) : kOob;
      buffer_load16_to_lds(rsA, uniform(lds0 + static_cast<uint32_t>(buf) * run_bytes + static_cast<uint32_t>(j) * (RPL * 128)), off,
                           __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(cc) * 128u));
    };
    auto load_b_tile = [&](int stage, int cc, int tap, bool live) __attribute__((always_inline)) {
      const bool cval = !ragged || cc * BK + piece * V < a.Cg;
      const uint32_t sob = __builtin_amdgcn_readfirstlane(b_at(tap, cc));
#pragma unroll
      for (int i = 0; i < RB; ++i)
        buffer_load16_to_lds(rsB, uniform(lds0 + b_base + static_cast<uint32_t>(stage) * (BN * 128) + i * (RPL * 128)),
                             live && b_live(i, cc, cval) ? b_row[i] : kOob, sob);
    };
    auto load_nothing = [&]() __attribute__((always_inline)) { buffer_load16_to_lds(rsA, lds0 + dump, kOob, 0); };
    // Which taps of which rows exist: bit `tap` of vmask[i] for this lane's row of the wave's row block i.
    uint32_t vmask[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int m = m0 + wm * (BM / WM) + i * 32 + (lane & 31);
      const bool ok = m < a.M;
      const int mm = ok ? m : 0;
      const int t = static_cast<int>(fdiv(static_cast<uint32_t>(mm), a.div_w[0]));
      const int x = mm - t * a.Q;
      const int y = t - static_cast<int>(fdiv(static_cast<uint32_t>(t), a.div_h[0])) * a.P;
      uint32_t bits = 0;
#pragma unroll
      for (int tap = 0; tap < 9; ++tap) {
        const int dyo = FWD ? tap / 3 - 1 : 1 - tap / 3, dxo = FWD ? tap % 3 - 1 : 1 - tap % 3;
        const bool v = ok && static_cast<unsigned>(y + dyo) < static_cast<unsigned>(a.H) &&
                       static_cast<unsigned>(x + dxo) < static_cast<unsigned>(a.W);
        bits |= v ? (1u << tap) : 0u;
      }
      vmask[i] = bits;
    }
    // One tap's fragments, and their products.
    struct Frags {
      Vec16 a[4][TM], b[4][TN];
    };
    struct TapAddr {
      int a[4];
      const unsigned char *sa, *sb;
    };
    auto tap_addr = [&](int buf, int bslot, int tap) __attribute__((always_inline)) {
      const int dyo = FWD ? tap / 3 - 1 : 1 - tap / 3, dxo = FWD ? tap % 3 - 1 : 1 - tap % 3;
      const int rl = (lane & 31) + (dyo + 1) * Wd + (dxo + 1);  // row of the run this lane's row 0 reads
      const int swz = (rl >> 1) & 7;
      TapAddr r;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) r.a[kk] = rl * 128 + (((2 * kk + (lane >> 5)) ^ swz) << 4);
      r.sa = smem + static_cast<uint32_t>(buf) * run_bytes + wm * (BM / WM) * 128;
      r.sb = smem + b_base + bslot * (BN * 128) + (DG ? 0 : wn * (BN / WN) * 128);
      return r;
    };
    auto tap_read = [&](Frags& f, const TapAddr& at, int kk) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < TM; ++i) f.a[kk][i].u = *reinterpret_cast<const uint4*>(at.sa + i * 32 * 128 + at.a[kk]);
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        if constexpr (DG) f.b[kk][j] = wgrad_read_frag<T, BRB>(at.sb, bt_base[j], kk);
        else f.b[kk][j].u = *reinterpret_cast<const uint4*>(at.sb + j * 32 * 128 + frag_off[kk]);
      }
    };
    struct TapMask {
      uint32_t m[TM];
    };
    auto tap_mask = [&](int tap) __attribute__((always_inline)) {
      TapMask r;
#pragma unroll
      for (int i = 0; i < TM; ++i) r.m[i] = ((vmask[i] >> tap) & 1u) ? 0xffffffffu : 0u;
      return r;
    };
    auto masked_mma = [&](Vec16 (&fa)[TM], const Vec16 (&fb)[TN], const TapMask& mk) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        fa[i].u.x &= mk.m[i]; fa[i].u.y &= mk.m[i]; fa[i].u.z &= mk.m[i]; fa[i].u.w &= mk.m[i];
#pragma unroll
        for (int j = 0; j < TN; ++j) Mma<T>::run(fb[j], fa[i], acc[i][j]);
      }
    };
    // KS: a wave multiplies the whole tile with its quarter of every chunk (k step `wave`).
    struct FragsKw {
      Vec16 a[TM], b[TN];
    };
    const int kw_slot = 2 * wave + (lane >> 5);
    const int kw_boff = (lane & 31) * 128 + ((kw_slot ^ ((lane >> 1) & 7)) << 4);
    auto kw_read = [&](FragsKw& f, int buf, int bslot, int tap) __attribute__((always_inline)) {
      const int dyo = FWD ? tap / 3 - 1 : 1 - tap / 3, dxo = FWD ? tap % 3 - 1 : 1 - tap % 3;
      const int rl = (lane & 31) + (dyo + 1) * Wd + (dxo + 1);
      const int aoff = rl * 128 + ((kw_slot ^ ((rl >> 1) & 7)) << 4);
      const unsigned char* sa = smem + static_cast<uint32_t>(buf) * run_bytes;
      const unsigned char* sb = smem + b_base + bslot * (BN * 128);
#pragma unroll
      for (int i = 0; i < TM; ++i) f.a[i].u = *reinterpret_cast<const uint4*>(sa + i * 32 * 128 + aoff);
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        if constexpr (DG) f.b[j] = wgrad_read_frag<T, BRB>(sb, bt_base[j], wave);
        else f.b[j].u = *reinterpret_cast<const uint4*>(sb + j * 32 * 128 + kw_boff);
      }
    };
    if constexpr (TAPS == 3) {
      // A step is a filter row: three taps.  Its three weight tiles come D steps ahead into a ring of D + 1 slots, the next
      // chunk's run in the chunk's first steps.
      constexpr int D = igemm_row_ahead<T, KS>(), NSLOT = D + 1, LB3 = 3 * RB;
      constexpr int NA_MIN = (BM + 4 + RPL - 1) / RPL;  // load passes of a run, at least
      auto load_row = [&](int slot, int cc, int row, bool live) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 3; ++t) load_b_tile(3 * slot + t, cc, 3 * row + t, live);
      };
      for (int j = 0; j < NA; ++j) load_run_pass(j, 0, 0);
#pragma unroll
      for (int r = 0; r < D; ++r) load_row(r, 0, r, true);
      int slot = 0;
      for (int cc = 0; cc < cpt; ++cc) {
        const int buf = cc & 1;  // (one chunk: 0)
        const bool more = cc + 1 < cpt;
#pragma unroll
        for (int row = 0; row < 3; ++row) {
          // What this row reads has landed: its weights were requested D steps ago, behind which D - 1 steps of LB3 loads each and
          // (D = 3) the run's passes of this chunk's first step may be in flight.  Nobody reads the slot that is filled next any more.
          if (D == 3 && row > 0 && more) wait_loads_then_barrier<(D - 1) * LB3 + (D == 3 ? NA_MIN : 0)>();
          else wait_loads_then_barrier<(D - 1) * LB3>();
          auto load_next = [&]() __attribute__((always_inline)) {
            const int to = slot >= 1 ? slot - 1 : NSLOT - 1;
            if constexpr (D == 3) {
              load_row(to, cc + 1, row, more);  // (past the last chunk a load of nothing, for the count)
              if (row == 0 && more)
                for (int j = 0; j < NA; ++j) load_run_pass(j, cc + 1, buf ^ 1);
            } else {
              if (row < 2) load_row(to, cc, row + 1, true);
              else if (more) load_row(to, cc + 1, 0, true);
              if (more) {
#pragma unroll
                for (int j = 3 * row; j < 3 * row + 3; ++j)  // (nine passes at most; the host checked NA <= 8)
                  if (j < NA) load_run_pass(j, cc + 1, buf ^ 1);
              }
            }
          };
          if constexpr (KS) {
            FragsKw f[3];
            TapMask mk[3];
#pragma unroll
            for (int t = 0; t < 3; ++t) {
              kw_read(f[t], buf, 3 * slot + t, 3 * row + t);
              mk[t] = tap_mask(3 * row + t);
            }
            __builtin_amdgcn_sched_barrier(0);
            load_next();
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < 3; ++t) masked_mma(f[t].a, f[t].b, mk[t]);
            __builtin_amdgcn_sched_barrier(0);
          } else {
            load_next();
            Frags f[2];  // a tap's fragments are read while the tap before it is multiplied
            auto read_all = [&](Frags& to, int t) __attribute__((always_inline)) {
              const TapAddr at = tap_addr(buf, 3 * slot + t, 3 * row + t);
#pragma unroll
              for (int kk = 0; kk < 4; ++kk) tap_read(to, at, kk);
            };
            read_all(f[0], 0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < 3; ++t) {
              if (t < 2) read_all(f[(t + 1) & 1], t + 1);
              const TapMask mk = tap_mask(3 * row + t);
              __builtin_amdgcn_sched_barrier(0);
#pragma unroll
              for (int kk = 0; kk < 4; ++kk) masked_mma(f[t & 1].a[kk], f[t & 1].b[kk], mk);
              __builtin_amdgcn_sched_barrier(0);
            }
          }
          slot = slot == NSLOT - 1 ? 0 : slot + 1;
        }
      }
    } else {
      auto compute_tap = [&](int buf, int bstage, int tap) __attribute__((always_inline)) {
        Frags f;
        constexpr int AH = (TM + TN <= 3) ? 4 : 1;
        const TapAddr at = tap_addr(buf, bstage, tap);
        const TapMask mk = tap_mask(tap);
#pragma unroll
        for (int kk = 0; kk < AH; ++kk) tap_read(f, at, kk);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          if (kk + AH < 4) {
            tap_read(f, at, kk + AH);
            __builtin_amdgcn_sched_barrier(0);
          }
          masked_mma(f.a[kk], f.b[kk], mk);
          __builtin_amdgcn_sched_barrier(0);
        }
      };
      if constexpr (PAIRED) {
        // The weights come one tap ahead, and behind them a pass of the next chunk's run, which may stay in flight for one more tap:
        // it comes from memory, the weights from the L2.
        for (int j = 0; j < NA; ++j) load_run_pass(j, 0, 0);
        load_b_tile(0, 0, 0, true);
        int bstage = 0;
        bool pass_behind = false;  // the tap before requested a pass of the next run behind its weights
        for (int cc = 0; cc < cpt; ++cc) {
          const int buf = cpt > 1 ? (cc & 1) : 0;
          const bool more = cc + 1 < cpt;
#pragma unroll
          for (int tap = 0; tap < 9; ++tap) {
            if (pass_behind) wait_loads_then_barrier<1>();
            else wait_loads_then_barrier<0>();
            if (tap < 8 || more) load_b_tile(bstage ^ 1, tap < 8 ? cc : cc + 1, (tap + 1) % 9, true);  // the tile of the tap before: free again
            pass_behind = more && tap < NA;
            if (pass_behind) load_run_pass(tap, cc + 1, buf ^ 1);
            compute_tap(buf, bstage, tap);
            bstage ^= 1;
          }
        }
      } else {
        // Prologue: the first run, the weight tiles of steps 0 and 1.  Every step of the loop then issues RB + 1
        // loads (the weight tile two steps ahead; one pass of the next chunk's run, or a load of nothing), so at its
        // top "at most RB + 1 outstanding" means: everything up to the step before the previous one has landed.
        for (int j = 0; j < NA; ++j) load_run_pass(j, 0, 0);
        load_b_tile(0, 0, 0, true);
        load_b_tile(1, 0, 1, true);
        load_nothing();
        int bstage = 0;
        for (int cc = 0; cc < cpt; ++cc) {
          const int buf = cpt > 1 ? (cc & 1) : 0;
#pragma unroll
          for (int tap = 0; tap < 9; ++tap) {
            wait_loads_then_barrier<RB + 1>();
            const int tap2 = (tap + 2) % 9, cc2 = cc + (tap + 2 >= 9 ? 1 : 0);
            load_b_tile(bstage >= 1 ? bstage - 1 : NSB - 1, cc2, tap2, cc2 < cpt);  // the tile of step - 1: free again
            if (tap < NA && cc + 1 < cpt) load_run_pass(tap, cc + 1, buf ^ 1);
            else load_nothing();
            compute_tap(buf, bstage, tap);
            bstage = bstage == NSB - 1 ? 0 : bstage + 1;
          }
        }
      }
    }
    // (the loads still in flight carry nothing and land in the dump area or in weight tiles nobody reads again;
    // they are waited for before the output stage reuses LDS)
    wait_loads_then_barrier<0>();
  } else {
    tap_setup();
    float* const in_tab = reinterpret_cast<float*>(smem + (BNIN ? a.in_lds : 0));  // [2][nchunks * BK]: scale, bias
    if constexpr (BNIN) {
      const int kpad = allchunks * BK;
      for (int c = tid; c < kpad; c += NT) {
        float sc = 0.f, bi = 0.f;
        if (c < a.Cg) bn_coeffs(a.in_gamma[c], a.in_beta[c], a.in_mean[c], a.in_rstd[c], &sc, &bi);
        in_tab[c] = sc;
        in_tab[kpad + c] = bi;
      }
      __syncthreads();
    }
    if constexpr (DEEP) {
      // Buffers of 16 KB: B0 A0 A1 B1 A2 (a reduction of one chunk has the first two, of two the first four).  Chunk k: A was requested two
      // chunks ago, B one; behind the wait only A of chunk k + 1 may still be in flight.
      static_assert(!DEEP || BM == BN, "buffers of one size");
      auto buf_a = [](int i) __attribute__((always_inline)) { return static_cast<uint32_t>(i + 1 + (i >> 1)) * (BM * 128); };
      auto buf_b = [](int i) __attribute__((always_inline)) { return static_cast<uint32_t>(3 * i) * (BM * 128); };
      if (nchunks > 0) {
        load_a(wave_dst + buf_a(0));
        load_b(wave_dst + buf_b(0), b_cc, sob);
      }
      if (nchunks > 1) load_a(wave_dst + buf_a(1));
      int ia = 0;
      for (int kc = 0; kc < nchunks; ++kc) {
        if (kc + 1 < nchunks) wait_loads_then_barrier<RA>(); else wait_loads_then_barrier<0>();
        compute(smem + buf_a(ia), smem + buf_b(kc & 1), [&]() __attribute__((always_inline)) {
          if (kc + 1 < nchunks) load_b(wave_dst + buf_b((kc & 1) ^ 1), b_cc, sob);
          if (kc + 2 < nchunks) load_a(wave_dst + buf_a(ia >= 1 ? ia - 1 : 2));
        });
        ia = ia == 2 ? 0 : ia + 1;
      }
    } else if constexpr (LEAN) {
      // Buffers B A0 A1.  Chunk k: A was requested two chunks ago, B behind chunk k - 1's products; only A of chunk k + 1 may still be in flight.
      auto buf_a = [](int i) __attribute__((always_inline)) { return static_cast<uint32_t>(BN + i * BM) * 128; };
      if (nchunks > 0) {
        load_a(wave_dst + buf_a(0));
        load_b(wave_dst, b_cc, sob);
      }
      if (nchunks > 1) load_a(wave_dst + buf_a(1));
      for (int kc = 0; kc < nchunks; ++kc) {
        if (kc + 1 < nchunks) wait_loads_then_barrier<RA>(); else wait_loads_then_barrier<0>();
        compute(smem + buf_a(kc & 1), smem, [] {});
        if (kc + 1 < nchunks) {
          lds_reads_then_barrier();  // every wave's fragments of B and of this A are in registers
          load_b(wave_dst, b_cc, sob);
          if (kc + 2 < nchunks) load_a(wave_dst + buf_a(kc & 1));
        }
      }
    } else {
#pragma unroll
      for (int c = 0; c < NSTAGE - 1; ++c)
        if (c < nchunks) load_chunk(c);
      int stage = 0;
      for (int kc = 0; kc < nchunks; ++kc) {
        if constexpr (KS) {  // (nobody else reads this wave's buffers: the next loads go out before the wait)
          if (kc + NSTAGE - 1 < nchunks) load_chunk(stage >= 1 ? stage - 1 : NSTAGE - 1);
          ring_wait<NSTAGE + 1, NL, false>(nchunks - 1 - kc);
        } else {
          ring_wait<NSTAGE, NL>(nchunks - 1 - kc);
          if (kc + NSTAGE - 1 < nchunks) load_chunk(stage >= 1 ? stage - 1 : NSTAGE - 1);  // buffer (kc - 1) mod NSTAGE
        }
        if constexpr (BNIN) {
          // every thread transforms, in place, the vectors of chunk kc that its own loads brought (its slot of its
          // rows holds piece `piece`, i.e. channels kc*BK + piece*V ..), then a second barrier
          float scale[V], bias[V];
          const int kpad = allchunks * BK;
#pragma unroll
          for (int par = 0; par < (KS ? 2 : 1); ++par) {
            const int at = (first_chunk + kc) * BK + piece_of(par) * V;
            load_floats<V>(in_tab + at, scale);
            load_floats<V>(in_tab + kpad + at, bias);
#pragma unroll
            for (int i = par; i < RA; i += KS ? 2 : 1) {
              uint4* p = reinterpret_cast<uint4*>(smem + (OWN ? wave * (NSTAGE * STAGE) : 0) + stage * STAGE + (lrow + RPL * i) * 128 + slot * 16);
              Vec16 v;
              v.u = *p;
              *p = bn_relu_vector<T>(v, scale, bias).u;
            }
          }
          if (!KS) lds_writes_then_barrier();  // (KS: the wave's own LDS operations stay in order)
        }
        const unsigned char* const tile = smem + (OWN ? wave * (NSTAGE * STAGE) : 0) + stage * STAGE;
        compute(tile, tile + BM * 128, [] {});
        stage = stage == NSTAGE - 1 ? 0 : stage + 1;
      }
    }
  }
  if constexpr (KS) {
    // wave w takes rows g = w (four consecutive output channels) of every 32x32 block from the four partial tiles
    float4* red = reinterpret_cast<float4*>(smem);  // [wave][i][j][g][lane]
    __syncthreads();
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          red[(((wave * TM + i) * TN + j) * 4 + g) * 64 + lane] =
              make_float4(acc[i][j][g * 4], acc[i][j][g * 4 + 1], acc[i][j][g * 4 + 2], acc[i][j][g * 4 + 3]);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        float4 r[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) r[w] = red[(((w * TM + i) * TN + j) * 4 + wave) * 64 + lane];
        acc[i][j][0] = ((r[0].x + r[1].x) + r[2].x) + r[3].x;
        acc[i][j][1] = ((r[0].y + r[1].y) + r[2].y) + r[3].y;
        acc[i][j][2] = ((r[0].z + r[1].z) + r[2].z) + r[3].z;
        acc[i][j][3] = ((r[0].w + r[1].w) + r[2].w) + r[3].w;
      }
  }
  if constexpr (AFF) {
    if (DEEP) __syncthreads();  // (prm_s lies in the ring)
    if (tid < BN) {
      float sc, bi;
      bn_coeffs(pg, pb, pm, static_cast<float>(1.0 / sqrt(static_cast<double>(pr) + static_cast<double>(a.aff_eps))), &sc, &bi);
      prm_s[tid] = sc; prm_s[BN + tid] = bi;
    }
    lds_writes_then_barrier();
  } else if constexpr (KS) {
    __syncthreads();  // the output tile below reuses the exchange buffers
  } else if constexpr (DGS && EARLY) {
    // (every load has landed; the wait is for the compiler, which counts stores with loads and would wait for a row's operands behind the store of
    // the row before: 256 <- 64 at 56x56, batch 40 38 -> 35 us)
    wait_loads_then_barrier<0>();  // the output tile below reuses the pipeline buffers
  } else {
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  }

  // Epilogue.  acc[i][j][v]: output channel n = j*32 + (v/4)*8 + (lane/32)*4 + v%4, pixel m = i*32 + lane%32.
  // The tile goes to LDS in the storage type, or in float when a bf16 data gradient has an addend.
  // What a launch's output stage does is chosen once per workgroup, with a copy of the loops each: tests inside them were two branches per
  // element, 130 a wave and tile in data gradients with sums (with sums at batch 256: 64 <- 64 3x3 at 56x56 113 -> 99 us; 128 <- 128 3x3 at 28x28
  // 93 -> 86).  The forward sums keep their one test per row: with rows past the end added as zeros instead 30 layers at batch 256 1905 -> 1950 us.
  const bool wide = sizeof(T) == 2 && (AFF || DGS) && a.addend != nullptr;
  auto stage_tile = [&](auto wide_tile, auto relu) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int row = wm * (BM / WM) + i * 32 + (lane & 31);
#pragma unroll
        for (int g0 = 0; g0 < (KS ? 1 : 4); ++g0) {
          const int g = KS ? wave : g0;
          const int col = wn * (BN / WN) + j * 32 + g * 8 + (lane >> 5) * 4;
          unsigned char* dst = smem + row * CP + col * sizeof(T);
          float4 v = make_float4(acc[i][j][g0 * 4 + 0], acc[i][j][g0 * 4 + 1], acc[i][j][g0 * 4 + 2], acc[i][j][g0 * 4 + 3]);
          if constexpr (AFF) {
            const float4 sc = *reinterpret_cast<const float4*>(prm_s + col), bi = *reinterpret_cast<const float4*>(prm_s + BN + col);
            v = make_float4(bn_affine(v.x, sc.x, bi.x), bn_affine(v.y, sc.y, bi.y), bn_affine(v.z, sc.z, bi.z), bn_affine(v.w, sc.w, bi.w));
            if (decltype(relu)::value) v = make_float4(fmaxf(v.x, 0.f), fmaxf(v.y, 0.f), fmaxf(v.z, 0.f), fmaxf(v.w, 0.f));
          }
          if (decltype(wide_tile)::value) *reinterpret_cast<float4*>(smem + row * CPW + col * 4) = v;
          else if (sizeof(T) == 2) *reinterpret_cast<uint2*>(dst) = make_uint2(float2_to_bf16x2_bits(v.x, v.y), float2_to_bf16x2_bits(v.z, v.w));
          else *reinterpret_cast<float4*>(dst) = v;
        }
      }
  };
  if (AFF && a.aff_relu && !a.addend) stage_tile(std::false_type{}, std::bool_constant<AFF>{});
  else if ((AFF || DGS) && sizeof(T) == 2 && wide) stage_tile(std::bool_constant<(AFF || DGS) && sizeof(T) == 2>{}, std::false_type{});
  else stage_tile(std::false_type{}, std::false_type{});
  if (DGS && tid < BN) {
    float sc, bi;
    bn_coeffs(pg, pb, pm, pr, &sc, &bi);
    prm_s[tid] = sc; prm_s[BN + tid] = bi; prm_s[2 * BN + tid] = pr; prm_s[3 * BN + tid] = -pm * pr;
  }
  __syncthreads();
  const OutTensor<T, THROUGH> out(static_cast<T*>(a.out), a.out_through);
  if constexpr (AFF) {
    if (a.addend != nullptr) {
      auto rows = [&](auto relu, auto whole) __attribute__((always_inline)) {
#pragma unroll
        for (int pass = 0; pass < NPASS; ++pass) {
          const int row = orow + pass * RPP, m = m0 + row;
          float r[V], t[V];
          Elem<T>::unpack(av[pass], r);
          load_floats<V>(reinterpret_cast<const float*>(smem + row * CPW) + op * V, t);
#pragma unroll
          for (int j = 0; j < V; ++j) {
            t[j] += r[j];
            if (decltype(relu)::value) t[j] = fmaxf(t[j], 0.f);
          }
          Vec16 o;
          Elem<T>::pack(t, o);
          if (decltype(whole)::value || (m < Mc && col_ok)) out.store(static_cast<int64_t>(m) * a.Ncols + n, o);
        }
      };
      // (a tile without rows or columns past the last stores without a test per row, which kept the LDS reads of a row behind the store of the
      // one before: evaluation at batch 256 4380 -> 4260 us; not worth a copy of the stage without a residual, 4260 -> 4253)
      const bool whole = m0 + BM <= Mc && n0 + BN <= a.Ncols;
      if (a.aff_relu) {
        if (whole) rows(std::true_type{}, std::true_type{});
        else rows(std::true_type{}, std::false_type{});
      } else {
        rows(std::false_type{}, std::false_type{});
      }
      return;
    }
  }
  if (AFF || DGP || (MODE == 0 && a.partial == nullptr)) {
#pragma unroll
    for (int pass = 0; pass < NPASS; ++pass) {
      const int row = orow + pass * RPP;
      const int m = m0 + row;
      if (m < Mc && n < a.Ncols) {
        const int pix = classes ? pixel(row) : m;
        Vec16 v;
        v.u = *reinterpret_cast<const uint4*>(smem + row * CP + op * 16);
        out.store(static_cast<int64_t>(pix) * a.Ncols + n, v);
      }
    }
    return;
  }

  // Output stage with batch-norm sums: every thread owns V channels and NPASS rows of the tile.
  float s1[V], s2[V];
#pragma unroll
  for (int j = 0; j < V; ++j) s1[j] = s2[j] = 0.f;
  if (MODE == 0) {
    float shift[V];
    Vec16 k0;
    k0.u = *reinterpret_cast<const uint4*>(smem + op * 16);  // row m0 of the tile always exists
    Elem<T>::unpack(k0, shift);
#pragma unroll
    for (int pass = 0; pass < NPASS; ++pass) {
      const int row = orow + pass * RPP;
      const int m = m0 + row;
      if (m < Mc && col_ok) {
        Vec16 v;
        v.u = *reinterpret_cast<const uint4*>(smem + row * CP + op * 16);
        out.store(static_cast<int64_t>(m) * a.Ncols + n, v);
        float f[V];
        Elem<T>::unpack(v, f);
#pragma unroll
        for (int j = 0; j < V; ++j) {
          const float d = f[j] - shift[j];
          s1[j] += d;
          s2[j] = fmaf(d, d, s2[j]);
        }
      }
    }
  } else if constexpr (DGS) {
    float scale[V], bias[V], rs[V], nmr[V];
#pragma unroll
    for (int j = 0; j < V; ++j) {
      scale[j] = prm_s[op * V + j]; bias[j] = prm_s[BN + op * V + j];
      rs[j] = prm_s[2 * BN + op * V + j]; nmr[j] = prm_s[3 * BN + op * V + j];
    }
    // masked: the BN layer's recorded ReLU bits are there; added: a second branch; whole: no row or column of the tile is past the last (a test
    // per row is a branch per row: step at batch 256 18.28 -> 18.20 ms without them; the forward sums gain nothing by it)
    // (opaque: where a launch may have no bits the compiler would move what is made of them up to their loads, in front of the main loop, and wait there)
    auto opaque = [](uint32_t bits) __attribute__((always_inline)) {
      if constexpr (EARLY) asm("" : "+v"(bits));
      return bits;
    };
    auto rows = [&](auto masked, auto added, auto whole) __attribute__((always_inline)) {
#pragma unroll
      for (int pass = 0; pass < NPASS; ++pass) {
        if (!EARLY && pass % GROUP == 0) {
          if (pass > 0) __builtin_amdgcn_sched_barrier(0);  // (the scheduler would request a group in front of the one before, and hold both)
          load_output_operands(pass);
        }
        const int row = orow + pass * RPP;
        if (!decltype(whole)::value && !(m0 + row < Mc && col_ok)) continue;  // (its operands are another pixel's: not even zero times them)
        Vec16 v;
        float g[V], xf[V];
        if constexpr (decltype(added)::value) {
          float ad[V];
          Elem<T>::unpack(keep_bits<T>(av[pass], opaque(ab[pass])), ad);
          // (in bf16 the tile lies in LDS in float)
          load_floats<V>(reinterpret_cast<const float*>(smem + row * (sizeof(T) == 2 ? CPW : CP)) + op * V, g);
#pragma unroll
          for (int j = 0; j < V; ++j) g[j] += ad[j];
          Elem<T>::pack(g, v);
        } else {
          v.u = *reinterpret_cast<const uint4*>(smem + row * CP + op * 16);
        }
        const int pix = classes ? pixel(row) : m0 + row;
        out.store(static_cast<int64_t>(pix) * a.Ncols + n, v);
        if constexpr (decltype(masked)::value) v = keep_bits<T>(v, opaque(zb[pass]));
        Elem<T>::unpack(v, g);  // the sums range over the stored (rounded) values
        Elem<T>::unpack(xv[pass], xf);
#pragma unroll
        for (int j = 0; j < V; ++j) {
          const float gm = decltype(masked)::value || bn_affine(xf[j], scale[j], bias[j]) > 0.f ? g[j] : 0.f;
          s1[j] += gm;
          s2[j] = fmaf(gm, fmaf(xf[j], rs[j], nmr[j]), s2[j]);
        }
      }
    };
    auto form = [&](auto masked, auto added) __attribute__((always_inline)) {
      if (m0 + BM <= Mc && n0 + BN <= a.Ncols) rows(masked, added, std::true_type{});
      else rows(masked, added, std::false_type{});
    };
    if (a.bn_zmask) {
      if (a.addend) form(std::true_type{}, std::true_type{});
      else form(std::true_type{}, std::false_type{});
    } else {
      if (a.addend) form(std::false_type{}, std::true_type{});
      else form(std::false_type{}, std::false_type{});
    }
  }
  // The per-thread sums of a column meet through LDS: [row group][plane][column], over the tile buffer
  // (every thread is done with its rows of the tile), then one thread per plane and column adds the RPP row
  // groups in order.  (Wave shuffles here -- 6 * V of them per thread -- cost more than the whole loop above.)
  float kshift = 0.f;
  if (MODE == 0 && tid < BN) kshift = Elem<T>::load(reinterpret_cast<const T*>(smem) + tid);  // row m0 of the tile
  __syncthreads();
  float* cs = reinterpret_cast<float*>(smem);
  static_assert(2 * BN <= NT && NPASS >= 1, "one thread per plane and column");
#pragma unroll
  for (int j = 0; j < V; j += 4) {
    *reinterpret_cast<float4*>(cs + (orow * 2 + 0) * BN + op * V + j) = make_float4(s1[j], s1[j + 1], s1[j + 2], s1[j + 3]);
    *reinterpret_cast<float4*>(cs + (orow * 2 + 1) * BN + op * V + j) = make_float4(s2[j], s2[j + 1], s2[j + 2], s2[j + 3]);
  }
  __syncthreads();
  if (MODE == 0) {
    // one thread per column
    if (tid < BN && n0 + tid < a.Ncols) {
      float t1 = 0.f, t2 = 0.f;
#pragma unroll 8
      for (int r = 0; r < RPP; ++r) {
        t1 += cs[(r * 2 + 0) * BN + tid];
        t2 += cs[(r * 2 + 1) * BN + tid];
      }
      const int64_t at = bn_sums_at(mt, n0 + tid, a.mtiles);
      if (a.partial_wide) reinterpret_cast<double2*>(a.partial)[at] = bn_tile_sums(kshift, t1, t2, min(BM, Mc - m0));
      else reinterpret_cast<BnTileRow*>(a.partial)[at] = BnTileRow{kshift, t1, t2};
    }
    return;
  }
  if (tid < 2 * BN) {
    const int pl = tid & 1, ch = tid >> 1;
    float t = 0.f;
#pragma unroll 8
    for (int r = 0; r < RPP; ++r) t += cs[(r * 2 + pl) * BN + ch];
    if (n0 + ch < a.Ncols) a.partial[2 * bn_sums_at(mt, n0 + ch, a.mtiles) + pl] = t;
  }
}

// ------------------------------------------------------- layout helper kernels
// Stem input: x [N][H][W][3] -> xp [N][H+6][Wp][4], zero border (3 pixels each side, Wp - W - 3 on the
// right) and zero 4th channel, so that a 7-tap filter row is 8 pixels = 32 contiguous elements.
template <typename T>
__global__ __launch_bounds__(256) void stem_pad_input_kernel(const T* __restrict__ x, T* __restrict__ xp,
                                                             int N, int H, int W, int Hp, int Wp) {
  // grid: (padded row, padded rows, images)
  const int wq = blockIdx.x * 256 + threadIdx.x;
  if (wq >= Wp) return;
  const int hq = blockIdx.y, n = blockIdx.z;
  const int64_t i = (static_cast<int64_t>(n) * Hp + hq) * Wp + wq;
  const int h = hq - 3, w = wq - 3;
  T v[4] = {0, 0, 0, 0};
  if (h >= 0 && h < H && w >= 0 && w < W) {
    const T* s = x + ((static_cast<int64_t>(n) * H + h) * W + w) * 3;
    v[0] = s[0]; v[1] = s[1]; v[2] = s[2];
  }
  T* d = xp + i * 4;
  d[0] = v[0]; d[1] = v[1]; d[2] = v[2]; d[3] = v[3];
}
// Stem weights: w [K][7][7][3] -> wp [K][8][8][4] with zeros in filter row 7, tap column 7 and channel 3.
template <typename T>
__global__ __launch_bounds__(256) void stem_pad_weight_kernel(const T* __restrict__ w, T* __restrict__ wp, int K) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= K * kStemK) return;
  const int c = i & 3, s = (i >> 2) & 7, r = (i >> 5) & 7, k = i >> 8;
  wp[i] = (c < 3 && s < 7 && r < 7) ? w[((k * 7 + r) * 7 + s) * 3 + c] : static_cast<T>(0);
}
// ------------------------------------------------------------------ host side
template <typename T, int BM, int BN, int WM, int WN, int MODE, bool LIN, bool BNIN, bool THROUGH>
static void launch_igemm_through(IgemmArgs a, const char* tag, int64_t grid, hipStream_t s) {
  constexpr bool KS = WM * WN == 1;
  constexpr int NT = KS ? 256 : 64 * WM * WN;
  constexpr int stage = (BM + BN) * 128 * (KS ? 4 : 1);  // (KS: every wave has a ring)
  constexpr int es = static_cast<int>(sizeof(T));
  // the output stage reuses the ring: the tile (in float when a bf16 data gradient adds a second branch) and
  // the column sums of the fused batch norm
  constexpr bool deep = igemm_deep_a<T, BM, BN, WM, WN, MODE, BNIN, false>();
  constexpr int col_sums = (NT / (BN * es / 16)) * 2 * BN * 4;
  constexpr int exchange = KS ? 4 * BM * BN * 4 : 0;     // (KS: the four partial tiles)
  constexpr int behind = deep ? 2 * BN * 4 : 0;          // (behind the output tile: MODE 2's coefficients)
  constexpr int out_most = std::max({igemm_out_tile<BM, BN>() + behind, col_sums, exchange});
  static std::once_flag once;
  constexpr int deep_ring = (2 * BN + 3 * BM) * 128;
  constexpr bool lean = igemm_lean_b<T, BM, BN, WM, WN, MODE, BNIN, false>();
  constexpr int lean_ring = (BN + 2 * BM) * 128;
  static_assert(!deep || (deep_ring <= 80 * 1024 && out_most <= deep_ring), "two workgroups per compute unit");
  static_assert(!lean || 3 * std::max({lean_ring, BM * (BN * es + 16), col_sums}) <= 160 * 1024, "three workgroups per compute unit");
  constexpr int nring = KS ? igemm_ks_ring<BM, BN, BNIN>() : igemm_ring<BM, BN, WM * WN>();
  // input-side BN coefficients: two floats per channel, at most 4096 channels (KS: 2048)
  constexpr int kInTabMax = 8 * (KS ? 2048 : 4096);
  std::call_once(once, [] {
    allow_big_lds(igemm_kernel<T, BM, BN, WM, WN, MODE, LIN, BNIN, 0, THROUGH>,
                  std::max({nring * stage, out_most, deep ? deep_ring : 0}) + (BNIN ? kInTabMax : 0));
  });
  // A short reduction never touches the later ring buffers, and an output tile in the storage type is half as large as in float; with
  // less LDS more workgroups fit a CU (the 1x1 layers with 64 channels, the largest pixel counts of the net, have a single chunk).
  const int chunks = a.R * a.S * a.cpt;
  const int ring = deep ? (chunks >= 3 ? deep_ring : chunks * stage) : lean ? (chunks >= 2 ? lean_ring : stage) : (!KS && chunks < nring ? (chunks < 1 ? 1 : chunks) : nring) * stage;
  const bool wide = es == 2 && (MODE == 2 || (MODE == 1 && a.addend != nullptr));
  const int out_need = std::max({(wide ? igemm_out_tile<BM, BN>() : BM * (BN * es + 16)) + behind, col_sums, exchange});
  int lds = ring > out_need ? ring : out_need;
  if (BNIN) {
    a.in_lds = lds;
    lds += 8 * a.R * a.S * a.cpt * (128 / es);
  }
  RN50_LAUNCH(tag, (igemm_kernel<T, BM, BN, WM, WN, MODE, LIN, BNIN, 0, THROUGH>), dim3(static_cast<unsigned>(grid)), dim3(NT), lds, s, a);
}
// Tiles of 128 columns: the rules give them to outputs of 6.6 MB and more (384 tiles of 128 rows, 192 of 256, by more than 64 columns;
// smaller ones only with a few rows by tens of thousands of columns), so they are compiled for outputs that are written through.
template <int BN>
constexpr bool igemm_always_through() { return BN > 64; }
template <typename T, int BM, int BN, int WM, int WN, int MODE, bool LIN, bool BNIN = false>
static void launch_igemm_mode(const IgemmArgs& a, const char* tag, int64_t grid, hipStream_t s) {
  if constexpr (!igemm_always_through<BN>()) {
    if (!a.out_through) return launch_igemm_through<T, BM, BN, WM, WN, MODE, LIN, BNIN, false>(a, tag, grid, s);
  }
  launch_igemm_through<T, BM, BN, WM, WN, MODE, LIN, BNIN, true>(a, tag, grid, s);
}
// The halo kernel (3x3, stride 1, padding 1): LDS bytes of its main loop for an image width, or 0 when the shape
// does not fit it (a run of more than 8 load passes where there is another chunk whose run is loaded beside this one's taps, more LDS than a
// compute unit has).
static bool igemm_halo_shape(const IgemmArgs& a);
// (the kernel's static arrays come on top; a compute unit has 160 KB, for two workgroups by rows with 2x2 waves)
constexpr int kHaloLdsMax = 152 * 1024, kHaloRowLdsMax = 78 * 1024, kHaloRowGroups = 512, kHaloPairLdsMax = 80 * 1024;
template <typename T, int BM, int BN, int WM, int WN>
static int halo_lds_bytes(int W, int cpt, int taps) {
  constexpr bool KS = WM * WN == 1;
  constexpr int NW = WM * WN == 1 ? 4 : WM * WN, RPL = NW * 8;
  const int passes = (BM + 2 * W + 2 + RPL - 1) / RPL;
  if (passes > 8 && (cpt > 1 || BM != 256 || BN != 64)) return 0;  // (a chunk's taps load the next one's run)
  const int runs = (cpt > 1 ? 2 : 1) * passes * RPL * 128;
  if (igemm_halo_paired<BM, BN, WM, WN>()) return runs + 2 * BN * 128 <= kHaloPairLdsMax ? runs + 2 * BN * 128 : 0;
  const int bytes = runs + (taps == 3 ? 3 * (igemm_row_ahead<T, KS>() + 1) * BN * 128 : 3 * BN * 128 + NW * 1024);
  return bytes <= (taps == 3 && !KS ? kHaloRowLdsMax : kHaloLdsMax) ? bytes : 0;
}
template <typename T, int BM, int BN, int WM, int WN, int MODE, int TAPS, bool THROUGH>
static void launch_igemm_halo_through(IgemmArgs a, const char* tag, int64_t grid, int main_lds, hipStream_t s) {
  constexpr bool KS = WM * WN == 1;
  constexpr int NT = KS ? 256 : 64 * WM * WN;
  constexpr int es = static_cast<int>(sizeof(T));
  constexpr int out_tile = igemm_out_tile<BM, BN>();
  constexpr int col_sums = (NT / (BN * es / 16)) * 2 * BN * 4;
  constexpr int exchange = KS ? 4 * BM * BN * 4 : 0;     // (KS: the four partial tiles)
  constexpr bool paired = igemm_halo_paired<BM, BN, WM, WN>();
  constexpr int behind = paired ? (MODE == 1 ? 4 : 2) * BN * 4 : 0;  // (the output stage's coefficients)
  constexpr int out_need = std::max({out_tile + behind, col_sums, exchange});
  static_assert(!paired || out_need <= kHaloPairLdsMax, "two workgroups per compute unit");
  static std::once_flag once;
  std::call_once(once, [] { allow_big_lds(igemm_kernel<T, BM, BN, WM, WN, MODE, false, false, TAPS, THROUGH>, kHaloLdsMax); });
  const int lds = main_lds > out_need ? main_lds : out_need;
  RN50_LAUNCH(tag, (igemm_kernel<T, BM, BN, WM, WN, MODE, false, false, TAPS, THROUGH>), dim3(static_cast<unsigned>(grid)), dim3(NT), lds, s, a);
}
template <typename T, int BM, int BN, int WM, int WN, int MODE, int TAPS>
static void launch_igemm_halo(const IgemmArgs& a, const char* tag, int64_t grid, int main_lds, hipStream_t s) {
  if constexpr (!igemm_always_through<BN>()) {
    if (!a.out_through) return launch_igemm_halo_through<T, BM, BN, WM, WN, MODE, TAPS, false>(a, tag, grid, main_lds, s);
  }
  launch_igemm_halo_through<T, BM, BN, WM, WN, MODE, TAPS, true>(a, tag, grid, main_lds, s);
}
template <typename T, int BM, int BN, int WM, int WN, int TAPS>
static void launch_igemm_halo_mode(const IgemmArgs& a, const char* tag, int64_t grid, int main_lds, hipStream_t s) {
  if (a.mode == 2) launch_igemm_halo<T, BM, BN, WM, WN, 2, TAPS>(a, tag, grid, main_lds, s);
  else if (a.mode == 0) launch_igemm_halo<T, BM, BN, WM, WN, 0, TAPS>(a, tag, grid, main_lds, s);
  else if (a.partial) launch_igemm_halo<T, BM, BN, WM, WN, 1, TAPS>(a, tag, grid, main_lds, s);
  else launch_igemm_halo<T, BM, BN, WM, WN, 3, TAPS>(a, tag, grid, main_lds, s);
}
// Tuning builds can force any tile on any layer; the product compiles what the rules below can choose.
#ifdef RN50_TUNING
constexpr bool kTuning = true;
#else
constexpr bool kTuning = false;
#endif
template <typename T, int BM, int BN, int WM, int WN>
static void launch_igemm_cfg(IgemmArgs a, const char* tag, hipStream_t s) {
  a.ntn = static_cast<int>(ceil_div(a.Ncols, BN));
  a.nimg = a.M / (a.P * a.Q);
  // stride-2 data gradient: four parity classes of the output pixels, each with its own row tiles
  const int64_t tiles_per_class = ceil_div(static_cast<int64_t>(a.nimg) * ((a.P + 1) / 2) * ((a.Q + 1) / 2), BM);
  const bool classes = a.mode == 1 && a.stride == 2;
  a.fill = classes && a.R == 1 && a.S == 1 && a.partial == nullptr;
  a.mtiles = static_cast<int>(classes ? (a.fill ? 1 : 4) * tiles_per_class : ceil_div(a.M, BM));
  const int64_t grid = static_cast<int64_t>(a.mtiles) * a.ntn;
  a.out_through = writes_through(static_cast<int64_t>(a.M) * a.Ncols * sizeof(T), igemm_always_through<BN>() ? 0 : kConvThroughBytes);
  a.partial_wide = bn_self_finalizes(a.mtiles, false);
  a.div_ntn = make_fastdiv(a.ntn);
  // 1x1 filter, stride 1, no padding: row m of the output is pixel m of the gathered tensor
  const bool linear = a.R == 1 && a.S == 1 && a.stride == 1 && a.pad == 0 && !a.pair && a.H == a.P && a.W == a.Q;
  for (int c = 0; c < 2; ++c) {
    a.div_w[c] = make_fastdiv(classes ? (a.Q - c + 1) >> 1 : a.Q);
    a.div_h[c] = make_fastdiv(classes ? (a.P - c + 1) >> 1 : a.P);
  }
  if (linear) {
    if constexpr (BM <= 128 || kTuning) {  // (the tiles of 256 rows are igemm_halo_tile's alone)
      if (a.mode == 1 && a.partial) launch_igemm_mode<T, BM, BN, WM, WN, 1, true>(a, tag, grid, s);
      else if (a.mode == 1) launch_igemm_mode<T, BM, BN, WM, WN, 3, true>(a, tag, grid, s);
      else if (a.mode == 2) launch_igemm_mode<T, BM, BN, WM, WN, 2, true>(a, tag, grid, s);
      else if (a.in_gamma) launch_igemm_mode<T, BM, BN, WM, WN, 0, true, true>(a, tag, grid, s);
      else launch_igemm_mode<T, BM, BN, WM, WN, 0, true>(a, tag, grid, s);
    }
    return;
  }
  if (igemm_halo_shape(a)) {
    if constexpr (BM <= 64) {  // by filter rows
      const int lds = WM * WN == 1 || grid <= kHaloRowGroups ? halo_lds_bytes<T, BM, BN, WM, WN>(a.W, a.cpt, 3) : 0;
      if (lds) return launch_igemm_halo_mode<T, BM, BN, WM, WN, 3>(a, tag, grid, lds, s);
    }
    if constexpr (WM * WN > 1) {
      const int lds = halo_lds_bytes<T, BM, BN, WM, WN>(a.W, a.cpt, 1);
      if (lds) return launch_igemm_halo_mode<T, BM, BN, WM, WN, 1>(a, tag, grid, lds, s);
    }
  }
  if constexpr (BM != 256 || BN != 64 || kTuning) {  // (igemm_halo_tile takes the 256x64 tile where its run fits)
    if (a.mode == 2) launch_igemm_mode<T, BM, BN, WM, WN, 2, false>(a, tag, grid, s);
    else if (a.mode == 0) launch_igemm_mode<T, BM, BN, WM, WN, 0, false>(a, tag, grid, s);
    else if (a.partial) launch_igemm_mode<T, BM, BN, WM, WN, 1, false>(a, tag, grid, s);
    else launch_igemm_mode<T, BM, BN, WM, WN, 3, false>(a, tag, grid, s);
  }
}

// Tile per layer shape.  The compiled shapes: rows x columns of the workgroup tile, waves along rows x columns.
struct TileShape {
  int bm, bn, wm, wn;
};
#define RN50_IGEMM_SHAPES(X) X(64, 64, 2, 2) X(128, 64, 2, 2) X(256, 64, 4, 1) X(128, 128, 2, 2) X(256, 128, 4, 2) X(64, 64, 1, 1)
#define RN50_IGEMM_SHAPE_BF16(X) X(32, 64, 1, 1)
#define RN50_IGEMM_SHAPE_F32(X) X(32, 32, 1, 1)
// The tile of a layer shape: M rows (output pixels; of one parity class for a stride-2 data gradient, `live` of
// whose four classes have any taps), Ncols output channels, `chunks` 128-byte steps of the reduction.  The rule
// is fitted to per-layer sweeps of all compiled shapes over ResNet-50's 23 convolution shapes at batch 40 and at
// batch 256 (profiles/conv_tile_sweep_*.txt: summed over the shapes within 1 % of the best tiles): the largest tile that still leaves about one and a half
// workgroups per compute unit wins -- larger tiles load fewer operand bytes per flop (the main loop's bound) but with a smaller
// grid the latencies of a workgroup's load -> LDS -> MFMA chain are exposed; a reduction of one chunk has nothing to reuse and
// takes the smallest tile (64 -> 64 at 56x56, batch 256, forward / data gradient 28.5 / 28.4 us against 29.1 / 29.0 with 128x64 and 31.2 / 31.4 with
// 128x128), except in bf16 with more than 64 columns and kCover tiles of 128x128 or more: that one reads A half as often.  By what the
// output stage does, 64 channels at 56x56, operands from memory, us, 64x64 -> 128x128 (profiles/conv_one_chunk_tile_sweep.txt):
//  - forward, with its sums (118 registers and 35 KB: four workgroups per compute unit): 64 -> 256 at batch 18 / 40 / 256 11.6 -> 8.6 / 25.5 ->
//    19.8 / 152 -> 98.  Every size, also from warm caches;
//  - data gradient without sums (128 registers: four): 8.7 -> 7.2 / 22.3 -> 17.6 / 129 -> 91 (warm 7.3 -> 6.5 / 13.2 -> 12.6 / 135 -> 92);
//  - data gradient with sums (225 registers: two), evaluation (158 registers and 69 KB: two): from an output of half the last-level cache on.  Data
//    gradient with sums at batch 40 / 100 / 256 35.0 -> 32.2 / 80.6 -> 71.5 / 199 -> 175; with a second branch, whose tile lies in LDS in float, the
//    128x64 tile of the same rows of sums is a little faster still (101 -> 93.4, 128x128 97.0 / 253 -> 232, 234); evaluation with the residual at batch
//    16 / 40 / 64 / 100 / 256 9.8 -> 12.0 / 23.9 -> 27.6 / 37 -> 43 / 66 -> 64 / 169 -> 149.  (The line was drawn where data gradients with sums lost
//    below it too, before their operands were requested early; now 128x64 and 128x128 are 6 to 8 % faster there as well, from batch 18 on.)
// In float the products take longer than the loads and the tile (68 KB in LDS) leaves two workgroups: 32 -> 256 at batch 64 with sums 61 -> 67, from
// warm caches 45 -> 61.
enum class TileUse { kForward, kAffine, kGrad, kGradSums, kGradSumsAdd };  // what the output stage does (MODE 0, 2, 3, 1, 1)
constexpr int64_t kOneChunkBytes = 128 << 20;
static TileShape igemm_tile(int64_t M, int Ncols, int chunks, bool strided_dgrad, int live, TileUse use, int dtype) {
  const int64_t classes = strided_dgrad ? live : 1;
  auto groups = [&](int bm, int bn) { return ceil_div(M, bm) * ceil_div(Ncols, bn) * classes; };
  constexpr int64_t kCover = 384;  // workgroups: one and a half per compute unit (two four-wave workgroups fit each)
  // (not the eight-wave 256x128 tile, also in the largest data gradients, which had it from 1536 tiles on: 22 shapes at batch 256
  // 3668 -> 3504 us without it, 128 1812 -> 1775; in the step at batch 256 19.49 -> 19.31 ms)
  if (Ncols > 64 && groups(128, 128) >= kCover) {
    const int64_t out_bytes = M * (strided_dgrad ? 4 : 1) * Ncols * 2;  // (asked in bf16)
    const bool large = use == TileUse::kForward || use == TileUse::kGrad || out_bytes >= kOneChunkBytes;
    if (chunks > 1) return TileShape{128, 128, 2, 2};
    if (dtype == RN50_BF16 && large) return use == TileUse::kGradSumsAdd ? TileShape{128, 64, 2, 2} : TileShape{128, 128, 2, 2};
  }
  if (chunks >= 8 && groups(128, 64) >= kCover) return TileShape{128, 64, 2, 2};
  return TileShape{64, 64, 2, 2};
}
// The tile of a 3x3 / stride 1 / padding 1 layer, which runs the halo main loop (forward and data gradient
// alike): fitted to sweeps of the compiled shapes over ResNet-50's four such layers at batch 40 and 256.  The
// eight-wave 256x128 tile, or two 128x128 ones per compute unit (PAIRED), once the former gives three quarters of the compute units a
// workgroup, else 128x64 while that leaves one and a half workgroups per compute unit, else 64x64.
constexpr int kHaloTallWidth = 63, kHaloPairWidth = 31;
// Of the two tiles of 128 columns, whether the paired one: where it fills fewer rounds of the grid.  A round of either takes about as long (bf16: 36 steps
// 33 us, 18 18 us; float nine times that); 256x128 tiles make ceil(tiles / 256) of them, pairs tiles / 512 and for the rest one more, or 0.55 of one where
// it leaves every compute unit a single tile at most.  us, forward / data gradient, 256x128 -> pairs (profiles/conv_halo_pairs_sweep.txt), bf16: 128 -> 128
// at 28x28, batch 256 (4 rounds, 3.55) 77.2 / 82.0 -> 65.2 / 67.2, 200 (3, 2.55) 55.7 / 58.2 -> 47.6 / 47.6, 90 (2, 1.55) 35.2 / 36.1 -> 28.4 / 28.8; 256 ->
// 256 at 14x14, 200 (2, 1.55) 59.8 / 62.1 -> 49.2 / 50.6.  Float likewise: 128 -> 128, 256 611 / 589 -> 509 / 510, 90 291 / 290 -> 219 / 224; 256 -> 256,
// 200 574 / 570 -> 433 / 438.  At equal rounds the two are within 5 % of each other: bf16 in one round the taller (512 -> 512 at 7x7, batch 256 56.0 /
// 60.6 -> 58.4 / 60.1; 128 -> 128 with sums, 64 19.8 -> 20.6), in two and more, and float, the pairs (128 -> 128, 128 36.7 / 37.6 -> 35.3 / 35.9; float 296 / 295
// -> 287 / 288); the taller one, which loads its weights half as often, stays.
static bool igemm_halo_pairs(int64_t tall, int64_t pairs) {  // (tiles of 256 and of 128 rows)
  const int64_t rest = pairs % 512;
  return 20 * (pairs / 512) + (rest == 0 ? 0 : rest <= 256 ? 11 : 20) < 20 * ceil_div(tall, 256);
}
static TileShape igemm_halo_tile(int64_t M, int Ncols, int cpt, int W) {
  auto groups = [&](int bm, int bn) { return ceil_div(M, bm) * ceil_div(Ncols, bn); };
  // One chunk of channels into at most 64 columns: four waves of 64x64 one above the other read two thirds of the fragment bytes per product
  // of the 128x64 tile's 64x32 waves, and a run of 256 + 2W + 2 pixels with its weights still leaves a compute unit two workgroups
  // (kHaloTallWidth: 12 load passes).  64 -> 64 at 56x56, us, forward / data gradient: batch 256 89.8 / 102.4 -> 67.3 / 74.2, 90 34.4 / 39.3 ->
  // 28.0 / 30.5, 40 16.1 / 18.5 -> 12.4 / 15.1, 32 15.4 / 18.2 -> 11.7 / 13.7.  In float, whose products are the bound, it is the rounds of the grid
// that decide, two workgroups against three of the 128x64 tile (32 -> 64 forward, batch 32 46.7 -> 40.2, 64 81 -> 81, 128 149 -> 138; 63x63, batch 40 59 -> 62, 64
// 94 -> 83).
  if (Ncols <= 64 && cpt == 1 && W <= kHaloTallWidth && groups(256, 64) >= 384) return TileShape{256, 64, 4, 1};
  if (Ncols > 64 && groups(256, 128) >= 192)
    return W <= kHaloPairWidth && igemm_halo_pairs(groups(256, 128), groups(128, 128)) ? TileShape{128, 128, 2, 2} : TileShape{256, 128, 4, 2};
  if (groups(128, 64) >= 384) return TileShape{128, 64, 2, 2};
  return TileShape{64, 64, 2, 2};
}
// A 3x3 filter with stride 1 and padding 1 (the gathered tensor and the output have the same pixel grid): the
// layers of the halo main loop.  The launch and the callers that size the batch-norm sums (one row per row tile)
// both go through halo_filter / igemm_halo_tile, so they agree on the tile.
static bool halo_filter(int R, int S, int stride, int pad) {
#ifdef RN50_TUNING  // tuning builds only: RN50_NO_HALO sends these layers down the general path
  static const bool off = getenv("RN50_NO_HALO") != nullptr;
  if (off) return false;
#endif
  return R == 3 && S == 3 && stride == 1 && pad == 1;
}
static bool igemm_halo_shape(const IgemmArgs& a) {
  return halo_filter(a.R, a.S, a.stride, a.pad) && !a.pair && a.H == a.P && a.W == a.Q;
}
// The tile of a launch.  rows: output pixels (of one parity class for a stride-2 data gradient, `live` of whose four classes
// have any taps); taps x cpt 128-byte chunks of reduction; lin_fwd_channels: input channels of a 1x1 stride-1 forward
// layer (else 0), whose coefficient table bounds the K-split kernels.  (The rows of sums of a data gradient are the same with a second
// branch and without: their callers do not know which.)
// Where 64x64 tiles would give at most one workgroup per compute unit and there are chunks for four waves, the waves split K
// (KS; 3x3 / stride 1 layers by filter rows); at half of that or less the tile is halved again (in float, whose MFMAs take sixteen times as
// long per chunk, in both directions), so that twice (four times) as many compute units work; with 257 to 512 tiles the two workgroups per
// compute unit of the shared ring do better.  Limits of 0 / 128 / 256 / 384 / 512 tiles, ms: step at batch 12 2.49 / 2.46 / 2.41 / 2.59 /
// 2.59, 24 3.37 / 3.36 / 3.32 / 3.48 / 3.50, 40 4.29 / 4.29 / 4.26 / 4.26 / 4.47; float gradients at batch 2 3.64 / 2.20 / 2.17 / 2.17 / 2.24, 8
// 4.66 / 4.04 / 3.80 / 3.80 / 4.08, 16 6.55 / 6.41 / 6.05 / 6.06 / 6.30; evaluation at batch 16 0.63 / 0.60 / 0.57 / 0.57 / 0.66
// (profiles/step_time_against_dispatch_constants.txt; layer by layer: profiles/conv_tile_sweep_*.txt).
static TileShape pick_tile(int64_t rows, int Ncols, int chunks, bool strided_dgrad, int live, int halo_width, int lin_fwd_channels,
                           TileUse use, int dtype) {
#ifdef RN50_TUNING  // tuning builds only: RN50_IGEMM_TILE=bm,bn,wm,wn forces a compiled tile shape
  if (const char* e = getenv("RN50_IGEMM_TILE")) {
    TileShape f{0, 0, 0, 0};
    if (sscanf(e, "%d,%d,%d,%d", &f.bm, &f.bn, &f.wm, &f.wn) == 4) {
#define X(BM, BN, WM, WN) if (f.bm == BM && f.bn == BN && f.wm == WM && f.wn == WN) return f;
      RN50_IGEMM_SHAPES(X)
      if (dtype == RN50_F32) { RN50_IGEMM_SHAPE_F32(X) } else { RN50_IGEMM_SHAPE_BF16(X) }
#undef X
    }
  }
#endif
  const int64_t groups64 = ceil_div(rows, 64) * ceil_div(Ncols, 64) * (strided_dgrad ? live : 1);
  if (chunks >= 4 && lin_fwd_channels <= 2048 && groups64 <= 256) {
    if (groups64 > 128) return TileShape{64, 64, 1, 1};
    return dtype == RN50_F32 ? TileShape{32, 32, 1, 1} : TileShape{32, 64, 1, 1};
  }
  return halo_width > 0 ? igemm_halo_tile(rows, Ncols, chunks / 9, halo_width) : igemm_tile(rows, Ncols, chunks, strided_dgrad, live, use, dtype);
}
template <typename T>
static void launch_igemm(const IgemmArgs& a, const char* tag, hipStream_t s) {
  const bool classes = a.mode == 1 && a.stride == 2;
  const int64_t rows = classes ? static_cast<int64_t>(a.M / (a.P * a.Q)) * ((a.P + 1) / 2) * ((a.Q + 1) / 2) : a.M;
  const TileUse use = a.mode == 0 ? TileUse::kForward : a.mode == 2 ? TileUse::kAffine : !a.partial ? TileUse::kGrad
                      : a.addend ? TileUse::kGradSumsAdd : TileUse::kGradSums;
  const bool lin_fwd = a.mode != 1 && a.R == 1 && a.S == 1 && a.stride == 1 && a.pad == 0 && !a.pair;
  const TileShape t = pick_tile(rows, a.Ncols, a.R * a.S * a.cpt, classes, a.R * a.S > 1 ? 4 : 1,
                                igemm_halo_shape(a) ? a.W : 0, lin_fwd ? a.Cg : 0, use, sizeof(T) == 2 ? RN50_BF16 : RN50_F32);
#define X(BM, BN, WM, WN) if (t.bm == BM && t.bn == BN && t.wm == WM && t.wn == WN) launch_igemm_cfg<T, BM, BN, WM, WN>(a, tag, s);
  RN50_IGEMM_SHAPES(X)
  if constexpr (sizeof(T) == 4) { RN50_IGEMM_SHAPE_F32(X) } else { RN50_IGEMM_SHAPE_BF16(X) }
#undef X
  if (a.partial) {  // (a stride-2 data gradient has the tiles of four classes of pixels)
    const int mtiles = static_cast<int>((classes ? 4 : 1) * ceil_div(rows, t.bm));
    if (bn_reduces(mtiles)) bn_reduce_rows(a.partial, mtiles, t.bm, a.M, a.Ncols, a.mode == 1, s);
  }
}

static int check_conv(const rn50_conv_desc* d, const char* who) {
  RN50_REQUIRE(d, RN50_ERR_INVALID, "%s: null descriptor", who);
  RN50_REQUIRE(d->N > 0 && d->H > 0 && d->W > 0 && d->Cin > 0 && d->Cout > 0 && d->R > 0 && d->S > 0 &&
                   d->stride > 0 && d->pad >= 0,
               RN50_ERR_INVALID, "%s: non-positive size", who);
  RN50_REQUIRE(d->dtype == RN50_F32 || d->dtype == RN50_BF16, RN50_ERR_INVALID, "%s: dtype %d", who, d->dtype);
  const int V = 16 / esize(d->dtype);
  RN50_REQUIRE(d->H + 2 * d->pad >= d->R && d->W + 2 * d->pad >= d->S, RN50_ERR_INVALID, "%s: filter larger than padded input", who);
  RN50_REQUIRE(d->Cout % V == 0, RN50_ERR_UNSUPPORTED, "%s: Cout=%d is not a multiple of %d", who, d->Cout, V);
  RN50_REQUIRE(d->Cin % V == 0 || is_stem(d), RN50_ERR_UNSUPPORTED,
               "%s: Cin=%d is neither a multiple of %d nor the 7x7/2 pad-3 stem", who, d->Cin, V);
  RN50_REQUIRE(d->pad < d->R && d->pad < d->S, RN50_ERR_UNSUPPORTED, "%s: pad >= filter size", who);
  RN50_REQUIRE(!is_stem(d) || (d->N <= 65535 && d->H + 6 <= 65535), RN50_ERR_UNSUPPORTED,
               "%s: stem with N=%d, H=%d is beyond the padding kernel's launch grid", who, d->N, d->H);
  const int P = out_dim(d->H, d->pad, d->R, d->stride), Q = out_dim(d->W, d->pad, d->S, d->stride);
  const int64_t lim = ((1ll << 31) - 1) / esize(d->dtype);  // byte offsets are 31-bit
  RN50_REQUIRE(static_cast<int64_t>(d->N) * (d->H + 6) * (d->W + 16) * (d->Cin < 4 ? 4 : d->Cin) < lim &&
                   static_cast<int64_t>(d->N) * P * Q * d->Cout < lim &&
                   static_cast<int64_t>(d->Cout) * d->R * d->S * (d->Cin < 4 ? 32 : d->Cin) < lim,
               RN50_ERR_UNSUPPORTED, "%s: a tensor is 2 GiB or larger", who);
  return RN50_OK;
}

}  // namespace rn50

using namespace rn50;

// Internal entry points shared with the whole-step driver (declared in step_internal.h).
namespace rn50 {

int conv_desc_check(const rn50_conv_desc* d, const char* who) { return check_conv(d, who); }

void stem_pad_input(const rn50_conv_desc* d, const void* x, void* xp, hipStream_t s) {
  const StemGeom g = stem_geom(d);
  const dim3 grid(static_cast<unsigned>(ceil_div(g.Wp, 256)), g.Hp, d->N);
  if (d->dtype == RN50_BF16)
    RN50_LAUNCH("stem_pad", stem_pad_input_kernel<uint16_t>, grid, dim3(256), 0, s,
                       static_cast<const uint16_t*>(x), static_cast<uint16_t*>(xp), d->N, d->H, d->W, g.Hp, g.Wp);
  else
    RN50_LAUNCH("stem_pad", stem_pad_input_kernel<float>, grid, dim3(256), 0, s,
                       static_cast<const float*>(x), static_cast<float*>(xp), d->N, d->H, d->W, g.Hp, g.Wp);
}

size_t stem_padded_input_bytes(const rn50_conv_desc* d) { return stem_geom(d).xp_bytes; }
size_t stem_padded_weight_bytes(const rn50_conv_desc* d) { return stem_geom(d).wp_bytes; }

static int chunks_per_tap(int channels, int dtype) { return static_cast<int>(ceil_div(channels * esize(dtype), 128)); }
// stride-2 data gradient: four parity classes of ceil(N * ceil(H/2) * ceil(W/2) / bm) row tiles each
static PartialRows class_tile_rows(const rn50_conv_desc* d) {
  const int64_t rows = static_cast<int64_t>(d->N) * ((d->H + 1) / 2) * ((d->W + 1) / 2);
  const int bm = pick_tile(rows, d->Cin, d->R * d->S * chunks_per_tap(d->Cout, d->dtype), true, d->R * d->S > 1 ? 4 : 1,
                           0, 0, TileUse::kGradSums, d->dtype).bm;
  return PartialRows{bm, static_cast<int>(4 * ceil_div(rows, bm))};
}
PartialRows fwd_partial_rows(const rn50_conv_desc* d) {
  if (const PartialRows pr = stem_partial_rows(d); pr.num) return pr;
  const int64_t M = static_cast<int64_t>(d->N) * out_dim(d->H, d->pad, d->R, d->stride) * out_dim(d->W, d->pad, d->S, d->stride);
  // the chunk count as the launch computes it (the bf16 stem runs as 4 taps of one chunk, the float stem as 7)
  const int chunks = is_stem(d) ? (d->dtype == RN50_BF16 ? 4 : 7) : d->R * d->S * chunks_per_tap(d->Cin, d->dtype);
  const bool lin = d->R == 1 && d->S == 1 && d->stride == 1 && d->pad == 0;
  const int bm = pick_tile(M, d->Cout, chunks, false, 4, halo_filter(d->R, d->S, d->stride, d->pad) ? d->W : 0, lin ? d->Cin : 0,
                           TileUse::kForward, d->dtype).bm;
  return PartialRows{bm, static_cast<int>(ceil_div(M, bm))};
}
int64_t dgrad_partial_rows_bound(const rn50_conv_desc* d) {
  const int64_t plain = ceil_div(static_cast<int64_t>(d->N) * d->H * d->W, 32);
  const int64_t classes = 4 * ceil_div(static_cast<int64_t>(d->N) * ((d->H + 1) / 2) * ((d->W + 1) / 2), 32);
  return d->stride == 2 && classes > plain ? classes : plain;
}
PartialRows dgrad_partial_rows(const rn50_conv_desc* d) {
  if (d->stride == 2) return class_tile_rows(d);
  const int64_t M = static_cast<int64_t>(d->N) * d->H * d->W;
  const int bm = pick_tile(M, d->Cin, d->R * d->S * chunks_per_tap(d->Cout, d->dtype), false, 4,
                           halo_filter(d->R, d->S, d->stride, d->pad) ? d->W : 0, 0, TileUse::kGradSums, d->dtype).bm;
  return PartialRows{bm, static_cast<int>(ceil_div(M, bm))};
}

static IgemmArgs stem_igemm_args(const rn50_conv_desc* d, const void* xp, const void* wp, void* y) {
  const StemGeom g = stem_geom(d);
  IgemmArgs a{};
  a.act = xp; a.wgt = wp; a.out = y;
  a.P = out_dim(d->H, 3, 7, 2); a.Q = out_dim(d->W, 3, 7, 2);
  a.M = d->N * a.P * a.Q; a.Ncols = d->Cout; a.Ktot = kStemK;
  a.H = g.Hp; a.W = g.Wp; a.PS = 4; a.stride = 2; a.pad = 0; a.mode = 0; a.S = 1;
  a.cpt = 1;
  // A filter row is 8 padded taps x 4 channels = 32 elements: a whole 128-byte chunk in float, half of
  // one in bf16, where two filter rows share a chunk (4 "taps" of 64 elements; the 8th row is zero weights).
  a.pair = d->dtype == RN50_BF16;
  a.R = a.pair ? 4 : 7;
  a.Cg = a.pair ? 64 : 32;
  a.act_bytes = static_cast<uint32_t>(static_cast<size_t>(d->N) * g.Hp * g.Wp * 4 * esize(d->dtype));
  a.wgt_bytes = static_cast<uint32_t>(static_cast<size_t>(d->Cout) * kStemK * esize(d->dtype));
  return a;
}

static void set_affine(IgemmArgs& a, const BnAffine& f) {
  a.mode = 2;
  a.bn_gamma = f.gamma; a.bn_beta = f.beta; a.bn_mean = f.mean; a.aff_var = f.var;
  a.aff_eps = f.eps; a.aff_relu = f.relu; a.addend = f.residual;
}
// Forward of the stem from an already padded input; wp is scratch for the padded weights.
void stem_fwd_padded(const rn50_conv_desc* d, const void* xp, const void* w, void* wp, void* y, float* bn_partial,
                     hipStream_t s, const BnAffine* affine) {
  if (stem_fwd_run(d, xp, w, y, bn_partial, s, affine)) return;
  const int nw = d->Cout * kStemK;
  IgemmArgs a = stem_igemm_args(d, xp, wp, y);
  a.partial = bn_partial;
  if (affine) set_affine(a, *affine);
  if (d->dtype == RN50_BF16) {
    RN50_LAUNCH("stem_pad", stem_pad_weight_kernel<uint16_t>, dim3(ceil_div(nw, 256)), dim3(256), 0, s,
                       static_cast<const uint16_t*>(w), static_cast<uint16_t*>(wp), d->Cout);
    launch_igemm<uint16_t>(a, "conv_fwd", s);
  } else {
    RN50_LAUNCH("stem_pad", stem_pad_weight_kernel<float>, dim3(ceil_div(nw, 256)), dim3(256), 0, s,
                       static_cast<const float*>(w), static_cast<float*>(wp), d->Cout);
    launch_igemm<float>(a, "conv_fwd", s);
  }
}

void fwd_run(const rn50_conv_desc* d, const void* x, const void* w, void* y, float* bn_partial, hipStream_t s,
             const char* tag, const BnIn* in, const BnAffine* affine, unsigned long long* slots) {
  IgemmArgs a{};
  a.act = x; a.wgt = w; a.out = y; a.partial = bn_partial; a.slots = slots;
  if (in) { a.in_gamma = in->gamma; a.in_beta = in->beta; a.in_mean = in->mean; a.in_rstd = in->rstd; }
  a.P = out_dim(d->H, d->pad, d->R, d->stride); a.Q = out_dim(d->W, d->pad, d->S, d->stride);
  a.M = d->N * a.P * a.Q; a.Ncols = d->Cout; a.Ktot = d->R * d->S * d->Cin;
  a.H = d->H; a.W = d->W; a.PS = d->Cin; a.Cg = d->Cin; a.R = d->R; a.S = d->S; a.stride = d->stride; a.pad = d->pad;
  a.mode = 0;
  a.act_bytes = static_cast<uint32_t>(static_cast<size_t>(d->N) * d->H * d->W * d->Cin * esize(d->dtype));
  a.wgt_bytes = static_cast<uint32_t>(static_cast<size_t>(d->Cout) * a.Ktot * esize(d->dtype));
  a.cpt = static_cast<int>(ceil_div(d->Cin * esize(d->dtype), 128));
  if (affine) set_affine(a, *affine);
  if (d->dtype == RN50_BF16) launch_igemm<uint16_t>(a, tag, s); else launch_igemm<float>(a, tag, s);
}

// What conv_dgrad's callers are asked for (the size of the weights).  The kernels read the weights as they lie and
// nothing is written there any more; the query and the checks stay as the interface has them.
static size_t dgrad_ws_bytes(const rn50_conv_desc* d) {
  return align_up(static_cast<size_t>(d->Cout) * d->R * d->S * d->Cin * esize(d->dtype), 256);
}
void dgrad_run(const rn50_conv_desc* d, const void* dy, const void* w, void* dx, const BnBwdSums* bn, hipStream_t s,
               const char* tag) {
  IgemmArgs a{};
  a.act = dy; a.wgt = w; a.out = dx;
  if (bn) {
    a.partial = bn->partial; a.bn_x = bn->x;
    a.bn_gamma = bn->gamma; a.bn_beta = bn->beta; a.bn_mean = bn->mean; a.bn_rstd = bn->rstd;
    a.slots = bn->slots; a.addend_even = bn->addend_even; a.addend = bn->addend; a.bn_zmask = bn->relu_mask; a.addend_mask = bn->addend ? bn->addend_mask : nullptr;
  }
  a.P = d->H; a.Q = d->W;
  a.H = out_dim(d->H, d->pad, d->R, d->stride); a.W = out_dim(d->W, d->pad, d->S, d->stride);
  a.M = d->N * d->H * d->W; a.Ncols = d->Cin; a.Ktot = d->R * d->S * d->Cout;
  a.PS = d->Cout; a.Cg = d->Cout; a.R = d->R; a.S = d->S; a.stride = d->stride; a.pad = d->pad;
  a.mode = 1;
  a.act_bytes = static_cast<uint32_t>(static_cast<size_t>(d->N) * a.H * a.W * d->Cout * esize(d->dtype));
  a.wgt_bytes = static_cast<uint32_t>(static_cast<size_t>(d->Cin) * a.Ktot * esize(d->dtype));
  a.cpt = static_cast<int>(ceil_div(d->Cout * esize(d->dtype), 128));
  if (d->dtype == RN50_BF16) launch_igemm<uint16_t>(a, tag, s); else launch_igemm<float>(a, tag, s);
}

}  // namespace rn50

extern "C" size_t conv_fwd_workspace_bytes(const rn50_conv_desc* d) {
  if (!d || check_conv(d, "conv_fwd_workspace_bytes")) return 0;
  if (!is_stem(d)) return 0;
  const StemGeom g = stem_geom(d);
  return g.xp_bytes + g.wp_bytes;
}
extern "C" size_t conv_dgrad_workspace_bytes(const rn50_conv_desc* d) {
  if (!d || check_conv(d, "conv_dgrad_workspace_bytes")) return 0;
  return dgrad_ws_bytes(d);
}
extern "C" size_t conv_wgrad_workspace_bytes(const rn50_conv_desc* d) {
  if (!d || check_conv(d, "conv_wgrad_workspace_bytes")) return 0;
  return wgrad_partial_bytes(d) + (is_stem(d) ? stem_geom(d).xp_bytes : 0);
}

extern "C" int conv_fwd(const rn50_conv_desc* d, const void* x, const void* w, void* y, void* workspace,
                        size_t workspace_bytes, void* stream) {
  clear_error();
  if (int rc = check_conv(d, "conv_fwd")) return rc;
  RN50_REQUIRE(x && w && y, RN50_ERR_INVALID, "conv_fwd: null pointer");
  RN50_REQUIRE(aligned16(x) && aligned16(w) && aligned16(y) && aligned16(workspace), RN50_ERR_ALIGN,
               "conv_fwd: pointer not 16-byte aligned");
  const size_t need = conv_fwd_workspace_bytes(d);
  RN50_REQUIRE(workspace_bytes >= need && (need == 0 || workspace), RN50_ERR_WORKSPACE,
               "conv_fwd: workspace %zu < %zu bytes", workspace_bytes, need);
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (is_stem(d)) {
    unsigned char* ws = static_cast<unsigned char*>(workspace);
    stem_pad_input(d, x, ws, s);
    stem_fwd_padded(d, ws, w, ws + stem_geom(d).xp_bytes, y, nullptr, s);
  } else {
    fwd_run(d, x, w, y, nullptr, s);
  }
  return launch_status("conv_fwd");
}

extern "C" int conv_dgrad(const rn50_conv_desc* d, const void* dy, const void* w, void* dx, void* workspace,
                          size_t workspace_bytes, void* stream) {
  clear_error();
  if (int rc = check_conv(d, "conv_dgrad")) return rc;
  RN50_REQUIRE(!is_stem(d) && d->Cin % (16 / esize(d->dtype)) == 0, RN50_ERR_UNSUPPORTED,
               "conv_dgrad: the 3-channel stem has no data gradient here (the network input needs none)");
  RN50_REQUIRE(d->stride == 1 || d->stride == 2, RN50_ERR_UNSUPPORTED, "conv_dgrad: stride %d", d->stride);
  RN50_REQUIRE(dy && w && dx && workspace, RN50_ERR_INVALID, "conv_dgrad: null pointer");
  RN50_REQUIRE(aligned16(dy) && aligned16(w) && aligned16(dx) && aligned16(workspace), RN50_ERR_ALIGN,
               "conv_dgrad: pointer not 16-byte aligned");
  RN50_REQUIRE(workspace_bytes >= dgrad_ws_bytes(d), RN50_ERR_WORKSPACE, "conv_dgrad: workspace %zu < %zu bytes",
               workspace_bytes, dgrad_ws_bytes(d));
  hipStream_t s = static_cast<hipStream_t>(stream);
  dgrad_run(d, dy, w, dx, nullptr, s);
  return launch_status("conv_dgrad");
}

extern "C" int conv_wgrad(const rn50_conv_desc* d, const void* x, const void* dy, float* dw, void* workspace,
                          size_t workspace_bytes, void* stream) {
  clear_error();
  if (int rc = check_conv(d, "conv_wgrad")) return rc;
  RN50_REQUIRE(x && dy && dw, RN50_ERR_INVALID, "conv_wgrad: null pointer");
  RN50_REQUIRE(aligned16(x) && aligned16(dy) && aligned16(dw) && aligned16(workspace), RN50_ERR_ALIGN,
               "conv_wgrad: pointer not 16-byte aligned");
  const size_t need = conv_wgrad_workspace_bytes(d);
  RN50_REQUIRE(workspace_bytes >= need && (need == 0 || workspace), RN50_ERR_WORKSPACE,
               "conv_wgrad: workspace %zu < %zu bytes", workspace_bytes, need);
  hipStream_t s = static_cast<hipStream_t>(stream);
  unsigned char* ws = static_cast<unsigned char*>(workspace);
  if (is_stem(d)) {
    stem_pad_input(d, x, ws, s);
    wgrad_run(d, ws, dy, dw, ws + stem_geom(d).xp_bytes, s);
  } else {
    wgrad_run(d, x, dy, dw, ws, s);
  }
  return launch_status("conv_wgrad");
}

// ---- fused batch-norm sums (the BN side is in bn.hip)
extern "C" size_t conv_bn_sums_bytes(const rn50_conv_desc* d) {
  if (!d || check_conv(d, "conv_bn_sums_bytes")) return 0;
  // one row per output tile of at least 32 pixels
  const int P = out_dim(d->H, d->pad, d->R, d->stride), Q = out_dim(d->W, d->pad, d->S, d->stride);
  const size_t fwd = bn_sums_bytes(ceil_div(static_cast<int64_t>(d->N) * P * Q, 32), d->Cout, kBnWideSumBytes);
  const size_t bwd = bn_sums_bytes(dgrad_partial_rows_bound(d), d->Cin, kBnBwdSumBytes);
  return align_up(fwd > bwd ? fwd : bwd, 256);
}

extern "C" int conv_fwd_bn_sums(const rn50_conv_desc* d, const void* x, const void* w, void* y, float* sums,
                                size_t sums_bytes, void* workspace, size_t workspace_bytes, void* stream) {
  clear_error();
  if (int rc = check_conv(d, "conv_fwd_bn_sums")) return rc;
  RN50_REQUIRE(x && w && y && sums, RN50_ERR_INVALID, "conv_fwd_bn_sums: null pointer");
  RN50_REQUIRE(aligned16(x) && aligned16(w) && aligned16(y) && aligned16(workspace) && aligned16(sums),
               RN50_ERR_ALIGN, "conv_fwd_bn_sums: pointer not 16-byte aligned");
  const size_t need = conv_fwd_workspace_bytes(d);
  RN50_REQUIRE(workspace_bytes >= need && (need == 0 || workspace), RN50_ERR_WORKSPACE,
               "conv_fwd_bn_sums: workspace %zu < %zu bytes", workspace_bytes, need);
  RN50_REQUIRE(sums_bytes >= conv_bn_sums_bytes(d), RN50_ERR_WORKSPACE, "conv_fwd_bn_sums: sums %zu < %zu bytes",
               sums_bytes, conv_bn_sums_bytes(d));
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (is_stem(d)) {
    unsigned char* ws = static_cast<unsigned char*>(workspace);
    stem_pad_input(d, x, ws, s);
    stem_fwd_padded(d, ws, w, ws + stem_geom(d).xp_bytes, y, sums, s);
  } else {
    fwd_run(d, x, w, y, sums, s);
  }
  return launch_status("conv_fwd_bn_sums");
}

extern "C" int conv_dgrad_bn_sums(const rn50_conv_desc* d, const void* dy, const void* w, void* dx,
                                  const void* addend, const uint8_t* addend_mask, const void* bn_x,
                                  const uint8_t* relu_mask, const float* gamma, const float* beta,
                                  const float* save_mean, const float* save_rstd, float* sums,
                                  size_t sums_bytes, void* workspace, size_t workspace_bytes, void* stream) {
  clear_error();
  if (int rc = check_conv(d, "conv_dgrad_bn_sums")) return rc;
  RN50_REQUIRE(!is_stem(d) && d->Cin % (16 / esize(d->dtype)) == 0, RN50_ERR_UNSUPPORTED,
               "conv_dgrad_bn_sums: the 3-channel stem has no data gradient here");
  RN50_REQUIRE(d->stride == 1 || d->stride == 2, RN50_ERR_UNSUPPORTED, "conv_dgrad_bn_sums: stride %d", d->stride);
  RN50_REQUIRE(dy && w && dx && workspace && bn_x && gamma && beta && save_mean && save_rstd && sums,
               RN50_ERR_INVALID, "conv_dgrad_bn_sums: null pointer");
  RN50_REQUIRE(aligned16(dy) && aligned16(w) && aligned16(dx) && aligned16(workspace) && aligned16(bn_x) &&
                   aligned16(sums) && aligned16(addend) && aligned16(gamma) && aligned16(beta) &&
                   aligned16(save_mean) && aligned16(save_rstd),
               RN50_ERR_ALIGN, "conv_dgrad_bn_sums: pointer not 16-byte aligned");
  RN50_REQUIRE(workspace_bytes >= dgrad_ws_bytes(d), RN50_ERR_WORKSPACE,
               "conv_dgrad_bn_sums: workspace %zu < %zu bytes", workspace_bytes, dgrad_ws_bytes(d));
  RN50_REQUIRE(sums_bytes >= conv_bn_sums_bytes(d), RN50_ERR_WORKSPACE, "conv_dgrad_bn_sums: sums %zu < %zu bytes",
               sums_bytes, conv_bn_sums_bytes(d));
  RN50_REQUIRE(!addend_mask || addend, RN50_ERR_INVALID, "conv_dgrad_bn_sums: addend_mask without addend");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const BnBwdSums bn{bn_x, gamma, beta, save_mean, save_rstd, sums, addend, relu_mask, addend_mask};
  dgrad_run(d, dy, w, dx, &bn, s);
  return launch_status("conv_dgrad_bn_sums");
}

// ---- convolution whose input is the output of a BN+ReLU layer that is applied on the fly
static int check_bn_in(const rn50_conv_desc* d, const char* who) {
  RN50_REQUIRE(d->R == 1 && d->S == 1 && d->stride == 1 && d->pad == 0, RN50_ERR_UNSUPPORTED,
               "%s: only 1x1 convolutions with stride 1 and no padding take their input through a BN layer", who);
  RN50_REQUIRE(d->Cin <= 4096, RN50_ERR_UNSUPPORTED, "%s: Cin=%d > 4096", who, d->Cin);
  return RN50_OK;
}
extern "C" int conv_fwd_bn_in(const rn50_conv_desc* d, const void* x, const float* in_gamma, const float* in_beta,
                              const float* in_mean, const float* in_rstd, const void* w, void* y, float* sums,
                              size_t sums_bytes, void* stream) {
  clear_error();
  if (int rc = check_conv(d, "conv_fwd_bn_in")) return rc;
  if (int rc = check_bn_in(d, "conv_fwd_bn_in")) return rc;
  RN50_REQUIRE(x && w && y && in_gamma && in_beta && in_mean && in_rstd, RN50_ERR_INVALID, "conv_fwd_bn_in: null pointer");
  RN50_REQUIRE(aligned16(x) && aligned16(w) && aligned16(y) && aligned16(sums), RN50_ERR_ALIGN,
               "conv_fwd_bn_in: pointer not 16-byte aligned");
  RN50_REQUIRE(!sums || sums_bytes >= conv_bn_sums_bytes(d), RN50_ERR_WORKSPACE, "conv_fwd_bn_in: sums %zu < %zu bytes",
               sums_bytes, conv_bn_sums_bytes(d));
  const BnIn in{in_gamma, in_beta, in_mean, in_rstd};
  fwd_run(d, x, w, y, sums, static_cast<hipStream_t>(stream), "conv_fwd", &in);
  return launch_status("conv_fwd_bn_in");
}
extern "C" int conv_wgrad_bn_in(const rn50_conv_desc* d, const void* x, const float* in_gamma, const float* in_beta,
                                const float* in_mean, const float* in_rstd, const void* dy, float* dw, void* workspace,
                                size_t workspace_bytes, void* stream) {
  clear_error();
  if (int rc = check_conv(d, "conv_wgrad_bn_in")) return rc;
  if (int rc = check_bn_in(d, "conv_wgrad_bn_in")) return rc;
  RN50_REQUIRE(x && dy && dw && in_gamma && in_beta && in_mean && in_rstd, RN50_ERR_INVALID, "conv_wgrad_bn_in: null pointer");
  RN50_REQUIRE(aligned16(x) && aligned16(dy) && aligned16(dw) && aligned16(workspace), RN50_ERR_ALIGN,
               "conv_wgrad_bn_in: pointer not 16-byte aligned");
  const size_t need = conv_wgrad_workspace_bytes(d);
  RN50_REQUIRE(workspace_bytes >= need && (need == 0 || workspace), RN50_ERR_WORKSPACE,
               "conv_wgrad_bn_in: workspace %zu < %zu bytes", workspace_bytes, need);
  const BnIn in{in_gamma, in_beta, in_mean, in_rstd};
  wgrad_run(d, x, dy, dw, workspace, static_cast<hipStream_t>(stream), &in);
  return launch_status("conv_wgrad_bn_in");
}
