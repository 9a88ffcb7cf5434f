// Training-mode batch normalization fused with ReLU and the residual add
// (Sec. II and III-A3 of the paper: statistics over the local batch only;
// appendix log: epsilon 1e-5, scale and centre on, momentum 0.9).
//
// All kernels are HBM-bound.  x is [m][C] with channels contiguous, so a
// workgroup of 256 threads is laid out as TY rows x TX 16-byte channel vectors
// (TX*16 B contiguous per row, consecutive rows contiguous in memory), every
// thread keeps its own channels in registers while it walks down the rows, and
// rows are only combined once per workgroup through LDS.
//
// Forward:  stats (per-workgroup partial sums) -> finalize (mean, rstd) -> apply.
// Backward: reduce (partial sums of g and g*xhat) -> finalize (dgamma, dbeta) -> apply.
// The first pass of either direction can be left to the convolution that produces
// the tensor (its output stage writes the same rows of partial sums, one per
// output tile): the *_from_partials entry points then run finalize + apply only.
// Partial sums are combined in a fixed order, so results are bitwise reproducible.
//
// Variance uses shifted sums: every row of partials is summed in float about a shift K of its own (the first
// element its producer saw), S1 = sum(x-K), S2 = sum((x-K)^2), and stored either moved to shift 0, in double, or with its
// shift; all combining is in double.  Nowhere does float rounding see the cancellation of the plain E[x^2]-E[x]^2 form.
// (Forms and layout of the rows: bn_sums_at.)
#include <stdlib.h>

#include <algorithm>

#include "common.h"
#include "step_internal.h"

namespace rn50 {

constexpr int kBnRows = 4;  // rows a thread loads before it touches any of them (memory-level parallelism)

// 16 bytes at a uniform address plus a lane's byte offset: the address costs the lanes nothing.  A row's offset of fewer than 256 rows
// fits 32 bits up to this many channels.
constexpr int kBnLaneOffsetChannels = 1 << 21;
template <typename T>
__device__ __forceinline__ Vec16 load16_at(const T* uniform_base, uint32_t lane_bytes) {
  return load16(reinterpret_cast<const T*>(reinterpret_cast<const unsigned char*>(uniform_base) + lane_bytes));
}

struct BnGeom {
  int V;        // elements per 16-byte vector
  int cvecs;    // C / V
  int tx_log2;  // TX = 1 << tx_log2 threads across channel vectors
  int gy;       // workgroups across channel vectors
  int rpb;      // rows per workgroup
  int nblk;     // workgroups across rows
};

static BnGeom bn_geom(int64_t m, int C, int dtype) {
  BnGeom g;
  g.V = dtype == RN50_BF16 ? 8 : 4;
  g.cvecs = C / g.V;
  g.tx_log2 = 0;
  while ((1 << g.tx_log2) < g.cvecs && g.tx_log2 < 5) ++g.tx_log2;
  const int TX = 1 << g.tx_log2, TY = 256 / TX;
  g.gy = static_cast<int>(ceil_div(g.cvecs, TX));
  // rows per thread: aim at ~1024 workgroups in all, but at least 64 rows per workgroup so that the
  // per-workgroup partial sums stay a few percent of the tensor; a multiple of the 4 rows whose loads
  // are issued together
  const int64_t nblk_target = 1024 / g.gy > 0 ? 1024 / g.gy : 1;
  int64_t rpt = ceil_div(m, static_cast<int64_t>(TY) * nblk_target);
  if (rpt * TY < 64) rpt = ceil_div(64, TY);
  rpt = ceil_div(rpt, kBnRows) * kBnRows;
  const int64_t rpb = rpt * TY;
  g.rpb = static_cast<int>(rpb);
  g.nblk = static_cast<int>(ceil_div(m, rpb));
  return g;
}

// Geometry of the stand-alone sums passes (statistics, backward sums).  Small layers are summed in at most 128 row blocks of
// at least 32 rows, as doubles, and their apply pass finalizes by itself (bn_apply_kernel's FIN): a finalize launch costs
// about 4 us whatever it computes, reading 128 rows of sums in every apply workgroup 1 to 2 -- as long as the workgroups
// are few: beyond kBnSelfElems the sums they read together are as many bytes as the tensor.  Nine layers, both directions, batch
// 4 / 8 / 40: 211 / 231 / 469 us; never 219 / 240 / 464; up to 8192 rows 209 / 231 / 465; up to 16 M elements 212 / 240 / 480
// (profiles/bn_standalone_sums_forms.txt; 28x28x128 at batch 40, 31,360 rows, is 3 us slower for it, 56x56x64 at batch 8 1 us faster).
// Larger layers: up to kBnSumsGroups workgroups whose threads load their eight rows (kBnSumsRows) once.  Workgroups that
// loop over more rows all load at the same time and all compute at the same time.
constexpr int64_t kBnSelfRows = 32768, kBnSelfElems = 4 << 20;
constexpr int kBnSumsGroups = 4096, kBnSumsRows = 8;
static bool bn_self_sums(int64_t m, int C) { return m <= kBnSelfRows && m * C <= kBnSelfElems; }
static BnGeom bn_sums_geom(int64_t m, int C, int dtype) {
  BnGeom g = bn_geom(m, C, dtype);
  const int TY = 256 >> g.tx_log2;
  if (bn_self_sums(m, C)) {
    const int64_t rows = std::max<int64_t>(ceil_div(m, 128), 32);
    g.rpb = static_cast<int>(ceil_div(rows, TY) * TY);
  } else {
    const int64_t rows = ceil_div(m * g.gy, static_cast<int64_t>(TY) * kBnSumsGroups);  // per thread
    g.rpb = static_cast<int>(ceil_div(rows, kBnSumsRows) * kBnSumsRows) * TY;
  }
  g.nblk = static_cast<int>(ceil_div(m, g.rpb));
  return g;
}

// The elementwise passes have no sums to combine, so their geometry is free: at most `target` workgroups,
// each thread streaming 4 to 32 rows.  Measured inside the training step (profiles/step_time_against_dispatch_constants.txt)
// and on a plain copy kernel: many small workgroups that make one round of loads each stream faster than few
// long-running ones (a 16-byte-per-thread copy of 1 GiB runs at 6.2 TB/s, the same copy by 2,048 looping workgroups
// at 4.9), so the target is high enough that every thread of ResNet-50's layers takes its minimum of 4 rows.
constexpr int kBnApplyGroups = 16384, kBnBwdApplyGroups = 16383;  // (distinct values: the tuning override tells them apart)
static BnGeom bn_apply_geom(int64_t m, int C, int dtype, int target) {
  BnGeom g = bn_geom(m, C, dtype);
#ifdef RN50_TUNING  // tuning builds only: RN50_BN_TARGET=forward,backward workgroup targets of the apply passes
  if (const char* e = getenv("RN50_BN_TARGET")) {
    int tf = 0, tb = 0;
    if (sscanf(e, "%d,%d", &tf, &tb) == 2) target = target == kBnApplyGroups ? tf : tb;
  }
#endif
  const int TY = 256 >> g.tx_log2;
  int64_t rpt = ceil_div(m * g.gy, static_cast<int64_t>(TY) * target);
  rpt = ceil_div(rpt, kBnRows) * kBnRows;
  if (rpt > 32) rpt = 32;
  g.rpb = static_cast<int>(rpt) * TY;
  g.nblk = static_cast<int>(ceil_div(m, g.rpb));
  return g;
}

// Geometry of an apply pass that finalizes by itself: column slices of 8 vectors (TY = 32 rows per pass), about
// kBnSelfFinalizeGroups workgroups, every thread a multiple of 4 rows.
constexpr int kBnSelfFinalizeGroups = 768;
static void bn_self_finalize_geom(int64_t m, int C, int V, int* gy_out, int* rpb_out) {
  int target = kBnSelfFinalizeGroups;
#ifdef RN50_TUNING  // tuning builds only: RN50_BN_FIN_TARGET=workgroups
  if (const char* e = getenv("RN50_BN_FIN_TARGET")) target = atoi(e) > 0 ? atoi(e) : target;
#endif
  const int TY = 32;
  const int gy = static_cast<int>(ceil_div(C / V, 8));
  const int64_t nblk_target = target / gy > 0 ? target / gy : 1;
  int64_t rpt = ceil_div(m, TY * nblk_target);
  rpt = ceil_div(rpt, kBnRows) * kBnRows;
  *gy_out = gy;
  *rpb_out = static_cast<int>(rpt) * TY;
}

// The per-thread sums (2V values: V channels of two quantities) of a workgroup meet: rows of one wave by shuffles, the four
// waves through LDS, in a fixed order.  Thread t < TX * V then owns channel t of the workgroup's column slice: true, with
// the two sums.  (A tree over LDS with every thread's 16 values side by side took longer than a small layer's loads.)
template <int V>
__device__ __forceinline__ bool combine_sums(float* acc, float* lds, int tx_log2, float* t1, float* t2) {
  const int TX = 1 << tx_log2, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int off = TX; off < 64; off <<= 1) {
#pragma unroll
    for (int j = 0; j < 2 * V; ++j) acc[j] += __shfl_xor(acc[j], off, 64);
  }
  if (lane < TX) {
#pragma unroll
    for (int j = 0; j < 2 * V; ++j) lds[(wave * 2 * V + j) * TX + lane] = acc[j];
  }
  __syncthreads();
  if (static_cast<int>(threadIdx.x) >= TX * V) return false;
  const int col = threadIdx.x / V, j = threadIdx.x % V;
  float a[4], b[4];
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    a[w] = lds[(w * 2 * V + j) * TX + col];
    b[w] = lds[(w * 2 * V + V + j) * TX + col];
  }
  *t1 = (a[0] + a[1]) + (a[2] + a[3]);
  *t2 = (b[0] + b[1]) + (b[2] + b[3]);
  return true;
}

// ------------------------------------------------------------------- forward
// Sums of a row block, about a shift of its own channel's first element, stored in either form (wide: doubles).  Bound by the
// bytes in flight: eight rows per thread are requested before the first is used (with four, and the LDS tree at the end, 64 MB
// took 29 us).  A batch of rows that are all there (nearly every one) has one offset per lane behind uniform row addresses and no test per
// row; an address of 64 bits per row, clamped, delayed the loads of small layers by as much as they take (bf16, batch 40: 56x56x64 8.9 ->
// 7.5 us, 28x28x128 7.5 -> 5.2, 14x14x256 5.3 -> 4.5; 64 MB the same; the nine layers' both directions 521 -> 506, float at batch 8 298 ->
// 281).  The apply passes lose by the same change (step at batch 12 1.6 %, 40 and 256 0.6 %: they need the row offsets again to store).
template <typename T>
__global__ __launch_bounds__(256) void bn_stats_kernel(const T* __restrict__ x, int64_t m, int C,
                                                       int tx_log2, int rpb, int wide,
                                                       float* __restrict__ partial) {
  constexpr int V = Elem<T>::VEC, U = kBnSumsRows;
  __shared__ float lds[4 * 2 * V * 32];
  const int TX = 1 << tx_log2, TY = 256 >> tx_log2;
  const int tcol = threadIdx.x & (TX - 1), trow = threadIdx.x >> tx_log2;
  const int col = blockIdx.y * TX + tcol;
  float acc[2 * V], K[V];
#pragma unroll
  for (int j = 0; j < 2 * V; ++j) acc[j] = 0.f;
  const int64_t r0 = static_cast<int64_t>(blockIdx.x) * rpb;
  const int64_t r1 = min(r0 + rpb, m);
  if (col < C / V) {
    const T* p = x + static_cast<int64_t>(col) * V;
    const Vec16 k0 = load16(p);
    const uint32_t lane_off = (static_cast<uint32_t>(trow) * C + static_cast<uint32_t>(col) * V) * sizeof(T);
    Vec16 v[U];
    bool first = true;
    auto add = [&](const Vec16& w) __attribute__((always_inline)) {
      float f[V];
      Elem<T>::unpack(w, f);
#pragma unroll
      for (int j = 0; j < V; ++j) {
        const float d = f[j] - K[j];
        acc[j] += d;
        acc[V + j] = fmaf(d, d, acc[V + j]);
      }
    };
    for (int64_t rb = r0; rb < r1; rb += U * TY) {
      const bool whole = rb + U * TY <= r1 && C <= kBnLaneOffsetChannels;
      if (whole) {
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = load16_at(x + (rb + u * TY) * C, lane_off);
      } else {
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = load16(p + min(rb + trow + u * TY, r1 - 1) * C);
      }
      if (first) Elem<T>::unpack(k0, K);
      first = false;
      if (whole) {
#pragma unroll
        for (int u = 0; u < U; ++u) add(v[u]);
      } else {
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (rb + trow + u * TY < r1) add(v[u]);
      }
    }
  }
  float t1, t2;
  const int c = blockIdx.y * TX * V + threadIdx.x;
  if (!combine_sums<V>(acc, lds, tx_log2, &t1, &t2) || c >= C) return;
  const float k = Elem<T>::load(x + c);
  const int64_t at = bn_sums_at(blockIdx.x, c, gridDim.x);
  if (wide) reinterpret_cast<double2*>(partial)[at] = bn_tile_sums(k, t1, t2, static_cast<int>(r1 - r0));
  else reinterpret_cast<BnTileRow*>(partial)[at] = BnTileRow{k, t1, t2};
}

// Finalize passes, for layers with more rows of partial sums than an apply pass should add up itself.  A workgroup takes
// kFinCh of the eight channels whose rows are contiguous: thread (channel ch, group g) adds rows g, g + G, ... in order,
// kFinRows of them requested at once, then the G groups are added by a fixed tree; all in double.  The pass is a chain of
// load latencies in front of everything that follows it, so there are as many groups as leave a thread a few rows; and its
// workgroups are small, because beside the weight gradients one of sixteen waves waits for a compute unit to empty.
constexpr int kFinCh = 2, kFinRows = 8, kFinThreads = 256;
static int finalize_grid(int C) { return static_cast<int>(ceil_div(C, kFinCh)); }
// Adds (s1, s2) over the groups of the workgroup; the totals of channel ch are in the threads of group 0.
__device__ __forceinline__ void finalize_combine(double* s1, double* s2) {
  __shared__ double red[2][kFinThreads / 64][kFinCh];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, ch = threadIdx.x % kFinCh;
#pragma unroll
  for (int off = 32; off >= kFinCh; off >>= 1) {
    *s1 += __shfl_xor(*s1, off, 64);
    *s2 += __shfl_xor(*s2, off, 64);
  }
  if (lane < kFinCh) {
    red[0][wave][ch] = *s1;
    red[1][wave][ch] = *s2;
  }
  __syncthreads();
  if (threadIdx.x < kFinCh) {
#pragma unroll
    for (int w = 1; w < kFinThreads / 64; ++w) {
      *s1 += red[0][w][ch];
      *s2 += red[1][w][ch];
    }
  }
}

// Forward: adds a row of sums over n rows of x to s1 = sum(x - k0), s2 = sum((x - k0)^2).
__device__ __forceinline__ void add_tile_row(const BnTileRow& v, double n, double k0, double* s1, double* s2) {
  const double e = static_cast<double>(v.k) - k0, d1 = static_cast<double>(v.s1);
  *s1 += d1 + n * e;
  *s2 += static_cast<double>(v.s2) + e * (2.0 * d1 + n * e);
}
__device__ __forceinline__ double rows_of(int b, int nrows, int rpp, int64_t m) {  // rows of x behind row b of the sums
  return static_cast<double>(b == nrows - 1 ? m - static_cast<int64_t>(b) * rpp : rpp);
}

// First reduction of many tile rows: workgroup (piece of eight channels, share of the rows) adds its share up to one row of
// doubles, forward about the shift of the layer's first tile (add_tile_row, as the finalize launch does it).  Thread (channel,
// group g of 32) takes rows g, g + 32, ... in order; groups by a fixed tree.
// The finalize launch alone has a workgroup per two channels, so at 64 channels 32 compute units read 12544 rows, 24 of every
// 96 bytes each: bound by one unit's load instructions (25 us behind an idle chip, 35 to 87 beside the weight gradients).  Here
// a row's 96 (64) bytes are read together and 8 x 64 workgroups share the rows, and the finalize launch is left with 64 rows:
// 12544 rows, step at batch 256: 64 channels 25 -> 14, 256 channels 33 -> 16 us with both launches, beside the weight gradients
// 55 to 87 -> 25 to 60; the step 20.27 -> 20.15 ms.  At 3136 rows the finalize launch alone takes 9 us, as long as both.
template <bool BWD>
__global__ __launch_bounds__(256) void bn_reduce_rows_kernel(const float* __restrict__ partial, int nrows, int per, int rpp,
                                                             int64_t m, double2* __restrict__ out) {
  __shared__ double red[2][4][8];
  const int ch = threadIdx.x & 7, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t base = bn_sums_at(0, blockIdx.x * 8 + ch, nrows);
  const int b0 = blockIdx.y * per, b1 = min(b0 + per, nrows);
  double s1 = 0.0, s2 = 0.0;
  if constexpr (BWD) {
    const float2* p = reinterpret_cast<const float2*>(partial) + base;
    for (int b = b0 + (threadIdx.x >> 3); b < b1; b += 32 * kFinRows) {
      float2 v[kFinRows];
#pragma unroll
      for (int u = 0; u < kFinRows; ++u) v[u] = p[min(b + u * 32, b1 - 1) * 8];
#pragma unroll
      for (int u = 0; u < kFinRows; ++u) {
        if (b + u * 32 < b1) {
          s1 += static_cast<double>(v[u].x);
          s2 += static_cast<double>(v[u].y);
        }
      }
    }
  } else {
    const BnTileRow* p = reinterpret_cast<const BnTileRow*>(partial) + base;
    const double k0 = static_cast<double>(p[0].k);
    for (int b = b0 + (threadIdx.x >> 3); b < b1; b += 32 * kFinRows) {
      BnTileRow v[kFinRows];
#pragma unroll
      for (int u = 0; u < kFinRows; ++u) v[u] = p[min(b + u * 32, b1 - 1) * 8];
#pragma unroll
      for (int u = 0; u < kFinRows; ++u)
        if (b + u * 32 < b1) add_tile_row(v[u], rows_of(b + u * 32, nrows, rpp, m), k0, &s1, &s2);
    }
  }
#pragma unroll
  for (int off = 32; off >= 8; off >>= 1) {
    s1 += __shfl_xor(s1, off, 64);
    s2 += __shfl_xor(s2, off, 64);
  }
  if (lane < 8) {
    red[0][wave][ch] = s1;
    red[1][wave][ch] = s2;
  }
  __syncthreads();
  if (threadIdx.x >= 8) return;
  out[bn_sums_at(blockIdx.y, blockIdx.x * 8 + ch, kBnReducedRows)] =
      make_double2(((red[0][0][ch] + red[0][1][ch]) + red[0][2][ch]) + red[0][3][ch],
                   ((red[1][0][ch] + red[1][1][ch]) + red[1][2][ch]) + red[1][3][ch]);
}
void bn_reduce_rows(float* sums, int nrows, int rpp, int64_t m, int C, bool backward, hipStream_t s) {
  const dim3 grid(static_cast<unsigned>(ceil_div(C, 8)), kBnReducedRows);
  const int per = static_cast<int>(ceil_div(nrows, kBnReducedRows));
  double2* out = bn_reduced_rows(sums, nrows, C, backward);
  if (backward) RN50_LAUNCH("bn_bwd_finalize", bn_reduce_rows_kernel<true>, grid, dim3(256), 0, s, sums, nrows, per, rpp, m, out);
  else RN50_LAUNCH("bn_finalize", bn_reduce_rows_kernel<false>, grid, dim3(256), 0, s, sums, nrows, per, rpp, m, out);
}

// What a pass that finalizes statistics gets: the rows of sums and where the results go (backward: mean_out = dbeta, rstd_out =
// dgamma).
struct BnFinArgs {
  const float* partial;
  int nrows, rpp;      // tile rows, rows of x behind each
  const double2* wide; // finalize launch and shared: rows of doubles instead (bn_reduced_rows, or about zero with partial null)
  int nwide;
  float eps, momentum;
  float *mean_out, *rstd_out, *running_mean, *running_var;
  // shared
  unsigned long long* slots;  // per channel: the two results, or kBnSlotEmpty
  int groups, polls;          // finalizing workgroups; how often the others ask for their results
  int nblk;                   // applying workgroups per column slice
};

// Forward: mean and 1/std of kFinCh channels by the 256 threads of a workgroup, from rows of sums over rpp rows of x each (the last
// over what is left of m), with their shifts; or (wide not null) rows of doubles: about zero (for a layer whose apply pass is left
// to its consumer), or reduced, about the shift of partial's first row.  True in the threads that hold a channel's results;
// `store`: they also go to memory.
__device__ __forceinline__ bool finalize_channels_fwd(const BnFinArgs& f, int group, int64_t m, int C, bool store, float* mean_r,
                                                      float* rstd_r) {
  constexpr int G = kFinThreads / kFinCh;
  const int c = group * kFinCh + threadIdx.x % kFinCh;
  int nrows = f.nrows;
  const BnTileRow* p = reinterpret_cast<const BnTileRow*>(f.partial) + bn_sums_at(0, c, nrows);  // (the last piece of C is padded)
  const double k0 = f.partial ? static_cast<double>(p[0].k) : 0.0;
  double s1 = 0.0, s2 = 0.0;
  if (f.wide) {
    const double2* pd = f.wide + bn_sums_at(0, c, f.nwide);
    for (int b = threadIdx.x / kFinCh; b < f.nwide; b += G) {
      s1 += pd[b * 8].x;
      s2 += pd[b * 8].y;
    }
    nrows = 0;
  }
  for (int b = threadIdx.x / kFinCh; b < nrows; b += kFinRows * G) {
    BnTileRow v[kFinRows];
#pragma unroll
    for (int u = 0; u < kFinRows; ++u) v[u] = p[min(b + u * G, nrows - 1) * 8];
#pragma unroll
    for (int u = 0; u < kFinRows; ++u)
      if (b + u * G < nrows) add_tile_row(v[u], rows_of(b + u * G, nrows, f.rpp, m), k0, &s1, &s2);
  }
  finalize_combine(&s1, &s2);
  if (threadIdx.x >= kFinCh || c >= C) return false;
  const double d = s1 / static_cast<double>(m), mean = k0 + d;
  double var = s2 / static_cast<double>(m) - d * d;
  if (var < 0.0) var = 0.0;
  *mean_r = static_cast<float>(mean);
  *rstd_r = static_cast<float>(1.0 / sqrt(var + static_cast<double>(f.eps)));
  if (store) {
    f.mean_out[c] = *mean_r;
    f.rstd_out[c] = *rstd_r;
    if (f.running_mean) f.running_mean[c] = f.momentum * f.running_mean[c] + (1.f - f.momentum) * static_cast<float>(mean);
    if (f.running_var) f.running_var[c] = f.momentum * f.running_var[c] + (1.f - f.momentum) * static_cast<float>(var);
  }
  return true;
}
// Backward: (dbeta, dgamma) likewise.
__device__ __forceinline__ bool finalize_channels_bwd(const BnFinArgs& f, int group, int C, bool store, float* dbeta_r,
                                                      float* dgamma_r) {
  constexpr int G = kFinThreads / kFinCh;
  const int c = group * kFinCh + threadIdx.x % kFinCh;
  int nrows = f.nrows;
  const float2* p = reinterpret_cast<const float2*>(f.partial) + bn_sums_at(0, c, nrows);
  double s1 = 0.0, s2 = 0.0;
  if (f.wide) {
    const double2* pd = f.wide + bn_sums_at(0, c, f.nwide);
    for (int b = threadIdx.x / kFinCh; b < f.nwide; b += G) {
      s1 += pd[b * 8].x;
      s2 += pd[b * 8].y;
    }
    nrows = 0;
  }
  for (int b = threadIdx.x / kFinCh; b < nrows; b += kFinRows * G) {
    float2 v[kFinRows];
#pragma unroll
    for (int u = 0; u < kFinRows; ++u) v[u] = p[min(b + u * G, nrows - 1) * 8];
#pragma unroll
    for (int u = 0; u < kFinRows; ++u) {
      if (b + u * G < nrows) {
        s1 += static_cast<double>(v[u].x);
        s2 += static_cast<double>(v[u].y);
      }
    }
  }
  finalize_combine(&s1, &s2);
  if (threadIdx.x >= kFinCh || c >= C) return false;
  *dbeta_r = static_cast<float>(s1);
  *dgamma_r = static_cast<float>(s2);
  if (store) {
    f.mean_out[c] = *dbeta_r;
    f.rstd_out[c] = *dgamma_r;
  }
  return true;
}
template <bool BWD>
__device__ __forceinline__ bool finalize_channels(const BnFinArgs& f, int group, int64_t m, int C, bool store, float* a, float* b) {
  return BWD ? finalize_channels_bwd(f, group, C, store, a, b) : finalize_channels_fwd(f, group, m, C, store, a, b);
}
template <bool BWD>
__global__ __launch_bounds__(kFinThreads) void bn_finalize_kernel(int64_t m, int C, const BnFinArgs f) {
  request_kernel_args<16 + sizeof(BnFinArgs)>();
  float a, b;
  finalize_channels<BWD>(f, blockIdx.x, m, C, true, &a, &b);
}

// Where an apply pass has its statistics from.  kFinGiven: from memory, a finalize launch has stored them.  kFinSelf: every
// workgroup adds up the tile rows of its channels.  kFinShared: the first `groups` workgroups of the same launch finalize, two
// channels each, and publish the two results of a channel as one 64-bit word; the others request their rows of x and then ask
// for the words of their channels.  Two launches in one: 11 to 13 us for 4.6 to 5.5 + 1.5 (between them) + 7 at 56x56, batch 40.  Four
// workgroups of these kernels are on a compute unit at a time (117 to 126 registers, as without the sharing), 1024 on the chip; those of
// a larger grid that come later find the results there.  The step with the sharing for grids of at most 0 / 1024 / 2048 / 4096 workgroups /
// all, ms (profiles/step_time_against_dispatch_constants.txt):
//   batch 12 2.498 / 2.438 / 2.439 / 2.439 / 2.439, 24 3.368 / 3.336 / 3.320 / 3.319 / 3.317, 40 4.272 / 4.244 / 4.235 / 4.235 / 4.236,
//   90 8.070 / 8.029 / 8.029 / 7.978 / 7.954, 256 19.17 / 19.16 / 19.17 / 19.16 / 19.09, float at batch 8 4.013 / 4.004 / 4.016 /
//   4.011 / 4.014;
// with the present kernels, 2048 / all: batch 90 8.029 / 7.984, 128 at 192 px 8.295 / 8.244, 256 19.10 / 19.06, 40 the same.  (Stand-alone calls,
// their sums passes making the words empty, gained nothing from it: batch 40 520 / 523 us, batch 200 2004 / 2019.)
// kFinSelf stays for its few rows: with kFinShared in its place (from 0 / 40 / 64 rows on) batch 12 loses 2.3 / 0.2 / 0.2 %.
// The word is the message: relaxed atomics at device scope, nothing else is passed by memory within the launch.  It is made empty
// by the convolution that produces the sums (IgemmArgs::slots).  No progress is assumed of the finalizing workgroups: after
// `polls` unanswered questions a workgroup computes what it needs itself, in the same order, so every wait ends and the results
// do not depend on who computed them.
enum BnFin { kFinGiven, kFinSelf, kFinShared };
__device__ __forceinline__ void publish_results(unsigned long long* slot, float a, float b) {
  unsigned long long v = static_cast<unsigned long long>(__float_as_uint(b)) << 32 | __float_as_uint(a);
  if (v == kBnSlotEmpty) v = 0x7fc000007fc00000ull;  // (two NaNs)
  __hip_atomic_store(slot, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The results of the `width` channels (at most 256) from c0 on into LDS; ends with a barrier.
template <bool BWD>
__device__ __forceinline__ void await_results(const BnFinArgs& f, int64_t m, int C, int c0, int width, float* a_s, float* b_s) {
  const int tid = threadIdx.x;
  bool missing = false;
  if (tid < width && c0 + tid < C) {
    missing = true;
    for (int i = 0; i < f.polls && missing; ++i) {
      const unsigned long long v = __hip_atomic_load(f.slots + c0 + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (v != kBnSlotEmpty) {
        a_s[tid] = __uint_as_float(static_cast<uint32_t>(v));
        b_s[tid] = __uint_as_float(static_cast<uint32_t>(v >> 32));
        missing = false;
      } else {
        __builtin_amdgcn_s_sleep(2);
      }
    }
  }
  if (__syncthreads_or(missing)) {
    for (int i = 0; i < width && c0 + i < C; i += kFinCh) {
      float a, b;
      if (finalize_channels<BWD>(f, (c0 + i) / kFinCh, m, C, false, &a, &b)) {
        a_s[i + tid] = a;
        b_s[i + tid] = b;
      }
      __syncthreads();  // (before the next ones use the same LDS)
    }
  }
}

// Forward statistics of the CS channels from c0 on, by all 256 threads of a workgroup, into mean_s / rstd_s (LDS).
// Thread (channel ch, part p) adds tile rows p, p + P, ... in order, the P parts
// are added in order: a fixed order, the same in every workgroup that computes these channels.  Ends with a barrier.
template <int CS>
__device__ __forceinline__ void finalize_slice_fwd(const BnFinArgs& f, int64_t m, int C, int c0, bool writer,
                                                   float* mean_s, float* rstd_s) {
  constexpr int P = 256 / CS, U = 4;
  __shared__ double red[2][256];
  const int ch = threadIdx.x % CS, part = threadIdx.x / CS;
  const int c = min(c0 + ch, C - 1);
  const double2* pk = reinterpret_cast<const double2*>(f.partial) + bn_sums_at(0, c, f.nrows);
  double s1 = 0.0, s2 = 0.0;
  for (int b = part; b < f.nrows; b += P * U) {
    double2 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = pk[min(b + u * P, f.nrows - 1) * 8];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (b + u * P < f.nrows) {
        s1 += v[u].x;
        s2 += v[u].y;
      }
    }
  }
  red[0][threadIdx.x] = s1;
  red[1][threadIdx.x] = s2;
  __syncthreads();
  if (threadIdx.x < CS) {
    double t1 = red[0][ch], t2 = red[1][ch];
#pragma unroll
    for (int q = 1; q < P; ++q) {
      t1 += red[0][q * CS + ch];
      t2 += red[1][q * CS + ch];
    }
    const double mean = t1 / static_cast<double>(m);
    double var = t2 / static_cast<double>(m) - mean * mean;
    if (var < 0.0) var = 0.0;
    const float mf = static_cast<float>(mean), rf = static_cast<float>(1.0 / sqrt(var + static_cast<double>(f.eps)));
    mean_s[ch] = mf;
    rstd_s[ch] = rf;
    if (writer && c0 + ch < C) {
      f.mean_out[c] = mf;
      f.rstd_out[c] = rf;
      if (f.running_mean) f.running_mean[c] = f.momentum * f.running_mean[c] + (1.f - f.momentum) * mf;
      if (f.running_var) f.running_var[c] = f.momentum * f.running_var[c] + (1.f - f.momentum) * static_cast<float>(var);
    }
  }
  __syncthreads();
}

// FIN: where the statistics come from (BnFin).  kFinSelf: every workgroup for the 8 vector columns it applies (tx_log2 = 3), and
// the first row block of every column slice stores them: no finalize launch in front.  For layers with few tile rows the redundant
// reads of the sums are far cheaper than a launch on the step's dependency chain (about 4 us whatever it computes).  kFinShared: a
// one-dimensional grid.
// LAST (apply passes of both directions): nobody reads the operands again for a long while, as in a training step, where the
// next layers are larger than the caches: their loads bypass the caches, which keep what the next kernel reads -- the output,
// the weight gradient's operands.  Whole step: batch 40 4.506 -> 4.457 ms, batch 256 20.90 -> 20.55 (stores past the caches
// made batch 40 slower).  Not for the calls of one operation, whose next one may read the same tensor: bn_relu_fwd and then
// bn_relu_bwd over ResNet-50's layers at batch 40 take 589 us with these loads and 523 without.
template <typename T, BnFin FIN, bool LAST, bool THROUGH>
__global__ __launch_bounds__(256) void bn_apply_kernel(const T* __restrict__ x,
                                                       const float* __restrict__ gamma,
                                                       const float* __restrict__ beta,
                                                       const float* __restrict__ mean,
                                                       const float* __restrict__ rstd,
                                                       const T* __restrict__ residual,
                                                       T* __restrict__ y, uint8_t* __restrict__ relu_mask,
                                                       int64_t m, int C, int tx_log2, int rpb, int mode,
                                                       int through, const BnFinArgs fin) {
  constexpr int V = Elem<T>::VEC;
  request_kernel_args<96 + sizeof(BnFinArgs)>();
  const OutTensor<T, THROUGH> out(y, through);
  const int TX = 1 << tx_log2, TY = 256 >> tx_log2;
  const int tcol = threadIdx.x & (TX - 1), trow = threadIdx.x >> tx_log2;
  int bx = blockIdx.x, by = blockIdx.y;
  if constexpr (FIN == kFinShared) {
    if (bx < fin.groups) {
      float a, b;
      if (finalize_channels<false>(fin, bx, m, C, true, &a, &b)) publish_results(fin.slots + bx * kFinCh + threadIdx.x, a, b);
      return;
    }
    bx -= fin.groups;
    by = bx / fin.nblk;
    bx -= by * fin.nblk;
  }
  const int col = by * TX + tcol;
  constexpr int kStats = FIN == kFinSelf ? 8 * V : (FIN == kFinShared ? 32 * V : 1);
  __shared__ __align__(16) float mean_s[kStats], rstd_s[kStats];
  if (FIN == kFinGiven && col >= C / V) return;
  const bool live = col < C / V;  // (else: every thread takes part in the statistics)
  const int64_t r0 = static_cast<int64_t>(bx) * rpb;
  const int64_t r1 = min(r0 + rpb, m);
  int64_t r = r0 + trow;
  int64_t off[kBnRows];
  Vec16 vx[kBnRows], vr[kBnRows];
  auto load_rows = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < kBnRows; ++u) {
      off[u] = min(r + u * TY, r1 - 1) * C + static_cast<int64_t>(col) * V;
      vx[u] = LAST ? load16_stream(x + off[u]) : load16(x + off[u]);
    }
    if (mode == 2) {
#pragma unroll
      for (int u = 0; u < kBnRows; ++u) vr[u] = LAST ? load16_stream(residual + off[u]) : load16(residual + off[u]);
    }
  };
  // the first rows are requested before the per-channel values, so both arrive in one round trip
  if (live && r < r1) load_rows();
  float scale[V], bias[V], cg[V], cb[V], cm[V], cr[V];
  if (live) {
    load_floats<V>(gamma + col * V, cg);
    load_floats<V>(beta + col * V, cb);
  }
  if constexpr (FIN != kFinGiven) {
    if constexpr (FIN == kFinSelf) finalize_slice_fwd<8 * V>(fin, m, C, by * 8 * V, bx == 0, mean_s, rstd_s);
    else await_results<false>(fin, m, C, by * TX * V, TX * V, mean_s, rstd_s);
    if (!live) return;
    load_floats<V>(mean_s + tcol * V, cm);
    load_floats<V>(rstd_s + tcol * V, cr);
  } else {
    load_floats<V>(mean + col * V, cm);
    load_floats<V>(rstd + col * V, cr);
  }
#pragma unroll
  for (int j = 0; j < V; ++j) bn_coeffs(cg[j], cb[j], cm[j], cr[j], &scale[j], &bias[j]);
  for (; r < r1; r += kBnRows * TY) {
    if (r != r0 + trow) load_rows();
#pragma unroll
    for (int u = 0; u < kBnRows; ++u) {
      if (r + u * TY < r1) {
        float f[V];
        Elem<T>::unpack(vx[u], f);
        if (mode == 2) {
          float rr[V];
          Elem<T>::unpack(vr[u], rr);
#pragma unroll
          for (int j = 0; j < V; ++j) f[j] = fmaxf(bn_affine(f[j], scale[j], bias[j]) + rr[j], 0.f);
        } else if (mode == 1) {
#pragma unroll
          for (int j = 0; j < V; ++j) f[j] = fmaxf(bn_affine(f[j], scale[j], bias[j]), 0.f);
        } else {
#pragma unroll
          for (int j = 0; j < V; ++j) f[j] = bn_affine(f[j], scale[j], bias[j]);
        }
        Vec16 o;
        Elem<T>::pack(f, o);
        out.store(off[u], o);
        if (relu_mask) {  // bit j: stored output j is positive; one byte per 16-byte vector
          float zf[V];
          Elem<T>::unpack(o, zf);
          uint32_t bits = 0;
#pragma unroll
          for (int j = 0; j < V; ++j) bits |= (zf[j] > 0.f ? 1u : 0u) << j;
          relu_mask[off[u] / V] = static_cast<uint8_t>(bits);
        }
      }
    }
  }
}

// ------------------------------------------------------------------ backward
// The backward kernels are compiled per operand set, so that a thread only holds registers for what its
// launch reads: DZ2 = a second gradient branch is added; ZK = where the ReLU decision comes from
// (0: recomputed from x, or no ReLU; 1: the forward output z; 2: the recorded bits).
// The operands of kBnRows rows, loaded before any is used.
template <bool DZ2, int ZK>
struct BwdRows {
  Vec16 x[kBnRows], dz[kBnRows], dz2[DZ2 ? kBnRows : 1], z[ZK == 1 ? kBnRows : 1];
  uint32_t zbits[ZK == 2 ? kBnRows : 1];
  int64_t off[kBnRows];
};
template <bool LAST, typename T, bool DZ2, int ZK>
__device__ __forceinline__ void load_bwd_rows(BwdRows<DZ2, ZK>& b, const T* dz, const T* dz2, const T* x,
                                              const T* z, const uint8_t* zmask, int64_t r, int64_t r1, int TY,
                                              int C, int col) {
  constexpr int V = Elem<T>::VEC;
#pragma unroll
  for (int u = 0; u < kBnRows; ++u) {
    b.off[u] = min(r + u * TY, r1 - 1) * C + static_cast<int64_t>(col) * V;
    b.x[u] = LAST ? load16_stream(x + b.off[u]) : load16(x + b.off[u]);
    b.dz[u] = LAST ? load16_stream(dz + b.off[u]) : load16(dz + b.off[u]);
  }
  if (DZ2) {
#pragma unroll
    for (int u = 0; u < kBnRows; ++u) b.dz2[DZ2 ? u : 0] = load16(dz2 + b.off[u]);
  }
  if (ZK == 2) {
#pragma unroll
    for (int u = 0; u < kBnRows; ++u) b.zbits[ZK == 2 ? u : 0] = zmask[b.off[u] / V];
  } else if (ZK == 1) {
#pragma unroll
    for (int u = 0; u < kBnRows; ++u) b.z[ZK == 1 ? u : 0] = load16(z + b.off[u]);
  }
}

// The same where all of the workgroup's rows from rb on are there (b.off is left alone).
template <typename T, bool DZ2, int ZK>
__device__ __forceinline__ void load_bwd_whole_rows(BwdRows<DZ2, ZK>& b, const T* dz, const T* dz2, const T* x, const T* z,
                                                    const uint8_t* zmask, int64_t rb, int TY, int C, uint32_t lane_elem) {
  constexpr int V = Elem<T>::VEC;
  const uint32_t lane_off = lane_elem * static_cast<uint32_t>(sizeof(T)), lane_vec = lane_elem / V;
#pragma unroll
  for (int u = 0; u < kBnRows; ++u) {
    const int64_t at = (rb + u * TY) * C;
    b.x[u] = load16_at(x + at, lane_off);
    b.dz[u] = load16_at(dz + at, lane_off);
  }
#pragma unroll
  for (int u = 0; u < kBnRows; ++u) {
    const int64_t at = (rb + u * TY) * C;
    if (DZ2) b.dz2[DZ2 ? u : 0] = load16_at(dz2 + at, lane_off);
    if (ZK == 2) b.zbits[ZK == 2 ? u : 0] = (zmask + at / V)[lane_vec];
    else if (ZK == 1) b.z[ZK == 1 ? u : 0] = load16_at(z + at, lane_off);
  }
}

// g = (dz + dz2) * mask for one 16-byte vector.
template <typename T, bool DZ2, int ZK>
__device__ __forceinline__ void masked_grad(const BwdRows<DZ2, ZK>& b, int u, const float* xf, const float* scale,
                                            const float* bias, int mode, float* g) {
  constexpr int V = Elem<T>::VEC;
  const Vec16& vdz = b.dz[u];
  const Vec16& vdz2 = b.dz2[DZ2 ? u : 0];
  const Vec16& vz = b.z[ZK == 1 ? u : 0];
  const uint32_t zbits = b.zbits[ZK == 2 ? u : 0];
  constexpr bool has_dz2 = DZ2, has_z = ZK == 1, has_zbits = ZK == 2;
  Elem<T>::unpack(vdz, g);
  if (has_dz2) {
    float g2[V];
    Elem<T>::unpack(vdz2, g2);
#pragma unroll
    for (int j = 0; j < V; ++j) g[j] += g2[j];
  }
  if (mode >= 1) {
    if (has_zbits) {
#pragma unroll
      for (int j = 0; j < V; ++j) g[j] = (zbits >> j) & 1u ? g[j] : 0.f;
    } else if (has_z) {
      float zf[V];
      Elem<T>::unpack(vz, zf);
#pragma unroll
      for (int j = 0; j < V; ++j) g[j] = zf[j] > 0.f ? g[j] : 0.f;
    } else {
#pragma unroll
      for (int j = 0; j < V; ++j) g[j] = bn_affine(xf[j], scale[j], bias[j]) > 0.f ? g[j] : 0.f;
    }
  }
}

template <typename T, bool DZ2, int ZK>
__global__ __launch_bounds__(256) void bn_bwd_reduce_kernel(
    const T* __restrict__ dz, const T* __restrict__ dz2, const T* __restrict__ x,
    const T* __restrict__ z, const uint8_t* __restrict__ zmask, const float* __restrict__ gamma,
    const float* __restrict__ beta,
    const float* __restrict__ mean, const float* __restrict__ rstd, int64_t m, int C, int tx_log2,
    int rpb, int mode, float* __restrict__ partial) {
  constexpr int V = Elem<T>::VEC;
  __shared__ float lds[4 * 2 * V * 32];
  const int TX = 1 << tx_log2, TY = 256 >> tx_log2;
  const int tcol = threadIdx.x & (TX - 1), trow = threadIdx.x >> tx_log2;
  const int col = blockIdx.y * TX + tcol;
  const bool active = col < C / V;
  float acc[2 * V];
#pragma unroll
  for (int j = 0; j < 2 * V; ++j) acc[j] = 0.f;
  if (active) {
    float scale[V], bias[V], rs[V], nmr[V], cg[V], cb[V], cm[V];
    load_floats<V>(gamma + col * V, cg);
    load_floats<V>(mean + col * V, cm);
    load_floats<V>(rstd + col * V, rs);
    if (beta) {
      load_floats<V>(beta + col * V, cb);
    } else {
#pragma unroll
      for (int j = 0; j < V; ++j) cb[j] = 0.f;
    }
#pragma unroll
    for (int j = 0; j < V; ++j) {
      nmr[j] = -cm[j] * rs[j];
      bn_coeffs(cg[j], cb[j], cm[j], rs[j], &scale[j], &bias[j]);
    }
    const int64_t r0 = static_cast<int64_t>(blockIdx.x) * rpb;
    const int64_t r1 = min(r0 + rpb, m);
    const uint32_t lane_elem = static_cast<uint32_t>(trow) * C + static_cast<uint32_t>(col) * V;
    auto add = [&](const BwdRows<DZ2, ZK>& b, int u) __attribute__((always_inline)) {
      float xf[V], g[V];
      Elem<T>::unpack(b.x[u], xf);
      masked_grad<T, DZ2, ZK>(b, u, xf, scale, bias, mode, g);
#pragma unroll
      for (int j = 0; j < V; ++j) {
        acc[j] += g[j];
        acc[V + j] = fmaf(g[j], fmaf(xf[j], rs[j], nmr[j]), acc[V + j]);
      }
    };
    for (int64_t rb = r0; rb < r1; rb += kBnRows * TY) {
      BwdRows<DZ2, ZK> b;
      if (rb + kBnRows * TY <= r1 && C <= kBnLaneOffsetChannels) {
        load_bwd_whole_rows<T, DZ2, ZK>(b, dz, dz2, x, z, zmask, rb, TY, C, lane_elem);
#pragma unroll
        for (int u = 0; u < kBnRows; ++u) add(b, u);
      } else {
        load_bwd_rows<false, T, DZ2, ZK>(b, dz, dz2, x, z, zmask, rb + trow, r1, TY, C, col);
#pragma unroll
        for (int u = 0; u < kBnRows; ++u)
          if (rb + trow + u * TY < r1) add(b, u);
      }
    }
  }
  float t1, t2;
  const int c = blockIdx.y * TX * V + threadIdx.x;
  if (!combine_sums<V>(acc, lds, tx_log2, &t1, &t2) || c >= C) return;
  reinterpret_cast<float2*>(partial)[bn_sums_at(blockIdx.x, c, gridDim.x)] = make_float2(t1, t2);
}

// Backward sums (sum g, sum g * xhat) of the CS channels from c0 on, by all 256 threads, in double and in the fixed order of
// finalize_slice_fwd; dbeta / dgamma land in db_s / dg_s (LDS).  Ends with a barrier.
template <int CS>
__device__ __forceinline__ void finalize_slice_bwd(const BnFinArgs& f, int C, int c0, bool writer, float* db_s,
                                                   float* dg_s) {
  constexpr int P = 256 / CS, U = 4;
  __shared__ double red[2][256];
  const int ch = threadIdx.x % CS, part = threadIdx.x / CS;
  const int c = min(c0 + ch, C - 1);
  const float2* pk = reinterpret_cast<const float2*>(f.partial) + bn_sums_at(0, c, f.nrows);
  double s1 = 0.0, s2 = 0.0;
  for (int b = part; b < f.nrows; b += P * U) {
    float2 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = pk[min(b + u * P, f.nrows - 1) * 8];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (b + u * P < f.nrows) {
        s1 += static_cast<double>(v[u].x);
        s2 += static_cast<double>(v[u].y);
      }
    }
  }
  red[0][threadIdx.x] = s1;
  red[1][threadIdx.x] = s2;
  __syncthreads();
  if (threadIdx.x < CS) {
    double t1 = red[0][ch], t2 = red[1][ch];
#pragma unroll
    for (int q = 1; q < P; ++q) {
      t1 += red[0][q * CS + ch];
      t2 += red[1][q * CS + ch];
    }
    db_s[ch] = static_cast<float>(t1);
    dg_s[ch] = static_cast<float>(t2);
    if (writer && c0 + ch < C) {
      f.mean_out[c] = static_cast<float>(t1);  // dbeta
      f.rstd_out[c] = static_cast<float>(t2);  // dgamma
    }
  }
  __syncthreads();
}

// FIN, LAST: as in bn_apply_kernel -- kFinSelf: the pass adds up the per-tile sums of its 8 vector columns itself
// (tx_log2 = 3) and the first row block of every column slice stores dgamma / dbeta.
template <typename T, bool DZ2, int ZK, BnFin FIN, bool LAST, bool THROUGH>
__global__ __launch_bounds__(256) void bn_bwd_apply_kernel(
    const T* __restrict__ dz, const T* __restrict__ dz2, const T* __restrict__ x,
    const T* __restrict__ z, const uint8_t* __restrict__ zmask, const float* __restrict__ gamma,
    const float* __restrict__ beta,
    const float* __restrict__ mean, const float* __restrict__ rstd,
    const float* __restrict__ dgamma, const float* __restrict__ dbeta, T* __restrict__ dx,
    T* __restrict__ dres, int64_t m, int C, int tx_log2, int rpb, int mode, int through, const BnFinArgs fin) {
  constexpr int V = Elem<T>::VEC;
  request_kernel_args<136 + sizeof(BnFinArgs)>();
  const OutTensor<T, THROUGH> out(dx, through);
  const int TX = 1 << tx_log2, TY = 256 >> tx_log2;
  const int tcol = threadIdx.x & (TX - 1), trow = threadIdx.x >> tx_log2;
  int bx = blockIdx.x, by = blockIdx.y;
  if constexpr (FIN == kFinShared) {
    if (bx < fin.groups) {
      float a, b;
      if (finalize_channels<true>(fin, bx, m, C, true, &a, &b)) publish_results(fin.slots + bx * kFinCh + threadIdx.x, a, b);
      return;
    }
    bx -= fin.groups;
    by = bx / fin.nblk;
    bx -= by * fin.nblk;
  }
  int col = by * TX + tcol;
  constexpr int kStats = FIN == kFinSelf ? 8 * V : (FIN == kFinShared ? 32 * V : 1);
  __shared__ __align__(16) float db_s[kStats], dg_s[kStats];
  if (FIN == kFinGiven && col >= C / V) return;
  const bool live = col < C / V;  // (else: every thread takes part in the sums)
  if (!live) col = C / V - 1;      // (its loads stay in range; it leaves before it stores anything)
  const int64_t r0 = static_cast<int64_t>(bx) * rpb;
  const int64_t r1 = min(r0 + rpb, m);
  int64_t r = r0 + trow;
  // the first rows are requested before the per-channel values, so both arrive in one round trip
  BwdRows<DZ2, ZK> b;
  if (live && r < r1) load_bwd_rows<LAST, T, DZ2, ZK>(b, dz, dz2, x, z, zmask, r, r1, TY, C, col);
  const float inv_m = 1.0f / static_cast<float>(m);
  float scale[V], bias[V], rs[V], nmr[V], mg[V], mgx[V], cg[V], cb[V], cm[V];
  load_floats<V>(gamma + col * V, cg);
  load_floats<V>(mean + col * V, cm);
  load_floats<V>(rstd + col * V, rs);
  if constexpr (FIN != kFinGiven) {
    if constexpr (FIN == kFinSelf) finalize_slice_bwd<8 * V>(fin, C, by * 8 * V, bx == 0, db_s, dg_s);
    else await_results<true>(fin, m, C, by * TX * V, TX * V, db_s, dg_s);
    if (!live) return;
    load_floats<V>(db_s + tcol * V, mg);
    load_floats<V>(dg_s + tcol * V, mgx);
  } else {
    load_floats<V>(dbeta + col * V, mg);
    load_floats<V>(dgamma + col * V, mgx);
  }
  if (beta) {
    load_floats<V>(beta + col * V, cb);
  } else {
#pragma unroll
    for (int j = 0; j < V; ++j) cb[j] = 0.f;
  }
#pragma unroll
  for (int j = 0; j < V; ++j) {
    nmr[j] = -cm[j] * rs[j];
    bn_coeffs(cg[j], cb[j], cm[j], rs[j], &scale[j], &bias[j]);
    mg[j] *= inv_m;
    mgx[j] *= inv_m;
  }
  for (; r < r1; r += kBnRows * TY) {
    if (r != r0 + trow) load_bwd_rows<LAST, T, DZ2, ZK>(b, dz, dz2, x, z, zmask, r, r1, TY, C, col);
#pragma unroll
    for (int u = 0; u < kBnRows; ++u) {
      if (r + u * TY < r1) {
        float xf[V], g[V], o[V];
        Elem<T>::unpack(b.x[u], xf);
        masked_grad<T, DZ2, ZK>(b, u, xf, scale, bias, mode, g);
#pragma unroll
        for (int j = 0; j < V; ++j) {
          const float xh = fmaf(xf[j], rs[j], nmr[j]);
          o[j] = scale[j] * (g[j] - mg[j] - xh * mgx[j]);
        }
        Vec16 ov;
        Elem<T>::pack(o, ov);
        out.store(b.off[u], ov);
        if (mode == 2 && dres) {
          Vec16 gv;
          Elem<T>::pack(g, gv);
          store16(dres + b.off[u], gv);
        }
      }
    }
  }
}

static int check_desc(const rn50_bn_desc* d, const char* who) {
  RN50_REQUIRE(d, RN50_ERR_INVALID, "%s: null descriptor", who);
  RN50_REQUIRE(d->N > 0 && d->H > 0 && d->W > 0 && d->C > 0, RN50_ERR_INVALID,
               "%s: non-positive size N=%d H=%d W=%d C=%d", who, d->N, d->H, d->W, d->C);
  RN50_REQUIRE(d->dtype == RN50_F32 || d->dtype == RN50_BF16, RN50_ERR_INVALID, "%s: dtype %d", who, d->dtype);
  RN50_REQUIRE(d->mode >= 0 && d->mode <= 2, RN50_ERR_INVALID, "%s: mode %d", who, d->mode);
  RN50_REQUIRE(d->C % (d->dtype == RN50_BF16 ? 8 : 4) == 0, RN50_ERR_UNSUPPORTED,
               "%s: C=%d is not a multiple of the 16-byte vector", who, d->C);
  RN50_REQUIRE(d->eps >= 0.f, RN50_ERR_INVALID, "%s: eps < 0", who);
  return RN50_OK;
}

int bn_desc_check(const rn50_bn_desc* d, const char* who) { return check_desc(d, who); }

static size_t bn_ws_bytes(const rn50_bn_desc* d) {
  const int64_t m = static_cast<int64_t>(d->N) * d->H * d->W;
  const BnGeom g = bn_sums_geom(m, d->C, d->dtype);
  return align_up(bn_sums_bytes(g.nblk, d->C, bn_self_sums(m, d->C) ? kBnWideSumBytes : kBnTileRowBytes), 256);
}

// finalize + apply from partial statistics rows (see bn_finalize_kernel).  reduces: their producer is a convolution, which
// leaves them reduced where they are many.  share (or null): finalize and apply in one launch where that is two.
template <typename T, bool LAST>
static void launch_fwd_tail(const rn50_bn_desc* d, int64_t m, const void* x,
                            const float* gamma, const float* beta, const void* residual, void* y,
                            uint8_t* relu_mask, float* save_mean, float* save_rstd, float* rm, float* rv,
                            float momentum, const float* partial, int nrows, int rpp, bool self, bool reduces, const BnShare* share,
                            hipStream_t s) {
  const int through = writes_through(m * d->C * sizeof(T));
  BnFinArgs fin{};
  fin.partial = partial; fin.nrows = nrows; fin.rpp = rpp;
  fin.eps = d->eps; fin.momentum = momentum;
  fin.mean_out = save_mean; fin.rstd_out = save_rstd; fin.running_mean = rm; fin.running_var = rv;
#define RN50_FWD_APPLY_T(FIN, THROUGH, GRID, MEAN, RSTD, TXL, RPB)                                                                 \
  RN50_LAUNCH("bn_apply", (bn_apply_kernel<T, FIN, LAST, THROUGH>), GRID, dim3(256), 0, s, static_cast<const T*>(x), gamma, beta, MEAN, \
              RSTD, static_cast<const T*>(residual), static_cast<T*>(y), relu_mask, m, d->C, TXL, RPB, d->mode, through, fin)
#define RN50_FWD_APPLY(FIN, GRID, MEAN, RSTD, TXL, RPB)                    \
  do {                                                                     \
    if (through) RN50_FWD_APPLY_T(FIN, true, GRID, MEAN, RSTD, TXL, RPB);  \
    else RN50_FWD_APPLY_T(FIN, false, GRID, MEAN, RSTD, TXL, RPB);         \
  } while (0)
  if (self && y) {
    // few tile rows: the apply pass finalizes for itself
    int gy, rpb;
    bn_self_finalize_geom(m, d->C, d->dtype == RN50_BF16 ? 8 : 4, &gy, &rpb);
    RN50_FWD_APPLY(kFinSelf, dim3(static_cast<unsigned>(ceil_div(m, rpb)), gy), nullptr, nullptr, 3, rpb);
    return;
  }
  if (self) {
    fin.wide = reinterpret_cast<const double2*>(partial); fin.nwide = nrows; fin.partial = nullptr;
  } else if (reduces && bn_reduces(nrows)) {
    fin.wide = bn_reduced_rows(partial, nrows, d->C, false); fin.nwide = kBnReducedRows;
  }
  const BnGeom ga = bn_apply_geom(m, d->C, d->dtype, kBnApplyGroups);
  if constexpr (LAST) {  // (only a step shares)
    if (share && y) {
      fin.slots = share->slots; fin.groups = finalize_grid(d->C); fin.polls = share->polls; fin.nblk = ga.nblk;
      RN50_FWD_APPLY(kFinShared, dim3(fin.groups + static_cast<unsigned>(ga.nblk) * ga.gy), nullptr, nullptr, ga.tx_log2, ga.rpb);
      return;
    }
  }
  RN50_LAUNCH("bn_finalize", bn_finalize_kernel<false>, dim3(finalize_grid(d->C)), dim3(kFinThreads), 0, s, m, d->C, fin);
  if (!y) return;  // statistics only: the consumer applies the layer while it loads its operand
  RN50_FWD_APPLY(kFinGiven, dim3(ga.nblk, ga.gy), save_mean, save_rstd, ga.tx_log2, ga.rpb);
#undef RN50_FWD_APPLY
#undef RN50_FWD_APPLY_T
}

template <typename T>
static void launch_fwd(const rn50_bn_desc* d, const BnGeom& g, int64_t m, const void* x,
                       const float* gamma, const float* beta, const void* residual, void* y,
                       uint8_t* relu_mask, float* save_mean, float* save_rstd, float* rm, float* rv,
                       float momentum, float* partial, hipStream_t s) {
  const bool self = bn_self_sums(m, d->C);
  RN50_LAUNCH("bn_stats", bn_stats_kernel<T>, dim3(g.nblk, g.gy), dim3(256), 0, s, static_cast<const T*>(x), m, d->C, g.tx_log2, g.rpb, self ? 1 : 0, partial);
  launch_fwd_tail<T, false>(d, m, x, gamma, beta, residual, y, relu_mask, save_mean, save_rstd, rm, rv, momentum,
                     partial, g.nblk, g.rpb, self, false, nullptr, s);
}

// finalize + apply from partial sums rows [sum g, sum g*xhat]
template <typename T, bool LAST>
static void launch_bwd_tail(const rn50_bn_desc* d, int64_t m, const void* dz,
                            const void* dz2, const void* x, const void* z, const uint8_t* zmask,
                            const float* gamma, const float* beta, const float* mean, const float* rstd,
                            void* dx, void* dres, float* dgamma, float* dbeta, const float* partial,
                            int nrows, bool self, bool reduces, const BnShare* share, hipStream_t s) {
  BnGeom ga = bn_apply_geom(m, d->C, d->dtype, kBnBwdApplyGroups);
  const int through = writes_through(m * d->C * sizeof(T));
  BnFinArgs fin{};
  fin.partial = partial; fin.nrows = nrows; fin.mean_out = dbeta; fin.rstd_out = dgamma;
  if (!self && reduces && bn_reduces(nrows)) {
    fin.wide = bn_reduced_rows(partial, nrows, d->C, true); fin.nwide = kBnReducedRows;
  }
  dim3 grid;
  if (self) {
    // few tile rows: the apply pass adds them up itself
    ga.tx_log2 = 3;
    bn_self_finalize_geom(m, d->C, ga.V, &ga.gy, &ga.rpb);
    ga.nblk = static_cast<int>(ceil_div(m, ga.rpb));
    grid = dim3(ga.nblk, ga.gy);
  } else if (share) {
    fin.slots = share->slots; fin.groups = finalize_grid(d->C); fin.polls = share->polls; fin.nblk = ga.nblk;
    grid = dim3(fin.groups + static_cast<unsigned>(ga.nblk) * ga.gy);
  } else {
    RN50_LAUNCH("bn_bwd_finalize", bn_finalize_kernel<true>, dim3(finalize_grid(d->C)), dim3(kFinThreads), 0, s, m, d->C, fin);
    grid = dim3(ga.nblk, ga.gy);
  }
#define RN50_BWD_APPLY_T(DZ2, ZK, FIN, THROUGH)                                                                           \
  RN50_LAUNCH("bn_bwd_apply", (bn_bwd_apply_kernel<T, DZ2, ZK, FIN, LAST, THROUGH>), grid, dim3(256), 0, s,                  \
              static_cast<const T*>(dz), static_cast<const T*>(dz2), static_cast<const T*>(x),                     \
              static_cast<const T*>(z), zmask, gamma, beta, mean, rstd, dgamma, dbeta, static_cast<T*>(dx),        \
              static_cast<T*>(dres), m, d->C, ga.tx_log2, ga.rpb, d->mode, through, fin)
#define RN50_BWD_APPLY_K(DZ2, ZK, FIN)                                                    \
  do {                                                                           \
    if (through) RN50_BWD_APPLY_T(DZ2, ZK, FIN, true); else RN50_BWD_APPLY_T(DZ2, ZK, FIN, false); \
  } while (0)
#define RN50_BWD_APPLY(DZ2, ZK)                                                  \
  do {                                                                           \
    if (self) {                                                                   \
      RN50_BWD_APPLY_K(DZ2, ZK, kFinSelf);                                        \
      break;                                                                      \
    }                                                                             \
    if constexpr (LAST) {                                                         \
      if (share) {                                                                \
        RN50_BWD_APPLY_K(DZ2, ZK, kFinShared);                                    \
        break;                                                                    \
      }                                                                           \
    }                                                                             \
    RN50_BWD_APPLY_K(DZ2, ZK, kFinGiven);                                         \
  } while (0)
  const int zk = d->mode == 0 ? 0 : (zmask ? 2 : (z ? 1 : 0));
  if constexpr (!LAST) {  // (a step has one gradient, and its ReLU decisions from recorded bits or x)
    if (dz2) {
      if (zk == 2) RN50_BWD_APPLY(true, 2); else if (zk == 1) RN50_BWD_APPLY(true, 1); else RN50_BWD_APPLY(true, 0);
      return;
    }
    if (zk == 1) {
      RN50_BWD_APPLY(false, 1);
      return;
    }
  }
  if (zk == 2) RN50_BWD_APPLY(false, 2); else RN50_BWD_APPLY(false, 0);
#undef RN50_BWD_APPLY
#undef RN50_BWD_APPLY_K
#undef RN50_BWD_APPLY_T
}

template <typename T, bool LAST>
static void launch_bwd(const rn50_bn_desc* d, const BnGeom& g, int64_t m, const void* dz,
                       const void* dz2, const void* x, const void* z, const uint8_t* zmask,
                       const float* gamma, const float* beta, const float* mean, const float* rstd, void* dx,
                       void* dres, float* dgamma, float* dbeta, float* partial, hipStream_t s) {
  const bool self = bn_self_sums(m, d->C);
#define RN50_BWD_REDUCE(DZ2, ZK)                                                                                 \
  RN50_LAUNCH("bn_bwd_reduce", (bn_bwd_reduce_kernel<T, DZ2, ZK>), dim3(g.nblk, g.gy), dim3(256), 0, s,            \
              static_cast<const T*>(dz), static_cast<const T*>(dz2), static_cast<const T*>(x),                     \
              static_cast<const T*>(z), zmask, gamma, beta, mean, rstd, m, d->C, g.tx_log2, g.rpb, d->mode, partial)
  const int zk = d->mode == 0 ? 0 : (zmask ? 2 : (z ? 1 : 0));
  if (dz2) {
    if (zk == 2) RN50_BWD_REDUCE(true, 2); else if (zk == 1) RN50_BWD_REDUCE(true, 1); else RN50_BWD_REDUCE(true, 0);
  } else {
    if (zk == 2) RN50_BWD_REDUCE(false, 2); else if (zk == 1) RN50_BWD_REDUCE(false, 1); else RN50_BWD_REDUCE(false, 0);
  }
#undef RN50_BWD_REDUCE
  launch_bwd_tail<T, LAST>(d, m, dz, dz2, x, z, zmask, gamma, beta, mean, rstd, dx, dres, dgamma, dbeta, partial,
                     g.nblk, self, false, nullptr, s);
}

// Entry points for the whole-step driver (last_reader) and the fused C-ABI calls: the sums come from the output stage
// of the convolution that produced x (forward) or dz (backward).
template <typename T, bool LAST>
static void fwd_from_partials(const rn50_bn_desc* d, const void* x, const float* partial, int nrows, int rpp,
                              const float* gamma, const float* beta, const void* residual, void* y, uint8_t* relu_mask,
                              float* save_mean, float* save_rstd, float* rm, float* rv, float momentum, const BnShare* share,
                              hipStream_t s) {
  launch_fwd_tail<T, LAST>(d, static_cast<int64_t>(d->N) * d->H * d->W, x, gamma, beta, residual, y, relu_mask, save_mean,
                           save_rstd, rm, rv, momentum, partial, nrows, rpp, bn_self_finalizes(nrows, false), true, share, s);
}
void bn_fwd_from_partials(const rn50_bn_desc* d, const void* x, const float* partial, int nrows, int rpp,
                          const float* gamma, const float* beta, const void* residual, void* y,
                          uint8_t* relu_mask, float* save_mean, float* save_rstd, float* rm, float* rv,
                          float momentum, bool last_reader, hipStream_t s, const BnShare* share) {
  auto* run = d->dtype == RN50_BF16 ? (last_reader ? fwd_from_partials<uint16_t, true> : fwd_from_partials<uint16_t, false>)
                                    : (last_reader ? fwd_from_partials<float, true> : fwd_from_partials<float, false>);
  run(d, x, partial, nrows, rpp, gamma, beta, residual, y, relu_mask, save_mean, save_rstd, rm, rv, momentum, share, s);
}
// Evaluation mode: 1/sqrt(running_var + eps) per channel, then the training pass's apply kernel with the
// moving averages in place of the batch statistics.
__global__ __launch_bounds__(256) void bn_infer_rstd_kernel(const float* __restrict__ running_var, float eps, int C,
                                                            float* __restrict__ rstd) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c < C) rstd[c] = static_cast<float>(1.0 / sqrt(static_cast<double>(running_var[c]) + static_cast<double>(eps)));
}
static void infer_run(const rn50_bn_desc* d, const void* x, const float* gamma, const float* beta,
                      const float* running_mean, const float* running_var, const void* residual, void* y,
                      float* rstd_scratch, hipStream_t s) {
  const int64_t m = static_cast<int64_t>(d->N) * d->H * d->W;
  hipLaunchKernelGGL(bn_infer_rstd_kernel, dim3(static_cast<unsigned>(ceil_div(d->C, 256))), dim3(256), 0, s,
                     running_var, d->eps, d->C, rstd_scratch);
  const BnGeom ga = bn_apply_geom(m, d->C, d->dtype, kBnApplyGroups);
  if (d->dtype == RN50_BF16)
    RN50_LAUNCH("bn_apply", (bn_apply_kernel<uint16_t, kFinGiven, false, false>), dim3(ga.nblk, ga.gy), dim3(256), 0, s, static_cast<const uint16_t*>(x), gamma, beta, running_mean, rstd_scratch, static_cast<const uint16_t*>(residual), static_cast<uint16_t*>(y), static_cast<uint8_t*>(nullptr), m, d->C, ga.tx_log2, ga.rpb, d->mode, 0, BnFinArgs{});
  else
    RN50_LAUNCH("bn_apply", (bn_apply_kernel<float, kFinGiven, false, false>), dim3(ga.nblk, ga.gy), dim3(256), 0, s, static_cast<const float*>(x), gamma, beta, running_mean, rstd_scratch, static_cast<const float*>(residual), static_cast<float*>(y), static_cast<uint8_t*>(nullptr), m, d->C, ga.tx_log2, ga.rpb, d->mode, 0, BnFinArgs{});
}

template <typename T, bool LAST>
static void bwd_from_partials(const rn50_bn_desc* d, const void* dz, const void* x, const uint8_t* relu_mask,
                              const float* gamma, const float* beta, const float* mean, const float* rstd,
                              const float* partial, int nrows, void* dx, void* dres, float* dgamma, float* dbeta,
                              const BnShare* share, hipStream_t s) {
  launch_bwd_tail<T, LAST>(d, static_cast<int64_t>(d->N) * d->H * d->W, dz, nullptr, x, nullptr, relu_mask, gamma, beta, mean,
                           rstd, dx, dres, dgamma, dbeta, partial, nrows, bn_self_finalizes(nrows, true), true, LAST ? share : nullptr, s);
}
void bn_bwd_from_partials(const rn50_bn_desc* d, const void* dz, const void* x, const uint8_t* relu_mask,
                          const float* gamma, const float* beta, const float* mean, const float* rstd,
                          const float* partial, int nrows, void* dx, void* dres, float* dgamma, float* dbeta,
                          bool last_reader, hipStream_t s, const BnShare* share) {
  auto* run = d->dtype == RN50_BF16 ? (last_reader ? bwd_from_partials<uint16_t, true> : bwd_from_partials<uint16_t, false>)
                                    : (last_reader ? bwd_from_partials<float, true> : bwd_from_partials<float, false>);
  run(d, dz, x, relu_mask, gamma, beta, mean, rstd, partial, nrows, dx, dres, dgamma, dbeta, share, s);
}
void bn_bwd_run(const rn50_bn_desc* d, const void* dz, const void* dz2, const void* x, const void* z,
                const uint8_t* relu_mask, const float* gamma, const float* beta, const float* mean, const float* rstd,
                void* dx, void* dres, float* dgamma, float* dbeta, float* scratch, bool last_reader, hipStream_t s) {
  const int64_t m = static_cast<int64_t>(d->N) * d->H * d->W;
  const BnGeom g = bn_sums_geom(m, d->C, d->dtype);
  last_reader = last_reader && !dz2 && !z;  // (what is compiled: no step passes either)
  auto* run = d->dtype == RN50_BF16 ? (last_reader ? launch_bwd<uint16_t, true> : launch_bwd<uint16_t, false>)
                                    : (last_reader ? launch_bwd<float, true> : launch_bwd<float, false>);
  run(d, g, m, dz, dz2, x, z, relu_mask, gamma, beta, mean, rstd, dx, dres, dgamma, dbeta, scratch, s);
}

// ------------------------------------------------------- BN + ReLU + max-pool, forward
// The layer's output is needed by the pool alone (the backward pass works on the winners), so it is not stored: a thread makes
// kPoolRows pooled rows of one column and vector out of 2 * kPoolRows + 1 input rows, every element rounded to the storage type
// before it is compared, as if it had been stored.  bf16: a non-negative value's bits order like integers, so (bits, 15 - window
// position) in one word finds the maximum and its first position with one three-way maximum per row.
// Bound by memory (the input once, a quarter of it and the winners written): 298 -> 132 us at batch 256, 44 -> 23 us at batch 40
// against the apply pass and maxpool_fwd; the step 20.15 -> 19.93 ms.  (The same fusion backward, the gradient gathered from the
// pool's windows in the sums and in the apply pass, took 735 + 543 us instead of 226 + 202 + 252: four windows' operands per
// element cost more than the tensor.)
constexpr int kPoolRows = 2;
template <typename T>
__global__ __launch_bounds__(256) void bn_relu_maxpool_kernel(const T* __restrict__ x, const float* __restrict__ gamma,
                                                              const float* __restrict__ beta, const float* __restrict__ mean,
                                                              const float* __restrict__ rstd, T* __restrict__ y,
                                                              uint8_t* __restrict__ argmax, int H, int W, int C, int P, int Q,
                                                              FastDiv div_cv) {
  // grid: (vectors of one pooled row, groups of kPoolRows pooled rows, images)
  constexpr int V = Elem<T>::VEC;
  const int cv = C / V;
  const int xi = blockIdx.x * 256 + threadIdx.x;
  if (xi >= Q * cv) return;
  const int q = static_cast<int>(fdiv(static_cast<uint32_t>(xi), div_cv)), c0 = (xi - q * cv) * V;
  const int p0 = blockIdx.y * kPoolRows, n = blockIdx.z;
  constexpr int NR = 2 * kPoolRows + 1;
  Vec16 v[NR][3];
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    const int ih = min(max(2 * p0 - 1 + i, 0), H - 1);
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      const int iw = min(max(2 * q - 1 + s, 0), W - 1);
      v[i][s] = load16_stream(x + ((static_cast<int64_t>(n) * H + ih) * W + iw) * C + c0);
    }
  }
  float scale[V], bias[V];
  {
    float cg[V], cb[V], cm[V], cr[V];
    load_floats<V>(gamma + c0, cg);
    load_floats<V>(beta + c0, cb);
    load_floats<V>(mean + c0, cm);
    load_floats<V>(rstd + c0, cr);
#pragma unroll
    for (int j = 0; j < V; ++j) bn_coeffs(cg[j], cb[j], cm[j], cr[j], &scale[j], &bias[j]);
  }
  const bool left = 2 * q - 1 >= 0, right = 2 * q + 1 < W;
  // per input row: the largest of its three values and its position s (the first one of equals)
  float best[sizeof(T) == 4 ? NR : 1][V];
  uint32_t key[NR][V];  // bf16: bits << 16 | 3 - s; float: s
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    float f[3][V];
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      Elem<T>::unpack(v[i][s], f[s]);
#pragma unroll
      for (int j = 0; j < V; ++j) f[s][j] = fmaxf(bn_affine(f[s][j], scale[j], bias[j]), 0.f);
    }
    if constexpr (sizeof(T) == 2) {
#pragma unroll
      for (int j = 0; j < V; j += 2) {
        uint32_t lo[3], hi[3];
#pragma unroll
        for (int s = 0; s < 3; ++s) {
          const uint32_t b = float2_to_bf16x2_bits(f[s][j], f[s][j + 1]) & 0x7fff7fffu;  // (no -0)
          lo[s] = (b << 16) | (3u - s);
          hi[s] = (b & 0xffff0000u) | (3u - s);
        }
        const uint32_t l0 = left ? lo[0] : 0u, h0 = left ? hi[0] : 0u, l2 = right ? lo[2] : 0u, h2 = right ? hi[2] : 0u;
        key[i][j] = max(max(l0, lo[1]), l2);
        key[i][j + 1] = max(max(h0, hi[1]), h2);
      }
    } else {
#pragma unroll
      for (int j = 0; j < V; ++j) {
        float b = left ? f[0][j] : f[1][j];
        uint32_t at = left ? 0u : 1u;
        if (f[1][j] > b) { b = f[1][j]; at = 1; }
        if (right && f[2][j] > b) { b = f[2][j]; at = 2; }
        best[i][j] = b;
        key[i][j] = at;
      }
    }
  }
#pragma unroll
  for (int k = 0; k < kPoolRows; ++k) {
    const int p = p0 + k;
    if (p >= P) break;
    const bool top = 2 * p - 1 >= 0, bottom = 2 * p + 1 < H;  // (row 2p is in the image)
    Vec16 o;
    uint32_t at[V];
    if constexpr (sizeof(T) == 2) {
      uint32_t m[V];
#pragma unroll
      for (int j = 0; j < V; ++j) {  // 3 - s + 12 - 3 r = 15 - position
        const uint32_t a0 = top ? key[2 * k][j] + 12u : 0u, a1 = key[2 * k + 1][j] + 9u, a2 = bottom ? key[2 * k + 2][j] + 6u : 0u;
        m[j] = max(max(a0, a1), a2);
        at[j] = 15u - (m[j] & 15u);
      }
#pragma unroll
      for (int j = 0; j < V; j += 2) {
        const uint32_t w = (m[j] >> 16) | (m[j + 1] & 0xffff0000u);
        if (j == 0) o.u.x = w; else if (j == 2) o.u.y = w; else if (j == 4) o.u.z = w; else o.u.w = w;
      }
    } else {
#pragma unroll
      for (int j = 0; j < V; ++j) {
        float b = top ? best[2 * k][j] : best[2 * k + 1][j];
        at[j] = top ? key[2 * k][j] : 3u + key[2 * k + 1][j];
        if (best[2 * k + 1][j] > b) { b = best[2 * k + 1][j]; at[j] = 3u + key[2 * k + 1][j]; }
        if (bottom && best[2 * k + 2][j] > b) { b = best[2 * k + 2][j]; at[j] = 6u + key[2 * k + 2][j]; }
        o.f[j & 3] = b;
      }
    }
    const int64_t i = ((static_cast<int64_t>(n) * P + p) * Q + q) * C + c0;
    store16(y + i, o);
    const uint32_t w0 = at[0] | at[1] << 8 | at[2] << 16 | at[3] << 24;
    if constexpr (V == 8) *reinterpret_cast<uint2*>(argmax + i) = make_uint2(w0, at[4] | at[5] << 8 | at[6] << 16 | at[7] << 24);
    else *reinterpret_cast<uint32_t*>(argmax + i) = w0;
  }
}
void bn_relu_maxpool(const rn50_bn_desc* d, const void* x, const float* gamma, const float* beta, const float* mean,
                     const float* rstd, void* pooled, uint8_t* argmax, hipStream_t s) {
  const int P = (d->H - 1) / 2 + 1, Q = (d->W - 1) / 2 + 1, cv = d->C / (d->dtype == RN50_BF16 ? 8 : 4);
  const dim3 grid(static_cast<unsigned>(ceil_div(static_cast<int64_t>(Q) * cv, 256)), static_cast<unsigned>(ceil_div(P, kPoolRows)), d->N);
  if (d->dtype == RN50_BF16)
    RN50_LAUNCH("bn_apply", bn_relu_maxpool_kernel<uint16_t>, grid, dim3(256), 0, s, static_cast<const uint16_t*>(x), gamma, beta, mean, rstd, static_cast<uint16_t*>(pooled), argmax, d->H, d->W, d->C, P, Q, make_fastdiv(cv));
  else
    RN50_LAUNCH("bn_apply", bn_relu_maxpool_kernel<float>, grid, dim3(256), 0, s, static_cast<const float*>(x), gamma, beta, mean, rstd, static_cast<float*>(pooled), argmax, d->H, d->W, d->C, P, Q, make_fastdiv(cv));
}

}  // namespace rn50

using namespace rn50;

extern "C" size_t bn_relu_fwd_workspace_bytes(const rn50_bn_desc* d) {
  if (!d || d->N <= 0 || d->H <= 0 || d->W <= 0 || d->C <= 0) return 0;
  return bn_ws_bytes(d);
}
extern "C" size_t bn_relu_bwd_workspace_bytes(const rn50_bn_desc* d) {
  return bn_relu_fwd_workspace_bytes(d);
}

extern "C" int bn_relu_fwd(const rn50_bn_desc* d, const void* x, const float* gamma,
                           const float* beta, const void* residual, void* y, uint8_t* relu_mask,
                           float* save_mean, float* save_rstd, float* running_mean, float* running_var,
                           float momentum, void* workspace, size_t workspace_bytes, void* stream) {
  clear_error();
  if (int rc = check_desc(d, "bn_relu_fwd")) return rc;
  RN50_REQUIRE(x && gamma && beta && y && save_mean && save_rstd && workspace, RN50_ERR_INVALID,
               "bn_relu_fwd: null pointer");
  RN50_REQUIRE((d->mode == 2) == (residual != nullptr), RN50_ERR_INVALID,
               "bn_relu_fwd: residual must be given exactly in mode 2");
  RN50_REQUIRE(aligned16(x) && aligned16(y) && aligned16(residual) && aligned16(workspace) &&
                   aligned16(gamma) && aligned16(beta) && aligned16(save_mean) && aligned16(save_rstd),
               RN50_ERR_ALIGN, "bn_relu_fwd: pointer not 16-byte aligned");
  RN50_REQUIRE(workspace_bytes >= bn_ws_bytes(d), RN50_ERR_WORKSPACE,
               "bn_relu_fwd: workspace %zu < %zu bytes", workspace_bytes, bn_ws_bytes(d));
  const int64_t m = static_cast<int64_t>(d->N) * d->H * d->W;
  const BnGeom g = bn_sums_geom(m, d->C, d->dtype);
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (d->dtype == RN50_BF16)
    launch_fwd<uint16_t>(d, g, m, x, gamma, beta, residual, y, relu_mask, save_mean, save_rstd, running_mean,
                         running_var, momentum, static_cast<float*>(workspace), s);
  else
    launch_fwd<float>(d, g, m, x, gamma, beta, residual, y, relu_mask, save_mean, save_rstd, running_mean,
                      running_var, momentum, static_cast<float*>(workspace), s);
  return launch_status("bn_relu_fwd");
}

extern "C" int bn_relu_bwd(const rn50_bn_desc* d, const void* dz, const void* dz2, const void* x,
                           const void* z, const uint8_t* relu_mask, const float* gamma, const float* beta,
                           const float* save_mean, const float* save_rstd, void* dx,
                           void* dresidual, float* dgamma, float* dbeta, void* workspace,
                           size_t workspace_bytes, void* stream) {
  clear_error();
  if (int rc = check_desc(d, "bn_relu_bwd")) return rc;
  RN50_REQUIRE(dz && x && gamma && save_mean && save_rstd && dx && dgamma && dbeta && workspace,
               RN50_ERR_INVALID, "bn_relu_bwd: null pointer");
  RN50_REQUIRE(d->mode != 2 || z || relu_mask, RN50_ERR_INVALID, "bn_relu_bwd: mode 2 needs z or relu_mask");
  RN50_REQUIRE(d->mode != 1 || z || relu_mask || beta, RN50_ERR_INVALID,
               "bn_relu_bwd: mode 1 needs z, relu_mask, or beta to recompute the ReLU mask");
  RN50_REQUIRE(aligned16(dz) && aligned16(dz2) && aligned16(x) && aligned16(z) && aligned16(dx) &&
                   aligned16(dresidual) && aligned16(workspace) && aligned16(gamma) && aligned16(beta) &&
                   aligned16(save_mean) && aligned16(save_rstd) && aligned16(dgamma) && aligned16(dbeta),
               RN50_ERR_ALIGN, "bn_relu_bwd: pointer not 16-byte aligned");
  RN50_REQUIRE(workspace_bytes >= bn_ws_bytes(d), RN50_ERR_WORKSPACE,
               "bn_relu_bwd: workspace %zu < %zu bytes", workspace_bytes, bn_ws_bytes(d));
  bn_bwd_run(d, dz, dz2, x, z, relu_mask, gamma, beta, save_mean, save_rstd, dx, dresidual, dgamma, dbeta,
             static_cast<float*>(workspace), false, static_cast<hipStream_t>(stream));
  return launch_status("bn_relu_bwd");
}

// ---- batch norm from sums fused into the producing convolution (conv_fwd_bn_sums / conv_dgrad_bn_sums)
extern "C" int bn_relu_fwd_from_sums(const rn50_bn_desc* d, const rn50_conv_desc* producer, const void* x,
                                     const float* sums, const float* gamma, const float* beta,
                                     const void* residual, void* y, uint8_t* relu_mask, float* save_mean,
                                     float* save_rstd, float* running_mean, float* running_var, float momentum,
                                     void* stream) {
  clear_error();
  if (int rc = check_desc(d, "bn_relu_fwd_from_sums")) return rc;
  RN50_REQUIRE(producer && conv_bn_sums_bytes(producer) > 0, RN50_ERR_INVALID,
               "bn_relu_fwd_from_sums: bad producer descriptor");
  RN50_REQUIRE(x && sums && gamma && beta && y && save_mean && save_rstd, RN50_ERR_INVALID,
               "bn_relu_fwd_from_sums: null pointer");
  RN50_REQUIRE((d->mode == 2) == (residual != nullptr), RN50_ERR_INVALID,
               "bn_relu_fwd_from_sums: residual must be given exactly in mode 2");
  RN50_REQUIRE(aligned16(x) && aligned16(y) && aligned16(residual) && aligned16(sums) && aligned16(gamma) &&
                   aligned16(beta) && aligned16(save_mean) && aligned16(save_rstd),
               RN50_ERR_ALIGN, "bn_relu_fwd_from_sums: pointer not 16-byte aligned");
  const int P = (producer->H + 2 * producer->pad - producer->R) / producer->stride + 1;
  const int Q = (producer->W + 2 * producer->pad - producer->S) / producer->stride + 1;
  RN50_REQUIRE(producer->N == d->N && P == d->H && Q == d->W && producer->Cout == d->C &&
                   producer->dtype == d->dtype,
               RN50_ERR_INVALID, "bn_relu_fwd_from_sums: the producer's output is not this layer's input");
  const PartialRows pr = fwd_partial_rows(producer);
  bn_fwd_from_partials(d, x, sums, pr.num, pr.rows, gamma, beta, residual, y, relu_mask, save_mean, save_rstd,
                       running_mean, running_var, momentum, false, static_cast<hipStream_t>(stream));
  return launch_status("bn_relu_fwd_from_sums");
}

extern "C" int bn_relu_bwd_from_sums(const rn50_bn_desc* d, const rn50_conv_desc* producer, const void* dz,
                                     const void* x, const uint8_t* relu_mask, const float* gamma,
                                     const float* beta, const float* save_mean, const float* save_rstd,
                                     const float* sums, void* dx, void* dresidual, float* dgamma, float* dbeta,
                                     void* stream) {
  clear_error();
  if (int rc = check_desc(d, "bn_relu_bwd_from_sums")) return rc;
  RN50_REQUIRE(d->mode == 1 || d->mode == 2, RN50_ERR_UNSUPPORTED, "bn_relu_bwd_from_sums: mode %d (needs a ReLU)",
               d->mode);
  RN50_REQUIRE(d->mode != 2 || relu_mask, RN50_ERR_INVALID, "bn_relu_bwd_from_sums: mode 2 needs relu_mask");
  RN50_REQUIRE(producer && conv_bn_sums_bytes(producer) > 0, RN50_ERR_INVALID,
               "bn_relu_bwd_from_sums: bad producer descriptor");
  RN50_REQUIRE(dz && x && gamma && beta && save_mean && save_rstd && sums && dx && dgamma && dbeta,
               RN50_ERR_INVALID, "bn_relu_bwd_from_sums: null pointer");
  RN50_REQUIRE(aligned16(dz) && aligned16(x) && aligned16(dx) && aligned16(sums) && aligned16(dresidual) &&
                   aligned16(gamma) && aligned16(beta) && aligned16(save_mean) && aligned16(save_rstd) &&
                   aligned16(dgamma) && aligned16(dbeta),
               RN50_ERR_ALIGN, "bn_relu_bwd_from_sums: pointer not 16-byte aligned");
  RN50_REQUIRE(producer->N == d->N && producer->H == d->H && producer->W == d->W && producer->Cin == d->C &&
                   producer->dtype == d->dtype,
               RN50_ERR_INVALID, "bn_relu_bwd_from_sums: the producer's input is not this layer's output");
  const PartialRows pr = dgrad_partial_rows(producer);
  bn_bwd_from_partials(d, dz, x, relu_mask, gamma, beta, save_mean, save_rstd, sums, pr.num, dx,
                       d->mode == 2 ? dresidual : nullptr, dgamma, dbeta, false, static_cast<hipStream_t>(stream));
  return launch_status("bn_relu_bwd_from_sums");
}

extern "C" size_t bn_relu_infer_workspace_bytes(const rn50_bn_desc* d) {
  if (!d || d->C <= 0) return 0;
  return align_up(static_cast<size_t>(d->C) * sizeof(float), 256);
}

extern "C" int bn_relu_infer(const rn50_bn_desc* d, const void* x, const float* gamma, const float* beta,
                             const float* running_mean, const float* running_var, const void* residual, void* y,
                             void* workspace, size_t workspace_bytes, void* stream) {
  clear_error();
  if (int rc = check_desc(d, "bn_relu_infer")) return rc;
  RN50_REQUIRE(x && gamma && beta && running_mean && running_var && y && workspace, RN50_ERR_INVALID,
               "bn_relu_infer: null pointer");
  RN50_REQUIRE((d->mode == 2) == (residual != nullptr), RN50_ERR_INVALID,
               "bn_relu_infer: residual must be given exactly in mode 2");
  RN50_REQUIRE(aligned16(x) && aligned16(y) && aligned16(residual) && aligned16(workspace) && aligned16(gamma) &&
                   aligned16(beta) && aligned16(running_mean) && aligned16(running_var),
               RN50_ERR_ALIGN, "bn_relu_infer: pointer not 16-byte aligned");
  RN50_REQUIRE(workspace_bytes >= bn_relu_infer_workspace_bytes(d), RN50_ERR_WORKSPACE,
               "bn_relu_infer: workspace %zu < %zu bytes", workspace_bytes, bn_relu_infer_workspace_bytes(d));
  infer_run(d, x, gamma, beta, running_mean, running_var, residual, y, static_cast<float*>(workspace),
            static_cast<hipStream_t>(stream));
  return launch_status("bn_relu_infer");
}
