// Shared by the convolution files: buffer descriptors and loads, the workgroup renumbering, the input-side batch norm,
// the geometry of the padded stem.
#pragma once
#include "common.h"
#include "step_internal.h"

namespace rn50 {

// Workgroups are dealt to the 8 XCDs round-robin; renumber them so that consecutive logical ids
// (which share rows of the activation tile) run on the same XCD and meet in its L2.
__device__ __forceinline__ int xcd_remap(int id, int n) {
  const int xcd = id & 7, idx = id >> 3;
  const int q = n >> 3, rem = n & 7;
  return xcd < rem ? xcd * (q + 1) + idx : rem * (q + 1) + (xcd - rem) * q + idx;
}

// relu(bn(x)) of one 16-byte vector with the arithmetic of the stand-alone BN pass (bn_affine, one rounding to
// the storage type), so that a convolution reading it sees bit for bit the tensor that pass would have stored.
template <typename T>
__device__ __forceinline__ Vec16 bn_relu_vector(const Vec16& v, const float* scale, const float* bias) {
  constexpr int V = 16 / sizeof(T);
  float f[V];
  Elem<T>::unpack(v, f);
#pragma unroll
  for (int j = 0; j < V; ++j) f[j] = fmaxf(bn_affine(f[j], scale[j], bias[j]), 0.f);
  Vec16 o;
  Elem<T>::pack(f, o);
  return o;
}
// The vector with zeros (+0) where an element's bit is not set.  In bf16 by pairs, two 16-bit shifts for two elements' masks: a test and a
// selection per element are twice the instructions.
template <typename T>
__device__ __forceinline__ Vec16 keep_bits(const Vec16& v, uint32_t bits) {
  Vec16 o;
  if constexpr (sizeof(T) == 2) {
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    typedef short s16x2 __attribute__((ext_vector_type(2)));
    const u16x2 both = __builtin_bit_cast(u16x2, bits | bits << 16);
    auto mask = [&](int i) __attribute__((always_inline)) {  // of elements 2i and 2i + 1: bit to sign, sign to all
      const u16x2 up = both << u16x2{static_cast<unsigned short>(15 - 2 * i), static_cast<unsigned short>(14 - 2 * i)};
      return __builtin_bit_cast(uint32_t, __builtin_bit_cast(s16x2, up) >> s16x2{15, 15});
    };
    o.u = make_uint4(v.u.x & mask(0), v.u.y & mask(1), v.u.z & mask(2), v.u.w & mask(3));
  } else {
    auto mask = [&](int j) __attribute__((always_inline)) { return static_cast<uint32_t>(static_cast<int>(bits << (31 - j)) >> 31); };
    o.u = make_uint4(v.u.x & mask(0), v.u.y & mask(1), v.u.z & mask(2), v.u.w & mask(3));
  }
  return o;
}
constexpr uint32_t kOob = 0x80000000u;  // buffer offset beyond every tensor: the load returns zeros

// Barrier behind LDS writes of this wave (s_barrier alone does not wait for them), leaving vector-memory loads in flight.
__device__ __forceinline__ void lds_writes_then_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0); vmcnt, expcnt: no wait
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
// Barrier behind LDS reads of this wave, whose buffers loads overwrite right behind it: the same waits.
__device__ __forceinline__ void lds_reads_then_barrier() { lds_writes_then_barrier(); }

// A 16-byte buffer load with LDS as its destination (buffer_load_dwordx4 ... lds): lane l of the wave writes its 16
// bytes to LDS address lds_addr + 16*l (lds_addr uniform, taken from M0), so one instruction fills 1 KB; lanes
// whose offset is out of range write zeros.  Nothing passes through registers; the transfer is counted by
// vmcnt like any other vector-memory load.  Written as assembly on purpose: the compiler would make every
// later LDS read wait for ALL outstanding loads of this kind (it cannot tell the ring buffers apart), which
// is the prefetch distance this kernel lives on; the waits are placed by hand (wait_loads_then_barrier).
typedef int rsrc_words __attribute__((ext_vector_type(4)));
__device__ __forceinline__ rsrc_words make_rsrc_words(const void* p, uint32_t bytes) {
  const uint64_t addr = reinterpret_cast<uint64_t>(p);
  rsrc_words r;
  r.x = static_cast<int>(addr);
  r.y = static_cast<int>((addr >> 32) & 0xffffu);  // stride 0: a raw buffer
  r.z = static_cast<int>(bytes);
  r.w = 0x00020000;
  return r;
}
__device__ __forceinline__ void buffer_load16_to_lds(rsrc_words r, uint32_t lds_addr, uint32_t voffset, uint32_t soffset) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               :
               : "s"(lds_addr), "v"(voffset), "s"(r), "s"(soffset)
               : "memory");  // (m0 is reserved: the compiler keeps nothing in it across statements)
}
// Wait until at most N of this wave's vector-memory loads are outstanding, then the workgroup barrier, without
// the full memory fence of __syncthreads() (which would also wait for the loads of the chunks still in flight).
template <int N, bool BARRIER = true>
__device__ __forceinline__ void wait_loads_then_barrier() {
  static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
  // s_waitcnt immediate on gfx9: vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt[5:4] << 14; 7 / 15 = no wait
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
  if (BARRIER) __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Top of iteration kc of a ring of NSTAGE chunk buffers (loads NSTAGE-1 chunks ahead, NL load instructions per
// thread and chunk): wait until this wave's loads of chunk kc have landed -- those of the chunks behind it that
// have been issued, at most NSTAGE-2 of them and none past the last chunk, may stay in flight -- then the barrier.
// (BARRIER = false: a ring that only this wave fills and reads.)
template <int NSTAGE, int NL, bool BARRIER = true>
__device__ __forceinline__ void ring_wait(int chunks_after) {
  static_assert(NSTAGE >= 2 && NSTAGE <= 5 && NL * (NSTAGE - 2) < 64, "ring depth");
  const int ahead = chunks_after < NSTAGE - 2 ? chunks_after : NSTAGE - 2;
  if (NSTAGE >= 5 && ahead == 3) wait_loads_then_barrier<(NSTAGE >= 5 ? 3 : 0) * NL, BARRIER>();
  else if (NSTAGE >= 4 && ahead == 2) wait_loads_then_barrier<(NSTAGE >= 4 ? 2 : 0) * NL, BARRIER>();
  else if (NSTAGE >= 3 && ahead == 1) wait_loads_then_barrier<(NSTAGE >= 3 ? 1 : 0) * NL, BARRIER>();
  else wait_loads_then_barrier<0, BARRIER>();
}

// LDS tiles of the weight gradient are [k row][column] with rows of RBY = 16 * (columns per 16 bytes ...) bytes,
// filled by LDS-destination loads (RBY/16 lanes per row).  The 16-byte slots of a row are stored permuted,
// slot s of row r at s ^ wgrad_swz(r), so that the fragment reads below touch every bank once:
//   bf16, 128-byte rows: a transposing read's 32 lanes take 64 bytes of 4 consecutive rows -- rows two apart
//                        share their banks, so they swap halves;
//   bf16, 256-byte rows: the same 4 rows all start at bank 0 -- each is rotated by a different 64 bytes;
//   float:               lanes 32-63 read the row 4 below lanes 0-31 -- it is shifted by 128 bytes.
template <typename T, int RBY>
__device__ __forceinline__ int wgrad_swz(int row) {
  if (RBY == 64 || (sizeof(T) == 4 && RBY == 128)) return 0;  // rows too short to permute
  if (sizeof(T) == 4) return ((row >> 2) & 1) << 3;
  return RBY == 128 ? ((row >> 1) & 1) << 2 : (row & 3) << 2;
}
// Byte offset, inside a tile, of this lane's first read for the MFMA operand "32 columns from col0 x one k step"
// at k step 0; step kk is KSTEP * kk rows further down.
template <typename T, int RBY>
__device__ __forceinline__ int wgrad_frag_base(int lane, int col0) {
  if (sizeof(T) == 2) {
    // ds_read_b64_tr_b16: within 16 lanes, lane t supplies the address of row t/4, columns 4*(t%4)..+3 and
    // receives column t of rows 0..3.  Two reads (rows +0 and +4) give 8 k values of column lane%32.
    const int g = lane >> 4, t = lane & 15;
    const int krow = 8 * (g >> 1) + (t >> 2);
    const int cb = 2 * (col0 + 16 * (g & 1) + 4 * (t & 3));
    return krow * RBY + (((cb >> 4) ^ wgrad_swz<T, RBY>(krow)) << 4) + (cb & 15);
  }
  const int krow = (lane >> 5) * 4;  // + j, j = 0..3: the permutation only looks at bit 2
  const int cb = 4 * (col0 + (lane & 31));
  return krow * RBY + (((cb >> 4) ^ wgrad_swz<T, RBY>(krow)) << 4) + (cb & 15);
}
template <typename T, int RBY>
__device__ __forceinline__ Vec16 wgrad_read_frag(const unsigned char* tile, int base, int kk) {
  Vec16 v;
  if constexpr (sizeof(T) == 2) {
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef s16x4 __attribute__((address_space(3))) * lds_ptr;
    const unsigned char* p0 = tile + base + kk * 16 * RBY;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p0));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p0 + 4 * RBY));
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v.h[j] = static_cast<uint16_t>(lo[j]);
      v.h[4 + j] = static_cast<uint16_t>(hi[j]);
    }
  } else {
    const unsigned char* p = tile + base + kk * 8 * RBY;
#pragma unroll
    for (int j = 0; j < 4; ++j) v.f[j] = *reinterpret_cast<const float*>(p + j * RBY);
  }
  return v;
}

template <typename K>
inline void allow_big_lds(K kernel, int bytes) {
  if (bytes > 48 * 1024) (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

inline int out_dim(int in, int pad, int k, int stride) { return (in + 2 * pad - k) / stride + 1; }
inline bool is_stem(const rn50_conv_desc* d) {
  return d->Cin == 3 && d->R == 7 && d->S == 7 && d->stride == 2 && d->pad == 3;
}
inline int esize(int dtype) { return dtype == RN50_BF16 ? 2 : 4; }

constexpr int kStemK = 256;  // padded reduction length of the stem: 8 filter rows x 8 taps x 4 channels
// Geometry of the padded stem: 7 "taps" (filter rows) of 32 elements on pixels of 4 channels.
struct StemGeom {
  int Hp, Wp;
  size_t xp_bytes, wp_bytes;
};
inline StemGeom stem_geom(const rn50_conv_desc* d) {
  StemGeom g;
  g.Hp = d->H + 6;
  g.Wp = (d->W + 6 + 2 + 3) / 4 * 4;  // room for the 8th (zero-weight) tap, row pitch a multiple of 16 bytes
  g.xp_bytes = align_up(static_cast<size_t>(d->N) * g.Hp * g.Wp * 4 * esize(d->dtype), 256);
  g.wp_bytes = align_up(static_cast<size_t>(d->Cout) * kStemK * esize(d->dtype), 256);
  return g;
}

// stem.hip: the bf16 stem from the padded image (false: a shape it does not take; the general kernel's turn), and the rows
// of batch-norm sums it leaves (num = 0: likewise).
bool stem_fwd_run(const rn50_conv_desc* d, const void* xp, const void* w, void* y, float* bn_partial, hipStream_t s,
                  const BnAffine* affine);
PartialRows stem_partial_rows(const rn50_conv_desc* d);

}  // namespace rn50
