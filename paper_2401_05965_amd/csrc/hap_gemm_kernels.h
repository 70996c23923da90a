/*
 * Device code of the tiled GEMM kernels and the host templates that launch them, shared by the translation units that
 * instantiate them (hap_gemm.hip, hap_gemm_pp.hip, hap_gemm_dma.hip); see hap_gemm.hip for the overview.
 */
#ifndef HAP_GEMM_KERNELS_H
#define HAP_GEMM_KERNELS_H

#include <hip/hip_runtime.h>

#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <type_traits>

#include "hap_gemm.h"

namespace hap_gemm_detail {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef int i32x4_t __attribute__((ext_vector_type(4)));

#define LDS_PTR(T, p) ((__attribute__((address_space(3))) T*)(p))

#if defined(HAP_GEMM_EXPERIMENT)
// (development harness only) wall-clock stamps of every workgroup: 0 start, 1 main loop start, 2 main loop end, 3 end, 4..7 after each
// 32-row block of the epilogue
__device__ unsigned long long hap_exp_stamps[8 * 2048];
#define HAP_EXP_STAMP(i) do { if (threadIdx.x == 0 && blockIdx.x < 2048) hap_exp_stamps[blockIdx.x * 8 + (i)] = __builtin_amdgcn_s_memrealtime(); } while (0)
#else
#define HAP_EXP_STAMP(i) do { } while (0)
#endif


constexpr unsigned kOobOffset = 0x80000000u;  // beyond any num_records we pass: reads as zero
constexpr int64_t kViewLimitBytes = 2147483000;  // reach of the tiled kernels' 32-bit buffer offsets: operand views stay below it
constexpr int kRsrcFlags = 0x00020000;        // raw buffer, 32-bit data format

struct SegArg {
  const void* a;   // aligned-down base of this segment's A view
  const void* b;
  int k;           // logical contracted length of the segment
  unsigned a_bytes, b_bytes;  // valid extent from the aligned bases
  int pad;
};

struct GemmArgs {
  int M, N;            // logical extent of C
  int skewM, skewN;    // physical columns preceding logical 0 in an M-/N-contiguous operand; for a K-contiguous B, skewN rows of the
                       // tile grid precede its first row (the grid then sits on C's 16-byte chunks)
  int skewK;           // physical k preceding logical 0 in a K-contiguous operand
  int nseg;
  int tiles_m, tiles_n;
  int vec_store;       // C (and preact) rows are 16-byte addressable: whole-chunk stores allowed
  int cdelta;          // columns by which tile columns are shifted in the store patch so that its 16-byte chunks coincide with
                       // 16-byte chunks of C's address space (0 when C has the B operand's phase; see epilogue_transposed)
  int kpair;           // 1: gemm_kpair_kernel
  int ksplit;          // >1: each output tile is computed by ksplit workgroups over disjoint K-tile ranges, fp32 partials go to `partial`
  float* partial;      // [group][tile][ksplit][BM][BN] fp32 workspace when ksplit > 1
  int ntiles;          // K tiles (of 64) over all segments
  long long lda, ldb, ldc, ldp;
  void* c;
  void* preact;
  const void* bias;
  int act, accumulate;
  const void* dact_preact;   // optional [M x N] in C's dtype, leading dimension ldd: C = (product + bias) * act'(dact_preact)
  long long ldd;
  // Grouped launch (gridDim.y groups): a workgroup works on one of `groups` independent products that differ only in their base
  // addresses (byte strides below) and, when group_len is given, in the valid length of one axis.
  int ragged;              // 0: every group is M x N x k;  1: group_len bounds M;  2: group_len bounds the contraction (nseg == 1)
  const int* group_len;    // device array [groups], or nullptr
  long long ga, gb, gc, gp, gbias, gd;
  SegArg seg[HAP_GEMM_MAX_SEG];
};

/* What the workgroup's group changes: valid rows, contracted length of the single segment (-1: as in
 * the segment table), byte offsets of the operands and outputs. */
struct GroupView {
  int M, k;
  long long oa, ob;
};

__device__ __forceinline__ GroupView group_view(const GemmArgs& args, int grp) {
  GroupView g;
  g.M = args.M; g.k = -1;
  g.oa = grp * args.ga; g.ob = grp * args.gb;
  if (args.ragged) {
    int len = __builtin_amdgcn_readfirstlane(args.group_len[grp]);
    len = len < 0 ? 0 : len;
    if (args.ragged == 1) g.M = len < args.M ? len : args.M;
    else g.k = len < args.seg[0].k ? len : args.seg[0].k;
  }
  return g;
}

/* The arguments as the epilogue of this workgroup's group sees them. */
__device__ __forceinline__ GemmArgs group_outputs(const GemmArgs& args, const GroupView& g, int grp) {
  GemmArgs e = args;
  e.M = g.M;
  e.c = static_cast<char*>(args.c) + grp * args.gc;
  if (args.preact) e.preact = static_cast<char*>(args.preact) + grp * args.gp;
  if (args.bias) e.bias = static_cast<const char*>(args.bias) + grp * args.gbias;
  if (args.dact_preact) e.dact_preact = static_cast<const char*>(args.dact_preact) + grp * args.gd;
  return e;
}

/* Compile-time loop: f(std::integral_constant<int, 0>) ... f(std::integral_constant<int, N-1>). */
template <int N, int I = 0, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>());
    static_for<N, I + 1>(f);
  }
}

/* Values that are the same in every lane but that the compiler cannot prove uniform (they depend on
 * a table entry picked by a loop-carried index) are pinned to scalar registers; otherwise every
 * buffer instruction using them is wrapped in a per-lane "waterfall" loop. */
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ const void* uni(const void* p) {
  const unsigned long long v = reinterpret_cast<unsigned long long>(p);
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v), hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
  return reinterpret_cast<const void*>(((unsigned long long)hi << 32) | lo);
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(uni(base)), 0, uni((int)bytes), kRsrcFlags);
}

/* One wave-wide direct load: lane l's 16 bytes at (voff + soff) of the buffer land at lds + 16*l.
 * `lds` must be wave-uniform.  The host pass of hipcc has no such builtin, hence the guard. */
__device__ __forceinline__ void dma16(__amdgpu_buffer_rsrc_t rsrc, char* lds, unsigned voff, unsigned soff) {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, LDS_PTR(void, lds), 16, voff, soff, 0, 0);
#else
  (void)rsrc; (void)lds; (void)voff; (void)soff;
#endif
}

/* erf by the rational-times-Gaussian form of Abramowitz & Stegun 7.1.26 (absolute error <= 1.5e-7, far
 * inside the fp32 and bf16 output tolerances): one reciprocal, one exponential and five multiply-adds
 * instead of the branchy library routine, because the epilogue evaluates it for every output element. */
__device__ __forceinline__ float erf_fast(float x) {
  const float ax = fabsf(x);
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, ax, 1.0f));
  float p = fmaf(1.061405429f, t, -1.453152027f);
  p = fmaf(p, t, 1.421413741f);
  p = fmaf(p, t, -0.284496736f);
  p = fmaf(p, t, 0.254829592f);
  const float e = __builtin_amdgcn_exp2f(ax * ax * -1.4426950408889634f);
  return copysignf(1.0f - p * t * e, x);
}
__device__ __forceinline__ float gelu_erf(float x) { return 0.5f * x * (1.0f + erf_fast(x * 0.70710678118654752f)); }
/* d gelu / dx = Phi(x) + x phi(x); exp(-x^2/2) serves both the erf approximation (its argument is x/sqrt 2) and phi */
__device__ __forceinline__ float gelu_erf_grad(float x) {
  const float ax = fabsf(x) * 0.70710678118654752f;
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, ax, 1.0f));
  float p = fmaf(1.061405429f, t, -1.453152027f);
  p = fmaf(p, t, 1.421413741f);
  p = fmaf(p, t, -0.284496736f);
  p = fmaf(p, t, 0.254829592f);
  const float e = __builtin_amdgcn_exp2f(x * x * -0.7213475204444817f);
  const float half_erf = copysignf(fmaf(p * t, -0.5f * e, 0.5f), x);      // erf(x / sqrt 2) / 2
  return fmaf(x, 0.3989422804014327f * e, 0.5f + half_erf);
}

template <typename T> struct Elem;
template <> struct Elem<__bf16> {
  static constexpr int kStep = 16;  // k per MFMA (v_mfma_f32_32x32x16_bf16)
};
template <> struct Elem<float> {
  static constexpr int kStep = 2;   // v_mfma_f32_32x32x2_f32
};

/* Swizzled position of 16-byte chunk c in LDS row `row`.  The LDS of gfx950 serves 256 bytes per clock
 * (64 banks x 4 bytes): a 128-bit read is conflict free when every 16 consecutive lanes cover 16
 * different chunk positions modulo 256 bytes, a transposing 64-bit read when every 32 lanes do.
 *   K-contiguous tile: 16 lanes read the same logical chunk of 16 consecutive rows -> XOR the chunk
 *     index with the row's index inside its 256-byte group.
 *   M/N-contiguous tile (rows are 256 bytes or more): 32 lanes read 64 contiguous bytes of each of 4
 *     consecutive rows -> XOR bits 2..3 of the chunk index with row & 3.  Rows of 128 bytes (the 64-wide tiles of
 *     gemm_small_kernel) have eight chunks and lie two to a sweep: XOR bits 1..2, with which the four rows fill it as well. */
template <bool KC, int CPR>
__device__ __forceinline__ int swz(int row, int c) {
  if constexpr (KC) {
    constexpr int RPS = CPR >= 16 ? 1 : 16 / CPR;    // rows per 256-byte bank sweep
    constexpr int MASK = (CPR >= 16 ? 16 : CPR) - 1;
    return c ^ ((row / RPS) & MASK);
  } else {
    static_assert(CPR >= 8, "M/N-contiguous tiles need rows of at least 128 bytes");
    if constexpr (CPR >= 16) return c ^ ((row & 3) << 2);
    else return c ^ ((row & 3) << 1);
  }
}

template <typename T> __device__ __forceinline__ void store_c(T* p, float v);
template <> __device__ __forceinline__ void store_c<float>(float* p, float v) { *p = v; }
template <> __device__ __forceinline__ void store_c<__bf16>(__bf16* p, float v) { *p = (__bf16)v; }
template <typename T> __device__ __forceinline__ float load_s(const T* p);
template <> __device__ __forceinline__ float load_s<float>(const float* p) { return *p; }
template <> __device__ __forceinline__ float load_s<__bf16>(const __bf16* p) { return (float)*p; }

/* Loads one operand tile's chunks owned by this thread into registers.
 * KC:  rows = ROWS (m or n), chunk c covers k in [c*EPC, (c+1)*EPC)
 * !KC: rows = BK (k), chunk c covers m (or n) in [c*EPC, ...)                                   */
template <typename T, bool KC, int ROWS, int BK, int NT>
struct TileLoader {
  static constexpr int ES = sizeof(T);
  static constexpr int EPC = 16 / ES;
  static constexpr int LROWS = KC ? ROWS : BK;
  static constexpr int CPR = (KC ? BK : ROWS) / EPC;
  static constexpr int CPT = LROWS * CPR / NT;
  static_assert(LROWS * CPR % NT == 0, "tile chunks must divide evenly over threads");

  i32x4_t regs[CPT];

  /* mn0: first physical row (KC) or column (!KC) of the tile in the MN direction.
   * mn_lim: physical MN extent.  k0: first physical k of the tile; kskew/kend: logical k range in
   * physical coordinates [kskew, kend).  ld in elements.                                        */
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rsrc, int tid, int mn0, int mn_lim, long long ld,
                                       int k0, int kskew, int kend) {
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      const int id = tid + i * NT;
      const int row = id / CPR, c = id % CPR;
      unsigned off;
      if constexpr (KC) {
        const int mn = mn0 + row, kp = k0 + c * EPC;
        const bool ok = mn < mn_lim && kp < kend && kp + EPC > kskew;
        off = ok ? (unsigned)(((long long)mn * ld + kp) * ES) : kOobOffset;
      } else {
        const int kl = k0 + row, mn = mn0 + c * EPC;
        const bool ok = kl >= kskew && kl < kend && mn < mn_lim;
        off = ok ? (unsigned)(((long long)(kl - kskew) * ld + mn) * ES) : kOobOffset;
      }
      regs[i] = __builtin_bit_cast(i32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rsrc, off, 0, 0));
    }
  }

  /* Zeroes elements outside [kskew, kend) of K-contiguous chunks (needed on a segment's first and
   * last tile only; callers skip it elsewhere). */
  __device__ __forceinline__ void mask_k(int tid, int k0, int kskew, int kend) {
    if constexpr (KC) {
#pragma unroll
      for (int i = 0; i < CPT; ++i) {
        const int id = tid + i * NT;
        const int c = id % CPR;
        const int kp = k0 + c * EPC;
        if (kp < kskew || kp + EPC > kend) {
          T v[EPC];
          __builtin_memcpy(v, &regs[i], 16);
#pragma unroll
          for (int e = 0; e < EPC; ++e)
            if (kp + e < kskew || kp + e >= kend) v[e] = (T)0.0f;
          __builtin_memcpy(&regs[i], v, 16);
        }
      }
    }
  }

  __device__ __forceinline__ void store(char* lds, int tid) {
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      const int id = tid + i * NT;
      const int row = id / CPR, c = id % CPR;
      *reinterpret_cast<i32x4_t*>(lds + row * (CPR * 16) + swz<KC, CPR>(row, c) * 16) = regs[i];
    }
  }
};

/* MFMA operand fragment for a 32-row block starting at LDS row/column `mn` (multiple of 32) and
 * k-step kk of the tile. */
template <typename T, bool KC, int ROWS, int BK>
struct Frag;

template <bool KC, int ROWS, int BK>
struct Frag<__bf16, KC, ROWS, BK> {
  typedef bf16x8_t type;
  static constexpr int CPR = (KC ? BK : ROWS) / 8;
  static __device__ __forceinline__ type read(const char* lds, int mn, int kk, int lane) {
    if constexpr (KC) {
      const int row = mn + (lane & 31);
      const int c = kk * 2 + (lane >> 5);
      return __builtin_bit_cast(type, *reinterpret_cast<const i32x4_t*>(lds + row * (CPR * 16) + swz<true, CPR>(row, c) * 16));
    } else {
      const int g = lane >> 4, i = lane & 15;
      const int col = mn + (g & 1) * 16 + (i & 3) * 4;
      const int krow = kk * 16 + (g >> 1) * 8 + (i >> 2);
      const int c = col >> 3, sub = (col & 7) * 2;
      const char* p0 = lds + krow * (CPR * 16) + swz<false, CPR>(krow, c) * 16 + sub;
      const char* p1 = lds + (krow + 4) * (CPR * 16) + swz<false, CPR>(krow + 4, c) * 16 + sub;
      s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4_t, p0));
      s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4_t, p1));
      typedef short s16x8_t __attribute__((ext_vector_type(8)));
      s16x8_t v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      return __builtin_bit_cast(type, v);
    }
  }
};

/* The same two fragment fetches as FragReader::read, written as instructions of their own.  The compiler treats every
 * LDS read it knows about as possibly aliasing the direct-to-LDS loads in flight and waits for ALL of them (vmcnt 0)
 * in front of it, which would drain a ring of several tiles on every tile.  These reads are ordered by hand instead:
 * the kernel waits for the awaited tile's loads (vmcnt) and a barrier before it reads a slot, and for the LDS counter
 * before it uses the values.  `off` is a compile-time byte offset (below 65536). */
template <int OFF>
__device__ __forceinline__ bf16x8_t lds_read_b128_at(unsigned addr) {
  i32x4_t v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
  return __builtin_bit_cast(bf16x8_t, v);
}
template <int OFF_LO, int OFF_HI>
__device__ __forceinline__ bf16x8_t lds_read_tr_pair_at(unsigned addr) {
  typedef int i32x2_t __attribute__((ext_vector_type(2)));
  i32x2_t lo, hi;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(lo) : "v"(addr), "n"(OFF_LO));
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(hi) : "v"(addr), "n"(OFF_HI));
  i32x4_t v = {lo[0], lo[1], hi[0], hi[1]};
  return __builtin_bit_cast(bf16x8_t, v);
}

/* The same bf16 fragment fetch with the address arithmetic folded.  The swizzles are XORs, so the byte
 * address of the fragment of 32-row block i (rows wave_mn + 32 i ..) at k-step kk of a tile is
 *   K-contiguous:    ((lane constant + tile address) ^ (kk << 5)) + i * 32 rows
 *   M/N-contiguous:  (lane constant ^ (block index << 6)) + tile address + kk * 16 rows (+ 4 rows, second half)
 * and a wave keeps one register (K-contiguous) or one per block (M/N-contiguous) instead of an address
 * per fragment.  Tile addresses are multiples of 512 bytes. */
template <bool KC, int ROWS, int BK, int NBLK>
struct FragReader {
  static constexpr int CPR = (KC ? BK : ROWS) / 8;
  static constexpr int ROWB = CPR * 16;
  unsigned at[KC ? 1 : NBLK];
  __device__ __forceinline__ void init(int lane, int wave_mn) {
    if constexpr (KC) {
      const int r = lane & 31, h = lane >> 5;
      at[0] = (unsigned)((wave_mn + r) * ROWB + ((h ^ swz<true, CPR>(r, 0)) << 4));
    } else {
      static_assert(CPR >= 8, "M/N-contiguous fragment addressing assumes rows of 128 bytes or more");
      const int g = lane >> 4, i = lane & 15;
      const int x = i >> 2, cl = (g & 1) * 2 + ((i & 3) >> 1);
      const unsigned lc = (unsigned)(((g >> 1) * 8 + x) * ROWB) + ((unsigned)((x << (CPR >= 16 ? 6 : 5)) ^ (cl << 4)) | (unsigned)(i & 1) * 8u);
#pragma unroll
      for (int b = 0; b < NBLK; ++b) at[b] = lc ^ (unsigned)(((wave_mn >> 5) + b) << 6);
    }
  }
  /* read() with the hand-ordered LDS instructions (see lds_read_b128_at); BLK and KKI fold into the offset field. */
  template <int BLK, int KKI>
  __device__ __forceinline__ bf16x8_t read_unordered(unsigned tile) const {
    if constexpr (KC) return lds_read_b128_at<BLK * 32 * ROWB>((at[0] + tile) ^ (unsigned)(KKI << 5));
    else return lds_read_tr_pair_at<KKI * 16 * ROWB, KKI * 16 * ROWB + 4 * ROWB>(at[BLK] + tile);
  }
  __device__ __forceinline__ bf16x8_t read(unsigned tile, int blk, int kk) const {
    if constexpr (KC) {
      const unsigned addr = ((at[0] + tile) ^ (unsigned)(kk << 5)) + (unsigned)(blk * 32 * ROWB);
      return __builtin_bit_cast(bf16x8_t, *(LDS_PTR(const i32x4_t, (unsigned long)addr)));
    } else {
      const unsigned addr = at[blk] + tile + (unsigned)(kk * 16 * ROWB);
      s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4_t, (unsigned long)addr));
      s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4_t, (unsigned long)(addr + 4 * ROWB)));
      typedef short s16x8_t __attribute__((ext_vector_type(8)));
      s16x8_t v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      return __builtin_bit_cast(bf16x8_t, v);
    }
  }
};

__device__ __forceinline__ unsigned lds_addr(const void* p) { return (unsigned)(unsigned long)LDS_PTR(const char, p); }

template <bool KC, int ROWS, int BK>
struct Frag<float, KC, ROWS, BK> {
  typedef float type;
  static constexpr int CPR = (KC ? BK : ROWS) / 4;
  static __device__ __forceinline__ type read(const char* lds, int mn, int kk, int lane) {
    if constexpr (KC) {
      const int row = mn + (lane & 31);
      const int k = kk * 2 + (lane >> 5);
      return *reinterpret_cast<const float*>(lds + row * (CPR * 16) + swz<true, CPR>(row, k >> 2) * 16 + (k & 3) * 4);
    } else {
      const int krow = kk * 2 + (lane >> 5);
      const int col = mn + (lane & 31);
      return *reinterpret_cast<const float*>(lds + krow * (CPR * 16) + swz<false, CPR>(krow, col >> 2) * 16 + (col & 3) * 4);
    }
  }
};

__device__ __forceinline__ f32x16_t mfma(bf16x8_t a, bf16x8_t b, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x16_t mfma(float a, float b, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

/* Workgroup id -> tile, keeping the workgroups that share an XCD (ids congruent mod 8 are
 * dispatched to the same die and L2) on a compact block of the tile grid. */
__device__ __forceinline__ int xcd_logical(int bid, int nblocks) {
  constexpr int XCDS = 8;
  const int xcd = bid % XCDS, local = bid / XCDS;
  const int q = nblocks / XCDS, r = nblocks % XCDS;
  return xcd * q + (xcd < r ? xcd : r) + local;
}

__device__ __forceinline__ void tile_of_logical(int logical, int tiles_m, int tiles_n, int* tm, int* tn) {
  constexpr int GM = 4;
  const int per_group = GM * tiles_n;
  const int group = logical / per_group, in_group = logical % per_group;
  const int first_m = group * GM;
  const int gsize = tiles_m - first_m < GM ? tiles_m - first_m : GM;
  *tm = first_m + in_group % gsize;
  *tn = in_group / gsize;
}

__device__ __forceinline__ void tile_of_block(int bid, int nblocks, int tiles_m, int tiles_n, int* tm, int* tn) {
  tile_of_logical(xcd_logical(bid, nblocks), tiles_m, tiles_n, tm, tn);
}

/* Which group, output tile and K split a workgroup of the tiled kernels works on.  A single product keeps
 * the map above.  In a grouped launch (gridDim.y groups of gridDim.x workgroups, dispatched x-fastest)
 * the XCD-contiguous renumbering runs over ALL workgroups, so an XCD works through whole groups one
 * after the other (a group's tiles share its operands in that XCD's L2) and every XCD gets the same
 * number of workgroups whatever the group count. */
struct BlockPos { int grp, out_tile, split, tm, tn; };
__device__ __forceinline__ BlockPos block_pos(const GemmArgs& args) {
  BlockPos b;
  const int ksplit = args.ksplit;
  if (gridDim.y == 1) {
    b.grp = 0;
    b.out_tile = blockIdx.x / ksplit; b.split = blockIdx.x - b.out_tile * ksplit;
    tile_of_block(b.out_tile, gridDim.x / ksplit, args.tiles_m, args.tiles_n, &b.tm, &b.tn);
  } else {
    const int logical = xcd_logical(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
    b.grp = logical / (int)gridDim.x;
    const int in_group = logical - b.grp * (int)gridDim.x;
    b.out_tile = in_group / ksplit; b.split = in_group - b.out_tile * ksplit;
    tile_of_logical(b.out_tile, args.tiles_m, args.tiles_n, &b.tm, &b.tn);
  }
  return b;
}

/* The arguments of the epilogue that leaves a split's raw fp32 tile [bm][bn] in the workspace: bias, activation and the real store
 * happen in the reduction kernel. */
__device__ __forceinline__ GemmArgs partial_outputs(const GemmArgs& args, const BlockPos& bp, int bm, int bn) {
  GemmArgs pa = args;
  pa.c = args.partial + (((long long)bp.grp * (gridDim.x / args.ksplit) + bp.out_tile) * args.ksplit + bp.split) * (bm * bn);
  pa.ldc = bn; pa.M = bm; pa.N = bn; pa.skewM = 0; pa.skewN = 0;
  pa.preact = nullptr; pa.bias = nullptr; pa.act = HAP_ACT_NONE; pa.accumulate = 0; pa.vec_store = 1; pa.cdelta = 0; pa.dact_preact = nullptr;
  return pa;
}

/* Writes a wave's TM x TN accumulator tiles.  Accumulator element e of lane l is row
 * (e/4)*8 + (l/32)*4 + e%4, column l%32 of its 32x32 tile.  (row0, col0): physical origin of the
 * wave tile; rows / columns outside the logical extent are dropped. */
template <typename T, typename TC, int TM, int TN>
__device__ __forceinline__ void epilogue(const GemmArgs& args, f32x16_t (&acc)[TM][TN], int row0, int col0, int lane) {
  TC* C = static_cast<TC*>(args.c);
  TC* P = static_cast<TC*>(args.preact);
  const T* bias = static_cast<const T*>(args.bias);
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int n = col0 + j * 32 + (lane & 31) - args.skewN;
    const bool n_ok = n >= 0 && n < args.N;
    const float bv = (bias && n_ok) ? load_s<T>(bias + n) : 0.0f;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int m = row0 + i * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3) - args.skewM;
        if (n_ok && m >= 0 && m < args.M) {
          float v = acc[i][j][e] + bv;
          if (P) store_c<TC>(P + (long long)m * args.ldp + n, v);
          if (args.act == HAP_ACT_GELU_ERF) v = gelu_erf((float)(TC)v);     // the activation sees the value as stored
          if (args.dact_preact) v *= gelu_erf_grad(load_s<TC>(static_cast<const TC*>(args.dact_preact) + (long long)m * args.ldd + n));
          TC* dst = C + (long long)m * args.ldc + n;
          if (args.accumulate) v += load_s<TC>(dst);
          store_c<TC>(dst, v);
        }
      }
    }
  }
}

template <typename T, typename TC, bool AKC, bool BKC, int BM, int BN, int BK, int WGM, int WGN>
__global__ __launch_bounds__(64 * WGM * WGN) void gemm_kernel(const GemmArgs args) {
  constexpr int NT = 64 * WGM * WGN;
  constexpr int ES = sizeof(T);
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  constexpr int KSTEP = Elem<T>::kStep;
  static_assert(WTM % 32 == 0 && WTN % 32 == 0 && BK % KSTEP == 0, "tile shape");

  __shared__ __attribute__((aligned(16))) char lds_a[BM * BK * ES];
  __shared__ __attribute__((aligned(16))) char lds_b[BN * BK * ES];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm0 = (wave / WGN) * WTM, wn0 = (wave % WGN) * WTN;
  // With split-K, ksplit consecutive workgroups share an output tile and take consecutive K-tile ranges.
  const BlockPos bp = block_pos(args);
  const int ksplit = args.ksplit, split = bp.split, tm = bp.tm, tn = bp.tn;
  const int m0 = tm * BM, n0 = tn * BN;                 // physical tile origin
  const GroupView gv = group_view(args, bp.grp);
  const int m_lim = args.skewM + gv.M, n_lim = args.skewN + args.N;
  if (args.ragged == 1 && (gv.M == 0 || m0 >= m_lim)) return;   // the group's rows end before this tile
  const int all_tiles = gv.k >= 0 ? (args.skewK + gv.k + BK - 1 >= BK ? (args.skewK + gv.k + BK - 1) / BK : 1) : args.ntiles;

  TileLoader<T, AKC, BM, BK, NT> la;
  TileLoader<T, BKC, BN, BK, NT> lb;

  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

  // this workgroup's range [first, first + ntiles) of the K tiles of all segments laid end to end
  const int first = (int)((long long)all_tiles * split / ksplit);
  int ntiles = (int)((long long)all_tiles * (split + 1) / ksplit) - first;
  int seg = 0, skip = first;
  while (seg + 1 < args.nseg) {
    const int in_seg = (args.skewK + args.seg[seg].k + BK - 1) / BK;
    if (skip < in_seg) break;
    skip -= in_seg;
    seg = uni(seg + 1);
  }
  // loader state runs one tile ahead of the compute
  int k0 = skip * BK;
  int kend = uni(args.skewK + (gv.k >= 0 ? gv.k : args.seg[seg].k));
  __amdgpu_buffer_rsrc_t ra = make_rsrc(static_cast<const char*>(args.seg[seg].a) + gv.oa, args.seg[seg].a_bytes);
  __amdgpu_buffer_rsrc_t rb = make_rsrc(static_cast<const char*>(args.seg[seg].b) + gv.ob, args.seg[seg].b_bytes);

  auto fetch = [&]() {
    la.load(ra, tid, m0, m_lim, args.lda, k0, args.skewK, kend);
    lb.load(rb, tid, n0, n_lim, args.ldb, k0, args.skewK, kend);
  };
  auto commit = [&](int ck0, int ckend) {
    if (ck0 < args.skewK || ck0 + BK > ckend) {
      la.mask_k(tid, ck0, args.skewK, ckend);
      lb.mask_k(tid, ck0, args.skewK, ckend);
    }
    la.store(lds_a, tid);
    lb.store(lds_b, tid);
  };

  if (ntiles > 0) fetch();
  while (ntiles > 0) {     // (a split's share of a contraction shortened on the device side can be empty)
    const int ck0 = k0, ckend = kend;
    // advance the loader to the next tile
    k0 += BK;
    bool more = --ntiles > 0;
    if (more && k0 >= kend) {
      ++seg;
      if (seg < args.nseg) {
        k0 = 0;
        seg = uni(seg);
        kend = uni(args.skewK + args.seg[seg].k);
        ra = make_rsrc(static_cast<const char*>(args.seg[seg].a) + gv.oa, args.seg[seg].a_bytes);
        rb = make_rsrc(static_cast<const char*>(args.seg[seg].b) + gv.ob, args.seg[seg].b_bytes);
      } else {
        more = false;
      }
    }
    commit(ck0, ckend);
    __syncthreads();
    if (more) fetch();
#pragma unroll
    for (int kk = 0; kk < BK / KSTEP; ++kk) {
      typename Frag<T, AKC, BM, BK>::type fa[TM];
      typename Frag<T, BKC, BN, BK>::type fb[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[i] = Frag<T, AKC, BM, BK>::read(lds_a, wm0 + i * 32, kk, lane);
#pragma unroll
      for (int j = 0; j < TN; ++j) fb[j] = Frag<T, BKC, BN, BK>::read(lds_b, wn0 + j * 32, kk, lane);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = mfma(fa[i], fb[j], acc[i][j]);
    }
    if (!more) break;
    __syncthreads();
  }

  if (ksplit > 1) {
    const GemmArgs pa = partial_outputs(args, bp, BM, BN);
    epilogue<T, float, TM, TN>(pa, acc, wm0, wn0, lane);
    return;
  }
  epilogue<T, TC, TM, TN>(group_outputs(args, gv, bp.grp), acc, m0 + wm0, n0 + wn0, lane);
}

/* Epilogue of the direct-to-LDS kernels.  Their accumulators are TRANSPOSED tiles (the MFMA is fed
 * B-fragment first), so element e of lane l belongs to output row l%32 and columns
 * (e/4)*8 + (l/32)*4 + e%4: four consecutive columns per register quad.  Each wave passes one
 * 32-row block at a time through a private LDS patch and writes it out as whole 16-byte chunks,
 * eight (bf16) or four (fp32) lanes per 128-byte line, instead of 2-byte scattered stores.
 * Bias, activation, the optional pre-activation copy and fp32 accumulation are applied on the way.
 * Falls back to element stores where the destination is not 16-byte addressable or at ragged ends. */
template <typename TC> struct Vec16;
template <> struct Vec16<__bf16> { typedef __bf16 type __attribute__((ext_vector_type(8))); };
template <> struct Vec16<float> { typedef float type __attribute__((ext_vector_type(4))); };

/* MODE 0: bias, optional pre-activation copy (a pass of its own), optional accumulation; no activation.
 * MODE 1 (DACT): the product times act'(dact_preact); no bias, activation, copy or accumulation (the host sees to that).
 * MODE 2 (ACTP): activation, with the optional pre-activation copy in the SAME pass through the patch: the pre-activation chunk is
 *         stored as it comes out of the patch and the activation is applied to those same, already rounded values,
 *         H = act(round(P)) - what a framework computes that stores P and then applies the activation to the stored tensor, and
 *         the point at which the backward evaluates act'.  Every epilogue of the engine rounds before the activation, with or
 *         without a copy, so a layer's output does not depend on whether its pre-activation is kept. */
template <typename T, typename TC, int TM, int TN, bool SHIFTED, int MODE>
__device__ __forceinline__ void epilogue_transposed_impl(const GemmArgs& args, f32x16_t (&acc)[TM][TN], int row0, int col0, int lane, char* patch) {
  constexpr bool DACT = MODE == 1, ACTP = MODE == 2;
  constexpr int ES = sizeof(TC);
  constexpr int EPC = 16 / ES;
  constexpr int COLS = TN * 32;
  constexpr int ROWB = COLS * ES + 16;            // padded row of the LDS patch
  constexpr int CH = COLS * ES / 16;              // 16-byte chunks per row
  typedef typename Vec16<TC>::type vec_t;
  TC* C = static_cast<TC*>(args.c);
  TC* P = static_cast<TC*>(args.preact);
  const T* bias = static_cast<const T*>(args.bias);
  const int h = lane >> 5, ml = lane & 31;
  const bool vec_ok = args.vec_store != 0;
  // A shard's columns start anywhere (column 8402 of a bf16 matrix is byte 16804), so C's 16-byte chunks need not coincide with the
  // tile's: the tile is written into the patch `delta` columns to the right (the row padding takes the overflow), which makes patch
  // chunk c the destination chunk that starts at tile column c * EPC - delta; only row ends are then stored element by element.
  const int delta = SHIFTED ? args.cdelta : 0;
  constexpr int nchunks = SHIFTED ? CH + 1 : CH;
  // this lane's bias values: the same 4 consecutive columns of every 8-column group, for all row blocks and passes
  // (DACT: the host admits no bias either, which frees these registers for the pre-activation chunks below)
  float bv[DACT ? 1 : TN][4][4];
  if constexpr (!DACT) {
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const int n = col0 + j * 32 + g * 8 + h * 4 + x - args.skewN;
          bv[j][g][x] = (bias && n >= 0 && n < args.N) ? load_s<T>(bias + n) : 0.0f;
        }
  }
  constexpr int ITS = (32 * nchunks + 63) / 64;          // 16-byte chunks of one 32-row block per lane
  // (row, column, valid part) of the chunk this lane stores in iteration `it` of row block i
  auto chunk_at = [&](int i, int it, int* m, int* n, int* t_lo, int* t_hi) -> bool {
    const int idx = it * 64 + lane;
    const int r = idx / nchunks, c = idx % nchunks;
    *m = row0 + i * 32 + r - args.skewM;
    *n = col0 + c * EPC - delta - args.skewN;
    // (a patch chunk also ends where the tile's columns end: what lies beyond was not written in this pass)
    *t_lo = c * EPC - delta < 0 ? delta - c * EPC : 0;
    *t_hi = c * EPC - delta + EPC > COLS ? COLS - (c * EPC - delta) : EPC;
    return (!SHIFTED || idx < 32 * nchunks) && *m >= 0 && *m < args.M && *n + *t_lo < args.N && *n + *t_hi > 0;
  };
  // DACT: all pre-activation chunks of the wave's tile are requested now, in one burst, so that the stores below wait for one
  // memory round trip instead of one per chunk
  // (an fp32 tile has twice the chunks: there the requests go out one row block at a time, ahead of that block's patch traffic)
  constexpr int BURST = ES == 2 ? TM : 1;
  vec_t pvs[DACT ? BURST : 1][DACT ? ITS : 1];
  auto request_preact = [&](int i, int slot) {
#pragma unroll
    for (int it = 0; it < ITS; ++it) {
      int m, n, t_lo, t_hi;
      // (a chunk that this wave stores only part of - its other columns belong to the neighbouring wave's tile - is still read whole)
      if (chunk_at(i, it, &m, &n, &t_lo, &t_hi) && vec_ok && n >= 0 && n + EPC <= args.N)
        pvs[slot][it] = *reinterpret_cast<const vec_t*>(static_cast<const TC*>(args.dact_preact) + (long long)m * args.ldd + n);
    }
  };
  if constexpr (DACT && BURST == TM) {
#pragma unroll
    for (int i = 0; i < TM; ++i) request_preact(i, i);
  }
#pragma unroll
  for (int i = 0; i < TM; ++i) {
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
      if (pass == 0 && (DACT || ACTP || !P)) continue;
      if constexpr (DACT && BURST < TM) request_preact(i, 0);
      TC* dst_base = pass == 0 ? P : C;
      const long long ldd = pass == 0 ? args.ldp : args.ldc;
      // registers -> LDS patch [32 rows][COLS]
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int cl = j * 32 + g * 8 + h * 4;            // first of 4 consecutive columns
          TC v[4];
#pragma unroll
          for (int x = 0; x < 4; ++x) {
            float f = acc[i][j][g * 4 + x];
            if constexpr (!DACT) f += bv[j][g][x];
            v[x] = (TC)f;
          }
          if constexpr (!SHIFTED) {
            __builtin_memcpy(patch + ml * ROWB + cl * ES, v, 4 * ES);
          } else {
            TC* q = reinterpret_cast<TC*>(patch + ml * ROWB) + cl + delta;
#pragma unroll
            for (int x = 0; x < 4; ++x) q[x] = v[x];
          }
        }
      // Order the patch accesses of this wave only: LDS operations of a wave execute in order, so a
      // wait on the LDS counter is enough (a fence would also drain the global stores in flight).
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_wave_barrier();
      // LDS patch -> global, 16 bytes per lane.  (An fp32 tile has eight iterations per block; all of them in flight at once, each
      // with its chunk, its address and - when accumulating - the old chunk, overflowed the registers the accumulators leave.)
      constexpr int kStoreUnroll = (ES == 4 && !DACT) ? 2 : ITS;
#pragma unroll kStoreUnroll
      for (int it = 0; it < ITS; ++it) {
        int m, n, t_lo, t_hi;
        if (!chunk_at(i, it, &m, &n, &t_lo, &t_hi)) continue;
        const int idx = it * 64 + lane;
        const int r = idx / nchunks, c = idx % nchunks;
        vec_t val = *reinterpret_cast<const vec_t*>(patch + r * ROWB + c * 16);
        TC* dst = dst_base + (long long)m * ldd + n;
        const TC* dpre = DACT ? static_cast<const TC*>(args.dact_preact) + (long long)m * args.ldd + n : nullptr;
        // (vec_ok implies that dact_preact shares C's 16-byte phase and pitch rule.)  The multiplication is done once, for whole
        // chunks, before the lanes part into chunk stores and element stores; elements of a partly stored chunk that lie outside
        // this wave's columns hold patch leftovers and are dropped below.
        const bool pv_ok = DACT && vec_ok && n >= 0 && n + EPC <= args.N;
        if constexpr (DACT) {
          if (pv_ok) {
            const vec_t pv = pvs[BURST == TM ? i : 0][it];
#pragma unroll
            for (int x = 0; x < EPC; ++x) val[x] = (TC)((float)val[x] * gelu_erf_grad((float)pv[x]));
          }
        }
        // ACTP: keep the pre-activation chunk, apply the activation to the whole chunk once (leftover elements are dropped below)
        vec_t pre = val;
        TC* pdst = ACTP ? P + (long long)m * args.ldp + n : nullptr;
        if constexpr (ACTP) {
#pragma unroll
          for (int x = 0; x < EPC; ++x) val[x] = (TC)gelu_erf((float)val[x]);
        }
        if (vec_ok && n >= 0 && n + EPC <= args.N && t_lo == 0 && t_hi == EPC) {
          // The pre-activation copy is read again only by the backward: it goes out non-temporally and leaves the caches to the operands.
          // Against a plain store, forward + backward: ten experts 737 -> 729 us, a 315-wide MLP slice over 50432 tokens 478 -> 471, an
          // 8402-wide one over 8192 2922 -> 2907; small layers and whole encoder layers within 0.3 %.  The output itself is what the next
          // product reads and stays a plain store.
          if constexpr (ACTP) {
            if (P) {
              if constexpr (ES == 2) __builtin_nontemporal_store(pre, reinterpret_cast<vec_t*>(pdst));
              else *reinterpret_cast<vec_t*>(pdst) = pre;
            }
          }
          if (!DACT && pass == 1 && args.accumulate) {
            const vec_t old = *reinterpret_cast<const vec_t*>(dst);
#pragma unroll
            for (int x = 0; x < EPC; ++x) val[x] = (TC)((float)val[x] + (float)old[x]);
          }
          *reinterpret_cast<vec_t*>(dst) = val;
        } else {
          // Rare (a chunk cut by a row end or by the wave's strip, or a destination that is not 16-byte addressable): element by
          // element, straight from the patch, as a real loop - unrolled eight-fold into every iteration above it made the epilogue
          // several times the size of the instruction cache, and the waves waited for code, not for data.
          // (read through an LDS-space pointer: a generic one makes the load a flat instruction, which counts on the memory
          // counter as well and makes every later wait for patch data a wait for the global stores in flight)
          const unsigned pe = lds_addr(patch + r * ROWB + c * 16);
#pragma unroll 1
          for (int x = t_lo; x < t_hi; ++x) {
            if (n + x < 0 || n + x >= args.N) continue;
            float f = (float)*LDS_PTR(const TC, (unsigned long)(pe + x * ES));
            if constexpr (ACTP) { if (P) store_c<TC>(pdst + x, f); f = gelu_erf(f); }
            if constexpr (DACT) f = (float)(TC)f * gelu_erf_grad(load_s<TC>(dpre + x));
            if (!DACT && pass == 1 && args.accumulate) f += load_s<TC>(dst + x);
            store_c<TC>(dst + x, f);
          }
        }
      }
      // Order the patch accesses of this wave only: LDS operations of a wave execute in order, so a
      // wait on the LDS counter is enough (a fence would also drain the global stores in flight).
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_wave_barrier();
    }
    HAP_EXP_STAMP(4 + (i & 3));
  }
}

template <typename T, typename TC, int TM, int TN>
__device__ __forceinline__ void epilogue_transposed(const GemmArgs& args, f32x16_t (&acc)[TM][TN], int row0, int col0, int lane, char* patch) {
  if (args.dact_preact) {
    if (args.cdelta) epilogue_transposed_impl<T, TC, TM, TN, true, 1>(args, acc, row0, col0, lane, patch);
    else epilogue_transposed_impl<T, TC, TM, TN, false, 1>(args, acc, row0, col0, lane, patch);
  } else if (args.act == HAP_ACT_GELU_ERF) {
    if (args.cdelta) epilogue_transposed_impl<T, TC, TM, TN, true, 2>(args, acc, row0, col0, lane, patch);
    else epilogue_transposed_impl<T, TC, TM, TN, false, 2>(args, acc, row0, col0, lane, patch);
  } else if (args.cdelta) epilogue_transposed_impl<T, TC, TM, TN, true, 0>(args, acc, row0, col0, lane, patch);
  else epilogue_transposed_impl<T, TC, TM, TN, false, 0>(args, acc, row0, col0, lane, patch);
}

/* ---------------------------------------------------------------------------------------------
 * bf16 main kernel: global -> LDS by buffer loads that write LDS directly (no register staging),
 * STAGES-deep ring of tiles, one barrier per tile.
 *
 * A wave-wide direct load writes 64 lanes x 16 bytes to CONSECUTIVE LDS bytes, so the XOR swizzle is
 * applied on the global side: the lane that fills LDS chunk position p of a row fetches the chunk
 * whose swizzled position is p.  Interior tiles use precomputed per-lane offsets plus one scalar
 * offset per tile; the first / last tile of a segment recompute validity per chunk and, for
 * K-contiguous operands, zero the elements outside the logical k range in LDS once the data landed.
 * ------------------------------------------------------------------------------------------- */
template <bool KC, int ROWS, int BK, int NT>
struct DmaLoader {
  static constexpr int EPC = 8;
  static constexpr int LROWS = KC ? ROWS : BK;
  static constexpr int CPR = (KC ? BK : ROWS) / EPC;
  static constexpr int CPT = LROWS * CPR / NT;
  static constexpr int TILE_BYTES = ROWS * BK * 2;
  static_assert(LROWS * CPR % NT == 0, "tile chunks must divide evenly over threads");

  unsigned base[CPT];   // byte offset of this lane's chunk for k0 = 0, or the out-of-range marker

  /* LDS position id -> (row, logical chunk) */
  static __device__ __forceinline__ void where(int id, int* row, int* c) {
    *row = id / CPR;
    *c = swz<KC, CPR>(*row, id % CPR);
  }

  /* mn0: the tile's first physical row / column; [mn_lo, mn_lim): the physical range that holds the operand's logical rows /
   * columns.  A K-contiguous operand's rows may be placed mn_lo rows into the tile grid (so that the OUTPUT's columns fall on
   * its 16-byte chunks): grid rows below mn_lo do not exist and read as zero.  mn_lo is 0 for an M-/N-contiguous operand,
   * whose skew is part of its aligned-down base address. */
  __device__ __forceinline__ void init(int tid, int mn0, int mn_lo, int mn_lim, long long ld) {
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      int row, c;
      where(tid + i * NT, &row, &c);
      if constexpr (KC) {
        const int mn = mn0 + row;
        base[i] = (mn >= mn_lo && mn < mn_lim) ? (unsigned)(((long long)(mn - mn_lo) * ld + c * EPC) * 2) : kOobOffset;
      } else {
        const int mn = mn0 + c * EPC;
        base[i] = mn < mn_lim ? (unsigned)(((long long)row * ld + mn) * 2) : kOobOffset;
      }
    }
  }

  /* Byte offset of a tile starting at physical k0: k0 elements along a row (KC) or (k0 - kskew) rows. */
  static __device__ __forceinline__ unsigned tile_offset(int k0, int kskew, long long ld) {
    if constexpr (KC) return (unsigned)k0 * 2u;
    else return (unsigned)((long long)(k0 - kskew) * ld * 2);
  }

  /* Interior tile: every k of the tile is inside the logical range; soff = tile_offset() >= 0 goes in
   * the instruction's scalar offset. */
  __device__ __forceinline__ void issue(__amdgpu_buffer_rsrc_t rsrc, char* lds, int tid, unsigned soff) const {
    const int wave_first = uni(tid & ~63);      // pinned to a scalar register: it feeds M0, the LDS address of the direct load
#pragma unroll
    for (int i = 0; i < CPT; ++i) dma16(rsrc, lds + (wave_first + i * NT) * 16, base[i], soff);
  }

  /* The loads i of an interior tile with i % nparts == part.  A tile's loads are spread between the
   * MFMA groups of the previous tile: issued back to back they fill the memory queue and the wave
   * blocks on it instead of feeding the matrix unit.  `part` and `nparts` fold at compile time. */
  __device__ __forceinline__ void issue_part(__amdgpu_buffer_rsrc_t rsrc, char* lds, int tid, unsigned soff, int part, int nparts) const {
    const int wave_first = (tid & ~63);
#pragma unroll
    for (int i = 0; i < CPT; ++i)
      if (i % nparts == part) dma16(rsrc, lds + (wave_first + i * NT) * 16, base[i], soff);
  }

  /* Edge tile: validity along k decided per chunk; the tile offset (which may be "negative" for the
   * rows a skewed first tile does not use) is added per lane so valid chunks get an exact offset. */
  __device__ __forceinline__ unsigned edge_offset(int i, int tid, unsigned toff, int k0, int kskew, int kend) const {
    int row, c;
    where(tid + i * NT, &row, &c);
    bool ok;
    if constexpr (KC) { const int kp = k0 + c * EPC; ok = kp < kend && kp + EPC > kskew; }
    else { const int kl = k0 + row; ok = kl >= kskew && kl < kend; }
    return ok && base[i] != kOobOffset ? base[i] + toff : kOobOffset;
  }
  __device__ __forceinline__ void edge_offsets(unsigned (&off)[CPT], int tid, unsigned toff, int k0, int kskew, int kend) const {
#pragma unroll
    for (int i = 0; i < CPT; ++i) off[i] = edge_offset(i, tid, toff, k0, kskew, kend);
  }
  __device__ __forceinline__ void issue_edge(__amdgpu_buffer_rsrc_t rsrc, char* lds, int tid, unsigned toff, int k0, int kskew, int kend) const {
    const int wave_first = (tid & ~63);
#pragma unroll
    for (int i = 0; i < CPT; ++i) dma16(rsrc, lds + (wave_first + i * NT) * 16, edge_offset(i, tid, toff, k0, kskew, kend), 0);
  }

  /* After the edge tile landed: zero elements outside [kskew, kend) in this thread's own chunks. */
  __device__ __forceinline__ void fixup(char* lds, int tid, int k0, int kskew, int kend) const {
    if constexpr (KC) {
#pragma unroll
      for (int i = 0; i < CPT; ++i) {
        int row, c;
        where(tid + i * NT, &row, &c);
        const int kp = k0 + c * EPC;
        if (kp < kend && kp + EPC > kskew && (kp < kskew || kp + EPC > kend)) {
          i32x4_t* q = reinterpret_cast<i32x4_t*>(lds + (tid + i * NT) * 16);
          bf16x8_t v = __builtin_bit_cast(bf16x8_t, *q);
#pragma unroll
          for (int e = 0; e < EPC; ++e)
            if (kp + e < kskew || kp + e >= kend) v[e] = (__bf16)0.0f;
          *q = __builtin_bit_cast(i32x4_t, v);
        }
      }
    }
  }
};

template <typename TC, bool AKC, bool BKC, int BM, int BN, int BK, int WGM, int WGN, int STAGES>
__global__ __launch_bounds__(64 * WGM * WGN, (WGM * WGN <= 4 ? 2 : 1))   /* the 4-wave kernel is built to share a compute unit with a second workgroup: two waves per SIMD */ void gemm_dma_kernel(const GemmArgs args) {
  typedef __bf16 T;
  constexpr int NT = 64 * WGM * WGN;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2, STAGE_BYTES = A_BYTES + B_BYTES;
  typedef DmaLoader<AKC, BM, BK, NT> LA;
  typedef DmaLoader<BKC, BN, BK, NT> LB;
  constexpr int LOADS_PER_TILE = LA::CPT + LB::CPT;

  extern __shared__ __attribute__((aligned(1024))) char smem[];   // FragReader needs tile addresses that are multiples of 512

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm0 = (wave / WGN) * WTM, wn0 = (wave % WGN) * WTN;
  // With split-K, ksplit consecutive workgroups share an output tile and take consecutive K-tile ranges.
  const BlockPos bp = block_pos(args);
  const int ksplit = args.ksplit, split = bp.split, tm = bp.tm, tn = bp.tn;
  const int m0 = tm * BM, n0 = tn * BN;
  const GroupView gv = group_view(args, bp.grp);
  const int m_lim = args.skewM + gv.M, n_lim = args.skewN + args.N;
  if (args.ragged == 1 && (gv.M == 0 || m0 >= m_lim)) return;   // the group's rows end before this tile
  const int all_tiles = gv.k >= 0 ? (args.skewK + gv.k + BK - 1 >= BK ? (args.skewK + gv.k + BK - 1) / BK : 1) : args.ntiles;

  LA la; LB lb;
  la.init(tid, m0, AKC ? args.skewM : 0, m_lim, args.lda);
  lb.init(tid, n0, BKC ? args.skewN : 0, n_lim, args.ldb);
  FragReader<AKC, BM, BK, TM> fra;
  FragReader<BKC, BN, BK, TN> frb;
  fra.init(lane, wm0);
  frb.init(lane, wn0);

  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

  // this workgroup's range [first, first + ntiles) of the K tiles of all segments laid end to end
  const int first = (int)((long long)all_tiles * split / ksplit);
  const int ntiles = (int)((long long)all_tiles * (split + 1) / ksplit) - first;
  int seg0 = 0, skip = first;
  while (seg0 + 1 < args.nseg) {
    const int in_seg = (args.skewK + args.seg[seg0].k + BK - 1) / BK;
    if (skip < in_seg) break;
    skip -= in_seg;
    seg0 = uni(seg0 + 1);
  }
  // producer state (runs STAGES-1 tiles ahead of the consumer)
  int pseg = seg0, pk0 = skip * BK, pkend = uni(args.skewK + (gv.k >= 0 ? gv.k : args.seg[seg0].k)), pslot = 0;
  __amdgpu_buffer_rsrc_t ra = make_rsrc(static_cast<const char*>(args.seg[seg0].a) + gv.oa, args.seg[seg0].a_bytes);
  __amdgpu_buffer_rsrc_t rb = make_rsrc(static_cast<const char*>(args.seg[seg0].b) + gv.ob, args.seg[seg0].b_bytes);
  // consumer state: k range of the tile being consumed (for the edge fix-up)
  int cseg = seg0, ck0 = pk0, ckend = pkend, cslot = 0;
  constexpr int KK = BK / 16;
  constexpr int MF = TM * TN;                       // MFMAs per k-step

  auto advance_producer = [&]() {
    pslot = pslot + 1 == STAGES ? 0 : pslot + 1;
    pk0 += BK;
    if (pk0 >= pkend && pseg + 1 < args.nseg) {
      pseg = uni(pseg + 1);
      pk0 = 0;
      pkend = uni(args.skewK + args.seg[pseg].k);
      ra = make_rsrc(static_cast<const char*>(args.seg[pseg].a) + gv.oa, args.seg[pseg].a_bytes);
      rb = make_rsrc(static_cast<const char*>(args.seg[pseg].b) + gv.ob, args.seg[pseg].b_bytes);
    }
  };

  // prologue: request the first STAGES-1 tiles
#pragma unroll
  for (int s = 0; s < STAGES - 1; ++s)
    if (s < ntiles) {
      char* pa = smem + pslot * STAGE_BYTES;
      la.issue_edge(ra, pa, tid, LA::tile_offset(pk0, args.skewK, args.lda), pk0, args.skewK, pkend);
      lb.issue_edge(rb, pa + A_BYTES, tid, LB::tile_offset(pk0, args.skewK, args.ldb), pk0, args.skewK, pkend);
      advance_producer();
    }

  // One K tile.  FAST: the tile consumed and the tile requested are both interior tiles of their segments (all k
  // valid) and a request is due: no per-chunk validity, no fix-up, no data-dependent branch between the MFMAs, so
  // the whole tile is one scheduling region.  Otherwise the general form.
  auto tile = [&](int t, auto fast_tag) __attribute__((always_inline)) {
    constexpr bool FAST = decltype(fast_tag)::value;
    char* sa = smem + cslot * STAGE_BYTES;
    char* sb = sa + A_BYTES;
    // tile t must have landed; up to STAGES-2 newer tiles may stay in flight
    if (STAGES > 2 && t + STAGES - 2 < ntiles) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((STAGES - 2) * LOADS_PER_TILE) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (!FAST && (ck0 < args.skewK || ck0 + BK > ckend)) {
      la.fixup(sa, tid, ck0, args.skewK, ckend);
      lb.fixup(sb, tid, ck0, args.skewK, ckend);
    }
    ck0 += BK;
    if (!FAST && ck0 >= ckend && cseg + 1 < args.nseg) { cseg = uni(cseg + 1); ck0 = 0; ckend = uni(args.skewK + args.seg[cseg].k); }
    __syncthreads();          // tile visible to all waves; every wave is done with the slot refilled below

    // the next request goes out in pieces between the MFMA groups of this tile (interior tiles), or
    // at once (first / last tile of a segment, where validity is decided per chunk)
    const bool produce = FAST || t + STAGES - 1 < ntiles;
    const bool edge = !FAST && (pk0 < args.skewK || pk0 + BK > pkend);
    char* pa = smem + pslot * STAGE_BYTES;
    char* pb = pa + A_BYTES;
    const unsigned soa = LA::tile_offset(pk0, args.skewK, args.lda);
    const unsigned sob = LB::tile_offset(pk0, args.skewK, args.ldb);
    if (!FAST && produce && edge) {
      la.issue_edge(ra, pa, tid, soa, pk0, args.skewK, pkend);
      lb.issue_edge(rb, pb, tid, sob, pk0, args.skewK, pkend);
    }
    const bool spread = !FAST && produce && !edge;
    constexpr bool kAtOnce = AKC && BKC;   // measured: with two 128-bit-read operands the whole request right after the barrier is faster, otherwise spread

    // fragments run kFragAhead k-steps ahead of the MFMAs that use them: a wave that has its SIMD to itself
    // (its partner waits at the barrier) must not stall on LDS latency between k-steps
    constexpr int kFragAhead = KK > 3 ? 3 : (KK > 2 ? 2 : 1), NB = kFragAhead + 1;
    bf16x8_t fa[NB][TM], fb[NB][TN];
    const unsigned ta = lds_addr(sa), tb = lds_addr(sb);
#pragma unroll
    for (int k0 = 0; k0 < kFragAhead; ++k0) {
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[k0][i] = fra.read(ta, i, k0);
#pragma unroll
      for (int j = 0; j < TN; ++j) fb[k0][j] = frb.read(tb, j, k0);
    }
    // The scheduling fences keep this order: without them the compiler moves each fragment read down to just before
    // the MFMA that uses it (fewer live registers), and the wave then waits on LDS in front of every MFMA.
    if (FAST) __builtin_amdgcn_sched_barrier(0);
    if (FAST && kAtOnce) { la.issue(ra, pa, tid, soa); lb.issue(rb, pb, tid, sob); __builtin_amdgcn_sched_barrier(0); }
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const int cur = kk % NB, nxt = (kk + kFragAhead) % NB;
      if (kk + kFragAhead < KK) {
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[nxt][i] = fra.read(ta, i, kk + kFragAhead);
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[nxt][j] = frb.read(tb, j, kk + kFragAhead);
        if (FAST) __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int x = 0; x < MF / 2; ++x) acc[x / TN][x % TN] = mfma(fb[cur][x % TN], fa[cur][x / TN], acc[x / TN][x % TN]);
      if ((FAST && !kAtOnce) || spread) la.issue_part(ra, pa, tid, soa, kk, KK);
      if (FAST) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int x = MF / 2; x < MF; ++x) acc[x / TN][x % TN] = mfma(fb[cur][x % TN], fa[cur][x / TN], acc[x / TN][x % TN]);
      if ((FAST && !kAtOnce) || spread) lb.issue_part(rb, pb, tid, sob, kk, KK);
      if (FAST) __builtin_amdgcn_sched_barrier(0);
    }
    if (FAST) {      // the producer stays inside its segment
      pslot = pslot + 1 == STAGES ? 0 : pslot + 1;
      pk0 += BK;
    } else if (produce) {
      advance_producer();
    }
    cslot = cslot + 1 == STAGES ? 0 : cslot + 1;
  };
  // interior for the consumer: all of [ck0, ck0+BK) valid and not the segment's last tile; for the producer likewise,
  // and its next position stays inside the segment
  auto fast = [&](int t) {
    return t + STAGES - 1 < ntiles && ck0 >= args.skewK && ck0 + 2 * BK <= ckend && pk0 >= args.skewK && pk0 + 2 * BK <= pkend;
  };
  for (int t = 0; t < ntiles;) {
    for (; t < ntiles && !fast(t); ++t) tile(t, std::false_type());
    for (; t < ntiles && fast(t); ++t) tile(t, std::true_type());
  }

  __syncthreads();   // every wave is done reading the ring: reuse it as per-wave store patches
  if (ksplit > 1) {
    const GemmArgs pa = partial_outputs(args, bp, BM, BN);
    epilogue_transposed<T, float, TM, TN>(pa, acc, wm0, wn0, lane, smem + wave * (32 * (TN * 32 * 4 + 16)));
    return;
  }
  epilogue_transposed<T, TC, TM, TN>(group_outputs(args, gv, bp.grp), acc, m0 + wm0, n0 + wn0, lane, smem + wave * (32 * (TN * 32 * (int)sizeof(TC) + 16)));
}

/* ---------------------------------------------------------------------------------------------
 * bf16 main kernel for 256 x 256 output tiles: the same direct-to-LDS loads, swizzles and fragment
 * addressing as gemm_dma_kernel, with the eight waves run as two groups that alternate between a
 * memory phase and a matrix phase, half a K tile apart ("ping-pong").
 *
 * A SIMD hosts one wave of each group (waves w and w + 4).  For K tile u a wave first runs
 *   Mem(u): fetch ALL of its fragments of tile u from LDS into registers, request the tile STAGES-1
 *           ahead from global memory, wait for its own chunks of tile u+1 (zeroing ragged k ends),
 * then, after a barrier,
 *   Cmp(u): nothing but the tile's MFMAs, at raised priority,
 * and another barrier.  Group 1 enters the loop one barrier later than group 0, so whenever one wave
 * of a SIMD is in Cmp the other is in Mem: the matrix unit always has a wave that issues nothing but
 * MFMAs, and the LDS reads and load issue of the other wave hide behind them instead of delaying
 * every wave's first MFMA after a common barrier.
 *
 * Ring discipline (phase p = interval between consecutive barriers; group 0 runs Mem(u) in phase 2u,
 * group 1 in phase 2u+1):
 *   - tile v is first read in phase 2v; every wave has waited for its own chunks of tile v in its
 *     Mem(v-1), i.e. by the barrier that ends phase 2v-1 (tile 0: before the first barrier);
 *   - the request issued in Mem(u) overwrites the slot of tile u-1, which both groups finished
 *     reading (LDS counter waited) by the barrier that ends phase 2u-1.
 * ------------------------------------------------------------------------------------------- */
#if !defined(HAP_PP_PRIO)
#define HAP_PP_PRIO 1
#endif
constexpr bool kPingPongPrio = HAP_PP_PRIO != 0;    // raise the wave's priority for its matrix phase
#if !defined(HAP_PP_DEFER)
#define HAP_PP_DEFER 1
#endif
constexpr bool kPingPongDefer = HAP_PP_DEFER != 0;  // group 0 awaits the next tile behind its MFMAs instead of in its memory phase
template <int N> __device__ __forceinline__ void wait_vmcnt() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

/* Fragment addressing of the ping-pong kernel: every address is (a register computed once before the K loop) +
 * (a compile-time offset in the instruction), so fetching a tile's fragments costs no vector ALU work at all - the
 * other wave of the SIMD owns the vector ALU port with its MFMAs meanwhile.  The ring lies at byte `ring` of LDS and
 * is wider than the 16-bit offset field reaches, hence one base register per 64 KiB of it. */
template <bool KC, int ROWS, int BK, int NBLK, int NH>
struct PinnedFrag {
  static constexpr int KK = BK / 16;
  static constexpr int CPR = (KC ? BK : ROWS) / 8;
  static constexpr int ROWB = CPR * 16;
  static constexpr int NB = KC ? KK : NBLK;      // K-contiguous: one base per k-step (the swizzle XOR); M/N-contiguous: one per 32-column block
  unsigned base[NB][NH];
  __device__ __forceinline__ void init(int lane, int wave_mn, unsigned ring) {
    FragReader<KC, ROWS, BK, NBLK> fr;
    fr.init(lane, wave_mn);
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int h = 0; h < NH; ++h) base[b][h] = (KC ? (fr.at[0] ^ (unsigned)(b << 5)) : fr.at[b]) + ring + (unsigned)h * 65536u;
  }
  /* Fragment of 32-row block BLK at k-step KKI of the tile that starts OFF bytes into the ring. */
  template <int OFF, int BLK, int KKI>
  __device__ __forceinline__ bf16x8_t read() const {
    constexpr int H = OFF >> 16, LO = OFF & 0xffff;
    if constexpr (KC) {
      static_assert(LO + BLK * 32 * ROWB < 65536, "offset field");
      return lds_read_b128_at<LO + BLK * 32 * ROWB>(base[KKI][H]);
    } else {
      static_assert(LO + KKI * 16 * ROWB + 4 * ROWB < 65536, "offset field");
      return lds_read_tr_pair_at<LO + KKI * 16 * ROWB, LO + KKI * 16 * ROWB + 4 * ROWB>(base[BLK][H]);
    }
  }
};

template <typename TC, bool AKC, bool BKC, int BM, int BN, int BK, int WGM, int WGN, int STAGES>
__global__ __launch_bounds__(64 * WGM * WGN) void gemm_pp_kernel(const GemmArgs args) {
  typedef __bf16 T;
  constexpr int NT = 64 * WGM * WGN;
  constexpr int NW = WGM * WGN;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2, STAGE_BYTES = A_BYTES + B_BYTES;
  constexpr int NH = (STAGES * STAGE_BYTES + 65535) / 65536;
  typedef DmaLoader<AKC, BM, BK, NT> LA;
  typedef DmaLoader<BKC, BN, BK, NT> LB;
  constexpr int LPT = LA::CPT + LB::CPT;            // loads per thread and tile
  constexpr int KK = BK / 16;
  static_assert(STAGES >= 2 && STAGES <= 5 && (STAGES - 1) * LPT < 64, "ring depth");

  extern __shared__ __attribute__((aligned(1024))) char smem[];
  HAP_EXP_STAMP(0);

  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
  const int wm0 = (wave / WGN) * WTM, wn0 = (wave % WGN) * WTN;
  const bool late_group = wave >= NW / 2;            // waves w and w + NW/2 share a SIMD
  const BlockPos bp = block_pos(args);
  const int ksplit = args.ksplit, split = bp.split, tm = bp.tm, tn = bp.tn;
  const int m0 = tm * BM, n0 = tn * BN;
  const GroupView gv = group_view(args, bp.grp);
  const int m_lim = args.skewM + gv.M, n_lim = args.skewN + args.N;
  if (args.ragged == 1 && (gv.M == 0 || m0 >= m_lim)) return;
  const int all_tiles = gv.k >= 0 ? (args.skewK + gv.k + BK - 1 >= BK ? (args.skewK + gv.k + BK - 1) / BK : 1) : args.ntiles;

  LA la; LB lb;
  la.init(tid, m0, AKC ? args.skewM : 0, m_lim, args.lda);
  lb.init(tid, n0, BKC ? args.skewN : 0, n_lim, args.ldb);
  PinnedFrag<AKC, BM, BK, TM, NH> fra;
  PinnedFrag<BKC, BN, BK, TN, NH> frb;
  fra.init(lane, wm0, lds_addr(smem));
  frb.init(lane, wn0, lds_addr(smem));

  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

  const int first = (int)((long long)all_tiles * split / ksplit);
  const int ntiles = (int)((long long)all_tiles * (split + 1) / ksplit) - first;
  int seg0 = 0, skip = first;
  while (seg0 + 1 < args.nseg) {
    const int in_seg = (args.skewK + args.seg[seg0].k + BK - 1) / BK;
    if (skip < in_seg) break;
    skip -= in_seg;
    seg0 = uni(seg0 + 1);
  }
  // request cursor (runs STAGES-1 tiles ahead) and landing cursor (the next tile whose arrival is awaited); tile v lives in slot v % STAGES
  int pseg = seg0, pk0 = skip * BK, pkend = uni(args.skewK + (gv.k >= 0 ? gv.k : args.seg[seg0].k)), issued = 0;
  __amdgpu_buffer_rsrc_t ra = make_rsrc(static_cast<const char*>(args.seg[seg0].a) + gv.oa, args.seg[seg0].a_bytes);
  __amdgpu_buffer_rsrc_t rb = make_rsrc(static_cast<const char*>(args.seg[seg0].b) + gv.ob, args.seg[seg0].b_bytes);
  int lseg = seg0, lk0 = pk0, lkend = pkend;

  auto request = [&](auto slot_tag) {
    constexpr int SLOT = decltype(slot_tag)::value;
    char* pa = smem + SLOT * STAGE_BYTES;
    char* pb = pa + A_BYTES;
    const unsigned soa = LA::tile_offset(pk0, args.skewK, args.lda), sob = LB::tile_offset(pk0, args.skewK, args.ldb);
    if (pk0 < args.skewK || pk0 + BK > pkend) {      // first / last tile of a segment: validity per chunk
      la.issue_edge(ra, pa, tid, soa, pk0, args.skewK, pkend);
      lb.issue_edge(rb, pb, tid, sob, pk0, args.skewK, pkend);
    } else {
      la.issue(ra, pa, wave << 6, soa);          // (issue() needs only the wave's first thread id, here already a scalar)
      lb.issue(rb, pb, wave << 6, sob);
    }
    pk0 += BK;
    ++issued;
    if (pk0 >= pkend && pseg + 1 < args.nseg) {
      pseg = uni(pseg + 1);
      pk0 = 0;
      pkend = uni(args.skewK + args.seg[pseg].k);
      ra = make_rsrc(static_cast<const char*>(args.seg[pseg].a) + gv.oa, args.seg[pseg].a_bytes);
      rb = make_rsrc(static_cast<const char*>(args.seg[pseg].b) + gv.ob, args.seg[pseg].b_bytes);
    }
  };
  // Waits until at most `newer` tiles requested after the awaited one are still in flight, then zeroes the awaited
  // tile's k elements outside the logical range (own chunks only) and moves the landing cursor on.
  auto land = [&](auto slot_tag, int newer) {
    constexpr int SLOT = decltype(slot_tag)::value;
    if (newer >= STAGES - 2) wait_vmcnt<(STAGES - 2) * LPT>();          // the steady state
    else if (STAGES > 3 && newer == 2) wait_vmcnt<(STAGES > 3 ? 2 : 0) * LPT>();
    else if (STAGES > 2 && newer == 1) wait_vmcnt<(STAGES > 2 ? 1 : 0) * LPT>();
    else wait_vmcnt<0>();
    if (lk0 < args.skewK || lk0 + BK > lkend) {
      char* sa = smem + SLOT * STAGE_BYTES;
      la.fixup(sa, tid, lk0, args.skewK, lkend);
      lb.fixup(sa + A_BYTES, tid, lk0, args.skewK, lkend);
    }
    lk0 += BK;
    if (lk0 >= lkend && lseg + 1 < args.nseg) { lseg = uni(lseg + 1); lk0 = 0; lkend = uni(args.skewK + args.seg[lseg].k); }
  };

  static_for<STAGES - 1>([&](auto s) { if (s < ntiles) request(s); });
  if (ntiles > 0) land(std::integral_constant<int, 0>(), issued - 1);
  __builtin_amdgcn_s_barrier();                      // tile 0 is in LDS for everybody
  HAP_EXP_STAMP(1);
  if (late_group) __builtin_amdgcn_s_barrier();      // group 1 runs one phase behind group 0

  // one K tile whose ring slot is known at compile time
  // FAST: the tile requested and the tile awaited are interior tiles of their segments and both cursors stay inside their
  // segments, a request is due and a tile follows - no per-chunk validity, no fix-up, no data-dependent branch at all.
  // (The two forms share ONE copy of the matrix phase: two copies of the tile body made the compiler shuffle the 128
  // accumulator registers between them through scratch memory.)
  auto tile = [&](auto slot_tag, const bool fast, int u) __attribute__((always_inline)) {
    constexpr int SLOT = decltype(slot_tag)::value;
    constexpr int PREV = (SLOT + STAGES - 1) % STAGES, NEXT = (SLOT + 1) % STAGES;
    // ---- Mem(u): all fragments of the tile, the request STAGES-1 tiles ahead (into the slot of tile u-1), arrival of tile u+1
    bf16x8_t fa[KK][TM], fb[KK][TN];
    static_for<KK>([&](auto kk) {
      static_for<TN>([&](auto j) { fb[kk][j] = frb.template read<SLOT * STAGE_BYTES + A_BYTES, j, kk>(); });
      static_for<TM>([&](auto i) { fa[kk][i] = fra.template read<SLOT * STAGE_BYTES, i, kk>(); });
    });
    if (fast) {
      char* pa = smem + PREV * STAGE_BYTES;
      la.issue(ra, pa, wave << 6, LA::tile_offset(pk0, args.skewK, args.lda));
      lb.issue(rb, pa + A_BYTES, wave << 6, LB::tile_offset(pk0, args.skewK, args.ldb));
      pk0 += BK;
      ++issued;
    } else {
      if (issued < ntiles) request(std::integral_constant<int, PREV>());
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // this wave's reads of tile u are done (its slot is refilled two phases on)
    if (fast) {
      // Tile u+1 is first read by group 0, in its memory phase behind the NEXT barrier but one (group 0's matrix phase lies
      // between).  Group 1 is one phase behind: the barrier that ends this memory phase is already the last one before that read,
      // so it waits here; group 0 has its whole matrix phase to go and waits behind its MFMAs.
      if (late_group || !kPingPongDefer) wait_vmcnt<(STAGES - 2) * LPT>();
      lk0 += BK;
    } else {
      if (u + 1 < ntiles) land(std::integral_constant<int, NEXT>(), issued - (u + 2));
    }
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    // ---- Cmp(u)
    if (kPingPongPrio) __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
#pragma unroll
      for (int x = 0; x < TM * TN; ++x) acc[x / TN][x % TN] = mfma(fb[kk][x % TN], fa[kk][x / TN], acc[x / TN][x % TN]);
    if (kPingPongPrio) __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
    // group 0 awaits its share of tile u+1 here: one more phase for the loads to arrive, and the wait is out of the memory phase
    // that group 1's MFMAs run against
    if (kPingPongDefer && fast && !late_group) wait_vmcnt<(STAGES - 2) * LPT>();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
  for (int u0 = 0; u0 < ntiles; u0 += STAGES) {
    const bool fast = issued + STAGES <= ntiles && pk0 >= args.skewK && pk0 + STAGES * BK < pkend &&
                      lk0 >= args.skewK && lk0 + STAGES * BK < lkend;
    static_for<STAGES>([&](auto s) { if (fast || u0 + s < ntiles) tile(s, fast, u0 + s); });
  }
  if (!late_group) __builtin_amdgcn_s_barrier();     // group 1's last matrix phase: after it nobody reads the ring any more
  HAP_EXP_STAMP(2);

  if (ksplit > 1) {
    const GemmArgs pa = partial_outputs(args, bp, BM, BN);
    epilogue_transposed<T, float, TM, TN>(pa, acc, wm0, wn0, lane, smem + wave * (32 * (TN * 32 * 4 + 16)));
    return;
  }
  epilogue_transposed<T, TC, TM, TN>(group_outputs(args, gv, bp.grp), acc, m0 + wm0, n0 + wn0, lane, smem + wave * (32 * (TN * 32 * (int)sizeof(TC) + 16)));
  HAP_EXP_STAMP(3);
}

/* ---------------------------------------------------------------------------------------------
 * bf16 kernel for short contractions: 128 x 128 tiles, four waves, three workgroups per compute unit.
 *
 * Over a few hundred k a workgroup spends longer in its prologue (the first tiles' way from memory) and epilogue (activation, stores) than
 * in its K loop, and a 256 x 256 tile, which has its compute unit to itself, overlaps neither with anything.  Here a K step of 32 in a
 * three-stage ring takes 48 KB of LDS and the waves at most 168 registers, so that three independent workgroups share a compute unit and
 * one's ends lie behind the others' MFMAs.  Bound: the operands' way from L2 (a tile of this size fetches twice what a 256-tile does per
 * MFMA), which is why long contractions go elsewhere.  Two workgroups of 256 x 128 per compute unit, tried for the same end, fetch less and
 * measured 5 to 10 % slower than three of 128 x 128 wherever either gained (50432 x 1024 over 315: 98 against 91 us, 74 before).
 * Four per compute unit (128 registers) spill in the epilogue: 90 there, but 74 against 60 without GeLU.
 *
 * A tile's loads go out behind the previous tile's fragment reads, two tiles ahead of their use; fragments are fetched whole, by hand-
 * ordered reads, and one barrier per tile separates a slot's last reader from its next request.
 * ------------------------------------------------------------------------------------------- */
template <typename TC, bool AKC, bool BKC>
__global__ __launch_bounds__(256, 3) void gemm_trio_kernel(const GemmArgs args) {
  typedef __bf16 T;
  constexpr int BM = 128, BN = 128, BK = 32, STAGES = 3, WGM = 2, WGN = 2, NT = 256;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2, STAGE_BYTES = A_BYTES + B_BYTES;
  typedef DmaLoader<AKC, BM, BK, NT> LA;
  typedef DmaLoader<BKC, BN, BK, NT> LB;
  constexpr int LPT = LA::CPT + LB::CPT;            // loads per thread and tile
  constexpr int KK = BK / 16;

  extern __shared__ __attribute__((aligned(1024))) char smem[];

  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
  const int wm0 = (wave / WGN) * WTM, wn0 = (wave % WGN) * WTN;
  const BlockPos bp = block_pos(args);
  const int m0 = bp.tm * BM, n0 = bp.tn * BN;
  const GroupView gv = group_view(args, bp.grp);
  const int m_lim = args.skewM + gv.M, n_lim = args.skewN + args.N;
  if (args.ragged == 1 && (gv.M == 0 || m0 >= m_lim)) return;
  const int all_tiles = gv.k >= 0 ? (args.skewK + gv.k + BK - 1 >= BK ? (args.skewK + gv.k + BK - 1) / BK : 1) : args.ntiles;

  LA la; LB lb;
  la.init(tid, m0, AKC ? args.skewM : 0, m_lim, args.lda);
  lb.init(tid, n0, BKC ? args.skewN : 0, n_lim, args.ldb);
  PinnedFrag<AKC, BM, BK, TM, 1> fra;
  PinnedFrag<BKC, BN, BK, TN, 1> frb;
  fra.init(lane, wm0, lds_addr(smem));
  frb.init(lane, wn0, lds_addr(smem));

  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

  const int ntiles = all_tiles;                      // (K is not split over workgroups)
  int pseg = 0, pk0 = 0, pkend = uni(args.skewK + (gv.k >= 0 ? gv.k : args.seg[0].k)), issued = 0;
  __amdgpu_buffer_rsrc_t ra = make_rsrc(static_cast<const char*>(args.seg[0].a) + gv.oa, args.seg[0].a_bytes);
  __amdgpu_buffer_rsrc_t rb = make_rsrc(static_cast<const char*>(args.seg[0].b) + gv.ob, args.seg[0].b_bytes);
  int lseg = 0, lk0 = 0, lkend = pkend;

  auto request = [&](auto slot_tag) {
    constexpr int SLOT = decltype(slot_tag)::value;
    char* pa = smem + SLOT * STAGE_BYTES;
    char* pb = pa + A_BYTES;
    const unsigned soa = LA::tile_offset(pk0, args.skewK, args.lda), sob = LB::tile_offset(pk0, args.skewK, args.ldb);
    if (pk0 < args.skewK || pk0 + BK > pkend) {      // first / last tile of a segment: validity per chunk
      la.issue_edge(ra, pa, tid, soa, pk0, args.skewK, pkend);
      lb.issue_edge(rb, pb, tid, sob, pk0, args.skewK, pkend);
    } else {
      la.issue(ra, pa, wave << 6, soa);
      lb.issue(rb, pb, wave << 6, sob);
    }
    pk0 += BK;
    ++issued;
    if (pk0 >= pkend && pseg + 1 < args.nseg) {
      pseg = uni(pseg + 1);
      pk0 = 0;
      pkend = uni(args.skewK + args.seg[pseg].k);
      ra = make_rsrc(static_cast<const char*>(args.seg[pseg].a) + gv.oa, args.seg[pseg].a_bytes);
      rb = make_rsrc(static_cast<const char*>(args.seg[pseg].b) + gv.ob, args.seg[pseg].b_bytes);
    }
  };
  auto land = [&](auto slot_tag, int newer) {
    constexpr int SLOT = decltype(slot_tag)::value;
    if (STAGES > 2 && newer >= 1) wait_vmcnt<(STAGES - 2) * LPT>();
    else wait_vmcnt<0>();
    if (lk0 < args.skewK || lk0 + BK > lkend) {
      char* sa = smem + SLOT * STAGE_BYTES;
      la.fixup(sa, tid, lk0, args.skewK, lkend);
      lb.fixup(sa + A_BYTES, tid, lk0, args.skewK, lkend);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    lk0 += BK;
    if (lk0 >= lkend && lseg + 1 < args.nseg) { lseg = uni(lseg + 1); lk0 = 0; lkend = uni(args.skewK + args.seg[lseg].k); }
  };

  static_for<STAGES - 1>([&](auto s) { if (s < ntiles) request(s); });
  if (ntiles > 0) land(std::integral_constant<int, 0>(), issued - 1);
  __builtin_amdgcn_s_barrier();                      // tile 0 is in LDS for everybody

  auto tile = [&](auto slot_tag, const bool fast, int u) __attribute__((always_inline)) {
    constexpr int SLOT = decltype(slot_tag)::value;
    constexpr int PREV = (SLOT + STAGES - 1) % STAGES, NEXT = (SLOT + 1) % STAGES;
    bf16x8_t fa[KK][TM], fb[KK][TN];
    static_for<KK>([&](auto kk) {
      static_for<TN>([&](auto j) { fb[kk][j] = frb.template read<SLOT * STAGE_BYTES + A_BYTES, j, kk>(); });
      static_for<TM>([&](auto i) { fa[kk][i] = fra.template read<SLOT * STAGE_BYTES, i, kk>(); });
    });
    if (fast) {
      char* pa = smem + PREV * STAGE_BYTES;
      la.issue(ra, pa, wave << 6, LA::tile_offset(pk0, args.skewK, args.lda));
      lb.issue(rb, pa + A_BYTES, wave << 6, LB::tile_offset(pk0, args.skewK, args.ldb));
      pk0 += BK;
      ++issued;
    } else {
      if (issued < ntiles) request(std::integral_constant<int, PREV>());
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
#pragma unroll
      for (int x = 0; x < TM * TN; ++x) acc[x / TN][x % TN] = mfma(fb[kk][x % TN], fa[kk][x / TN], acc[x / TN][x % TN]);
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
    if (fast) {
      wait_vmcnt<(STAGES - 2) * LPT>();
      lk0 += BK;
    } else {
      if (u + 1 < ntiles) land(std::integral_constant<int, NEXT>(), issued - (u + 2));
    }
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
  for (int u0 = 0; u0 < ntiles; u0 += STAGES) {
    const bool fast = issued + STAGES <= ntiles && pk0 >= args.skewK && pk0 + STAGES * BK < pkend &&
                      lk0 >= args.skewK && lk0 + STAGES * BK < lkend;
    static_for<STAGES>([&](auto s) { if (fast || u0 + s < ntiles) tile(s, fast, u0 + s); });
  }

  epilogue_transposed<T, TC, TM, TN>(group_outputs(args, gv, bp.grp), acc, m0 + wm0, n0 + wn0, lane, smem + wave * (32 * (TN * 32 * (int)sizeof(TC) + 16)));
}

/* ---------------------------------------------------------------------------------------------
 * bf16 kernel for outputs of few 128 x 128 tiles: two wave groups share ONE tile, each contracts its half of the workgroup's K
 * tiles in a ring of its own, and the halves meet in LDS before the epilogue, of which each group does one half.
 *
 * Such outputs (at most one tile per compute unit) need the contraction split to put two waves on every SIMD.  Split over two
 * workgroups it costs the fp32 partial tiles and a dependent reduction launch; here the split stays inside the compute unit.
 *
 * The groups alternate between a memory phase and a matrix phase as in gemm_pp_kernel (waves w and w + 4 share a SIMD; group 1 runs
 * one barrier behind): in lockstep, with one barrier per K tile for all eight waves, both waves of a SIMD wait for LDS and then both
 * want the matrix unit (1.06 us per pair of K tiles at 248 workgroups against 0.68 for two independent workgroups).
 * A group's tile u is read in its Mem(u); from the barrier behind it on the slot is free, and the request for tile u + 2 goes out
 * between the MFMAs of Cmp(u).  It has Cmp(u), Mem(u+1), Cmp(u+1) to arrive: at the end of Cmp(u+1) everything but the newest
 * request has landed.  Requests past the group's last tile are issued out of range (no memory access, zeros), so that the count
 * of loads in flight is always the same.
 * ------------------------------------------------------------------------------------------- */
template <typename TC, bool AKC, bool BKC>
__global__ __launch_bounds__(512) void gemm_kpair_kernel(const GemmArgs args) {
  typedef __bf16 T;
  constexpr int BM = 128, BN = 128, BK = 64, NT = 256, TM = 2, TN = 2, KK = BK / 16;
  constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2, STAGE_BYTES = A_BYTES + B_BYTES;
  typedef DmaLoader<AKC, BM, BK, NT> LA;
  typedef DmaLoader<BKC, BN, BK, NT> LB;
  constexpr int LPT = LA::CPT + LB::CPT;

  extern __shared__ __attribute__((aligned(1024))) char smem_all[];

  const int kg = uni((int)threadIdx.x / NT);         // wave group
  const int tid = threadIdx.x - kg * NT, lane = tid & 63, wave = uni(tid >> 6);
  char* const smem = smem_all + kg * (2 * STAGE_BYTES);
  const int wm0 = (wave >> 1) * 64, wn0 = (wave & 1) * 64;
  const BlockPos bp = block_pos(args);
  const int ksplit = args.ksplit, tm = bp.tm, tn = bp.tn;
  const int m0 = tm * BM, n0 = tn * BN;
  const GroupView gv = group_view(args, bp.grp);
  const int m_lim = args.skewM + gv.M, n_lim = args.skewN + args.N;
  if (args.ragged == 1 && (gv.M == 0 || m0 >= m_lim)) return;
  const int all_tiles = gv.k >= 0 ? (args.skewK + gv.k + BK - 1 >= BK ? (args.skewK + gv.k + BK - 1) / BK : 1) : args.ntiles;

  LA la; LB lb;
  la.init(tid, m0, AKC ? args.skewM : 0, m_lim, args.lda);
  lb.init(tid, n0, BKC ? args.skewN : 0, n_lim, args.ldb);
  PinnedFrag<AKC, BM, BK, TM, 1> fra;
  PinnedFrag<BKC, BN, BK, TN, 1> frb;
  fra.init(lane, wm0, lds_addr(smem));
  frb.init(lane, wn0, lds_addr(smem));

  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

  // the K tiles of this group: the first or the second half of the workgroup's (group 1 takes the odd one, so it never has fewer)
  const int first_of_both = (int)((long long)all_tiles * bp.split / ksplit);
  const int both = (int)((long long)all_tiles * (bp.split + 1) / ksplit) - first_of_both;
  const int steps = both - both / 2;
  const int first = first_of_both + (kg ? both / 2 : 0), ntiles = kg ? steps : both / 2;
  int seg0 = 0, skip = first;
  while (seg0 + 1 < args.nseg) {
    const int in_seg = (args.skewK + args.seg[seg0].k + BK - 1) / BK;
    if (skip < in_seg) break;
    skip -= in_seg;
    seg0 = uni(seg0 + 1);
  }
  int pseg = seg0, pk0 = skip * BK, pkend = uni(args.skewK + (gv.k >= 0 ? gv.k : args.seg[seg0].k)), prepared = 0;
  __amdgpu_buffer_rsrc_t ra = make_rsrc(static_cast<const char*>(args.seg[seg0].a) + gv.oa, args.seg[seg0].a_bytes);
  __amdgpu_buffer_rsrc_t rb = make_rsrc(static_cast<const char*>(args.seg[seg0].b) + gv.ob, args.seg[seg0].b_bytes);
  int lseg = seg0, lk0 = pk0, lkend = pkend;

  // offsets of the next tile to request
  unsigned va[LA::CPT], vb[LB::CPT], soa = 0, sob = 0;
  auto prepare = [&]() {
    if (prepared >= ntiles) {
#pragma unroll
      for (int i = 0; i < LA::CPT; ++i) va[i] = kOobOffset;
#pragma unroll
      for (int i = 0; i < LB::CPT; ++i) vb[i] = kOobOffset;
      soa = 0; sob = 0;
      return;
    }
    if (prepared > 0) {
      pk0 += BK;
      if (pk0 >= pkend && pseg + 1 < args.nseg) {
        pseg = uni(pseg + 1);
        pk0 = 0;
        pkend = uni(args.skewK + args.seg[pseg].k);
        ra = make_rsrc(static_cast<const char*>(args.seg[pseg].a) + gv.oa, args.seg[pseg].a_bytes);
        rb = make_rsrc(static_cast<const char*>(args.seg[pseg].b) + gv.ob, args.seg[pseg].b_bytes);
      }
    }
    ++prepared;
    soa = LA::tile_offset(pk0, args.skewK, args.lda); sob = LB::tile_offset(pk0, args.skewK, args.ldb);
    if (pk0 < args.skewK || pk0 + BK > pkend) {      // first / last tile of a segment: validity per chunk
      la.edge_offsets(va, tid, soa, pk0, args.skewK, pkend);
      lb.edge_offsets(vb, tid, sob, pk0, args.skewK, pkend);
      soa = 0; sob = 0;
    } else {
#pragma unroll
      for (int i = 0; i < LA::CPT; ++i) va[i] = la.base[i];
#pragma unroll
      for (int i = 0; i < LB::CPT; ++i) vb[i] = lb.base[i];
    }
  };
  auto request = [&](int slot, int i) {              // load i of LPT
    char* const pa = smem + slot * STAGE_BYTES + (wave << 6) * 16;
    if (i < LA::CPT) dma16(ra, pa + i * NT * 16, va[i], soa);
    else dma16(rb, pa + A_BYTES + (i - LA::CPT) * NT * 16, vb[i - LA::CPT], sob);
  };
  // all but the newest request have landed: zero the awaited tile's k elements outside the logical range (own chunks only)
  auto land = [&](int slot) {
    wait_vmcnt<LPT>();
    if (lk0 < args.skewK || lk0 + BK > lkend) {
      char* const sa = smem + slot * STAGE_BYTES;
      la.fixup(sa, tid, lk0, args.skewK, lkend);
      lb.fixup(sa + A_BYTES, tid, lk0, args.skewK, lkend);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    lk0 += BK;
    if (lk0 >= lkend && lseg + 1 < args.nseg) { lseg = uni(lseg + 1); lk0 = 0; lkend = uni(args.skewK + args.seg[lseg].k); }
  };

#pragma unroll
  for (int u = 0; u < 2; ++u) {
    prepare();
#pragma unroll
    for (int i = 0; i < LPT; ++i) request(u, i);
  }
  if (ntiles > 0) land(0);
  __builtin_amdgcn_s_barrier();                      // the first tiles are in LDS
  if (kg) __builtin_amdgcn_s_barrier();              // group 1 runs one phase behind group 0

  auto tile = [&](auto slot_tag, int u) __attribute__((always_inline)) {
    constexpr int SLOT = decltype(slot_tag)::value;
    // ---- Mem(u): all fragments of the tile; where the request of tile u + 2 goes
    bf16x8_t fa[KK][TM], fb[KK][TN];
    static_for<KK>([&](auto kk) {
      static_for<TN>([&](auto j) { fb[kk][j] = frb.template read<SLOT * STAGE_BYTES + A_BYTES, j, kk>(); });
      static_for<TM>([&](auto i) { fa[kk][i] = fra.template read<SLOT * STAGE_BYTES, i, kk>(); });
    });
    prepare();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // this wave's reads of tile u are done
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    // ---- Cmp(u)
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
#pragma unroll
      for (int x = 0; x < TM * TN; ++x) {
        acc[x / TN][x % TN] = mfma(fb[kk][x % TN], fa[kk][x / TN], acc[x / TN][x % TN]);
        const int at = kk * TM * TN + x;
        if (at % 2 == 1 && at / 2 < LPT) {
          __builtin_amdgcn_sched_barrier(0);
          request(SLOT, at / 2);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
    if (u + 1 < ntiles) land(1 - SLOT);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
  static_assert(LPT <= KK * TM * TN / 2, "one request behind every second MFMA");
  for (int u = 0; u < ntiles; u += 2) {
    tile(std::integral_constant<int, 0>(), u);
    if (u + 1 < ntiles) tile(std::integral_constant<int, 1>(), u + 1);
  }
  wait_vmcnt<0>();                                   // (the out-of-range requests still write zeros into the ring)
  if (!kg) {
    __builtin_amdgcn_s_barrier();                    // group 1's last matrix phase
    for (int t = ntiles; t < steps; ++t) { __builtin_amdgcn_s_barrier(); __builtin_amdgcn_s_barrier(); }   // its tile more than group 0 has
  }
  __syncthreads();

  // Each group keeps row block `kg` of its waves' tiles and hands the other one over: per register quad the 256 threads write
  // consecutive 16-byte chunks, 32 KB per group.
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  f32x4* const handed = reinterpret_cast<f32x4*>(smem_all) + (1 - kg) * (TN * 4 * NT);
  const f32x4* const received = reinterpret_cast<f32x4*>(smem_all) + kg * (TN * 4 * NT);
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      f32x4 v;
#pragma unroll
      for (int x = 0; x < 4; ++x) v[x] = kg ? acc[0][j][q * 4 + x] : acc[1][j][q * 4 + x];
      handed[(j * 4 + q) * NT + tid] = v;
    }
  __syncthreads();
  f32x16_t sum[1][TN];
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 v = received[(j * 4 + q) * NT + tid];
#pragma unroll
      for (int x = 0; x < 4; ++x) sum[0][j][q * 4 + x] = (kg ? acc[1][j][q * 4 + x] : acc[0][j][q * 4 + x]) + v[x];
    }
  __syncthreads();                                   // the exchange area becomes store patches
  const int wm = wm0 + kg * 32;
  char* const patch = smem_all + (kg * 4 + wave) * (32 * (TN * 32 * 4 + 16));
  if (ksplit > 1) {
    const GemmArgs pa = partial_outputs(args, bp, BM, BN);
    epilogue_transposed<T, float, 1, TN>(pa, sum, wm, wn0, lane, patch);
    return;
  }
  epilogue_transposed<T, TC, 1, TN>(group_outputs(args, gv, bp.grp), sum, m0 + wm, n0 + wn0, lane, patch);
}

/* Stores four consecutive columns n .. n + 3 of output row m (n may precede the first column or run past the last one) as the one-pass
 * epilogues would: bias, pre-activation copy, activation or activation backward, accumulation, conversion.  whole: all four columns exist
 * and every tensor's four lie on a boundary of their size, so that each is one access; else element by element. */
template <typename T, typename TC>
__device__ __forceinline__ void store_quad(const GemmArgs& args, int m, int n, const float (&sum)[4], bool whole) {
  typedef TC quad_t __attribute__((ext_vector_type(4)));
  TC* const C = static_cast<TC*>(args.c) + (long long)m * args.ldc + n;
  TC* const P = args.preact ? static_cast<TC*>(args.preact) + (long long)m * args.ldp + n : nullptr;
  const T* const bias = args.bias ? static_cast<const T*>(args.bias) + n : nullptr;
  const TC* const dpre = args.dact_preact ? static_cast<const TC*>(args.dact_preact) + (long long)m * args.ldd + n : nullptr;
  if (whole) {
    quad_t d, old, pre, out;
    if (dpre) d = *reinterpret_cast<const quad_t*>(dpre);
    if (args.accumulate) old = *reinterpret_cast<const quad_t*>(C);
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      float v = sum[x];
      if (bias) v += load_s<T>(bias + x);
      pre[x] = (TC)v;
      if (args.act == HAP_ACT_GELU_ERF) v = gelu_erf((float)(TC)v);     // the activation sees the value as stored
      if (dpre) v *= gelu_erf_grad((float)d[x]);
      if (args.accumulate) v += (float)old[x];
      out[x] = (TC)v;
    }
    if (P) *reinterpret_cast<quad_t*>(P) = pre;
    *reinterpret_cast<quad_t*>(C) = out;
    return;
  }
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    if (n + x < 0 || n + x >= args.N) continue;
    float v = sum[x];
    if (bias) v += load_s<T>(bias + x);
    if (P) store_c<TC>(P + x, v);
    if (args.act == HAP_ACT_GELU_ERF) v = gelu_erf((float)(TC)v);
    if (dpre) v *= gelu_erf_grad(load_s<TC>(dpre + x));
    if (args.accumulate) v += load_s<TC>(C + x);
    store_c<TC>(C + x, v);
  }
}

/* Whether the quad at row m, column n is whole (see store_quad). */
template <typename TC>
__device__ __forceinline__ bool quad_is_whole(const GemmArgs& args, int m, int n) {
  uintptr_t at = (uintptr_t)(static_cast<const TC*>(args.c) + (long long)m * args.ldc + n);
  if (args.preact) at |= (uintptr_t)(static_cast<const TC*>(args.preact) + (long long)m * args.ldp + n);
  if (args.dact_preact) at |= (uintptr_t)(static_cast<const TC*>(args.dact_preact) + (long long)m * args.ldd + n);
  return n >= 0 && n + 4 <= args.N && at % (4 * sizeof(TC)) == 0;
}

/* Whether all quads at multiples of four columns are. */
template <typename TC>
__device__ __forceinline__ bool all_quads_are_whole(const GemmArgs& args) {
  uintptr_t at = (uintptr_t)args.c | (uintptr_t)args.ldc * sizeof(TC);
  if (args.preact) at |= (uintptr_t)args.preact | (uintptr_t)args.ldp * sizeof(TC);
  if (args.dact_preact) at |= (uintptr_t)args.dact_preact | (uintptr_t)args.ldd * sizeof(TC);
  return args.N % 4 == 0 && at % (4 * sizeof(TC)) == 0;
}

/* ---------------------------------------------------------------------------------------------
 * bf16 kernel for the smallest outputs: eight waves share one BM x 64 tile, each contracts an eighth of K with a ring of its own.
 *
 * Bound: latency.  A product of a few hundred rows has a few dozen 128-tiles; spread over the chip by splitting K over workgroups it
 * pays for fp32 partial tiles and a dependent reduction launch, longer together than the product.  Tiles of 32 or 64 rows give the chip
 * enough workgroups without one, and with the contraction cut in eight a wave's share is a handful of steps, most of whose loads are in
 * flight at once.  The rings are private to the waves, so nothing waits at a barrier before the partial sums meet in LDS.
 * ------------------------------------------------------------------------------------------- */
template <int BM> constexpr int kSmallStages = BM == 32 ? 3 : 2;
template <int BM> constexpr int kSmallLds = 8 * kSmallStages<BM> * (BM + 64) * 32 * 2;

template <typename TC, bool AKC, bool BKC, int BM>
__global__ __launch_bounds__(512) void gemm_small_kernel(const GemmArgs args) {
  typedef __bf16 T;
  constexpr int BN = 64, BK = 32, NW = 8, STAGES = kSmallStages<BM>, KK = BK / 16;
  constexpr int TM = BM / 32, TN = BN / 32;
  constexpr int A_BYTES = BM * BK * 2, STAGE_BYTES = A_BYTES + BN * BK * 2;
  typedef DmaLoader<AKC, BM, BK, 64> LA;
  typedef DmaLoader<BKC, BN, BK, 64> LB;
  constexpr int LPT = LA::CPT + LB::CPT;
  static_assert(STAGES * STAGE_BYTES >= TM * TN * 16 * 64 * 4, "a wave's ring holds its partial sums");

  extern __shared__ __attribute__((aligned(1024))) char smem_all[];
  const int lane = threadIdx.x & 63, wave = uni((int)threadIdx.x >> 6);
  char* const smem = smem_all + wave * (STAGES * STAGE_BYTES);
  const BlockPos bp = block_pos(args);
  const int m0 = bp.tm * BM, n0 = bp.tn * BN;
  const GroupView gv = group_view(args, bp.grp);
  const int m_lim = args.skewM + gv.M, n_lim = args.skewN + args.N;
  if (args.ragged == 1 && (gv.M == 0 || m0 >= m_lim)) return;
  const int all_tiles = gv.k >= 0 ? (args.skewK + gv.k + BK - 1 >= BK ? (args.skewK + gv.k + BK - 1) / BK : 1) : args.ntiles;

  LA la; LB lb;
  la.init(lane, m0, AKC ? args.skewM : 0, m_lim, args.lda);
  lb.init(lane, n0, BKC ? args.skewN : 0, n_lim, args.ldb);
  PinnedFrag<AKC, BM, BK, TM, 1> fra;
  PinnedFrag<BKC, BN, BK, TN, 1> frb;
  fra.init(lane, 0, lds_addr(smem));
  frb.init(lane, 0, lds_addr(smem));

  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

  // this wave's range of the K tiles of all segments laid end to end
  const int first = (int)((long long)all_tiles * wave / NW), ntiles = (int)((long long)all_tiles * (wave + 1) / NW) - first;
  int seg0 = 0, skip = first;
  while (seg0 + 1 < args.nseg) {
    const int in_seg = (args.skewK + args.seg[seg0].k + BK - 1) / BK;
    if (skip < in_seg) break;
    skip -= in_seg;
    seg0 = uni(seg0 + 1);
  }
  int pseg = seg0, pk0 = skip * BK, pkend = uni(args.skewK + (gv.k >= 0 ? gv.k : args.seg[seg0].k)), issued = 0;
  __amdgpu_buffer_rsrc_t ra = make_rsrc(static_cast<const char*>(args.seg[seg0].a) + gv.oa, args.seg[seg0].a_bytes);
  __amdgpu_buffer_rsrc_t rb = make_rsrc(static_cast<const char*>(args.seg[seg0].b) + gv.ob, args.seg[seg0].b_bytes);
  int lseg = seg0, lk0 = pk0, lkend = pkend;
  auto request = [&](auto slot_tag) {
    constexpr int SLOT = decltype(slot_tag)::value;
    char* const pa = smem + SLOT * STAGE_BYTES;
    const unsigned soa = LA::tile_offset(pk0, args.skewK, args.lda), sob = LB::tile_offset(pk0, args.skewK, args.ldb);
    la.issue_edge(ra, pa, lane, soa, pk0, args.skewK, pkend);
    lb.issue_edge(rb, pa + A_BYTES, lane, sob, pk0, args.skewK, pkend);
    pk0 += BK;
    ++issued;
    if (pk0 >= pkend && pseg + 1 < args.nseg) {
      pseg = uni(pseg + 1);
      pk0 = 0;
      pkend = uni(args.skewK + args.seg[pseg].k);
      ra = make_rsrc(static_cast<const char*>(args.seg[pseg].a) + gv.oa, args.seg[pseg].a_bytes);
      rb = make_rsrc(static_cast<const char*>(args.seg[pseg].b) + gv.ob, args.seg[pseg].b_bytes);
    }
  };
  static_for<STAGES>([&](auto s) { if (s < ntiles) request(s); });
  auto tile = [&](auto slot_tag, int u) __attribute__((always_inline)) {
    constexpr int SLOT = decltype(slot_tag)::value;
    const int newer = issued - (u + 1);              // tiles requested after this one: their loads may stay in flight
    if (newer >= 2) wait_vmcnt<2 * LPT>();
    else if (newer == 1) wait_vmcnt<LPT>();
    else wait_vmcnt<0>();
    if (lk0 < args.skewK || lk0 + BK > lkend) {      // zero the k elements outside the segment
      char* const sa = smem + SLOT * STAGE_BYTES;
      la.fixup(sa, lane, lk0, args.skewK, lkend);
      lb.fixup(sa + A_BYTES, lane, lk0, args.skewK, lkend);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    lk0 += BK;
    if (lk0 >= lkend && lseg + 1 < args.nseg) { lseg = uni(lseg + 1); lk0 = 0; lkend = uni(args.skewK + args.seg[lseg].k); }
    bf16x8_t fa[KK][TM], fb[KK][TN];
    static_for<KK>([&](auto kk) {
      static_for<TN>([&](auto j) { fb[kk][j] = frb.template read<SLOT * STAGE_BYTES + A_BYTES, j, kk>(); });
      static_for<TM>([&](auto i) { fa[kk][i] = fra.template read<SLOT * STAGE_BYTES, i, kk>(); });
    });
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    if (issued < ntiles) request(slot_tag);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
#pragma unroll
      for (int x = 0; x < TM * TN; ++x) acc[x / TN][x % TN] = mfma(fb[kk][x % TN], fa[kk][x / TN], acc[x / TN][x % TN]);
    __builtin_amdgcn_sched_barrier(0);
  };
  for (int u0 = 0; u0 < ntiles; u0 += STAGES)
    static_for<STAGES>([&](auto s) { if (u0 + s < ntiles) tile(s, u0 + s); });

  // the partial sums meet: register quad by register quad, 64 lanes next to each other, each wave's in its own ring
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  f32x4* const mine = reinterpret_cast<f32x4*>(smem);
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        f32x4 v;
#pragma unroll
        for (int x = 0; x < 4; ++x) v[x] = acc[i][j][q * 4 + x];
        mine[((i * TN + j) * 4 + q) * 64 + lane] = v;
      }
  __syncthreads();
  const GemmArgs out = group_outputs(args, gv, bp.grp);
#pragma unroll
  for (int b = 0; b < TM * TN * 4 / NW; ++b) {
    const int at = b * NW + wave, i = at / (TN * 4), j = at / 4 % TN, q = at % 4;
    f32x4 t = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int w = 0; w < NW; ++w) t += reinterpret_cast<const f32x4*>(smem_all + w * (STAGES * STAGE_BYTES))[at * 64 + lane];
    const int m = m0 + i * 32 + (lane & 31) - args.skewM, n = n0 + j * 32 + q * 8 + (lane >> 5) * 4 - args.skewN;
    const float v[4] = {t[0], t[1], t[2], t[3]};
    if (m >= 0 && m < out.M && n < out.N && n + 4 > 0) store_quad<T, TC>(out, m, n, v, quad_is_whole<TC>(out, m, n));
  }
}

/* Split-K reduction: sums the ksplit fp32 partial tiles of every output tile and applies what the
 * one-pass epilogue would have (bias, pre-activation copy, activation, accumulation, conversion),
 * storing only the logical rows / columns.  One thread per 4 consecutive columns. */
template <typename T, typename TC, int BM, int BN>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const GemmArgs args_in, int out_tiles) {
  const GemmArgs args = group_outputs(args_in, group_view(args_in, blockIdx.y), blockIdx.y);   // blockIdx.y: group
  constexpr int QPT = BM * BN / 4;                 // column quads per tile
  const long long gid = (long long)blockIdx.x * 256 + threadIdx.x;
  const int tile = (int)(gid / QPT), q = (int)(gid % QPT);
  if (tile >= out_tiles) return;
  int tm, tn;
  if (gridDim.y == 1) tile_of_block(tile, out_tiles, args.tiles_m, args.tiles_n, &tm, &tn);   // the maps of block_pos()
  else tile_of_logical(tile, args.tiles_m, args.tiles_n, &tm, &tn);
  const int r = q / (BN / 4), c4 = (q % (BN / 4)) * 4;
  const int m = tm * BM + r - args.skewM, n = tn * BN + c4 - args.skewN;
  if (m < 0 || m >= args.M || n >= args.N || n + 4 <= 0) return;
  typedef float f32x4_t __attribute__((ext_vector_type(4)));
  f32x4_t sum = {0.0f, 0.0f, 0.0f, 0.0f};
  const float* p = args.partial + ((long long)blockIdx.y * out_tiles + tile) * args.ksplit * (BM * BN) + r * BN + c4;
  for (int s = 0; s < args.ksplit; ++s) sum += *reinterpret_cast<const f32x4_t*>(p + (long long)s * (BM * BN));
  const float v[4] = {sum[0], sum[1], sum[2], sum[3]};
  // One way for the whole launch: a wave that holds whole and cut quads runs the epilogue twice.  This kernel alone, 1419 x 539 in two splits with
  // GeLU: element by element 5.2 us, whole quads with cut ones between them 5.6; 1408 x 544, all whole: 5.1 element by element, 4.9.
  store_quad<T, TC>(args, m, n, v, args.skewN % 4 == 0 && all_quads_are_whole<TC>(args));
}

/* ------------------------------------------------------------------------------------------- launching */

inline int esize(int dtype) { return dtype == HAP_BF16 ? 2 : 4; }

/* Sums the partial tiles of a launch that split K (tile BM x BN). */
template <typename T, typename TC, int BM, int BN>
int launch_splitk_reduce(const GemmArgs& a, int groups, hipStream_t st) {
  const int out_tiles = a.tiles_m * a.tiles_n;
  const long long threads = (long long)out_tiles * (BM * BN / 4);
  hipLaunchKernelGGL((splitk_reduce_kernel<T, TC, BM, BN>), dim3((unsigned)((threads + 255) / 256), groups), dim3(256), 0, st, a, out_tiles);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hap_fail(HAP_EDEVICE, "split-K reduce launch: %s", hipGetErrorString(e));
  return HAP_OK;
}

/* Launches one of the direct-to-LDS kernels with `smem` bytes of LDS, and the reduction behind it when K is split.  `configured`
 * belongs to the kernel: the LDS attribute has to be set on the kernel's copy on every device (benign race: idempotent). */
template <typename TC, int BM, int BN, bool SPLITS = true>
int launch_lds_kernel(void (*kernel)(const GemmArgs), bool (&configured)[64], size_t smem, int threads, const GemmArgs& a, int groups, hipStream_t st) {
  int device = 0;
  if (hipGetDevice(&device) != hipSuccess || device < 0 || device >= 64) device = -1;
  if (device < 0 || !configured[device]) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return hap_fail(HAP_EDEVICE, "cannot reserve %zu bytes of LDS: %s", smem, hipGetErrorString(e));
    if (device >= 0) configured[device] = true;
  }
  hipLaunchKernelGGL(kernel, dim3(a.tiles_m * a.tiles_n * a.ksplit, groups), dim3(threads), smem, st, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hap_fail(HAP_EDEVICE, "gemm launch: %s", hipGetErrorString(e));
  if constexpr (SPLITS) return a.ksplit > 1 ? launch_splitk_reduce<__bf16, TC, BM, BN>(a, groups, st) : HAP_OK;
  return HAP_OK;
}

/* Defined in the translation unit that instantiates the kernels in question. */
int run_pp(const hap_gemm_problem* p, const GemmArgs& a, int groups, hipStream_t st);             // hap_gemm_pp.hip: gemm_pp_kernel, 256 x 256
int run_trio(const hap_gemm_problem* p, const GemmArgs& a, int groups, hipStream_t st);           // hap_gemm_trio.hip: gemm_trio_kernel
int run_small(const hap_gemm_problem* p, const GemmArgs& a, int bm, int groups, hipStream_t st);  // hap_gemm_small.hip: gemm_small_kernel of bm rows
int run_dma(const hap_gemm_problem* p, const GemmArgs& a, int tile, int groups, hipStream_t st);  // hap_gemm_dma.hip: gemm_dma_kernel of 128- or
                                                                                                  // 256-tiles, gemm_kpair_kernel

}  // namespace hap_gemm_detail

#endif
