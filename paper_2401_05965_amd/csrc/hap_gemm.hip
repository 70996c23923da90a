/*
 * GEMM engine of libhap for gfx950 (CDNA4): bf16 / fp32 MFMA, LDS-tiled, ragged edges handled by
 * predication instead of padding the problem.
 *
 * Data movement.  A tile of each operand is fetched as 16-byte chunks with raw buffer loads
 * (an out-of-range chunk costs no memory access and reads as zero) and stored in LDS in the
 * operand's own contiguous direction:
 *   K-contiguous operand  -> LDS rows are m (or n), chunks run along k; MFMA fragments come from
 *                            one 128-bit LDS read per lane;
 *   M/N-contiguous operand-> LDS rows are k, chunks run along m (or n); fragments come from the
 *                            transposing LDS read of gfx950 (ds_read_b64_tr_b16), which hands each
 *                            lane 4 consecutive k of one column.
 * 16-byte chunks are XOR-swizzled inside a row so both kinds of fragment read are bank-conflict free.
 *
 * Raggedness.  Shard ranges start at arbitrary elements (e.g. column 13443 of a bf16 matrix), so the
 * launcher aligns every operand base DOWN to 16 bytes and passes the number of leading elements
 * (skew) that do not belong to the shard.  Leading / trailing elements along k are zeroed in
 * registers before they reach LDS; leading / trailing rows and columns of C are simply not stored.
 *
 * Kernels.  gemm_pp_kernel: bf16, 256 x 256 tiles, two wave groups that alternate a memory phase and a matrix phase over a
 * 4-stage ring of direct-to-LDS K tiles (all layouts but "both operands K-contiguous").  gemm_dma_kernel: bf16, two-stage ring,
 * 256 x 256 (both operands K-contiguous) and 128 x 128 (small outputs, remainder strips).  gemm_trio_kernel: bf16, 128 x 128, three
 * workgroups per compute unit, short contractions.  gemm_kpair_kernel: bf16, 128 x 128, at
 * most one tile per compute unit, two wave groups that split the tile's contraction.  gemm_small_kernel: bf16, 32 x 64 and 64 x 64, the
 * smallest outputs, eight waves that split the contraction.  gemm_kernel: register-staged, fp32
 * and what the direct kernels cannot address.  gemm_skinny_f32_kernel: fp32 products of few rows, contraction split over
 * the waves of a workgroup.  gemm_rank_f32_kernel: fp32 products over few k of two M-/N-contiguous operands; linear_bwd_f32_kernel:
 * both in one launch.  gemm_generic_kernel: scalar fallback.  Epilogues: bias, GeLU, pre-activation copy, fp32
 * accumulation, or the product times gelu'(saved pre-activation) - the activation backward of the layer that produced the
 * output's tensor.
 */
#include "hap_gemm_kernels.h"

namespace hap_gemm_detail {

/* ---------------------------------------------------------------------------------------------
 * fp32 products of few output rows (a layer whose batch shard is a few dozen samples: the single fully-connected layer
 * of the smallest workload, 38 / 26 rows of 64).  Such a product has far too few output tiles for the chip, and splitting its
 * contraction over workgroups costs a second, dependent launch for the reduction - on this machine about as long as the product
 * itself.  Here the split happens INSIDE a workgroup: one workgroup owns one 16-row block or up to 64 rows of 16 output columns, its 16 waves each
 * contract 1/16 of K with v_mfma_f32_16x16x4_f32, and their partial tiles are summed through LDS in a fixed order (deterministic).
 *   A (K-contiguous): lane (row r = lane % 16, k-quad q = lane / 16) fetches the 4 consecutive k values 16c + 4q .. + 3 of a
 *   16-wide chunk c as one 16-byte load and feeds element s to step s; B's lane (k-quad q, column) supplies the same k, so the
 *   order in which a chunk's k values are consumed is a permutation that both operands share.
 * ------------------------------------------------------------------------------------------- */
struct SkinnyArgs {
  int M, N, K;
  long long lda, ldb, ldc, ldp;
  const float* a; const float* b; float* c; float* preact; const float* bias;
  int act, accumulate;
};

typedef float f32x4_t __attribute__((ext_vector_type(4)));

/* RB: 16-row blocks of a workgroup (blockIdx.y counts them; skinny_f32_row_blocks() chooses).  1: 38
 * rows of a 1024-wide layer are 64 workgroups of three row blocks or 192 of one, each with a third of the MFMAs and of the A
 * traffic (the weight is then read three times, out of L2); with all rows in one workgroup (4) the weight is read once, for outputs
 * wide enough to fill the chip by themselves.  That layer's forward, backward and factor rebuild: 38.2 us with 4, 31.9 with 1. */
template <bool BKC, int RB>
__device__ __forceinline__ void skinny_f32_tile(const SkinnyArgs& g, int bx, int by, float (*red)[16 * RB][16]) {
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, r = lane & 15, kq = lane >> 4;
  const int n0 = bx * 16, col = n0 + r, row0 = by * (16 * RB);
  const int rb = (g.M - row0 + 15) >> 4;             // 16-row blocks in use
  const int kslice = ((g.K + 255) >> 8) << 4;        // k values per wave, a multiple of 16
  const int kb0 = wave * kslice;
  const int kb1 = kb0 + kslice < g.K ? kb0 + kslice : g.K;      // (K is a multiple of 4: a lane's quad is inside or outside as a whole)
  f32x4_t acc[RB];
#pragma unroll
  for (int i = 0; i < RB; ++i) acc[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  for (int kb = kb0; kb < kb1; kb += 64) {
    f32x4_t av[4][RB], bv[4];
    // all loads of four chunks first, then their MFMAs
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int kk = kb + 16 * c + 4 * kq;
      const bool kin = kk < kb1;
      bv[c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      if (kin && col < g.N) {
        if constexpr (BKC) bv[c] = *reinterpret_cast<const f32x4_t*>(g.b + (long long)col * g.ldb + kk);
        else {
#pragma unroll
          for (int x = 0; x < 4; ++x) bv[c][x] = g.b[(long long)(kk + x) * g.ldb + col];
        }
      }
#pragma unroll
      for (int i = 0; i < RB; ++i) {
        const int row = row0 + i * 16 + r;
        av[c][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        if (i < rb && kin && row < g.M) av[c][i] = *reinterpret_cast<const f32x4_t*>(g.a + (long long)row * g.lda + kk);
      }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int i = 0; i < RB; ++i)
          if (i < rb) acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[c][i][x], bv[c][x], acc[i], 0, 0, 0);
  }
  // accumulator element v of lane l is output (row 4 * (l / 16) + v, column l % 16) of its 16-row block
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) red[wave][i * 16 + 4 * kq + v][r] = acc[i][v];
  __syncthreads();
  const int lrow = tid >> 4, row = row0 + lrow, c = tid & 15, n = n0 + c;
  if (lrow >= 16 * RB || row >= g.M || n >= g.N) return;
  float v = 0.f;
#pragma unroll
  for (int w = 0; w < 16; ++w) v += red[w][lrow][c];
  if (g.bias) v += g.bias[n];
  if (g.preact) g.preact[(long long)row * g.ldp + n] = v;
  if (g.act == HAP_ACT_GELU_ERF) v = gelu_erf(v);
  float* dst = g.c + (long long)row * g.ldc + n;
  if (g.accumulate) v += *dst;
  *dst = v;
}

template <bool BKC, int RB>
__global__ __launch_bounds__(1024) void gemm_skinny_f32_kernel(const SkinnyArgs g) {
  __shared__ float red[16][16 * RB][16];             // one partial [rows][columns] tile per wave: 16 KB per row block
  skinny_f32_tile<BKC, RB>(g, blockIdx.x, blockIdx.y, red);
}

/* ---------------------------------------------------------------------------------------------
 * fp32 products of two M-/N-contiguous operands over few k (the weight gradient of a layer whose batch shard is a few dozen rows, the
 * rebuild from such factors): dW[m][n] = sum over k of X[k][m] dY[k][n].
 * Bound: latency.  The operands' rows are the MFMA's lanes, so fragments come straight from global memory, 128 bytes per row and half
 * wave: no LDS, no barrier on the way, and a wave has the loads of 32 k values in flight before its first MFMA.  A wave owns one 32 x 32
 * tile; with KG = 4 four waves share it, each takes every fourth chunk of 16 k values, and the four meet in LDS in a fixed order.  The
 * waves of the first tile row also add up their columns of B where the caller asks (the bias gradient: B is in their registers anyway).
 * ------------------------------------------------------------------------------------------- */
struct RankArgs {
  int M, N, nseg, accumulate;
  int tiles_n;                      // workgroup tiles (64 x 64) along N
  long long lda, ldb, ldc;
  float* c;
  float* colsum;                    // [N] sums over all k of B, or nullptr
  const float* a[HAP_GEMM_MAX_SEG];
  const float* b[HAP_GEMM_MAX_SEG];
  int k[HAP_GEMM_MAX_SEG];          // > 0
};

/* CK: k values of a chunk.  FOLD: no chain of additions longer than 128 k values.  Left out in linear_bwd_f32_kernel, whose callers keep to
 * kUnfoldedK values in all, 128 for each of its four wave groups: the second set of accumulators would take the registers with which two
 * workgroups share a compute unit. */
constexpr int kUnfoldedK = 4 * 128;

template <int KG, int CK, bool FOLD>
__device__ __forceinline__ void rank_f32_tile(const RankArgs& g, int tile, float* red) {
  const int lane = threadIdx.x & 63, wave = uni((int)threadIdx.x >> 6), cl = lane & 31, h = lane >> 5;
  const int grp = wave >> 2, w = wave & 3;
  const int tm = tile / g.tiles_n, tn = tile - tm * g.tiles_n;
  const int m0 = (tm * 2 + (w >> 1)) * 32, n0 = (tn * 2 + (w & 1)) * 32;
  const bool sums = g.colsum && m0 == 0;
  // lane offsets of k = h; lanes beyond the matrix read out of range (zeros), and so do k beyond the segment
  const unsigned va = m0 + cl < g.M ? (unsigned)((h * g.lda + m0 + cl) * 4) : kOobOffset;
  const unsigned vb = n0 + cl < g.N ? (unsigned)((h * g.ldb + n0 + cl) * 4) : kOobOffset;
  f32x16_t acc, folded;
#pragma unroll
  for (int e = 0; e < 16; ++e) { acc[e] = 0.0f; folded[e] = 0.0f; }
  float cs[2] = {0.0f, 0.0f}, cst = 0.0f;
  int seg = 0, k0 = 0, k = g.nseg ? uni(g.k[0]) : 0;  // next chunk
  auto skip = [&](int chunks) {
    for (int i = 0; i < chunks && seg < g.nseg; ++i) {
      k0 += CK;
      if (k0 >= k) { seg = uni(seg + 1); k0 = 0; k = seg < g.nseg ? uni(g.k[seg]) : 0; }
    }
  };
  float av[2][CK / 2], bv[2][CK / 2];
  int len[2];                                        // k values of the two chunks in registers, 0: none
  auto load = [&](auto which) {
    constexpr int Q = decltype(which)::value;
    len[Q] = 0;
    if (seg >= g.nseg) return;
    const __amdgpu_buffer_rsrc_t ra = make_rsrc(g.a[seg], (unsigned)(((long long)(k - 1) * g.lda + g.M) * 4));
    const __amdgpu_buffer_rsrc_t rb = make_rsrc(g.b[seg], (unsigned)(((long long)(k - 1) * g.ldb + g.N) * 4));
    len[Q] = k - k0 < CK ? k - k0 : CK;
    // (the whole offset goes in the lanes' part: the range check does not hold for a scalar offset beyond the extent)
    const unsigned oa = va + (unsigned)((long long)k0 * g.lda * 4), ob = vb + (unsigned)((long long)k0 * g.ldb * 4);
#pragma unroll
    for (int i = 0; i < CK / 2; ++i) {
      av[Q][i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(ra, oa + i * (unsigned)(g.lda * 8), 0, 0));
      bv[Q][i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rb, ob + i * (unsigned)(g.ldb * 8), 0, 0));
    }
    skip(KG);
  };
  auto contract = [&](auto which) {
    constexpr int Q = decltype(which)::value;
#pragma unroll
    for (int i = 0; i < CK / 2; ++i) {
      if (i % 2 == 0 && len[Q] <= 2 * i) break;
      acc = mfma(av[Q][i], bv[Q][i], acc);
      if (sums) cs[i & 1] += bv[Q][i];
    }
  };
  if (m0 < g.M && n0 < g.N) {
    skip(grp);
    load(std::integral_constant<int, 0>());
    load(std::integral_constant<int, 1>());
    for (int done = 0; len[0] > 0; ++done) {
      if (FOLD && done == 64 / CK) {
        folded += acc; cst += cs[0] + cs[1];
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[e] = 0.0f;
        cs[0] = cs[1] = 0.0f;
        done = 0;
      }
      contract(std::integral_constant<int, 0>());
      load(std::integral_constant<int, 0>());
      if (len[1] > 0) contract(std::integral_constant<int, 1>());
      load(std::integral_constant<int, 1>());
    }
    if (FOLD) acc += folded;
    cst += cs[0] + cs[1];
  }
  cst += __shfl_xor(cst, 32, 64);
  constexpr int EW = 16 / KG;                        // accumulator elements that a wave stores
  const int e0 = grp * EW;
  if constexpr (KG > 1) {
    float* const sums_at = red + KG * 4 * 16 * 64;   // [group][wave column][32]
#pragma unroll
    for (int e = 0; e < 16; ++e) red[((grp * 4 + w) * 16 + e) * 64 + lane] = acc[e];
    if (sums && h == 0) sums_at[(grp * 2 + (w & 1)) * 32 + cl] = cst;
    __syncthreads();
    if (sums) {
      cst = 0.0f;
#pragma unroll
      for (int q = 0; q < KG; ++q) cst += sums_at[(q * 2 + (w & 1)) * 32 + cl];
    }
  }
  if (m0 >= g.M || n0 + cl >= g.N) return;
  if (sums && grp == 0 && h == 0) g.colsum[n0 + cl] = cst;
#pragma unroll
  for (int x = 0; x < EW; ++x) {
    const int e = KG > 1 ? e0 + x : x;
    float v;
    if constexpr (KG > 1) {
      v = 0.0f;
#pragma unroll
      for (int q = 0; q < KG; ++q) v += red[((q * 4 + w) * 16 + e) * 64 + lane];
    } else {
      v = acc[x];
    }
    const int m = m0 + (e >> 2) * 8 + h * 4 + (e & 3);
    if (m < g.M) {
      float* dst = g.c + (long long)m * g.ldc + n0 + cl;
      *dst = g.accumulate ? *dst + v : v;
    }
  }
}

constexpr int kRankRed = 4 * 4 * 16 * 64 + 4 * 2 * 32;     // floats of LDS with KG = 4

template <int KG>
__global__ __launch_bounds__(256 * KG) void gemm_rank_f32_kernel(const RankArgs g) {
  __shared__ float red[KG > 1 ? kRankRed : 1];
  rank_f32_tile<KG, 16, true>(g, blockIdx.x, red);
}

/* bwd-data of few rows and the weight (and bias) gradient of the same layer in one launch: neither fills the chip and neither needs the
 * other.  The first `nrank` workgroups take the weight gradient, over at most kUnfoldedK rows, nx x (rows / 16) the data gradient.
 * Bound: latency; 64 registers at most, so that two workgroups of 1024 threads share a compute unit (38 x 1024 x 1024: 8.0 us with 55
 * registers, 9.7 with 89). */
__global__ __launch_bounds__(1024, 8) void linear_bwd_f32_kernel(const RankArgs w, const SkinnyArgs x, int nrank, int nx) {
  __shared__ float red[kRankRed];
  if ((int)blockIdx.x < nrank) { rank_f32_tile<4, 8, false>(w, blockIdx.x, red); return; }
  const int id = blockIdx.x - nrank;
  skinny_f32_tile<true, 1>(x, id % nx, id / nx, reinterpret_cast<float (*)[16][16]>(red));
}

/* Compute units of the current device (256 on MI355X); the planner's round arithmetic uses it.  Asked once per device, the device once per
 * product (each question costs a small product's call some hundredths of a microsecond): look_up_cu_count() on entry, for its thread. */
static thread_local int t_cus = 256;
static inline int cu_count() { return t_cus; }
static void look_up_cu_count() {
  static int cached[64] = {};
  int device = 0;
  if (hipGetDevice(&device) != hipSuccess || device < 0 || device >= 64) { t_cus = 256; return; }
  if (cached[device] == 0) {     // benign race: every thread stores the same value
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || n < 8) n = 256;
    cached[device] = n;
  }
  t_cus = cached[device];
}

inline long long cdiv(long long a, long long b) { return (a + b - 1) / b; }

constexpr size_t kSmallTileBytes = 128 * 128 * sizeof(float);     // a partial tile
constexpr long long kShortContraction = 24;                      // K tiles of 64 up to which the planner compares microseconds (us_256() below)

/* What the planner weighs the kernels by (below). */
long long workgroup_splits(const hap_gemm_problem* p, long long tiles, long long slots, long long steps, int min_steps, size_t tile_bytes);
bool kpair_applies(const hap_gemm_problem* p, long long tiles, long long nk);
int kpair_splits(const hap_gemm_problem* p, long long tiles, long long nk, double* us);
double us_256(const hap_gemm_problem* p, long long n, long long nk);
bool trio_applies(const hap_gemm_problem* p, long long n, long long nk, double* us);

/* 16-row blocks per workgroup with which gemm_skinny_f32_kernel takes the product: 1, 4 (all rows, at most 64), or 0 where it does not.
 * Microseconds, what ran before -> one row block:
 *   forward, rows x in x out:  64 x 2048 x 2048 22.3 -> 16.3    100 x 1024 x 1024 13.1 -> 8.3    256 x 512 x 512: 11.2 -> 6.2    256 x 1024 x 1024 17.6 -> 14.2
 *   bwd-data:  128 x 1024 x 1024 13.4 -> 9.2    512 x 512 x 512 12.4 -> 10.8 (1024 workgroups)
 * More than 64 rows: one row block each, where the tiled kernel could split K as long as the rounds of workgroups over the compute units,
 * times K, are at most 4096 (5120 in a single round):
 *   one round, 80 to 256 workgroups, K = 4096 / 5120 / 6144:  forward 17.7 -> 13.8 / 20.0 -> 18.8 / 21.7 -> 22.8, bwd-data 18.5 -> 16.1 / 20.3 -> 19.6 / 22.0 -> 23.2
 *   two rounds, 258 workgroups, K = 2048 / 2560:  18.2 -> 15.5 / 19.8 -> 20.2, 17.3 -> 16.3 / 19.3 -> 20.6
 *   three rounds, 516 workgroups, K = 1300 / 1536:  17.3 -> 15.9 / 17.3 -> 19.0    four rounds, K = 1024 / 2048: 17.4 -> 14.2 / 27.0 -> 29.9
 *   more:  256 x 2048 x 512 16.5 -> 18.8 (2048 workgroups)
 * and, where it could not (no workspace, or a weight whose rows are not on the 16-byte grid and go to the scalar kernel), up to a thousand
 * workgroups of a million k values in all (without a workspace 688 workgroups over K = 1300 39.3 -> 17.6).
 * Up to 64 rows: all rows in one workgroup where the columns alone give half of the compute units one: 38 x 512 x 4096 7.0 as one row
 * block each 8.5, 64 x 1024 x 4096 12.7 and 16.1; and three row blocks of a forward over a long K, whose weight would be read three times:
 * 38 x 1024 x 1600 8.4 and 7.7, 38 x 2048 x 1600 14.9 and 15.4, 38 x 8192 x 2048 54.0 and 58.7 (bwd-data 56.0 and 53.4, 50 rows 69.0 and 63.2). */
static int skinny_f32_row_blocks(const hap_gemm_problem* p) {
  if (p->in_dtype != HAP_F32 || p->c_dtype != HAP_F32 || !p->a_kcontig || p->nseg != 1) return 0;
  if (p->groups > 1 || p->group_len || p->force_generic || p->tile || p->dact) return 0;
  const int64_t K = p->k[0];
  if (K < 256 || K % 4 || K > 0x7fffffff || (p->N + 63) / 64 >= 128) return 0;      // enough 64-wide tiles: the tiled kernel fills the chip by itself
  if (p->lda % 4 || (uintptr_t)p->a[0] % 16) return 0;
  if (p->b_kcontig && (p->ldb % 4 || (uintptr_t)p->b[0] % 16)) return 0;
  const int64_t columns = (p->N + 15) / 16, rows = (p->M + 15) / 16, cus = cu_count(), groups = columns * rows;
  if (p->M > 64) {
    if (rows > 4 * cus || groups > 4 * cus || groups * K > 4096 * cus) return 0;
    if (p->ldb % 4 || workgroup_splits(p, cdiv(p->M, 64) * cdiv(p->N, 64), 4 * cus, cdiv(K, 64), 2, 64 * 64 * sizeof(float)) < 2) return 1;
    return cdiv(groups, cus) * K <= (groups <= cus ? 5120 : 4096) ? 1 : 0;
  }
  if (groups <= cus) return 1;
  return columns * 2 <= cus && (rows > 3 || p->b_kcontig || K <= 1536) ? 1 : 4;
}

/* Whether a product goes to gemm_rank_f32_kernel: as many k values as its waves contract in the time that the tiled kernel and, where it
 * splits K, the reduction behind it take.  Microseconds, tiled -> this kernel:
 *   1024 x 1024 (256 tiles of 64 x 64) over k = 38 / 256 / 512 / 2048: 8.2 -> 5.2 / 17.2 -> 9.0 / 25.2 -> 13.7 / 50.6 -> 43.0
 *   512 x 512 (64 tiles) over 200 / 400 / 512 / 1024: 11.9 -> 7.5 / 12.8 -> 10.9 / 12.2 -> 13.0 / 17.7 -> 22.5    1024 x 512 over 2048: 34.2 -> 42.4
 *   2048 x 2048 (1024 tiles) over 64 / 450 / 512: 14.4 -> 11.6 / 44.4 -> 40.6 / 45.9 -> 46.1    300 x 300 (25 tiles) over 448: 11.1 -> 12.0 */
static bool rank_f32_applies(const hap_gemm_problem* p) {
  if (p->in_dtype != HAP_F32 || p->c_dtype != HAP_F32 || p->a_kcontig || p->b_kcontig || p->M <= 0 || p->N <= 0) return false;
  if (p->groups > 1 || p->group_len || p->force_generic || p->tile || p->dact || p->act != HAP_ACT_NONE || p->bias || p->preact) return false;
  const int64_t tiles = ((p->M + 63) / 64) * ((p->N + 63) / 64);
  int64_t most = tiles * 7 < 2048 ? tiles * 7 : 2048, k = 0;
  if (tiles > 2 * cu_count()) most = 448;
  else if (most < 256) most = 256;
  if (tiles > 0x7fffffff || p->M > 0x7fffffff || p->N > 0x7fffffff) return false;
  for (int s = 0; s < p->nseg; ++s) {
    if (p->k[s] <= 0) continue;
    if ((uintptr_t)p->a[s] % 4 || (uintptr_t)p->b[s] % 4) return false;
    // every offset that a lane forms, also past the segment's end, stays below the out-of-range marker
    if ((p->k[s] + 16) * p->lda * 4 + p->M * 4 >= kViewLimitBytes || (p->k[s] + 16) * p->ldb * 4 + p->N * 4 >= kViewLimitBytes) return false;
    k += p->k[s];
  }
  return k <= most;
}

/* Scalar fallback for operand views the tiled kernel cannot address with aligned 16-byte chunks
 * (leading dimension not a multiple of 16 bytes, or differently skewed K-contiguous operands). */
struct GenericArgs {
  int M, N, nseg;
  long long lda, ldb, ldc, ldp;
  int a_kcontig, b_kcontig;
  void* c; void* preact; const void* bias;
  int act, accumulate;
  const void* dact_preact; long long ldd;
  int ragged;                        // as in GemmArgs; blockIdx.z is the group
  const int* group_len;
  long long ga, gb, gc, gp, gbias, gd;   // byte strides between groups
  const void* a[HAP_GEMM_MAX_SEG];
  const void* b[HAP_GEMM_MAX_SEG];
  int k[HAP_GEMM_MAX_SEG];
};

template <typename T, typename TC>
__global__ __launch_bounds__(256) void gemm_generic_kernel(const GenericArgs g) {
  const int n = blockIdx.x * 16 + (threadIdx.x & 15);
  const int m = blockIdx.y * 16 + (threadIdx.x >> 4);
  const int grp = blockIdx.z;
  int len = g.ragged ? g.group_len[grp] : 0;
  len = len < 0 ? 0 : len;
  const int M = g.ragged == 1 && len < g.M ? len : g.M;
  if (m >= M || n >= g.N) return;
  float acc = 0.0f;
  for (int s = 0; s < g.nseg; ++s) {
    const T* A = reinterpret_cast<const T*>(static_cast<const char*>(g.a[s]) + grp * g.ga);
    const T* B = reinterpret_cast<const T*>(static_cast<const char*>(g.b[s]) + grp * g.gb);
    const int ks = g.ragged == 2 && len < g.k[s] ? len : g.k[s];
    for (int k = 0; k < ks; ++k) {
      const float av = load_s<T>(g.a_kcontig ? A + (long long)m * g.lda + k : A + (long long)k * g.lda + m);
      const float bv = load_s<T>(g.b_kcontig ? B + (long long)n * g.ldb + k : B + (long long)k * g.ldb + n);
      acc = fmaf(av, bv, acc);
    }
  }
  if (g.bias) acc += load_s<T>(reinterpret_cast<const T*>(static_cast<const char*>(g.bias) + grp * g.gbias) + n);
  if (g.preact) store_c<TC>(reinterpret_cast<TC*>(static_cast<char*>(g.preact) + grp * g.gp) + (long long)m * g.ldp + n, acc);
  if (g.act == HAP_ACT_GELU_ERF) acc = gelu_erf((float)(TC)acc);     // the activation sees the value as stored
  if (g.dact_preact) acc *= gelu_erf_grad(load_s<TC>(reinterpret_cast<const TC*>(static_cast<const char*>(g.dact_preact) + grp * g.gd) + (long long)m * g.ldd + n));
  TC* dst = reinterpret_cast<TC*>(static_cast<char*>(g.c) + grp * g.gc) + (long long)m * g.ldc + n;
  if (g.accumulate) acc += load_s<TC>(dst);
  store_c<TC>(dst, acc);
}

constexpr int kPingPongBK = 32;   // K step of the ping-pong kernel

struct Plan {
  bool tiled;
  int skewM, skewN, skewK;
  int bm, bn;       // tile
  int bk;           // K step of the kernel that will run (the K-tile counts handed to it are in this unit)
  int dma;          // 1: bf16, direct-to-LDS kernel; 0: fp32, register-staged kernel
  bool pingpong;    // 256 x 256 tiles run by gemm_pp_kernel
  bool small;       // BM x 64 tiles run by gemm_small_kernel
};

/* Rows of the tiles with which gemm_small_kernel takes a bf16 product (32 or 64), 0 where it does not: at most one tile per compute unit
 * (a workgroup's rings fill its LDS), of 32 rows where there are compute units for that, over contractions that a wave's eighth of does
 * not take longer than the split over workgroups that the other kernels make.  Microseconds, what ran before -> this kernel:
 *   tiles of 32, forward:  197 x 1024 x 1260 13.6 -> 6.7    512 x 512 x 512 9.9 -> 5.6    400 x 1024 x 1024 12.2 -> 7.0 (208 tiles)
 *   tiles of 64:  forward 1024 x 1024 x 1024 12.4 -> 9.0, with GeLU 17.1 -> 10.7    bwd-weight 768 x 768 over 1500 rows 15.3 -> 8.9
 *   beyond 256 tiles of 64:  1500 x 768 x 768 11.5 -> 13.6 (288)    2000 x 640 x 1024 11.1 -> 14.4
 * Long contractions end it where the others can split theirs (in steps of 32; 2500 random sizes, pitches and epilogues over 62 to 162 steps, time
 * here over time there, geometric mean / worst):
 *   tiles of 32:  up to 64 of them, 152 to 159 steps 0.85 / 1.16    65 to 128, 128 to 135 steps 0.82 / 1.02, 144 to 151 0.98 / 1.24
 *                 beyond, 112 to 119 steps 0.90 / 1.00, 120 to 124 0.95 / 1.06
 *                 experts' bwd-data, each with a weight of its own to read once per 32 rows, more than 64 tiles: 96 to 103 steps 0.81 / 1.02, 104 to 111
 *                 0.91 / 1.08, 112 to 124 0.96 / 1.19
 *   tiles of 64, forward:  88 to 95 steps 0.92 / 1.01, 100 to 107 0.99 / 1.06    bwd-data:  84 to 87 steps 0.92 / 1.01, 92 to 95 0.99 / 1.05,
 *                 experts' 88 to 95 1.07 / 1.11, 108 to 111 1.05 / 1.13
 *   tiles of 64, bwd-weight:  up to 32 of them, 136 to 143 steps 0.95 / 1.08, 152 to 159 1.01 / 1.22    33 to 128, 104 to 111 steps 0.86 / 0.96, 112 to 119
 *                 0.93 / 1.05, 128 to 135 0.98 / 1.14    beyond, 120 to 124 steps 0.95 / 1.01
 * Without a workspace for their partial tiles they take 1.2 to 2.7 times as long as this kernel wherever it applies. */
int small_rows(const hap_gemm_problem* p, const Plan& pl) {
  if (p->in_dtype != HAP_BF16 || p->tile == 256 || (!p->a_kcontig && p->b_kcontig)) return 0;
  if (p->c_dtype == HAP_F32 && p->a_kcontig) return 0;       // (a form no product of the path has)
  const long long cus = cu_count(), groups = p->groups > 1 ? p->groups : 1;
  long long steps = 0, nk = 0;
  for (int s = 0; s < p->nseg; ++s) {
    if (p->k[s] <= 0) continue;
    steps += (pl.skewK + p->k[s] + 31) / 32;
    nk += (pl.skewK + p->k[s] + 63) / 64;
  }
  const long long columns = groups * ((p->N + pl.skewN + 63) / 64);
  for (int bm = p->a_kcontig ? 32 : 64; bm <= 64; bm *= 2) {      // (an M-contiguous operand's LDS rows are 128 bytes or more)
    const long long tiles = columns * ((p->M + pl.skewM + bm - 1) / bm);
    if (tiles > cus) continue;
    long long most = tiles * 2 > cus ? 124 : 160;
    if (workgroup_splits(p, groups * cdiv(p->M + pl.skewM, 128) * cdiv(p->N + pl.skewN, 128), 2 * cus, nk, 4, kSmallTileBytes) > 1) {
      if (bm == 32) most = tiles * 4 <= cus ? 160 : ((groups > 1 || p->group_len) && p->b_kcontig ? 103 : (tiles * 2 > cus ? 124 : 136));
      else if (p->a_kcontig) most = p->b_kcontig ? 87 : 95;
      else most = tiles * 2 > cus ? 124 : (tiles * 8 > cus ? 112 : 144);
    }
    return steps <= most ? bm : 0;
  }
  return 0;
}

/* Decides whether the aligned-chunk kernel can address the operands and with which skews. */
Plan make_plan(const hap_gemm_problem* p) {
  Plan pl = {false, 0, 0, 0, 0, 0, 64, 0, false, false};
  if (p->force_generic) return pl;
  const int es = esize(p->in_dtype);
  if ((p->lda * es) % 16 || (p->ldb * es) % 16) return pl;
  if (p->groups > 1 && ((p->ga * es) % 16 || (p->gb * es) % 16)) return pl;   // every group needs the first one's 16-byte phase
  int sa = -1, sb = -1;
  for (int s = 0; s < p->nseg; ++s) {
    if (p->k[s] == 0) continue;
    const int xa = (int)(((uintptr_t)p->a[s] % 16) / es), xb = (int)(((uintptr_t)p->b[s] % 16) / es);
    if (((uintptr_t)p->a[s] % es) || ((uintptr_t)p->b[s] % es)) return pl;
    if (sa < 0) { sa = xa; sb = xb; }
    else if (sa != xa || sb != xb) return pl;
  }
  if (sa < 0) { sa = sb = 0; }
  if (p->a_kcontig && p->b_kcontig && sa != sb) return pl;
  // K-contiguous operands: a K tile fetches 64 or 128 consecutive bytes of every row, so the K-tile grid is laid on 128-byte
  // (else 64-byte) boundaries of the operand's own address space where the pitch allows it - the view's first k then sits up
  // to 63 elements into its first tile, which is masked like any skew.  Fetches that straddle cache sectors cost 10-20 %.
  if (p->in_dtype == HAP_BF16 && !(p->groups > 1) && (p->a_kcontig || p->b_kcontig)) {
    for (int gran = 128; gran >= 32; gran /= 2) {
      if ((p->a_kcontig && (p->lda * es) % gran) || (p->b_kcontig && (p->ldb * es) % gran)) continue;
      int ka = -1, kb = -1;
      bool ok = true;
      for (int s = 0; s < p->nseg && ok; ++s) {
        if (p->k[s] == 0) continue;
        const int xa = (int)(((uintptr_t)p->a[s] % gran) / es), xb = (int)(((uintptr_t)p->b[s] % gran) / es);
        if (ka < 0) { ka = xa; kb = xb; }
        else ok = (!p->a_kcontig || ka == xa) && (!p->b_kcontig || kb == xb);
      }
      if (!ok || ka < 0 || (p->a_kcontig && p->b_kcontig && ka != kb)) continue;
      if (p->a_kcontig) sa = ka;
      if (p->b_kcontig) sb = kb;
      break;
    }
  }
  pl.skewK = p->a_kcontig ? sa : (p->b_kcontig ? sb : 0);
  pl.skewM = p->a_kcontig ? 0 : sa;
  pl.skewN = p->b_kcontig ? 0 : sb;
  // A K-contiguous B has no preferred column origin of its own (its rows are the output's columns), so the tile grid is laid on
  // the 16-byte chunks of the OUTPUT instead: the reduction rule's dX[:, k_j] of a whole tensor starts at an arbitrary column, and
  // with the grid on its chunks the epilogue stores whole chunks everywhere but at the matrix's two ends.
  if (p->b_kcontig && p->in_dtype == HAP_BF16 && !(p->groups > 1) && !p->group_len) {
    const int ces = esize(p->c_dtype), cepc = 16 / ces;
    if ((uintptr_t)p->c % ces == 0 && p->ldc % cepc == 0) pl.skewN = (int)(((uintptr_t)p->c % 16) / ces);
  }
  // operand views must stay below 2 GiB so 32-bit buffer offsets and the out-of-range marker work
  for (int s = 0; s < p->nseg; ++s) {
    const double ea = p->a_kcontig ? ((double)(p->M - 1) * p->lda + pl.skewK + p->k[s]) : ((double)(p->k[s] - 1) * p->lda + pl.skewM + p->M);
    const double eb = p->b_kcontig ? ((double)(p->N - 1) * p->ldb + pl.skewK + p->k[s]) : ((double)(p->k[s] - 1) * p->ldb + pl.skewN + p->N);
    if (ea * es >= (double)kViewLimitBytes || eb * es >= (double)kViewLimitBytes) return pl;
  }
  pl.tiled = true;
  if (p->in_dtype == HAP_F32) pl.bm = pl.bn = 64;
  else if (const int rows = small_rows(p, pl)) {
    pl.bm = rows; pl.bn = 64; pl.bk = 32;
    pl.dma = 1;
    pl.small = true;
  } else {
    bool big = p->tile ? p->tile == 256 : (p->M + pl.skewM > 128 && p->N + pl.skewN > 128);
    if (big && !p->tile && (p->groups > 1 || p->group_len)) {
      // A grouped launch is not cut into strips: all tiles of all groups, big or small; by microseconds or by rounds: of big tiles (one per
      // CU, time 1; as split-K spreads a few of them over the chip at about a third of a round for the partial-tile traffic) and of small
      // ones (two per CU, 0.6 per round, 0.3 when half empty).
      // Microseconds are the better up to kShortContraction, and for weight gradients past 96 K tiles and, with bf16 outputs, wherever big
      // tiles fill more than half of the chip.  Small -> big tiles, experts x rows x columns over K, where only microseconds say big:
      //   10 x 768 x 3072 over 1024 to 2048 rows 125 -> 107    12 x 1024 x 1976 over up to 5878 275 -> 212    5 x 256 x 3680 over 9545 186 -> 118
      // and where they say so wrongly:
      //   7 x 256 x 2960 over 3094 50.5 -> 54.3    5 x 2048 x 696 over 5767 81.6 -> 86.1    bwd-data 6 x 2039 x 1024 over 1640 50.8 -> 63.6
      const long long g = p->groups > 1 ? p->groups : 1;
      const long long nb = g * ((p->M + pl.skewM + 255) / 256) * ((p->N + pl.skewN + 255) / 256);
      const long long ns = g * ((p->M + pl.skewM + 127) / 128) * ((p->N + pl.skewN + 127) / 128);
      const long long nk = (pl.skewK + p->k[0] + 63) / 64, cus = cu_count();
      const bool long_us = !p->a_kcontig && (nk > 96 || (nb * 2 > cus && p->c_dtype == HAP_BF16));
      double tb, ts;
      if (nk <= kShortContraction || long_us) {
        trio_applies(p, ns, nk, &ts);
        if (kpair_applies(p, ns, nk)) kpair_splits(p, ns, nk, &ts);
        tb = us_256(p, nb, nk);
      } else {
        tb = nb * 2 <= cus ? 0.35 + 1.0 / (double)(cus / nb) : (double)cdiv(nb, cus);
        ts = ns <= cus ? 0.3 : 0.6 * (double)cdiv(ns, 2 * cus);
      }
      big = tb <= ts;
    }
    pl.bm = pl.bn = big ? 256 : 128;
    pl.dma = 1;
    // 256-tiles: the ping-pong kernel, except when both operands are K-contiguous (bwd-data), where the two-stage kernel
    // with 128-byte rows per K tile is the faster one
    // ... and except the shortest contractions, over which the four-stage ring does not fill.  Two-stage -> ping-pong, microseconds:
    // forward 15360 rows x 3072 over K = 64 / 128 / 320: 31.3 -> 33.4 / 35.5 -> 37.3 / 52.8 -> 55.3, 16384 x 2048 over 384: 41.1 -> 42.6
    // (with GeLU 63.1 -> 62.2); from seven K tiles on the ping-pong kernel is ahead: forward 15360 x 3072 over 512 / 768 / 1024:
    // 71.4 -> 65.7 / 83.4 -> 78.2 / 100.1 -> 94.0, bwd-weight 4096 x 8192 over 256 / 400 / 768 rows: 33.1 -> 33.3 / 44.7 -> 41.6 / 61.1 -> 57.7
    long long nk64 = 0;
    for (int s = 0; s < p->nseg; ++s) nk64 += p->k[s] > 0 ? (pl.skewK + p->k[s] + 63) / 64 : 0;
    const bool short_k = nk64 < 7 && !(!p->a_kcontig && p->b_kcontig);
    pl.pingpong = big && !(p->a_kcontig && p->b_kcontig) && !short_k;
    pl.bk = pl.pingpong ? kPingPongBK : 64;
  }
  return pl;
}

template <typename T, typename TC, bool AKC, bool BKC, int BM, int BN, int BK, int WGM, int WGN>
int launch_tiled(const GemmArgs& a, int groups, hipStream_t st) {
  const int out_tiles = a.tiles_m * a.tiles_n;
  hipLaunchKernelGGL((gemm_kernel<T, TC, AKC, BKC, BM, BN, BK, WGM, WGN>), dim3(out_tiles * a.ksplit, groups), dim3(64 * WGM * WGN), 0, st, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hap_fail(HAP_EDEVICE, "gemm launch: %s", hipGetErrorString(e));
  return a.ksplit > 1 ? launch_splitk_reduce<T, TC, BM, BN>(a, groups, st) : HAP_OK;
}

template <typename T, typename TC, int BM, int BN, int BK, int WGM, int WGN>
int dispatch_layout(const hap_gemm_problem* p, const GemmArgs& a, int groups, hipStream_t st) {
  if (p->a_kcontig && p->b_kcontig) return launch_tiled<T, TC, true, true, BM, BN, BK, WGM, WGN>(a, groups, st);
  if (p->a_kcontig && !p->b_kcontig) return launch_tiled<T, TC, true, false, BM, BN, BK, WGM, WGN>(a, groups, st);
  if (!p->a_kcontig && !p->b_kcontig) return launch_tiled<T, TC, false, false, BM, BN, BK, WGM, WGN>(a, groups, st);
  return launch_tiled<T, TC, false, true, BM, BN, BK, WGM, WGN>(a, groups, st);
}

template <typename T, typename TC>
int dispatch_tile(const hap_gemm_problem* p, const Plan& pl, const GemmArgs& a, int groups, hipStream_t st) {
  if constexpr (sizeof(T) == 4) {
    return dispatch_layout<T, TC, 64, 64, 64, 2, 2>(p, a, groups, st);
  } else {
    if (pl.small) return run_small(p, a, pl.bm, groups, st);
    return pl.pingpong ? run_pp(p, a, groups, st) : run_dma(p, a, pl.bm, groups, st);
  }
}


/* Into how many workgroups the launcher splits the contraction of `tiles` output tiles (1: not at all): over the idle slots, with at
 * least min_steps K steps for each, at most sixteen, and as far as the caller's workspace holds the partial tiles. */
long long workgroup_splits(const hap_gemm_problem* p, long long tiles, long long slots, long long steps, int min_steps, size_t tile_bytes) {
  long long g = slots / tiles;
  if (g > steps / min_steps) g = steps / min_steps;
  if (g > 16) g = 16;
  const long long held = p->ws ? (long long)(p->ws_bytes / ((size_t)tiles * tile_bytes)) : 0;
  if (g > held) g = held;
  return g < 2 ? 1 : g;
}

/* Whether 128-tiles of this product run in gemm_kpair_kernel: at most one tile per compute unit, and two K tiles for each of its two
 * wave groups.  The alternative is the 4-wave kernel, which fills the chip by splitting K over workgroups where it has a workspace.
 * The limits lie where the two cross (microseconds, 4-wave -> K-pair, three operand sets in turn, MI355X):
 *   K tiles, 88 output tiles:  3: forward 8.7 -> 8.8, bwd-data 8.6 -> 8.9    4: 9.2 -> 8.9, 9.1 -> 8.9    5: 9.7 -> 9.4, 9.6 -> 9.4
 *   output tiles, K = 1024:    256: 29.9 -> 15.6    272: 20.8 -> 25.9    320: 20.8 -> 25.4
 *   without a workspace:       88 tiles over K = 512 / 1024 / 4096  12.2 -> 10.4 / 17.9 -> 13.2 / 50 -> 28
 * Past 128 K tiles, where the operands stream from HBM, tile counts that leave compute units idle here but not there stay with the 4-wave
 * kernel where it can split K (160 tiles: 62 %, as three splits 94 %; forward over K = 6144 / 7680 / 10240 44.6 -> 41.8 / 52.3 -> 50.3 / 70.7 -> 78.2;
 * in between the two are within 5 %, and the line lies where kpair_splits() raises the cost of a step, so that the planner weighs the
 * kernel that will run).
 * (The smallest outputs run in gemm_small_kernel, which make_plan() asks first.  An M-contiguous A with a K-contiguous B is a form no product
 * of the path has; the kernel is not built for it.) */
bool kpair_applies(const hap_gemm_problem* p, long long tiles, long long nk) {
  const long long cus = cu_count();
  if (p->in_dtype != HAP_BF16 || (!p->a_kcontig && p->b_kcontig) || tiles > cus || nk < 4) return false;
  if (workgroup_splits(p, tiles, 2 * cus, nk, 4, kSmallTileBytes) == 1) return true;
  const long long here = cus / tiles * tiles * 2, there = 2 * cus / tiles * tiles;      // of 2 * cus wave groups
  return nk <= 128 || here * 20 >= there * 17;
}

/* Into how many workgroups that kernel splits K (1: no partial tiles, no reduction launch) and the estimated time in microseconds.
 * Measured: a step (a K tile for each wave group) takes 0.6 with few compute units busy and 0.9 with all, 1.15 there over long
 * contractions, whose operands stream from HBM (256 tiles, K = 50432: 462 in all against 345 for 64 256-tiles with K split in
 * four); 6 for prologue, exchange and epilogue, 4 / 1.5 more for GeLU / its backward in an epilogue that runs on few compute units
 * only; a reduction launch 1.2 and 0.03 per partial tile written and read back.  128 tiles over K = 1024: whole 13, split in
 * two 23; 64 tiles over K = 4096: whole 28, split in four 23.  (Where the step cost rises: 240 and 256 tiles take 0.9 per step at 65 steps,
 * 0.95 to 1.1 at 76, 1.1 at 84.  Between 65 and 76 some sizes are 5 to 20 % faster here than what the planner takes instead, single
 * forward sizes as much slower, 180 tiles over 152 K tiles 85 against 71; 64 is where none of them loses.) */
int kpair_splits(const hap_gemm_problem* p, long long tiles, long long nk, double* us) {
  const long long cus = cu_count();
  const size_t ws_splits = p->ws ? p->ws_bytes / ((size_t)tiles * kSmallTileBytes) : 0;
  int best = 1;
  *us = 0.0;
  for (int s = 1; s <= 16; ++s) {
    if (s > 1 && (tiles * s > cus || nk < 4 * s || (size_t)s > ws_splits)) break;
    const long long steps = cdiv(nk, 2 * s);
    const double busy = (double)(tiles * s) / (double)cus;
    double t = (double)steps * (steps > 64 && busy > 0.5 ? 1.15 : 0.6 + 0.3 * busy) + 6.0;
    t += s > 1 ? 1.2 + 0.03 * (double)(tiles * s) : (p->act != HAP_ACT_NONE ? 4.0 : (p->dact != HAP_ACT_NONE ? 1.5 : 0.0));
    if (s == 1 || t < *us) { best = s; *us = t; }
  }
  return best;
}

/* Relative time of n output tiles of 128x128 (one 256x256 tile on one CU = 1): a small tile does a
 * quarter of the work at lower efficiency, and two of them share a CU. */
static double small_tiles_time(long long n) {
  if (n <= 0) return 0.0;
  const int kCUs = cu_count();
  // measured: a round of 512 small tiles takes 0.58 of a round of 256 big ones; a last round that leaves every CU at
  // most one small tile 0.36 (the tile has the CU to itself)
  const long long full = n / (2 * kCUs), rest = n % (2 * kCUs);
  return 0.58 * (double)full + (rest == 0 ? 0.0 : (rest <= kCUs ? 0.36 : 0.58));
}

/* Estimated microseconds of the bf16 kernels, for the planner.  From least-squares fits over 240 random shapes (M, N 300 to 50000, K 64 to 8400,
 * aligned and not) x five products, each forced through every kernel: standard error 3 to 10 %.  Over those of at most 24 K tiles the
 * choice that these make is 1.0 to 1.5 % slower than the fastest kernel of each (geometric mean, by product), by whole rounds, whatever the
 * epilogue and the contraction, 4 to 16 %.  Over 24 to 48 K tiles the two are alike, beyond 48 the rounds are 1 to 1.5 % better for bwd-data:
 * there a tile's epilogue matters little and what the operands' pitches cost a kernel much.  fp32 outputs: 400 more shapes (300 to 16384 each
 * way, K 32 to 1536) as weight gradients and as rebuilds of two factors; the choice is 0.8 % slower than the fastest kernel, 1.2 % with the
 * bf16 outputs' terms (which lose up to 13 % at K = 64: 3479 x 3072 14.8 -> 16.7), 1.8 % by whole rounds.
 * Over 1200 fresh products of up to 24 K tiles, those of the small-output and the K-pair kernel among them: forward / with GeLU / bwd-data / with
 * gelu' / weight gradient / in fp32 1.2 / 1.4 / 1.4 / 1.9 / 1.3 / 1.0 % off the fastest kernel, by whole rounds 3.0 / 4.3 / 5.8 / 9.3 / 8.0 / 1.2; of the
 * 860 that take 15 us or more, rounds are more than 3 % better for 21 (forward 14701 x 680 over 737 30.1 against 34.5), worse for 202. */
enum { kPlain = 0, kGelu = 1, kDact = 2, kF32 = 3 };     // what the epilogue does; kF32: a weight gradient's or factor rebuild's fp32 output

int epilogue_kind(const hap_gemm_problem* p) {
  if (p->act != HAP_ACT_NONE) return kGelu;
  if (p->dact != HAP_ACT_NONE) return kDact;
  return p->c_dtype == HAP_F32 ? kF32 : kPlain;
}

/* n 256-tiles.  A K tile of 64 takes 1.5 with all compute units at it (1.65 when both operands are K-contiguous), down to half with few;
 * prologue, epilogue and stores of a round 9.5, with GeLU and the pre-activation copy or with the activation backward 20.  fp32 outputs: 1.65
 * per K tile, 11.5 per round, 3.9 instead of 5.5 per launch.  Fewer tiles
 * than compute units, as the launcher splits K over the idle ones: 1.55 and 18 with the reduction (24 with
 * GeLU in it), 0.025 per partial tile (88 tiles over K = 16384, split in two: 199; 68 over 1402 in three: 35, with GeLU 43; 80 over 5312: 68). */
double us_256(const hap_gemm_problem* p, long long n, long long nk) {
  const long long cus = cu_count();
  const long long g = workgroup_splits(p, n, cus, nk, 4, 4 * kSmallTileBytes);
  const int e = epilogue_kind(p);
  if (g > 1) return (double)nk / (double)g * 1.55 + (e == kPlain || e == kF32 ? 18.0 : 24.0) + 0.025 * (double)(n * g);
  const double kt = (double)nk * ((p->a_kcontig && p->b_kcontig) || e == kF32 ? 1.65 : 1.5), round = e == kPlain ? 9.5 : (e == kF32 ? 11.5 : 20.0);
  const double rest = (double)(n % cus) / (double)cus;
  return (e == kF32 ? 3.9 : 5.5) + (double)(n / cus) * (kt + round) + (rest > 0.0 ? kt * (0.5 + 0.5 * rest) + round : 0.0);
}

/* Whether 128-tiles that do not run in gemm_kpair_kernel run in gemm_trio_kernel, and the estimated time either way.  n: tiles.  What
 * separates the two is the price of a workgroup: with three of them on a compute unit one's prologue and epilogue lie behind the others'
 * MFMAs; per K tile they are alike, or the two-workgroup kernel is ahead (both operands K-contiguous).  Up to two tiles per
 * compute unit are all under way at once in either kernel: over 280 such products three workgroups took 0.99 to 1.17 times as long (geometric
 * means by form and length, forward with GeLU of experts 1.04).  Microseconds, two -> three workgroups (2 x 64 KB of LDS against 3 x 48):
 *   forward 50432 x 315 over 1024 61 -> 54, with GeLU 79 -> 68; 50432 x 1024 over 315 74 -> 60, 112 -> 91
 *   bwd-data with the activation backward 17947 x 614 over 200 49.7 -> 30.7
 *   long contractions:  forward 16384 x 2731 over 2048 209 -> 199, bwd-data 16384 x 2048 over 2731 188 -> 231 */
bool trio_applies(const hap_gemm_problem* p, long long n, long long nk, double* us) {
  static const double four_fixed[4] = {3.0, 4.0, 4.5, 4.3}, four_tile[4] = {3.0, 5.7, 5.0, 3.25};      // by epilogue_kind()
  static const double trio_fixed[4] = {6.0, 7.0, 7.5, 0.0}, trio_tile[4] = {1.7, 4.1, 3.3, 0.0};        // (not built for fp32 outputs)
  const long long cus = cu_count();
  const int e = epilogue_kind(p);
  const bool kk = p->a_kcontig && p->b_kcontig;
  const long long g = workgroup_splits(p, n, 2 * cus, nk, 4, kSmallTileBytes);
  if (g > 1) {
    *us = (double)nk / (double)g * 1.05 + 5.0 + 3.0 + 0.00625 * (double)(n * g);
    return false;
  }
  // tiles that a compute unit works through, a lone one at 1.4 and 1.3 times its share of a full load
  const long long four_rest = cdiv(n % (2 * cus), cus), trio_rest = cdiv(n % (3 * cus), cus);
  const double four_load = 2.0 * (double)(n / (2 * cus)) + (four_rest == 1 ? 1.4 : (double)four_rest);
  const double trio_load = 3.0 * (double)(n / (3 * cus)) + (trio_rest == 1 ? 1.3 : (double)trio_rest);
  const double four = four_fixed[e] + four_load * (0.475 * (double)nk + four_tile[e]);
  const double trio = trio_fixed[e] + trio_load * ((kk ? 0.56 : 0.485) * (double)nk + trio_tile[e]);
  const bool built = p->c_dtype == HAP_BF16 && p->in_dtype == HAP_BF16 && (p->a_kcontig || !p->b_kcontig);
  const bool take = built && n > 2 * cus && nk <= kShortContraction && trio <= four;
  *us = take ? trio : four;
  return take;
}

/* The sub-problem of p over logical rows [m_lo, m_hi) and columns [n_lo, n_hi). */
hap_gemm_problem sub_problem(const hap_gemm_problem* p, int64_t m_lo, int64_t m_hi, int64_t n_lo, int64_t n_hi, int tile) {
  hap_gemm_problem q = *p;
  const int es = esize(p->in_dtype), ces = esize(p->c_dtype);
  q.M = m_hi - m_lo; q.N = n_hi - n_lo; q.tile = tile;
  for (int s = 0; s < p->nseg; ++s) {
    q.a[s] = static_cast<const char*>(p->a[s]) + (p->a_kcontig ? m_lo * p->lda : m_lo) * es;
    q.b[s] = static_cast<const char*>(p->b[s]) + (p->b_kcontig ? n_lo * p->ldb : n_lo) * es;
  }
  q.c = static_cast<char*>(p->c) + (m_lo * p->ldc + n_lo) * ces;
  if (p->preact) q.preact = static_cast<char*>(p->preact) + (m_lo * p->ldp + n_lo) * ces;
  if (p->dact_preact) q.dact_preact = static_cast<const char*>(p->dact_preact) + (m_lo * p->ldd + n_lo) * ces;
  if (p->bias) q.bias = static_cast<const char*>(p->bias) + n_lo * es;
  return q;
}

}  // namespace hap_gemm_detail

using namespace hap_gemm_detail;

static int64_t g_view_limit = kViewLimitBytes;
static int64_t g_cut_products = 0;      // products run in pieces so far (testing aid, not synchronised)

// Launches of gemm_kpair_kernel, gemm_small_kernel, gemm_trio_kernel and splitk_reduce_kernel so far (testing aid)
static int64_t g_kpair_products = 0, g_small_products = 0, g_trio_products = 0, g_split_products = 0;

extern "C" int64_t hap_debug_kpair_products(void) { return __atomic_load_n(&g_kpair_products, __ATOMIC_RELAXED); }
extern "C" int64_t hap_debug_small_products(void) { return __atomic_load_n(&g_small_products, __ATOMIC_RELAXED); }
extern "C" int64_t hap_debug_trio_products(void) { return __atomic_load_n(&g_trio_products, __ATOMIC_RELAXED); }
extern "C" int64_t hap_debug_split_products(void) { return __atomic_load_n(&g_split_products, __ATOMIC_RELAXED); }

/* Test hook (declared in hap_internal.h, not part of the public interface): lowers the reach at which operand views are
 * cut so the cutting can be exercised on small inputs; returns how many products have run in pieces so far. */
extern "C" int64_t hap_debug_set_gemm_view_limit(int64_t bytes) {
  g_view_limit = bytes > 0 && bytes < kViewLimitBytes ? bytes : kViewLimitBytes;
  return g_cut_products;
}

/* Operand views of 2 GiB and more.  The product is cut on the host so that every piece stays inside that reach:
 * a K-contiguous operand by rows (row or column blocks of C, one launch each), an M- / N-contiguous operand, whose
 * rows are k, along the contraction (more segments of the same launch; cuts at multiples of 64 keep every piece's
 * 16-byte phase).  Returns true if it ran the product (status in *rc), false if nothing needs cutting or a cut is
 * not possible (more than HAP_GEMM_MAX_SEG pieces, unaligned leading dimensions): the caller goes on as before. */
static bool run_large(const hap_gemm_problem* p, void* stream, int* rc) {
  const int es = esize(p->in_dtype);
  if ((p->lda * es) % 16 || (p->ldb * es) % 16) return false;
  const double limit = (double)g_view_limit / es;       // elements
  const int64_t slack = 16;                              // skew and chunk rounding
  int64_t kmax = 0;
  for (int s = 0; s < p->nseg; ++s) kmax = p->k[s] > kmax ? p->k[s] : kmax;
  // rows r of pitch ld and width w with ((r - 1) * ld + w + slack) elements inside the reach
  auto rows_fit = [&](int64_t ld, int64_t w, int64_t granule) -> int64_t {
    const double r = (limit - (double)(w + slack)) / (double)ld;
    return r < (double)granule ? 0 : (int64_t)(r / granule) * granule;
  };
  auto too_big = [&](int64_t rows, int64_t ld, int64_t w) { return (double)(rows - 1) * ld + w + slack >= limit; };
  if (p->a_kcontig && too_big(p->M, p->lda, kmax)) {
    const int64_t r = rows_fit(p->lda, kmax, 256);
    if (r == 0) return false;
    ++g_cut_products;
    for (int64_t lo = 0; lo < p->M; lo += r) {
      const hap_gemm_problem q = sub_problem(p, lo, lo + r < p->M ? lo + r : p->M, 0, p->N, p->tile);
      if ((*rc = hap_gemm_run(&q, stream))) return true;
    }
    *rc = HAP_OK;
    return true;
  }
  if (p->b_kcontig && too_big(p->N, p->ldb, kmax)) {
    const int64_t r = rows_fit(p->ldb, kmax, 256);
    if (r == 0) return false;
    ++g_cut_products;
    for (int64_t lo = 0; lo < p->N; lo += r) {
      const hap_gemm_problem q = sub_problem(p, 0, p->M, lo, lo + r < p->N ? lo + r : p->N, p->tile);
      if ((*rc = hap_gemm_run(&q, stream))) return true;
    }
    *rc = HAP_OK;
    return true;
  }
  bool cut = false;
  for (int s = 0; s < p->nseg; ++s)
    cut = cut || (!p->a_kcontig && too_big(p->k[s], p->lda, p->M)) || (!p->b_kcontig && too_big(p->k[s], p->ldb, p->N));
  if (!cut) return false;
  int64_t piece = INT64_MAX;
  if (!p->a_kcontig) piece = rows_fit(p->lda, p->M, 64);
  if (!p->b_kcontig) { const int64_t r = rows_fit(p->ldb, p->N, 64); piece = r < piece ? r : piece; }
  if (piece == 0) return false;
  hap_gemm_problem q = *p;
  q.nseg = 0;
  for (int s = 0; s < p->nseg; ++s)
    for (int64_t k0 = 0; k0 < p->k[s]; k0 += piece) {
      if (q.nseg == HAP_GEMM_MAX_SEG) return false;
      q.a[q.nseg] = static_cast<const char*>(p->a[s]) + (p->a_kcontig ? k0 : k0 * p->lda) * es;
      q.b[q.nseg] = static_cast<const char*>(p->b[s]) + (p->b_kcontig ? k0 : k0 * p->ldb) * es;
      q.k[q.nseg] = p->k[s] - k0 < piece ? p->k[s] - k0 : piece;
      ++q.nseg;
    }
  if (q.nseg == 0) return false;
  ++g_cut_products;
  *rc = hap_gemm_run(&q, stream);
  return true;
}

/* 256x256 tiles on 256 CUs quantise badly: 33 tile columns of 32 rows are 4.1 rounds of work that take
 * 5.  The engine therefore cuts the output into a part whose big tiles fill whole rounds and a
 * remainder strip computed with 128x128 tiles (or 256-tiles whose K range is split over the idle compute units), when its cost model says
 * that is faster: the sum of two launches, each with its fixed part. */
static int run_auto_tiled(const hap_gemm_problem* p, const Plan& pl, void* stream) {
  const int kCUs = cu_count();
  const long long Mp = p->M + pl.skewM, Np = p->N + pl.skewN;
  const long long tm = cdiv(Mp, 256), tn = cdiv(Np, 256);
  const long long sm = cdiv(Mp, 128), sn = cdiv(Np, 128);
  long long nk = 0;                 // K tiles of the contraction
  for (int s = 0; s < p->nseg; ++s) nk += p->k[s] > 0 ? cdiv(pl.skewK + p->k[s], 64) : 0;
  // Time of n 256-tiles, and of a part that may run on either tile: microseconds for short contractions, rounds of 256-tiles for long ones.
  const bool is_short = nk <= kShortContraction;
  auto us_128 = [&](long long n) {
    double us;
    trio_applies(p, n, nk, &us);
    if (kpair_applies(p, n, nk)) {     // (where it applies, it is at least as fast as the 4-wave kernel)
      double pair;
      kpair_splits(p, n, nk, &pair);
      if (pair < us || nk > 128) us = pair;
    }
    return us;
  };
  // A part of few big tiles over a long contraction: 128-tiles (two per CU) or 256-tiles, either with the K range split over
  // the idle slots as the launcher will do it.  Measured on this chip (microseconds): a workgroup spends 2.0 per K tile
  // on a 256-tile and 1.05 on a 128-tile that shares its CU, plus 7 / 5 for prologue and epilogue; a split costs 3 for
  // the reduction launch and 0.025 / 0.00625 per partial tile written and read back.
  auto few_tiles_us = [&](long long tiles, long long slots, size_t tile_bytes, double per_ktile, double fixed, double per_partial) {
    const long long g = workgroup_splits(p, tiles, slots, nk, 4, tile_bytes);
    const double rounds = (double)cdiv(tiles * g, slots);
    return rounds * ((double)nk / (double)g * per_ktile + fixed) + (g > 1 ? 3.0 + (double)(tiles * g) * per_partial : 0.0);
  };
  const double round_us = (double)nk * 2.0 + 7.0;
  auto big_time = [&](long long n) { return is_short ? us_256(p, n, nk) : (double)cdiv(n, kCUs); };
  auto part_time = [&](long long big_tiles, long long small_tiles, int* tile) {
    double tb, ts;
    if (is_short) {
      tb = us_256(p, big_tiles, nk);
      ts = us_128(small_tiles);
    } else if (big_tiles < kCUs) {
      tb = few_tiles_us(big_tiles, kCUs, 4 * kSmallTileBytes, 2.0, 7.0, 0.025) / round_us;
      ts = few_tiles_us(small_tiles, 2 * kCUs, kSmallTileBytes, 1.05, 5.0, 0.00625);
      if (kpair_applies(p, small_tiles, nk)) {
        double pair;
        kpair_splits(p, small_tiles, nk, &pair);
        if (pair < ts || nk > 128) ts = pair;
      }
      ts /= round_us;
    } else {
      tb = (double)cdiv(big_tiles, kCUs);
      ts = small_tiles_time(small_tiles);
    }
    *tile = tb <= ts ? 256 : 128;
    return tb <= ts ? tb : ts;
  };
  int strip_tile = 128, whole_tile;
  double best = part_time(tm * tn, sm * sn, &whole_tile);
  int choice = whole_tile == 128 ? 1 : 0;       // 0: all big, 1: all small, 2: split columns, 3: split rows
  long long cut = 0;
  // a plan of two launches pays for the second one: the strip starts when the last big tile has finished (~10 us; part of every
  // estimate in microseconds)
  const double second_launch = is_short ? 0.0 : 10.0 / round_us;
  for (long long c = tn - 1; c >= 1; --c)
    if ((tm * c) % kCUs == 0) {
      int tl;
      const double t = big_time(tm * c) + part_time(tm * (tn - c), sm * cdiv(Np - c * 256, 128), &tl) + second_launch;
      if (t < best - 1e-9) { best = t; choice = 2; cut = c; strip_tile = tl; }
      break;
    }
  for (long long r = tm - 1; r >= 1; --r)
    if ((tn * r) % kCUs == 0) {
      int tl;
      const double t = big_time(tn * r) + part_time(tn * (tm - r), sn * cdiv(Mp - r * 256, 128), &tl) + second_launch;
      if (t < best - 1e-9) { best = t; choice = 3; cut = r; strip_tile = tl; }
      break;
    }
  hap_gemm_problem q;
  int rc;
  switch (choice) {
    case 1:
      q = sub_problem(p, 0, p->M, 0, p->N, 128);
      return hap_gemm_run(&q, stream);
    case 2: {
      const int64_t n_cut = cut * 256 - pl.skewN;
      q = sub_problem(p, 0, p->M, 0, n_cut, 256);
      if ((rc = hap_gemm_run(&q, stream))) return rc;
      q = sub_problem(p, 0, p->M, n_cut, p->N, strip_tile);
      return hap_gemm_run(&q, stream);
    }
    case 3: {
      const int64_t m_cut = cut * 256 - pl.skewM;
      q = sub_problem(p, 0, m_cut, 0, p->N, 256);
      if ((rc = hap_gemm_run(&q, stream))) return rc;
      q = sub_problem(p, m_cut, p->M, 0, p->N, strip_tile);
      return hap_gemm_run(&q, stream);
    }
    default:
      q = sub_problem(p, 0, p->M, 0, p->N, 256);
      return hap_gemm_run(&q, stream);
  }
}

static SkinnyArgs skinny_args(const hap_gemm_problem* p) {
  SkinnyArgs g;
  g.M = (int)p->M; g.N = (int)p->N; g.K = (int)p->k[0];
  g.lda = p->lda; g.ldb = p->ldb; g.ldc = p->ldc; g.ldp = p->ldp;
  g.a = static_cast<const float*>(p->a[0]); g.b = static_cast<const float*>(p->b[0]);
  g.c = static_cast<float*>(p->c); g.preact = static_cast<float*>(p->preact); g.bias = static_cast<const float*>(p->bias);
  g.act = p->act; g.accumulate = p->accumulate;
  return g;
}

static RankArgs rank_args(const hap_gemm_problem* p, float* colsum) {
  RankArgs g;
  g.M = (int)p->M; g.N = (int)p->N; g.accumulate = p->accumulate;
  g.lda = p->lda; g.ldb = p->ldb; g.ldc = p->ldc;
  g.c = static_cast<float*>(p->c); g.colsum = colsum;
  g.tiles_n = (int)cdiv(p->N, 64);
  g.nseg = 0;
  for (int s = 0; s < p->nseg; ++s) {
    if (p->k[s] <= 0) continue;
    g.a[g.nseg] = static_cast<const float*>(p->a[s]); g.b[g.nseg] = static_cast<const float*>(p->b[s]); g.k[g.nseg] = (int)p->k[s];
    ++g.nseg;
  }
  return g;
}

static int run_rank_f32(const RankArgs& g, hipStream_t st) {
  const dim3 grid((unsigned)(cdiv(g.M, 64) * g.tiles_n));
  // (enough tiles to give every SIMD four waves: one wave each takes a whole tile, 2048 x 2048 over 64: 15.6 -> 11.6 us)
  if (grid.x > 2u * cu_count()) hipLaunchKernelGGL(gemm_rank_f32_kernel<1>, grid, dim3(256), 0, st, g);
  else hipLaunchKernelGGL(gemm_rank_f32_kernel<4>, grid, dim3(1024), 0, st, g);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? HAP_OK : hap_fail(HAP_EDEVICE, "fp32 few-k gemm launch: %s", hipGetErrorString(e));
}

/* Whether two fp32 matrices (rows of `cols` elements, ld apart) share addresses; NULL or empty ones do not. */
static bool overlap_f32(const void* a, int64_t rows_a, int64_t cols_a, int64_t lda, const void* b, int64_t rows_b, int64_t cols_b, int64_t ldb) {
  if (!a || !b || rows_a <= 0 || cols_a <= 0 || rows_b <= 0 || cols_b <= 0) return false;
  const char *pa = static_cast<const char*>(a), *pb = static_cast<const char*>(b);
  return pa < pb + ((rows_b - 1) * ldb + cols_b) * 4 && pb < pa + ((rows_a - 1) * lda + cols_a) * 4;
}

int hap_gemm_run_bwd_f32(const hap_gemm_problem* dx, const hap_gemm_problem* dw, float* dbias, int* taken, void* stream) {
  *taken = 0;
  look_up_cu_count();
  if (!rank_f32_applies(dw)) return HAP_OK;
  {
    // The products apart run one after the other, so that one may write where an earlier one has read; together they must not.
    const int64_t tokens = dw->k[0], in = dw->M, out = dw->N;
    const struct { const void* p; int64_t rows, cols, ld; } input[3] = {{dw->a[0], tokens, in, dw->lda}, {dw->b[0], tokens, out, dw->ldb},
                                                                        {dx ? dx->b[0] : nullptr, in, out, dx ? dx->ldb : 0}},
        output[3] = {{dw->c, in, out, dw->ldc}, {dbias, 1, out, out}, {dx ? dx->c : nullptr, tokens, in, dx ? dx->ldc : 0}};
    for (int o = 0; o < 3; ++o) {
      for (int i = 0; i < 3; ++i)
        if (overlap_f32(output[o].p, output[o].rows, output[o].cols, output[o].ld, input[i].p, input[i].rows, input[i].cols, input[i].ld)) return HAP_OK;
      for (int i = 0; i < o; ++i)
        if (overlap_f32(output[o].p, output[o].rows, output[o].cols, output[o].ld, output[i].p, output[i].rows, output[i].cols, output[i].ld)) return HAP_OK;
    }
  }
  hipStream_t st = static_cast<hipStream_t>(stream);
  const RankArgs w = rank_args(dw, dbias);
  *taken = 1;
  if (dx && dx->M > 0 && dx->N > 0 && dw->k[0] <= kUnfoldedK && skinny_f32_row_blocks(dx) == 1) {
    const long long nrank = cdiv(dw->M, 64) * w.tiles_n, nx = cdiv(dx->N, 16), rows = cdiv(dx->M, 16);
    // (workgroups that the chip holds at once; twice as many over short contractions: 200 rows x 512 x 512 18.7 us apart, 9.1 together,
    // 400 x 512 x 512 21.3 and 13.6; over k = 1024 100 x 1024 x 1024 15.1 and 15.6.  38 x 1024 x 1024: 11.0 and 8.0.)
    if (nrank + nx * rows <= (dx->k[0] <= 512 ? 4 : 2) * cu_count()) {
      hipLaunchKernelGGL(linear_bwd_f32_kernel, dim3((unsigned)(nrank + nx * rows)), dim3(1024), 0, st, w, skinny_args(dx), (int)nrank, (int)nx);
      const hipError_t e = hipGetLastError();
      return e == hipSuccess ? HAP_OK : hap_fail(HAP_EDEVICE, "fp32 layer backward launch: %s", hipGetErrorString(e));
    }
  }
  if (dx) { const int rc = hap_gemm_run(dx, stream); if (rc) return rc; }
  return run_rank_f32(w, st);
}

int hap_gemm_run(const hap_gemm_problem* p, void* stream) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (p->M <= 0 || p->N <= 0) return HAP_OK;
  look_up_cu_count();
  if (p->M > 0x7fffffff || p->N > 0x7fffffff) return hap_fail(HAP_EUNSUPPORTED, "GEMM extent exceeds 2^31");
  if (p->accumulate && p->c_dtype != HAP_F32) return hap_fail(HAP_EINVAL, "accumulate needs an fp32 output");
  if (p->in_dtype == HAP_F32 && p->c_dtype != HAP_F32) return hap_fail(HAP_EUNSUPPORTED, "fp32 inputs need fp32 output");
  if (p->dact != HAP_ACT_NONE) {
    if (p->dact != HAP_ACT_GELU_ERF || !p->dact_preact) return hap_fail(HAP_EINVAL, "bad activation backward in the epilogue (dact %d)", p->dact);
    if (p->act != HAP_ACT_NONE || p->accumulate || p->preact || p->bias)
      return hap_fail(HAP_EINVAL, "an epilogue with an activation backward has no bias, activation, pre-activation copy or accumulation");
  }
  const int es = esize(p->in_dtype), ces_out = esize(p->c_dtype);
  const int groups = p->groups > 1 ? p->groups : 1;
  const bool grouped = groups > 1 || p->group_len;
  if (grouped) {
    if (p->nseg != 1) return hap_fail(HAP_EINVAL, "a grouped product has one contracted segment");
    if (groups > 65535) return hap_fail(HAP_EUNSUPPORTED, "more than 65535 groups");
    if (p->group_len && p->group_ragged != 1 && p->group_ragged != 2) return hap_fail(HAP_EINVAL, "group_len needs group_ragged 1 or 2");
    if (p->k[0] > 0x7fffffff) return hap_fail(HAP_EUNSUPPORTED, "segment longer than 2^31");
  }
  const int ragged = p->group_len ? p->group_ragged : 0;
  if (!grouped && !p->force_generic) {
    int rc;
    if (run_large(p, stream, &rc)) return rc;
  }
  if (rank_f32_applies(p)) return run_rank_f32(rank_args(p, nullptr), st);
  if (const int row_blocks = skinny_f32_row_blocks(p)) {
    const SkinnyArgs g = skinny_args(p);
    const unsigned nb = (unsigned)((p->N + 15) / 16), rb = (unsigned)((p->M + 15) / 16);
    if (row_blocks == 1) {
      if (p->b_kcontig) hipLaunchKernelGGL((gemm_skinny_f32_kernel<true, 1>), dim3(nb, rb), dim3(1024), 0, st, g);
      else hipLaunchKernelGGL((gemm_skinny_f32_kernel<false, 1>), dim3(nb, rb), dim3(1024), 0, st, g);
    } else if (p->b_kcontig) hipLaunchKernelGGL((gemm_skinny_f32_kernel<true, 4>), dim3(nb), dim3(1024), 0, st, g);
    else hipLaunchKernelGGL((gemm_skinny_f32_kernel<false, 4>), dim3(nb), dim3(1024), 0, st, g);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hap_fail(HAP_EDEVICE, "skinny fp32 gemm launch: %s", hipGetErrorString(e));
    return HAP_OK;
  }
  const Plan pl = make_plan(p);
  if (pl.tiled && pl.dma && p->tile == 0 && pl.bm == 256 && !grouped) return run_auto_tiled(p, pl, stream);

  if (!pl.tiled) {
    GenericArgs g;
    g.M = (int)p->M; g.N = (int)p->N; g.nseg = 0;
    g.lda = p->lda; g.ldb = p->ldb; g.ldc = p->ldc; g.ldp = p->ldp;
    g.a_kcontig = p->a_kcontig; g.b_kcontig = p->b_kcontig;
    g.c = p->c; g.preact = p->preact; g.bias = p->bias; g.act = p->act; g.accumulate = p->accumulate;
    g.dact_preact = p->dact ? p->dact_preact : nullptr; g.ldd = p->ldd;
    g.ragged = ragged; g.group_len = p->group_len;
    g.ga = p->ga * es; g.gb = p->gb * es; g.gc = p->gc * ces_out; g.gp = p->gp * ces_out; g.gbias = p->gbias * es; g.gd = p->gd * ces_out;
    for (int s = 0; s < p->nseg; ++s) {
      if (p->k[s] <= 0) continue;
      if (p->k[s] > 0x7fffffff) return hap_fail(HAP_EUNSUPPORTED, "segment longer than 2^31");
      g.a[g.nseg] = p->a[s]; g.b[g.nseg] = p->b[s]; g.k[g.nseg] = (int)p->k[s]; ++g.nseg;
    }
    dim3 grid((unsigned)((p->N + 15) / 16), (unsigned)((p->M + 15) / 16), (unsigned)groups);
    if (grid.y > 65535u) return hap_fail(HAP_EUNSUPPORTED, "generic GEMM fallback: too many rows");
    if (p->in_dtype == HAP_BF16 && p->c_dtype == HAP_BF16) hipLaunchKernelGGL((gemm_generic_kernel<__bf16, __bf16>), grid, dim3(256), 0, st, g);
    else if (p->in_dtype == HAP_BF16) hipLaunchKernelGGL((gemm_generic_kernel<__bf16, float>), grid, dim3(256), 0, st, g);
    else hipLaunchKernelGGL((gemm_generic_kernel<float, float>), grid, dim3(256), 0, st, g);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hap_fail(HAP_EDEVICE, "generic gemm launch: %s", hipGetErrorString(e));
    return HAP_OK;
  }

  GemmArgs a;
  a.M = (int)p->M; a.N = (int)p->N;
  a.skewM = pl.skewM; a.skewN = pl.skewN; a.skewK = pl.skewK;
  a.lda = p->lda; a.ldb = p->ldb; a.ldc = p->ldc; a.ldp = p->ldp;
  a.c = p->c; a.preact = p->preact; a.bias = p->bias; a.act = p->act; a.accumulate = p->accumulate;
  a.dact_preact = p->dact ? p->dact_preact : nullptr; a.ldd = p->ldd;
  a.ragged = ragged; a.group_len = p->group_len;
  a.ga = p->ga * es; a.gb = p->gb * es; a.gc = p->gc * ces_out; a.gp = p->gp * ces_out; a.gbias = p->gbias * es; a.gd = p->gd * ces_out;
  a.tiles_m = (int)((p->M + pl.skewM + pl.bm - 1) / pl.bm);
  a.tiles_n = (int)((p->N + pl.skewN + pl.bn - 1) / pl.bn);
  a.nseg = 0;
  for (int s = 0; s < p->nseg; ++s) {
    if (p->k[s] <= 0) continue;
    SegArg& sg = a.seg[a.nseg++];
    const int skew_a = p->a_kcontig ? pl.skewK : pl.skewM, skew_b = p->b_kcontig ? pl.skewK : pl.skewN;
    sg.a = static_cast<const char*>(p->a[s]) - (size_t)skew_a * es;
    sg.b = static_cast<const char*>(p->b[s]) - (size_t)skew_b * es;
    sg.k = (int)p->k[s];
    const long long ea = p->a_kcontig ? ((p->M - 1) * p->lda + pl.skewK + p->k[s]) : ((p->k[s] - 1) * p->lda + pl.skewM + p->M);
    const long long eb = p->b_kcontig ? ((p->N - 1) * p->ldb + pl.skewK + p->k[s]) : ((p->k[s] - 1) * p->ldb + pl.skewN + p->N);
    // Extents are rounded up to whole 16-byte chunks: the hardware range check works per dword, and
    // a chunk that starts inside the view must come back whole (its tail is discarded by the kernel).
    // An aligned chunk never crosses a page, so the bytes past the view are still mapped memory.
    sg.a_bytes = (unsigned)((ea * es + 15) / 16 * 16);
    sg.b_bytes = (unsigned)((eb * es + 15) / 16 * 16);
    sg.pad = 0;
  }
  if (a.nseg == 0) {   // empty contraction: the product is zero; run one empty segment so the epilogue still applies
    a.nseg = 1;
    a.seg[0].a = p->c; a.seg[0].b = p->c; a.seg[0].k = 0; a.seg[0].a_bytes = 0; a.seg[0].b_bytes = 0; a.seg[0].pad = 0;
  }
  {
    // Whole-chunk stores need rows of C (and of the pre-activation copy, with C's phase) that start on the same 16-byte phase;
    // the phase itself is arbitrary: cdelta shifts the tile inside the store patch onto C's chunk grid.
    const int ces = esize(p->c_dtype), cepc = 16 / ces;
    a.vec_store = ((uintptr_t)p->c % ces) == 0 && p->ldc % cepc == 0 &&
                  (!p->preact || (((uintptr_t)p->preact % 16) == ((uintptr_t)p->c % 16) && p->ldp % cepc == 0)) &&
                  (groups == 1 || (p->gc % cepc == 0 && (!p->preact || p->gp % cepc == 0))) &&
                  (!(p->dact && p->dact_preact) || (((uintptr_t)p->dact_preact % 16) == ((uintptr_t)p->c % 16) && p->ldd % cepc == 0 &&
                                                    (groups == 1 || p->gd % cepc == 0)));
    const int skew_c = (int)(((uintptr_t)p->c % 16) / ces);       // columns of C's 16-byte chunk that precede logical column 0
    a.cdelta = a.vec_store ? ((skew_c - pl.skewN) % cepc + cepc) % cepc : 0;
  }
  a.ntiles = 0;
  a.kpair = 0;
  a.ksplit = 1;
  a.partial = nullptr;
  {
    const int bk = pl.bk;                // the chosen kernel's K step
    for (int s = 0; s < a.nseg; ++s) a.ntiles += (pl.skewK + a.seg[s].k + bk - 1) / bk;
    if (a.ntiles == 0) a.ntiles = 1;     // empty contraction still runs one (all-zero) tile
  }
  if (pl.dma || p->in_dtype == HAP_F32) {
    // Split-K when the output tiles cannot occupy the chip: spread each tile's K range over the idle CUs,
    // keeping at least 4 K tiles per workgroup (2 for the small fp32 tiles, whose loop is bound by one load
    // latency per tile), as far as the caller's workspace allows.
    const long long out_tiles = (long long)a.tiles_m * a.tiles_n * groups;
    const int kCUs = cu_count();
    const long long slots = pl.bm == 256 ? kCUs : (pl.bm == 128 ? 2 * kCUs : 4 * kCUs);
    const int min_tiles = pl.bm == 64 ? 2 : 4 * (64 / pl.bk);      // in K steps of the chosen kernel
    a.ksplit = pl.small ? 1 : (int)workgroup_splits(p, out_tiles, slots, a.ntiles, min_tiles, (size_t)pl.bm * pl.bn * sizeof(float));
    if (pl.small) __atomic_fetch_add(&g_small_products, 1, __ATOMIC_RELAXED);
    if (pl.dma && pl.bm == 128 && kpair_applies(p, out_tiles, a.ntiles)) {
      double us;
      a.kpair = 1;
      __atomic_fetch_add(&g_kpair_products, 1, __ATOMIC_RELAXED);
      a.ksplit = kpair_splits(p, out_tiles, a.ntiles, &us);
    }
    double us;
    if (pl.dma && pl.bm == 128 && !a.kpair && trio_applies(p, out_tiles, a.ntiles, &us)) {
      a.ntiles = 0;                      // its K step is 32
      for (int s = 0; s < a.nseg; ++s) a.ntiles += (pl.skewK + a.seg[s].k + 31) / 32;
      if (a.ntiles == 0) a.ntiles = 1;
      __atomic_fetch_add(&g_trio_products, 1, __ATOMIC_RELAXED);
      return run_trio(p, a, groups, st);
    }
    if (a.ksplit > 1) {
      a.partial = static_cast<float*>(p->ws);
      __atomic_fetch_add(&g_split_products, 1, __ATOMIC_RELAXED);
    }
  }
  if (p->in_dtype == HAP_BF16 && p->c_dtype == HAP_BF16) return dispatch_tile<__bf16, __bf16>(p, pl, a, groups, st);
  if (p->in_dtype == HAP_BF16) return dispatch_tile<__bf16, float>(p, pl, a, groups, st);
  return dispatch_tile<float, float>(p, pl, a, groups, st);
}
