/*
 * Data movement of an All-Gather over unevenly sharded tensors, as one device performs it
 * (Sec. 2.2; Sec. 2.3.1 and Fig. "comm_opt": padded All-Gather vs grouped Broadcast).
 *
 * Both layouts end with the same step: piece j (a padded slot, or the shard at its own size) is
 * copied to its range of the sharded axis of the full tensor.  All m pieces move in ONE launch:
 * blockIdx.y is the piece, the blocks of a piece stride over its rows x 16-byte chunks.  Shard sizes
 * are arbitrary integers, so nothing is assumed about alignment (see the kernel).
 * "Pad" (shard -> front of the device's send slot) is the same copy with a single piece.
 * A Reduce-Scatter over uneven shards needs equal pieces as well (Sec. 2.3.1): there the device cuts
 * its full partial tensor into m capacity-sized slots, shard range first, zeros behind.
 */
#include <hip/hip_runtime.h>

#include <stdint.h>

#include "hap_internal.h"
#include "hap_move.h"

namespace {

constexpr int kMaxPieces = HAP_SFB_MAX_DEVICES;

struct PieceArgs {
  int m;
  char* out;
  long long ld_out;                  // bytes
  const char* src[kMaxPieces];
  long long ld_src[kMaxPieces];      // bytes
  long long dst_off[kMaxPieces];     // bytes from out to the piece's first element
  long long rows[kMaxPieces];
  long long width[kMaxPieces];       // valid bytes per row
};

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

/* One row range of a piece: rows x width bytes of dst, of which the first vrows x vwidth come from src and the rest is zeros. */
struct Move {
  const char* src;
  char* dst;
  long long lds, ldd;                // bytes
  long long rows, width, vrows, vwidth;
};

/* 16-byte chunks of the destination's rows, aligned in the DESTINATION's address space: whole chunks are written with one aligned 16-byte
 * store and read from wherever the source happens to lie (global loads need no alignment on this target); chunks that straddle the
 * row's ends or the shard's edge go unit by unit (UNIT: 4, 2 or 1 bytes, whatever all addresses are
 * multiples of).  A row has at most (width + 30) / 16 chunks: width / 16 rounded up where all rows start on one, and where
 * only some do, these leave the last index empty.
 * Bound: HBM.  A workgroup moves 256 * UNROLL consecutive chunks of the piece, row after row; a thread has UNROLL loads in flight before its
 * first store and finds its row with a reciprocal.  STREAM: non-temporal stores (see streamed()).
 * One chunk per thread in small moves (2000 x 1333 bf16: two 1 us slower, four 3 us) and in moves of row shards; streamed moves of column
 * shards, whose rows are shorter and end in cut chunks, take two, and four where a full tensor is cut into slots.  Microseconds with one / two / four,
 * buffers not touched since 1.6 GB ago (in brackets one chunk, a 64-bit division each, edges byte after byte and plain stores):
 *   assemble  8192 x 16384 in three column shards 100 / 102 / 110 (107)    100000 x 1024 113 / 98 / 103 (125)    row shards of 16384 x 8192 84 / 88 / 92 (92)
 *   split     8192 x 16384 in three column slots 130 / 130 / 132 (164)     100000 x 1024 155 / 126 / 124 (233)    60000 x 1500 155 / 134 / 120 (238)
 *             row slots of 16384 x 8192 101 / 103 / 107 (114), of 60000 x 1500 86 / 97 / 106 (103) */
template <int UNROLL, bool STREAM, typename UNIT>
__device__ __forceinline__ void move_rows(const Move& m) {
  const bool aligned = ((reinterpret_cast<uintptr_t>(m.dst) | (uintptr_t)m.ldd) & 15) == 0;
  const hap_move::Walk w = hap_move::walk_of(m.rows, m.width, aligned);
  const long long nch = w.per_row, total = w.total, span = (long long)gridDim.x * (256 * UNROLL);
  const double inv = 1.0 / (double)nch;
  for (long long base = (long long)blockIdx.x * (256 * UNROLL) + threadIdx.x; base < total; base += span) {
    u32x4 v[UNROLL];
    long long row[UNROLL], lo[UNROLL];
    bool whole[UNROLL];               // a whole chunk, of data or of zeros; else units or nothing
    // row and chunk of the linear index: the quotient from a reciprocal is off by one at most (total < 2^52)
    long long r = (long long)((double)base * inv), k = base - r * nch;
    if (k < 0) { --r; k += nch; }
    if (k >= nch) { ++r; k -= nch; }
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      if (u > 0) {
        r += w.over; k += w.step;
        if (k >= nch) { ++r; k -= nch; }
      }
      const long long i = base + u * 256;
      row[u] = r;
      lo[u] = 16 * k - (long long)(reinterpret_cast<uintptr_t>(m.dst + r * m.ldd) & 15);       // first byte of the chunk within the row
      const long long hi = lo[u] + 16;
      const bool data = r < m.vrows && hi <= m.vwidth, zeros = r >= m.vrows || lo[u] >= m.vwidth;
      whole[u] = i < total && lo[u] >= 0 && hi <= m.width && (data || zeros);
      v[u] = u32x4{0u, 0u, 0u, 0u};
      if (whole[u] && data) __builtin_memcpy(&v[u], m.src + r * m.lds + lo[u], 16);
    }
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      if (base + u * 256 >= total) continue;
      const long long r = row[u], at = lo[u];
      char* const drow = m.dst + r * m.ldd;
      if (whole[u]) {
        if constexpr (STREAM) __builtin_nontemporal_store(v[u], reinterpret_cast<u32x4*>(drow + at));
        else *reinterpret_cast<u32x4*>(drow + at) = v[u];
      } else {
        // all units are fetched before the first is stored: one trip to memory instead of up to sixteen
        constexpr int N = 16 / (int)sizeof(UNIT);
        const hap_move::Units c = hap_move::units_of(at, m.width, r < m.vrows ? m.vwidth : 0, (int)sizeof(UNIT));
        const UNIT* const sp = reinterpret_cast<const UNIT*>(m.src + r * m.lds + at);           // dereferenced inside the shard only
        UNIT* const dp = reinterpret_cast<UNIT*>(drow + at);
        UNIT unit[N];
#pragma unroll
        for (int x = 0; x < N; ++x) {
          unit[x] = 0;
          if (x >= c.first && x < c.data) unit[x] = sp[x];
        }
#pragma unroll
        for (int x = 0; x < N; ++x)
          if (x >= c.first && x < c.last) dp[x] = unit[x];
      }
    }
  }
}

template <int UNROLL, bool STREAM, typename UNIT>
__global__ __launch_bounds__(256) void copy_pieces_kernel(const PieceArgs a) {
  const int j = blockIdx.y;
  move_rows<UNROLL, STREAM, UNIT>({a.src[j], a.out + a.dst_off[j], a.ld_src[j], a.ld_out, a.rows[j], a.width[j], a.rows[j], a.width[j]});
}

/* f(value of the widest unit type that every address is a multiple of) */
template <typename F>
void with_unit(uintptr_t phases, F&& f) {
  if (phases % 4 == 0) f(uint32_t());
  else if (phases % 2 == 0) f(uint16_t());
  else f(uint8_t());
}

/* Whether a launch that writes `bytes` in all stores non-temporally: from 72 MB on.  Below, whoever reads the result next
 * finds it in the caches, and what the stores save is less than what the reader loses; beyond, little of it would still be there.
 * Microseconds, plain -> non-temporal, buffers not touched since 1.6 GB ago, with a copy of the result behind the move (without it):
 *   assemble:  30 MB 27.3 -> 30.4 (19.5 -> 18.1)    53 MB 42.1 -> 46.5 (28.3 -> 26.5)    78 MB 70.1 -> 66.5 (40.1 -> 38.0)    128 MB 120.2 -> 106.0 (56.9 -> 52.2)
 *   split:     47 MB 36.4 -> 40.2 (25.4 -> 22.4)    70 MB 54.2 -> 56.1 (34.7 -> 30.7)    82 MB 66.7 -> 63.2 (37.1 -> 33.4)    197 MB 169.3 -> 153.6 (84.1 -> 74.5)
 *   pad:       36 MB 25.1 -> 29.2 (16.1 -> 14.9)    66 MB 47.7 -> 52.1 (30.0 -> 27.8)    80 MB 64.0 -> 61.6 (34.9 -> 32.2)    131 MB 112.7 -> 106.6 (52.8 -> 49.8)
 * Pad, assemble and split of one tensor in turn, 26 of 40 to 160 MB, the line at 72 / 128 MB: 3 x 102 MB of columns 104.5 / 120.2, 4 x 90 MB of columns
 * 90.6 / 113.5, 5 x 72 MB of rows 73.4 / 81.8; none is slower with 72, whether a pass repeats on its buffers or goes around three sets of them.
 * Past the last-level cache the two are alike with a reader (assemble 256 MB 213.0 -> 213.9, 500 MB 415.0 -> 416.5), without one the gain stays (110.1 -> 100.6). */
inline bool streamed(long long bytes) { return bytes >= (72LL << 20); }

inline dim3 move_grid(long long chunks, int unroll, int pieces) {
  long long gx = (chunks + 256 * unroll - 1) / (256 * unroll);
  if (gx > 256 * 32) gx = 256 * 32;        // grid-stride beyond 32 blocks per CU and piece
  return dim3((unsigned)gx, (unsigned)pieces);
}

/* columns: the pieces are column ranges. */
int launch_pieces(const PieceArgs& a, bool columns, hipStream_t s) {
  long long most = 0, bytes = 0;
  uintptr_t phases = (uintptr_t)a.out | (uintptr_t)a.ld_out;       // its lowest bits: what every address is a multiple of
  for (int j = 0; j < a.m; ++j) {
    if (a.rows[j] <= 0 || a.width[j] <= 0) continue;
    phases |= (uintptr_t)a.src[j] | (uintptr_t)a.ld_src[j] | (uintptr_t)a.dst_off[j] | (uintptr_t)a.width[j];
    const long long chunks = a.rows[j] * ((a.width[j] + 30) / 16);
    most = chunks > most ? chunks : most;
    bytes += a.rows[j] * a.width[j];
  }
  if (most == 0) return HAP_OK;
  with_unit(phases, [&](auto unit) {
    using U = decltype(unit);
    if (!streamed(bytes)) hipLaunchKernelGGL((copy_pieces_kernel<1, false, U>), move_grid(most, 1, a.m), dim3(256), 0, s, a);
    else if (columns) hipLaunchKernelGGL((copy_pieces_kernel<2, true, U>), move_grid(most, 2, a.m), dim3(256), 0, s, a);
    else hipLaunchKernelGGL((copy_pieces_kernel<1, true, U>), move_grid(most, 1, a.m), dim3(256), 0, s, a);
  });
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hap_fail(HAP_EDEVICE, "piece copy launch: %s", hipGetErrorString(e));
  return HAP_OK;
}

struct SplitArgs {
  const char* src;
  long long ld_src;                  // bytes
  long long srows, swidth;           // extent of every slot: rows, bytes per row
  char* dst[kMaxPieces];
  long long ld_dst[kMaxPieces];      // bytes
  long long src_off[kMaxPieces];     // bytes from src to the shard's first element
  long long vrows[kMaxPieces];       // the shard's part of the slot: rows, bytes per row; the rest is zero-filled
  long long vwidth[kMaxPieces];
};

/* The reverse movement: slot j (blockIdx.y) receives shard j's range of the full tensor and zeros up to the slot's extent. */
template <int UNROLL, bool STREAM, typename UNIT>
__global__ __launch_bounds__(256) void split_pieces_kernel(const SplitArgs a) {
  const int j = blockIdx.y;
  move_rows<UNROLL, STREAM, UNIT>({a.src + a.src_off[j], a.dst[j], a.ld_src, a.ld_dst[j], a.srows, a.swidth, a.vrows[j], a.vwidth[j]});
}

int check_desc(const hap_gather_desc* d) {
  if (!d) return hap_fail(HAP_EINVAL, "descriptor is NULL");
  if (d->rows < 0 || d->cols < 0) return hap_fail(HAP_EINVAL, "negative tensor size");
  if (d->dim != 0 && d->dim != 1) return hap_fail(HAP_EINVAL, "dim must be 0 or 1");
  if (d->elem_bytes != 1 && d->elem_bytes != 2 && d->elem_bytes != 4 && d->elem_bytes != 8) return hap_fail(HAP_EINVAL, "elem_bytes must be 1, 2, 4 or 8");
  if (d->m < 1 || d->m > kMaxPieces) return hap_fail(HAP_EINVAL, "m = %d outside [1, %d]", d->m, kMaxPieces);
  return HAP_OK;
}

}  // namespace

extern "C" {

int64_t hap_allgather_capacity(const hap_gather_desc* d) {
  hap_clear_error();
  if (check_desc(d)) return -1;
  int64_t cap = 0;
  for (int j = 0; j < d->m; ++j) {
    int64_t lo, hi;
    if (hap_shard_range(d->m, d->offsets, d->dim == 0 ? d->rows : d->cols, j, &lo, &hi)) return -1;
    if (hi - lo > cap) cap = hi - lo;
  }
  return cap;
}

int hap_allgather_pad(const hap_gather_desc* d, int shard_index, const void* shard, int64_t ld_shard, void* slot, int64_t ld_slot, void* stream) {
  hap_clear_error();
  int rc = check_desc(d);
  if (rc) return rc;
  int64_t lo, hi;
  if ((rc = hap_shard_range(d->m, d->offsets, d->dim == 0 ? d->rows : d->cols, shard_index, &lo, &hi))) return rc;
  const int64_t r = d->dim == 0 ? hi - lo : d->rows, c = d->dim == 0 ? d->cols : hi - lo;
  if (r == 0 || c == 0) return HAP_OK;
  if (!shard || !slot) return hap_fail(HAP_EINVAL, "NULL pointer");
  if (ld_shard < c || ld_slot < c) return hap_fail(HAP_ESHAPE, "leading dimension below the shard's width %lld", (long long)c);
  PieceArgs a = {};
  a.m = 1; a.out = static_cast<char*>(slot); a.ld_out = ld_slot * d->elem_bytes;
  a.src[0] = static_cast<const char*>(shard); a.ld_src[0] = ld_shard * d->elem_bytes;
  a.rows[0] = r; a.width[0] = c * d->elem_bytes;
  return launch_pieces(a, d->dim == 1, static_cast<hipStream_t>(stream));
}

int hap_allgather_assemble(const hap_gather_desc* d, const void* const* pieces, const int64_t* ld_pieces, void* out, int64_t ld_out, void* stream) {
  hap_clear_error();
  int rc = check_desc(d);
  if (rc) return rc;
  if (!pieces || !ld_pieces) return hap_fail(HAP_EINVAL, "NULL piece table");
  if (ld_out < d->cols) return hap_fail(HAP_ESHAPE, "ld_out below cols");
  PieceArgs a = {};
  a.m = d->m; a.out = static_cast<char*>(out); a.ld_out = ld_out * d->elem_bytes;
  for (int j = 0; j < d->m; ++j) {
    int64_t lo, hi;
    if ((rc = hap_shard_range(d->m, d->offsets, d->dim == 0 ? d->rows : d->cols, j, &lo, &hi))) return rc;
    const int64_t r = d->dim == 0 ? hi - lo : d->rows, c = d->dim == 0 ? d->cols : hi - lo;
    if (r == 0 || c == 0) continue;                      // an empty shard contributes nothing
    if (!pieces[j] || !out) return hap_fail(HAP_EINVAL, "piece %d or out is NULL", j);
    if (ld_pieces[j] < c) return hap_fail(HAP_ESHAPE, "piece %d: leading dimension %lld below its width %lld", j, (long long)ld_pieces[j], (long long)c);
    a.src[j] = static_cast<const char*>(pieces[j]); a.ld_src[j] = ld_pieces[j] * d->elem_bytes;
    a.dst_off[j] = (d->dim == 0 ? lo * ld_out : lo) * d->elem_bytes;
    a.rows[j] = r; a.width[j] = c * d->elem_bytes;
  }
  return launch_pieces(a, d->dim == 1, static_cast<hipStream_t>(stream));
}

int hap_reducescatter_split(const hap_gather_desc* d, const void* full, int64_t ld_full, void* const* slots, const int64_t* ld_slots, void* stream) {
  hap_clear_error();
  int rc = check_desc(d);
  if (rc) return rc;
  if (!slots || !ld_slots) return hap_fail(HAP_EINVAL, "NULL slot table");
  const int64_t cap = hap_allgather_capacity(d);
  if (cap < 0) return HAP_ESHAPE;
  const int64_t srows = d->dim == 0 ? cap : d->rows, scols = d->dim == 0 ? d->cols : cap;
  if (srows == 0 || scols == 0) return HAP_OK;
  if (!full) return hap_fail(HAP_EINVAL, "full is NULL");
  if (ld_full < d->cols) return hap_fail(HAP_ESHAPE, "ld_full below cols");
  SplitArgs a = {};
  a.src = static_cast<const char*>(full); a.ld_src = ld_full * d->elem_bytes;
  a.srows = srows; a.swidth = scols * d->elem_bytes;
  for (int j = 0; j < d->m; ++j) {
    int64_t lo, hi;
    if ((rc = hap_shard_range(d->m, d->offsets, d->dim == 0 ? d->rows : d->cols, j, &lo, &hi))) return rc;
    if (!slots[j]) return hap_fail(HAP_EINVAL, "slot %d is NULL", j);
    if (ld_slots[j] < scols) return hap_fail(HAP_ESHAPE, "slot %d: leading dimension %lld below the slot's width %lld", j, (long long)ld_slots[j], (long long)scols);
    a.dst[j] = static_cast<char*>(slots[j]); a.ld_dst[j] = ld_slots[j] * d->elem_bytes;
    a.src_off[j] = (d->dim == 0 ? lo * ld_full : lo) * d->elem_bytes;
    a.vrows[j] = d->dim == 0 ? hi - lo : d->rows;
    a.vwidth[j] = (d->dim == 0 ? d->cols : hi - lo) * d->elem_bytes;
  }
  const long long chunks = srows * ((a.swidth + 30) / 16);
  uintptr_t phases = (uintptr_t)a.src | (uintptr_t)a.ld_src | (uintptr_t)a.swidth;
  for (int j = 0; j < d->m; ++j) phases |= (uintptr_t)a.dst[j] | (uintptr_t)a.ld_dst[j] | (uintptr_t)a.src_off[j] | (uintptr_t)a.vwidth[j];
  const bool stream_stores = streamed(srows * a.swidth * d->m);
  with_unit(phases, [&](auto unit) {
    using U = decltype(unit);
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (!stream_stores) hipLaunchKernelGGL((split_pieces_kernel<1, false, U>), move_grid(chunks, 1, d->m), dim3(256), 0, s, a);
    else if (d->dim == 1) hipLaunchKernelGGL((split_pieces_kernel<4, true, U>), move_grid(chunks, 4, d->m), dim3(256), 0, s, a);
    else hipLaunchKernelGGL((split_pieces_kernel<1, true, U>), move_grid(chunks, 1, d->m), dim3(256), 0, s, a);
  });
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hap_fail(HAP_EDEVICE, "slot split launch: %s", hipGetErrorString(e));
  return HAP_OK;
}

}  // extern "C"
