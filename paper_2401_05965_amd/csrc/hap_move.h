/*
 * Index arithmetic of the piece copies (hap_gather.hip): which 16-byte chunks a move has, and which part of a cut chunk belongs to the row
 * and to the shard.  Plain constexpr functions: device code calls them, and a host compiler can run them over sizes that no test buffer has.
 */
#ifndef HAP_MOVE_H
#define HAP_MOVE_H

namespace hap_move {

/* The chunks of `rows` rows of `width` bytes, numbered row after row; a thread walks them 256 apart.  An empty move has none (a device that
 * owns nothing still has its place in the launch). */
struct Walk {
  long long per_row, total;
  int over, step;                    // 256 chunks on: `over` rows and `step` chunks (and one more row where that passes the row's last one)
};

/* aligned: all rows start on a 16-byte boundary; else a row may straddle one chunk more. */
constexpr Walk walk_of(long long rows, long long width, bool aligned) {
  if (rows <= 0 || width <= 0) return {1, 0, 0, 0};
  const long long per_row = (width + (aligned ? 15 : 30)) / 16;
  const int short_row = per_row < 256 ? (int)per_row : 0;
  const int over = short_row ? 256 / short_row : 0;
  return {per_row, rows * per_row, over, 256 - over * short_row};
}

/* Units of `unit` bytes of the chunk whose first byte is byte `at` of a row (negative where it starts before the row): [first, last) lie in
 * the row of `width` bytes, those of them before `data` in the shard's `vwidth` bytes (0 for a row behind the shard's last). */
struct Units { int first, last, data; };

constexpr Units units_of(long long at, long long width, long long vwidth, int unit) {
  const int n = 16 / unit;
  const int first = at < 0 ? (int)-at / unit : 0;
  const int last = at + 16 < width ? n : (int)((width - at) / unit);
  const long long left = vwidth - at;                        // (a shard may end any distance before the chunk: compared before it is narrowed)
  return {first, last, left <= 0 ? 0 : left / unit < last ? (int)(left / unit) : last};
}

}  // namespace hap_move

#endif
