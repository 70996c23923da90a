/*
 * Index arithmetic of the piece copies (hap_gather.hip): which 16-byte chunks a move has.  Plain constexpr functions: device code calls them,
 * and a host compiler can run them over sizes that no test buffer has.
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

}  // namespace hap_move

#endif
