"""The index arithmetic of the piece copies (csrc/hap_move.h), compiled for the host with the undefined-behaviour sanitizer and compared with
counting: moves of devices that own nothing, rows longer than 2^31 bytes, cut chunks of all phases."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2401_05965_amd", "csrc")

SOURCE = r"""
#include <cstdio>
#include <cstdlib>
#include <initializer_list>
#include "hap_move.h"
using namespace hap_move;
static void fail(const char* what, long long a, long long b, long long c, long long d) {
  std::printf("%s: %lld %lld %lld %lld\n", what, a, b, c, d);
  std::exit(1);
}
int main() {
  const long long widths[] = {0, 1, 15, 16, 17, 31, 255, 256, 300, 4080, 4096, 4097, 1 << 20, 3LL << 31};
  for (long long rows = 0; rows <= 3; ++rows)
    for (long long width : widths)
      for (int aligned = 0; aligned < 2; ++aligned) {
        const Walk w = walk_of(rows, width, aligned);
        if (rows == 0 || width == 0) { if (w.total != 0) fail("empty", rows, width, aligned, w.total); continue; }
        // the last byte of a row lies in the last chunk, on or off the 16-byte grid
        if (w.total != rows * w.per_row || w.per_row * 16 < width + (aligned ? 0 : 15) || w.per_row * 16 > width + (aligned ? 15 : 30)) fail("chunks", rows, width, aligned, w.per_row);
        for (long long at = 0; at < w.total && at < 2000; at += 37) {
          long long r = at / w.per_row, k = at % w.per_row;
          for (int u = 1; u <= 3; ++u) {
            r += w.over; k += w.step;
            if (k >= w.per_row) { ++r; k -= w.per_row; }
            if (r != (at + 256 * u) / w.per_row || k != (at + 256 * u) % w.per_row) fail("walk", rows, width, aligned, at);
          }
        }
      }
  // byte by byte: which units of a chunk lie in the row, which of those in the shard
  for (int unit = 1; unit <= 4; unit *= 2)
    for (int phase = 0; phase < 16; phase += unit)
      for (long long width : {4LL, 16LL, 20LL, 48LL, (3LL << 31) + 4})
        for (long long vwidth : {0LL, 4LL, 12LL, 16LL, 20LL, 44LL, 3LL << 31, (3LL << 31) + 4}) {
          if (vwidth > width) continue;
          const long long chunks = (width + phase + 15) / 16;
          for (long long k = 0; k < chunks; k = k == 3 && chunks > 8 ? chunks - 3 : k + 1) {
            const long long at = 16 * k - phase;
            const Units c = units_of(at, width, vwidth, unit);
            for (int x = 0; x < 16 / unit; ++x) {
              const long long b = at + x * unit;
              if ((x >= c.first && x < c.last) != (b >= 0 && b < width)) fail("in the row", unit, at, width, vwidth);
              if ((x >= c.first && x < c.data) != (b >= 0 && b < vwidth)) fail("in the shard", unit, at, width, vwidth);
            }
          }
        }
  std::puts("ok");
}
"""


def test_chunks_of_empty_moves_and_of_rows_beyond_2_gib(tmp_path):
    src, exe = tmp_path / "move.cpp", tmp_path / "move"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    done = subprocess.run([str(exe)], capture_output=True, text=True)
    assert done.returncode == 0 and done.stdout == "ok\n", done.stdout + done.stderr
