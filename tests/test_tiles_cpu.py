"""The projections' tile arithmetic, compiled for the host from the header that the kernels
include."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2511_22009_amd", "csrc")


def _compiled(tmp_path_factory, name, body):
    d = tmp_path_factory.mktemp(name)
    src, exe = str(d / (name + ".cpp")), str(d / name)
    with open(src, "w") as f:
        f.write(body)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, src, "-o", exe], check=True)
    return exe


ROWS = r"""
#include <cstdio>
#include "sf_tiles.h"
// Every residual epilogue pass over tiles of BM rows in steps of RP rows: prints the first
// item whose loaded row is not one of the M rows (or not its own where it has one), or whose
// gate slot is not one of the M / ntok samples.
int main() {
  const int tiles[][2] = {{64, 32}, {128, 32}, {128, 64}, {256, 32}, {256, 128}};
  long seen = 0, past = 0;
  for (int rows = 1; rows <= 16; ++rows)
    for (int ntok = 1; ntok <= 40; ++ntok)
      for (const auto& t : tiles) {
        const int M = rows * ntok;
        for (int m0 = 0; m0 < M; m0 += t[0])
          for (int p0 = m0; p0 < m0 + t[0]; p0 += t[1])
            for (int m = p0; m < p0 + t[1]; ++m)
              for (int col = 0; col < 2; ++col) {
                const bool in = m < M && col == 0;
                const int got = sf::loaded_row(in, m, p0, M);
                ++seen;
                past += p0 >= M;
                if (got < 0 || got >= M || got / ntok >= rows || (in && got != m)) {
                  std::printf("M %d ntok %d tile %d pass at %d item %d: row %d\n", M, ntok, t[0], p0, m, got);
                  return 1;
                }
              }
      }
  std::printf("ok %ld %ld\n", seen, past);
  return 0;
}
"""


def test_residual_epilogue_items_read_rows_that_exist(tmp_path_factory):
    """Items outside the tile load from a row of the matrix also in a pass that starts past its
    end (a 64-row tile of 1 to 32 rows, the last tile of a ragged batch)."""
    r = subprocess.run([_compiled(tmp_path_factory, "rows", ROWS)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
    ok, seen, past = r.stdout.split()
    assert ok == "ok" and int(past) > 1000, r.stdout
