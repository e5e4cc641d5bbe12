"""Rules of the kernels and their dispatch, compiled for the host from the header that the
kernels include."""
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
#include "sf_rules.h"
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


SOFTMAX = r"""
#include <cmath>
#include <cstdio>
#include <cstring>
#include <initializer_list>
#include <limits>
#include "sf_rules.h"
static uint32_t bits(float f) { uint32_t u; std::memcpy(&u, &f, 4); return u; }
static uint32_t bf16_pattern(float p) {  // round to nearest even, kept in the high half
  uint32_t u = bits(p);
  if (p != p) return (u | 0x400000u) & 0xffff0000u;
  return (u + 0x7fffu + ((u >> 16) & 1u)) & 0xffff0000u;
}
// s: the lane's largest score less the offset. p: 2^s off by up to one unit in the last place,
// and any bf16 pattern in the low half.
int main() {
  long looked = 0, n = 0;
  auto check = [&](float s) {
    const float e = std::exp2(s);
    for (int k = -1; k <= 1; ++k) {
      const float p = k == 0 ? e : std::nextafter(e, k < 0 ? 0.0f : std::numeric_limits<float>::infinity());
      for (uint32_t low : {0u, 0xffffu})
        for (bool first : {false, true}) {
          const bool looks = sf::softmax_looks(bf16_pattern(p) | low, first);
          const bool must = s > 64.0f || (first && s < -64.0f) || s != s;
          const bool may = must || std::fabs(std::fabs(s) - 64.0f) < 0.006f || (first && s < -64.0f);
          ++n;
          looked += looks;
          if ((must && !looks) || (looks && !may)) {
            std::printf("score %.9g first %d: looks %d\n", s, (int)first, (int)looks);
            return false;
          }
        }
    }
    return true;
  };
  for (float edge : {64.0f, -64.0f}) {
    float lo = edge, hi = edge;
    for (int i = 0; i < 3000; ++i) {  // every float next to the edge, then ever wider steps
      if (!check(lo) || !check(hi)) return 1;
      lo = i < 1000 ? std::nextafter(lo, -1e9f) : lo - 1e-5f * (i - 999);
      hi = i < 1000 ? std::nextafter(hi, 1e9f) : hi + 1e-5f * (i - 999);
    }
  }
  const float inf = std::numeric_limits<float>::infinity();
  for (float s : {-inf, -200.0f, -100.0f, -1.0f, 0.0f, 63.0f, 100.0f, 127.9f, 128.0f, 500.0f, inf,
                  std::numeric_limits<float>::quiet_NaN()})
    if (!check(s)) return 1;
  std::printf("ok %ld %ld\n", looked, n);
  return 0;
}
"""


def test_softmax_step_looks_at_every_score_past_the_range(tmp_path_factory):
    """The check on rounded probabilities lets no score by that the check on scores (more than
    64 from the offset) would catch, at either edge, and takes little more than those."""
    r = subprocess.run([_compiled(tmp_path_factory, "softmax", SOFTMAX)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
    assert r.stdout.startswith("ok"), r.stdout


TILES = r"""
#include <cstdio>
#include <cstdlib>
#include "sf_rules.h"
int main(int argc, char** argv) {  // M N kind ...: the tile of each, and whether it is compiled for that kind
  const char* const names[] = {"kTile128", "kTile128x288", "kTile256x192", "kHalf128x96", "kHalf128", "kHalf64",
                               "kPipe128x192", "kPipe128", "kPipe64", "kPipeHalf128x192", "kPipeHalf128"};
  for (int i = 1; i + 4 < argc; i += 5) {
    const auto kind = (sf::EpiKind)std::atoi(argv[i + 4]);
    const sf::GemmTile t = sf::choose_gemm_tile(std::atoi(argv[i]), std::atoi(argv[i + 1]), std::atoi(argv[i + 2]),
                                                std::atoi(argv[i + 3]), kind);
    std::printf("%s %d\n", names[t], (int)sf::gemm_tile_used(t, kind));
  }
  return 0;
}
"""
KINDS = {"QKV": 0, "RES_GATE": 1, "GELU": 2, "RES": 3, "RES_GATE_MLP": 4, "KVX": 5}


def _chosen(exe, asked):
    args = [str(v) for M, N, K, ntok, kind in asked for v in (M, N, K, ntok, KINDS[kind])]
    out = subprocess.run([exe] + args, capture_output=True, text=True, timeout=60, check=True).stdout.split()
    return out[0::2], out[1::2]


def test_tiles_of_the_projection_cases(tmp_path_factory):
    """The GPU test's cases take the tiles that it names, a row alone the 64 x 64 ones, and among
    them they take every tile."""
    from test_gpu_gemm_tiles import CASES
    exe = _compiled(tmp_path_factory, "tiles", TILES)
    seen = set()
    for D, _, mlp, H, Wd, B, want in CASES.values():
        shapes = [(3 * D, D, "QKV"), (D, D, "RES_GATE"), (mlp, D, "GELU"), (D, mlp, "RES_GATE_MLP")]
        ntok = (H // 2) * (Wd // 2)
        for rows in (B, 1):
            tiles, _ = _chosen(exe, [(rows * ntok, N, K, ntok, kind) for N, K, kind in shapes])
            if rows == 1:
                want = " ".join("kHalf64" if N <= 768 and (N % 96 == 0 or N % 128 == 0) else "kPipe64"
                                for N, _, _ in shapes)
            assert tiles == want.split(), (D, rows)
            seen |= set(tiles)
    assert len(seen) == 11, seen


def test_every_tile_that_is_chosen_is_compiled(tmp_path_factory):
    """Over widths, rows and epilogues: a tile that the launcher has no kernel for is never
    chosen, and M never changes which of the two orders of sums a width gets."""
    exe = _compiled(tmp_path_factory, "tiles", TILES)
    asked = [(M, N, K, ntok, kind) for N in list(range(8, 1600, 56)) + [96, 128, 384, 512, 640, 768, 2304, 3456, 6144, 8192]
             for M, ntok in ((1, 1), (30, 30), (195, 195), (1024, 1024), (2760, 920), (4095, 195), (7800, 195),
                             (16384, 1024), (65536, 4096)) for K in (8, 768, 8192) for kind in KINDS]
    for i in range(0, len(asked), 2000):
        part = asked[i:i + 2000]
        tiles, used = _chosen(exe, part)
        for (M, N, K, ntok, kind), tile, ok in zip(part, tiles, used):
            assert ok == "1", (M, N, K, ntok, kind, tile)
            assert ("Half" in tile) == (N <= 768 and (N % 96 == 0 or N % 128 == 0)), (M, N, K, ntok, kind, tile)
