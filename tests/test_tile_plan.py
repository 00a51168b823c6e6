"""Address arithmetic of the tiled GEMM and the choice between the prompt attentions, compiled for the host and
enumerated."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_28166_amd", "csrc")

OFFSETS = r"""
#include <cstdio>
#include <initializer_list>
#include "tile_plan.h"
// every weight fragment that the tiles of an N-row matrix fetch lies inside the packed matrix, and inside the tile
// it is the fragment of its own block
int main() {
  const int rows[] = {1, 31, 32, 33, 127, 128, 129, 224, 255, 256, 257, 544, 31972, 32001, 151936};
  for (int n : rows)
    for (int bn : {128, 256})
      for (int k : {256, 512, 1024}) {
        const int nblk = (n + 31) / 32, kfr = k / 16;
        for (int b0 = 0; b0 < nblk; b0 += bn / 32)
          for (int f = 0; f < bn / 16; ++f)
            for (int kc = 0; kc < k / 32; kc += k / 32 - 1) {
              const long off = tandem::tile_weight_offset(f, kc, kfr, nblk - b0);
              const long at = (long)b0 * kfr * 1024 + off;
              const bool own = b0 + f / 2 >= nblk || off == ((long)(f / 2) * kfr + 2 * kc + f % 2) * 1024;
              if (off < 0 || at + 1024 > (long)nblk * kfr * 1024 || !own) {
                printf("N %d, tile of %d rows, K %d: block %d, fragment %d, chunk %d at %ld of %ld\n", n, bn, k, b0, f,
                       kc, at, (long)nblk * kfr * 1024);
                return 1;
              }
            }
      }
  return 0;
}
"""


def _run(tmp_path, source):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(source)
    subprocess.run(["g++", "-std=c++17", "-O1", f"-I{CSRC}", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_weight_fragments_lie_inside_the_matrix(tmp_path):
    _run(tmp_path, OFFSETS)


ATTENTION = r"""
#include <cstdio>
#include "tile_plan.h"
// {kv heads, heads per group, head size, row groups, longest prompt, waves that split the positions}
int main() {
  const int c[][6] = {
      {4, 4, 64, 32, 512, 1},  {4, 4, 64, 128, 2040, 1},  {4, 4, 64, 512, 2040, 0}, {4, 4, 64, 128, 512, 0},
      {4, 4, 64, 64, 128, 0},  {4, 4, 64, 256, 256, 0},   {8, 4, 128, 8, 128, 1},   {8, 4, 128, 128, 2040, 0},
      {8, 2, 128, 32, 512, 1}, {8, 2, 128, 512, 2040, 0}, {2, 8, 64, 128, 2040, 1}, {2, 8, 64, 128, 512, 0},
      {8, 1, 128, 8, 128, 1},  {8, 1, 128, 512, 2040, 1},
      // the GPU parity cases: a few prompts (up to 20 groups a pass), then 240 groups
      {2, 4, 64, 20, 96, 1},   {2, 4, 128, 20, 96, 1},    {1, 2, 128, 20, 96, 1},   {2, 8, 64, 20, 96, 1},
      {1, 8, 128, 20, 96, 1},  {2, 4, 64, 240, 96, 0},    {2, 2, 64, 240, 96, 0},   {2, 4, 128, 240, 96, 0},
      {2, 2, 128, 240, 96, 0}, {2, 8, 64, 240, 96, 0},    {2, 8, 128, 240, 96, 0}};
  for (const auto& x : c)
    if (tandem::prompt_splits_positions(256, x[0], x[1], x[2], x[3], x[4]) != (x[5] != 0)) {
      printf("%d kv heads, groups of %d, head size %d, %d row groups, %d positions\n", x[0], x[1], x[2], x[3], x[4]);
      return 1;
    }
  return 0;
}
"""


def test_prompt_attention_of_each_shape(tmp_path):
    _run(tmp_path, ATTENTION)
