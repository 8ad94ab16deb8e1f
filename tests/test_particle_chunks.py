"""The list of particle chunks near the largest particle number an int holds: a
small host program built with the kernels' header lists the chunks of tiles that
end at 2^31 - 1 (as the sort's kernel does) and checks that they cover the tile in
order, none beyond it and none past the counted entries."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1502_02935_amd", "csrc")

PROGRAM = r"""
#include <climits>
#include <cstdio>
#include <vector>
#include "mhd_kernels.hpp"
int main() {
  using namespace mhd;
  const int sizes[] = {0, 1, kChunk - 1, kChunk, kChunk + 1, 3 * kChunk, 5000, INT_MAX};
  for (int c : sizes)
    for (int first : {0, INT_MAX - c}) {
      const int want = (int)(((long long)c + kChunk - 1) / kChunk);
      if (chunk_count(c) != want) return std::printf("count of %d\n", c), 1;
      std::vector<int> list(1 + 3 * (size_t)(want + 2), -7);
      if (list_chunks(list.data(), 1, 9, first, c) != 1 + want) return std::printf("end of %d\n", c), 1;
      long long at = first;
      for (int k = 1; k <= want; ++k) {
        const int* r = &list[1 + 3 * (size_t)k];
        const long long n = (long long)r[2] - r[1];
        if (r[0] != 9 || r[1] != at || n < 1 || n > kChunk) return std::printf("chunk %d of %d\n", k, c), 1;
        at += n;
      }
      if (at != (long long)first + c || list[1 + 3 * (size_t)(want + 1)] != -7 || list[3] != -7)
        return std::printf("cover of %d\n", c), 1;
    }
  std::puts("ok");
  return 0;
}
"""


def test_chunks_up_to_the_largest_index(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    src, exe = tmp_path / "chunks.hip", tmp_path / "chunks"
    src.write_text(PROGRAM)
    subprocess.run([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-I", CSRC, "-I",
                    os.path.join(ROOT, "include"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
