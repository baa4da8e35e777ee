"""Work distribution of the persistent kernels (ppt_work.h): whatever the number of wavefronts, their tickets hand out
every batch exactly once, although each wavefront stops at the first ticket of its own counter beyond the end."""
import os
import subprocess

import pytest

CLANG = "/opt/rocm/llvm/bin/clang++"
HEADER_DIR = os.path.join(os.path.dirname(__file__), "..", "paper_2607_13265_amd", "csrc")
PROGRAM = r"""
#include "ppt_work.h"
#include <cstdio>
#include <vector>
int main() {
    for (int waves = 4; waves <= 72; waves += 4)
        for (int batches : {0, 1, 3, 4, 5, 15, 16, 17, 31, 63, 64, 65, 200, 1001}) {
            std::vector<int> seen(batches, 0), next(ppt::WORK_SHARDS, 0);
            std::vector<bool> done(waves, false);
            const int shards = ppt::work_shards(waves);
            for (int left = waves; left > 0;)  // the wavefronts in turn, the last ones most often
                for (int w = 0; w < waves; ++w)
                    for (int k = 0; k <= w % 3 && !done[w]; ++k) {
                        const int shard = w & (shards - 1), b = ppt::work_batch(next[shard]++, shard, shards);
                        if (b >= batches) { done[w] = true; --left; }
                        else ++seen[b];
                    }
            for (int b = 0; b < batches; ++b)
                if (seen[b] != 1) { std::printf("%d wavefronts, %d batches: batch %d taken %d times\n", waves, batches, b, seen[b]); return 1; }
        }
    return 0;
}
"""


def test_every_batch_is_taken_once(tmp_path):
    if not os.path.exists(CLANG):
        pytest.skip("no clang")
    src, exe = tmp_path / "w.cpp", tmp_path / "w"
    src.write_text(PROGRAM)
    subprocess.run([CLANG, "-std=c++17", "-O1", "-I", HEADER_DIR, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
