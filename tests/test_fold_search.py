"""The folded enumeration's job search, compiled for the CPU with a loop in the
wave's place: every first and last chunk of every job must lead to that job,
on both sides of the 64 and 4,096 jobs that one and two rounds can tell apart."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1907_12933_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "fold_search.h"

int main() {
    const int sizes[] = {1, 2, 63, 64, 65, 127, 128, 4032, 4095, 4096, 4097, 4160, 4200, 5016, 8191, 262144, 262145, 270001};
    for (int n : sizes) {
        std::vector<long long> begin;
        long long at = 0;
        for (int j = 0; j < n; ++j) {
            begin.push_back(at);
            at += 1 + j % 7;
        }
        for (int j = 0; j < n; ++j)
            for (long long chunk : {begin[j], (j + 1 < n ? begin[j + 1] : at) - 1}) {
                const int got = ibmc::fold_search(n, [&](int first, int step, int m) {
                    int c = 0;
                    for (int lane = 0; lane < 64; ++lane) c += lane * step < m && begin[first + lane * step] <= chunk;
                    return c;
                });
                if (got != j) {
                    std::printf("%d jobs: chunk %lld of job %d leads to %d\n", n, chunk, j, got);
                    return 1;
                }
            }
    }
    return 0;
}
"""


def test_every_chunk_finds_its_job(tmp_path):
    src, exe = tmp_path / "search.cpp", tmp_path / "search"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
