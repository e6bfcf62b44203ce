"""The weights of a node whose list ends at the last positions an int32 offset can have, in the lanes' shares of a
few lanes, a wavefront and a workgroup: every weight once, nothing outside the list (the arrays end where the list
does, in address space that is only reserved)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <sys/mman.h>
#include "hnv_weights.h"

template <int U> static int check(int32_t *idx, float *wn, uint32_t end, uint32_t len, uint32_t lanes)
{
    const uint32_t begin = end - len;
    float w[97];
    double want = 0.0, got = 0.0;
    for (int i = 0; i < 97; ++i)
        w[i] = 1.0f + (float)i;
    for (uint32_t j = begin; j < end; ++j) {
        idx[j] = 1000 + (int32_t)(j % 97);
        wn[j] = 0.0f;
        want += w[j % 97];
    }
    for (uint32_t l = 0; l < lanes; ++l)
        got += hnv::sum_weights<U>(idx, w, 1000, begin + l, end, lanes, wn);
    for (uint32_t j = begin; j < end; ++j)
        if (wn[j] != w[j % 97])
            return 1;
    return got == want ? 0 : 2;     // whole numbers, so the order does not matter
}

int main()
{
    const uint32_t end = 0x7ffffffeu;      // one below the largest accepted number of incidences
    const size_t bytes = 4 * (size_t)end;
    int32_t *idx = (int32_t *)mmap(nullptr, bytes, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    float *wn = (float *)mmap(nullptr, bytes, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (idx == MAP_FAILED || wn == MAP_FAILED)
        return 77;
    const int bad = check<2>(idx, wn, end, 64, 4) + 10 * check<8>(idx, wn, end, 65, 64) +
                    100 * check<8>(idx, wn, end, 2048, 64) + 1000 * check<8>(idx, wn, end, 5001, 256);
    std::printf("%d\n", bad);
    return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_lists_that_end_at_the_last_offset(tmp_path):
    src, exe = tmp_path / "weights.cpp", str(tmp_path / "weights")
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Wno-unknown-pragmas", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2103_09660_amd", "csrc"), str(src), "-o", exe], check=True)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    if run.returncode == 77:
        pytest.skip("no address space")
    assert run.returncode == 0 and run.stdout.strip() == "0", (run.returncode, run.stdout)
