"""The rules of the small models' one-launch passes (host code)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2505_16162_amd", "csrc")

DRIVER = r'''
#include <cstdio>
#include <cstdlib>
#include "small_plan.h"
int main(int, char **v) {
    const int H = atoi(v[1]), hd = atoi(v[2]), rows = atoi(v[3]), len = atoi(v[4]);
    printf("%d %d\n", ks::small_wait(H, hd, rows, len), ks::SM_ITEMS);
}
'''


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("small")
    (tmp / "driver.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-o", str(tmp / "driver"), str(tmp / "driver.cpp")], check=True)
    return lambda *args: [int(x) for x in subprocess.run([str(tmp / "driver")] + [str(a) for a in args], check=True, capture_output=True, text=True).stdout.split()]


@pytest.mark.parametrize("heads,hd,rows,length", [(1, 64, 1, 1), (4, 64, 16, 300), (16, 64, 8, 8000), (16, 64, 9, 8000), (2, 128, 1, 6000), (20, 128, 8, 9000), (64, 64, 5, 9000)])
def test_the_wait_covers_the_attention(driver, heads, hd, rows, length):
    """A workgroup takes its (row, head) items one after the other, each a round of loads and a reduction per 1024 / (hd / 4) positions of keys and of
    values, 1.1 us measured: twice that, and what any other step may take. In ticks of 10 ns."""
    wait, side_by_side = driver(heads, hd, rows, length)
    turns = -(-heads * rows // side_by_side)
    rounds = 2 * -(-length // (1024 // (hd // 4)))
    assert wait * 10e-3 >= 350 + 2.2 * turns * rounds
    assert wait * 10e-3 < 50000        # a launch that cannot be whole is given up within some tens of milliseconds
