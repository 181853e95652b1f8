"""Which prompts on the any-shape kernels take their rows side by side (prompt_plan.h), against whole prompts measured on an MI355X."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_16162_amd", "csrc")

DRIVER = r'''
#include <cstdio>
#include <cstdlib>
#include "prompt_plan.h"
int main(int n, char **v) {
    for (int i = 1; i + 2 < n; i += 3) {
        knnssd_model_cfg g{};
        g.weight_dtype = atoi(v[i]); g.d_model = atoi(v[i + 1]);
        printf("%d\n", ks::prompt_rows(g, atoi(v[i + 2])));
    }
}
'''


@pytest.fixture(scope="module")
def rows(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("prompt")
    (tmp / "driver.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-o", str(tmp / "driver"), str(tmp / "driver.cpp")], check=True)
    return lambda cases: [int(x) for x in subprocess.run([str(tmp / "driver")] + [str(a) for c in cases for a in c], check=True, capture_output=True, text=True).stdout.split()]


# (bf16 weights, columns, rows): us in passes, side by side in launches of up to 256 rows, of up to 128
MEASURED = [((0, 72, 33), 151, 112, None), ((0, 520, 17), 222, 105, None), ((0, 520, 250), 2362, 348, None), ((0, 4104, 17), 1552, 1214, None), ((0, 5128, 25), 3080, 2506, None),
            ((0, 8008, 17), 3288, 2381, None), ((0, 8008, 250), 42103, 24299, None), ((1, 72, 17), 99, 85, None), ((1, 520, 250), 1954, 366, 410), ((1, 1000, 17), 249, 134, None),
            ((1, 2504, 17), 305, 248, None), ((1, 2504, 129), 3424, 2191, 2328), ((1, 3000, 17), 343, 309, None), ((1, 3008, 250), 3903, 3005, 2771), ((1, 3304, 17), 408, 424, None),
            ((1, 3304, 33), 684, 650, None), ((1, 3600, 25), 538, 597, None), ((1, 3600, 33), 742, 712, None), ((1, 4104, 17), 672, 726, None), ((1, 4104, 250), 8067, 7906, 7099),
            ((1, 4304, 33), 1024, 963, None), ((1, 4608, 25), 868, 998, None), ((1, 4608, 250), 8219, 8466, 7479), ((1, 4808, 33), 1343, 1424, None), ((1, 5128, 17), 885, 1000, None),
            ((1, 5128, 49), 2240, 2128, None), ((1, 5128, 250), 9653, 10329, 8977), ((1, 5304, 500), 20074, 21680, 18669), ((1, 5504, 250), 9999, 11299, 9599),
            ((1, 6008, 17), 955, 1194, None), ((1, 6008, 64), 2929, 3129, None), ((1, 6008, 250), 11514, 14405, None), ((1, 8008, 112), 11379, 11503, None)]


def test_prompts_take_the_faster_way(rows):
    for (case, passes, full, half), got in zip(MEASURED, rows([m[0] for m in MEASURED])):
        taken = passes if got == 0 else (full if half is None or got == 256 else half)
        assert got in (0, 256) or half is not None or got >= case[2], case
        assert taken <= 1.02 * min(t for t in (passes, full, half) if t), case


def test_launches_hold_the_prompt(rows):
    """Whole passes' rows each (the head reads the prompt's last pass of rows from one launch), never more than there is room for, about equal."""
    cases = [(b, d, n) for b in (0, 1) for d in (8, 2800, 2808, 3200, 3208, 4700, 4704, 5600, 5608) for n in range(1, 1100)]
    for (b, d, n), r in zip(cases, rows(cases)):
        assert r % 16 == 0 and 0 <= r <= 256
        assert n > 16 or r == 0
        if r and b and d > 2800:
            assert r <= 128 and -(-n // r) == -(-n // 128)
