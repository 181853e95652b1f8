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
int main(int n, char **v) {
    if (n == 2) {        // a word per pass: w runs whole, b is broken up; what was chosen
        ks::SmallHold h;
        int broken = 0;
        for (const char *p = v[1]; *p; ++p) {
            const bool held = h.hold(broken);
            putchar(held ? '1' : '0'); putchar(' ');
            broken += !held && *p == 'b';
        }
        return 0;
    }
    const int H = atoi(v[1]), hd = atoi(v[2]), rows = atoi(v[3]), len = atoi(v[4]);
    printf("%d %d", ks::small_wait(H, hd, rows, len), ks::SM_ITEMS);
    for (int n_attn = 0; n_attn <= 12; ++n_attn) printf(" %d %d", ks::small_faster(H, hd, false, n_attn, rows, len), ks::small_faster(H, hd, true, n_attn, rows, len));
    printf("\n");
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
    wait, side_by_side = driver(heads, hd, rows, length)[:2]
    turns = -(-heads * rows // side_by_side)
    rounds = 2 * -(-length // (1024 // (hd // 4)))
    assert wait * 10e-3 >= 350 + 2.2 * turns * rounds
    assert wait * 10e-3 < 50000        # a launch that cannot be whole is given up within some tens of milliseconds


# measured on an MI355X, GPU us as launches / in one launch inside generations: (heads, head size, rows, context, bf16, attention sublayers)
MEASURED = [((4, 64, 1, 30, 0, 4), 87, 55), ((4, 64, 1, 250, 0, 4), 96, 74), ((4, 64, 1, 1400, 0, 4), 179, 215), ((4, 64, 5, 1400, 0, 4), 191, 235),
            ((2, 128, 1, 600, 0, 4), 152, 194), ((2, 128, 5, 250, 0, 4), 115, 126), ((16, 64, 5, 250, 0, 4), 107, 115), ((32, 64, 5, 250, 0, 4), 115, 149),
            ((32, 64, 5, 600, 0, 4), 153, 221), ((8, 128, 1, 1400, 0, 4), 319, 392), ((4, 64, 1, 30, 0, 12), 224, 141), ((4, 64, 1, 1400, 0, 12), 543, 614),
            ((2, 128, 5, 1400, 0, 1), 75, 95), ((16, 64, 1, 250, 0, 1), 39, 30), ((2, 128, 1, 250, 0, 1), 42, 32), ((4, 64, 1, 600, 1, 4), 118, 99),
            ((4, 64, 1, 1400, 1, 4), 153, 188), ((2, 128, 1, 1400, 1, 4), 253, 367), ((32, 64, 5, 600, 1, 4), 150, 221), ((8, 128, 5, 600, 1, 12), 571, 639),
            ((8, 128, 1, 30, 1, 12), 233, 172), ((4, 64, 5, 250, 1, 4), 113, 102), ((2, 128, 1, 6000, 1, 1), 212, 409)]


def test_passes_take_the_faster_way(driver):
    for (heads, hd, rows, ctx, bf16, n_attn), launches, one in MEASURED:
        faster = driver(heads, hd, rows, ctx + rows)[2:]
        chosen = one if faster[2 * n_attn + bf16] else launches
        assert chosen <= 1.1 * min(one, launches), (heads, hd, rows, ctx, bf16, n_attn)      # a fit: within a tenth around the crossing


def test_longer_contexts_and_more_rows_never_turn_to_one_launch(driver):
    for heads, hd in ((1, 64), (16, 64), (4, 128)):
        for rows in (1, 5, 16):
            last = None
            for length in list(range(16, 700, 31)) + [2000, 8000]:
                now = driver(heads, hd, rows, length)[2:]
                assert now[0] == now[1] == 1                     # no attention: nothing depends on the context
                if last is not None:
                    assert all(b <= a for a, b in zip(last, now))
                last = now
            assert not any(last[2:])
    assert all(b <= a for a, b in zip(driver(4, 64, 5, 300)[2:], driver(4, 64, 9, 300)[2:]))


def test_broken_launches_are_not_tried_again_at_once(driver):
    def held_after(passes):                 # lengths of the runs of passes held back
        return [len(r) for r in "".join(map(str, driver(passes))).split("0") if r]
    assert held_after("w" * 500) == []
    assert held_after("w" * 10 + "b" + "w" * 200) == [64]
    assert held_after("b" * 5000)[:7] == [64, 128, 256, 512, 1024, 1024, 1024]     # on a GPU that stays busy
    assert held_after("b" + "w" * 64 + "b" + "w" * 1000) == [64, 128]
    assert held_after("b" + "w" * 200 + "b" + "w" * 200) == [64, 64]               # a second disturbance, much later
