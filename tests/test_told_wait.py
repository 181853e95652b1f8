"""How the host waits for a pass's word (told_wait.h), against a clock and a stream that are made up: it sees the word when it comes however
long the pass lasts, asks the stream rarely, and ends when the stream has ended without the word."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_16162_amd", "csrc")

# a look, a question to the stream and a rest take 50 ns, 1 us and 100 ns (a yield 1 us); times in ns
DRIVER = r'''
#include <cstdio>
#include <cstdlib>
#include "told_wait.h"
int main(int, char **v) {
    const long long word = atoll(v[1]), end = atoll(v[2]);        // the word comes, the stream ends; -1: never
    long long t = 0;
    int asked = 0, yields = 0;
    const bool came = ks::told_wait([&] { t += 50; return word >= 0 && t >= word; }, [&] { ++asked; t += 1000; return end >= 0 && t >= end; },
                                    [&] { return t / 1000; }, [&](bool yield) { yields += yield; t += yield ? 1000 : 100; });
    printf("%d %lld %d %d\n", came, t, asked, yields);
}
'''


@pytest.fixture(scope="module")
def wait(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("told")
    (tmp / "driver.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-o", str(tmp / "driver"), str(tmp / "driver.cpp")], check=True)
    return lambda *args: [int(x) for x in subprocess.run([str(tmp / "driver")] + [str(a) for a in args], check=True, capture_output=True, text=True,
                                                          timeout=60).stdout.split()]


MS = 1000 * 1000


@pytest.mark.parametrize("word", [0, 30 * 1000, 700 * 1000, 2 * MS, 4999 * 1000, 5 * MS, 5160 * 1000, 17 * MS, 400 * MS])
@pytest.mark.parametrize("behind", [300, 40 * 1000, 50 * MS])          # the stream ends so long after the word
def test_the_word_is_seen_when_it_comes(wait, word, behind):
    came, t, asked, yields = wait(word, word + behind)
    assert came == 1 and t - word <= 5 * 1000           # a look, a rest and at most one question to the stream
    assert asked <= word // (5 * MS)                    # the stream is asked now and then at most
    assert (yields > 0) == (word > 2 * MS + 10 * 1000)


@pytest.mark.parametrize("end", [0, 100 * 1000, 5160 * 1000, 33 * MS])
def test_a_stream_that_ends_without_the_word_ends_the_wait(wait, end):
    came, t, asked, _ = wait(-1, end)
    assert came == 0 and t <= end + 6 * MS


def test_a_word_between_the_last_look_and_the_end_counts(wait):
    """The stream is asked at 5 ms for the first time; the word is written while it answers."""
    _, t, asked, _ = wait(-1, 5 * MS)
    assert asked == 1
    came, t2, asked, _ = wait(t - 60, 5 * MS)
    assert came == 1 and t2 == t
