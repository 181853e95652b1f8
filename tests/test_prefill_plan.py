"""The prefill's tile plan (host code): the GPU tests' prompts reach every build of the product, and every plan covers its
matrix and its token rows."""
import os
import re
import subprocess

import pytest

from test_gpu_prefill_tiles import OPERAND_PROMPTS, OPERANDS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2505_16162_amd", "csrc")

DRIVER = r'''
#include <cstdio>
#include <cstdlib>
#include "prefill_plan.h"
int main(int n, char **v) {
    knnssd_model_cfg g{};
    g.d_model = atoi(v[1]); g.n_heads = atoi(v[2]); g.n_kv_heads = atoi(v[3]); g.head_dim = atoi(v[4]); g.d_ffn = atoi(v[5]);
    for (int i = 6; i < n; ++i)
        for (int w = 0; w < ks::PF_OPS; ++w) {
            const ks::PfPlan p = ks::pf_plan(g, w, (atoi(v[i]) + 15) / 16);
            printf("%d %d %d %d %d %d %d %d %d\n", atoi(v[i]), w, p.tb, p.S, p.epilogue(w), p.own_sums(w), p.n_mt * p.tm(), p.out_rows(), p.n_mr * p.tm());
        }
}
'''


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("plan")
    (tmp / "driver.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-o", str(tmp / "driver"), str(tmp / "driver.cpp")], check=True)

    def run(shape, lengths):
        args = [shape[k] for k in ("d_model", "n_heads", "n_kv_heads", "head_dim", "d_ffn")] + list(lengths)
        out = subprocess.run([str(tmp / "driver")] + [str(a) for a in args], check=True, capture_output=True, text=True).stdout
        keys = ("n", "which", "tb", "S", "epilogue", "own", "rows", "out_rows", "pair_rows")
        return [dict(zip(keys, map(int, line.split()))) for line in out.splitlines()]
    return run


def test_gpu_prompts_reach_every_build(plans):
    text = open(os.path.join(CSRC, "knnssd.hip")).read()
    kinds = ("PF_PARTS", "PF_SWIGLU", "PF_ROPE")
    builds = {(int(tb), kinds.index(epi), int(own == "true"))
              for tb, epi, own in re.findall(r"^    pf_build<\d+, (\d+), \d+, \d+, \w+, (\w+), (\w+)>\(f\);", text, re.M)}
    assert len(builds) == 7
    assert {(p["tb"], p["epilogue"], p["own"]) for p in plans(OPERANDS, OPERAND_PROMPTS)} == builds


@pytest.mark.parametrize("shape", [OPERANDS, dict(d_model=5120, n_heads=40, n_kv_heads=8, head_dim=128, d_ffn=13824),
                                   dict(d_model=320, n_heads=2, n_kv_heads=1, head_dim=64, d_ffn=352)])
def test_plans_cover_rows_and_tokens(plans, shape):
    kinds = set()
    text = open(os.path.join(CSRC, "knnssd.hip")).read()
    for tb, epi, own in re.findall(r"^    pf_build<\d+, (\d+), \d+, \d+, \w+, (\w+), (\w+)>\(f\);", text, re.M):
        kinds.add((int(tb), ("PF_PARTS", "PF_SWIGLU", "PF_ROPE").index(epi), int(own == "true")))
    qd, kvd = shape["n_heads"] * shape["head_dim"], shape["n_kv_heads"] * shape["head_dim"]
    width = [qd, shape["d_model"], 2 * shape["d_ffn"], shape["d_model"]]
    k = [shape["d_model"], qd, shape["d_model"], shape["d_ffn"]]
    for p in plans(shape, list(range(1, 700, 13)) + [1024, 1025, 4096, 15360]):
        w = p["which"]
        assert (p["tb"], p["epilogue"], p["own"]) in kinds, p          # a build for every plan
        assert p["out_rows"] >= p["n"]
        assert 1 <= p["S"] <= 16 and p["S"] <= k[w] // 32
        if w == 0:
            assert p["pair_rows"] >= qd + kvd and p["rows"] - p["pair_rows"] >= kvd
        else:
            assert p["rows"] >= width[w] and p["rows"] - width[w] < 256
