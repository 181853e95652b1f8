"""The prefill's choice of tiles as the library makes it (host code): every build is reached by the prompts of a GPU test, every plan has
a build, and tiles that finish their rows themselves walk all of K."""
import os
import re
import subprocess

import pytest

from test_gpu_prefill_tiles import OPERAND_PROMPTS, OPERANDS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2505_16162_amd", "csrc")
WIDE = dict(d_model=4096, n_heads=32, n_kv_heads=32, head_dim=128, d_ffn=6016)
PROMPTS = (170, 192, 193, 330, 385, 560, 700, 1300)
# 256 x 256 tiles with K in parts: QKV rows of the first, residual rows of the second
SPLIT = ((dict(d_model=4608, n_heads=32, n_kv_heads=32, head_dim=128, d_ffn=320), (208,)),
         (dict(d_model=2560, n_heads=64, n_kv_heads=1, head_dim=128, d_ffn=320), (1184,)))

DRIVER = r'''
#include <cstdio>
#include <cstdlib>
#include "prefill_plan.h"
int main(int n, char **v) {
    knnssd_model_cfg g{};
    g.d_model = atoi(v[1]); g.n_heads = atoi(v[2]); g.n_kv_heads = atoi(v[3]); g.head_dim = atoi(v[4]); g.d_ffn = atoi(v[5]);
    for (int i = 6; i < n; ++i)
        for (int w = 0; w < ks::PF_OPS; ++w) {
            const ks::PfPlan p = ks::pf_choose(g, w, (atoi(v[i]) + 15) / 16);
            printf("%d %d %d %d %d %d %d %d %d %d\n", atoi(v[i]), w, p.tb, p.S, p.epilogue(w), p.own_sums(w), p.G, p.n_mt * p.tm(), p.out_rows(), p.parts(w));
        }
}
'''


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("wide")
    (tmp / "driver.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-o", str(tmp / "driver"), str(tmp / "driver.cpp")], check=True)

    def run(shape, lengths):
        args = [shape[k] for k in ("d_model", "n_heads", "n_kv_heads", "head_dim", "d_ffn")] + list(lengths)
        out = subprocess.run([str(tmp / "driver")] + [str(a) for a in args], check=True, capture_output=True, text=True).stdout
        keys = ("n", "which", "tb", "S", "epilogue", "own", "G", "rows", "out_rows", "parts")
        return [dict(zip(keys, map(int, line.split()))) for line in out.splitlines()]
    return run


def _builds():
    text = open(os.path.join(CSRC, "knnssd.hip")).read()
    kinds = ("PF_PARTS", "PF_SWIGLU", "PF_ROPE")
    found = re.findall(r"^    pf_build(?:_wide)?<(?:\d+, )?(\d+), (?:\d+, \d+, \w+, )?(\w+), (\w+)>\(f\);", text, re.M)
    return {(int(tb), kinds.index(epi), int(own == "true")) for tb, epi, own in found}


def test_gpu_prompts_reach_every_build(plans):
    builds = _builds()
    assert len(builds) == 13
    reached = {(p["tb"], p["epilogue"], p["own"]) for shape, lengths in ((WIDE, PROMPTS), (OPERANDS, OPERAND_PROMPTS)) + SPLIT
               for p in plans(shape, lengths) if p["G"] == 0}
    assert reached == builds, builds ^ reached


@pytest.mark.parametrize("shape", [WIDE, dict(d_model=5120, n_heads=40, n_kv_heads=8, head_dim=128, d_ffn=13824),
                                   dict(d_model=320, n_heads=2, n_kv_heads=1, head_dim=64, d_ffn=352)])
def test_every_plan_has_a_build(plans, shape):
    builds = _builds()
    qd = shape["n_heads"] * shape["head_dim"]
    width = [qd, shape["d_model"], 2 * shape["d_ffn"], shape["d_model"]]
    for p in plans(shape, list(range(17, 900, 13)) + [1024, 1025, 4096, 15360]):
        if p["G"] == 0:
            assert (p["tb"], p["epilogue"], p["own"]) in builds, p
            assert p["epilogue"] == 0 or p["S"] == 1, p
        assert p["out_rows"] >= p["n"] and p["rows"] >= width[p["which"]]
        assert p["parts"] or p["which"] in (0, 2)      # the residual rows are always finished by a row kernel
