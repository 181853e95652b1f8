"""How short prompts' products are dealt to workgroups (host code): equal runs over the tiles' pairs of steps, the number of parts a
row kernel reads per tile, and the row tiles a run touches."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_16162_amd", "csrc")

DRIVER = r'''
#include <cstdio>
#include <cstdlib>
#include "prefill_plan.h"
int main(int n, char **v) {
    knnssd_model_cfg g{};
    g.d_model = atoi(v[1]); g.n_heads = atoi(v[2]); g.n_kv_heads = atoi(v[3]); g.head_dim = atoi(v[4]); g.d_ffn = atoi(v[5]);
    for (int w = 0; w < ks::PF_OPS; ++w)
        for (int tt = 2; tt <= 5; ++tt) {
            const ks::PfPlan p = ks::pf_choose(g, w, tt), r = ks::pf_tiles(g, w, tt);
            const int K = w == ks::PF_O ? g.n_heads * g.head_dim : (w == ks::PF_DOWN ? g.d_ffn : g.d_model), KP = (K / 32 + 1) / 2, units = p.n_mt * KP;
            printf("%d %d %d %d %d %d %d %d\n", w, tt, p.G, p.S, p.n_mt * p.tm(), p.out_rows(), (int)(p.parts(w)), (int)(p.tb == r.tb && p.S == r.S));
            if (!p.G) continue;
            // every unit belongs to the run that pf_share gives it to; parts and tiles of a run by counting
            int most = 0, touched = 0;
            for (int g0 = 0; g0 < p.G; ++g0) {
                const int a = ks::pf_share(units, p.G, g0), b = ks::pf_share(units, p.G, g0 + 1);
                if (b <= a) { puts("empty run"); return 1; }
                for (int u = a; u < b; ++u)
                    if (ks::pf_share_owner(units, p.G, u) != g0) { puts("owner"); return 1; }
                if ((b - 1) / KP - a / KP + 1 > touched) touched = (b - 1) / KP - a / KP + 1;
            }
            for (int t = 0; t < p.n_mt; ++t) {
                const int parts = ks::pf_share_owner(units, p.G, (t + 1) * KP - 1) - ks::pf_share_owner(units, p.G, t * KP) + 1;
                if (parts > most) most = parts;
            }
            if (most != p.S || touched > ks::PF_THIN_TILES) { printf("parts %d of %d, tiles %d\n", most, p.S, touched); return 1; }
        }
    if (ks::pf_share(1000, 7, 7) != 1000 || ks::pf_share(1000, 7, 0) != 0) return 1;
    return 0;
}
'''


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("thin")
    (tmp / "driver.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-o", str(tmp / "driver"), str(tmp / "driver.cpp")], check=True)
    return str(tmp / "driver")


CHAIN = r'''
#include <cstdio>
#include <cstdlib>
#include "prefill_plan.h"
int main(int n, char **v) {
    knnssd_model_cfg g{};
    g.d_model = atoi(v[1]); g.n_heads = atoi(v[2]); g.n_kv_heads = atoi(v[3]); g.head_dim = atoi(v[4]); g.d_ffn = atoi(v[5]);
    for (int w = 0; w < ks::PF_OPS; ++w)
        for (int tt = 2; tt <= 3; ++tt) {
            const ks::PfPlan p = ks::pf_choose(g, w, tt), r = ks::pf_plan(g, w, tt);
            if (!p.G || !r.own_sums(w)) continue;
            const int K = w == ks::PF_O ? g.n_heads * g.head_dim : (w == ks::PF_DOWN ? g.d_ffn : g.d_model), KP = (K / 32 + 1) / 2, units = p.n_mt * KP;
            const int run = (units + p.G - 1) / p.G < KP ? (units + p.G - 1) / p.G : KP;       // pairs of steps
            printf("%d %d %d %d %d\n", run, ks::PF_THIN_FOLD, p.S, (K / 32 + r.S - 1) / r.S, r.S);
        }
}
'''


@pytest.mark.parametrize("shape", [(4096, 32, 32, 128, 11008), (5120, 40, 40, 128, 13824), (5120, 40, 8, 128, 13824), (3200, 25, 25, 128, 8640), (8192, 64, 8, 128, 28672)])
def test_no_sum_has_more_roundings_in_a_row_than_with_tiles(tmp_path, shape):
    """Steps within a fold, folds and parts, against steps within a part and parts of the 128 x 64 tiles (both add a step's planes on their own)."""
    (tmp_path / "chain.cpp").write_text(CHAIN)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, "-o", str(tmp_path / "chain"), str(tmp_path / "chain.cpp")], check=True)
    lines = subprocess.run([str(tmp_path / "chain")] + [str(v) for v in shape], check=True, capture_output=True, text=True).stdout.splitlines()
    assert lines
    for line in lines:
        run, fold, parts, steps, tile_parts = map(int, line.split())
        assert min(2 * fold, 2 * run) + -(-run // fold) + parts <= steps + tile_parts, line


@pytest.mark.parametrize("shape,thin", [((4096, 32, 32, 128, 11008), {0, 2, 3}), ((5120, 40, 40, 128, 13824), {0, 1, 2, 3}), ((2080, 4, 2, 128, 6048), {2}),
                                        ((320, 2, 1, 64, 352), set()), ((64, 2, 1, 64, 120000), set()), ((8192, 64, 8, 128, 28672), {0, 1, 2, 3})])
def test_runs_cover_the_steps(driver, shape, thin):
    """`thin`: the matrices (QKV, O, gate+up, down) that prompts of up to three token tiles stream this way."""
    out = subprocess.run([driver] + [str(v) for v in shape], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    d, h, kvh, hd, f = shape
    width = [(h + 2 * kvh) * hd, d, 2 * f, d]
    for line in out.stdout.splitlines():
        w, tt, g, s, rows, out_rows, parts, same = map(int, line.split())
        assert (g > 0) == (w in thin and tt <= 3), line
        assert g > 0 or same, line
        assert rows >= width[w] and out_rows >= 16 * tt
        assert not g or (parts and 1 <= s)
