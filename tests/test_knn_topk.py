"""K > 1 nearest anchors with a majority vote, batched queries: oracle pins (CPU) and GPU parity."""
import os
import subprocess
import numpy as np
import pytest
import torch

from oracle import knnssd_oracle as O
from paper_2505_16162_amd import synth


def _table(n, d, n_dom, seed, sigma=0.3):
    anchors, labels, centres = synth.make_anchors(d, n, n_dom, sigma, seed=seed)
    return anchors, labels, centres


def test_k1_is_the_routing_argmax():
    anchors, labels, centres = _table(200, 64, 5, seed=1)
    masks = np.zeros((5, 8), dtype=np.uint8)
    for i in range(20):
        q = synth.make_domain_query(centres, i % 5, 0.3, seed=50 + i).numpy()
        n_star, dom, _, _ = O.knn_select(q, anchors.numpy(), labels.numpy(), masks)
        order, cos, d1 = O.knn_topk_vote(q, anchors.numpy(), labels.numpy(), 1)
        assert order == [n_star] and d1 == dom


def test_topk_against_brute_force_and_planted_neighbours():
    rng = np.random.default_rng(3)
    anchors = rng.standard_normal((40, 16))
    labels = np.arange(40) % 4
    q = rng.standard_normal(16)
    # brute force written out: cosine of every pair, full sort
    cos = [float(np.dot(q, a) / (np.linalg.norm(q) * np.linalg.norm(a))) for a in anchors]
    want = sorted(range(40), key=lambda n: (-np.float32(cos[n]), n))[:7]
    order, scores, _ = O.knn_topk_vote(q, anchors, labels, 7)
    assert order == want
    assert np.allclose(scores, [cos[n] for n in want], atol=1e-12)
    assert all(scores[i] >= scores[i + 1] for i in range(6))
    # planted: three anchors are positive multiples of the query -> cosine 1, index order among them
    anchors[[31, 5, 17]] = np.outer([2.0, 0.5, 7.0], q)
    order, scores, _ = O.knn_topk_vote(q, anchors, labels, 3)
    assert order == [5, 17, 31] and np.allclose(scores, 1.0)


def test_vote_rule():
    q = np.array([1.0, 0.0])
    # ranked by cosine: anchors 0,1,2,3,4 with labels B A A B C
    ang = [0.01, 0.02, 0.03, 0.04, 0.05]
    anchors = np.array([[np.cos(t), np.sin(t)] for t in ang])
    labels = np.array([1, 0, 0, 1, 2])
    assert O.knn_topk_vote(q, anchors, labels, 1)[2] == 1
    assert O.knn_topk_vote(q, anchors, labels, 3)[2] == 0          # A has two of three
    assert O.knn_topk_vote(q, anchors, labels, 2)[2] == 1          # one each: the better-ranked label
    assert O.knn_topk_vote(q, anchors, labels, 4)[2] == 1          # two each: B's best anchor ranks first
    assert O.knn_topk_vote(q, anchors, labels, 5)[2] == 1


@pytest.mark.gpu
@pytest.mark.parametrize("n,k,nq", [(40, 1, 1), (777, 3, 5), (777, 16, 4), (5000, 8, 9)])
def test_gpu_topk_matches_oracle(n, k, nq):
    from paper_2505_16162_amd import binding
    from gpu_common import make_pair
    shape = synth.small_shape("knnk", d_ffn=704, max_seq=64)
    n_dom = 5
    w, orc, gpu = make_pair(shape, seed=2, max_anchors=n)
    anchors, labels, centres = _table(n, shape.d_model, n_dom, seed=9)
    masks = synth.make_block_masks(shape.n_blocks, n_dom, 1, seed=6)
    gpu.knnssd_set_anchors(anchors, labels, masks)
    queries = torch.stack([synth.make_domain_query(centres, i % n_dom, 0.3, seed=300 + i) for i in range(nq)])
    idx, cos, dom = gpu.knnssd_knn_topk(queries, k)
    for i in range(nq):
        order, scores, d = O.knn_topk_vote(queries[i].numpy(), anchors.numpy(), labels.numpy(), k)
        # fp32 sums on the GPU against fp64 in the oracle: the ranking is unique wherever neighbouring scores differ
        # by more than the rounding error, which seeded Gaussian data satisfies with a wide margin
        assert idx[i] == order, (i, idx[i], order)
        assert np.allclose(cos[i], scores, atol=2e-6)
        assert dom[i] == d
    # the K = 1 result is the routing call's
    a1, d1, _ = gpu.knnssd_select_skipset(queries[0])
    assert [a1] == gpu.knnssd_knn_topk(queries[:1], 1)[0][0] and d1 == gpu.knnssd_knn_topk(queries[:1], 1)[2][0]
    with pytest.raises(binding.KnnSsdError):
        gpu.knnssd_knn_topk(queries, 17)
    with pytest.raises(binding.KnnSsdError):
        gpu.knnssd_knn_topk(torch.zeros_like(queries), k)      # zero-norm query
    gpu.close()


@pytest.mark.gpu
@pytest.mark.parametrize("n,k", [(16, 16), (20, 16), (70, 5), (3000, 16), (9000, 7)])
def test_gpu_topk_ties_short_tables_and_bad_anchors(n, k):
    """The selection's own edges: exact ties (every anchor stored several times, so equal scores must come out lowest
    index first, across the lanes, wavefronts and slices that rank parts of the table), tables shorter than a
    wavefront's share or than K allows to be dropped, and a non-finite anchor anywhere in the table."""
    from paper_2505_16162_amd import binding
    from gpu_common import make_pair
    shape = synth.small_shape("knnties", d_ffn=704, max_seq=64)
    n_dom = 4
    w, orc, gpu = make_pair(shape, seed=2, max_anchors=n)
    base, _, centres = _table((n + 3) // 4, shape.d_model, n_dom, seed=11)
    # copies of one anchor sit a quarter of the table apart (different lanes, wavefronts, slices); scaled copies have
    # the same cosine up to rounding only, so the copies are exact
    anchors = torch.cat([base, base, base, base])[:n].contiguous()
    labels = (torch.arange(n) % n_dom).to(torch.int32)
    masks = synth.make_block_masks(shape.n_blocks, n_dom, 1, seed=6)
    gpu.knnssd_set_anchors(anchors, labels, masks)
    queries = torch.stack([synth.make_domain_query(centres, i % n_dom, 0.3, seed=40 + i) for i in range(4)])
    idx, cos, dom = gpu.knnssd_knn_topk(queries, k)
    for i in range(4):
        order, scores, d = O.knn_topk_vote(queries[i].numpy(), anchors.numpy(), labels.numpy(), k)
        assert idx[i] == order, (i, idx[i], order)
        assert np.allclose(cos[i], scores, atol=2e-6)
        assert dom[i] == d
    a1, d1, _ = gpu.knnssd_select_skipset(queries[1])
    assert a1 == idx[1][0]
    bad = anchors.clone()
    bad[n - 1, 3] = float("nan")
    gpu.knnssd_set_anchors(bad, labels, masks)
    with pytest.raises(binding.KnnSsdError):
        gpu.knnssd_knn_topk(queries, min(k, 2))
    with pytest.raises(binding.KnnSsdError):
        gpu.knnssd_select_skipset(queries[0])
    gpu.close()


@pytest.mark.gpu
@pytest.mark.timeout(600)
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_gpu_scan_of_a_large_table_matches_oracle(dtype):
    """The regime in which the scan is bound by HBM: 100 000 anchors of dimension 5120 (2 GB in fp32, 1 GB in bf16),
    the routing arg-max and the 8 nearest with their vote against the exhaustive oracle. A bf16 table is rounded
    once by the caller; both sides then search the same rounded values."""
    from paper_2505_16162_amd import binding
    n, d, n_dom, k = 100_000, 5120, 5, 8
    shape = synth.small_shape("knn_big", n_blocks=1, d_model=d, n_heads=40, n_kv_heads=40, head_dim=128, d_ffn=1024,
                              vocab=1024, max_seq=64)
    w = synth.make_weights(shape, device="cuda:0", seed=3)
    gpu = binding.KnnSsd(shape, w, max_anchors=n)
    print("anchors", flush=True)
    # sigma 1: neighbouring scores are well apart (a table of near-duplicates would make the ranking a coin toss)
    anchors, labels, centres = synth.make_anchors(d, n, n_dom, 1.0, seed=21, device="cuda:0")
    if dtype == "bf16":
        anchors = anchors.to(torch.bfloat16)
    masks = synth.make_block_masks(shape.n_blocks, n_dom, 1, seed=6)
    gpu.knnssd_set_anchors(anchors, labels, masks)
    a64 = anchors.float().cpu().numpy()          # the stored values, exactly
    lab = labels.cpu().numpy()
    queries = torch.stack([synth.make_domain_query(centres.cpu(), i % n_dom, 1.0, seed=700 + i) for i in range(3)])
    print("gpu", flush=True)
    idx, cos, dom = gpu.knnssd_knn_topk(queries, k)
    for i in range(3):
        print("oracle query", i, flush=True)
        order, scores, dvote = O.knn_topk_vote(queries[i].numpy(), a64, lab, k)
        gaps = [scores[r] - scores[r + 1] for r in range(k - 1)]
        assert idx[i] == order, (i, idx[i], order, min(gaps))
        assert np.allclose(cos[i], scores, atol=3e-6)
        assert dom[i] == dvote
        n_star, d_star, mask, _ = O.knn_select(queries[i].numpy(), a64, lab, masks.numpy())
        a1, d1, m1 = gpu.knnssd_select_skipset(queries[i])
        assert (a1, d1, m1) == (n_star, d_star, mask.tolist())
    gpu.close()


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,n,d", [("bf16", 8191, 264), ("bf16", 8192, 264), ("bf16", 8195, 1000), ("bf16", 9001, 8), ("bf16", 16385, 512), ("bf16", 33000, 520),
                                       ("fp32", 32767, 72), ("fp32", 32768, 256), ("fp32", 32771, 264), ("fp32", 40002, 520),
                                        ("bf16", 11468, 2048), ("bf16", 11469, 2056), ("bf16", 16384, 2560), ("bf16", 16387, 2504), ("bf16", 33001, 2048),
                                        ("fp32", 11471, 2056), ("fp32", 12001, 4104), ("fp32", 16384, 4104), ("fp32", 17001, 4104), ("fp32", 33002, 8),
                                        ("bf16", 131072, 8), ("bf16", 131075, 264), ("fp32", 131073, 248)])
def test_gpu_scan_kernels_agree(dtype, n, d):
    """Around the sizes from which two, three or four queries take the streaming scan: rows in whole and broken blocks, tables that end within
    a wavefront's four anchors, fewer and more groups of them than wavefronts. Every query gets the same bits alone (the
    other kernel) as among two, three or four; against 64 bits; a non-finite anchor is met in both."""
    from paper_2505_16162_amd import binding
    shape = synth.small_shape("knn_scan", n_blocks=1, d_model=d, max_seq=64)
    gpu = binding.KnnSsd(shape, synth.make_weights(shape, seed=4), max_anchors=n)
    anchors, labels, centres = synth.make_anchors(d, n, 5, 1.0, seed=31)
    if dtype == "bf16":
        anchors = anchors.to(torch.bfloat16)
    masks = synth.make_block_masks(1, 5, 0, seed=6)
    gpu.knnssd_set_anchors(anchors, labels, masks)
    queries = torch.stack([synth.make_domain_query(centres, i % 5, 1.0, seed=800 + i) for i in range(4)])
    a64 = anchors.double()
    want = (a64 @ queries.double().T / a64.norm(dim=1, keepdim=True)) / queries.double().norm(dim=1)
    one = [gpu.knnssd_knn_topk(queries[i:i + 1], 9) for i in range(4)]
    for nq in (2, 3, 4):
        idx, cos, dom = gpu.knnssd_knn_topk(queries[:nq], 9)
        for i in range(nq):
            assert (idx[i], cos[i], dom[i]) == (one[i][0][0], one[i][1][0], one[i][2][0]), (nq, i)
    for i in range(4):
        # fp32 sums of d terms of either sign: a few units in the last place of the score
        assert np.allclose(one[i][1][0], want[one[i][0][0], i].numpy(), atol=2e-6)
        assert np.allclose(one[i][1][0], torch.topk(want[:, i], 9).values.numpy(), atol=2e-6)
    bad = anchors.clone()
    bad[n - 1, d - 1] = float("inf")
    gpu.knnssd_set_anchors(bad, labels, masks)
    for nq in (1, 3):
        with pytest.raises(binding.KnnSsdError):
            gpu.knnssd_knn_topk(queries[:nq], 2)
    gpu.close()


@pytest.fixture(scope="module")
def streams(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("scan")
    (tmp / "driver.cpp").write_text("""
#include <cstdio>
#include <cstdlib>
#include "knn_plan.h"
int main(int n, char **v) { for (int i = 1; i + 3 < n; i += 4) printf("%d ", ks::knn_streams(atoi(v[i]), atoi(v[i + 1]), atoi(v[i + 2]), atoi(v[i + 3]))); }
""")
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_16162_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", csrc, "-o", str(tmp / "driver"), str(tmp / "driver.cpp")], check=True)
    return lambda cases: [int(x) for x in subprocess.run([str(tmp / "driver")] + [str(a) for c in cases for a in c], check=True, capture_output=True, text=True).stdout.split()]


def test_scans_take_the_faster_kernel(streams):
    """Whole calls measured on an MI355X in us: (queries, bf16, anchors, elements), the kernel that reads its queries from the cache, the streaming one."""
    measured = [((2, 1, 8192, 5120), 52.5, 58.7), ((3, 1, 8192, 256), 41.3, 42.8), ((2, 1, 24000, 1000), 46.8, 49.2), ((4, 1, 50000, 512), 50.9, 53.7),
                ((2, 1, 100000, 512), 55.3, 58.5), ((2, 1, 200000, 1000), 100.1, 105.2), ((2, 1, 32768, 2048), 68.1, 61.1), ((4, 1, 65536, 2048), 99.7, 82.6),
                ((3, 1, 200000, 5120), 416.7, 365.2), ((4, 1, 200000, 5120), 470.5, 371.9), ((2, 1, 4096, 8192), 54.8, 63.6), ((3, 1, 200000, 256), 79.7, 73.7),
                ((2, 0, 8192, 5120), 64.5, 73.4), ((2, 0, 50000, 2048), 98.5, 108.2), ((2, 0, 24000, 4096), 99.0, 106.5), ((2, 0, 50000, 4096), 163.6, 178.1),
                ((2, 0, 50000, 1000), 68.4, 73.7), ((3, 0, 100000, 2048), 162.9, 173.3), ((3, 0, 16384, 4096), 92.5, 82.7), ((4, 0, 24000, 5120), 138.7, 123.0),
                ((2, 0, 16384, 8192), 137.5, 121.5), ((2, 0, 200000, 256), 87.1, 71.5), ((4, 0, 200000, 256), 90.8, 79.4), ((1, 0, 200000, 5120), 640, 657),
                ((1, 1, 200000, 5120), 353, 355), ((3, 0, 20000, 5120), 109.6, 117.3), ((4, 0, 20000, 4096), 99.2, 102.5), ((4, 1, 20000, 5120), 104, 92), ((3, 0, 100000, 512), 68.8, 72.4)]
    for (case, multi, stream), chosen in zip(measured, streams([m[0] for m in measured])):
        assert chosen == (stream < multi), case


def test_routing_takes_the_faster_ranking(tmp_path):
    """Whole routing calls measured on an MI355X in us: (anchors, elements), one workgroup, slices; from KNN_RANK_ONE anchors on the slices rank. A
    tenth of a microsecond or two is noise."""
    measured = [((8, 256), 18.9, 20.1), ((1000, 256), 20.2, 21.3), ((4097, 256), 21.1, 22.4), ((8000, 1000), 25.0, 26.5), ((8192, 256), 22.6, 24.3), ((8192, 5120), 44.4, 45.8),
                ((10000, 1000), 26.6, 27.9), ((12000, 64), 23.9, 24.2), ((12000, 2048), 34.5, 35.2), ((13000, 256), 24.8, 24.9), ((13000, 5120), 60.7, 60.9),
                ((14000, 256), 25.1, 25.1), ((14000, 2048), 37.4, 37.0), ((14000, 5120), 62.6, 62.2), ((16000, 1000), 31.4, 30.3), ((20000, 5120), 81.7, 80.6), ((100000, 256), 74.9, 44.5)]
    (tmp_path / "driver.cpp").write_text('#include <cstdio>\n#include "knn_plan.h"\nint main() { printf("%d", ks::KNN_RANK_ONE); }\n')
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_16162_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-I", csrc, "-o", str(tmp_path / "driver"), str(tmp_path / "driver.cpp")], check=True)
    least = int(subprocess.run([str(tmp_path / "driver")], check=True, capture_output=True, text=True).stdout)
    for (anchors, _), one, slices in measured:
        assert (slices if anchors >= least else one) <= min(one, slices) + 0.2, anchors


def test_kernel_pairs_of_the_gpu_test_cross_every_edge(streams):
    """The sizes of test_gpu_scan_kernels_agree take both kernels for each query count and type."""
    sizes = [m for m in test_gpu_scan_kernels_agree.pytestmark if m.name == "parametrize"][0].args[1]
    for q in (2, 3, 4):
        for dtype in ("bf16", "fp32"):
            taken = streams([(q, int(dtype == "bf16"), n, d) for t, n, d in sizes if t == dtype])
            assert set(taken) == {0, 1}, (q, dtype)
    assert not any(streams([(1, b, n, d) for b in (0, 1) for _, n, d in sizes]))
