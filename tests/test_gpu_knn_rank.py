"""The ranking behind a scan at the edges of its slices: one workgroup with entries past its registers, two slices, a short
last slice; ties across slices, negative scores, and the best anchors in the first or last places of a slice."""
import pytest
import torch

from oracle import knnssd_oracle as O
from paper_2505_16162_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.mark.timeout(120)
@pytest.mark.parametrize("n", [15, 1023, 4096, 4097, 8191, 8192, 8193, 12289, 40960])
@pytest.mark.parametrize("k", [1, 7, 15])
def test_rank_at_slice_edges(n, k):
    d, n_dom = 64, 5
    g = torch.Generator().manual_seed(n * 17 + k)
    anchors = torch.randn(n, d, generator=g)
    queries = torch.randn(3, d, generator=g)
    anchors[-1] = 2.0 * queries[0]                        # cosine 1 in the last place
    if n > 4097:
        anchors[4095], anchors[4096] = queries[1], queries[1]      # the same score on both sides of a slice edge: the lower index first
    anchors[0] = -queries[2]                              # the worst one first
    labels = torch.randint(0, n_dom, (n,), generator=g).int()
    shape = synth.ModelShape("rank", 1, d, 1, 1, 64, 64, 64, 16, "fp32", "fp32")
    gpu = binding.KnnSsd(shape, synth.make_weights(shape, seed=1), max_anchors=n)
    gpu.knnssd_set_anchors(anchors.cuda(), labels.cuda(), synth.make_block_masks(1, n_dom, 0, seed=2))
    for _ in range(2):                                    # the arrival counters are as they were
        idx, cos, dom = gpu.knnssd_knn_topk(queries.cuda(), k)
    for i in range(3):
        order, scores, want_dom = O.knn_topk_vote(queries[i].numpy(), anchors.numpy(), labels.numpy(), k)
        # fp32 sums of 64 products: scores closer than 1e-6 may change places
        for r in range(k):
            assert abs(cos[i][r] - scores[r]) <= 1e-6, (i, r)
            assert idx[i][r] == order[r] or abs(float(scores[r]) - cos[i][r]) <= 1e-6
        assert len(set(idx[i])) == k
        if list(idx[i]) == list(order):
            assert dom[i] == want_dom
        one, one_dom, _ = gpu.knnssd_select_skipset(queries[i].cuda())
        assert one == idx[i][0] and one_dom == int(labels[one])
    if n > 4097 and k > 1:
        assert idx[1][:2] == [4095, 4096]
    assert idx[0][0] == n - 1
    gpu.close()
