"""The ranking behind a scan at the edges of its slices: one workgroup with entries past its registers, two slices, a short
last slice; ties across slices, negative scores, and the best anchors in the first or last places of a slice."""
import pytest
import torch

from oracle import knnssd_oracle as O
from paper_2505_16162_amd import binding, synth

pytestmark = pytest.mark.gpu


def _check(query, anchors, labels, k, idx, cos, dom):
    """One query's result against the oracle. TOL: fp32 sums of 64 products of a unit query's size; two scores each off by as much may change places
    if they are closer than twice that."""
    TOL = 1e-6
    exact = O.cosine_scores(query.numpy().astype("float64"), anchors.numpy().astype("float64"))
    order, scores, _ = O.knn_topk_vote(query.numpy(), anchors.numpy(), labels.numpy(), min(k + 1, len(exact)))
    assert len(set(idx)) == k
    for r in range(k):
        assert abs(cos[r] - exact[idx[r]]) <= TOL, r          # the cosine of the anchor that was returned
        assert abs(cos[r] - scores[r]) <= TOL, r              # ... which is the one of this rank, unless neighbours in the order are that close
        apart = (r == 0 or scores[r - 1] - scores[r] > 2 * TOL) and (r + 1 == len(scores) or scores[r] - scores[r + 1] > 2 * TOL)
        assert idx[r] == order[r] or not apart, r
        assert r == 0 or cos[r - 1] > cos[r] or (cos[r - 1] == cos[r] and idx[r - 1] < idx[r]), r
    voted = [int(labels[n]) for n in idx]
    assert dom == max(voted, key=lambda lab: (voted.count(lab), -voted.index(lab)))


@pytest.mark.timeout(120)
@pytest.mark.parametrize("n", [16, 1023, 4096, 4097, 8191, 8192, 8193, 12289, 13499, 13500, 40960])
@pytest.mark.parametrize("k", [1, 7, 15, 16])
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
        _check(queries[i], anchors, labels, k, idx[i], cos[i], dom[i])
        one, one_dom, _ = gpu.knnssd_select_skipset(queries[i].cuda())
        assert one == idx[i][0] and one_dom == int(labels[one])
    if n > 4097 and k > 1:
        assert idx[1][:2] == [4095, 4096]
    assert idx[0][0] == n - 1
    gpu.close()
