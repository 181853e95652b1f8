"""The times of a generation: drafts' and verifications', from the device's clock, are the whole decode between the events around it; with no
draft, a fixed count, the confidence stop (passes enqueued in vain among them), on each kind of kernels."""
import pytest

from paper_2505_16162_amd import binding, synth

pytestmark = pytest.mark.gpu

KINDS = {
    "one launch": dict(weight_dtype="fp32", kv_dtype="fp32", n_blocks=4, vocab=1024, max_seq=200),
    "launches": dict(weight_dtype="fp32", kv_dtype="fp32", n_blocks=4, vocab=1024, max_seq=200),
    "tuned": dict(n_blocks=3, d_ffn=704, vocab=1500, max_seq=200),
}


@pytest.mark.timeout(120)
@pytest.mark.parametrize("kind", sorted(KINDS))
def test_draft_and_verify_times_are_the_whole_decode(kind):
    shape = synth.small_shape("times", **KINDS[kind])
    w = synth.make_weights(shape, seed=91, gains="random", std=0.05)
    gpu = binding.KnnSsd(shape, w)
    assert gpu.packed == (kind == "tuned")
    if kind == "launches":
        gpu.knnssd_set_pass_mode("launches")
    prompt = synth.make_prompt(shape.vocab, 40, seed=92).tolist()
    gpu.knnssd_set_skipset([1, 1] + [0, 0] * (shape.n_blocks - 1))
    for max_draft, conf in ((0, 0.0), (4, 0.0), (15, 0.0), (4, 0.02), (8, 0.9), (3, 1e-6)):
        missing = []
        for turn in range(4):                # the first one loads code
            _, st = gpu.knnssd_generate(prompt, 90, max_draft, conf, route=False)
            decode = st["ns_total"] - st["ns_prefill"] - st["ns_knn"]
            missing.append(decode - st["ns_draft"] - st["ns_verify"])
            print("case", kind, max_draft, conf, st, flush=True)
            assert (st["ns_draft"] == 0) == (st["drafted"] == 0) and st["ns_draft"] >= 0 and st["ns_verify"] > 0
            assert st["rounds"] == st["verify_passes"] and st["drafted"] == st["draft_passes"]
        # outside of them: the launch in front of the first round, the event behind the last one (30 to 60 us; the host may have been held up once)
        assert min(missing) >= -20e3 and sorted(missing)[1] <= 150e3 and decode > 2e6, (missing, decode)
    gpu.close()
