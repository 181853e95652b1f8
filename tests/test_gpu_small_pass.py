"""Passes of small models in one launch: the smallest widths (one value per workgroup in some steps), ragged ones, both head sizes,
grouped-query heads, weights just under and over the size up to which a pass is one launch, skipped sublayers, contexts of
several rounds of the attention, every row count the builds split at. Logits against the oracle (and a row's logits the same however
many rows share its pass), and many contexts at once on streams of their own: more workgroups than the chip holds."""
import threading

import pytest
import torch

from paper_2505_16162_amd import binding, synth
from gpu_common import logits_close, make_pair

pytestmark = pytest.mark.gpu

# block bytes of "under" / "over": 8 x 1024 x 1024 is the limit
SHAPES = {
    "least": dict(n_blocks=1, d_model=8, n_heads=1, n_kv_heads=1, head_dim=64, d_ffn=64, vocab=17, max_seq=200),
    "ragged": dict(n_blocks=3, d_model=248, n_heads=3, n_kv_heads=1, head_dim=128, d_ffn=72, vocab=1003, max_seq=300),
    "wide_ffn": dict(n_blocks=2, d_model=72, n_heads=2, n_kv_heads=2, head_dim=64, d_ffn=1096, vocab=513, max_seq=200),
    "under": dict(n_blocks=1, d_model=520, n_heads=4, n_kv_heads=2, head_dim=64, d_ffn=832, vocab=600, max_seq=120),
    "over": dict(n_blocks=1, d_model=520, n_heads=4, n_kv_heads=2, head_dim=64, d_ffn=1120, vocab=600, max_seq=120),
}


@pytest.mark.timeout(300)
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("name", sorted(SHAPES))
def test_logits_and_rows(name, dtype):
    shape = synth.small_shape("small_%s_%s" % (name, dtype), weight_dtype=dtype, kv_dtype=dtype, **SHAPES[name])
    w, orc, gpu = make_pair(shape, seed=61, std=0.05)
    assert not gpu.packed
    n_all = shape.max_seq - 20
    tokens = synth.make_prompt(shape.vocab, n_all + 16, seed=62).tolist()
    rows = orc.forward(tokens, 0, None)
    for ctx in sorted({1, 15, 17, 63, 65, n_all}):
        print("case", shape.name, ctx, flush=True)
        gpu.knnssd_prefill(tokens[:ctx])
        kept = {}
        for n in (16, 1, 2, 3, 4, 5, 6, 9, 10, 15):
            gpu.knnssd_verify(tokens[ctx:ctx + n], ctx)
            for r in {0, n // 2, n - 1}:
                got = gpu.knnssd_get_logits(r).clone()
                if r in kept:
                    assert torch.equal(got, kept[r]), (ctx, n, r)
                kept[r] = got
        for r, got in kept.items():
            ok, err = logits_close(got.numpy(), rows[ctx + r], shape)
            assert ok, (ctx, r, err)
    gpu.close()


@pytest.mark.timeout(300)
@pytest.mark.parametrize("mask", [(0, 1), (1, 0), (1, 1)])
def test_skipped_sublayers(mask):
    shape = synth.small_shape("small_mask", weight_dtype="fp32", kv_dtype="fp32", n_blocks=3, d_model=136, n_heads=2, n_kv_heads=1, head_dim=64,
                              d_ffn=200, vocab=311, max_seq=64)
    w, orc, gpu = make_pair(shape, seed=63, std=0.05)
    tokens = synth.make_prompt(shape.vocab, 30, seed=64).tolist()
    skip = list(mask) + [0, 0] + list(mask)
    gpu.knnssd_set_skipset(skip)
    gpu.knnssd_prefill(tokens[:20])
    orc.forward(tokens[:20], 0, None)
    for i in range(20, 26):
        gpu.knnssd_draft_step(tokens[i], i)
        want = orc.forward([tokens[i]], i, skip)[0]
        ok, err = logits_close(gpu.knnssd_get_logits(0).numpy(), want, shape)
        assert ok, (i, err)
    gpu.close()


@pytest.mark.timeout(300)
def test_many_contexts_at_once():
    shape = synth.small_shape("small_streams", weight_dtype="fp32", kv_dtype="fp32", n_blocks=4, vocab=1024, max_seq=96)
    w = {k: ([{n: t.cuda() for n, t in b.items()} for b in v] if k == "blocks" else v.cuda()) for k, v in synth.make_weights(shape, seed=65, gains="random", std=0.05).items()}
    prompts = [synth.make_prompt(shape.vocab, 20 + i, seed=70 + i).tolist() for i in range(10)]
    skip = [0, 0, 1, 1, 0, 0, 1, 1]

    def one(gpu, prompt):
        gpu.knnssd_set_skipset(skip)
        return gpu.knnssd_generate(prompt, 40, 4, 0.0, route=False)[0]

    alone = binding.KnnSsd(shape, w)
    want = [one(alone, p) for p in prompts]
    alone.close()
    ctxs = []
    for _ in prompts:
        with torch.cuda.stream(torch.cuda.Stream()):
            ctxs.append(binding.KnnSsd(shape, w))
    torch.cuda.synchronize()
    got = [None] * len(prompts)

    def run(i):
        for _ in range(3):
            got[i] = one(ctxs[i], prompts[i])

    threads = [threading.Thread(target=run, args=(i,)) for i in range(len(prompts))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for c in ctxs:
        c.close()
    assert got == want
