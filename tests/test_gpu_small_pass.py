"""Passes of small models in one launch: the smallest widths (one value per workgroup in some steps), ragged ones, both head sizes,
grouped-query heads, weights just under and over the size up to which a pass is one launch, skipped sublayers, contexts of
several rounds of the attention, every row count the builds split at. Logits against the oracle (and a row's logits the same however
many rows share its pass), launches whose workgroups give up waiting (all that a pass leaves behind is that of a launch per step,
bit for bit), and contexts in threads on streams of their own."""
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
    gpu.knnssd_set_pass_mode("one")         # wherever the pass fits
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
    gpu.knnssd_set_pass_mode("one")
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


BROKEN = dict(n_blocks=3, d_model=136, n_heads=3, n_kv_heads=1, head_dim=64, d_ffn=200, vocab=311, max_seq=96)


def _everything(gpu, tokens, skip):
    """What a prompt in three chunks (two of them without a head), draft steps with skipped sublayers, verifications of every build's row
    count and a generation return and leave in memory."""
    out = []
    gpu.kv.zero_()
    gpu.knnssd_set_skipset(skip)
    first, hidden = gpu.knnssd_prefill(tokens[:37])
    out += [first, hidden.cpu(), gpu.knnssd_get_logits(4), gpu.kv.cpu()]
    for i in range(3):
        out += [gpu.knnssd_draft_step(tokens[37 + i], 37 + i), gpu.knnssd_get_logits(0)]      # token and probability
    out.append(gpu.kv.cpu())
    for n in (16, 1, 2, 3, 5, 9):
        out.append(gpu.knnssd_verify(tokens[37:37 + n], 37))
        out += [gpu.knnssd_get_logits(r) for r in range(n)]
    out.append(gpu.kv.cpu())
    out += [gpu.knnssd_generate(tokens[:20], 12, 4, conf, route=False)[0] for conf in (0.0, 0.5)]
    out.append(gpu.kv.cpu())
    return out


def _same(a, b):
    return len(a) == len(b) and all(torch.equal(x, y) if isinstance(x, torch.Tensor) else x == y for x, y in zip(a, b))


@pytest.mark.timeout(300)
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_broken_up_launches_leave_what_whole_ones_leave(dtype):
    """A workgroup (the first, one in between, the last, every one) gives up its first wait in some block or in the head, the others theirs
    when the bound on it runs out; the one that stays runs the pass alone."""
    shape = synth.small_shape("small_broken_" + dtype, weight_dtype=dtype, kv_dtype=dtype, **BROKEN)
    w, orc, gpu = make_pair(shape, seed=66, std=0.05)
    tokens = synth.make_prompt(shape.vocab, 60, seed=67).tolist()
    skip = [0, 0, 1, 1, 0, 0]
    gpu.knnssd_set_pass_mode("launches")
    want = _everything(gpu, tokens, skip)
    assert gpu.knnssd_pass_counts() == (0, 0)
    gpu.knnssd_set_pass_mode("one")
    assert _same(_everything(gpu, tokens, skip), want)
    whole, broken = gpu.knnssd_pass_counts()
    assert whole > 12
    for wg, block in [(0, 0), (0, 3), (17, 0), (17, 2), (63, 1), (63, 3), (64, 0), (64, 2)]:
        print("case", dtype, wg, block, flush=True)
        gpu.knnssd_set_pass_mode("one", wg, block)
        before = gpu.knnssd_pass_counts()
        assert _same(_everything(gpu, tokens, skip), want), (wg, block)
        after = gpu.knnssd_pass_counts()
        assert after[0] - before[0] >= whole - 4
        # the head's wait is not met by the two chunks of a prompt that have no head; nor is a block by drafts that skip it
        assert after[1] - before[1] >= (whole if block == 0 else 8), (wg, block, before, after)
    gpu.knnssd_set_pass_mode("one")
    before = gpu.knnssd_pass_counts()
    assert _same(_everything(gpu, tokens, skip), want)
    print("broken up without a quitter:", gpu.knnssd_pass_counts()[1] - before[1], "of", gpu.knnssd_pass_counts()[0] - before[0])
    gpu.close()


@pytest.mark.timeout(300)
def test_a_pass_without_a_result_fails_the_call():
    shape = synth.small_shape("small_no_result", weight_dtype="fp32", kv_dtype="fp32", **BROKEN)
    w, orc, gpu = make_pair(shape, seed=68, std=0.05)
    tokens = synth.make_prompt(shape.vocab, 60, seed=69).tolist()
    skip = [0, 0, 1, 1, 0, 0]
    gpu.knnssd_set_pass_mode("one")
    want = _everything(gpu, tokens, skip)
    calls = [lambda: gpu.knnssd_verify(tokens[37:40], 37), lambda: gpu.knnssd_draft_step(tokens[37], 37), lambda: gpu.knnssd_prefill(tokens[:40]),
             lambda: gpu.knnssd_generate(tokens[:20], 12, 4, 0.0, route=False), lambda: gpu.knnssd_generate(tokens[:20], 12, 4, 0.5, route=False)]
    for block in (0, shape.n_blocks):
        for i, call in enumerate(calls):
            print("case", block, i, flush=True)
            gpu.knnssd_set_pass_mode("one")
            gpu.knnssd_prefill(tokens[:37])
            gpu.knnssd_set_pass_mode("one", 65, block)
            with pytest.raises(binding.KnnSsdError, match="without a result"):
                call()
    gpu.knnssd_set_pass_mode("one")
    assert _same(_everything(gpu, tokens, skip), want)
    gpu.close()


@pytest.mark.timeout(300)
@pytest.mark.parametrize("heads,hd,rows", [(16, 64, 9), (48, 64, 3), (15, 128, 9), (2, 128, 1), (2, 128, 2)])
def test_long_contexts_stay_whole(heads, hd, rows):
    """A context of thousands of positions, with more (row, head) items than are worked on side by side and with hardly any: the others'
    waits last."""
    shape = synth.small_shape("small_long", weight_dtype="bf16", kv_dtype="bf16", n_blocks=1, d_model=72, n_heads=heads, n_kv_heads=1, head_dim=hd, d_ffn=64,
                              vocab=100, max_seq=6000)
    gpu = binding.KnnSsd(shape, synth.make_weights(shape, seed=75, std=0.05), generic_kernels=True)
    tokens = synth.make_prompt(shape.vocab, 5900, seed=76).tolist()
    ctx = 5850
    gpu.knnssd_prefill(tokens[:ctx])
    out = {}
    for mode in ("launches", "one"):
        gpu.knnssd_set_pass_mode(mode)
        before = gpu.knnssd_pass_counts()
        for _ in range(3):
            out[mode] = [gpu.knnssd_verify(tokens[ctx:ctx + rows], ctx)] + [gpu.knnssd_get_logits(r) for r in range(rows)]
        after = gpu.knnssd_pass_counts()
        assert after[0] - before[0] == 3 * (mode == "one") and after[1] == before[1], (mode, before, after)
    assert _same(out["one"], out["launches"])
    gpu.close()


@pytest.mark.timeout(300)
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_the_choice_between_the_ways_changes_nothing(dtype):
    """Prompts, drafts and verifications on both sides of the context up to which a pass runs in one launch."""
    shape = synth.small_shape("small_choice_" + dtype, weight_dtype=dtype, kv_dtype=dtype, n_blocks=2, d_model=72, n_heads=4, n_kv_heads=2, head_dim=128,
                              d_ffn=104, vocab=211, max_seq=900)
    gpu = binding.KnnSsd(shape, synth.make_weights(shape, seed=77, std=0.05), generic_kernels=True)
    tokens = synth.make_prompt(shape.vocab, 900, seed=78).tolist()
    out, counts = {}, {}
    for mode in ("launches", "one", "auto"):
        gpu.knnssd_set_pass_mode(mode)
        before = gpu.knnssd_pass_counts()[0]
        gpu.kv.zero_()
        out[mode] = [gpu.knnssd_prefill(tokens[:870])[1].cpu()]
        for ctx in (40, 860):
            out[mode].append(gpu.knnssd_verify(tokens[ctx:ctx + 5], ctx))
            out[mode] += [gpu.knnssd_get_logits(r) for r in range(5)]
            gpu.knnssd_prefill(tokens[:ctx])
            out[mode] += [gpu.knnssd_draft_step(tokens[ctx], ctx), gpu.knnssd_get_logits(0), gpu.kv.cpu()]
            gpu.knnssd_prefill(tokens[:870])
        counts[mode] = gpu.knnssd_pass_counts()[0] - before
    assert _same(out["one"], out["launches"]) and _same(out["auto"], out["launches"])
    assert 0 == counts["launches"] < counts["auto"] < counts["one"]
    gpu.close()


@pytest.mark.timeout(300)
def test_a_broken_launch_is_followed_by_launches():
    shape = synth.small_shape("small_hold", weight_dtype="fp32", kv_dtype="fp32", **BROKEN)
    w, orc, gpu = make_pair(shape, seed=79, std=0.05)
    tokens = synth.make_prompt(shape.vocab, 40, seed=80).tolist()
    gpu.knnssd_prefill(tokens[:16])
    step = lambda: (gpu.knnssd_draft_step(tokens[16], 16), gpu.knnssd_get_logits(0).tolist())
    want = step()
    gpu.knnssd_set_pass_mode("auto", 3)
    whole, broken = gpu.knnssd_pass_counts()
    assert step() == want and gpu.knnssd_pass_counts() == (whole + 1, broken + 1)
    for i in range(64):
        assert step() == want and gpu.knnssd_pass_counts() == (whole + 1, broken + 1), i
    assert step() == want and gpu.knnssd_pass_counts() == (whole + 2, broken + 2)
    gpu.knnssd_set_pass_mode("auto")
    for i in range(128):
        assert step() == want and gpu.knnssd_pass_counts() == (whole + 2, broken + 2), i
    assert step() == want and gpu.knnssd_pass_counts() == (whole + 3, broken + 2)
    gpu.close()


@pytest.mark.timeout(300)
def test_a_round_knows_that_the_pass_before_was_broken_up():
    """A generation waits for a pass's number, not for the stream: the broken-up launch is counted before the number is there, so the very
    next pass is held back."""
    shape = synth.small_shape("small_hold_rounds", weight_dtype="fp32", kv_dtype="fp32", **BROKEN)
    w = synth.make_weights(shape, seed=81, std=0.05)
    prompt = synth.make_prompt(shape.vocab, 40, seed=82).tolist()
    for wg in (0, 3, 63, 64):
        gpu = binding.KnnSsd(shape, w, generic_kernels=True)
        want = gpu.knnssd_generate(prompt, 30, 0)[0]
        gpu.knnssd_set_pass_mode("auto", wg)
        whole, broken = gpu.knnssd_pass_counts()
        assert whole > 0 and broken == 0
        assert gpu.knnssd_generate(prompt, 30, 0)[0] == want          # 29 passes of one row, each waited for
        assert gpu.knnssd_pass_counts() == (whole + 1, 1), wg
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
    print("(one-launch passes, broken up):", [c.knnssd_pass_counts() for c in ctxs])
    for c in ctxs:
        c.close()
    assert got == want
