"""The many-row prefill at the edges of its tiles: prompts just below, at and above 16-, 64-, 128- and 256-row tiles, on
shapes whose row tiles are partly empty (rotary pairs, value rows, gate / up pairs and residual rows that do not fill a
whole tile), whose decode-layout tiles have few rows or differ from workgroup to workgroup, and whose reductions are split
into several parts. Everything is compared with the oracle: first token, hidden state, logits, cached keys and values."""
import numpy as np
import pytest
import torch

from oracle import knnssd_oracle as O
from paper_2505_16162_amd import binding, synth
from gpu_common import logits_close, make_pair
from test_gpu_parity_benchmark_shapes import _kv_close

pytestmark = pytest.mark.gpu

SHAPES = {
    # 2 query heads on 1 kv head: 96 rotary pairs and 64 value rows, less than one tile each; 10 column steps
    "pt_small": dict(d_model=320, n_heads=2, n_kv_heads=1, head_dim=64, d_ffn=352, vocab=700),
    # more rows than workgroups in the decode layout, unequal shares (some workgroups own one 16-row tile, some two)
    "pt_uneven": dict(d_model=4352, n_heads=10, n_kv_heads=2, head_dim=128, d_ffn=2080, vocab=1500, n_blocks=1),
    # long reduction over few output rows: K in many parts
    "pt_long_k": dict(d_model=288, n_heads=4, n_kv_heads=4, head_dim=64, d_ffn=8224, vocab=600, n_blocks=1),
}


@pytest.mark.timeout(300)
@pytest.mark.parametrize("name", sorted(SHAPES))
def test_prompt_lengths_round_the_tile_edges(name):
    shape = synth.small_shape(name, **dict(dict(max_seq=600), **SHAPES[name]))
    w, orc, gpu = make_pair(shape, seed=21, std=0.05 if shape.d_model < 1000 else 0.02)
    assert gpu.packed
    longest = 530
    prompt = synth.make_prompt(shape.vocab, longest, seed=22).tolist()
    # causal: one oracle run over the longest prompt holds the cached rows of every prefix, and the hidden state and
    # logits of a prefix are those of its last row
    rows, hid = orc.forward(prompt, 0, None, want_hidden=True)
    for n in (17, 31, 32, 33, 64, 65, 128, 129, 200, 256, 257, 511, 530):
        print("case", name, n, flush=True)
        first, hidden = gpu.knnssd_prefill(prompt[:n])
        ok, err = logits_close(gpu.knnssd_get_logits((n - 1) % 16).numpy(), rows[n - 1], shape)
        assert ok, (n, err)
        herr = np.abs(hidden.cpu().numpy() - hid[n - 1]).max() / np.abs(hid[n - 1]).max()
        assert herr <= 5e-3, (n, herr)      # the bound the logits have by default: the head is linear in it
        margin = O.top2_margin(rows[n - 1])
        assert first == O.argmax_lowest(rows[n - 1]) or margin < 1e-3, (n, margin)
        for blk in range(shape.n_blocks):
            for pos in sorted({0, 15, 16, n // 2, (n - 1) // 16 * 16, n - 2, n - 1}):
                for got, want in zip(gpu.knnssd_read_kv(blk, pos), orc.read_kv(blk, pos)):
                    _kv_close(got.numpy(), want)
    gpu.close()


@pytest.mark.timeout(300)
@pytest.mark.parametrize("what", ["large", "tiny", "zero", "wide_row"])
def test_weights_and_activations_of_any_magnitude(what):
    """Weights of 32 and more, whole matrices below 2^-24, rows whose values span many orders of magnitude, all-zero matrices:
    the prefill's operands are three bf16 planes of the fp32 activations and the bf16 weights as they are, whatever their
    range. The result is the oracle's. Two prompts each: the second one starts where the first ended."""
    shape = synth.small_shape("pt_wide", d_model=320, n_heads=4, n_kv_heads=2, head_dim=64, d_ffn=352, vocab=700, max_seq=400)
    w = synth.make_weights(shape, seed=31, gains="random", std=0.05)
    b0 = w["blocks"][0]
    if what == "large":
        b0["wd"][7, 11] = 100.0
        b0["wq"][3, 5] = -64.0
    elif what == "tiny":
        b0["wv"] *= 2.0 ** -24
        b0["wo"] *= 2.0 ** 9
    elif what == "zero":
        b0["wo"].zero_()
    else:
        b0["wg"] *= (2.0 ** (-10.0 * torch.rand(b0["wg"].shape, generator=torch.Generator().manual_seed(5)))).to(b0["wg"].dtype)
        b0["attn_norm"][::7] *= 300.0          # activations that span orders of magnitude as well
    orc, gpu = O.OracleModel(shape, w), binding.KnnSsd(shape, w)
    prompt = synth.make_prompt(shape.vocab, 300, seed=32).tolist()
    rows, hid = orc.forward(prompt, 0, None, want_hidden=True)
    for n in (290, 45):
        print("case", what, n, flush=True)
        _, hidden = gpu.knnssd_prefill(prompt[:n])
        ok, err = logits_close(gpu.knnssd_get_logits((n - 1) % 16).numpy(), rows[n - 1], shape)
        assert ok, (n, err)
        for blk in range(shape.n_blocks):
            for pos in (0, n // 2, n - 1):
                for got, want in zip(gpu.knnssd_read_kv(blk, pos), orc.read_kv(blk, pos)):
                    _kv_close(got.numpy(), want)
    gpu.close()


# one block whose plan takes, over these lengths, 128 x 64, 256 x 128 and 256 x 256 tiles for the QKV rows, with K split and whole
OPERANDS = dict(d_model=4096, n_heads=32, n_kv_heads=32, head_dim=128, d_ffn=6016, vocab=64, n_blocks=1)
OPERAND_PROMPTS = (45, 100, 520, 700, 1045)


@pytest.mark.timeout(300)
def test_operands_keep_every_bit():
    """Value rows whose weights let all but the last bit of an activation cancel, take one activation past another that is 2^36
    times as large, hold a weight of 2^-40 beside one of 1 (that meets a zero), or a single small one: every product is exact and
    every partial sum fits 24 bits, so the cached value is the closed form below, rounded to bf16 once (2^-8) behind the fp32 norm
    factor (2^-20)."""
    shape = synth.small_shape("pt_operands", max_seq=1060, **OPERANDS)
    w = synth.make_weights(shape, seed=41, gains="random", std=0.02)
    d, b0 = shape.d_model, w["blocks"][0]
    j, k, l, far = 8, 9, 10, 2041          # three columns of one group of eight; one far away
    w["embed"][:, [j, k, l]] = 1.0
    w["embed"][0::2, far] = 2.0 ** 36      # even tokens: the other activations are nothing beside it
    b0["attn_norm"][j], b0["attn_norm"][k], b0["attn_norm"][l] = 1 + 2.0 ** -12 + 2.0 ** -23, 1 + 2.0 ** -12, 1.5
    b0["wv"].zero_()
    b0["wv"][0::4, j], b0["wv"][0::4, k] = 1.0, -1.0
    b0["wv"][1::4, j] = 1.0
    b0["wv"][2::4, l], b0["wv"][2::4, l + 1] = 1.5 * 2.0 ** -40, 1.0
    w["embed"][:, l + 1] = 0.0
    b0["wv"][3::4, l] = 2.0 ** -14
    # products gain * x that fp32 rounds up, beside columns that hold the rounded product: they cancel
    g = torch.rand(4000, generator=torch.Generator().manual_seed(47)) + 1.0
    g = g[(g * 1.3671875).double() > g.double() * 1.3671875][:8]
    up = torch.arange(64, 96, 4)
    w["embed"][:, up], w["embed"][:, up + 1] = 1.3671875, 1.0
    b0["attn_norm"][up], b0["attn_norm"][up + 1] = g, g * 1.3671875
    for i, c in enumerate(up.tolist()):
        b0["wv"][4 * i + 3, l], b0["wv"][4 * i + 3, c], b0["wv"][4 * i + 3, c + 1] = 0.0, 1.0, -1.0
    gpu = binding.KnnSsd(shape, w)
    assert gpu.packed
    embed = w["embed"].double()
    rs = 1.0 / torch.sqrt((embed * embed).mean(dim=1) + shape.rms_eps)
    row = torch.tensor([2.0 ** -23, 1 + 2.0 ** -12 + 2.0 ** -23, 1.5 * 1.5 * 2.0 ** -40, 1.5 * 2.0 ** -14], dtype=torch.float64)
    row = row.repeat(shape.kv_dim // 4)
    row[3:32:4] = 0.0
    prompt = synth.make_prompt(shape.vocab, 1050, seed=42).tolist()
    for n in OPERAND_PROMPTS:
        print("case", n, flush=True)
        gpu.knnssd_prefill(prompt[:n])
        for pos in sorted({0, 1, 15, n // 2, n // 2 + 1, n - 2, n - 1}):
            want = row * rs[prompt[pos]]
            got = gpu.knnssd_read_kv(0, pos)[1].double()
            rel = (got - want).abs() / want.clamp(min=1e-30)
            assert rel.max() <= 2.0 ** -8 + 2.0 ** -20, (n, pos, prompt[pos] % 2, int(rel.argmax()) % 4, float(rel.max()))
    gpu.close()


@pytest.mark.timeout(300)
def test_every_tile_against_the_oracle():
    """The same lengths with ordinary weights: over them every build of the product runs."""
    shape = synth.small_shape("pt_builds", max_seq=1060, **dict(OPERANDS, vocab=600))
    w, orc, gpu = make_pair(shape, seed=43, std=0.02)
    prompt = synth.make_prompt(shape.vocab, OPERAND_PROMPTS[-1], seed=44).tolist()
    rows, hid = orc.forward(prompt, 0, None, want_hidden=True)
    for n in OPERAND_PROMPTS:
        print("case", n, flush=True)
        _, hidden = gpu.knnssd_prefill(prompt[:n])
        ok, err = logits_close(gpu.knnssd_get_logits((n - 1) % 16).numpy(), rows[n - 1], shape)
        assert ok, (n, err)
        herr = np.abs(hidden.cpu().numpy() - hid[n - 1]).max() / np.abs(hid[n - 1]).max()
        assert herr <= 5e-3, (n, herr)
        for pos in sorted({0, 15, 16, n // 2, n - 2, n - 1}):
            for got, want in zip(gpu.knnssd_read_kv(0, pos), orc.read_kv(0, pos)):
                _kv_close(got.numpy(), want)
    gpu.close()


@pytest.mark.timeout(300)
@pytest.mark.parametrize("hd", [64, 128])
def test_chunks_of_a_prompt_are_weighed_alike(hd):
    """Scores near 10^6 whose maximum grows by 8 (unscaled) from one 64-position chunk to the next: the weights of earlier chunks
    have to follow to fp32 accuracy, though the exponent itself is only known to 2^-8 there. Everything in front of the
    softmax is exact (rows of +-1 with eps = 0 have an RMS of 1, the scores are whole numbers below 2^24 and the two score
    dimensions do not rotate), so the hidden state has a closed form; fp32 sums of 200 weights: 10^-5."""
    d, n = 256, 200
    shape = synth.ModelShape("pt_softmax", 1, d, 2, 2, hd, 352, 64, 240, "bf16", "bf16", rope_base=1e30, rms_eps=0.0)
    w = synth.make_weights(shape, seed=45, gains="ones", std=0.02)
    b0 = w["blocks"][0]
    for name in ("wq", "wk", "wv", "wo", "wd"):
        b0[name].zero_()
    sign = torch.randint(0, 2, (shape.vocab, d), generator=torch.Generator().manual_seed(46)) * 2 - 1
    sign[:, 0] = 1                                                       # column 0: one
    sign[:, 1], sign[:, 2] = -1, -1                                      # columns 1 and 2: the token's kind, tokens 0, 1 and 2
    sign[1:, 1], sign[2:, 2] = 1, 1
    w["embed"].copy_(sign)
    a, b = hd // 2 - 1, hd // 2 - 2                                      # the slowest rotations
    b0["wq"][a, 0], b0["wk"][a, 0] = 1000.0, 1000.0
    b0["wq"][b, 0], b0["wk"][b, 0] = 1.0, 8.0
    b0["wk"][b, 1], b0["wk"][b, 2] = 4.0, 4.0                            # 0, 8, 16 by kind
    b0["wv"][0, 0], b0["wv"][0, 1] = 0.5, 0.5                            # 0, 1, 1
    b0["wo"][3, 0] = 1.0
    gpu = binding.KnnSsd(shape, w)
    assert gpu.packed
    kind = np.zeros(n, dtype=np.int64)
    kind[70:130], kind[140:] = 1, 2
    _, hidden = gpu.knnssd_prefill(kind.tolist())
    e = np.exp(8.0 * (kind - 2) / np.sqrt(hd))
    x = sign[2].double().numpy()
    x[3] += (e * (kind > 0)).sum() / e.sum()
    want = x / np.sqrt((x * x).mean())
    assert abs(hidden.cpu().numpy()[3] / want[3] - 1) <= 1e-5, (hidden.cpu().numpy()[3], want[3])
    gpu.close()
