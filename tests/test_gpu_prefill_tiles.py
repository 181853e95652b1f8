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
def test_weights_that_two_fp16_planes_do_or_do_not_hold(what):
    """Weights of 32 and more, or whole runs of weights below 2^-15, go through three bf16 planes instead of two fp16 ones
    (the kernels find out, the prompt runs again); rows whose values span many orders of magnitude and all-zero matrices
    stay with two. Either way the result is the oracle's. Two prompts each: the second one starts where the first ended."""
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
