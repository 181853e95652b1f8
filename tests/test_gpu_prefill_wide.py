"""Prompts whose products take the 256 x 192 tiles of the prefill, and the 256 x 128 and 256 x 192 ones that finish their rows themselves,
against the oracle: lengths below, at and above a tile, on the shape whose plans test_prefill_wide_plan.py checks."""
import numpy as np
import pytest

from paper_2505_16162_amd import synth
from gpu_common import logits_close, make_pair
from test_gpu_parity_benchmark_shapes import _kv_close
from test_prefill_wide_plan import PROMPTS, SPLIT, WIDE

pytestmark = pytest.mark.gpu


@pytest.mark.timeout(300)
@pytest.mark.parametrize("dims,lengths", ((WIDE, PROMPTS),) + SPLIT)
def test_wide_tiles_against_the_oracle(dims, lengths):
    shape = synth.small_shape("pt_wide_tiles", max_seq=1320, n_blocks=1, vocab=600, **dims)
    w, orc, gpu = make_pair(shape, seed=61, std=0.02)
    assert gpu.packed
    prompt = synth.make_prompt(shape.vocab, lengths[-1], seed=62).tolist()
    rows, hid = orc.forward(prompt, 0, None, want_hidden=True)
    for n in lengths:
        print("case", n, flush=True)
        _, hidden = gpu.knnssd_prefill(prompt[:n])
        ok, err = logits_close(gpu.knnssd_get_logits((n - 1) % 16).numpy(), rows[n - 1], shape)
        assert ok, (n, err)
        herr = np.abs(hidden.cpu().numpy() - hid[n - 1]).max() / np.abs(hid[n - 1]).max()
        assert herr <= 5e-3, (n, herr)      # the bound the logits have by default: the head is linear in it
        for pos in sorted({0, 15, 16, 191, 192, n // 2, n - 2, n - 1} & set(range(n))):
            for got, want in zip(gpu.knnssd_read_kv(0, pos), orc.read_kv(0, pos)):
                _kv_close(got.numpy(), want)
    gpu.close()
