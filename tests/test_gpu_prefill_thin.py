"""Short prompts over matrices large enough to be streamed by prefill_thin_kernel, against the oracle: an odd number of 32-column
steps (the last pair of a tile is half empty), runs that cross from one row tile into the next, row tiles that are partly
empty, both token widths at their edges."""
import numpy as np
import pytest

from paper_2505_16162_amd import synth
from gpu_common import logits_close, make_pair
from test_gpu_parity_benchmark_shapes import _kv_close

pytestmark = pytest.mark.gpu

SHAPES = {
    "thin_odd": dict(d_model=2080, n_heads=4, n_kv_heads=2, head_dim=128, d_ffn=6048, vocab=500),       # gate+up: 65 steps, 48 tiles
    "thin_all": dict(d_model=4096, n_heads=40, n_kv_heads=8, head_dim=128, d_ffn=8224, vocab=500),      # QKV, gate+up, down (257 steps)
}


@pytest.mark.timeout(300)
@pytest.mark.parametrize("name", sorted(SHAPES))
def test_short_prompts_stream_large_matrices(name):
    shape = synth.small_shape(name, n_blocks=1, max_seq=64, **SHAPES[name])
    w, orc, gpu = make_pair(shape, seed=51, std=0.02)
    assert gpu.packed
    prompt = synth.make_prompt(shape.vocab, 48, seed=52).tolist()
    rows, hid = orc.forward(prompt, 0, None, want_hidden=True)
    for n in (17, 31, 32, 33, 47, 48):
        print("case", name, n, flush=True)
        first, hidden = gpu.knnssd_prefill(prompt[:n])
        ok, err = logits_close(gpu.knnssd_get_logits((n - 1) % 16).numpy(), rows[n - 1], shape)
        assert ok, (n, err)
        herr = np.abs(hidden.cpu().numpy() - hid[n - 1]).max() / np.abs(hid[n - 1]).max()
        assert herr <= 5e-3, (n, herr)      # the bound the logits have by default: the head is linear in it
        for pos in sorted({0, 15, 16, n - 2, n - 1}):
            for got, want in zip(gpu.knnssd_read_kv(0, pos), orc.read_kv(0, pos)):
                _kv_close(got.numpy(), want)
    gpu.close()
