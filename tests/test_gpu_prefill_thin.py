"""Short prompts over matrices large enough to be streamed by prefill_thin_kernel, against the oracle: an odd number of 32-column
steps (the last pair of a tile is half empty), runs that cross from one row tile into the next, row tiles that are partly
empty, both token widths at their edges."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2505_16162_amd import binding, synth
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


def _least_workspace(lib, cfg):
    """The smallest workspace that knnssd_create takes for a stream-order context of this cfg; asked with fp32 matrices, with which it ends
    with KNNSSD_ESHAPE behind the size check."""
    cfg = type(cfg).from_buffer_copy(cfg)
    cfg.weight_dtype = 0
    h, w, fake = ctypes.c_void_p(), binding.Weights(), ctypes.c_void_p(0x100000)
    kv = lib.knnssd_kvcache_bytes(ctypes.byref(cfg)) * 2
    lo, hi = 0, lib.knnssd_workspace_bytes(ctypes.byref(cfg))
    while hi - lo > 1:
        mid = (lo + hi) // 2
        rc = lib.knnssd_create(ctypes.byref(cfg), ctypes.byref(w), fake, kv, fake, mid, None, ctypes.byref(h))
        assert rc in (-1, -2)
        lo, hi = (lo, mid) if rc == -2 else (mid, hi)
    return hi


@pytest.mark.timeout(300)
def test_a_workspace_without_room_for_the_parts_will_do():
    """A context over the smallest workspace that is accepted: prompts take the plain tiles, stay inside the buffer, and agree with the oracle."""
    shape = synth.small_shape("thin_room", n_blocks=1, max_seq=64, d_model=2560, n_heads=8, n_kv_heads=2, head_dim=128, d_ffn=6048, vocab=500)
    w, orc, gpu = make_pair(shape, seed=51, std=0.02)
    prompt = synth.make_prompt(shape.vocab, 48, seed=52).tolist()
    rows, hid = orc.forward(prompt, 0, None, want_hidden=True)
    lib = gpu.lib
    least, full = _least_workspace(lib, gpu.cfg), lib.knnssd_workspace_bytes(ctypes.byref(gpu.cfg))
    assert least < full
    ws = torch.full((least + 65536,), 0x5a, dtype=torch.uint8, device="cuda")
    h = ctypes.c_void_p()
    assert lib.knnssd_create(ctypes.byref(gpu.cfg), ctypes.byref(gpu.w), gpu.kv.data_ptr(), gpu.kv.numel(), ws.data_ptr(), least,
                             ctypes.c_void_p(gpu.stream.cuda_stream), ctypes.byref(h)) == 0
    for n in (17, 33, 48):
        print("case", n, flush=True)
        first, hidden, logits = ctypes.c_int32(), torch.empty(shape.d_model, device="cuda"), torch.empty(shape.vocab)
        assert lib.knnssd_prefill(h, (ctypes.c_int32 * n)(*prompt[:n]), n, hidden.data_ptr(), ctypes.byref(first)) == 0
        assert lib.knnssd_get_logits(h, (n - 1) % 16, logits.data_ptr()) == 0
        ok, err = logits_close(logits.numpy(), rows[n - 1], shape)
        assert ok, (n, err)
        herr = np.abs(hidden.cpu().numpy() - hid[n - 1]).max() / np.abs(hid[n - 1]).max()
        assert herr <= 5e-3, (n, herr)
    assert bool((ws[least:] == 0x5a).all())
    assert lib.knnssd_destroy(h) == 0
    gpu.close()
