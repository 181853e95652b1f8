"""Prompts on the any-shape kernels take their rows side by side; a context that sends prompts through 16-row passes is the reference, bit
for bit: hidden state, logits, cache. Lengths around a chunk (8), a pass (16) and a launch's rows (256; 128 with wide bf16 rows), all pairs of storage types, ragged
widths. And a passes-then-prompt mix: a prompt after a verification starts from the same state."""
import ctypes

import pytest
import torch

from paper_2505_16162_amd import binding, synth

pytestmark = pytest.mark.gpu

LENGTHS = (16, 17, 23, 24, 25, 32, 33, 64, 128, 129, 161, 255, 256, 257, 272, 521)


@pytest.mark.timeout(120)
@pytest.mark.parametrize("wt,kt,hd,h,kvh,d,f", [("fp32", "fp32", 64, 4, 2, 264, 504), ("bf16", "bf16", 128, 3, 1, 328, 1000), ("bf16", "fp32", 64, 5, 1, 72, 40),
                                                ("fp32", "bf16", 128, 2, 2, 1016, 88), ("bf16", "bf16", 64, 2, 1, 2808, 72), ("bf16", "fp32", 64, 1, 1, 3208, 64)])
def test_prompt_rows_have_the_bits_of_passes(wt, kt, hd, h, kvh, d, f):
    shape = synth.ModelShape("rows", 2, d, h, kvh, hd, f, 613, 560, wt, kt)
    w = synth.make_weights(shape, seed=71, gains="random", std=0.05)
    side, passes = binding.KnnSsd(shape, w, generic_kernels=True), binding.KnnSsd(shape, w, generic_kernels=True, chunked_prefill=True)
    assert not side.packed
    prompt = synth.make_prompt(shape.vocab, LENGTHS[-1], seed=72).tolist()
    kvt = torch.bfloat16 if kt == "bf16" else torch.float32
    for n in LENGTHS:
        print("case", wt, kt, n, flush=True)
        got = side.knnssd_prefill(prompt[:n])
        want = passes.knnssd_prefill(prompt[:n])
        assert got[0] == want[0] and torch.equal(got[1], want[1]), n
        row = (n - 1) % 16
        assert torch.equal(side.knnssd_get_logits(row), passes.knnssd_get_logits(row)), n
        kv = [c.kv.view(kvt).view(shape.n_blocks, 2, kvh, shape.max_seq, hd)[:, :, :, :n] for c in (side, passes)]
        assert torch.equal(kv[0], kv[1]), n
        tokens = prompt[n - 3:n]
        assert side.knnssd_verify(tokens, n) == passes.knnssd_verify(tokens, n)
        assert torch.equal(side.knnssd_get_logits(2), passes.knnssd_get_logits(2)), n
    side.close()
    passes.close()


@pytest.mark.timeout(60)
def test_a_workspace_without_room_for_the_rows_will_do():
    """A buffer of the size that 16-row passes need is accepted, whatever prefill_mode says; one byte less is refused."""
    shape = synth.ModelShape("rows_small", 1, 72, 2, 1, 64, 40, 100, 80, "bf16", "bf16")
    w = synth.make_weights(shape, seed=73, gains="random", std=0.05)
    prompt = synth.make_prompt(shape.vocab, 70, seed=74).tolist()
    gpu = binding.KnnSsd(shape, w, generic_kernels=True)
    want = gpu.knnssd_prefill(prompt)
    lib = gpu.lib
    chunked = binding.make_cfg(shape, 0)
    chunked.prefill_mode = 1
    need, full = lib.knnssd_workspace_bytes(ctypes.byref(chunked)), lib.knnssd_workspace_bytes(ctypes.byref(gpu.cfg))
    assert need < full
    ws = torch.empty(full, dtype=torch.uint8, device="cuda")
    for size, ok in ((need, True), (need - 1, False)):
        h = ctypes.c_void_p()
        rc = lib.knnssd_create(ctypes.byref(gpu.cfg), ctypes.byref(gpu.w), gpu.kv.data_ptr(), gpu.kv.numel() * gpu.kv.element_size(), ws.data_ptr(), size,
                               ctypes.c_void_p(gpu.stream.cuda_stream), ctypes.byref(h))
        assert (rc == 0) == ok
        if ok:
            first, hidden = ctypes.c_int32(), torch.empty(shape.d_model, device="cuda")
            toks = (ctypes.c_int32 * len(prompt))(*prompt)
            assert lib.knnssd_prefill(h, toks, len(prompt), hidden.data_ptr(), ctypes.byref(first)) == 0
            assert first.value == want[0] and torch.equal(hidden, want[1])
            assert lib.knnssd_destroy(h) == 0
    gpu.close()
