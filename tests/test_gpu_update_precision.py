"""Sums of the drafter update on inputs where the length of a chain of additions shows.

A sum of one large and many small terms, each below half a unit in the last place of the large one,
loses every small term that is added to the large one alone, and keeps those that were added up among
themselves first.  So the error counts the length of the longest chain, and bounds it exactly.
"""
import numpy as np
import pytest

import gpu_util as gu
import synth

pytestmark = pytest.mark.gpu

BASE = synth.TINY.replace(name="chain", n_layers=1, split_k=1, d_model=48, n_heads=1, n_kv_heads=1, head_dim=64, ffn_dim=32,
                          vocab=128, lora_rank=16)


def _zero_weights(shape):
    w = synth.make_weights(shape, 0)
    w.lm_head = np.zeros_like(w.lm_head)
    w.lora_A, w.lora_B = np.zeros_like(w.lora_A), np.zeros_like(w.lora_B)
    return w


def _update(shape, w, h, a):
    """Gradients of plain cross-entropy at tokens a (all rows accepted, uniform target logits)."""
    n = h.shape[0]
    eng, _ = gu.engine(shape, max_seq=64, weights=w)
    eng.prefill(synth.make_prompts(shape.vocab, 1, 4, 1))
    eng.write_buffer(h, a, np.zeros((n, shape.vocab), np.float32), np.ones(n, np.int8), np.ones(n, np.int8))
    st = eng.update_drafter(0.0, 1.0, 0.0, 0.0, 1.0, 0.0, lr=0.0, grads=True)
    gA, gB = st["grad_A"].cpu().numpy().astype(np.float64), st["grad_B"].cpu().numpy().astype(np.float64)
    eng.close()
    return gA, gB


@pytest.mark.parametrize("token", [0, 5, 17, 64, 127])
def test_du_adds_the_vocabulary_as_a_tree(token):
    """du = A_s^T g over the 128 vocabulary entries of one workgroup.  The logits are all equal, so g is
    p - 1 at the token and p = 1/128 elsewhere, and A_s makes the others' products 0.4 units of 2^-24
    beside one of 127/128 (half a unit there: 2^-25).  A chain of c products with the large one loses
    0.4 (c - 1) units; in a tree the four products of one MFMA lose 1.2, and each of the seven additions
    up to du at most half a unit: 4.7, with one unit for g and one for the product with h.  Chains of 32
    lose 10 to 12."""
    shape = BASE
    w = _zero_weights(shape)
    w.lora_A[:] = -0.4 * 2.0 ** -24 * shape.vocab
    w.lora_A[token] = 1.0
    h = np.linspace(0.5, 2.0, shape.d_model).astype(np.float32)[None]
    _, gB = _update(shape, w, h, np.array([token], np.int32))
    p = 1.0 / shape.vocab
    A = w.lora_A.astype(np.float64)
    du = shape.lora_gamma * (A[token] * (p - 1.0) + p * (A.sum(0) - A[token]))
    off = np.abs(gB / (du[:, None] * h.astype(np.float64)) - 1.0).max()
    assert off <= 6.7 * 2.0 ** -24, "%.2f units of 2^-24" % (off * 2.0 ** 24)


@pytest.mark.parametrize("vocab,rows", [(1008, 1), (1008, 16), (1008, 40), (1008, 60), (8448, 3), (8448, 33), (8448, 64)])
def test_logits_of_few_rows_have_no_long_chain(vocab, rows):
    """The logits' sum over K = 4096 in bf16, 128 chunks of 32 products.  Odd entries of the vocabulary
    are 16 exactly; even ones have 0.4 units of 2^-20 more per chunk, where one unit is half the spacing
    of fp32 beside 16.  Their ratio of probabilities shows what was kept: a chain of c chunks onto the 16
    loses 0.4 (c - 1) units, each addition of partial sums behind it rounds by at most one.  A wave per
    tile has chains of 6 chunks, two additions that join the parts of a block and one for each of six
    blocks: 10 units; the ring 8, two and four: 8.8.  Half a unit more for the two exponentials.  Chains
    of 32 lose 12.4 before the first of these additions."""
    shape = BASE.replace(d_model=4096, vocab=vocab, lora_rank=4, bf16=True)
    d = shape.d_model
    w = _zero_weights(shape)
    per = synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(np.float32([0.4 * 2.0 ** -20 / 32])))[0]
    head = np.zeros((vocab, d), np.float32)
    head[::2] = per
    head[:, 0] = 16.0
    w.lm_head = synth.f32_to_bf16_bits(head)
    w.lora_B[0, 0] = 1.0   # u = 1 for rank 0, A_s = 0: the logits are the head's alone
    h = np.ones((rows, d), np.float32)
    tokens = np.arange(rows, dtype=np.int32) * 2 + 1
    gA, _ = _update(shape, w, h, tokens)
    free = np.setdiff1d(np.arange(vocab), tokens)
    gA = gA[free, 0]
    odd, even = gA[free % 2 == 1], gA[free % 2 == 0]
    off = np.abs(np.log(even / odd[0]) - float(per) * (d - 1)).max()
    assert np.ptp(odd) == 0 and off <= 10.5 * 2.0 ** -20, "%.2f units of 2^-20" % (off * 2.0 ** 20)


def test_gradients_into_memory_that_is_not_the_devices_own():
    """Gradient buffers outside the context's device memory (here pinned host memory) are filled by a
    copy, with the same values as buffers on the device."""
    import ctypes

    import torch
    from paper_2510_05421_amd import _abi
    shape = BASE.replace(vocab=1008)
    eng, w = gu.engine(shape, max_seq=64, lora_A_std=0.02)
    buf = synth.make_buffer(shape.d_model, shape.vocab, 20, seed=11)
    eng.prefill(synth.make_prompts(shape.vocab, 1, 4, 1))
    got = []
    for where in ("device", "pinned", "mixed"):
        eng.write_buffer(buf.h, buf.a, buf.logits, buf.r, buf.fresh)
        torch.cuda.synchronize()
        gA = torch.zeros(shape.vocab, shape.lora_rank, pin_memory=True) if where == "pinned" else torch.zeros_like(eng.lora_A)
        gB = torch.zeros_like(eng.lora_B) if where == "device" else torch.zeros(shape.lora_rank, shape.d_model, pin_memory=True)
        torch.cuda.synchronize()
        args = _abi.UpdateArgs(0.7, 0.9, 0.4, 0.05, 1.3, 0.35, 0.0, 0.9, 0.999, 1e-8, 0, gA.data_ptr(), gB.data_ptr())
        assert eng.lib.dvi_update_drafter(eng.ctx, ctypes.byref(args), None) == _abi.OK
        torch.cuda.synchronize()
        got.append((gA.cpu().numpy().copy(), gB.cpu().numpy().copy()))
    eng.close()
    assert got[0][0].any() and got[0][1].any()
    for a, b in got[1:]:
        assert np.array_equal(a, got[0][0]) and np.array_equal(b, got[0][1])


@pytest.mark.parametrize("rows", [8, 48])
def test_small_updates_do_not_wait_for_a_cold_head(rows):
    """An update of few rows streams the head once, so it may not matter whether the last-level cache holds
    it: with a head of 262 MB the update after a gigabyte of other traffic takes at most a quarter longer
    than the one right after another update (ordinary loads: 1.4 times)."""
    import torch
    shape = BASE.replace(d_model=4096, vocab=32000, bf16=True)
    w = synth.make_weights(shape.replace(vocab=128), 0)
    zeros = np.zeros((shape.vocab, shape.d_model), np.uint16)
    w.shape, w.tok_emb, w.lm_head = shape, zeros, zeros
    w.lora_A, w.lora_B = np.zeros((shape.vocab, shape.lora_rank), np.float32), np.zeros((shape.lora_rank, shape.d_model), np.float32)
    eng, _ = gu.engine(shape, max_seq=64, weights=w)
    eng.prefill(np.ones((1, 4), np.int32))
    eng.write_buffer(np.ones((rows, shape.d_model), np.float32), np.zeros(rows, np.int32),
                     np.zeros((rows, shape.vocab), np.float32), np.ones(rows, np.int8), np.ones(rows, np.int8))
    other = torch.zeros(1 << 28, dtype=torch.float32, device="cuda")
    took = {}
    for cold in (False, True):
        ms = []
        for _ in range(25):
            if cold:
                other.add_(1.0)
            torch.cuda.synchronize()
            eng.update_drafter(0.7, 0.9, 0.4, lr=0.0)
            ms.append(eng.timings()["update"])
        took[cold] = float(np.median(ms[5:]))
    eng.close()
    assert took[True] <= 1.25 * took[False], "%.4f ms cold, %.4f ms warm" % (took[True], took[False])
