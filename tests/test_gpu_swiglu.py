"""silu(gate) * up over the whole range of the gate that fp32 can express, in prefill and in decoding.

One layer is built so that logit f shows feature f alone: every embedding is ones, the attention
contributes nothing, gate f is a chosen value G_f, the up projection a power of two that brings
silu(G_f) * up to [1, 2), the down projection and the head hand feature f to logit f.  G reaches down to
-88.5: exp(88.5) still fits fp32, while 1 / (1 + exp(88.5)) is below its normal range.

Against float64.  bf16 storage rounds the activation, and h before the head, to 8 bits: 2^-9 each, so
2^-7 per logit leaves twice their sum.  In fp32 an error of one unit of 2^-24 in the gate is one of
|G| units in exp(-G): 5e-5 is nine such units at |G| = 88.
"""
import numpy as np
import pytest

import gpu_util as gu
import synth

pytestmark = pytest.mark.gpu

WIDE = synth.TINY.replace(name="gate_range", n_layers=1, split_k=1, d_model=512, n_heads=4, n_kv_heads=4, head_dim=128,
                          ffn_dim=9216, vocab=1008)


def _weights(shape):
    w = synth.make_weights(shape, 1)
    d, F = shape.d_model, shape.ffn_dim

    def put(x):
        return synth.f32_to_bf16_bits(np.asarray(x, np.float32)) if shape.bf16 else np.asarray(x, np.float32)

    G = np.linspace(-88.5, 60.0, d)
    G[:3] = (-88.5, -88.0, -87.5)
    G = synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(G.astype(np.float32))).astype(np.float64)
    G[G == 0.0] = 0.5
    inv = 1.0 / np.sqrt(1.0 + shape.rms_eps)
    silu = (G * inv) / (1.0 + np.exp(-G * inv))
    up = np.exp2(-np.floor(np.log2(np.abs(silu)))) * np.sign(silu)
    gate, upm, down = np.zeros((F, d)), np.zeros((F, d)), np.zeros((d, F))
    gate[:d, 0], upm[:d, 1] = G, up
    down[np.arange(d), np.arange(d)] = 1.0
    head = np.zeros((shape.vocab, d))
    head[:d] = np.eye(d)
    l = w.layers[0]
    l["wo"], l["w_gate"], l["w_up"], l["w_down"] = put(np.zeros(l["wo"].shape)), put(gate), put(upm), put(down)
    w.tok_emb, w.lm_head = put(np.ones((shape.vocab, d))), put(head)
    h = 1.0 + silu * up * inv
    return w, h / np.sqrt(np.mean(h * h) + shape.rms_eps)


@pytest.mark.parametrize("bf16", [True, False], ids=["bf16", "fp32"])
@pytest.mark.parametrize("rows", [5, 40, 600])
def test_swiglu_over_the_range_of_the_gate(rows, bf16):
    shape = WIDE.replace(bf16=bf16)
    w, want = _weights(shape)
    tol = 2.0 ** -7 if bf16 else 5e-5
    eng, _ = gu.engine(shape, max_seq=rows + 8, weights=w)
    eng.prefill(synth.make_prompts(shape.vocab, 1, rows, 3))
    for what in ("prefill", "decode"):
        if what == "decode":
            eng.draft(1)
            eng.verify()
        got = eng.read_logits()[0, 0].astype(np.float64)
        off = np.abs(got[:shape.d_model] / want - 1.0)
        assert off.max() <= tol, "%s: feature %d off by %.3g" % (what, off.argmax(), off.max())
        assert not got[shape.d_model:].any()
    eng.close()
