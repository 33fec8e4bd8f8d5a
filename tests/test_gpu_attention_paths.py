"""Decode attention: the one-workgroup path of short contexts against the split path.

A sequence decoded alone at up to 256 positions (512 in bf16 at head dim 64) is attended to in one
workgroup per head, with the partials in LDS; beside a sequence of 600 positions the same rows go
through the split chunks and a merge from memory.  Both must commit the same tokens and leave, bitwise,
the same keys and values.
"""
import numpy as np
import pytest

import gpu_util as gu
import synth
from test_gpu_prefill_shapes import SHAPES

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["odd", "wide", "fp32", "fp32_128"])
@pytest.mark.parametrize("k,ctx", [(1, 1), (1, 255), (2, 63), (3, 64), (4, 254), (4, 257), (5, 191), (8, 250), (8, 505)])
def test_short_context_attention_equals_split_path(name, k, ctx):
    shape = SHAPES[name]
    w = synth.make_weights(shape, 3, lora_A_std=0.01)
    prompts = synth.make_prompts(shape.vocab, 2, 600, 5)
    lens = np.array([ctx, 600], np.int32)
    steps = 3
    cap = 600 + steps * k + 8
    eng, _ = gu.engine(shape, max_batch=2, max_seq=cap, weights=w)
    eng.prefill(prompts, lens)
    tok, n, m = eng.decode_steps(k, steps)
    end = int(eng.lengths()[0])
    kv = [eng.read_kv(l, 0, 0, end) for l in range(shape.n_layers)]
    eng.close()
    one, _ = gu.engine(shape, max_batch=1, max_seq=cap, weights=w)
    one.prefill(prompts[:1, :ctx])
    t1, n1, m1 = one.decode_steps(k, steps)
    assert np.array_equal(t1[:, 0], tok[:, 0]) and np.array_equal(n1[:, 0], n[:, 0]) and np.array_equal(m1[:, 0], m[:, 0])
    for l in range(shape.n_layers):
        kk, vv = one.read_kv(l, 0, 0, end)
        assert np.array_equal(kk, kv[l][0]) and np.array_equal(vv, kv[l][1]), "layer %d" % l
    one.close()


# enough kv heads in the batch for eight chunks in one workgroup, and few enough alone for the split
MANY = {
    "bf16_128": (SHAPES["wide"], 8, 4),
    "fp32_64": (SHAPES["fp32"].replace(name="many_64", d_model=256, n_heads=4, n_kv_heads=4, ffn_dim=64), 32, 2),
    "fp32_128": (SHAPES["fp32_128"].replace(name="many_128", d_model=128, n_heads=4, n_kv_heads=4, ffn_dim=64), 64, 1),
}


@pytest.mark.parametrize("name", sorted(MANY))
@pytest.mark.parametrize("ctx", [257, 383, 500])
def test_eight_chunks_in_one_workgroup_equal_split_path(name, ctx):
    """Sequences of 257 to 505 positions decoded in a batch whose heads fill enough of the chip for the
    one-workgroup path, against three of them decoded alone, whose chunks are split over workgroups."""
    shape, batch, k = MANY[name]
    w = synth.make_weights(shape, 3, lora_A_std=0.01)
    lens = np.array([ctx - b % 3 for b in range(batch)], np.int32)
    prompts = synth.make_prompts(shape.vocab, batch, ctx, 5)
    cap = ctx + k + 8
    eng, _ = gu.engine(shape, max_batch=batch, max_seq=cap, max_k_spec=k, weights=w)
    eng.prefill(prompts, lens)
    tok, n, m = eng.decode_steps(k, 1)
    ends, layer = eng.lengths(), shape.n_layers - 1
    for b in (0, 1, batch - 1):
        kv = eng.read_kv(layer, b, 0, int(ends[b]))
        one, _ = gu.engine(shape, max_batch=1, max_seq=cap, max_k_spec=k, weights=w)
        one.prefill(prompts[b:b + 1, :lens[b]])
        t1, n1, m1 = one.decode_steps(k, 1)
        assert np.array_equal(t1[:, 0], tok[:, b]) and np.array_equal(n1[:, 0], n[:, b]) and np.array_equal(m1[:, 0], m[:, b])
        kk, vv = one.read_kv(layer, 0, 0, int(ends[b]))
        assert np.array_equal(kk, kv[0]) and np.array_equal(vv, kv[1]), "sequence %d" % b
        one.close()
    eng.close()
