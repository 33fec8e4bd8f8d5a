"""Decode attention: the one-workgroup path of short contexts against the split path.

A sequence decoded alone at up to 512 positions is attended to in one workgroup per head, with the
partials in LDS; beside a sequence of 600 positions the same rows go through the split chunks and a
merge from memory.  Both must commit the same tokens and leave, bitwise, the same keys and values.
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
