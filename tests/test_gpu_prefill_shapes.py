"""Prefill at the edges of its launch shapes.

The many-row GEMM and the prefill attention pick a launch shape by rows and matrix: one token
group, a wave per tile, tiles from 64 x 64 to 128 x 256 with one or two workgroups per compute
unit, one-chunk stages for a K of an odd number of chunks, blocks of at most 8192 rows cut
anywhere in a prompt.  A row's arithmetic may not depend on any of that: a ragged batch must give,
bitwise, the keys, values and head logits of its sequences run one by one, and sequences short
enough for the float64 oracle must match it within the storage tolerance.
"""
import numpy as np
import pytest

import gpu_util as gu
import oracle
import synth
from oracle import dvi as odvi

pytestmark = pytest.mark.gpu

BASE = synth.TINY.replace(n_layers=2, split_k=1, vocab=1008)
SHAPES = {
    # K of 3, 4 and 5 chunks, two query heads per kv head, head dim 64
    "odd": BASE.replace(name="odd", d_model=96, n_heads=2, n_kv_heads=1, head_dim=64, ffn_dim=160, bf16=True),
    # 1152 gate/up tiles, head dim 128
    "wide": BASE.replace(name="wide", d_model=512, n_heads=4, n_kv_heads=4, head_dim=128, ffn_dim=9216, bf16=True),
    # the same width over 10 chunks of K, head dim 64
    "wide10": BASE.replace(name="wide10", d_model=320, n_heads=5, n_kv_heads=5, head_dim=64, ffn_dim=9216, bf16=True),
    # fp32, K of 3 and 5 chunks, head dim 64; and head dim 128
    "fp32": BASE.replace(name="fp32", d_model=48, n_heads=1, n_kv_heads=1, head_dim=64, ffn_dim=80),
    "fp32_128": BASE.replace(name="fp32_128", d_model=256, n_heads=6, n_kv_heads=2, head_dim=128, ffn_dim=512),
}
CASES = [
    ("odd", [1]), ("odd", [16]), ("odd", [17]), ("odd", [64, 1]), ("odd", [200, 130, 16]), ("odd", [1, 600, 17, 63]),
    ("odd", [3000, 2700, 3001]),
    ("wide", [9]), ("wide", [33]), ("wide", [64]), ("wide", [65, 2]), ("wide", [200]), ("wide", [300, 7]),
    ("wide", [65, 255, 280]), ("wide", [1100, 63, 128]), ("wide", [2100, 2100, 1999, 17]),
    ("wide10", [65, 2]), ("wide10", [255, 65]), ("wide10", [1100]),
    ("fp32", [5]), ("fp32", [33, 31]), ("fp32", [70, 33]), ("fp32", [520, 300]),
    ("fp32_128", [7]), ("fp32_128", [129, 64, 1]), ("fp32_128", [900, 700, 450]),
]


@pytest.mark.parametrize("name,lens", CASES, ids=["%s-%s" % (n, "+".join(map(str, l))) for n, l in CASES])
def test_ragged_prefill_equals_single_sequences(name, lens):
    shape = SHAPES[name]
    lens = np.array(lens, np.int32)
    B, P = lens.size, int(lens.max())
    w = synth.make_weights(shape, 3)
    prompts = synth.make_prompts(shape.vocab, B, P, 5)
    layer = shape.n_layers - 1
    eng, _ = gu.engine(shape, max_batch=B, max_seq=P + 8, weights=w)
    first = eng.prefill(prompts, lens)
    logits = eng.read_logits()[:, 0].copy()
    kv = [eng.read_kv(layer, b, 0, int(n)) for b, n in enumerate(lens)]
    assert np.array_equal(eng.lengths(), lens)
    eng.close()
    om = oracle.OracleModel(w)
    for b, n in enumerate(lens):
        one, _ = gu.engine(shape, max_batch=1, max_seq=P + 8, weights=w)
        f1 = one.prefill(prompts[b:b + 1, :n])
        assert f1[0] == first[b]
        assert np.array_equal(one.read_logits()[0, 0], logits[b]), "sequence %d: logits" % b
        k, v = one.read_kv(layer, 0, 0, int(n))
        assert np.array_equal(k, kv[b][0]) and np.array_equal(v, kv[b][1]), "sequence %d: keys or values" % b
        one.close()
        if n <= 300:
            ref = odvi.greedy_ar(om, prompts[b, :n], 1, keep_logits=True)
            gu.check_close(logits[b], ref.logits[0], shape, "sequence %d" % b)


UPDATES = [
    # a wave per tile: one to four token groups
    ("odd", 1, 16, 1008), ("odd", 16, 3, 1008), ("odd", 17, 16, 1008), ("odd", 65, 1, 1008), ("odd", 256, 3, 1008),
    ("wide", 48, 16, 1008), ("wide", 64, 3, 1008), ("fp32", 33, 18, 1008), ("fp32", 130, 16, 1008),
    # 64 x 64 tiles: up to 64 rows, four parts of K; more rows of a narrower matrix, one
    ("wide", 48, 16, 32016), ("wide", 64, 3, 32016), ("fp32_128", 48, 16, 32016), ("wide", 80, 16, 8464),
    # 64 x 128 tiles: four-chunk and two-chunk stages
    ("wide", 160, 16, 8464), ("wide10", 160, 3, 8464),
    # 128 x 128 tiles: more and fewer workgroups than compute units
    ("wide", 400, 16, 8464), ("wide", 128, 16, 32016), ("fp32_128", 100, 3, 32016),
    # 128 x 256 tiles: eight waves, four waves
    ("wide", 200, 18, 32016), ("fp32_128", 130, 3, 32016), ("wide", 300, 3, 32016), ("fp32_128", 300, 16, 32016),
    # one-chunk stages
    ("odd", 100, 16, 32016), ("odd", 300, 3, 32016), ("fp32", 100, 16, 32016),
]


@pytest.mark.parametrize("name,rows,r,vocab", UPDATES)
def test_update_logits_launch_shapes(name, rows, r, vocab):
    """The drafter update's logits GEMM in each of its launch shapes on 256 compute units, with ranks that
    are not a multiple of four and vocabularies that leave the last tiles partly empty among them.  The
    engine sums fp32 products of the oracle's own inputs (a few hundred terms, 6e-8 each): 1e-4 leaves two
    orders."""
    from oracle import update as oupd
    shape = SHAPES[name].replace(lora_rank=r, vocab=vocab)
    eng, w = gu.engine(shape, max_seq=64, lora_A_std=0.02, buffer_rows=max(256, rows))
    buf = synth.make_buffer(shape.d_model, shape.vocab, rows, seed=11)
    eng.prefill(synth.make_prompts(shape.vocab, 1, 8, 1))
    eng.write_buffer(buf.h, buf.a, buf.logits, buf.r, buf.fresh)
    c = oupd.Coeffs(c_kl=0.7, c_ce=0.9, c_pg=0.4, c_ent=0.05, tau=1.3, baseline=0.35)
    st = eng.update_drafter(c.c_kl, c.c_ce, c.c_pg, c.c_ent, c.tau, c.baseline, lr=0.0, grads=True)
    ref = oupd.loss_and_grad(w.as_f32(w.lm_head).astype(np.float64), w.lora_A.astype(np.float64),
                             w.lora_B.astype(np.float64), shape.lora_gamma, buf.h.astype(np.float64), buf.a, buf.logits,
                             buf.r, buf.fresh, c)
    eng.close()
    assert gu.rel_l2(st["grad_A"].cpu().numpy(), ref.dA) <= 1e-4
    assert gu.rel_l2(st["grad_B"].cpu().numpy(), ref.dB) <= 1e-4
