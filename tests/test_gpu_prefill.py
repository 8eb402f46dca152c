"""GPU parity of long prompts: chunks of hundreds of rows with an attention of their own (rotary + append, then causal
attention over the cache), against the oracle's forward over the whole prompt."""
import dataclasses

import numpy as np
import pytest

import paper_2510_02329_amd as sj
import synth
from oracle import selfjudge_oracle as orc
from tests import gpu_common as G
from tests import helpers
from tests.test_gpu_bf16 import SMALL

pytestmark = pytest.mark.gpu


# (dtype, q heads, kv heads, head dim, prompts fed one after the other).  The sizes sit at the edges of the path: one row
# more than a block, few-row kernels with more rows than their plan, 16-position tiles and their remainders, one row group
# and one row more, a group size that does not divide 16, and a prompt of two chunks.
CASES = [
    ("bf16", 8, 2, 128, [6, 16, 33]),
    ("bf16", 8, 2, 64, [7, 1, 31, 145]),
    ("bf16", 6, 2, 64, [32, 289]),
    ("bf16", 4, 4, 128, [64, 577]),
    ("fp32", 10, 2, 64, [15, 144]),
    ("fp32", 4, 4, 128, [300]),
]


@pytest.mark.parametrize("dtype,hq,hkv,hd,prompts", CASES)
def test_long_prompt_matches_oracle(dtype, hq, hkv, hd, prompts):
    shape = dataclasses.replace(SMALL, name=f"prefill_{dtype}_{hq}_{hd}", dtype=dtype, n_layers=2, n_q_heads=hq, n_kv_heads=hkv,
                                head_dim=hd, batch=2, gamma=4, temperature=1.0)
    src = synth.WeightSource(shape, seed=21, norm_jitter=0.1)
    cap = sum(prompts) + 3
    gpu = G.Gpu(shape, src, [40, cap])                   # the prompts go to the second sequence
    try:
        cfg = helpers.oracle_config(shape)
        W = helpers.oracle_weights(src)
        cache = orc.SeqCache(cfg, cap, storage=dtype)
        block = shape.gamma + 1
        for i, n in enumerate(prompts):
            prompt = synth.make_prompt(shape, 30 + i, n).tolist()
            L0 = cache.length
            print(f"prompt of {n} at {L0}", flush=True)
            sj.sj_prefill(gpu.model, gpu.kv, 1, prompt)
            fw = orc.block_forward(cfg, W, [cache], [prompt])[0]
            cache.length += n
            ln, pend = sj.sj_kv_state(gpu.kv, 2)
            assert ln.tolist() == [0, cache.length]
            for l in range(shape.n_layers):
                k, v = gpu.kv_rows(1, l, L0, n)
                G.close_enough(k, cache.k[l][:, L0:cache.length], dtype, f"K layer {l}")
                G.close_enough(v, cache.v[l][:, L0:cache.length], dtype, f"V layer {l}")
            # the rows of the last block of a chain of blocks, and after them the ones before
            rows = min(n, block)
            tail = n - (n - 1) // block * block
            order = list(range(n - tail, n)) + list(range(n - rows, n - tail))
            hn = sj.sj_debug_fetch(gpu.kv, sj.SJ_DBG_HIDDEN, np.empty((rows, shape.d_model), np.float32))
            G.close_enough(hn, fw["hn"][order], dtype, "hidden")
            logits = sj.sj_debug_fetch(gpu.kv, sj.SJ_DBG_LOGITS, np.empty((rows, shape.vocab), np.float32))
            G.close_enough(logits[:tail], fw["logits"][n - tail:], dtype, "logits")
            top2 = np.sort(fw["logits"][-1])[-2:]
            a, r = G.TOL[dtype]
            if top2[1] - top2[0] > 2 * (a + r * abs(top2[1])):
                assert pend[1] == int(np.argmax(fw["logits"][-1]))
            assert pend[1] == int(np.argmax(logits[tail - 1]))
    finally:
        gpu.close()


# The last layer of a prompt chunk goes on with the rows of the last block only: two rows (operand planes with rows side by side), seven (packed),
# twelve (not packed), 41 (the many-row kernels), tails that begin inside a tile of query columns, one layer and three, and a group
# that does not divide 16.
@pytest.mark.parametrize("dtype,layers,hq,hkv,gamma,prompts", [
    ("bf16", 1, 8, 2, 1, [3, 64]),
    ("bf16", 3, 6, 2, 6, [8, 47]),
    ("bf16", 1, 4, 4, 11, [5, 13, 130]),
    ("bf16", 2, 8, 2, 40, [42, 100]),
    ("fp32", 1, 10, 2, 2, [4, 33]),
    ("fp32", 2, 4, 2, 35, [37, 77]),
])
def test_last_layer_runs_over_the_last_block(dtype, layers, hq, hkv, gamma, prompts):
    shape = dataclasses.replace(SMALL, name=f"prefill_tail_{dtype}_{layers}_{gamma}", dtype=dtype, n_layers=layers, n_q_heads=hq, n_kv_heads=hkv,
                                head_dim=64, batch=1, gamma=gamma, temperature=1.0)
    src = synth.WeightSource(shape, seed=25, norm_jitter=0.1)
    cap, block = sum(prompts), gamma + 1
    gpu = G.Gpu(shape, src, [cap])
    try:
        cfg, W = helpers.oracle_config(shape), helpers.oracle_weights(src)
        cache = orc.SeqCache(cfg, cap, storage=dtype)
        for i, n in enumerate(prompts):
            prompt = synth.make_prompt(shape, 40 + i, n).tolist()
            L0 = cache.length
            sj.sj_prefill(gpu.model, gpu.kv, 0, prompt)
            fw = orc.block_forward(cfg, W, [cache], [prompt])[0]
            cache.length += n
            for l in range(layers):
                k, v = gpu.kv_rows(0, l, L0, n)
                G.close_enough(k, cache.k[l][:, L0:cache.length], dtype, f"K layer {l}")
                G.close_enough(v, cache.v[l][:, L0:cache.length], dtype, f"V layer {l}")
            rows, tail = min(n, block), n - (n - 1) // block * block
            order = list(range(n - tail, n)) + list(range(n - rows, n - tail))
            hn = sj.sj_debug_fetch(gpu.kv, sj.SJ_DBG_HIDDEN, np.empty((rows, shape.d_model), np.float32))
            G.close_enough(hn, fw["hn"][order], dtype, "hidden")
            logits = sj.sj_debug_fetch(gpu.kv, sj.SJ_DBG_LOGITS, np.empty((rows, shape.vocab), np.float32))
            G.close_enough(logits[:tail], fw["logits"][n - tail:], dtype, "logits")
    finally:
        gpu.close()


def test_prompt_buffers_come_with_the_first_long_prompt():
    """A cache object that sees no prompt longer than a block holds no buffers for prompt chunks."""
    import torch
    shape = dataclasses.replace(SMALL, name="prefill_memory", d_model=1024, d_ffn=4096, n_layers=1, batch=1, gamma=4)
    gpu = G.Gpu(shape, synth.WeightSource(shape, seed=23), [1024])
    free = lambda: (torch.cuda.synchronize(), torch.cuda.mem_get_info()[0])[1] / 2.0 ** 20  # noqa: E731
    try:
        prompt = synth.make_prompt(shape, 24, 700).tolist()
        f0 = free()
        kv = sj.sj_kv_create(gpu.model, 1, [1024])
        f1 = free()
        sj.sj_prefill(gpu.model, kv, 0, prompt[:5])            # one block
        f2 = free()
        sj.sj_prefill(gpu.model, kv, 0, prompt[5:600])
        f3 = free()
        sj.sj_kv_set_state(kv, 0, 0, 0)
        sj.sj_prefill(gpu.model, kv, 0, prompt)
        f4 = free()
        sj.sj_kv_free(kv)
        # cache 1 MB, workspace of 5 rows below 3 MB (logits, statistics, partials of at most 8 slices); planes of 576 rows alone are
        # 3 * 576 * (1024 + 1024 + 4096) * 2 = 20 MB.  Allocations come in pieces of 2 MB.
        assert f0 - f1 <= 12 and f2 == f1 and f2 - f3 >= 20 and f4 == f3, (f0 - f1, f1 - f2, f2 - f3, f3 - f4)
        assert free() >= f0 - 2
    finally:
        gpu.close()
