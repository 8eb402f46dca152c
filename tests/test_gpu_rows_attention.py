"""GPU parity of many-row attention in each of its forms: 8, 4 and 2 waves to a tile of 16 query columns (fewer than 512 tiles, fewer than
1024, more), with tiles left over in the last workgroup, for blocks of a batch over cached contexts and for prompt chunks."""
import dataclasses

import numpy as np
import pytest

import paper_2510_02329_amd as sj
import synth
from oracle import selfjudge_oracle as orc
from tests import gpu_common as G
from tests import helpers
from tests.test_gpu_bf16 import SMALL, _fill_caches

pytestmark = pytest.mark.gpu


def _waves_per_tile(shape, rps, nseq):
    tiles = (rps * (shape.n_q_heads // shape.n_kv_heads) + 15) // 16 * shape.n_kv_heads * nseq
    return 2 if tiles >= 1024 else 4 if tiles >= 512 else 8


@pytest.mark.parametrize("dtype,hq,hkv,hd,batch,gamma,planes,waves", [
    ("bf16", 16, 4, 128, 64, 8, 2, 4),          # 3 tiles per kv head and sequence: a wave group without a tile
    ("bf16", 16, 8, 64, 64, 8, 2, 2),           # 2 tiles: two of four groups without one
    ("bf16", 24, 8, 64, 52, 7, 1, 4),
    ("bf16", 20, 4, 128, 65, 15, 3, 2),         # 5 tiles
    ("fp32", 16, 8, 128, 43, 7, 1, 8),
    ("fp32", 18, 6, 64, 58, 10, 1, 2),          # 3 tiles
])
def test_blocks_of_a_batch(dtype, hq, hkv, hd, batch, gamma, planes, waves):
    shape = dataclasses.replace(SMALL, name=f"rows_attn_{dtype}_{hq}_{hkv}_{hd}_{batch}", dtype=dtype, n_layers=1, d_model=256, d_ffn=256, vocab=512,
                                n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, batch=batch, gamma=gamma)
    assert _waves_per_tile(shape, gamma + 1, batch) == waves
    src = synth.WeightSource(shape, seed=81, norm_jitter=0.1)
    lens = [(37 * b) % 290 for b in range(batch)]                # several steps of every wave, and none
    cap = [l + gamma + 1 for l in lens]
    gpu = G.Gpu(shape, src, cap)
    try:
        if dtype == "bf16":
            sj.sj_set_operand_planes(gpu.kv, planes)
        cfg = helpers.oracle_config(shape)
        caches = _fill_caches(shape, gpu, cfg, lens, seed=82, capacity=[(c + 63) // 64 * 64 for c in cap])
        draft = synth.make_draft(shape, seed=83)
        out = gpu.step(draft, 0.5, gamma)
        fw = orc.block_forward(cfg, helpers.oracle_weights(src), caches, [[caches[b].pending] + draft["tokens"][b].tolist() for b in range(batch)])
        scale = 20.0 if planes == 1 and dtype == "bf16" else 1.0         # one plane rounds every operand to 8 bits
        for b in range(batch):
            G.close_enough(out["hn"][b], fw[b]["hn"], dtype, f"hidden seq {b}", scale=scale)
            k, v = gpu.kv_rows(b, 0, lens[b], gamma + 1)
            G.close_enough(k, caches[b].k[0][:, lens[b]:lens[b] + gamma + 1], dtype, f"K seq {b}", scale=scale)
            G.close_enough(v, caches[b].v[0][:, lens[b]:lens[b] + gamma + 1], dtype, f"V seq {b}", scale=scale)
    finally:
        gpu.close()


@pytest.mark.parametrize("dtype,hq,hkv,hd,prompts,waves", [
    ("bf16", 32, 8, 64, [41, 299], [8, 4]),     # 75 tiles per kv head, over 41 cached keys
    ("bf16", 32, 8, 128, [545], [2]),           # 137 tiles
    ("fp32", 32, 8, 64, [515], [2]),            # 129 tiles
    ("fp32", 20, 4, 128, [1, 411], [None, 4]),  # 129 tiles of a group of 5 heads
])
def test_prompt_chunks(dtype, hq, hkv, hd, prompts, waves):
    shape = dataclasses.replace(SMALL, name=f"rows_attn_prompt_{dtype}_{hq}_{hd}", dtype=dtype, n_layers=1, d_model=256, d_ffn=256, vocab=512,
                                n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, batch=1, gamma=4)
    src = synth.WeightSource(shape, seed=91, norm_jitter=0.1)
    cap = sum(prompts)
    gpu = G.Gpu(shape, src, [cap])
    try:
        cfg, W = helpers.oracle_config(shape), helpers.oracle_weights(src)
        cache = orc.SeqCache(cfg, cap, storage=dtype)
        for i, n in enumerate(prompts):
            assert waves[i] is None or _waves_per_tile(shape, n, 1) == waves[i]
            prompt = synth.make_prompt(shape, 92 + i, n).tolist()
            L0 = cache.length
            sj.sj_prefill(gpu.model, gpu.kv, 0, prompt)
            fw = orc.block_forward(cfg, W, [cache], [prompt])[0]
            cache.length += n
            rows, tail = min(n, 5), n - (n - 1) // 5 * 5
            order = list(range(n - tail, n)) + list(range(n - rows, n - tail))
            hn = sj.sj_debug_fetch(gpu.kv, sj.SJ_DBG_HIDDEN, np.empty((rows, shape.d_model), np.float32))
            G.close_enough(hn, fw["hn"][order], dtype, "hidden")
            k, v = gpu.kv_rows(0, 0, L0, n)
            G.close_enough(k, cache.k[0][:, L0:cache.length], dtype, "K")
            G.close_enough(v, cache.v[0][:, L0:cache.length], dtype, "V")
    finally:
        gpu.close()


# The single launch over long contexts in its three batch sizes: partials of every number that a block of many rows can have, three query
# tiles to a workgroup, contexts of one and of seventeen key ranges.
@pytest.mark.parametrize("dtype,parts", [("fp32", p) for p in range(2, 9)] + [("bf16", 5), ("bf16", 7)])
def test_long_contexts_over_every_number_of_partials(dtype, parts):
    shape = dataclasses.replace(SMALL, name=f"partials_{dtype}_{parts}", dtype=dtype, n_layers=1, d_model=(128 if dtype == "fp32" else 256) * parts, d_ffn=256,
                                vocab=512, n_q_heads=12, n_kv_heads=3, head_dim=64, batch=5, gamma=8)
    src = synth.WeightSource(shape, seed=95, norm_jitter=0.1)
    lens, cap = [2090, 40, 0, 700, 1301], [2112] * 5
    gpu = G.Gpu(shape, src, cap)
    try:
        assert f"{parts} K-slice" in sj.sj_kernel_class_shape(gpu.kv, 1, 45)
        cfg = helpers.oracle_config(shape)
        caches = _fill_caches(shape, gpu, cfg, lens, seed=96, capacity=cap)
        draft = synth.make_draft(shape, seed=97)
        out = gpu.step(draft, 0.5, 8)
        fw = orc.block_forward(cfg, helpers.oracle_weights(src), caches, [[caches[b].pending] + draft["tokens"][b].tolist() for b in range(5)])
        for b in range(5):
            G.close_enough(out["hn"][b], fw[b]["hn"], dtype, f"hidden seq {b}")
            k, v = gpu.kv_rows(b, 0, lens[b], 9)
            G.close_enough(k, caches[b].k[0][:, lens[b]:lens[b] + 9], dtype, f"K seq {b}")
            G.close_enough(v, caches[b].v[0][:, lens[b]:lens[b] + 9], dtype, f"V seq {b}")
    finally:
        gpu.close()
