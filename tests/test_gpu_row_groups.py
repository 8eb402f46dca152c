"""GPU parity of the many-row GEMM over its row-group sizes: one group that fits the rows, several groups, remainders of every kind,
one, two and three operand planes - as verification steps and as the head alone."""
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


# rows = batch * (gamma + 1): edges of the groups of 64, 96, 128, 144 (two planes), 64, 144, 256, 288 (one), 64, 80, 96 (three), 64 and
# 144 (fp32), and several groups
@pytest.mark.parametrize("batch,gamma,planes,dtype", [(11, 2, 2, "bf16"), (16, 3, 2, "bf16"), (13, 4, 2, "bf16"), (12, 7, 2, "bf16"), (14, 8, 2, "bf16"),
                                                      (16, 7, 2, "bf16"), (15, 8, 2, "bf16"), (16, 8, 2, "bf16"), (29, 4, 2, "bf16"), (37, 6, 2, "bf16"),
                                                      (13, 4, 1, "bf16"), (17, 8, 1, "bf16"), (32, 8, 1, "bf16"), (13, 4, 3, "bf16"),
                                                      (37, 6, 3, "bf16"), (33, 8, 3, "bf16"), (16, 3, 3, "bf16"), (12, 7, 3, "bf16"),
                                                      (9, 3, 1, "fp32"), (29, 4, 1, "fp32"), (32, 4, 1, "fp32"), (32, 8, 1, "fp32")])
def test_step_over_row_groups(batch, gamma, planes, dtype):
    shape = dataclasses.replace(SMALL, name=f"groups_{batch}_{gamma}_{planes}_{dtype}", dtype=dtype, n_layers=1, batch=batch, gamma=gamma)
    _step_matches(shape, planes, dtype)


# The large-tile gate / up kernel, which needs some 200 tiles of 16 n-tiles x a row group: every group size at its edges (160, 192, 224,
# 256 rows and one more), two and three groups, fewer k-steps than stages, n-tiles that end in the middle of a tile, a second round of
# the chip, and the same rows with one plane, where the loader-wave kernel stays.
@pytest.mark.parametrize("batch,gamma,d,ffn,planes", [(29, 4, 64, 26304, 2), (32, 4, 64, 26240, 2), (23, 6, 128, 26304, 2), (24, 7, 64, 26304, 2),
                                                      (28, 7, 192, 26240, 2), (32, 7, 64, 26304, 2), (43, 5, 64, 13184, 2), (64, 8, 128, 10432, 2),
                                                      (57, 8, 64, 21184, 2), (32, 7, 64, 26304, 1)])
def test_step_on_large_tiles(batch, gamma, d, ffn, planes):
    shape = dataclasses.replace(SMALL, name=f"tiles_{batch}_{gamma}_{d}_{ffn}", n_layers=1, batch=batch, gamma=gamma, d_model=d, d_ffn=ffn,
                                n_q_heads=2, n_kv_heads=1, head_dim=64, vocab=512)
    _step_matches(shape, planes, "bf16", "gemm_tile" if planes == 2 else "gemm_rows8")


# The same tiles with the LM head's epilogue, on two planes and on one: the loader waves up to 64 rows, then every group size at its
# edges, halves of unequal row tiles, two groups, n-tiles that end in the middle of a tile, a second round of the chip, fewer
# k-steps than stages.
@pytest.mark.parametrize("batch,gamma,vocab,d,planes,kernel", [(8, 7, 52480, 64, 2, "gemm_rows8"), (13, 4, 52480, 64, 2, "groups of 96"),
                                                               (12, 7, 52608, 128, 2, "groups of 96"), (11, 8, 52480, 64, 2, "groups of 128"),
                                                               (16, 7, 52480, 192, 2, "groups of 128"), (43, 2, 52480, 128, 2, "groups of 144"),
                                                               (16, 8, 52608, 256, 2, "groups of 144"), (29, 4, 52480, 64, 2, "groups of 160"),
                                                               (28, 7, 52480, 128, 2, "groups of 224"), (32, 7, 52480, 64, 2, "groups of 256"),
                                                               (23, 6, 52480, 64, 2, "groups of 176"), (22, 7, 52608, 192, 2, "groups of 176"),
                                                               (28, 6, 52480, 128, 2, "groups of 208"), (26, 7, 52480, 64, 2, "groups of 208"),
                                                               (25, 8, 52480, 64, 2, "groups of 240"), (30, 7, 52608, 128, 2, "groups of 240"),
                                                               (42, 7, 26240, 64, 2, "groups of 176"),
                                                               (37, 6, 26240, 64, 2, "groups of 144"), (64, 4, 42752, 128, 2, "groups of 160"),
                                                               (8, 7, 52480, 64, 1, "gemm_rows8"), (13, 4, 52480, 64, 1, "groups of 96"),
                                                               (43, 2, 52480, 64, 1, "groups of 160"), (28, 7, 52480, 64, 1, "groups of 224"),
                                                               (45, 4, 52480, 64, 1, "groups of 256"), (32, 7, 52608, 256, 1, "groups of 256"),
                                                               (43, 5, 52480, 128, 1, "groups of 288"), (32, 8, 85248, 64, 1, "groups of 288"),
                                                               (37, 7, 26240, 192, 1, "groups of 160")])
def test_lm_head_on_large_tiles(batch, gamma, vocab, d, planes, kernel):
    shape = dataclasses.replace(SMALL, name=f"lm_{batch}_{gamma}_{vocab}_{d}_{planes}", n_layers=1, batch=batch, gamma=gamma, d_model=d, d_ffn=128,
                                n_q_heads=2, n_kv_heads=1, head_dim=64, vocab=vocab)
    _step_matches(shape, planes, "bf16", lm_head=kernel)


def _step_matches(shape, planes, dtype, gate_up="", lm_head=""):
    batch, gamma = shape.batch, shape.gamma
    src = synth.WeightSource(shape, seed=51, norm_jitter=0.1)
    lens = [(7 * b) % 40 for b in range(batch)]
    cap = [64] * batch
    gpu = G.Gpu(shape, src, cap)
    try:
        if dtype == "bf16":
            sj.sj_set_operand_planes(gpu.kv, planes)
        assert gate_up in sj.sj_kernel_class_shape(gpu.kv, 3, batch * (gamma + 1))
        named = sj.sj_kernel_class_shape(gpu.kv, 5, batch * (gamma + 1))
        assert lm_head in named and (not lm_head.startswith("groups") or "gemm_tile" in named), named
        cfg = helpers.oracle_config(shape)
        W = helpers.oracle_weights(src)
        caches = _fill_caches(shape, gpu, cfg, lens, seed=52, capacity=cap)
        draft = synth.make_draft(shape, seed=53)
        out = gpu.step(draft, 0.5, gamma)
        fw = orc.block_forward(cfg, W, caches, [[caches[b].pending] + draft["tokens"][b].tolist() for b in range(batch)])
        scale = 20.0 if dtype == "bf16" and planes == 1 else 1.0       # one plane rounds every operand to 8 bits
        for b in range(batch):
            G.close_enough(out["hn"][b], fw[b]["hn"], dtype, f"hidden seq {b}", scale=scale)
            G.close_enough(out["logits"][b], fw[b]["logits"], dtype, f"logits seq {b}", scale=scale)
        bad, _ = G.replay_matches(shape, out, draft, 0.5)
        assert not bad, bad
    finally:
        gpu.close()
