"""GPU parity of the residual epilogue (O / down projection + residual add + the next norm's operand in one launch, 1/rms applied by
the consumer) and of the packed operand planes, at the edges of their rules."""
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


# (dtype, d_model, q heads, kv heads, head dim, d_ffn, batch, gamma, planes): one n-tile a workgroup on both kernels (K of a few
# k-steps and of whole stages, ring depths 4 and 8), two and four tiles, 1 / 8 / 9 rows, one / two / three planes, fp32
CASES = [
    ("bf16", 512, 4, 2, 64, 192, 1, 7, 2),
    ("bf16", 512, 4, 2, 64, 1024, 2, 3, 2),
    ("bf16", 512, 16, 2, 64, 4096, 1, 1, 2),
    ("bf16", 512, 4, 2, 64, 1024, 3, 2, 2),
    ("bf16", 512, 4, 2, 64, 1024, 1, 4, 1),
    ("bf16", 512, 4, 2, 64, 1024, 1, 4, 3),
    ("bf16", 4160, 4, 2, 64, 2048, 1, 5, 2),
    ("bf16", 8256, 2, 1, 64, 512, 1, 2, 2),
    ("fp32", 320, 5, 5, 64, 448, 2, 3, 1),
    ("fp32", 4160, 2, 1, 64, 128, 1, 2, 1),
]


@pytest.mark.parametrize("dtype,d,hq,hkv,hd,f,batch,gamma,planes", CASES)
def test_residual_epilogue_matches_oracle(dtype, d, hq, hkv, hd, f, batch, gamma, planes):
    shape = dataclasses.replace(SMALL, name=f"resid_{dtype}_{d}_{f}", dtype=dtype, n_layers=3, d_model=d, n_q_heads=hq, n_kv_heads=hkv,
                                head_dim=hd, d_ffn=f, vocab=1024, batch=batch, gamma=gamma, weight_std=0.5 / d ** 0.5)
    src = synth.WeightSource(shape, seed=41, norm_jitter=0.1, judge_bias=0.1)
    lens = [70, 5, 131][:batch]
    cap = [l + 2 * (gamma + 1) + 3 for l in lens]
    gpu = G.Gpu(shape, src, cap)
    try:
        if dtype == "bf16":
            sj.sj_set_operand_planes(gpu.kv, planes)
        cfg = helpers.oracle_config(shape)
        W = helpers.oracle_weights(src)
        caches = _fill_caches(shape, gpu, cfg, lens, seed=42, capacity=cap)
        scale = 20.0 if dtype == "bf16" and planes == 1 else 1.0       # one plane rounds every operand to 8 bits
        for step in range(2):
            draft = synth.make_draft(shape, seed=43 + step)
            L0 = [c.length for c in caches]
            out = gpu.step(draft, 0.5, gamma)
            fw = orc.block_forward(cfg, W, caches, [[caches[b].pending] + draft["tokens"][b].tolist() for b in range(batch)])
            for b in range(batch):
                G.close_enough(out["hn"][b], fw[b]["hn"], dtype, f"hidden seq {b}", scale=scale)
                G.close_enough(out["logits"][b], fw[b]["logits"], dtype, f"logits seq {b}", scale=scale)
                n, nxt = int(out["accepted_len"][b]), int(out["next_token"][b])
                caches[b].length, caches[b].pending = L0[b] + 1 + n, nxt
            bad, _ = G.replay_matches(shape, out, draft, 0.5)
            assert not bad, bad
    finally:
        gpu.close()
