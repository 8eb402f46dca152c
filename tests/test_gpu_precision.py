"""Rounding of the running sums: where the operands are exact to 24 bits (fp32 storage; three bf16 planes), a many-row product is as close
to 64 bits as the few-row kernels' product of the same rows."""
import numpy as np
import pytest
import torch

import paper_2510_02329_amd as sj
import synth
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


def _logits(shape, src, hidden, batch, gamma, planes):
    """Device logits of the verification tail on given hidden states, with the model's rows in one call."""
    gpu = G.Gpu(synth.ModelShape(**{**shape.__dict__, "batch": batch, "gamma": gamma}), src, None, max_gamma=8)
    try:
        if planes:
            sj.sj_set_operand_planes(gpu.kv, planes)
        draft = synth.make_draft(gpu.shape, seed=3)
        h = torch.from_numpy(np.ascontiguousarray(hidden[:batch * (gamma + 1)])).to("cuda:0")
        return gpu.step(draft, 0.5, gamma, head_hidden=h)["logits"].reshape(batch * (gamma + 1), shape.vocab)
    finally:
        gpu.close()


@pytest.mark.parametrize("d", [1024, 8192])
def test_fp32_head_of_many_rows_is_as_exact_as_of_few(d):
    """One chain of sums over all of d has twice the error of the few-row kernel, whose waves share d."""
    shape = synth.ModelShape("precision_fp32", "fp32", 0, d, 4, 4, 64, 256, 1024, 10000.0, batch=37, gamma=3)
    src = synth.WeightSource(shape, seed=5)
    hidden = np.random.default_rng(6).standard_normal((37 * 8, d)).astype(np.float32)
    ref = hidden.astype(np.float64) @ synth.to_f64(src.tensor("lm_head", -1)).T
    rms = lambda got, n: float(np.sqrt(((got[:n] - ref[:n]) ** 2).mean()))  # noqa: E731
    few = rms(_logits(shape, src, hidden, 8, 3, 0), 32)
    for batch, gamma in ((12, 3), (37, 3), (37, 7)):     # 48, 148, 296 rows
        many = rms(_logits(shape, src, hidden, batch, gamma, 0), 32)
        print(f"d {d}, {batch * (gamma + 1)} rows: rms error {many:.3e}, 32 rows {few:.3e}", flush=True)
        assert many <= 1.1 * few


def test_three_plane_prompt_chunk_is_as_exact_as_blocks(monkeypatch):
    """The first layer's K / V rows of a prompt are bf16 roundings of one product: the share that rounds to the other neighbour of the
    64-bit value measures the product's error.  A chunk of 560 rows against blocks of 20 rows through the few-row kernels, in the shapes
    of the rule: there 304 against 281 elements, where the start-up measurement sometimes takes 3 n-tiles, 8 waves, 4 K-slices for the
    blocks, whose 32 chains of a product are half as long (227)."""
    monkeypatch.setenv("SJ_TUNE", "0")
    from oracle import selfjudge_oracle as orc
    from tests import helpers
    shape = synth.ModelShape("precision_planes", "bf16", 1, 4096, 8, 8, 128, 256, 512, 10000.0, batch=1, gamma=19)
    src = synth.WeightSource(shape, seed=7, norm_jitter=0.1)
    n = 560
    prompt = synth.make_prompt(shape, 8, n).tolist()
    cache = orc.SeqCache(helpers.oracle_config(shape), n, storage="bf16")
    orc.block_forward(helpers.oracle_config(shape), helpers.oracle_weights(src), [cache], [prompt])
    gpu = G.Gpu(shape, src, [n])
    share = {}
    try:
        sj.sj_set_operand_planes(gpu.kv, 3)
        for way, pieces in (("chunk", [prompt]), ("blocks", [prompt[i:i + 20] for i in range(0, n, 20)])):
            sj.sj_kv_set_state(gpu.kv, 0, 0, 0)
            for p in pieces:
                sj.sj_prefill(gpu.model, gpu.kv, 0, p)
            k, v = gpu.kv_rows(0, 0, 0, n)
            share[way] = sum(int((a != b[0][:, :n]).sum()) for a, b in ((k, cache.k), (v, cache.v)))
    finally:
        gpu.close()
    total = 2 * n * 1024
    print(f"of {total} stored elements take the other neighbour: chunk {share['chunk']}, blocks {share['blocks']}", flush=True)
    # counts of independent rare events: three standard deviations of their difference, and the 64-bit oracle itself is exact
    assert share["chunk"] <= share["blocks"] + 3.0 * np.sqrt(share["chunk"] + share["blocks"])


def test_fp32_residual_epilogue_is_as_exact_as_slices():
    """Blocks of up to 8 rows close a sub-layer without K-slices, larger ones with up to eight (the last layer always): the same
    rows either way."""
    import dataclasses
    from oracle import selfjudge_oracle as orc
    from tests import helpers
    from tests.test_gpu_bf16 import _fill_caches
    shape = synth.ModelShape("precision_resid", "fp32", 2, 512, 8, 8, 64, 16384, 512, 10000.0, batch=1, gamma=5, weight_std=0.05)
    src = synth.WeightSource(shape, seed=11, norm_jitter=0.1)
    cfg, W = helpers.oracle_config(shape), helpers.oracle_weights(src)
    err = {}
    for batch in (1, 2, 4):                                    # 6, 12, 24 rows; the first sequence is the same
        many = dataclasses.replace(shape, batch=batch)
        gpu = G.Gpu(many, src, [64] * batch)
        try:
            caches = _fill_caches(many, gpu, cfg, [20] * batch, seed=12, capacity=[64] * batch)
            draft = synth.make_draft(dataclasses.replace(shape, batch=4), seed=13)
            draft = {k: v[:batch] for k, v in draft.items()}
            out = gpu.step(draft, 0.5, 5)
            ref = orc.block_forward(cfg, W, caches[:1], [[caches[0].pending] + draft["tokens"][0].tolist()])[0]["hn"]
            err[batch] = float(np.sqrt(((out["hn"][0] - ref) ** 2).mean()))
        finally:
            gpu.close()
    print("rms error of the hidden states, 6 / 12 / 24 rows: %.3e %.3e %.3e" % tuple(err.values()), flush=True)
    assert err[1] <= 1.1 * max(err[2], err[4])
