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
