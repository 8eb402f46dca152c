"""GPU parity on the remaining named workloads: the verify-head microbenchmark (batch 64, gamma 8,
vocab 128256) and the 8B-shaped batch-16 / gamma-8 case with ragged cache lengths; the 70B-shaped
case is opt-in (minutes of weight generation)."""
import os

import numpy as np
import pytest
import torch

import paper_2510_02329_amd as sj
import synth
from oracle import selfjudge_oracle as orc
from tests import gpu_common as G
from tests import helpers
from tests.progress import say
from tests.test_gpu_bf16 import _compare_step, _fill_caches

pytestmark = pytest.mark.gpu


def test_verify_head_microbenchmark():
    """LM head -> softmax -> ratio test -> judge -> scan -> extra token on given final hidden states
    (576 rows): logits against the fp64 product, decisions exactly against the oracle's tail."""
    shape = synth.CONFIGS[1]
    src = synth.WeightSource(shape, seed=0, judge_bias=0.1)
    gpu = G.Gpu(shape, src, None)
    try:
        B, gamma, V, d = shape.batch, shape.gamma, shape.vocab, shape.d_model
        hidden = synth.make_hidden(shape, seed=0)                       # [R, d] bf16 bits
        draft = synth.make_draft(shape, seed=0)
        hid_dev = torch.from_numpy(hidden.view(np.int16)).to(gpu.dev)
        say("head step")
        out = gpu.step(draft, 0.5, gamma, head_hidden=hid_dev)
        h64 = synth.to_f64(hidden)
        logits = np.empty((B * (gamma + 1), V))
        for r0 in range(0, V, 16384):
            r1 = min(V, r0 + 16384)
            logits[:, r0:r1] = h64 @ synth.to_f64(src.tensor("lm_head", -1, (r0, r1))).T
        logits = logits.reshape(B, gamma + 1, V)
        w, bias = synth.to_f64(src.tensor("judge_w")), float(synth.to_f64(src.tensor("judge_b"))[0])
        err, worst = G.close_enough(out["logits"], logits, "bf16", "head logits")
        say("head logits max err %.3e (%.3f of the bound)" % (err, worst))
        n_acc = []
        for b in range(B):
            scores = np.array([orc.judge_score(w, bias, h64[b * (gamma + 1) + j]) for j in range(1, gamma + 1)])
            G.close_enough(out["judge_scores"][b], scores, "bf16", f"judge seq {b}")
            ref = orc.verify_tail(logits[b], scores, draft["tokens"][b], draft["probs"][b], draft["uniforms"][b],
                                  0.5, shape.temperature)
            bits = [(1 if a else 0) | (2 if g else 0) for a, g in zip(ref["align_bits"], ref["judge_bits"])]
            assert out["bits"][b].tolist() == bits, b
            assert int(out["accepted_len"][b]) == ref["accepted_len"], b
            n_acc.append(ref["accepted_len"])
            # the token draw sits on a flat distribution: exact on replay of the device's logits, and against
            # the pure oracle unless the uniform falls next to a cell boundary
            if int(out["next_token"][b]) != ref["next_token"]:
                rep = orc.verify_tail(out["logits"][b].astype(np.float64), scores, draft["tokens"][b], draft["probs"][b],
                                      draft["uniforms"][b], 0.5, shape.temperature)
                assert int(out["next_token"][b]) == rep["next_token"], b
        bad, _ = G.replay_matches(shape, out, draft, 0.5)
        assert not bad, bad
        assert 0 < np.mean(n_acc) < gamma          # the recipe exercises both accepts and rejects
    finally:
        gpu.close()


@pytest.fixture(scope="module")
def llama8b():
    shape = synth.CONFIGS[3]
    src = synth.WeightSource(shape, seed=0)
    say("loading 8B-shaped model")
    model = G.load_model(shape, src)
    yield shape, src, model
    sj.sj_model_free(model)


def test_llama8b_batch16_ragged(llama8b):
    """8B shape, batch 16, gamma 8, cache lengths U[512, 4096], capacity padded to 64."""
    shape, src, model = llama8b
    lens = shape.kv_lengths(0)
    cap = [int(l) + 64 for l in lens]
    gpu = G.Gpu.__new__(G.Gpu)
    gpu.shape, gpu.model, gpu.dev = shape, model, torch.device("cuda:0")
    gpu.kv = sj.sj_kv_create(model, shape.batch, cap)
    try:
        cfg = helpers.oracle_config(shape)
        W = helpers.oracle_weights(src, cache_items=0)
        say("filling caches", lens.tolist())
        caches = _fill_caches(shape, gpu, cfg, lens, seed=0, capacity=cap)
        draft = synth.make_draft(shape, seed=0)
        say("step")
        out, ref, stats = _compare_step(shape, gpu, cfg, W, caches, draft, 0.5, "8B b16")
        say("8B b16 logits max err %.3e worst err/bound %.2f" % stats["logits"])
    finally:
        sj.sj_kv_free(gpu.kv)


def _llama70b(force_rounding, scale):
    shape = synth.CONFIGS[4]
    src = synth.WeightSource(shape, seed=0)
    lens = shape.kv_lengths(0)
    cap = [int(l) + 64 for l in lens]
    say("loading 70B-shaped model")
    gpu = G.Gpu(shape, src, cap)
    try:
        cfg = helpers.oracle_config(shape)
        W0 = helpers.oracle_weights(src, cache_items=0)

        def W(name, layer=-1, rows=None):
            if name == "wq" and layer % 4 == 0:
                say(f"  oracle layer {layer}/{shape.n_layers}")
            return W0(name, layer, rows)

        caches = _fill_caches(shape, gpu, cfg, lens, seed=0, capacity=cap)
        draft = synth.make_draft(shape, seed=0)
        say("step")
        out, ref, stats = _compare_step(shape, gpu, cfg, W, caches, draft, 0.5, "70B", force_rounding=force_rounding, scale=scale)
        say("70B %s: logits max err %.3e worst err/bound %.3f" % ("replay on the device's stored rows" if force_rounding else
                                                                   "against the pure oracle", *stats["logits"]))
        # the same step with the operands exact
        sj.sj_set_operand_planes(gpu.kv, 3)
        sj.sj_kv_rewind(gpu.kv, lens, synth.make_pending(shape, 0), torch.cuda.current_stream())
        exact = gpu.step(draft, 0.5, shape.gamma)
        if not force_rounding:
            _measured_shapes(shape, gpu, lens, draft, ref)
        return stats, out, ref, draft, exact
    finally:
        gpu.close()


_measured70b = {}


def _measured_shapes(shape, gpu, lens, draft, ref):
    """The same step with two planes in the launch shapes that the start-up measurement picks, kept for the test of them."""
    tune = os.environ.pop("SJ_TUNE", None)
    try:
        sj.sj_set_operand_planes(gpu.kv, 2)
        sj.sj_set_temperature(gpu.model, shape.temperature)              # (a new launch graph: the one of the rule's shapes would be replayed)
        sj.sj_kv_rewind(gpu.kv, lens, synth.make_pending(shape, 0), torch.cuda.current_stream())
        say("70B measured shapes: " + ", ".join(sj.sj_kernel_class_shape(gpu.kv, c, shape.batch * (shape.gamma + 1)) for c in (1, 2, 4)))
        _measured70b.update(out=gpu.step(draft, 0.5, shape.gamma), ref=ref, draft=draft)
    finally:
        if tune is not None:
            os.environ["SJ_TUNE"] = tune


def test_llama70b_batch4(monkeypatch):
    """70B shape, batch 4, gamma 5, cache 2048, against the PURE oracle.  Bits and accepted lengths must match;
    hidden states and judge scores meet the bf16 bar.  The logits of this 80-layer random decoder sit AT the bar
    (measured 1.03 of it with two operand planes, 1.33 with three): a stored K / V element is the bf16 rounding of a
    value the two sides know to ~1e-6, near a rounding boundary they store neighbouring numbers, and 80 random layers
    amplify those one-ulp differences - it does not shrink with a more exact operand.  Asserted at twice the bar,
    with the measured figure printed; the replay below shows the same step inside 0.05 of the bar once both sides
    store the same rows.

    Emitted tokens must match, too, wherever the oracle's own draw decides them.  The first sequence's uniform lies
    3.5e-7 above the lower edge of its token's cell, which is 6.5e-7 wide, and the device's CDF is off by 2e-8 .. 7e-7
    there: 6.6e-7 with the shapes of the rule (the draw gives the token before), 2e-8 and 2.6e-7 with two choices of
    the start-up measurement (the oracle's token).  So the shapes are fixed here, and a token may be the
    oracle's neighbour where the uniform is closer to the edge between the two than 2e-6: three times that error.
    With three operand planes all four tokens are the oracle's."""
    monkeypatch.setenv("SJ_TUNE", "0")
    stats, out, ref, draft, exact = _llama70b(force_rounding=False, scale=2.0)
    d = stats["decisions"]
    assert d["unexcused"] == 0 and d["bit_excused"] == 0 and d["len_excused"] == 0 and d["token_excused"] <= 1
    for b, r in enumerate(ref):
        n, k_dev, k_ref = int(out["accepted_len"][b]), int(out["next_token"][b]), int(r["next_token"])
        w = r["p"][n] if n == draft["tokens"].shape[1] else np.maximum(0.0, r["p"][n] - np.asarray(draft["probs"][b, n], np.float64))
        edge = w[:max(k_dev, k_ref)].sum() / w.sum()                 # between the two, if they are neighbours
        gap = abs(float(draft["uniforms"][b, -1]) - edge)
        say(f"70B token {b}: {k_dev}, oracle {k_ref}, uniform {gap:.2e} from the lower edge")
        assert k_dev == k_ref or (abs(k_dev - k_ref) == 1 and gap < 2e-6), (b, k_dev, k_ref, gap)
        assert int(exact["accepted_len"][b]) == r["accepted_len"] and int(exact["next_token"][b]) == k_ref, (b, exact["next_token"][b], k_ref)


def test_llama70b_batch4_in_measured_shapes(monkeypatch):
    """The step of the test above in the shapes that the start-up measurement picks: the same bound on the logits (twice the bar), bits and lengths.
    How far the logits are off is a matter of which stored elements round the other way: over six drafts the worst element of a sequence is 0.2 to
    4.8 bars from that of exact operands, for a draft the same to 0.1 with 1, 2, 4 or 8 K-slices of any product - but for this draft's fourth
    sequence, 3.2 with one or two slices of QKV and 1.4 with four or eight, the number that both the rule and the measurement have."""
    if not _measured70b:
        monkeypatch.setenv("SJ_TUNE", "0")
        _llama70b(force_rounding=False, scale=2.0)
    out, ref, draft = (_measured70b[k] for k in ("out", "ref", "draft"))
    for b, r in enumerate(ref):
        err, worst = G.close_enough(out["logits"][b], r["logits"], "bf16", f"70B measured shapes, logits seq {b}", scale=2.0)
        say(f"70B measured shapes, sequence {b}: logits max err {err:.3e} worst err/bound {worst:.3f}")
    d = G.decisions_vs_oracle(synth.CONFIGS[4], out, ref, draft, 0.5)
    assert d["unexcused"] == 0 and d["bit_excused"] == 0 and d["len_excused"] == 0, d


@pytest.mark.skipif(os.environ.get("SJ_RUN_70B_REPLAY") != "1",
                    reason="replay check, not parity: the oracle adopts the device's stored K / V rows (several minutes; "
                           "run with SJ_RUN_70B_REPLAY=1)")
def test_llama70b_batch4_replay_on_device_rounding():
    _llama70b(force_rounding=True, scale=1.0)
