"""GPU parity of judge training (Sec. 3.4, appendix "Training Logistic Regressor"): every model of the C grid,
its validation ROC-AUC, the kept model and both thresholds against the CPU oracle; at the paper's size, the
optimality conditions that identify the unique optimum."""
import time

import numpy as np
import pytest
import torch

import paper_2510_02329_amd as sj
import synth
from oracle import judge_training_oracle as jt

pytestmark = pytest.mark.gpu


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def _auc_slack(scores, y, tol):
    """Pairs (acceptable, unacceptable) whose scores differ by less than tol: the ones whose order may
    legitimately differ between two computations that agree to tol / 2."""
    pos, neg = np.sort(scores[y == 1]), np.sort(scores[y == 0])
    close = np.searchsorted(neg, pos + tol) - np.searchsorted(neg, pos - tol)
    return close.sum() / (len(pos) * len(neg))


@pytest.mark.parametrize("n,n_val,d,seed", [(3000, 1000, 256, 1), (1501, 777, 1100, 2), (900, 300, 4100, 3)])
def test_judge_training_matches_oracle(n, n_val, d, seed):
    H, y = synth.make_judge_dataset(seed, n, d)
    Hv, yv = synth.make_judge_dataset(seed + 100, n_val, d)
    grid = jt.paper_c_grid()
    if d > 2048:
        grid = grid[[0, 4, 9]]                                # the oracle's dense Hessian is slow at this width
    out = sj.sj_judge_train(_dev(H), _dev(y), _dev(Hv), _dev(yv), grid, torch.cuda.current_stream())
    ref = jt.train_judge(H, y, Hv, yv, grid)
    tol_z = 1e-7
    for c, fit in enumerate(ref["fits"]):
        w_err = np.abs(out["w_all"][c, :d] - fit["w"]).max()
        b_err = abs(out["w_all"][c, d] - fit["b"])
        print(f"C = {grid[c]:.4g}: |w err| = {w_err:.2e}, |b err| = {b_err:.2e}, passes = {out['passes'][c]}", flush=True)
        assert w_err < 1e-8 * max(1.0, np.abs(fit["w"]).max() * 10) and b_err < 1e-8 * max(1.0, abs(fit["b"]) * 10)
        s_ref = jt.scores_of(Hv, fit["w"], fit["b"])
        assert abs(out["auc"][c] - ref["auc"][c]) <= _auc_slack(s_ref, yv, tol_z) + 1e-15
    assert out["best_index"] == ref["best_index"]
    assert np.abs(out["w"] - ref["w"]).max() < 1e-8 * max(1.0, 10 * np.abs(ref["w"]).max())
    # thresholds are validation scores of the kept model: equal up to the agreement of the scores
    assert abs(out["theta_f1"] - ref["theta_f1"]) < tol_z
    assert abs(out["theta_recall"] - ref["theta_recall"]) < tol_z
    # and they act the same on the validation set
    s = ref["val_scores"]
    margin = np.abs(s - ref["theta_f1"])
    safe = margin > tol_z
    assert ((s > out["theta_f1"]) == (s > ref["theta_f1"]))[safe].all()


def test_judge_training_argument_errors():
    H, y = synth.make_judge_dataset(1, 64, 32)
    Hd, yd = _dev(H), _dev(y)
    with pytest.raises(sj.SJError):
        sj.sj_judge_train(Hd, _dev(np.ones(64, np.int32)), Hd, yd, [1.0])            # one class only
    with pytest.raises(sj.SJError):
        sj.sj_judge_train(Hd, _dev(np.full(64, 2, np.int32)), Hd, yd, [1.0])          # not a label
    with pytest.raises(sj.SJError):
        sj.sj_judge_train(Hd, yd, Hd, yd, [0.0])                                     # C must be positive
    with pytest.raises(sj.SJError):
        sj.sj_judge_train(_dev(H[:, :30]), yd, _dev(H[:, :30]), yd, [1.0])            # d not a multiple of 4
    out = sj.sj_judge_train(Hd, yd, Hd, yd, [0.5])                                   # and the call still works after errors
    assert out["best_index"] == 0 and 0.5 <= out["auc"][0] <= 1.0


@pytest.mark.parametrize("n,d,C", [(2000, 8192, 0.01), (1000, 6144, 3.0), (513, 3072, 0.3)])
def test_judge_training_wide_rows_meet_optimality_conditions(n, d, C):
    """Feature widths of the larger targets (d 8192 = 70B-shaped: rows in two-row groups) where the oracle's dense
    Hessian is too slow: the returned point must be stationary for the strictly convex objective."""
    H, y = synth.make_judge_dataset(21, n, d)
    Hv, yv = synth.make_judge_dataset(22, 400, d)
    out = sj.sj_judge_train(_dev(H), _dev(y), _dev(Hv), _dev(yv), [C], torch.cuda.current_stream())
    w, b = out["w"], out["b"]
    Hd = H.astype(np.float64)
    s = 1.0 / (1.0 + np.exp(-(Hd @ w + b)))
    gmax = max(np.abs(w + C * ((s - y) @ Hd)).max(), abs(C * np.sum(s - y)))
    print(f"d = {d}: max |grad| = {gmax:.2e} after {out['passes'][0]} passes", flush=True)
    assert gmax <= 1e-9 * max(1.0, C * n)
    sv = jt.scores_of(Hv, w, b)
    assert abs(out["auc"][0] - jt.roc_auc(sv, yv)) <= _auc_slack(sv, yv, 1e-9) + 1e-15


def test_judge_training_at_paper_size_meets_optimality_conditions():
    """69,432 pairs of 4096 features (the paper's Llama-3.1-8B training set size), one C: the result must be the
    stationary point of the strictly convex objective - gradient recomputed on the CPU in fp64."""
    n, d, n_val = 69432, 4096, 4096
    H, y = synth.make_judge_dataset(11, n, d)
    Hv, yv = synth.make_judge_dataset(12, n_val, d)
    C = 0.0129
    Hd, yd, Hvd, yvd = _dev(H), _dev(y), _dev(Hv), _dev(yv)
    torch.cuda.synchronize()
    t0 = time.time()
    out = sj.sj_judge_train(Hd, yd, Hvd, yvd, [C], torch.cuda.current_stream())
    dt = time.time() - t0
    w, b = out["w"], out["b"]
    z = H.astype(np.float64) @ w + b                      # one fp64 pass on the host
    s = 1.0 / (1.0 + np.exp(-z))
    g_w = w + C * ((s - y) @ H.astype(np.float64))
    g_b = C * np.sum(s - y)
    gmax = max(np.abs(g_w).max(), abs(g_b))
    print(f"paper-size fit: {dt:.2f} s, {out['passes'][0]} passes over 1.14 GB, max |grad| = {gmax:.2e}", flush=True)
    assert gmax <= 1e-9 * max(1.0, C * n)
    sv = 1.0 / (1.0 + np.exp(-(Hv.astype(np.float64) @ w + b)))
    assert abs(out["auc"][0] - jt.roc_auc(sv, yv)) <= _auc_slack(sv, yv, 1e-9) + 1e-15
    assert abs(out["theta_recall"] - jt.best_recall_threshold(sv, yv)) < 1e-9
    assert abs(out["theta_f1"] - jt.best_f1_threshold(sv, yv)["theta"]) < 1e-9


@pytest.mark.parametrize("n,d,n_C", [(700, 512, 10), (61, 1024, 3), (5, 4, 2), (257, 2048, 5), (130, 2052, 6), (90, 6144, 3)])
def test_grid_equals_its_values_one_at_a_time(n, d, n_C):
    """Problems share the passes over the matrix (up to four at a time, two for wide rows) and take each other's place when one
    is done: every model of a grid is bit for bit the one that its C gives alone, over all forms of the pass (teams of 1, 2, 4
    and 8 waves a row, 1 - 4 column pieces a wave, rows left over, fewer rows than workgroups)."""
    H, y = synth.make_judge_dataset(31, n, d)
    y[:2] = [0, 1]
    Hd, yd = _dev(H), _dev(y)
    grid = np.logspace(-2, 0.5, n_C)
    out = sj.sj_judge_train(Hd, yd, Hd, yd, grid, torch.cuda.current_stream())
    for c in range(n_C):
        one = sj.sj_judge_train(Hd, yd, Hd, yd, [grid[c]], torch.cuda.current_stream())
        assert (out["w_all"][c] == one["w_all"][0]).all() and out["passes"][c] == one["passes"][0] and out["auc"][c] == one["auc"][0]
    x = np.concatenate([H.astype(np.float64), np.ones((n, 1))], axis=1)
    for c in range(n_C):
        w = out["w_all"][c]
        g = np.append(w[:d], 0.0) + grid[c] * (x.T @ (1.0 / (1.0 + np.exp(-(x @ w))) - y))
        assert np.abs(g).max() <= 2e-11 * max(1.0, grid[c] * n) + 1e-12 * np.abs(x).sum(axis=0).max() * grid[c]


@pytest.mark.parametrize("n_val,n_C", [(6000, 1), (4097, 2), (3, 4)])
def test_validation_over_every_launch_size(n_val, n_C):
    """Scores of one model or several over validation sets with more rows than the launch has waves, and with fewer than a
    workgroup has: AUC and thresholds against the definitions, on the scores of the returned weights."""
    d = 8
    H, y = synth.make_judge_dataset(51, 200, d)
    Hv, yv = synth.make_judge_dataset(52, n_val, d)
    y[:2] = yv[:2] = [0, 1]
    out = sj.sj_judge_train(_dev(H), _dev(y), _dev(Hv), _dev(yv), np.logspace(-2, 1, n_C), torch.cuda.current_stream())
    for c in range(n_C):
        w = out["w_all"][c]
        sv = jt.scores_of(Hv, w[:d], w[d])
        assert abs(out["auc"][c] - jt.roc_auc(sv, yv)) <= _auc_slack(sv, yv, 1e-9) + 1e-15
    sv = jt.scores_of(Hv, out["w"], out["b"])
    assert abs(out["theta_recall"] - jt.best_recall_threshold(sv, yv)) < 1e-9
    assert abs(out["theta_f1"] - jt.best_f1_threshold(sv, yv)["theta"]) < 1e-9


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("d", [8, 1028])
def test_features_that_are_not_finite_do_not_converge(value, d):
    H, y = synth.make_judge_dataset(61, 120, d)
    bad = H.copy()
    bad[77, d - 3] = value
    yd = _dev(y)
    with pytest.raises(sj.SJError, match="did not converge") as e:
        sj.sj_judge_train(_dev(bad), yd, _dev(H), yd, [0.1, 1.0, 10.0])
    assert e.value.code == -3
    assert sj.sj_judge_train(_dev(H), yd, _dev(H), yd, [0.1])["passes"][0] > 0


@pytest.mark.parametrize("n,d,n_C", [(1027, 256, 4), (1026, 260, 3), (2049, 508, 1), (300, 1028, 2), (1029, 4096, 3), (1030, 4092, 4), (40, 4100, 2), (41, 8188, 2)])
def test_every_model_is_stationary_at_the_edges_of_the_pass(n, d, n_C):
    """Whole and cut column pieces of a wave, groups of rows with one, two and three rows over, one to four slots in use: the gradient in
    64 bits on the CPU.  Bound: the solver's own tolerance, 1e-11 max(1, C n), and the rounding of its sums and of these."""
    H, y = synth.make_judge_dataset(41, n, d)
    y[:2] = [0, 1]
    grid = np.logspace(-2, 0.0, n_C)
    out = sj.sj_judge_train(_dev(H), _dev(y), _dev(H), _dev(y), grid, torch.cuda.current_stream())
    x = np.concatenate([H.astype(np.float64), np.ones((n, 1))], axis=1)
    for c in range(n_C):
        w = out["w_all"][c]
        g = np.append(w[:d], 0.0) + grid[c] * (x.T @ (1.0 / (1.0 + np.exp(-(x @ w))) - y))
        assert np.abs(g).max() <= 2e-11 * max(1.0, grid[c] * n) + 1e-12 * np.abs(x).sum(axis=0).max() * grid[c]
