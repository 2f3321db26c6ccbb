"""GPU parity of the listed windows through events that an idle device does not show by itself: workgroups that start after the
others are done, waits that run out.  Every kernel of these calls ends as in any other call.  Against the oracle, bit for bit."""
import contextlib

import numpy as np
import pytest
import torch

import oracle
import paper_1911_02497_amd as P
from gpu_util import assert_bits_equal, assert_select_equal, check_prune_against_oracle, up

pytestmark = pytest.mark.gpu

LATE, NO_SAMPLE, NO_VERDICT, ASK, NO_POSTS = 1, 2, 4, 8, 16              # csrc/host.h


@contextlib.contextmanager
def forced(what):
    lib = P.library()
    lib.condensa_test_force(what)
    try:
        yield
    finally:
        lib.condensa_test_force(0)


def _weights(kind, n):
    """What a list leaves open: thousands of ties cut in the middle, a crowded sample, nothing to keep."""
    w = np.random.default_rng(n).standard_normal(n).astype(np.float32) * np.float32(0.02)
    if kind == "zeros":
        w[np.abs(w) < 0.0329] = 0.0
    elif kind == "grid":
        w = (np.round(w * 1024) / 1024).astype(np.float32)
    elif kind == "atom":
        w[np.abs(w) > 0.035] = np.float32(-0.035)
    return w


def _check_all_calls(w, density, config=None):
    arrs, lams = [w, w[:777].copy()], [np.zeros_like(w), np.zeros(777, np.float32)]
    for outputs in ({"theta_f16": True}, {"in_place": True}):
        res = P.condensa_prune(up(arrs), [density], config=config, **outputs)
        torch.cuda.synchronize()
        check_prune_against_oracle(res, oracle.prune(arrs, [density], P.SCOPE_GLOBAL), P.SCOPE_GLOBAL, 2, f"{density} {config}")
    for pq in (False, True):
        call, ora = (P.condensa_lc_step_pq, oracle.lc_step_pq) if pq else (P.condensa_lc_step, oracle.lc_step)
        res = call(up(arrs), up(lams), 1e-3, density, config=config, **({"nnz": True} if pq else {}))
        torch.cuda.synchronize()
        want = ora(arrs, lams, 1e-3, density)
        assert_select_equal(P.select_records(res["results"])[0], want["select"], f"{density} {config} pq={pq}")
        for i in range(2):
            for name in ("theta", "lambda", "grad"):
                assert_bits_equal(res[name][i], want[name][i], f"{name} {i}")
            assert np.array_equal(res["mask"][i].cpu().numpy(), want["mask"][i])
        if pq:
            codes = [t.cpu().numpy().view(np.uint16) for t in res["theta_f16"]]
            assert int(res["nnz"].item()) == sum(int(((c & 0x7FFF) != 0).sum()) for c in codes)


@pytest.mark.parametrize("kind, density, config", [
    ("zeros", 0.05, None), ("zeros", 0.3, None), ("grid", 0.1, None), ("atom", 0.05, None), ("normal", 0.2, {"window_margin": 0}),
    ("normal", 0.2, {"cand_shift": 12}), ("normal", 0.0, None)])
@pytest.mark.parametrize("n", [200003, (1 << 21) + 3])
def test_workgroups_that_start_when_the_ranking_is_done(kind, density, config, n):
    """Records and counts of what the lists leave open stay as they were written."""
    with forced(LATE):
        _check_all_calls(_weights(kind, n), density, config)


@pytest.mark.parametrize("sizes", [[200003], [(1 << 21) + 3, 777], [300001, 9, 700000, 0, 66000]], ids=str)
@pytest.mark.parametrize("kind", ["normal", "zeros"])
def test_windows_whose_samples_do_not_come(sizes, kind):
    """The whole population is searched, beside populations with a lone sampling workgroup, which has nobody to wait for."""
    arrs = [_weights(kind, n) for n in sizes]
    for scope in (P.SCOPE_GLOBAL, P.SCOPE_PER_TENSOR):
        for ds in ([0.1], [0.02, 0.0, 0.1, 0.5, 1.0]):
            with forced(NO_SAMPLE):
                res = P.condensa_prune(up(arrs), ds, scope=scope, theta_f16=True)
            torch.cuda.synchronize()
            check_prune_against_oracle(res, oracle.prune(arrs, ds, scope), scope, len(arrs), f"{sizes} {kind} {ds}")
    with forced(NO_SAMPLE):
        _check_all_calls(arrs[0], 0.1)


@pytest.mark.parametrize("what", [NO_VERDICT, ASK, NO_POSTS, NO_POSTS | NO_VERDICT], ids=["leave", "ask", "no_posts", "no_posts_leave"])
@pytest.mark.parametrize("n", [140001, 300007, (1 << 21) + 3])
@pytest.mark.parametrize("ties", [0, 60, 900, 2040])
def test_entries_of_workgroups_that_do_not_stay(n, ties, what):
    """The entries of the threshold's bin are settled by the workgroups that posted them, by the one that ranks them when those have
    left, and by a search of everything when it does not get them: every decision, multiplier and code the same."""
    w = np.random.default_rng(n + ties).standard_normal(n).astype(np.float32)
    order = np.argsort(-np.abs(w), kind="stable")
    k = n // 7
    w[order[k - ties // 2:k + (ties + 1) // 2]] = np.abs(w[order[k]])      # the values next to the threshold become equal
    with forced(what):
        for d in (k / n, (k + ties // 3) / n):
            _check_all_calls(w, d * n / (n + 777))
        shifted = torch.empty(n + 1, dtype=torch.float32, device="cuda:0")[1:]
        shifted.copy_(torch.from_numpy(w))
        res = P.condensa_prune([shifted], [k / n], theta_f16=True)
        torch.cuda.synchronize()
        check_prune_against_oracle(res, oracle.prune([w], [k / n], P.SCOPE_GLOBAL), P.SCOPE_GLOBAL, 1, f"{n} {ties} {what}")
        assert P.select_records(res["results"])[0]["path"] == (3 if what & NO_POSTS else 2)
