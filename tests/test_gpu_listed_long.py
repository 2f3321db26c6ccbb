"""GPU parity of listed windows on lists of millions of entries (2^27 weights and more, one density; 3 2^26 and more are ranked by kernels of their own): bins of thousands of entries, ties in them,
workgroups that leave.  Against the radix levels, which the oracle anchors at sizes that it can sort; bit for bit."""
import contextlib
import time

import pytest
import torch

import paper_1911_02497_amd as P
from gpu_util import DEV
from paper_1911_02497_amd.binding import OP_PRUNE, OP_LC_STEP

pytestmark = pytest.mark.gpu

LATE, NO_VERDICT, ASK, NO_POSTS = 1, 4, 8, 16                            # csrc/host.h
FIELDS = ("n", "k", "n_gt", "n_tie_kept", "n_tie", "threshold_key", "tie_end")


@contextlib.contextmanager
def forced(what):
    lib = P.library()
    lib.condensa_test_force(what)
    try:
        yield
    finally:
        lib.condensa_test_force(0)


def _weights(kind, n):
    g = torch.Generator(device=DEV).manual_seed(n % 1000)
    w = torch.empty(n, dtype=torch.float32, device=DEV).normal_(0.0, 0.02, generator=g)
    if kind == "ties":                                     # the upper half of a bin's width around the threshold of 0.1: thousands of equal keys
        w[(w.abs() - 0.0329).abs() < 1e-6] = 0.0329
    return [w[:n // 3].view(-1, 1), w[n // 3:]]


def _same(a, b):
    return torch.equal(a.view(torch.int32) if a.dtype == torch.float32 else a, b.view(torch.int32) if b.dtype == torch.float32 else b)


@pytest.mark.timeout(300)
@pytest.mark.parametrize("kind", ["normal", "ties"])
@pytest.mark.parametrize("n", [(1 << 27) + 1, (3 << 26) - 1, 3 << 26, 400_000_003])
def test_prune_and_steps(kind, n):
    ws = _weights(kind, n)
    lam = [t * 0.0 for t in ws]
    for d in (0.1, 0.6):
        ref = P.condensa_prune(ws, [d], config={"select_path": 1})
        want = P.select_records(ref["results"])[0]
        step = P.condensa_lc_step(ws, lam, 1e-3, d, config={"select_path": 1})
        for what in (0, LATE, NO_VERDICT, ASK) if d == 0.1 else (0, NO_POSTS) if n < 1 << 28 else (0,):
            with forced(what):
                res = P.condensa_prune(ws, [d])
                got = P.select_records(res["results"])[0]
            assert all(got[f] == want[f] for f in FIELDS), (what, got, want)
            for name in ("theta", "mask"):
                assert all(_same(a, b) for a, b in zip(res[name][0], ref[name][0])), (what, name)
            with forced(what):
                res = P.condensa_lc_step(ws, lam, 1e-3, d)
            for name in ("theta", "lambda", "grad", "mask"):
                assert all(_same(a, b) for a, b in zip(res[name], step[name])), (what, name)
        pq = P.condensa_lc_step_pq(ws, lam, 1e-3, d, nnz=True)
        assert int(pq["nnz"].item()) == sum(int(((c & 0x7FFF) != 0).sum()) for c in pq["theta_f16"])
        assert all(_same(a, b) for a, b in zip(pq["mask"], step["mask"]))
        del ref, step, pq, res


@pytest.mark.timeout(300)
@pytest.mark.parametrize("scale,d", [(1.0, 0.1), (1.5, 0.4)])
def test_bins_of_tens_of_thousands(scale, d):
    """Rows whose sizes differ widen the window: some 30 thousand entries in the threshold's bin."""
    g = torch.Generator(device=DEV).manual_seed(5)
    w = torch.empty((131072, 4608), dtype=torch.float32, device=DEV).normal_(0.0, 0.02, generator=g)
    w *= torch.exp(scale * torch.empty((131072, 1), dtype=torch.float32, device=DEV).normal_(0.0, 1.0, generator=g))
    ws = [w[:100_000], w[100_000:]]
    lam = [t * 0.0 for t in ws]
    ref = P.condensa_prune(ws, [d], config={"select_path": 1})
    want = P.select_records(ref["results"])[0]
    for what in (0, LATE, NO_VERDICT, ASK, NO_POSTS, NO_POSTS | NO_VERDICT):
        with forced(what):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            res = P.condensa_prune(ws, [d])
            torch.cuda.synchronize()
            seconds = time.perf_counter() - t0
        got = P.select_records(res["results"])[0]
        assert all(got[f] == want[f] for f in FIELDS) and got["path"] == (3 if what & NO_POSTS else 2), (what, got, want)
        assert seconds < 0.5, (what, seconds)              # one workgroup goes over the list, not over the weights (seconds)
        for name in ("theta", "mask"):
            assert all(_same(a, b) for a, b in zip(res[name][0], ref[name][0])), (what, name)
        with forced(what):
            pq = P.condensa_lc_step_pq(ws, lam, 1e-3, d, nnz=True)
        assert all(_same(a, b) for a, b in zip(pq["mask"], ref["mask"][0])), what
        assert int(pq["nnz"].item()) == sum(int(((c & 0x7FFF) != 0).sum()) for c in pq["theta_f16"])


def _best(call):
    call()
    torch.cuda.synchronize()
    best = 1e9
    for _ in range(5):
        t0 = time.perf_counter()
        for _ in range(3):
            call()
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t0) / 3)
    return best


def _step_time(ws, lam):
    ws = P.TensorTable(ws)
    res = P.condensa_lc_step(ws, lam, 1e-3, 0.1, mask=False)
    return _best(lambda: P.condensa_lc_step(ws, lam, 1e-3, 0.1, mask=False, outputs=res, workspace=res["workspace"]))


# ties in the bin: about as many as are posted, more than one workgroup is sent, more than 2^18 (two binary digits less than binary16's)
@pytest.mark.timeout(300)
@pytest.mark.parametrize("n,digits", [(3 << 26, 10), (400_000_003, 10), (400_000_003, 8)])
def test_values_on_a_floating_point_grid(n, digits):
    ws = _weights("normal", n)
    for t in ws:
        bits = t.view(torch.int32)
        bits.add_(1 << (22 - digits)).bitwise_and_(-1 << (23 - digits))
    lam = [t * 0.0 for t in ws]
    for d in (0.1, 0.1003, 0.35):
        ref = P.condensa_prune(ws, [d], config={"select_path": 1})
        want = P.select_records(ref["results"])[0]
        assert want["n_tie"] > 40_000
        step = P.condensa_lc_step(ws, lam, 1e-3, d, config={"select_path": 1})
        for what in (0, LATE):
            with forced(what):
                res = P.condensa_prune(ws, [d])
                got = P.select_records(res["results"])[0]
            assert all(got[f] == want[f] for f in FIELDS) and got["path"] == 2, (what, got, want)      # nothing was left open
            for name in ("theta", "mask"):
                assert all(_same(a, b) for a, b in zip(res[name][0], ref[name][0])), (what, name)
            with forced(what):
                res = P.condensa_lc_step(ws, lam, 1e-3, d)
            for name in ("theta", "lambda", "grad", "mask"):
                assert all(_same(a, b) for a, b in zip(res[name], step[name])), (what, name)
        del ref, step, res
    pq = P.condensa_lc_step_pq(ws, lam, 1e-3, 0.1, nnz=True)
    assert int(pq["nnz"].item()) == sum(int(((c & 0x7FFF) != 0).sum()) for c in pq["theta_f16"])


@pytest.mark.timeout(300)
def test_workspaces_with_room_for_fewer_gathered_entries():
    n = (3 << 26) + 7
    ws = _weights("normal", n)
    for t in ws:
        t.view(torch.int32).add_(1 << 14).bitwise_and_(-1 << 15)         # 260 thousand ties
    lam = [t * 0.0 for t in ws]
    ref = P.condensa_lc_step(ws, lam, 1e-3, 0.1, config={"select_path": 1})
    want = P.select_records(ref["results"])[0]
    assert want["n_tie"] > 1 << 17
    full = P.condensa_workspace_bytes(OP_LC_STEP, n, 0, 2, 4, P.SCOPE_GLOBAL)            # (four densities: the lists alone)
    for size in (full, full - 256, full - 6 * (1 << 20)):
        res = P.condensa_lc_step(ws, lam, 1e-3, 0.1, workspace=torch.empty(size, dtype=torch.uint8, device=DEV))
        got = P.select_records(res["results"])[0]
        assert all(got[f] == want[f] for f in FIELDS), (size, got, want)
        for name in ("theta", "lambda", "grad", "mask"):
            assert all(_same(a, b) for a, b in zip(res[name], ref[name])), (size, name)
    with pytest.raises(P.CondensaError):
        P.condensa_lc_step(ws, lam, 1e-3, 0.1, workspace=torch.empty(full - 7 * (1 << 20), dtype=torch.uint8, device=DEV))


@pytest.mark.timeout(300)
def test_ties_do_not_set_the_time():
    """Counted by another sweep over weights and multipliers they took 1.5 times the step of other weights (1.04 times counted where they lie gathered)."""
    g = torch.Generator(device=DEV).manual_seed(5)
    ws = [torch.empty(603_979_776, dtype=torch.float32, device=DEV).normal_(0.0, 0.02, generator=g)]
    lam = [torch.zeros_like(ws[0])]
    other = _step_time(ws, lam)
    ws[0].copy_(ws[0].half())
    this = _step_time(ws, lam)
    assert this < 1.2 * other, (this, other)


def _rows_differ(n, scale):
    """n matrices of rows whose sizes are spread by e^scale to either side, and multipliers."""
    g, by_row = [torch.Generator(device=DEV).manual_seed(s) for s in (3, 7)]
    ws = [torch.empty((4096, 4608), dtype=torch.float32, device=DEV).normal_(0.0, 0.02, generator=g) for _ in range(n)]
    lam = [torch.empty((4096, 4608), dtype=torch.float32, device=DEV).normal_(0.0, 6e-6, generator=g) for _ in range(n)]
    for w in ws:
        w *= torch.exp(scale * torch.randn((4096, 1), device=DEV, generator=by_row))
    return ws, lam


@pytest.mark.timeout(300)
def test_workgroups_wait_for_the_one_that_ranks():
    """Hundreds of thousands of corrections: the workgroup that ranks did its own first, the others left meanwhile, and it settled their entries one after the
    other: 1.15 times the step of rows alike, 1.06 where it ranks at once."""
    alike, this = [_step_time(*_rows_differ(32, scale)) for scale in (0.0, 1.0)]
    assert this < 1.1 * alike, (this, alike)


@pytest.mark.timeout(300)
def test_rows_of_different_sizes_do_not_set_the_time():
    """Draws from such rows are skewed, and their mean left a million wrong decisions: 1.08 times the step of rows alike, 1.02 from their median."""
    alike, this = [_step_time(*_rows_differ(64, scale)) for scale in (0.0, 1.0)]
    assert this < 1.05 * alike, (this, alike)


# a selection that is a sweep of its own: either side of the lines between the two windows, and a workspace that has room for the lists alone
@pytest.mark.timeout(300)
@pytest.mark.parametrize("op,n", [("lc", (3 << 26) - 1), ("lc", 3 << 26), ("prune", (1 << 29) - 1), ("prune", (1 << 29) + 3)])
def test_two_sweeps(op, n):
    w = _weights("normal", n)
    d = 0.1
    lists = n // 4                                         # bytes: more than the lists take, less than the sampled window
    if op == "lc":
        lam = [t * 1e-4 for t in w]
        ref = P.condensa_lc_step(w, lam, 1e-3, d, config={"select_path": 1})
        names = ("theta", "lambda", "grad", "mask")
    else:
        ref = P.condensa_prune(w, [d], config={"select_path": 1})
        names = ("theta", "mask")
    want = P.select_records(ref["results"])[0]
    for ws in (None, torch.empty(lists, dtype=torch.uint8, device=DEV)):
        if ws is not None:
            assert n < 3 << 26 or lists < P.condensa_workspace_bytes(OP_LC_STEP if op == "lc" else OP_PRUNE, n, 0, 2, 1, P.SCOPE_GLOBAL)
        if op == "lc":
            mine = [t.clone() for t in lam]
            res = P.condensa_lc_step(w, mine, 1e-3, d, in_place=True, workspace=ws)
            res = dict(res, **{"lambda": mine})
            pairs = [(res[name], ref[name]) for name in names]
        else:
            res = P.condensa_prune(w, [d], workspace=ws, config={"fused_sweep": 1})
            pairs = [(res[name][0], ref[name][0]) for name in names]
            alone = P.select_records(P.condensa_prune(w, [d], theta=False, mask=False, workspace=ws)["results"])[0]
            assert all(alone[f] == want[f] for f in FIELDS), (alone, want)
        got = P.select_records(res["results"])[0]
        assert all(got[f] == want[f] for f in FIELDS), (got, want)
        assert all(_same(a, b) for x, y in pairs for a, b in zip(x, y))
        del res, pairs
