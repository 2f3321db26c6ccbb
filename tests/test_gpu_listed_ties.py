"""GPU parity of the listed windows on weights with many equal magnitudes (pruned before, widened from few bits): what the lists
leave open, by one workgroup and by the whole grid, one ranking and many, beside rankings that the lists resolve; windows of
256 sampling workgroups; list indices beyond 2^31.  Against the oracle, bit for bit, and against the time of radix levels."""
import threading
import time

import numpy as np
import pytest
import torch

import oracle
import paper_1911_02497_amd as P
from gpu_util import assert_bits_equal, assert_select_equal, check_prune_against_oracle, DEV, up

pytestmark = pytest.mark.gpu


def _tied(kind, n, seed):
    w = np.random.default_rng(seed).standard_normal(n).astype(np.float32) * np.float32(0.02)
    if kind == "zeros":                                      # nine tenths pruned before
        w[np.abs(w) < 0.0329] = 0.0
    elif kind == "grid8":
        s = np.abs(w).max() / np.float32(127)
        w = (np.round(w / s) * s).astype(np.float32)
    elif kind == "grid4":
        s = np.abs(w).max() / np.float32(7)
        w = (np.round(w / s) * s).astype(np.float32)
    elif kind == "e4m3":
        w = torch.from_numpy(w).to(torch.float8_e4m3fn).float().numpy()
    elif kind == "bf16":
        w = torch.from_numpy(w).bfloat16().float().numpy()
    return w


KINDS = ["zeros", "grid8", "grid4", "e4m3", "bf16"]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n", [5, 4097, 65536, 65537, 131072, 131073, 262144, 262149, (1 << 21) + 3, (1 << 23) + 5])
def test_one_population(kind, n):
    w = _tied(kind, n, n)
    kept = float(np.count_nonzero(w)) / n
    for ds in ([0.05], [kept], [0.3], [0.02, 0.1, 0.3, 0.9]):
        want = oracle.prune([w], ds, P.SCOPE_GLOBAL)
        res = P.condensa_prune(up([w]), ds, theta_f16=True)
        torch.cuda.synchronize()
        check_prune_against_oracle(res, want, P.SCOPE_GLOBAL, 1, f"{kind} {n} {ds}")
    shifted = torch.empty(n + 1, dtype=torch.float32, device=DEV)[1:]
    shifted.copy_(torch.from_numpy(w))
    res = P.condensa_prune([shifted], [0.3])
    torch.cuda.synchronize()
    check_prune_against_oracle(res, oracle.prune([w], [0.3], P.SCOPE_GLOBAL), P.SCOPE_GLOBAL, 1, f"{kind} {n} shifted")


@pytest.mark.parametrize("sizes", [[70, 9000, 0, 30000, 1, 65536], [70, 300001, 0, 9000, 1 << 20, 262144, 1, 2100000, 16385]], ids=["small", "mixed"])
@pytest.mark.parametrize("scope", [P.SCOPE_GLOBAL, P.SCOPE_PER_TENSOR])
@pytest.mark.parametrize("ds", [[0.12], [0.02, 0.1, 0.12, 0.5, 0.97]], ids=["one", "five"])
def test_models_of_tied_and_ordinary_tensors(sizes, scope, ds):
    kinds = ["normal"] + KINDS
    arrs = [_tied(kinds[(i * 2 + len(sizes)) % 6], n, 10 + i) for i, n in enumerate(sizes)]
    want = oracle.prune(arrs, ds, scope)
    for config in (None, {"window_margin": 0}, {"cand_shift": 12}):
        res = P.condensa_prune(up(arrs), ds, scope=scope, theta_f16=True, config=config)
        torch.cuda.synchronize()
        check_prune_against_oracle(res, want, scope, len(arrs), f"{sizes} {config}")


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n", [50000, 700003])
@pytest.mark.parametrize("pq", [False, True])
@pytest.mark.parametrize("in_place", [False, True])
def test_lc_step(kind, n, pq, in_place):
    arrs = [_tied(kind, n, 3), _tied(kind, 777, 4)]
    lams = [np.zeros_like(a) for a in arrs]
    mu = 1e-3
    for density in (0.05, 0.3):
        lam = up(lams)
        call = P.condensa_lc_step_pq if pq else P.condensa_lc_step
        res = call(up(arrs), lam, mu, density, in_place=in_place, **({"nnz": True} if pq else {}))
        torch.cuda.synchronize()
        ora = (oracle.lc_step_pq if pq else oracle.lc_step)(arrs, lams, mu, density)
        assert_select_equal(P.select_records(res["results"])[0], ora["select"])
        for i in range(len(arrs)):
            for name in ("theta", "lambda", "grad"):
                assert_bits_equal(res[name][i], ora[name][i], f"{name} {i}")
            assert np.array_equal(res["mask"][i].cpu().numpy(), ora["mask"][i])
        if pq:
            assert int(res["nnz"].item()) == sum(int(((t.cpu().numpy().view(np.uint16) & 0x7FFF) != 0).sum()) for t in res["theta_f16"])


def test_a_tile_that_lies_in_one_window():
    """Several densities: a wavefront whose elements all belong on one list, more than it can buffer."""
    rng = np.random.default_rng(1)
    w = rng.standard_normal(3_000_000).astype(np.float32)
    t = np.sort(np.abs(w))[::-1][int(0.1 * w.size)]
    near = (t * (1.0 + 1e-5 * rng.standard_normal(40_000))).astype(np.float32)
    arrs = [w, near]
    for ds in ([0.1, 0.4], [0.1 + 0.05 * j for j in range(10)]):
        res = P.condensa_prune(up(arrs), ds)
        torch.cuda.synchronize()
        check_prune_against_oracle(res, oracle.prune(arrs, ds, P.SCOPE_GLOBAL), P.SCOPE_GLOBAL, 2, str(len(ds)))


@pytest.mark.parametrize("kind", ["normal", "grid8", "zeros"])
def test_windows_of_256_sampling_workgroups(kind):
    arrs = [_tied(kind, (1 << 23) + 999, 1), _tied(kind, (1 << 23) + (1 << 21) + 1, 2), _tied(kind, 12345, 3)]
    want = oracle.prune(arrs, [0.07], P.SCOPE_PER_TENSOR)
    res = P.condensa_prune(up(arrs), [0.07], scope=P.SCOPE_PER_TENSOR)
    torch.cuda.synchronize()
    check_prune_against_oracle(res, want, P.SCOPE_PER_TENSOR, 3, kind)
    rng = np.random.default_rng(9)
    lams = [(rng.standard_normal(a.shape) * 2e-6).astype(np.float32) for a in arrs]
    res = P.condensa_lc_step(up(arrs), up(lams), 1e-3, 0.07)
    torch.cuda.synchronize()
    ora = oracle.lc_step(arrs, lams, 1e-3, 0.07)
    assert_select_equal(P.select_records(res["results"])[0], ora["select"])
    for i in range(3):
        for name in ("theta", "lambda", "grad"):
            assert_bits_equal(res[name][i], ora[name][i], f"{kind} {name} {i}")


def test_streams_and_threads_with_calls_that_are_left_open():
    """Calls on several streams at once, all of which end in the passes that the whole grid takes together."""
    models = [[_tied("zeros", 300000 + 7777 * i, i), _tied("grid4", 150000, 50 + i)] for i in range(4)]
    want = [oracle.prune(m, [0.3], P.SCOPE_PER_TENSOR) for m in models]
    got = [[] for _ in models]

    def work(i):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            d = up(models[i])
            for _ in range(20):
                got[i].append(P.condensa_prune(d, [0.3], scope=P.SCOPE_PER_TENSOR))
            s.synchronize()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(models))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for w, rs in zip(want, got):
        for r in rs:
            check_prune_against_oracle(r, w, P.SCOPE_PER_TENSOR, 2)


def test_captured_call_that_is_left_open():
    dev = up([_tied("grid4", 400000, 1), _tied("normal", 3000, 2)])
    res = P.condensa_prune(dev, [0.2], scope=P.SCOPE_PER_TENSOR)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        P.condensa_prune(dev, [0.2], scope=P.SCOPE_PER_TENSOR, outputs=res, workspace=res["workspace"])
    for i, kind in enumerate(("zeros", "normal", "e4m3")):
        arrs = [_tied(kind, 400000, 10 + i), _tied("zeros", 3000, 20 + i)]
        for d, a in zip(dev, arrs):
            d.copy_(torch.from_numpy(a))
        graph.replay()
        torch.cuda.synchronize()
        check_prune_against_oracle(res, oracle.prune(arrs, [0.2], P.SCOPE_PER_TENSOR), P.SCOPE_PER_TENSOR, 2, kind)


def _seconds(call):
    call()
    torch.cuda.synchronize()
    best = 1e9
    for _ in range(5):
        t0 = time.perf_counter()
        for _ in range(4):
            call()
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t0) / 4)
    return best


@pytest.mark.parametrize("kind", ["zeros", "grid8", "grid4", "e4m3"])
@pytest.mark.parametrize("form", ["layers", "search", "layer_searches"])
def test_tied_weights_take_no_longer_than_radix_levels(kind, form):
    """Every ranking of a call may be left open by its list; all of them then go through the same few passes.  One ranking
    after the other took 4 to 60 times as long as radix levels; the bound leaves room for noise."""
    dev = up([_tied(kind, n, n) for n in [262144 + 999 * i for i in range(12)] + [2359296] * 5])
    ds = {"layers": [0.2], "search": [0.005 * 100.0 ** (j / 9) for j in range(10)], "layer_searches": [0.05, 0.1, 0.3]}[form]
    scope = P.SCOPE_GLOBAL if form == "search" else P.SCOPE_PER_TENSOR
    took = {}
    for name, config in (("auto", None), ("radix", {"select_path": 1})):
        table = P.TensorTable(dev)
        res = P.condensa_prune(table, ds, scope, theta=form == "layers", config=config)
        took[name] = _seconds(lambda: P.condensa_prune(table, ds, scope, theta=form == "layers", outputs=res, workspace=res["workspace"], config=config))
    assert took["auto"] < 2.5 * took["radix"], took


def test_several_densities_of_more_than_2_31_weights():
    """List indices use all 32 bits.  Checked by what defines a mask: its count, the keys above and below the threshold, and the
    order of the kept ties."""
    n_each, densities = (1 << 29) + 12345, [0.03, 0.4]
    ws = []
    try:
        for t in range(4):
            g = torch.Generator(device=DEV).manual_seed(t)
            w = torch.empty(n_each, dtype=torch.float32, device=DEV).normal_(generator=g)
            ws.append(w.bfloat16().float() if t == 3 else w)
        total = 4 * n_each
        assert total > 1 << 31
        res = P.condensa_prune(ws, densities, theta=False)
        torch.cuda.synchronize()
        for j, d in enumerate(densities):
            rec = P.select_records(res["results"])[j]
            T, kept, above, ties, start = rec["threshold_key"], 0, 0, 0, 0
            for t, w in enumerate(ws):
                key, m = w.abs().view(torch.int32), res["mask"][j][t].bool()
                kept += int(m.sum())
                above += int((key > T).sum())
                assert bool((m | (key <= T)).all()) and not bool((m & (key < T)).any()), f"density {d} tensor {t}"
                eq = (key == T).nonzero().flatten()
                ties += eq.numel()
                assert torch.equal(m[eq], eq + start < rec["tie_end"]), f"density {d} tensor {t}: ties"
                start += w.numel()
                del key, m, eq
            assert kept == rec["k"] == round(d * total) and above == rec["n_gt"] and ties == rec["n_tie"], rec
    finally:
        del ws
        torch.cuda.empty_cache()
