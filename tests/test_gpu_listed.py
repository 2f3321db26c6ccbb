"""GPU parity of the listed windows (what the automatic choice takes for ordinary calls): sizes at the edges of the
rules (sampling workgroups, tiles, list segments), windows that miss or overlap, populations that crowd into a few
values, all rankings of both scopes; against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_1911_02497_amd as P
from gpu_util import assert_bits_equal, assert_select_equal, check_prune_against_oracle, DEV, up

pytestmark = pytest.mark.gpu

MISS = {"window_margin": 0}                       # windows of almost no width: the rankings go to the fallback


def _check_lc(arrs, lams, density, config=None, in_place=False, pq=False):
    mu = 1e-3
    dev, lam = up(arrs), up(lams)
    call = P.condensa_lc_step_pq if pq else P.condensa_lc_step
    res = call(dev, lam, mu, density, in_place=in_place, config=config, **({"nnz": True} if pq else {}))
    torch.cuda.synchronize()
    ora = (oracle.lc_step_pq if pq else oracle.lc_step)(arrs, lams, mu, density)
    assert_select_equal(P.select_records(res["results"])[0], ora["select"])
    for i in range(len(arrs)):
        for name in ("theta", "lambda", "grad"):
            assert_bits_equal(res[name][i], ora[name][i], f"{name} {i}")
        assert np.array_equal(res["mask"][i].cpu().numpy(), ora["mask"][i])
    if pq:
        codes = [res["theta_f16"][i].cpu().numpy().view(np.uint16) for i in range(len(arrs))]
        assert int(res["nnz"].item()) == sum(int(((c & 0x7FFF) != 0).sum()) for c in codes)


@pytest.mark.parametrize("n", [1, 255, 4096, 4097, 16384, (1 << 20), (1 << 20) + 3, (1 << 21), (1 << 21) + 5, (1 << 22) + 1])
@pytest.mark.parametrize("config", [None, MISS], ids=["window", "miss"])
def test_population_sizes(n, config):
    w = np.random.default_rng(n).standard_normal(n).astype(np.float32)
    for ds in ([0.3], [0.01, 0.2, 0.6]):
        res = P.condensa_prune(up([w]), ds, theta_f16=True, config=config)
        torch.cuda.synchronize()
        check_prune_against_oracle(res, oracle.prune([w], ds, P.SCOPE_GLOBAL), P.SCOPE_GLOBAL, 1, str(n))


@pytest.mark.parametrize("ds", [[0.1, 0.1], [0.1, 0.1001, 0.1002, 0.5], [1.0, 0.0, 0.5], [0.0, 0.0], [1.0, 1.0, 0.9999999],
                                [0.5 - 0.03 * j for j in range(16)]], ids=str)
@pytest.mark.parametrize("scope", [P.SCOPE_GLOBAL, P.SCOPE_PER_TENSOR])
@pytest.mark.parametrize("outputs", ["mask", "all"])
def test_windows_that_overlap_and_rankings_without_a_threshold(ds, scope, outputs):
    rng = np.random.default_rng(3)
    arrs = [rng.standard_normal(s).astype(np.float32) for s in ((300, 1111), (7,), (64, 32, 3, 3), (0,), (1 << 20,))]
    res = P.condensa_prune(up(arrs), ds, scope=scope, theta=outputs == "all", theta_f16=outputs == "all")
    torch.cuda.synchronize()
    check_prune_against_oracle(res, oracle.prune(arrs, ds, scope), scope, len(arrs))


@pytest.mark.parametrize("kind", ["zeros", "two_values", "all_equal", "levels", "edge"])
@pytest.mark.parametrize("scope", [P.SCOPE_GLOBAL, P.SCOPE_PER_TENSOR])
@pytest.mark.parametrize("ds", [[0.2], [0.05, 0.2, 0.7]], ids=["one", "three"])
def test_populations_that_crowd_into_few_values(kind, scope, ds):
    """Lists that overflow, bins that hold more than the gathering allows, thousands of ties cut in the middle."""
    rng = np.random.default_rng(4)
    w = rng.standard_normal((3, 400001)).astype(np.float32)
    if kind == "zeros":
        w[np.abs(w) < 1.6] = 0.0
    elif kind == "two_values":
        w = np.where(rng.random(w.shape) < 0.2, np.float32(0.5), np.float32(-0.25)).astype(np.float32)
    elif kind == "all_equal":
        w[:] = -3.0
    elif kind == "levels":
        w = (np.round(w * 16) / 16).astype(np.float32)
    else:
        w.reshape(-1)[: w.size // 3] = np.float32(1.2816)          # an atom right at one of the thresholds
    arrs = [np.ascontiguousarray(r) for r in w]
    res = P.condensa_prune(up(arrs), ds, scope=scope)
    torch.cuda.synchronize()
    check_prune_against_oracle(res, oracle.prune(arrs, ds, scope), scope, len(arrs), kind)


@pytest.mark.parametrize("config", [None, MISS, {"fused_sweep": 1}, {"cand_shift": 12}, {"sample_log2": 20}], ids=["window", "miss", "two_sweeps", "short_lists", "large_sample"])
@pytest.mark.parametrize("pq", [False, True])
@pytest.mark.parametrize("in_place", [False, True])
def test_lc_step(config, pq, in_place):
    rng = np.random.default_rng(5)
    shapes = [(64, 3, 3, 3), (513, 1027), (10, 512), (0,), (300001,)]
    arrs = [rng.standard_normal(s).astype(np.float32) * np.float32(0.05) for s in shapes]
    lams = [rng.standard_normal(s).astype(np.float32) * np.float32(2e-5) for s in shapes]
    _check_lc(arrs, lams, 0.1, config, in_place, pq)
    if pq:                                                           # kept values that underflow to zero in binary16
        _check_lc([a * np.float32(1e-7) for a in arrs], [l * np.float32(1e-7) for l in lams], 0.4, config, in_place, pq)


@pytest.mark.parametrize("config", [None, MISS], ids=["window", "miss"])
def test_per_tensor_population_sizes_in_one_call(config):
    """Lone sampling workgroups beside populations with many, one density and several; misaligned weights too."""
    rng = np.random.default_rng(6)
    arrs = [rng.standard_normal(n).astype(np.float32) for n in (5, (1 << 20) + 1, 0, 9000, (1 << 22) + 77, 1)]
    for ds in ([0.15], [0.02, 0.5]):
        want = oracle.prune(arrs, ds, P.SCOPE_PER_TENSOR)
        res = P.condensa_prune(up(arrs), ds, scope=P.SCOPE_PER_TENSOR, config=config)
        torch.cuda.synchronize()
        check_prune_against_oracle(res, want, P.SCOPE_PER_TENSOR, len(arrs))
        shifted = [torch.empty(a.size + 1, dtype=torch.float32, device=DEV)[1:] for a in arrs]
        for s, a in zip(shifted, arrs):
            s.copy_(torch.from_numpy(a))
        res = P.condensa_prune(shifted, ds, scope=P.SCOPE_PER_TENSOR, config=config)
        torch.cuda.synchronize()
        check_prune_against_oracle(res, want, P.SCOPE_PER_TENSOR, len(arrs))


def test_in_place_theta():
    w = np.random.default_rng(7).standard_normal(700001).astype(np.float32)
    dev = up([w])
    res = P.condensa_prune(dev, [0.25], in_place=True)
    torch.cuda.synchronize()
    check_prune_against_oracle(res, oracle.prune([w], [0.25], P.SCOPE_GLOBAL), P.SCOPE_GLOBAL, 1)


def test_special_values():
    """Infinities, NaN patterns, zeros and subnormals among ordinary weights, thresholds in every region."""
    rng = np.random.default_rng(8)
    w = rng.standard_normal(300000).astype(np.float32)
    w[:1000] = np.inf
    w[1000:2000] = -np.inf
    w[2000:2500] = np.nan
    w.view(np.uint32)[2500:3000] = 0xFFC12345
    w[3000:60000] = 0.0
    w[60000:120000] = -1e-42
    rng.shuffle(w)
    for ds in ([0.001], [0.005], [0.3], [0.7], [0.99], [0.001, 0.005, 0.3, 0.7, 0.99]):
        res = P.condensa_prune(up([w]), ds, theta_f16=True)
        torch.cuda.synchronize()
        check_prune_against_oracle(res, oracle.prune([w], ds, P.SCOPE_GLOBAL), P.SCOPE_GLOBAL, 1)


@pytest.mark.parametrize("case", ["tiny_among_large", "only_tiny", "many_ask_for_samples", "sixteen_densities", "density_ends"])
def test_sampling_workgroups(case):
    """Tensors too short to be sampled, PER_TENSOR populations that ask for more sampling workgroups than fit at once, the
    most rankings that one launch bounds, ranks at and beyond the ends of a sample."""
    rng = np.random.default_rng(11)
    scope, ds, shapes = P.SCOPE_GLOBAL, [0.1], [(3,), (700, 701), (1,), (2,), (5,), (90001,), (3, 1)]
    if case == "only_tiny":
        shapes = [(3,)] * 90
    elif case == "many_ask_for_samples":
        scope, shapes = P.SCOPE_PER_TENSOR, [(600, 451 + i) for i in range(16)] + [(2,), (40,)]
    elif case == "sixteen_densities":
        ds, shapes = [0.01 + 0.06 * j for j in range(16)], [(1300, 1001), (17,)]
    elif case == "density_ends":
        ds, shapes = [1e-6, 3e-4, 9e-4, 0.9992, 0.999999], [(1300, 1001)]
    arrs = [rng.standard_normal(s).astype(np.float32) for s in shapes]
    for d in ([ds] if len(ds) > 1 else [ds, [0.1, 0.6]]):
        res = P.condensa_prune(up(arrs), d, scope=scope)
        torch.cuda.synchronize()
        check_prune_against_oracle(res, oracle.prune(arrs, d, scope), scope, len(arrs), case)
    for d in ds if case == "density_ends" else ds[:1]:
        _check_lc(arrs, [rng.standard_normal(s).astype(np.float32) * np.float32(1e-4) for s in shapes], d)


@pytest.mark.parametrize("n", [131073, 262144, 300001, 4300007])
@pytest.mark.parametrize("ties", [0, 3, 60, 900, 2040, 2060, 9000])
def test_one_ranking_settled_by_the_launch_after_the_sweep(n, ties):
    """Bins of one entry and of as many as that launch ranks by itself, fewer and more; ties at the threshold that are cut in the
    middle, alone in their bin or among others."""
    rng = np.random.default_rng(n + ties)
    w = rng.standard_normal(n).astype(np.float32)
    order = np.argsort(-np.abs(w), kind="stable")
    k = n // 7
    w[order[k - ties // 2:k + (ties + 1) // 2]] = np.abs(w[order[k]])      # the values next to the threshold become equal
    lam = (rng.standard_normal(n) * 1e-7).astype(np.float32)
    for d in (k / n, (k - 1) / n, (k + ties // 3) / n):
        res = P.condensa_prune(up([w]), [d], theta_f16=True)
        torch.cuda.synchronize()
        check_prune_against_oracle(res, oracle.prune([w], [d], P.SCOPE_GLOBAL), P.SCOPE_GLOBAL, 1, str((n, ties)))
    _check_lc([w], [np.zeros_like(lam)], k / n, pq=True)
    _check_lc([w], [lam], k / n, pq=ties % 2 == 0)


@pytest.mark.parametrize("n", [140001, 1 << 20])               # 35 segments of the list: more of the bin's entries than a wavefront holds, and 257
@pytest.mark.parametrize("ties", [1900, 2049, 4000, 4097])     # the room for the entries of the threshold's bin: 4096
def test_threshold_bins_about_as_large_as_their_room(n, ties):
    rng = np.random.default_rng(ties)
    w = rng.standard_normal(n).astype(np.float32)
    w[rng.choice(n, ties, replace=False)] = np.float32(-1.25)
    above = int((np.abs(w) > 1.25).sum())
    for k in (above + 5, above + ties // 2):                   # at the first of the ties the list holds as many other elements
        res = P.condensa_prune(up([w]), [k / n], theta_f16=True)
        torch.cuda.synchronize()
        check_prune_against_oracle(res, oracle.prune([w], [k / n], P.SCOPE_GLOBAL), P.SCOPE_GLOBAL, 1, f"n={n} ties={ties} k={k}")


def test_a_population_whose_samplers_take_several_units():
    w = np.random.default_rng(26).standard_normal((1 << 26) + 4099).astype(np.float32)
    res = P.condensa_prune(up([w]), [0.6])
    torch.cuda.synchronize()
    check_prune_against_oracle(res, oracle.prune([w], [0.6], P.SCOPE_GLOBAL), P.SCOPE_GLOBAL, 1)


def test_sampling_workgroups_with_an_empty_sample():
    """A tensor among so many tensors too short to be sampled that only some of the 32 sampling workgroups meet it: the window is
    that of these alone, and its list (half of the population) holds it."""
    rng = np.random.default_rng(27)
    n_tiny = 8000                                            # 25 of 32 stretches of the population hold weights that are sampled
    tiny = rng.standard_normal((n_tiny, 4)).astype(np.float32)
    big = rng.standard_normal(200003).astype(np.float32)
    arrs = [big] + [t[:3] for t in tiny]
    dev = up([tiny])[0]
    config = {"cand_shift": 1, "window_margin": 16}
    res = P.condensa_prune(up([big]) + [dev[i, :3] for i in range(n_tiny)], [0.5], config=config)
    torch.cuda.synchronize()
    want = oracle.prune(arrs, [0.5], P.SCOPE_GLOBAL)
    rec = P.select_records(res["results"])[0]
    assert_select_equal(rec, want[0]["select"])
    assert rec["path"] == 2, "the window was opened by workgroups that sampled nothing"
    for t in range(0, len(arrs), 97):
        assert np.array_equal(res["mask"][0][t].cpu().numpy(), want[0]["mask"][t])


@pytest.mark.parametrize("n", [150001, 700001, (1 << 20) + 3, (1 << 22) + 1, (1 << 23) + 5])        # 32, 64 and 256 sampling workgroups
@pytest.mark.parametrize("kind", ["apart", "few_apart", "near_the_compressed"])
def test_windows_at_a_gap(n, kind):
    """Thresholds at the edge of a gap between the kept weights and the others, as a model has that is close to its compressed
    form: the window still holds them, though the mean of the samples' keys lies where no weights are."""
    rng = np.random.default_rng(n)
    kept = rng.random(n) < (0.1 if kind != "few_apart" else 0.003)
    if kind == "near_the_compressed":
        w = rng.standard_normal(n).astype(np.float32) * np.float32(0.02)
        kept = np.abs(w) > 0.0329
        w = np.where(kept, w, 0) + rng.standard_normal(n) * 2e-4
    else:
        w = np.where(kept, 0.05 + 0.05 * rng.random(n), 2e-4 * rng.random(n)) * rng.choice([-1.0, 1.0], n)
    w = w.astype(np.float32)
    share = int(kept.sum()) / n
    for ds in ([share], [share + 0.004], [share, 0.3, 0.5]):
        res = P.condensa_prune(up([w]), ds)
        torch.cuda.synchronize()
        check_prune_against_oracle(res, oracle.prune([w], ds, P.SCOPE_GLOBAL), P.SCOPE_GLOBAL, 1, f"{n} {kind} {ds}")
        assert [r["path"] for r in P.select_records(res["results"])] == [2] * len(ds), (n, kind, ds)
    _check_lc([w], [np.zeros_like(w)], share, pq=True)


@pytest.mark.parametrize("distinct", [2, 40, 3000, 1 << 20])
@pytest.mark.parametrize("n", [100001, 262149, 3000001])       # one workgroup a ranking; all rankings together
def test_threshold_bins_of_many_entries(n, distinct):
    """Tens of thousands of keys in a small part of the threshold's bin, with few and with many values among them: the levels that
    rank them end at comparable pairs, at one value, and at the first and last of them."""
    rng = np.random.default_rng(n + distinct)
    w = rng.standard_normal(n).astype(np.float32)
    m = n // 6
    near = np.float32(1.5).view(np.uint32) + rng.integers(0, distinct, m).astype(np.uint32)
    at = rng.choice(n, m, replace=False)
    w[at] = near.view(np.float32) * rng.choice([-1.0, 1.0], m).astype(np.float32)
    above = int((np.abs(w) >= 1.5).sum()) - int(((np.abs(w) >= 1.5) & (np.abs(w).view(np.uint32) < np.float32(1.5).view(np.uint32) + distinct)).sum())
    ks = [above + 1, above + m // 3, above + m - 1]
    for ds in ([k / n for k in ks[:1]], [k / n for k in ks[1:2]], [k / n for k in ks]):
        res = P.condensa_prune(up([w]), ds, theta_f16=True)
        torch.cuda.synchronize()
        check_prune_against_oracle(res, oracle.prune([w], ds, P.SCOPE_GLOBAL), P.SCOPE_GLOBAL, 1, f"{n} {distinct} {ds}")
    _check_lc([w], [np.zeros_like(w)], ks[1] / n, pq=True)
    arrs = [w, w[: n // 2].copy(), w[n // 3:].copy()]
    res = P.condensa_prune(up(arrs), [ks[1] / n], scope=P.SCOPE_PER_TENSOR)
    torch.cuda.synchronize()
    check_prune_against_oracle(res, oracle.prune(arrs, [ks[1] / n], P.SCOPE_PER_TENSOR), P.SCOPE_PER_TENSOR, 3, f"{n} {distinct}")


@pytest.mark.parametrize("ds", [[0.1], [0.02, 0.3]], ids=["one", "two"])
def test_populations_with_fewer_sampling_workgroups_than_they_ask_for(ds):
    """PER_TENSOR populations of every size class whose workgroups are cut to a quarter, or to 32, with rows of very different
    sizes: their lists still hold the windows."""
    rng = np.random.default_rng(31)
    shapes = [(3000, 3001)] + [(4608, 500 + 7 * i) for i in range(3)] + [(600, 451 + i) for i in range(12)] + [(9, 50)]
    arrs = [rng.standard_normal(s).astype(np.float32) * np.exp(rng.standard_normal((s[0], 1))).astype(np.float32) for s in shapes]
    res = P.condensa_prune(up(arrs), ds, scope=P.SCOPE_PER_TENSOR, theta=False)
    torch.cuda.synchronize()
    check_prune_against_oracle(res, oracle.prune(arrs, ds, P.SCOPE_PER_TENSOR), P.SCOPE_PER_TENSOR, len(arrs))
    paths = [r["path"] for r in P.select_records(res["results"])]
    for j in range(len(ds)):
        assert paths[j * len(arrs):j * len(arrs) + 4] == [2] * 4, paths


# A wavefront of the sweep over several densities buffers 256 listed entries of its 1024 elements: runs of them with fewer, as many, one more and
# all listed, for disjoint windows (masks alone, all outputs, an unaligned tensor) and overlapping ones
@pytest.mark.parametrize("listed", [255, 256, 257, 1024])
@pytest.mark.parametrize("ds", [[0.1, 0.4], [0.5, 0.02, 0.1, 0.3], [0.1, 0.1002, 0.4]], ids=str)
def test_wavefronts_with_many_listed_entries(listed, ds):
    n, per = 3 << 20, 1024
    rng = np.random.default_rng(listed)
    w = rng.standard_normal(n).astype(np.float32)
    marks = np.sort(np.abs(w))[::-1]
    T = np.array([marks[int(d * n)] for d in ds], np.float32)
    for run in range(0, n // per, 97):
        at = np.zeros(per, np.float32)
        near = T[np.arange(listed) % T.size].view(np.int32) + rng.permutation(listed).astype(np.int32) * 3 - listed         # distinct, a few hundred steps off
        at[rng.permutation(per)[:listed]] = near.view(np.float32) * rng.choice(np.array([-1, 1], np.float32), listed)
        w[run * per:(run + 1) * per] = at
    ora = oracle.prune([w], ds, P.SCOPE_GLOBAL)
    for all_outputs in (False, True):
        res = P.condensa_prune(up([w]), ds, theta=all_outputs, theta_f16=all_outputs)
        torch.cuda.synchronize()
        check_prune_against_oracle(res, ora, P.SCOPE_GLOBAL, 1, f"{listed} {all_outputs}")
    buf = torch.zeros(n + 1, dtype=torch.float32, device=DEV)
    buf[1:].copy_(torch.from_numpy(w))
    res = P.condensa_prune([buf[1:]], ds)
    torch.cuda.synchronize()
    check_prune_against_oracle(res, ora, P.SCOPE_GLOBAL, 1, f"{listed} not aligned")
