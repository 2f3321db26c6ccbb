"""GPU parity at the edges of the rankings of structures: one workgroup over the aggregates, one over a list of them, the rows'
staged sums and the tiles of the kept-id list, against the oracle (bit exact)."""
import numpy as np
import pytest

import oracle
import paper_1911_02497_amd as P
from gpu_util import up, with_form
from test_gpu_structure import _compare

pytestmark = pytest.mark.gpu

block_prune = with_form(P.condensa_block_prune, fill_keep_idx=True)
neuron_prune = with_form(P.condensa_neuron_prune, fill_keep_idx=True)


def _values(kind, n, seed):
    rng = np.random.default_rng(seed)
    if kind == "distinct":
        return rng.lognormal(0.0, 1.5, n).astype(np.float32)
    if kind == "equal":
        return np.full(n, 0.75, np.float32)
    if kind == "few":          # ties in every bin
        return rng.choice(np.array([0.0, 0.5, 0.5000001, 3.0], np.float32), n)
    v = rng.standard_normal(n).astype(np.float32)       # special
    v[:: max(n // 7, 1)] = 0.0
    v[1:: max(n // 5, 1)] = np.inf
    v[2:: max(n // 3, 1)] = 1e-42
    return v


def _neurons(values, length):
    """Rows whose aggregate is the square of a given value: the value once, zeros, and both signs of zero."""
    w = np.zeros((values.size, length), np.float32)
    w[np.arange(values.size), np.arange(values.size) % length] = values
    w[::2] *= -1.0
    return w


@pytest.mark.parametrize("kind", ["distinct", "equal", "few", "special"])
@pytest.mark.parametrize("n", [1, 2, 64, 255, 256, 257, 1023, 1025, 4095, 4096, 4097, 9001, 66000])
def test_one_ranking_of_n_rows(n, kind):
    w = _neurons(_values(kind, n, n), 3)
    dev = up([w])
    for d in (0.0, 1.0 / n, 0.013, 0.5, 1.0 - 1.0 / n, 1.0):
        _compare(neuron_prune(dev, d, P.SCOPE_GLOBAL), oracle.neuron_prune([w], d, P.SCOPE_GLOBAL), P.SCOPE_GLOBAL, [w], f"n={n} {kind} d={d}")


@pytest.mark.parametrize("length", [1, 3, 15, 16, 17, 31, 255, 256, 257, 511, 512, 513, 528, 769, 1025])
def test_sums_of_few_rows_of_some_length(length):
    rng = np.random.default_rng(length)
    ts = [rng.standard_normal((r, max(length - c, 1))).astype(np.float32) for r, c in ((33, 0), (1, 1), (64, 0), (31, 2))]
    ts[0][::5, :1] = np.inf
    ts[2][::3] *= 1e-30
    for scope in (P.SCOPE_GLOBAL, P.SCOPE_PER_TENSOR):
        _compare(neuron_prune(up(ts), 0.4, scope), oracle.neuron_prune(ts, 0.4, scope), scope, ts, f"length={length} scope={scope}")


def test_rows_of_more_tensors_than_the_search_holds():
    rng = np.random.default_rng(5)
    ts = [rng.standard_normal((1 + i % 3, 16 + i % 5)).astype(np.float32) for i in range(600)]
    _compare(neuron_prune(up(ts), 0.3, P.SCOPE_GLOBAL), oracle.neuron_prune(ts, 0.3, P.SCOPE_GLOBAL), P.SCOPE_GLOBAL, ts, "600 tensors")


# 1024 blocks a row of blocks: 2048 tiles of kept ids and more; without strips, which have no tiles, and with them
@pytest.mark.parametrize("config", [{"fused_sweep": 1}, None])
@pytest.mark.parametrize("rows", [1023, 1025, 2048, 2051])
def test_kept_ids_of_many_tiles(rows, config):
    rng = np.random.default_rng(rows)
    w = rng.choice(np.array([0.25, 0.5, 1.0], np.float32), (rows, 2048)) * rng.standard_normal((rows, 2048)).astype(np.float32)
    _compare(block_prune(up([w]), 1, 2, 0.31, P.SCOPE_GLOBAL, config=config), oracle.block_prune([w], 1, 2, 0.31, P.SCOPE_GLOBAL), P.SCOPE_GLOBAL, [w], f"rows={rows}")


@pytest.mark.parametrize("zeros", [0.5, 0.9, 0.999, 1.0])
def test_ranking_of_rows_pruned_before(zeros):
    n = 20000
    rng = np.random.default_rng(17)
    v = rng.lognormal(0.0, 0.2, n).astype(np.float32)
    v[rng.random(n) < zeros] = 0.0
    if zeros < 1.0:
        v[::1999] = 1e-18          # far below what a sample of the others shows
    w = _neurons(v, 3)
    kept = float(np.count_nonzero(v)) / n
    for d in (0.8 * kept, kept - 2.0 / n, kept, kept + 3.0 / n, 0.5 + 0.5 * kept):
        d = min(max(d, 0.0), 1.0)
        _compare(neuron_prune(up([w]), d, P.SCOPE_GLOBAL), oracle.neuron_prune([w], d, P.SCOPE_GLOBAL), P.SCOPE_GLOBAL, [w], f"zeros={zeros} d={d}")


@pytest.mark.parametrize("rows", [16384, 16385, 32768, 32769])      # where the staged sums of rows change their form
def test_sums_of_many_rows(rows):
    rng = np.random.default_rng(rows)
    w = rng.standard_normal((rows, 277)).astype(np.float32)
    _compare(neuron_prune(up([w]), 0.2, P.SCOPE_GLOBAL), oracle.neuron_prune([w], 0.2, P.SCOPE_GLOBAL), P.SCOPE_GLOBAL, [w], f"rows={rows}")


@pytest.mark.parametrize("shapes", [
    ((33, 40), (1, 1), (1, 2), (3, 1), (1, 3), (40, 64)),               # tensors of fewer than four elements
    ((32769, 36), (7, 64), (300, 20)),                                  # aligned, several lengths in a workgroup, the last one ragged
    ((33001, 19), (65, 17), (5, 131), (1, 18)),                         # not aligned, the last rows end within four elements of their tensor
    ((70001, 17), (300, 33), (1, 130)),                                 # rows of one piece, 256 to a workgroup
    ((65400, 64), (41, 33), (7, 131), (95, 2)),                         # few that are not aligned among many, in workgroups of both
    ((65537, 36), (3, 5001)),                                           # ... and long ones
])
def test_sums_of_rows_of_several_tensors(shapes):
    rng = np.random.default_rng(len(shapes))
    ts = [rng.standard_normal(s).astype(np.float32) for s in shapes]
    _compare(neuron_prune(up(ts), 0.4, P.SCOPE_GLOBAL), oracle.neuron_prune(ts, 0.4, P.SCOPE_GLOBAL), P.SCOPE_GLOBAL, ts, f"{shapes}")
