"""GPU parity of filter and neuron pruning whose aggregates are summed in the launch that begins the call (up to 80 tensors, up to 16 384 rows of up to 8 192):
both sides of each limit, tensors without weights and with fewer than four, a used workspace, both scopes; against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_1911_02497_amd as P
from gpu_util import up, with_form
from test_gpu_structure import _compare

pytestmark = pytest.mark.gpu

neuron_prune = with_form(P.condensa_neuron_prune, fill_keep_idx=True)


def _check(ts, density, scope, what):
    want = oracle.neuron_prune(ts, density, scope)
    dev = up(ts)
    for again in range(2):
        _compare(neuron_prune(dev, density, scope), want, scope, ts, f"{what} density={density} scope={scope} call {again}")


@pytest.mark.parametrize("scope", [P.SCOPE_GLOBAL, P.SCOPE_PER_TENSOR])
@pytest.mark.parametrize("n_tensors", [1, 2, 79, 80, 81])
def test_number_of_tensors(n_tensors, scope):
    rng = np.random.default_rng(n_tensors)
    ts = [(rng.standard_normal((1 + (5 * i) % 41, 17 + (11 * i) % 67)) * 0.1).astype(np.float32) for i in range(n_tensors)]
    if n_tensors > 2:
        ts[0] = np.zeros((0, 40), np.float32)              # no rows, at the start, within and at the end; then fewer than four weights
        ts[n_tensors // 2] = np.zeros((0, 3), np.float32)
        ts[-1] = np.zeros((0, 9), np.float32)
        ts[1] = np.array([[0.25, -3.0, 1e-42]], np.float32)
        ts[5] = np.array([[-7.0], [0.0]], np.float32)
    for density in (0.0, 0.3, 1.0):
        _check(ts, density, scope, f"{n_tensors} tensors")


@pytest.mark.parametrize("rows", [16383, 16384, 16385])             # 512 workgroups of 32 rows
@pytest.mark.parametrize("length", [8191, 8192, 8193])    # the longest row
def test_number_and_length_of_rows(rows, length):
    rng = np.random.default_rng(rows)
    ts = [rng.standard_normal((n, d)).astype(np.float32) for n, d in ((rows - 133, 33), (1, length), (132, 16))]
    ts[0][::7] = ts[0][3]                                   # equal rows
    for scope in (P.SCOPE_GLOBAL, P.SCOPE_PER_TENSOR):
        _check(ts, 0.37, scope, f"{rows} rows {length}")


def test_graph_and_stream():
    rng = np.random.default_rng(3)
    ts = [rng.standard_normal((60 + i, 27 * (1 + i % 4))).astype(np.float32) for i in range(12)]
    want = oracle.neuron_prune(ts, 0.4, P.SCOPE_GLOBAL)
    dev = up(ts)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        on_side = neuron_prune(dev, 0.4, P.SCOPE_GLOBAL)
    side.synchronize()
    _compare(on_side, want, P.SCOPE_GLOBAL, ts, "another stream")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        captured = neuron_prune(dev, 0.4, P.SCOPE_GLOBAL)
    for i in range(3):
        graph.replay()
        torch.cuda.synchronize()
        _compare(captured, want, P.SCOPE_GLOBAL, ts, f"replay {i}")
        _check(ts, 0.4, P.SCOPE_GLOBAL, "between replays")
