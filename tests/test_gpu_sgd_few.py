"""GPU parity of the learning-step update at the number of tensors where its tables change their route, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_1911_02497_amd as P
from gpu_util import assert_bits_equal, up

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shift", [0, 1])                 # 1: views one element into their buffers, no 128-bit accesses
@pytest.mark.parametrize("n_tensors", [1, 2, 63, 64, 65])
def test_sgd_step_of_n_tensors(n_tensors, shift):
    rng = np.random.default_rng(n_tensors)
    sizes = [(0, 1, 255, 256, 257, 8191, 8192, 8193, 20011)[(i + n_tensors) % 9] for i in range(n_tensors)]
    mk = lambda s: [(rng.standard_normal(n + shift) * s).astype(np.float32) for n in sizes]  # noqa: E731
    ws, gs, ths, ls, bs = mk(0.01), mk(1e-3), mk(0.01), mk(0.01), mk(1e-3)
    cut = lambda arrs: [a[shift:] for a in arrs]  # noqa: E731
    dev = [up(x) for x in (ws, gs, ths, ls, bs)]
    w, g, th, lam, b = [[t[shift:] for t in x] for x in dev]
    P.condensa_lc_sgd_step(w, g, th, lam, b, 1e-3, 0.1, 0.9)
    torch.cuda.synchronize()
    w_ora, b_ora = oracle.lc_sgd_step(cut(ws), cut(gs), cut(ths), cut(ls), cut(bs), 1e-3, 0.1, 0.9)
    for t in range(n_tensors):
        assert_bits_equal(w[t], w_ora[t], f"w {t}")
        assert_bits_equal(b[t], b_ora[t], f"buf {t}")


def test_pointer_tables_of_empty_views_and_missing_tensors():
    x = torch.arange(10, dtype=torch.float32, device="cuda")
    arr, p = P.binding._ptr_table([x, None, x[3:3], x[2:]])
    assert list(arr) == [x.data_ptr(), 0, 0, x.data_ptr() + 8] and p.value == arr.buffer_info()[0]
    assert P.binding._ptr_table(None) == (None, None) and P.binding._ptr_table([])[1].value
