"""GPU parity of the listed windows where a wavefront finds more entries than it can buffer, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_1911_02497_amd as P
from gpu_util import check_prune_against_oracle, up

pytestmark = pytest.mark.gpu


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
