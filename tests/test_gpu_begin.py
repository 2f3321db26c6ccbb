"""GPU parity of what every call starts with: tables of one launch and of two (more than 256 tensors, or tables beyond
one staging slot), more calls in flight than there are staging slots, from several threads and streams, behind a stream
that is busy for long, and after calls that failed once their first kernel was queued."""
import threading

import numpy as np
import pytest
import torch

import oracle
import paper_1911_02497_amd as P
from gpu_util import DEV, check_prune_against_oracle, up

pytestmark = pytest.mark.gpu


def _model(n_tensors, seed):
    rng = np.random.default_rng(seed)
    return [rng.standard_normal(int(rng.integers(1, 40)) if t % 7 else 8193).astype(np.float32) for t in range(n_tensors)]


@pytest.mark.parametrize("n_tensors", [1, 255, 256, 257, 700])
@pytest.mark.parametrize("densities", [[0.3], [0.05, 0.3, 0.9] * 5])
def test_tables_of_every_size(n_tensors, densities):
    arrs = _model(n_tensors, n_tensors)
    res = P.condensa_prune(up(arrs), densities)
    torch.cuda.synchronize()
    check_prune_against_oracle(res, oracle.prune(arrs, densities, P.SCOPE_GLOBAL), P.SCOPE_GLOBAL, n_tensors)


@pytest.mark.parametrize("n_tensors", [96, 97])
@pytest.mark.parametrize("scope", [P.SCOPE_GLOBAL, P.SCOPE_PER_TENSOR])
def test_the_sample_in_the_first_launch_and_in_one_of_its_own(n_tensors, scope):
    arrs = _model(n_tensors, n_tensors)
    res = P.condensa_prune(up(arrs), [0.3], scope=scope)
    torch.cuda.synchronize()
    check_prune_against_oracle(res, oracle.prune(arrs, [0.3], scope), scope, n_tensors)


def test_more_calls_in_flight_than_staging_slots():
    """Every call has its own table (and so its own image); none may be replaced before the device has read it."""
    models = [_model(3, 100 + i) for i in range(100)]
    dev = [up(m) for m in models]
    torch.cuda.synchronize()
    busy = torch.randn(4096, 4096, device=DEV)
    for _ in range(20):
        busy = busy @ busy * 1e-3                            # keeps the stream occupied while the calls are queued
    out = [P.condensa_prune(d, [0.25]) for d in dev]
    torch.cuda.synchronize()
    for m, r in zip(models, out):
        check_prune_against_oracle(r, oracle.prune(m, [0.25], P.SCOPE_GLOBAL), P.SCOPE_GLOBAL, 3)


def test_threads_and_streams_share_the_slots():
    models = [_model(5, 300 + i) for i in range(4)]
    want = [oracle.prune(m, [0.4], P.SCOPE_GLOBAL) for m in models]
    got = [[] for _ in models]

    def work(i):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            d = up(models[i])
            for _ in range(30):
                got[i].append(P.condensa_prune(d, [0.4]))
            s.synchronize()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(models))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for m, w, rs in zip(models, want, got):
        for r in rs:
            check_prune_against_oracle(r, w, P.SCOPE_GLOBAL, 5)


@pytest.mark.parametrize("n_tensors", [3, 700])
def test_a_busy_stream_holds_no_call_back_for_good(n_tensors):
    models = [_model(n_tensors, 500 + i) for i in range(3)]
    dev = [up(m) for m in models]
    torch.cuda.synchronize()
    torch.cuda._sleep(600_000_000)                           # some tenths of a second, longer than a call waits for a slot
    out = [P.condensa_prune(dev[i % 3], [0.25]) for i in range(40)]
    torch.cuda.synchronize()
    for i in (0, 1, 2, 37, 38, 39):
        check_prune_against_oracle(out[i], oracle.prune(models[i % 3], [0.25], P.SCOPE_GLOBAL), P.SCOPE_GLOBAL, n_tensors)


def test_calls_that_fail_after_their_launch_give_their_slots_back():
    """An error that the thread left behind (here: a device number that does not exist) is reported by the call's first launch
    check, after the kernel that reads the slot was queued.  More of these than there are slots, then ordinary calls."""
    m = _model(3, 7)
    d = up(m)
    res = P.condensa_prune(d, [0.25])
    again = lambda: P.condensa_prune(d, [0.25], outputs=res, workspace=res["workspace"])  # noqa: E731  (no launch but the library's)
    failed = 0
    for _ in range(40):
        P.library().hipSetDevice(9999)
        try:
            again()
        except P.CondensaError:
            failed += 1
    torch.cuda.synchronize()
    res["mask"][0][0].zero_()
    for _ in range(40):
        again()
    torch.cuda.synchronize()
    check_prune_against_oracle(res, oracle.prune(m, [0.25], P.SCOPE_GLOBAL), P.SCOPE_GLOBAL, 3, f"{failed} calls failed")
