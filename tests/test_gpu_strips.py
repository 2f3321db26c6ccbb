"""GPU parity of block pruning in strips (2-D blocks of up to 256 elements, 4097 to 2^24 of them, GLOBAL scope): the edges of strips, clipped blocks,
every alignment, windows that miss and bins that overflow; against the oracle, bit for bit."""
import contextlib

import numpy as np
import pytest
import torch

import oracle
import paper_1911_02497_amd as P
from gpu_util import DEV, up
from paper_1911_02497_amd.binding import OP_BLOCK_PRUNE
from test_gpu_structure import _compare

pytestmark = pytest.mark.gpu

LATE, NO_SAMPLE = 1, 2                                     # csrc/host.h


@contextlib.contextmanager
def forced(what):
    lib = P.library()
    lib.condensa_test_force(what)
    try:
        yield
    finally:
        lib.condensa_test_force(0)


def _check(arrs, block, density, what, dev=None, config=None, **kw):
    res = P.condensa_block_prune_nd(dev if dev is not None else up(arrs), block, density, P.SCOPE_GLOBAL, fill_keep_idx=True, config=config, **kw)
    torch.cuda.synchronize()
    _compare(res, oracle.block_prune_nd(arrs, block, density, P.SCOPE_GLOBAL), P.SCOPE_GLOBAL, arrs, what)
    return res


def _normal(shapes, seed):
    rng = np.random.default_rng(seed)
    return [(rng.standard_normal(s) * 0.02).astype(np.float32) for s in shapes]


# strips of one and several rows of blocks, pieces of a row, clipped blocks at both edges, rows of all remainders of four, narrow matrices
@pytest.mark.parametrize("block,shapes", [
    ((8, 8), [(512, 1024), (0, 8), (264, 520), (8, 8), (1024, 24)]),
    ((8, 8), [(515, 1028), (3, 4), (1200, 36)]),
    ((4, 4), [(300, 1604), (64, 4), (1000, 40)]),
    ((16, 16), [(1024, 1040), (720, 1000), (4096, 16)]),
    ((64, 4), [(700, 4096), (1111, 100)]),
    ((2, 64), [(301, 4096), (9001, 60)]),
    ((5, 5), [(650, 650), (1, 1), (2, 3), (333, 331), (700, 3)]),
    ((3, 7), [(200, 4099), (41, 6), (2000, 21)]),
    ((1, 3), [(128, 514), (5000, 2), (90, 1025)]),
    ((16, 16), [(1023, 1501), (50, 5), (3000, 17)]),
    ((256, 1), [(700, 2050), (3, 301)]),
    ((6, 6), [(602, 901), (601, 902), (600, 900)]),
])
@pytest.mark.parametrize("density", [0.03, 0.4, 0.9])
def test_strips(block, shapes, density):
    arrs = _normal(shapes, sum(block))
    arrs[0][:16, :16] = arrs[0][16:32, 16:32]              # equal blocks
    dev = up(arrs)
    before = P.condensa_launch_count()
    _check(arrs, block, density, f"{block} {density}", dev=dev)
    assert P.condensa_launch_count() - before == 3         # strips it was


def _same_as_radix(dev, block, density, launches):
    ref = P.condensa_block_prune_nd(dev, block, density, P.SCOPE_GLOBAL, fill_keep_idx=True, config={"select_path": 1})
    before = P.condensa_launch_count()
    res = P.condensa_block_prune_nd(dev, block, density, P.SCOPE_GLOBAL, fill_keep_idx=True)
    took = P.condensa_launch_count() - before
    assert took == 3 if launches == 3 else took > 3, took
    want, got = [P.select_records(r["results"])[0] for r in (ref, res)]
    assert all(got[f] == want[f] for f in ("n", "k", "n_gt", "n_tie_kept", "n_tie", "threshold_key", "tie_end")), (got, want)
    as_bits = {torch.float32: torch.int32, torch.float64: torch.int64}
    for name in ("theta", "mask", "sumsq", "norms", "keep_idx", "structure_mask"):
        for a, b in zip(*[(r[name] if isinstance(r[name], list) else [r[name]]) for r in (res, ref)]):
            assert torch.equal(a.view(as_bits.get(a.dtype, a.dtype)), b.view(as_bits.get(b.dtype, b.dtype))), name


# a whole number of strips short of 2^14 (the counts are added up by 64 below, by 512 from there on) and 2^22 blocks (a second round of draws), both, more; then
# bins with all their places, up to the 2^24 blocks that strips take at most, and one row of them more
@pytest.mark.parametrize("block,shape,launches", [
    ((4, 4), (4 * 2047, 4 * 2048), 3), ((4, 4), (4 * 2048, 4 * 2048), 3), ((4, 4), (4 * 2050 - 1, 4 * 2052), 3), ((3, 5), (3 * 2500, 5 * 2111 - 2), 3),
    ((2, 2), (8192, 8192), 3), ((2, 2), (8194, 8192), 4), ((1, 3), (5000, 3 * 3355 - 1), 3)])
def test_sizes_where_the_plan_changes(block, shape, launches):
    g = torch.Generator(device=DEV).manual_seed(shape[0])
    w = torch.empty(shape, dtype=torch.float32, device=DEV).normal_(0.0, 0.02, generator=g)
    for density in (0.3, 0.004):
        _same_as_radix([w], block, density, launches)
    w.mul_(2048).round_()                                  # many equal aggregates: bins overflow
    _same_as_radix([w], block, 0.3, launches)


@pytest.mark.parametrize("block", [(4, 4), (5, 5)])
def test_values_that_are_not_numbers(block):
    g = torch.Generator(device=DEV).manual_seed(9)
    w = torch.empty((1000, 1200), dtype=torch.float32, device=DEV).normal_(0.0, 0.02, generator=g)
    w[::23, ::7] = float("nan")
    w[5::31, ::5] = float("-inf")
    for density in (0.01, 0.2, 0.5, 0.95):
        _same_as_radix([w], block, density, 3)


@pytest.mark.parametrize("scale", [1e-24, 1e-20, 1e17, 1e21])          # squares that leave binary32, in which samples are summed
@pytest.mark.parametrize("block,shape", [((8, 8), (1024, 1032)), ((5, 5), (651, 650))])
def test_scales_beyond_the_sample(block, shape, scale):
    (a,) = _normal([shape], 8)
    for density in (0.05, 0.5):
        _check([a * np.float32(scale)], block, density, f"{scale} {density}")


def test_any_alignment_and_missing_outputs():
    (a,) = _normal([(600, 1024)], 1)
    for off in (0, 1, 2, 3):
        buf = torch.zeros(a.size + 4, dtype=torch.float32, device=DEV)
        w = buf[off:off + a.size].view(a.shape)
        w.copy_(torch.from_numpy(a))
        _check([a], (8, 8), 0.3, f"offset {off}", dev=[w])
    want = oracle.block_prune(([a]), 8, 8, 0.3, P.SCOPE_GLOBAL)
    for theta, mask in ((True, False), (False, True)):
        res = P.condensa_block_prune(up([a]), 8, 8, 0.3, theta=theta, mask=mask)
        if theta:
            assert np.array_equal(res["theta"][0].cpu().numpy().view(np.uint32), want["theta"][0].view(np.uint32))
        if mask:
            assert np.array_equal(res["mask"][0].cpu().numpy(), want["mask"][0])


@pytest.mark.parametrize("kind", ["zeros", "grid", "gap", "constant", "infinite"])
@pytest.mark.parametrize("block", [(4, 4), (5, 5)])
def test_many_equal_aggregates_and_gaps(kind, block):
    rng = np.random.default_rng(5)
    n = 200
    w = rng.standard_normal((n * block[0], n * block[1])).astype(np.float32)
    pick = np.kron(rng.random((n, n)) < 0.7, np.ones(block, bool))
    if kind == "zeros":
        w[pick] = np.float32(-0.0)
    elif kind == "grid":
        w = np.where(pick, np.float32(0.5), np.round(w)).astype(np.float32)
    elif kind == "gap":
        w[pick] *= np.float32(1e-3)
    elif kind == "constant":
        w[:] = 0.25
    else:
        w[::block[0] * 3, ::block[1]] = np.inf
    for d in (0.1, 0.3, 0.31, 0.5, 0.9):
        _check([w], block, d, f"{kind} {d}")


# the fallback: a threshold at a gap, in a bin that it gathers or beyond; ties there that end inside one of the workgroups' shares
@pytest.mark.parametrize("copies", [0, 60, 255, 700])
@pytest.mark.parametrize("block,n", [((4, 4), 200), ((5, 5), 180), ((2, 2), 400)])
def test_ties_at_a_gap(block, n, copies):
    rng = np.random.default_rng(copies)
    big = rng.random(n * n) < 0.5
    w = rng.standard_normal((n * block[0], n * block[1])).astype(np.float32) * np.where(np.kron(big.reshape(n, n), np.ones(block, bool)), np.float32(1), np.float32(1e-2))
    k = int(big.sum())
    blocks = w.reshape(n, block[0], n, block[1]).transpose(0, 2, 1, 3).reshape(n * n, -1)
    order = np.argsort(-(blocks.astype(np.float64) ** 2).sum(1))
    same = rng.choice(order[k - 900:k], copies, replace=False)
    blocks[same] = blocks[order[k - 1]]
    w = np.ascontiguousarray(blocks.reshape(n, n, *block).transpose(0, 2, 1, 3).reshape(w.shape))
    for at in (k - copies - 1, k - copies // 2, k - 1, k, k + 1):
        _check([w], block, (at + 0.25) / (n * n), f"{copies} {at}")
        with forced(LATE):
            _check([w], block, (at + 0.25) / (n * n), f"{copies} {at}, late")


@pytest.mark.parametrize("block,shapes", [((8, 8), [(512, 1024), (264, 520)]), ((5, 5), [(650, 651), (333, 331)])])
def test_windows_that_miss(block, shapes):
    arrs = _normal(shapes, 3)
    for d in (0.05, 0.5, 0.93):
        _check(arrs, block, d, f"no margin {d}", config={"window_margin": 0})
        for what in (LATE, NO_SAMPLE, LATE | NO_SAMPLE):
            with forced(what):
                _check(arrs, block, d, f"forced {what} {d}")


def test_more_tensors_than_one_launch_begins_and_capture():
    arrs = _normal([(40 + i % 7, 60 + i % 5) for i in range(120)], 4)
    dev = up(arrs)
    res = _check(arrs, (4, 4), 0.35, "120 tensors", dev=dev)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        P.condensa_block_prune_nd(dev, (4, 4), 0.35, outputs=res, workspace=res["workspace"])
    for seed in (7, 8, 9):
        new = _normal([a.shape for a in arrs], seed)
        for d, a in zip(dev, new):
            d.copy_(torch.from_numpy(a))
        P.condensa_block_prune(up(_normal([(64, 64)], 1)), 8, 8, 0.5)
        res["keep_idx"].fill_(-1)
        graph.replay()
        torch.cuda.synchronize()
        _compare(res, oracle.block_prune_nd(new, (4, 4), 0.35, P.SCOPE_GLOBAL), P.SCOPE_GLOBAL, new, f"replay {seed}")


def test_workspace_without_room_for_strips():
    arrs = _normal([(512, 1024), (264, 520)], 6)
    n, f = sum(a.size for a in arrs), 64 * 128 + 33 * 65
    short, full = [P.condensa_workspace_bytes(OP_BLOCK_PRUNE, n, f, 2, 1, P.SCOPE_GLOBAL, config=c) for c in ({"select_path": 1}, None)]
    assert short < full
    for size in (short, full - 256, full):
        _check(arrs, (8, 8), 0.3, f"{size} bytes", workspace=torch.empty(size, dtype=torch.uint8, device=DEV))
    with pytest.raises(P.CondensaError):
        P.condensa_block_prune_nd(up(arrs), (8, 8), 0.3, P.SCOPE_GLOBAL, workspace=torch.empty(short - 256, dtype=torch.uint8, device=DEV))
