"""GPU parity: condensa_lc_step against the oracle (every output bit exact)."""
import numpy as np
import pytest
import torch

import oracle
import paper_1911_02497_amd as P
from gpu_util import assert_bits_equal, assert_select_equal, DEV, Form, FORMS, up, with_form

pytestmark = pytest.mark.gpu

lc_step = with_form(P.condensa_lc_step)
lc_step_pq = with_form(P.condensa_lc_step_pq)


@pytest.fixture(params=["auto", "radix", "window", "window_narrow", "window_two_sweeps"], autouse=True)
def select_path(request):
    """Every case runs through the automatic choice (listed windows: one sweep, then lists of the keys around
    the thresholds), the radix levels, the sampled window (selection and apply in one sweep
    where the call allows it), a window whose margin is cut to a couple of sample ranks so that it
    regularly misses and falls back, and the window with separate selection and apply sweeps."""
    Form.config = FORMS[request.param]
    yield request.param
    Form.config = None


def _check(ws, ls, mu, d, what="", **kw):
    res = lc_step(up(ws), up(ls), mu, d, **kw)
    torch.cuda.synchronize()
    ora = oracle.lc_step(ws, ls, mu, d)
    assert_select_equal(P.select_records(res["results"])[0], ora["select"], what)
    for t in range(len(ws)):
        assert np.array_equal(res["mask"][t].cpu().numpy(), ora["mask"][t]), f"{what} mask {t}"
        assert_bits_equal(res["theta"][t], ora["theta"][t], f"{what} theta {t}")
        assert_bits_equal(res["lambda"][t], ora["lambda"][t], f"{what} lambda {t}")
        assert_bits_equal(res["grad"][t], ora["grad"][t], f"{what} grad {t}")
    return res, ora


def _gauss(shapes, seed, std):
    rng = np.random.default_rng(seed)
    return [(rng.standard_normal(s) * std).astype(np.float32) for s in shapes]


def test_several_tensors_ragged():
    shapes = [(8192 * 2 + 3,), (37, 41), (1,), (0,), (16, 8, 3, 3), (8191,)]
    ws, ls = _gauss(shapes, 1, 0.01), _gauss(shapes, 2, 0.01)
    for d in (0.0, 0.1, 0.5, 1.0):
        _check(ws, ls, 1e-3, d, f"d={d}")


def test_mu_schedule_values_and_denormals():
    shapes = [(5000,)]
    ws, ls = _gauss(shapes, 3, 0.01), _gauss(shapes, 4, 0.01)
    ls[0][:50] = np.float32(1e-41)            # denormal multipliers: the division must not flush them
    ws[0][50:100] = np.float32(3e-39)
    for j in (0, 1, 10, 49):
        _check(ws, ls, 1e-3 * 1.1 ** j, 0.1, f"mu_{j}")


def test_planted_ties_in_the_shifted_weights():
    n = 8192 * 4
    ws, ls = _gauss([(n,)], 5, 0.01), [np.zeros(n, np.float32)]
    for p in (7, 8191, 8192, 30000, 32767):
        ws[0][p] = np.float32(0.0123)
    n_gt = int((np.abs(ws[0]) > np.float32(0.0123)).sum())
    for extra in (2, 5):
        res, ora = _check(ws, ls, 1e-3, (n_gt + extra) / n, f"ties {extra}")
        assert ora["select"]["n_tie"] == 5 and ora["select"]["n_tie_kept"] == extra


def test_in_place_multiplier_update_and_optional_outputs():
    ws, ls = _gauss([(10000,), (333,)], 6, 0.01), _gauss([(10000,), (333,)], 7, 0.01)
    ora = oracle.lc_step(ws, ls, 1e-3, 0.2)
    dl = up(ls)
    res = lc_step(up(ws), dl, 1e-3, 0.2, in_place=True, theta=False, mask=False)
    torch.cuda.synchronize()
    for t in range(2):
        assert_bits_equal(dl[t], ora["lambda"][t], "in-place lambda")
        assert_bits_equal(res["grad"][t], ora["grad"][t], "grad")


def test_errors():
    w, l = torch.ones(8, device=DEV), torch.zeros(8, device=DEV)
    for mu in (0.0, -1.0, float("inf"), float("nan")):
        with pytest.raises(P.CondensaError) as e:
            lc_step([w], [l], mu, 0.5)
        assert e.value.code == -3
    with pytest.raises(P.CondensaError) as e:          # theta must not alias w
        lc_step([w], [l], 1e-3, 0.5, outputs={"theta": [w]})
    assert e.value.code == -6


# ---- composed scheme P+Q as the compression step, and the footprint objective ---------------------------

def test_pq_step_against_the_oracle():
    shapes = [(8192 * 2 + 3,), (37, 41), (0,), (16, 8, 3, 3)]
    ws, ls = _gauss(shapes, 11, 0.01), _gauss(shapes, 12, 0.01)
    ws[1][0, :8] = np.float32(1e-9)                     # tiny values: underflow to zero in binary16 if kept
    for mu, d in ((1e-3, 0.1), (1e-3, 1.0), (50.0, 0.5)):
        res = lc_step_pq(up(ws), up(ls), mu, d, nnz=True)
        torch.cuda.synchronize()
        ora = oracle.lc_step_pq(ws, ls, mu, d)
        assert_select_equal(P.select_records(res["results"])[0], ora["select"], f"mu={mu} d={d}")
        for t in range(len(ws)):
            assert np.array_equal(res["mask"][t].cpu().numpy(), ora["mask"][t])
            assert np.array_equal(res["theta_f16"][t].cpu().numpy().view(np.uint16), ora["theta_f16"][t]), f"theta16 {t}"
            for name in ("theta", "lambda", "grad"):
                assert_bits_equal(res[name][t], ora[name][t], f"{name} {t} mu={mu} d={d}")
        nnz = int(P.condensa_count_nonzero(res["theta_f16"]).item())
        assert nnz == oracle.count_nonzero(ora["theta_f16"])
        # the same objective as a by-product of the step: k less the kept values that underflow in binary16
        assert int(res["nnz"].item()) == oracle.count_nonzero(ora["theta_f16"]), f"fused non-zero count, mu={mu} d={d}"
        nnz32 = int(P.condensa_count_nonzero(res["theta"]).item())
        assert nnz32 == oracle.count_nonzero(ora["theta"])


def test_pq_step_with_theta_as_codes_only_leaves_reused_buffers_alone():
    """theta=False with an earlier call's buffers passed back in: the fp32 theta is not written (its buffer
    keeps what it held), the codes, the multipliers, the penalty gradient and the count are the oracle's."""
    shapes = [(8192 * 3 + 5,), (129, 67)]
    ws, ls = _gauss(shapes, 21, 0.01), _gauss(shapes, 22, 0.01)
    dw, dl = up(ws), up(ls)
    first = lc_step_pq(dw, dl, 1e-3, 0.5, nnz=True)
    torch.cuda.synchronize()
    for t in first["theta"]:
        t.fill_(7.0)
    res = lc_step_pq(dw, dl, 1e-3, 0.1, nnz=True, theta=False, mask=False, outputs=first)
    torch.cuda.synchronize()
    ora = oracle.lc_step_pq(ws, ls, 1e-3, 0.1)
    assert res["theta"] is None and res["mask"] is None
    for t in range(len(ws)):
        assert bool((first["theta"][t] == 7.0).all()), "the switched-off output was written"
        assert np.array_equal(res["theta_f16"][t].cpu().numpy().view(np.uint16), ora["theta_f16"][t]), f"theta16 {t}"
        assert_bits_equal(res["lambda"][t], ora["lambda"][t], f"lambda {t}")
        assert_bits_equal(res["grad"][t], ora["grad"][t], f"grad {t}")
    assert int(res["nnz"].item()) == oracle.count_nonzero(ora["theta_f16"])


def test_count_nonzero_edge_cases():
    x = torch.tensor([0.0, -0.0, 1e-30, -2.0, 3.0, float("nan")], device=DEV)
    assert int(P.condensa_count_nonzero([x]).item()) == 4
    q, _ = P.condensa_quantize(x)
    assert int(P.condensa_count_nonzero([q]).item()) == 3
    big = torch.ones(8192 * 5 + 7, device=DEV)
    big[::3] = 0
    want = int((big != 0).sum().item())
    assert int(P.condensa_count_nonzero([big, x, torch.zeros(0, device=DEV)]).item()) == want + 4
    assert int(P.condensa_count_nonzero([big[1:]]).item()) == int((big[1:] != 0).sum().item())   # misaligned view
    assert int(P.condensa_count_nonzero([]).item()) == 0
    # 16-bit and 8-bit floating-point codes: several chunks, a ragged tail, a misaligned view, empty tensors
    rng = np.random.default_rng(12)
    v = (rng.standard_normal(8192 * 9 + 1234) * (rng.random(8192 * 9 + 1234) < 0.4)).astype(np.float32)
    v[5], v[6] = -0.0, 1e-30
    for codes in (oracle.quantize_f16(v)[0], oracle.quantize_bf16(v)[0], oracle.quantize_fp8(v, oracle.FP8_E4M3)[0],
                  oracle.quantize_fp8(v, oracle.FP8_E5M2)[0]):
        as_torch = codes.view(np.int16) if codes.dtype == np.uint16 else codes
        d = torch.from_numpy(as_torch.copy()).to(DEV)
        assert int(P.condensa_count_nonzero([d, d[:0], d[:100]]).item()) == oracle.count_nonzero([codes, codes[:100]])
        assert int(P.condensa_count_nonzero([d[1:]]).item()) == oracle.count_nonzero([codes[1:]])
    q8, _ = P.condensa_quantize_fp8(x, P.FP8_E5M2)
    assert int(P.condensa_count_nonzero([q8]).item()) == 3


# ---- learning-step update with the penalty folded in ----------------------------------------------------

def test_sgd_step_with_penalty_against_the_oracle():
    shapes = [(8192 + 77,), (64, 32, 3, 3), (0,), (10, 512)]
    rng = np.random.default_rng(60)
    mk = lambda s: [(rng.standard_normal(sh) * s).astype(np.float32) for sh in shapes]  # noqa: E731
    ws, gs, ths, ls, bs = mk(0.01), mk(1e-3), mk(0.01), mk(0.01), mk(1e-3)
    for j in (0, 7):
        mu = P.condensa_mu_schedule(1e-3, 1.1, j)
        assert mu == oracle.mu_schedule(1e-3, 1.1, j)
        dw, db = up(ws), up(bs)
        P.condensa_lc_sgd_step(dw, up(gs), up(ths), up(ls), db, mu, 0.1, 0.9)
        torch.cuda.synchronize()
        w_ora, b_ora = oracle.lc_sgd_step(ws, gs, ths, ls, bs, mu, 0.1, 0.9)
        for t in range(len(ws)):
            assert_bits_equal(dw[t], w_ora[t], f"w {t}")
            assert_bits_equal(db[t], b_ora[t], f"buf {t}")
    # the fused update equals the unfused one: penalty gradient from condensa_lc_step, then a plain momentum step
    res = lc_step(up(ws), up(ls), 1e-3, 0.2)
    torch.cuda.synchronize()
    theta = [t.cpu().numpy() for t in res["theta"]]
    lam2 = [t.cpu().numpy() for t in res["lambda"]]
    w_f, b_f = oracle.lc_sgd_step(ws, gs, theta, lam2, bs, 1e-3, 0.1, 0.9)
    for t in range(len(ws)):
        g_pen = res["grad"][t].cpu().numpy()                       # mu (w - theta) - lambda'
        b = np.float32(0.9) * bs[t] + (gs[t] + g_pen)
        assert np.allclose(b, b_f[t], rtol=0, atol=2e-8) and np.allclose(ws[t] - np.float32(0.1) * b, w_f[t], rtol=0, atol=2e-8)
    w = torch.ones(8, device=DEV)
    with pytest.raises(P.CondensaError) as e:
        P.condensa_lc_sgd_step([w], [w], [torch.zeros(8, device=DEV)], [torch.zeros(8, device=DEV)], [torch.zeros(8, device=DEV)], 1e-3, 0.1, 0.9)
    assert e.value.code == -6


def test_misaligned_tensors_and_partial_outputs():
    """Pointers that are not 16-byte aligned take the scalar path of every sweep (also of the one-sweep
    form); outputs that are not asked for are skipped."""
    n = 8192 * 3 + 77
    ws, ls = _gauss([(n,), (1001,)], 21, 0.01), _gauss([(n,), (1001,)], 22, 0.01)
    ora = oracle.lc_step(ws, ls, 1e-3, 0.25)

    def shifted(a):                                     # same values, storage offset by one element
        big = torch.empty(a.size + 1, dtype=torch.float32, device=DEV)
        big[1:] = torch.from_numpy(a.reshape(-1)).to(DEV)
        return big[1:].view(a.shape)

    dw, dl = [shifted(a) for a in ws], [shifted(a) for a in ls]
    out_l = [shifted(np.zeros_like(a)) for a in ls]
    res = lc_step(dw, dl, 1e-3, 0.25, lambda_out=out_l, grad=False)
    torch.cuda.synchronize()
    assert res["grad"] is None
    for t in range(2):
        assert_bits_equal(res["theta"][t], ora["theta"][t], f"theta {t}")
        assert_bits_equal(out_l[t], ora["lambda"][t], f"lambda {t}")
        assert np.array_equal(res["mask"][t].cpu().numpy(), ora["mask"][t])
    res = lc_step(up(ws), up(ls), 1e-3, 0.25, theta=False, mask=False)
    torch.cuda.synchronize()
    for t in range(2):
        assert_bits_equal(res["lambda"][t], ora["lambda"][t], f"lambda only {t}")
        assert_bits_equal(res["grad"][t], ora["grad"][t], f"grad only {t}")


def test_same_step_twice_and_other_launch_shapes_give_the_same_bits():
    """Determinism of the L-C step: the same call twice, the apply sweep in workgroups of 64, 128 and 256
    threads, separate sweeps instead of one, and other sample / candidate sizes (other grids and segment
    counts) agree in every bit of theta, lambda', g, the mask and the record."""
    rng = np.random.default_rng(78)
    shapes = ((1200, 1024), (8192 * 30 + 5,), (128, 64, 3, 3))
    ws = [(rng.standard_normal(s) * 0.01).astype(np.float32) for s in shapes]
    ls = [(rng.standard_normal(s) * 0.01).astype(np.float32) for s in shapes]
    dw, dl = up(ws), up(ls)
    fields = ("n", "k", "n_gt", "n_tie_kept", "n_tie", "threshold_key", "tie_end")
    ref = lc_step(dw, dl, 1e-3, 0.1)
    torch.cuda.synchronize()
    ref_rec = P.select_records(ref["results"])[0]
    base = dict(Form.config)
    variants = [base] + [dict(base, apply_threads=n, fused_sweep=1) for n in (64, 128, 256)] + \
               [dict(base, sample_log2=16), dict(base, cand_shift=3), dict(base, select_path=1, apply_threads=256)]
    for cfg in variants:
        got = P.condensa_lc_step(dw, dl, 1e-3, 0.1, config=cfg)
        torch.cuda.synchronize()
        rec = P.select_records(got["results"])[0]
        assert all(rec[f] == ref_rec[f] for f in fields), (cfg, rec, ref_rec)
        for name in ("theta", "lambda", "grad"):
            for t in range(len(ws)):
                assert torch.equal(got[name][t].view(torch.int32), ref[name][t].view(torch.int32)), (cfg, name, t)
        for t in range(len(ws)):
            assert torch.equal(got["mask"][t], ref["mask"][t]), (cfg, t)
