"""GPU: products of more than 64 input rows on the fp16 matrix instruction (fp32 operands as two fp16 planes each)."""
import numpy as np
import pytest

from paper_1901_10997_amd import binding as B
from paper_1901_10997_amd import inputs
from parity_util import check_case, run_gpu

pytestmark = pytest.mark.gpu


def _product(X, W):
    _, y = B.lstm_bench_matmul(W.shape[0], X.shape[0], 1.0, B.LSTM_FMT_DENSE_MASKED, iters=1, want_product=True, X=X, W=W)
    return y


def _bound(K):
    """Relative to the result's norm: two operands kept to 2^-23 of each value at worst and the dropped product of the two low
    parts, 2^-22, taken as if all added up; and 3 K / 16 instructions whose sums are rounded, by 2^-24 of a sum that has grown to
    its full size (it grows to it, so that an instruction may round twice), like a random walk."""
    return 2.0 ** -23 * 4 + 2.0 ** -24 * np.sqrt(3 * K / 16)


@pytest.mark.parametrize("n,batch", [(1032, 130), (1036, 191), (2052, 330), (6404, 300), (2400, 1500), (4100, 1900), (4096, 4000), (4100, 3841)])
def test_product_over_the_tile_shapes(n, batch):
    """Each of the five tile shapes, whole tiles and remainders of rows, columns and k."""
    rng = np.random.default_rng(n + batch)
    X = rng.standard_normal((batch, n)).astype(np.float32)
    W = rng.uniform(-0.1, 0.1, (n, n)).astype(np.float32)
    y = _product(X, W)
    for rows in (slice(0, 160), slice(max(0, batch - 160), batch)):
        ref = X[rows].astype(np.float64) @ W.astype(np.float64).T
        d = y[rows] - ref
        assert np.linalg.norm(d) <= _bound(n) * np.linalg.norm(ref), (np.linalg.norm(d) / np.linalg.norm(ref), _bound(n))
        assert np.max(np.abs(d)) <= 8 * _bound(n) * np.sqrt(np.mean(ref ** 2))


@pytest.mark.parametrize("n,batch", [(1032, 130), (6404, 300), (2400, 1500), (4100, 1900)])
def test_masked_product_in_two_stages(n, batch):
    """Weights with many zeros: sums in stages.  What K rounded sums would add is gone: per stage of 128 k 24 rounded sums of a
    share of the result, then at most one per stage."""
    rng = np.random.default_rng(n)
    X = rng.standard_normal((batch, n)).astype(np.float32)
    W = (rng.uniform(-0.1, 0.1, (n, n)) * (rng.random((n, n)) < 0.15)).astype(np.float32)
    _, y = B.lstm_bench_matmul(n, batch, 1.0, B.LSTM_FMT_DENSE_MASKED, iters=1, want_product=True, X=X, W=W, mask=(W != 0).astype(np.uint8))
    rows = slice(max(0, batch - 160), batch)
    ref = X[rows].astype(np.float64) @ W.astype(np.float64).T
    bound = 2.0 ** -23 * 4 + 2.0 ** -24 * np.sqrt(24 + n / 128)
    assert np.linalg.norm(y[rows] - ref) <= bound * np.linalg.norm(ref), (np.linalg.norm(y[rows] - ref) / np.linalg.norm(ref), bound)


def test_rows_that_do_not_fit_two_fp16_planes():
    """Rows of any scale, with zeros, denormals, values far below the largest, infinities and NaN give what fp32 arithmetic
    gives: every finite row within the fp32 bound of its own result, every other one its infinities and NaN."""
    n, batch = 1032, 300
    rng = np.random.default_rng(3)
    X = rng.standard_normal((batch, n)).astype(np.float32)
    W = rng.uniform(-0.1, 0.1, (n, n)).astype(np.float32)
    W[:, 5] = 0.0
    X[0] = 0.0
    X[1] *= 1e-30
    X[2] *= 1e30
    X[3, 5] = 1e9                       # meets zeros only: the rest of the row is the result
    X[4] *= np.float32(2.0) ** -140     # denormals
    X[5] = 0.0
    X[5, 7] = 3.0
    X[66, 9] = np.inf
    X[67, 9] = -np.inf
    X[140, 5] = np.inf                  # times zero
    X[299, 1031] = np.nan
    y = _product(X, W)
    with np.errstate(invalid="ignore"):
        ref = X.astype(np.float64) @ W.astype(np.float64).T
    for r in range(batch):
        if r == 4:   # the fp32 instruction flushes products below its normal range
            assert np.max(np.abs(y[r])) <= 2.0 ** -126
        elif np.isfinite(ref[r]).all():
            assert np.linalg.norm(y[r] - ref[r]) <= 2 * _bound(n) * np.linalg.norm(ref[r]), r
        else:
            np.testing.assert_array_equal(y[r].astype(np.float64), ref[r])


def test_weights_that_do_not_fit_stay_with_the_fp32_instruction():
    n, batch = 1032, 130
    rng = np.random.default_rng(4)
    X = rng.standard_normal((batch, n)).astype(np.float32)
    W = rng.uniform(-0.1, 0.1, (n, n)).astype(np.float32)
    W[17, 3] = 1e9
    X[:, 3] = 0.0
    y = _product(X, W)
    ref = X.astype(np.float64) @ W.astype(np.float64).T
    d = np.linalg.norm(y - ref, axis=0) / np.linalg.norm(ref, axis=0)
    assert np.max(d) <= 2e-6, np.max(d)     # column 17 as close as the others


@pytest.mark.parametrize("L,bidir,D,H,T,Bn,keep,fmt", [
    (2, True, 533, 150, 12, 16, None, B.LSTM_FMT_DENSE_MASKED),     # padded rows, both directions in one launch
    (1, False, 1030, 70, 1, 130, 0.3, B.LSTM_FMT_ROW_COMPRESSED),
    (2, False, 512, 600, 20, 40, 0.17, B.LSTM_FMT_AUTO),
])
def test_forward_with_split_projections(L, bidir, D, H, T, Bn, keep, fmt):
    case = inputs.make_case(inputs.Workload(87, "split", L, bidir, D, H, T, Bn, "f32", 0.05, keep, "uniform"), k=H, random_state=True)
    desc, _ = check_case(case, fmt, B.LSTM_PLAN_AUTO)
    assert "l0.d0:proj=dense-split" in desc, desc


def test_infinite_input_reaches_kept_entries_only():
    """The mask selects: an infinity in the input changes the units that keep an entry in its column, no other."""
    case = inputs.make_case(inputs.Workload(87, "split_inf", 1, False, 1032, 70, 1, 130, "f32", 0.05, 0.3, "uniform"), k=9)
    fmt = B.LSTM_FMT_ROW_COMPRESSED
    before, desc = run_gpu(case, fmt, B.LSTM_PLAN_AUTO)
    assert "proj=dense-split" in desc, desc
    case.x[0, 77, 40] = np.inf
    after = run_gpu(case, fmt, B.LSTM_PLAN_AUTO)[0]
    kept = case.weights[(0, 0)]["Mx"].reshape(4, 70, 1032)[:, :, 40].any(axis=0)
    y0, y1 = before[0].reshape(130, 70), after[0].reshape(130, 70)
    assert 0 < kept.sum() < 70
    # (the row's neighbours in its tile are summed by the fp32 instruction too: the same within rounding)
    np.testing.assert_allclose(np.delete(y1, 77, 0), np.delete(y0, 77, 0), rtol=0, atol=1e-5)
    np.testing.assert_allclose(y1[77, ~kept], y0[77, ~kept], rtol=0, atol=1e-5)
    assert not np.isnan(y1[77, ~kept]).any()
    assert (y1[77, kept] != y0[77, kept]).mean() > 0.5    # (all but those whose only such entry is in the gate that meets c0 = 0)


def _marked(X, rows, rng):
    """Rows with one value that takes most of the others below 2^-16 of it."""
    X = X.copy()
    X[rows, rng.integers(0, X.shape[1], len(rows))] = 1e7
    return X


@pytest.mark.parametrize("keep", [1.0, 0.15])
@pytest.mark.parametrize("n,batch", [(1032, 130), (1036, 191), (6404, 300), (2400, 1500), (4100, 1900), (4096, 4000)])
def test_rows_without_a_plane_form_leave_the_others_as_they_were(n, batch, keep):
    """A row's result depends on that row alone, whatever the others are: the same bits; and the marked rows are within the bound of
    an fp32 sum (K rounded additions that add up like a random walk) of theirs."""
    rng = np.random.default_rng(n + batch)
    X = rng.standard_normal((batch, n)).astype(np.float32)
    W = (rng.uniform(-0.1, 0.1, (n, n)) * (rng.random((n, n)) < keep)).astype(np.float32)
    y = _product(X, W)
    for rows in (np.array([batch - 1]), rng.permutation(batch)[:batch // 3], np.sort(rng.permutation(batch)[:batch - 2]), np.arange(batch)):
        Xm = _marked(X, rows, rng)
        ym = _product(Xm, W)
        others = np.setdiff1d(np.arange(batch), rows)
        assert np.array_equal(ym[others], y[others])
        some = rows[rng.permutation(len(rows))[:120]]
        ref = Xm[some].astype(np.float64) @ W.astype(np.float64).T
        err = np.linalg.norm(ym[some] - ref, axis=1) / np.linalg.norm(ref, axis=1)
        assert np.max(err) <= 4 * 2.0 ** -24 * np.sqrt(n), (np.max(err), len(rows))


def test_non_finite_rows_leave_the_others_as_they_were():
    case = inputs.make_case(inputs.Workload(87, "split_inf", 1, True, 1032, 70, 1, 330, "f32", 0.05, 0.3, "uniform"), k=9)
    fmt = B.LSTM_FMT_ROW_COMPRESSED
    before, desc = run_gpu(case, fmt, B.LSTM_PLAN_AUTO)
    assert "proj=dense-split" in desc, desc
    rows = [0, 64, 65, 200, 329]
    case.x[0, rows, [1, 40, 77, 1031, 500]] = [np.inf, -np.inf, np.nan, np.inf, np.nan]
    after = run_gpu(case, fmt, B.LSTM_PLAN_AUTO)[0]
    for a, b in zip(after, before):
        a, b = a.reshape(-1, 330, a.shape[-1]), b.reshape(-1, 330, b.shape[-1])
        assert np.array_equal(np.delete(a, rows, 1), np.delete(b, rows, 1))
    # the units that keep no entry in the column: a sum over their kept entries, the same within rounding
    kept = case.weights[(0, 0)]["Mx"].reshape(4, 70, 1032)[:, :, 77].any(axis=0)
    y0, y1 = before[0].reshape(330, 140), after[0].reshape(330, 140)
    np.testing.assert_allclose(y1[65, :70][~kept], y0[65, :70][~kept], rtol=0, atol=1e-5)
    assert np.isnan(y1[65, :70][kept]).any()


def test_more_rows_than_one_launch_takes_and_unaligned_input():
    """40000 rows (a launch takes 32768), marked ones in both launches, from an address that is no multiple of 16 bytes; every launch
    looks at its own rows, and a call without a marked row gives the first one's bits again."""
    import torch
    D, H, Bn = 200, 300, 40000
    case = inputs.make_case(inputs.Workload(88, "split_rows", 1, False, D, H, 1, 64, "f32", 0.05, None, "uniform"), k=2)
    m = B.Lstm(1, D, H, False, B.LSTM_F32)
    m.set_weights_from(case.weights, B.LSTM_FMT_DENSE_MASKED)
    dev = torch.device("cuda:0")
    buf = torch.randn(Bn * D + 1, device=dev, generator=torch.Generator(device=dev).manual_seed(5))
    x = buf[1:].view(1, Bn, D)
    assert x.data_ptr() % 16 == 4
    first = m.forward(x, None, None)[0].clone()
    assert "proj=dense-split" in B.lstm_describe_plan(m.handle), B.lstm_describe_plan(m.handle)
    rows = torch.tensor([0, 5, 100, 32767, 32768, 39999], device=dev)
    keep = x[0, rows].clone()
    x[0, rows, 3] = 3e5
    y = m.forward(x, None, None)[0]
    others = torch.ones(Bn, dtype=torch.bool, device=dev)
    others[rows] = False
    assert torch.equal(y[0, others], first[0, others]) and not torch.equal(y[0, rows], first[0, rows])
    p = case.weights[(0, 0)]
    a = x[0, rows].double().cpu().numpy() @ p["Wx"].astype(np.float64).T + p["b"]
    f, i, o, g = (a[:, q * H:(q + 1) * H] for q in range(4))
    sig = lambda v: 0.5 * (1 + np.tanh(0.5 * v))
    ref = sig(o) * np.tanh(sig(i) * np.tanh(g))
    # a pre-activation of up to 3e5 * 0.05 sums 200 terms to 2^-24 of that each
    assert np.max(np.abs(y[0, rows].cpu().numpy() - ref)) <= 2.0 ** -24 * 15000 * np.sqrt(200)
    x[0, rows] = keep
    assert torch.equal(m.forward(x, None, None)[0], first)
    m.close()


def _f32_chain(X, W):
    """X . W^T as fp32 multiply-adds in the order of k: what the fp32 matrix instruction rounds, a zero term never does."""
    y = np.zeros((X.shape[0], W.shape[0]), np.float32)
    for k in range(X.shape[1]):
        y = (y.astype(np.float64) + X[:, k:k + 1].astype(np.float64) * W[:, k].astype(np.float64)).astype(np.float32)
    return y


def _error(y, ref):
    return np.linalg.norm(y - ref) / np.linalg.norm(ref)


@pytest.mark.parametrize("n,kept", [(640, 0.05), (1032, 0.02), (1032, 0.10), (1032, 0.45), (640, 0.8)])
@pytest.mark.parametrize("as_mask", [True, False])
def test_products_of_few_terms_are_no_further_from_64_bits(n, kept, as_mask):
    """Rows with few entries, by a mask or as zeros among the weights: no further from the exact product than a chain of fp32
    multiply-adds over the kept entries (the order of the sums moves either by a tenth or two)."""
    rng = np.random.default_rng(n)
    batch = 4096 if n == 640 else 2048
    X = rng.standard_normal((batch, n)).astype(np.float32)
    keep = rng.random((n, n)) < kept
    W = (rng.uniform(-0.1, 0.1, (n, n)) * keep).astype(np.float32)
    _, y = B.lstm_bench_matmul(n, batch, 1.0, B.LSTM_FMT_DENSE_MASKED, iters=1, want_product=True, X=X, W=W,
                               mask=keep.astype(np.uint8) if as_mask else None)
    ref = X[:200].astype(np.float64) @ W.astype(np.float64).T
    assert _error(y[:200], ref) <= 1.1 * _error(_f32_chain(X[:200], W), ref)


@pytest.mark.parametrize("n,batch", [(1032, 130), (2052, 330), (6404, 300), (2400, 1500), (4100, 1900)])
@pytest.mark.parametrize("kept", [0.1, 0.4])
def test_staged_sums_keep_what_the_planes_hold(n, batch, kept):
    """Weights with many zeros: the error does not grow with K.  Of each operand one value in four is off by half a last place of
    its fp32 form (rms 4e-8, two operands 5.6e-8), the product of the two low planes is left out (3.5e-8), a stage rounds 8 sums
    that grow to its own (4.9e-8), and the sums are added up with what that rounds off: 8.3e-8 of the product's norm, and half of
    that on top for the values between two powers of two that this takes in the middle."""
    rng = np.random.default_rng(n)
    X = rng.standard_normal((batch, n)).astype(np.float32)
    W = (rng.uniform(-0.1, 0.1, (n, n)) * (rng.random((n, n)) < kept)).astype(np.float32)
    y = _product(X, W)
    rows = slice(max(0, batch - 160), batch)
    ref = X[rows].astype(np.float64) @ W.astype(np.float64).T
    assert _error(y[rows], ref) <= 1.25e-7


def test_input_rows_of_few_terms_are_no_further_from_64_bits():
    """Input rows that are zero but for a few values (one-hot rows among them) beside full ones."""
    n, batch = 1032, 2048
    rng = np.random.default_rng(8)
    X = rng.standard_normal((batch, n)).astype(np.float32)
    W = rng.uniform(-0.1, 0.1, (n, n)).astype(np.float32)
    X[:40] = 0.0
    X[np.arange(40), rng.integers(0, n, 40)] = 1.0
    X[40:80] *= rng.random((40, n)) < 0.02
    X[80:90] = 0.0
    y = _product(X, W)
    ref = X[:200].astype(np.float64) @ W.astype(np.float64).T
    np.testing.assert_array_equal(y[:40].astype(np.float64), ref[:40])     # one term: exact
    assert _error(y[40:80], ref[40:80]) <= 1.1 * _error(_f32_chain(X[40:80], W), ref[40:80])
    assert not y[80:90].any()


def test_masked_layers_of_few_entries_keep_their_sums():
    """The H-LSTM and LSTM layers whose projection goes by the same rule."""
    for keep, want in ((0.05, "proj=dense,"), (0.30, "proj=dense-split,")):
        case = inputs.make_case(inputs.Workload(89, "few_terms", 1, True, 512, 160, 30, 20, "f32", 0.05, keep, "uniform", 160), k=4, random_state=True)
        desc, _ = check_case(case)
        assert want in desc, desc


def test_workspace_holds_planes_of_the_input_only_where_they_can_run():
    """At most 64 input rows are multiplied without them: the workspace has no room for them then."""
    D, H = 2000, 512
    m = B.Lstm(1, D, H, False, B.LSTM_F32)
    per_row = 4 * (4 * H + D)                                # pre-activations and the transposed input
    few, many = B.lstm_workspace_bytes(m.handle, 64, 1), B.lstm_workspace_bytes(m.handle, 4096, 1)
    assert few < 64 * (per_row + 4 * D // 2) and many > 4096 * (per_row + 4 * D)
    m.close()
