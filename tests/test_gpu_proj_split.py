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
    """Relative to the result's norm: two operands kept to 2^-23 of each value at worst, the dropped product of the two low
    parts 2^-22, and 3 K / 16 rounded sums of 2^-24 each that add up like a random walk."""
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
    """Weights with many zeros: sums in two stages.  What K rounded sums would add is gone: per stage of 128 k 24 rounded sums
    of a share of the result, then one per stage."""
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
