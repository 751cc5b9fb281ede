"""GPU: recurrences over kept entries whose exchanged values carry their readiness in a bit (gather_stamped in exchange.h),
against the fp64 oracle with the tolerances of parity_util: array lengths that are no multiple of a load, several launches
over the same words, ragged groups, NaN."""
import numpy as np
import pytest

from paper_1901_10997_amd import binding as B
from paper_1901_10997_amd import inputs
from parity_util import check_case, run_gpu

pytestmark = pytest.mark.gpu

CSR = B.LSTM_FMT_ROW_COMPRESSED


def _case(L, bidir, D, H, T, Bn, keep, G=0):
    w = inputs.Workload(130, f"stamped_L{L}_H{H}_G{G}_T{T}_B{Bn}", L, bidir, D, H, T, Bn, "f32", min(0.3, 1.5 / np.sqrt(keep * max(H, G, 16))),
                        keep, "uniform", G)
    return inputs.make_case(w, H + Bn + T, random_state=True)


@pytest.mark.parametrize("L,bidir,D,H,T,Bn,keep,G", [
    (3, True, 24, 37, 6, 2, 0.3, 53),      # odd widths, two columns per group: the last group of words is half full
    (3, False, 24, 53, 7, 3, 0.3, 37),     # a ragged group; workgroups with units of one vector only
    (4, False, 16, 130, 1, 5, 0.2, 96),    # one step per launch: h is never written, u once a layer
    (3, True, 40, 400, 5, 37, 0.1, 400),   # groups of several columns, the last one ragged
    (2, False, 24, 2000, 3, 40, 0.02, 300),   # several launches per layer
    (2, True, 640, 800, 4, 16, 0.2, 800),
])
def test_hlstm(L, bidir, D, H, T, Bn, keep, G):
    desc, _ = check_case(_case(L, bidir, D, H, T, Bn, keep, G), CSR)
    assert desc.count("rec=persist_batched-hlstm-csr") == L * (2 if bidir else 1), desc


@pytest.mark.parametrize("H,G,Bn", [(70, 96, 6), (131, 64, 3)])
def test_nan_stays_in_its_sequence(H, G, Bn):
    case = _case(1, True, 24, H, 6, Bn, 0.3, G)
    (y0, hT0, cT0), _ = run_gpu(case, CSR)
    b = Bn - 1
    case.c0[:, b, H // 2] = np.nan
    (y, hT, cT), desc = run_gpu(case, CSR)
    assert "persist_batched-hlstm-csr" in desc, desc
    assert np.isnan(y[0, b, H // 2]) and np.isnan(cT[0, b, H // 2])
    others = np.arange(Bn) != b
    for got, ref in ((y, y0), (hT, hT0), (cT, cT0)):
        np.testing.assert_array_equal(got[:, others], ref[:, others])


@pytest.mark.parametrize("L,bidir,D,H,T,Bn,keep", [
    (3, True, 24, 37, 6, 2, 0.3),         # an odd number of units, two columns per group: the last group of words is half full
    (3, False, 24, 131, 7, 3, 0.2),       # a ragged group
    (4, False, 16, 250, 1, 5, 0.2),       # one step per launch: nothing is published
    (3, True, 40, 402, 5, 37, 0.1),
    (3, False, 24, 1900, 3, 61, 0.02),    # several launches per layer, runs of unequal length
    (2, False, 64, 1500, 4, 20, 0.1),
])
def test_lstm(L, bidir, D, H, T, Bn, keep):
    desc, _ = check_case(_case(L, bidir, D, H, T, Bn, keep), CSR)
    assert desc.count("rec=persist_batched-q16") == L * (2 if bidir else 1), desc


@pytest.mark.parametrize("H,Bn", [(71, 6), (300, 3)])
def test_nan_stays_in_its_sequence_lstm(H, Bn):
    case = _case(1, True, 24, H, 6, Bn, 0.3)
    (y0, hT0, cT0), _ = run_gpu(case, CSR)
    b = Bn - 1
    case.c0[:, b, H // 2] = np.nan
    (y, hT, cT), desc = run_gpu(case, CSR)
    assert "persist_batched-q16" in desc, desc
    assert np.isnan(y[0, b, H // 2]) and np.isnan(cT[0, b, H // 2]) and np.isnan(y[1:, b, :H]).sum() > 1
    others = np.arange(Bn) != b
    for got, ref in ((y, y0), (hT, hT0), (cT, cT0)):
        np.testing.assert_array_equal(got[:, others], ref[:, others])
