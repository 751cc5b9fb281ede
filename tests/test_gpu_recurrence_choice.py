"""GPU: which recurrence LSTM_FMT_AUTO takes for a masked H-LSTM layer, at sizes where one side is at least a fifth faster (microseconds
per step over kept entries / dense in the comments), and its outputs against the fp64 oracle with the tolerances of parity_util."""
import numpy as np
import pytest

from paper_1901_10997_amd import inputs
from parity_util import check_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bidir,H,G,Bn,keep,takes", [
    (False, 212, 212, 1, 0.20, "persist-dense-hlstm"),        # 3.06 / 1.89
    (False, 291, 291, 1, 0.23, "persist-dense-hlstm"),        # 2.98 / 2.34
    (True, 848, 946, 1, 0.31, "persist-dense-hlstm"),         # 7.48 / 4.89
    (False, 1500, 1500, 1, 0.10, "persist_b1-hlstm-csr"),     # 3.5 / 6.9
    (False, 416, 416, 5, 0.12, "persist_batched-hlstm-csr"),  # 2.10 / 3.01
    (True, 87, 87, 55, 0.11, "persist_batched-hlstm-csr"),    # 1.87 / 2.23
])
def test_recurrence_of_a_masked_hlstm_layer(bidir, H, G, Bn, keep, takes):
    w = inputs.Workload(134, f"choice_H{H}_G{G}_B{Bn}", 1, bidir, 32, H, 60, Bn, "f32", min(0.2, 0.7 / np.sqrt(keep * H)), keep, "uniform", G)
    desc, _ = check_case(inputs.make_case(w, H + Bn, random_state=True))
    assert desc.count("rec=" + takes) == (2 if bidir else 1), desc
