"""GPU: H-LSTM stacks whose middle layer runs with launches per step between two layers of the recurrence over kept entries
(persist_batched_h.hip), against the fp64 oracle with the tolerances of parity_util.  The step kernels keep u where that recurrence
has its stamped words of u; with an odd number of steps what they leave there carries the stamp it would wait for."""
import numpy as np
import pytest

from paper_1901_10997_amd import binding as B
from paper_1901_10997_amd import inputs
from parity_util import check_case

pytestmark = pytest.mark.gpu


def _case(bidir, H, T, Bn, keep_middle, keep=0.1):
    w = inputs.Workload(132, f"between_H{H}_T{T}_B{Bn}", 3, bidir, 24, H, T, Bn, "f32", min(0.3, 1.5 / np.sqrt(keep * H)), keep, "uniform", H)
    case = inputs.make_case(w, H + T + Bn, random_state=True)
    rng = np.random.default_rng(H + T)
    for (l, _), v in case.weights.items():
        if l == 1:
            for name in ("1h", "2"):
                v["M" + name] = (rng.random((4 * H, H)) < keep_middle).astype(np.uint8)
                v["W" + name] *= np.float32(np.sqrt(keep / keep_middle))
    return case


@pytest.mark.parametrize("bidir,H,T,Bn,keep_middle,between", [
    (False, 420, 5, 3, 1.0, "csr"),            # rows of more than 384 entries
    (False, 420, 1, 6, 1.0, "csr"),
    (True, 420, 3, 3, 1.0, "csr"),
    (False, 420, 4, 3, 1.0, "csr"),            # an even number of steps
    (False, 1100, 3, 2, 0.28, "pair-csr"),     # too wide for the workgroups that the longest rows need
])
def test_step_layers_between(bidir, H, T, Bn, keep_middle, between):
    desc, _ = check_case(_case(bidir, H, T, Bn, keep_middle), B.LSTM_FMT_ROW_COMPRESSED)
    n = 2 if bidir else 1
    assert desc.count("rec=persist_batched-hlstm-csr") == 2 * n and desc.count("rec=hlstm-stepwise-" + between) == n, desc
