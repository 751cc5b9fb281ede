"""GPU: recurrences over kept entries whose batch is cut into runs of unequal length, a launch each over the same words: against the
fp64 oracle with the tolerances of parity_util, and no launch more than runs of equal length take (the words are cleared once)."""
import ctypes
import os

import numpy as np
import pytest

from paper_1901_10997_amd import binding as B
from paper_1901_10997_amd import inputs
from parity_util import check_case, run_gpu

pytestmark = pytest.mark.gpu

CSR = B.LSTM_FMT_ROW_COMPRESSED


def _case(L, H, G, T, Bn, keep):
    w = inputs.Workload(133, f"uneven_H{H}_G{G}_B{Bn}", L, False, 24, H, T, Bn, "f32", min(0.3, 1.5 / np.sqrt(keep * max(H, G, 16))), keep, "uniform", G)
    return inputs.make_case(w, H + Bn, random_state=True)


def _nodes(case):
    """Nodes of the graph that a forward is captured into."""
    import torch
    _, desc, model = run_gpu(case, CSR, return_model=True, cooperative=False)
    dev = torch.device("cuda:0")
    x, h0, c0 = (torch.from_numpy(a).to(dev) for a in (case.x, case.h0, case.c0))
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        model.forward(x, h0, c0, check=False)
    n = ctypes.c_size_t()
    hip = ctypes.CDLL(os.path.join(os.path.dirname(torch.__file__), "lib", "libamdhip64.so"))
    assert hip.hipGraphGetNodes(ctypes.c_void_p(g.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    torch.cuda.synchronize()
    model.close()
    return n.value, desc


@pytest.mark.parametrize("H,G,keep,uneven,even,runs", [
    (1900, 0, 0.02, 51, 52, 4),      # 12 and 13 columns: six groups of two, seven
    (2000, 300, 0.02, 38, 39, 3),    # 12 and 13: three groups of four, four
    (2000, 300, 0.02, 44, 45, 3),    # 14 and 15: four groups both
])
def test_words_are_cleared_once(H, G, keep, uneven, even, runs):
    case = _case(3, H, G, 4, uneven, keep)
    check_case(case, CSR)
    n, desc = _nodes(case)
    n_even, desc_even = _nodes(_case(3, H, G, 4, even, keep))
    assert desc.count(f"batch/{runs}") == 3 and desc_even.count(f"batch/{runs}") == 3, (desc, desc_even)
    assert n == n_even


def test_runs_of_unlike_shape():
    """16 and 17 columns of 1500 units take different shapes; the words are cleared between them, as for another layer."""
    desc, _ = check_case(_case(2, 1500, 0, 3, 50, 0.10), CSR)
    assert desc.count("batch/3") == 2, desc
