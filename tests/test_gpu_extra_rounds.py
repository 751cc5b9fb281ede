"""GPU: entries beyond a matrix's slots in the quarter-wave form, sixteen of a gate per round (quarter_wave.h), against the fp64
oracle with the tolerances of parity_util: one round (LSTM and projection; no more are ever packed) and one to three (H-LSTM), every unit
count per wave, the last units, other units' sums."""
import re

import numpy as np
import pytest

from paper_1901_10997_amd import binding as B
from paper_1901_10997_amd import inputs
from parity_util import check_case, run_gpu

pytestmark = pytest.mark.gpu

CSR = B.LSTM_FMT_ROW_COMPRESSED


def _mask(rng, units, cols, kept, extra):
    """Rows of `kept` entries; `extra` more in one row of gate 1 near the start, and in two rows of gate 3 at the end."""
    m = np.zeros((4, units, cols), dtype=np.uint8)
    more = np.zeros((4, units), dtype=int)
    more[1, 2] = extra
    more[3, units - 1] = extra // 3
    more[3, units - 2] = extra - extra // 3
    for q in range(4):
        for u in range(units):
            m[q, u, rng.choice(cols, kept + more[q, u], replace=False)] = 1
    return m.reshape(4 * units, cols)


def _case(L, bidir, D, H, T, Bn, kept, extra, G=0, keep=0.3):
    w = inputs.Workload(131, f"rounds_H{H}_G{G}_{kept}_{extra}", L, bidir, D, H, T, Bn, "f32", min(0.3, 1.5 / np.sqrt(kept)), keep, "uniform", G)
    case = inputs.make_case(w, H + Bn + extra, random_state=True)
    rng = np.random.default_rng(H + G + extra)
    for v in case.weights.values():
        for name, units, cols in (("M1h", G, H), ("M2", H, G)) if G else (("Mh", H, H),):
            v[name] = _mask(rng, units, cols, kept, extra)
    return case


@pytest.mark.parametrize("H,Bn,kept,extra,bidir", [
    (70, 3, 32, 1, True),
    (150, 2, 64, 16, False),
    (403, 5, 96, 16, True),        # a ragged last wave
    (1000, 20, 96, 16, False),
    (1500, 20, 64, 9, False),
    (1900, 61, 32, 16, False),     # several launches
])
def test_lstm(H, Bn, kept, extra, bidir):
    desc, _ = check_case(_case(2, bidir, 24, H, 5, Bn, kept, extra), CSR)
    n = 4 if bidir else 2
    assert desc.count(f"rec=persist_batched-q16+ovf(s{kept // 16},") == n, desc


@pytest.mark.parametrize("H,G,Bn,kept,extra", [
    (90, 75, 3, 32, 5),
    (90, 75, 3, 32, 20),           # two rounds
    (200, 211, 6, 64, 48),         # three
    (800, 800, 16, 96, 40),
    (300, 900, 5, 96, 48),         # workgroups without a unit of h
    (1000, 96, 18, 32, 33),        # ... of u
])
def test_hlstm(H, G, Bn, kept, extra):
    desc, _ = check_case(_case(2, True, 24, H, 5, Bn, kept, extra, G), CSR)
    assert desc.count(f"rec=persist_batched-hlstm-csr+ovf(s{kept // 16},") == 4, desc


@pytest.mark.parametrize("H,D,kept,extra", [(70, 533, 64, 16), (131, 2048, 96, 7), (64, 2048, 352, 16)])   # four units to a wave, three
def test_projection(H, D, kept, extra):
    case = _case(1, False, D, H, 13, 5, 32, 0)
    case.weights[(0, 0)]["Mx"] = _mask(np.random.default_rng(H), H, D, kept, extra)
    case.weights[(0, 0)]["Wx"] *= 0.2
    desc, _ = check_case(case, CSR)
    assert "proj=q16" in desc, desc


@pytest.mark.parametrize("H,G", [(150, 0), (90, 75)])
def test_infinite_weight_stays_in_its_unit(H, G):
    """An entry outside the slots, one step: no other unit's sums change (they are left out, not multiplied by zero)."""
    case = _case(1, False, 24, H, 1, 6, 32, 16, G)
    before, desc = run_gpu(case, CSR)
    assert "+ovf" in desc, desc
    v = case.weights[(0, 0)]
    name, units = ("2", H) if G else ("h", H)
    row = 3 * units + units - 2
    v["W" + name][row, np.flatnonzero(v["M" + name][row])[-1]] = np.inf
    after, _ = run_gpu(case, CSR)
    others = np.arange(H) != units - 2
    for a, b in zip(after, before):
        np.testing.assert_array_equal(a[..., others], b[..., others])
    assert not np.array_equal(after[0][..., units - 2], before[0][..., units - 2])


def _long_rows(mask, units, gate, first, rows, entries):
    m = mask.reshape(4, units, -1)
    m[gate, first:first + rows] = 0
    m[gate, first:first + rows, :entries] = 1


@pytest.mark.parametrize("name", ["h1", "2"])
def test_rows_that_only_rounds_can_hold(name):
    """Rows of 400 entries, 16 more than the most slots hold, three of a gate side by side: three rounds, and the recurrence takes them
    as it takes shorter ones, also where it is asked for."""
    H, G = 420, 410
    case = _case(1, False, 24, H, 5, 3, 32, 0, G)
    v = case.weights[(0, 0)]
    if name == "h1":
        _long_rows(v["M1h"], G, 1, 200, 3, 400)
        v["W1h"][G + 200:G + 203] *= 0.3
    else:
        _long_rows(v["M2"], H, 3, H - 3, 3, 400)
        v["W2"][4 * H - 3:] *= 0.3
    for plan in (B.LSTM_PLAN_AUTO, B.LSTM_PLAN_PERSISTENT):
        desc, _ = check_case(case, CSR, plan)
        assert "rec=persist_batched-hlstm-csr+ovf(s24," in desc, desc


def test_rounds_of_a_matrix_packed_again_lstm():
    """The shorter direction is packed again for the other's slots: nothing of it is outside them any more."""
    case = _case(1, True, 24, 300, 5, 3, 192, 16)                                          # 12 slots and a round
    desc, _ = check_case(case, CSR)
    assert desc.count("+ovf(s12,") == 2 and desc.count(",r1") == 2, desc
    case.weights[(0, 1)]["Mh"] = _mask(np.random.default_rng(1), 300, 300, 208, 0)         # 14 slots
    desc, _ = check_case(case, CSR)
    assert desc.count("q16(s14,") == 2 and not re.search(r",r\d", desc), desc


def test_rounds_of_a_matrix_packed_again_hlstm():
    case = _case(1, True, 24, 300, 5, 3, 192, 40, 300)
    desc, _ = check_case(case, CSR)
    assert desc.count("+ovf(s12,") == 2 and desc.count(",r3") == 2, desc
    case.weights[(0, 1)]["M2"] = _mask(np.random.default_rng(1), 300, 300, 240, 0)         # 16 slots: all four matrices
    desc, _ = check_case(case, CSR)
    assert desc.count("csr(s16,") == 2 and not re.search(r",r\d", desc), desc


@pytest.mark.parametrize("H,G,Bn,extra,shape", [
    (310, 305, 10, 7, "u3,b2,r1"),
    (310, 320, 18, 40, "u3,b2,r3"),
    (320, 310, 24, 48, "u3,b4,r3"),
    (382, 382, 29, 16, "u3,b4,r1"),
])
def test_hlstm_sixteen_slots_of_three_units(H, G, Bn, extra, shape):
    """The form whose weights leave the fewest registers for the entries outside its slots."""
    desc, _ = check_case(_case(2, True, 24, H, 5, Bn, 256, extra, G), CSR)
    assert desc.count(f"rec=persist_batched-hlstm-csr+ovf(s16,{shape})") == 4, desc
