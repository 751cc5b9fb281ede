"""GPU: consecutive bf16 layers of one width in one launch (persist_rows_bf16.hip), against the fp64 oracle with the tolerances
of parity_util, and the words that travel between its workgroups."""
import numpy as np
import pytest

from paper_1901_10997_amd import binding as B
from paper_1901_10997_amd import inputs
from parity_util import check_case, run_gpu
from test_gpu_graph import test_graph_replays_match_eager as graph_replays_match_eager

pytestmark = pytest.mark.gpu


def _case(L, D, H, T, Bn, k=0, bidir=False, keep=None):
    w = inputs.Workload(120, f"stack_L{L}_D{D}_H{H}_T{T}_B{Bn}", L, bidir, D, H, T, Bn, "bf16", min(0.2, 1.5 / np.sqrt(max(H, D))), keep, "uniform", 0)
    return inputs.make_case(w, H + Bn + k, random_state=True)


@pytest.mark.parametrize("L,D,H,T,Bn", [
    (2, 24, 3, 40, 2),        # less than a tile of units, seven words that fill up the last block
    (3, 33, 100, 40, 3),      # seven again
    (2, 64, 130, 33, 17),     # a row block and one row
    (5, 40, 203, 25, 33),     # groups of one XCD, five fill words
    (2, 64, 224, 1, 9),       # one step: every layer waits for the one below only
    (7, 20, 64, 50, 5),       # more layers than a launch takes
    (2, 31, 515, 20, 30),
    (2, 96, 900, 21, 18),     # rows in two sixteens per pass
    (2, 317, 1197, 12, 20),   # the compacted language model: part of W_x in LDS
    (2, 40, 1500, 12, 6),
    (3, 40, 384, 16, 150),    # several passes
])
def test_stack_matches_the_oracle(L, D, H, T, Bn):
    case = _case(L, D, H, T, Bn)
    desc, _ = check_case(case)
    if T > 2:
        assert "rows-stack" in desc, desc
    (a, _), (b, _) = run_gpu(case, cooperative=False), run_gpu(case, cooperative=True)
    for p, q in zip(a, b):
        np.testing.assert_array_equal(p, q)


@pytest.mark.parametrize("H,Bn", [(100, 5), (900, 18)])
def test_state_beyond_one_and_nan_stay_in_their_row(H, Bn):
    """h0 may have any value (it does not travel between workgroups); a NaN reaches every unit of its sequence and layers above,
    and no other row.  The stamps are a bit of the values."""
    case = _case(2, 40, H, 12, Bn)
    case.h0[:, 1] *= 9.0
    check_case(case)
    (y0, hT0, cT0), _ = run_gpu(case)
    b = Bn - 1
    case.c0[0, b, H // 2] = np.nan
    (y, hT, cT), desc = run_gpu(case)
    assert "rows-stack" in desc, desc
    assert np.isnan(y[1:, b]).all() and np.isnan(hT[:, b]).all() and np.isnan(cT[:, b]).all()
    others = np.arange(Bn) != b
    for got, ref in ((y, y0), (hT, hT0), (cT, cT0)):
        np.testing.assert_array_equal(got[:, others], ref[:, others])


def test_device_scope_only_gives_the_same_bits(monkeypatch):
    case = _case(4, 40, 256, 30, 8)
    a, desc = run_gpu(case)
    assert ",xcd)" in desc, desc
    monkeypatch.setenv("LSTM355_L2_HANDOVER", "0")
    b, _ = run_gpu(case)
    for p, q in zip(a, b):
        np.testing.assert_array_equal(p, q)


def test_masked_layer_in_the_stack_runs_apart():
    """A row-compressed layer has no place in a launch over dense ones: those by themselves, as before."""
    case = _case(3, 40, 300, 30, 6, keep=0.1)
    for l in (0, 2):
        case.weights[(l, 0)].update(Mx=None, Mh=None)
    desc, _ = check_case(case)
    assert "stack" not in desc and desc.count("rec=persist-mfma-rows(") == 2, desc


def test_stack_over_layers_of_another_width():
    """Widths 96, 200, 200, 200, 64: the three equal ones in one launch, between two that are not."""
    import torch
    widths, D, T, Bn = (96, 200, 200, 200, 64), 48, 30, 7
    rng = np.random.default_rng(5)
    bf = lambda a: torch.from_numpy(a.astype(np.float32)).bfloat16().float().numpy()
    weights = {}
    for l, H in enumerate(widths):
        d = D if l == 0 else widths[l - 1]
        weights[(l, 0)] = dict(Wx=bf(rng.uniform(-0.1, 0.1, (4 * H, d))), Wh=bf(rng.uniform(-0.1, 0.1, (4 * H, H))),
                               b=rng.uniform(-0.1, 0.1, 4 * H).astype(np.float32), Mx=None, Mh=None)
    x = torch.from_numpy(rng.standard_normal((T, Bn, D)).astype(np.float32)).cuda().bfloat16()
    outs = []
    for plan in (B.LSTM_PLAN_AUTO, B.LSTM_PLAN_STEPWISE):
        m = B.Lstm(len(widths), D, list(widths), False, B.LSTM_BF16)
        m.set_weights_from(weights)
        B.lstm_set_plan(m.handle, plan, 0)
        y, hT, cT = m.forward(x, None, None)
        outs.append([t.double().cpu().numpy().ravel() for t in (y, hT, cT)])
        desc = B.lstm_describe_plan(m.handle)
        assert desc.count("rows-stack") == (3 if plan == B.LSTM_PLAN_AUTO else 0), desc
        m.close()
    for a, b in zip(*outs):      # both round h to bf16 every step: an ulp of the operand, 2^-8, is the bf16 tolerance of parity_util
        assert np.linalg.norm(a - b) <= 2e-2 * np.linalg.norm(b)


@pytest.mark.parametrize("L,H,Bn", [(3, 96, 5), (4, 130, 9)])
def test_graph_replays(L, H, Bn):
    """(Narrow layers only: that test's weights of up to 0.3 make 900 units chaotic, 0.17 of the largest output apart from the oracle
    after twelve steps whichever kernel rounds h to bf16.)"""
    graph_replays_match_eager(L, False, 40, H, 12, Bn, "bf16", None, 0, "rows-stack")


@pytest.mark.parametrize("bidir,H,Bn,takes", [
    (False, 384, 256, "rows("),      # sixteen groups of one pass
    (False, 384, 384, "bf16;"),          # groups of two passes: the 32-row tiles
    (True, 384, 224, "rows("),       # two passes, both directions in a launch
    (True, 512, 384, "rows("),       # three
    (True, 512, 512, "bf16;"),           # four: the tiles, a launch per direction
])
def test_groups_of_rows_or_tiles(bidir, H, Bn, takes):
    w = inputs.Workload(121, f"rows_H{H}_B{Bn}", 1, bidir, 64, H, 6, Bn, "bf16", 1.5 / np.sqrt(H), None, "uniform", 0)
    desc, _ = check_case(inputs.make_case(w, H + Bn, random_state=True), oracle_cols=list(range(0, Bn, 13)) + [Bn - 1])
    assert desc.count("rec=persist-mfma-" + takes) == (2 if bidir else 1), desc


def test_workspace_of_a_larger_batch():
    """64 columns run as stacks and report more than 65, which do not: in a workspace made for 65 they run layer by layer."""
    import torch
    L, D, H, T, Bn = 6, 317, 800, 70, 64
    case = _case(L, D, H, T, Bn)
    dev = torch.device("cuda:0")
    m = B.Lstm(L, D, H, False, B.LSTM_BF16)
    m.set_weights_from(case.weights)
    x = torch.from_numpy(case.x).to(dev).to(torch.bfloat16)
    h0, c0 = torch.from_numpy(case.h0).to(dev), torch.from_numpy(case.c0).to(dev)
    need, larger = B.lstm_workspace_bytes(m.handle, T, Bn), B.lstm_workspace_bytes(m.handle, T, Bn + 1)
    assert need > larger
    outs = []
    for n, stacked in ((need, True), (larger, False)):
        ws = torch.empty(n, dtype=torch.uint8, device=dev)
        y, hT, cT = torch.empty((T, Bn, H), device=dev), torch.empty((L, Bn, H), device=dev), torch.empty((L, Bn, H), device=dev)
        B.lstm_forward(m.handle, T, Bn, x.data_ptr(), h0.data_ptr(), c0.data_ptr(), y.data_ptr(), hT.data_ptr(), cT.data_ptr(), ws.data_ptr(), n,
                       torch.cuda.current_stream().cuda_stream)
        B.lstm_check(m.handle)
        assert ("rows-stack" in B.lstm_describe_plan(m.handle)) == stacked
        outs.append([t.double().cpu().numpy() for t in (y, hT, cT)])
    m.close()
    for a, b in zip(*outs):      # both round h to bf16 every step: the bf16 tolerance of parity_util
        assert np.linalg.norm(a - b) <= 2e-2 * np.linalg.norm(b)


@pytest.mark.parametrize("L,bidir", [(70, False), (35, True)])
def test_more_initial_states_than_one_launch_lays_out(L, bidir):
    w = inputs.Workload(122, f"states_L{L}_{int(bidir)}", L, bidir, 16, 16, 5, 3, "bf16", 0.3, None, "uniform", 0)
    desc, _ = check_case(inputs.make_case(w, L, random_state=True))
    assert desc.count("rec=") - 1 <= desc.count("rec=persist-mfma-rows") > 20, desc   # (the binding's buffer cuts the rest off)
