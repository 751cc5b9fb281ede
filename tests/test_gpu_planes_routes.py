"""GPU: what holds for every exchanging kernel and every captured forward, for the kernels on fp16 planes and for those whose shapes
they took over: the hand-over through one XCD's L2, bounded waits, replays of a graph."""
import numpy as np
import pytest

from oracle import lstm_oracle as orc
from paper_1901_10997_amd import binding as B
from paper_1901_10997_amd import inputs
from parity_util import check_case, compare, run_gpu

pytestmark = pytest.mark.gpu

DENSE, CSR, AUTO = B.LSTM_FMT_DENSE_MASKED, B.LSTM_FMT_ROW_COMPRESSED, B.LSTM_PLAN_AUTO


def _wl(cid, L, bidir, D, H, T, Bn, keep=None, a=0.1):
    return inputs.Workload(cid, f"planes_L{L}_D{D}_H{H}_T{T}_B{Bn}", L, bidir, D, H, T, Bn, "f32", a, keep, "uniform")


@pytest.mark.parametrize("w,fmt,want", [
    (inputs.shrink(inputs.c4(), T=60), CSR, "rec=persist_batched-q16"),          # the kept entries, one batch group per XCD
    (inputs.shrink(inputs.c4(), T=60), B.LSTM_FMT_AUTO, ",xcd,split)"),
    (_wl(97, 1, True, 64, 800, 40, 16), DENSE, ",xcd,split)"),
    (_wl(97, 2, True, 64, 200, 40, 16), DENSE, ",xcd)"),                         # the fp32 instruction
])
def test_l2_handover_off_gives_the_same_bits(w, fmt, want, monkeypatch):
    case = inputs.make_case(w, 1)
    on, desc_on = run_gpu(case, fmt, cooperative=False)
    monkeypatch.setenv("LSTM355_L2_HANDOVER", "0")
    off, desc_off = run_gpu(case, fmt, cooperative=False)
    monkeypatch.delenv("LSTM355_L2_HANDOVER")
    assert desc_on == desc_off and all(want in d for d in desc_on.split(";") if d), desc_on
    for a, b in zip(on, off):
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32))


def test_expired_waits_are_reported_and_nothing_hangs(monkeypatch):
    """A bound of one poll: the forward is right or reports LSTM_ERR_TIMEOUT, and returns either way."""
    families = [(_wl(70, 1, True, 48, 200, 30, 12), lambda d: "rec=persist-dense-f32(t" in d and ",split)" not in d),
                (_wl(70, 1, True, 48, 400, 30, 12), lambda d: ",split)" in d)]
    monkeypatch.setenv("LSTM355_SPIN_LIMIT", "1")
    for w, route in families:
        case = inputs.make_case(w, 0, random_state=True)
        try:
            gpu, desc = run_gpu(case, DENSE, AUTO)
        except B.LstmError as e:
            assert e.code == B.LSTM_ERR_TIMEOUT
            continue
        assert route(desc), desc
        compare(gpu, orc.forward_case(case), "f32", w.name)
    monkeypatch.delenv("LSTM355_SPIN_LIMIT")
    for w, route in families:
        desc, _ = check_case(inputs.make_case(w, 0, random_state=True), DENSE, AUTO)
        assert route(desc), desc


@pytest.mark.parametrize("L,bidir,D,H,T,Bn,keep", [(2, True, 640, 400, 40, 16, None), (1, False, 1032, 600, 30, 20, 0.3)])
def test_graph_replays_match_eager(L, bidir, D, H, T, Bn, keep):
    """Projection and recurrence on planes, recorded once: replays with input rows that have no plane form, with a state beyond 1 and
    without either give the eager forward's bits, in any order."""
    import torch
    w = _wl(95, L, bidir, D, H, T, Bn, keep, a=0.05)
    case = inputs.make_case(w, 2, random_state=True)
    m = B.Lstm(L, D, H, bidir, B.LSTM_F32)
    m.set_weights_from(case.weights, DENSE)
    dev = torch.device("cuda:0")
    x0, h0, c0 = (torch.from_numpy(v).to(dev) for v in (case.x, case.h0, case.c0))
    x1, h1 = x0.clone(), h0.clone()
    x1.view(-1, D)[::7, 3] = 1e7
    x1.view(-1, D)[5, 9] = float("inf")
    h1[0, 2, 5] = 30.0
    sets = [(x0, h0), (x1, h0), (x0, h1), (x1, h1)]
    eager = [[t.cpu().numpy() for t in m.forward(x, h, c0)] for x, h in sets]
    desc = B.lstm_describe_plan(m.handle)
    assert all("proj=dense-split" in d and ",split)" in d for d in desc.split(";") if d), desc
    xs, hs = x0.clone(), h0.clone()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        outs = m.forward(xs, hs, c0, check=False)
    for k in (0, 1, 0, 2, 3, 0, 0, 1, 1):
        xs.copy_(sets[k][0])
        hs.copy_(sets[k][1])
        for o in outs:
            o.fill_(3.0)
        g.replay()
        torch.cuda.synchronize()
        B.lstm_check(m.handle)
        for want, got in zip(eager[k], outs):
            assert np.array_equal(want, got.cpu().numpy(), equal_nan=True), k
        again = m.forward(*sets[3 - k], c0)
        assert all(np.array_equal(a, b.cpu().numpy(), equal_nan=True) for a, b in zip(eager[3 - k], again)), k
    m.close()
