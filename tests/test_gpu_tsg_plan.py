"""The TSG call's first launch: the historical-token plan over many sequences
and frames, and the whole gate of a batch without any history.

Tolerances are those of the parity comparison (gpu_harness); the routes of a
batch without history are compared bit for bit.
"""
import numpy as np
import pytest

from paper_2603_00188_amd import workload as W

pytestmark = pytest.mark.gpu

F, T = W.FRAME, W.TEXT


@pytest.fixture(scope="module")
def torch_cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _batch(frames_per_seq, layers=1):
    """One sequence per entry: that many 3 x 5 frames, each followed by text."""
    seqs = [tuple([(T, 9)] + [s for i in range(n) for s in ((F, 3, 5), (T, 2 + i % 3))]) for n in frames_per_seq]
    return W.Workload("plan", layers, 4, 2, 4, (1, 4), tuple(seqs), W.Redundancy(frac=(0.1, 0.3), n_rects=(1, 1)),
                      ((1, 2), (1, 2)), seed=5)


@pytest.mark.parametrize("frames", [(3, 0, 1, 70, 2, 1, 0, 130, 5), (2,), (1, 1, 4)])
def test_plan_over_sequences(torch_cuda, frames):
    """More sequences than waves of a work-group, sequences of more frames than
    lanes, and sequences without frames or history between them."""
    from tests import gpu_harness as H
    w = _batch(frames)
    H.log(f"tsg plan {frames}: L={w.total_tokens}")
    case = H.Case(w)
    res = case.run()
    for kv in range(w.n_kv_heads):
        for s in range(case.lay.n_seqs):
            H.compare_unit(case, res, 0, kv, s)


@pytest.mark.parametrize("frames", [(1,), (0, 1, 1, 0, 1), (0, 0)])
def test_gate_without_history(torch_cuda, frames):
    """Without history the gate is open everywhere, rho is 0 and tau NaN, the
    same bits as from the two halves of the call."""
    import torch
    from tests import gpu_harness as H
    from paper_2603_00188_amd import stlite as S
    case = H.Case(_batch(frames, layers=3))
    p, o = case.prob, case.out
    outs = []
    for split in (False, True):
        o.rho.fill_(float("nan"))
        o.tau.fill_(7.0)
        o.gate.fill_(0xAB)
        if split:
            S.stlite_tsg_rho(p, case.dk, o.rho, o.ws_tsg)
            S.stlite_tsg_threshold(p, o.rho, o.tau, o.gate, o.ws_tsg)
        else:
            S.stlite_tsg_gate(p, case.dk, o.rho, o.tau, o.gate, o.ws_tsg)
        torch.cuda.synchronize()
        outs.append([x.cpu().numpy().copy() for x in (o.rho.view(torch.int32), o.tau.view(torch.int32), o.gate)])
    rho, tau, gate = outs[0]
    assert (rho == 0).all() and (gate == 1).all() and np.isnan(tau.view(np.float32)).all()
    for a, b in zip(*outs):
        assert np.array_equal(a, b)
    o.gate.fill_(0xAB)  # rho and tau are optional
    S.stlite_tsg_gate(p, case.dk, None, None, o.gate, o.ws_tsg)
    torch.cuda.synchronize()
    assert (o.gate.cpu().numpy() == 1).all()
