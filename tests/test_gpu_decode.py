"""GPU parity of decode attention (the decoding phase that consumes the
cache) over the full and the compacted cache, through the C ABI, against the
fp64 oracle.  Small workloads are compared on every unit; the 150,528-token
trajectory is checked on sampled units inside its full-size test."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("name", ["ragged", "tiles", "g1w1", "g8w64", "g16w32", "beta_tiny", "beta_one"])
def test_decode_small_all_units(torch_cuda, name):
    from tests import gpu_harness as H
    from tests.test_gpu_parity import SMALL
    w = SMALL[name]
    H.log(f"decode small {name}: L={w.total_tokens} seqs={len(w.seqs)} G={w.group}")
    case = H.Case(w)
    res = case.run()
    dec = H.run_decode(case)
    worst = 0.0
    for layer in range(w.n_layers):
        for kv in range(w.n_kv_heads):
            for s in range(case.lay.n_seqs):
                worst = max(worst, H.compare_decode(case, res, dec, layer, kv, s))
    H.log(f"decode small {name}: worst error / tolerance {worst:.3g}")
    if name == "beta_tiny":
        # a sequence whose budget is 0 has an empty compacted cache: out = 0
        empty = [s for s in range(case.lay.n_seqs) if case.cu_budget[s + 1] == case.cu_budget[s]]
        assert empty and not dec[2][:, empty].any()


def test_decode_config0_all_units(torch_cuda):
    from tests import gpu_harness as H
    from paper_2603_00188_amd import workload as W
    case = H.Case(W.config(0))
    res = case.run()
    dec = H.run_decode(case)
    for kv in range(case.w.n_kv_heads):
        H.compare_decode(case, res, dec, 0, kv, 0)
    # attention over the compacted cache differs from the full one (20 % of the rows)
    assert not np.allclose(dec[1], dec[2])


@pytest.mark.parametrize("lengths,layers", [((512, 1, 130, 17), 2), ((513, 1, 130, 17), 2), ((512, 16, 40, 5), 48)])
def test_decode_one_work_group_per_sequence(torch_cuda, lengths, layers):
    """The longest sequence that one work-group takes whole (512 rows), one row
    more, and a batch of too many such sequences for one round (4 x 96 units):
    every sequence of sampled units, full and compacted cache, same tolerance."""
    from tests import gpu_harness as H
    from tests.test_gpu_parity import T, _small
    w = _small([[(T, n)] for n in lengths], G=3, Hkv=2, window=1, beta=(1, 3), layers=layers)
    H.log(f"decode lengths {lengths} x {layers} layers")
    case = H.Case(w)
    res = case.run()
    dec = H.run_decode(case)
    for layer in (0, layers - 1):
        for kv in range(w.n_kv_heads):
            for s in range(case.lay.n_seqs):
                H.compare_decode(case, res, dec, layer, kv, s)
