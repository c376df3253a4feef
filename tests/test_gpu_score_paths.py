"""Which way a chunk of the window score's first pass takes, read from the
(offset, sum) pairs it leaves at the start of the workspace
([units][chunks][padded rows], log2 units): the lean pass gives the eight rows
of a group one common offset, the exact pass gives every row its own maximum.

The scores are compared with a float64 softmax, tolerance as in gpu_harness."""
import numpy as np
import pytest

from paper_2603_00188_amd import stlite as S
from tests.test_plans import score_chunks, score_waves

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def problem(lens, units, window, group):
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    return S.Problem(units, group, 1, window, cu, np.zeros(len(lens) + 1, np.int32), np.zeros((0, 3), np.int32),
                     S.budgets(cu, 1, 4))


def run(torch, p, q, k):
    """A [units][tokens] and the partials [units][chunks][padded rows][2]."""
    ws = torch.full((p.workspace_size(S.CALL_SCORE_WINDOW),), 0xFF, dtype=torch.uint8, device="cuda")
    a = torch.full((p.units, p.total_tokens), float("nan"), device="cuda")
    S.stlite_score_window(p, q, k, a, ws)
    torch.cuda.synchronize()
    shape = (p.units, score_chunks(p), score_waves(p)[1], 2)
    part = ws[:8 * int(np.prod(shape[:3]))].view(torch.float32).view(shape)
    return a.cpu().numpy(), part.cpu().numpy()


def reference(torch, p, q, k, unit, s):
    """float64 A of one sequence."""
    G, w = p.n_q_heads, p.window
    b, e = int(p.h["cu_seqlens"][s]), int(p.h["cu_seqlens"][s + 1])
    x = q[unit, s].double().reshape(G * w, 128) @ k[unit, b:e].double().T * 128 ** -0.5
    x = x.view(G, w, e - b)
    for i in range(w):
        x[:, i, e - b - w + i + 1:] = -torch.inf
    return (torch.softmax(x, -1).sum((0, 1)) / G).cpu().numpy()


def check(torch, p, q, k, a, unit, s):
    ref = reference(torch, p, q, k, unit, s)
    b, e = int(p.h["cu_seqlens"][s]), int(p.h["cu_seqlens"][s + 1])
    got = a[unit, b:e]
    err = np.abs(got - ref) / np.maximum(np.abs(ref), 1e-30)
    assert (err <= 1e-3).all(), f"unit {unit} seq {s}: {err.max():.3g} at {int(err.argmax())}"


@pytest.mark.parametrize("group,window", [(7, 1), (3, 1), (7, 37), (7, 61)])
def test_padding_rows_stay_out_of_the_offset(torch_cuda, group, window):
    """Rows that do not fill their group of eight, every logit of the sequence
    some 90 log2 units below 0: the group's offset is its real rows' maximum (a
    padding row's logits are 0), so the sums stay in range and the lean pass's
    one offset per group is kept."""
    torch = torch_cuda
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    p = problem([4096], 2, window, group)
    line = torch.randn((128,), generator=gen, device="cuda")
    line /= line.norm()
    q = (30.0 * line + 0.05 * torch.randn((2, 1, group, window, 128), generator=gen, device="cuda")).to(torch.bfloat16)
    k = (-24.0 * line + 0.05 * torch.randn((2, 4096, 128), generator=gen, device="cuda")).to(torch.bfloat16)
    a, part = run(torch, p, q, k)
    rows = group * window
    assert rows % 8 != 0
    for unit in range(2):
        check(torch, p, q, k, a, unit, 0)
        last = part[unit, :, rows // 8 * 8:rows, 0]  # the group with padding rows
        assert (last == last[:, :1]).all() and (last < -60).all(), last[:, :4]
