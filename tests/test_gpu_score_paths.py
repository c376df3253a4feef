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


# (group, window): row blocks, waves.  1: 1; 2: 1; 4: 2; 6: 3; 7: 4; 9: 5; 11: 6; 13: 7 (plain); 14: 8
# (two blocks split by key block between two waves); 16: 8
LAYOUTS = [(1, 1), (7, 8), (7, 16), (7, 24), (7, 32), (9, 32), (11, 32), (13, 32), (7, 64), (8, 64)]


@pytest.mark.parametrize("chunks", [5, 18])
@pytest.mark.parametrize("group,window", LAYOUTS)
def test_chunks_of_many_tiles(torch_cuda, group, window, chunks):
    """Chunks of 1024 keys (16 tiles; the plan of a batch of more than 256
    sequences), every wave layout, partials merged by pass 2 (5 chunks) and by
    the combine (18).  Keys aligned with a query of the last head, 150 log2 units
    above the rest:
      chunk 0, tiles 3, 7 and 10   the row's sum overflows: exact pass;
      chunk 1, first tile          the group's other rows underflow: exact pass;
      chunk 2                      none: lean pass;
      the last chunk, of 70 keys   the row of the last window position overflows
                                   in the second of two masked tiles: exact pass.
    """
    torch = torch_cuda
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    L = 1024 * (chunks - 1) + 70
    lens = [L] + [window + i % 5 for i in range(256)]
    p = problem(lens, 1, window, group)
    assert score_chunks(p) == chunks + 256, "the plan has to give chunks of 1024 keys"
    q = torch.randn((1, len(lens), group, window, 128), generator=gen, device="cuda").to(torch.bfloat16)
    k = torch.randn((1, p.total_tokens, 128), generator=gen, device="cuda")
    # (|q| about 11, logits in log2 units are q . k log2(e) / sqrt(128))
    first, last = (q[0, 0, group - 1, w].double() for w in (0, window - 1))
    spike = lambda x: (x / x.norm() * (150.0 / (x.norm() * 0.12751743))).float()
    spots = [200, 460, 700, 1024 + 10]
    k[0, spots] = spike(first)
    k[0, L - 2 if window > 1 else L - 1] = spike(last)
    k = k.to(torch.bfloat16)
    a, part = run(torch, p, q, k)
    for s in (0, 1, 2, 255, 256):
        check(torch, p, q, k, a, 0, s)
    assert not np.isnan(a).any()
    offset = part[0, :, :, 0]
    row, row_last = (group - 1) * window, group * window - 1
    assert offset[0, row] > 140, "overflow: the row's own maximum, far above the first tile's"
    assert offset[chunks - 1, row_last] > 140, "overflow behind the window's mask"
    assert offset[2, row] < 60
    rows = np.arange(group * window)
    group_of = rows[rows // 8 == row // 8]
    if len(group_of) > 1:
        others = group_of[group_of != row]
        assert (offset[1, others] < 100).all() and offset[1, row] > 140, "underflow: every row has its own maximum"
        assert (offset[2, group_of] == offset[2, row]).all(), "no spike: the group's common offset"
