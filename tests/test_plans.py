"""CPU tests of the host plans of the score and decode calls, read from their
workspace sizes: (max, sum) partials of rows_pad window rows per score chunk, a
16-head partial per decode chunk."""
import os
import time

import numpy as np
import pytest

from paper_2603_00188_amd import stlite as S

pytestmark = pytest.mark.skipif(not os.path.exists(S.LIB_PATH), reason="libstlite.so not built")


def problem(lens, units=4, window=8, group=7):
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    return S.Problem(units, group, 1, window, cu, np.zeros(len(lens) + 1, np.int32), np.zeros((0, 3), np.int32),
                     S.budgets(cu, 1, 5), device="cpu")


def _aligned(n):
    return (n + 255) // 256 * 256


def score_waves(p):
    """(waves, padded rows) of the score's layout: 32-row blocks, two per wave."""
    blocks = -(-p.n_q_heads // p.n_kv_heads * p.window // 32)
    per_wave = 2 if blocks >= 2 else 1
    waves = 8 if blocks == 14 else -(-blocks // per_wave)
    return waves, waves * per_wave * 32


def score_chunks(p):
    """Key chunks of the score call over all sequences."""
    _, rows_pad = score_waves(p)
    n = p.workspace_size(S.CALL_SCORE_WINDOW) - _aligned(p.units * p.n_seqs * rows_pad * 4)
    return n // (p.units * rows_pad * 8)  # (the alignment is less than one chunk's rows)


def score_chunk_keys(p):
    """The least chunk length that gives that many."""
    n, lens = score_chunks(p), np.diff(p.h["cu_seqlens"])
    return next(c for c in range(64, 16385, 64) if (-(-lens // c)).sum() == n)


@pytest.mark.parametrize("units", [1, 4, 24, 112])
@pytest.mark.parametrize("window", [1, 8, 32, 64])
@pytest.mark.parametrize("tokens", [912, 8192, 30000, 150528])
def test_score_merge_is_no_longer_than_its_chunks(units, window, tokens):
    """A row's partials are merged one chunk after another at about a quarter of
    a tile each, so the best split of a sequence that fits one round balances
    the two: the merge costs no more than the tiles of a chunk, start included
    (6 tiles), by more than the rounding of the split, and a second round is
    only taken where the first one is full."""
    p = problem([tokens], units, window)
    n = score_chunks(p)
    tiles = -(-tokens // (64 * n))  # of a chunk, at least
    slots = 256 * min(3, max(1, 8 // score_waves(p)[0]))
    rounds = -(-n * units // slots)
    assert n / 4 <= rounds * (tiles + 6) + 2, (n, tiles, rounds)
    assert rounds == 1 or tokens * units > 64 * slots, (n, tiles, rounds)


def test_score_rounds_count_the_lds_limit():
    """One-wave groups: the 48 KB key ring lets three of them share a CU, so 112
    units x 3392 tokens are cut into at most 768 work-groups, one round."""
    p = problem([3392], 112, 1)
    assert score_chunks(p) * 112 <= 768


@pytest.mark.parametrize("call", [S.CALL_SCORE_WINDOW, S.CALL_DECODE_FULL])
def test_short_sequences_plan_quickly(call):
    """The plan of a call tries chunks up to the longest sequence, for every
    sequence: 256 sequences of 100 tokens leave two lengths to try, 256 of
    16,384 leave 128 or more, so their plan takes a small part of the time (the
    same before the search ended there)."""
    def best(lens):
        p = problem(lens)
        times = []
        for _ in range(20):
            t = time.perf_counter()
            p.workspace_size(call)
            times.append(time.perf_counter() - t)
        return min(times)
    assert best([100] * 256) < 0.5 * best([16384] * 256)


@pytest.mark.parametrize("call", [S.CALL_SCORE_WINDOW, S.CALL_DECODE_FULL, S.CALL_DECODE_COMPACT])
@pytest.mark.parametrize("lens", [[8], [64] * 3, [65, 8, 64], [100] * 256, [512, 9, 130], [600] * 7, [8192, 8], [8200]])
def test_plan_sizes_hold_every_chunk(call, lens):
    """Edges of the search's end: the workspace holds a partial of every chunk
    of every sequence (at least one chunk each)."""
    p = problem(lens, units=4, window=8)
    size = p.workspace_size(call)
    if call == S.CALL_SCORE_WINDOW:
        assert len(lens) <= score_chunks(p) <= sum(-(-n // 64) for n in lens)
    else:
        rows = lens if call == S.CALL_DECODE_FULL else [n // 5 for n in lens]
        per = p.units * 16 * 4  # a chunk's maxima, and as much again for its sums
        used = sum(r > 0 for r in rows)
        assert per * 130 * used <= size <= per * 130 * sum(-(-r // 64) for r in rows) + 3 * 256


def decode_chunks(p):
    """Chunks of the decode call over the full cache, all sequences."""
    return p.workspace_size(S.CALL_DECODE_FULL) // (p.units * 16 * 4 * 130)


@pytest.mark.parametrize("units", [1, 4, 8, 16, 112])
@pytest.mark.parametrize("rows", [912, 2048, 4096, 8192, 16384, 62720, 150528])
def test_decode_merge_is_no_longer_than_its_chunks(units, rows):
    """The combine merges 16 chunks of a sequence at a time, one batch after
    another at about four 64-row steps each: it costs no more than the steps of
    the chunks, start included (4 steps), by more than one batch."""
    n = decode_chunks(problem([rows], units, 1))
    steps = -(-rows // (64 * n))  # of a chunk, at least
    rounds = -(-n * units // 512)
    assert 4 * -(-n // 16) <= rounds * (steps + 4) + 4, (n, steps, rounds)
