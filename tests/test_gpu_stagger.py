"""GPU: the staggered decode schedule at its edges.

Ranges of one to a few blocks (prologue copies, the last two periods), ranges whose pieces are
one block each (a wave of one parity skips pieces and reloads its queries every block, the row
state starts afresh in every period), row counts at the edges of the 32-row tiles and both
parities of every start.  Every row against the oracle (derived bounds and the tolerance of
check_sequence).  A bad page id at any place of a sequence gives NaN rows for that sequence and
leaves the others alone.
"""

import numpy as np
import pytest
import torch

from paper_2602_10718_amd import workloads as wl
from gpu_common import runner, reference, check_sequence

pytestmark = pytest.mark.gpu

LENS = [1, 64, 65, 130, 63, 0, 200, 3, 64, 321]


@pytest.mark.parametrize("rows", [(1, 1), (16, 2), (17, 1), (32, 1), (33, 1), (64, 1), (40, 2)])
@pytest.mark.parametrize("parts", [1, 2, 3, 5, 19])
def test_short_ranges_and_one_block_pieces(rows, parts):
    H, q_len = rows
    lens = [n if n == 0 or n >= q_len else q_len for n in LENS]
    w = wl.custom(B=len(lens), H=H, q_len=q_len, seq_lens=lens, causal=q_len == 2, seed=91, n_new=1)
    run = runner(w, num_splits=parts)
    run.out.fill_(12345.0)
    run.step()
    torch.cuda.synchronize()
    assert not (run.out == 12345.0).any()
    qn, qr = w.queries()
    for b in range(len(lens)):
        if lens[b]:
            check_sequence(run, b, reference(w, b, qn, qr), label=f"stagger H{H} q{q_len} parts{parts}")
        else:
            assert (run.out[b] == 0).all() and torch.isneginf(run.lse[b]).all()


@pytest.mark.parametrize("H", [16, 64])
@pytest.mark.parametrize("place", [0, 1, 2, 3, 4, 7])
def test_bad_page_marks_its_sequence_only(H, place):
    w = wl.custom(B=3, H=H, q_len=1, seq_lens=[129, 64 * 7 + 5, 300], seed=92, n_new=0)
    run = runner(w, num_splits=1)
    run.step()
    good = (run.out.clone(), run.lse.clone())
    run.page_table[1, place] = w.num_pages
    run.step()
    torch.cuda.synchronize()
    assert torch.isnan(run.out[1]).all() and torch.isnan(run.lse[1]).all()
    for b in (0, 2):
        assert torch.equal(run.out[b], good[0][b]) and torch.equal(run.lse[b], good[1][b])


@pytest.mark.parametrize("H", [32, 64, 128])
@pytest.mark.parametrize("B,n", [(1, 700), (3, 1500), (9, 130)])
def test_fewer_parts_than_asked_for(H, B, n):
    """Batches with few blocks use fewer parts than num_splits (the merge of a part costs as much as several blocks):
    the same rows as with every sequence in one piece, up to the order of float32 sums (2^-16 of a row's largest
    output: some 200 terms of at most that size, 2^-24 each)."""
    lens = [n, n // 2 + 1, 0, 64][:B] + [n] * max(0, B - 4)
    w = wl.custom(B=B, H=H, q_len=1, seq_lens=lens, seed=93, n_new=0)
    one = runner(w, unsplit=True)
    one.step()
    for parts in (7, 8, 40, 1000):
        run = runner(w, num_splits=parts, cache=(one.kv_latent, one.kv_scale, one.k_rope))
        run.out.fill_(12345.0)
        run.step()
        torch.cuda.synchronize()
        a, b = run.out.double().reshape(-1, 512), one.out.double().reshape(-1, 512)
        assert ((a - b).abs().amax(1) <= 2.0 ** -16 * b.abs().amax(1)).all()
