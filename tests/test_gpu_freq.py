"""The access tracker's counting kernel for long streams, at the edges of its chunks and with tables too small for the rows."""

from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2101_11714_amd import binding as B
from gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,rows,capacity", [(16_384, 3, 64), (16_385, 5000, 1 << 14), (17_409, 17_409, 1 << 15), (20_000, 64, 64), (20_001, 300, 64),
                                             (40_000, 20_000, 1 << 12)])
def test_long_streams(L, rows, capacity):
    rng = np.random.default_rng(L + rows)
    idx = rng.integers(0, rows, L).astype(np.int64) * 7919 + 11
    idx[: L // 4] = 11                                                       # a hot row
    freq = B.Freq(capacity, dev())
    B.tt_freq_reset(freq)
    true = {}
    for part in (idx, idx[::-1].copy()):
        B.tt_freq_update(freq, torch.from_numpy(part).to(dev()))
    for r, c in zip(*np.unique(idx, return_counts=True)):
        true[int(r)] = 2 * int(c)
    got_r, got_c = (torch.empty(capacity, dtype=torch.int64, device=dev()) for _ in range(2))
    n_out = torch.zeros(1, dtype=torch.int64, device=dev())
    B.tt_freq_export(freq, got_r, got_c, n_out)
    torch.cuda.synchronize()
    n, stats = int(n_out.item()), freq.stats.cpu().numpy()
    r, c = got_r[:n].cpu().numpy(), got_c[:n].cpu().numpy()
    assert np.unique(r).size == n == stats[0] == min(len(true), capacity)
    assert int(c.sum()) + int(stats[1]) == 2 * L                             # every access is counted or reported dropped
    # a row that is in the table has all of its accesses: none is ever taken out, and where it is full none comes in
    assert all(b == true[int(a)] for a, b in zip(r, c))


def test_padding_of_a_long_stream_is_in_no_rows_count():
    # -1 is no row (and, as a key, the counting kernel's mark of a free entry): every chunk has some before, between and after its rows
    rng = np.random.default_rng(5)
    idx = rng.integers(0, 900, 20_001).astype(np.int64)
    idx[rng.random(idx.size) < 0.3] = -1
    idx[:50] = -1
    freq = B.Freq(1 << 12, dev())
    B.tt_freq_reset(freq)
    B.tt_freq_update(freq, torch.from_numpy(idx).to(dev()))
    got_r, got_c = (torch.empty(freq.capacity, dtype=torch.int64, device=dev()) for _ in range(2))
    n_out = torch.zeros(1, dtype=torch.int64, device=dev())
    B.tt_freq_export(freq, got_r, got_c, n_out)
    n, stats = int(n_out.item()), freq.stats.cpu().numpy()
    order = np.argsort(got_r[:n].cpu().numpy())
    rows, counts = np.unique(idx[idx >= 0], return_counts=True)
    assert np.array_equal(got_r[:n].cpu().numpy()[order], rows) and np.array_equal(got_c[:n].cpu().numpy()[order], counts)
    assert stats[0] == rows.size and stats[1] == 0
