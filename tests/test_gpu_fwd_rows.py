"""The forward pass over distinct rows (tt_rows_fwd.h, tt_emb_fwd_rows) at the edges of its windows, blocks and counting tiles:
one position, a window one short of full, full and one over, every row different, one row, one slice, empty and ragged bags,
weights, few and many slices.  Against the oracle and bit for bit against itself; the binding's tt_emb_fwd takes it by the rule
of tt_emb_fwd_rows_pays, and the wave per bag where the stream is captured or no scratch memory is to be had."""
import threading

import numpy as np
import pytest
import torch

from oracle import tt_oracle as ora
from paper_2101_11714_amd import binding as B
from paper_2101_11714_amd import workloads as W
from gpu_util import DeviceTable, assert_close, dev
from test_gpu_rows import SHAPES, _rows

pytestmark = pytest.mark.gpu


def _table(kind, n, R, L, n_bags, m=(30, 20, 40), alpha=True):
    t = W.TableShape(m[0] * m[1] * m[2] - 3, m, n, (1, R, R, 1))
    rng = np.random.default_rng([L, R, n[0]])
    off = np.concatenate([[0], np.sort(rng.integers(0, L + 1, n_bags - 1)), [L]]).astype(np.int64)
    batch = W.Batch(_rows(kind, t, L, rng), off, np.zeros((n_bags, t.dim), np.float32), (0.5 + rng.random(L)).astype(np.float32) if alpha else None)
    return DeviceTable(W.Workload("fwd rows", (t,), n_bags, (0, 9), "uniform", 0.0, "normal0.1", 5), batch=batch)


def _run(d):
    outs = []
    for fill in (0x7F, 0xFF):                                # what was in the scratch memory does not matter
        ws = torch.full((B.fwd_rows_workspace_bytes(d.shape, d.L, d.n_bags),), fill, dtype=torch.uint8, device=dev())
        out = torch.full((d.n_bags, d.t.dim), float("nan"), dtype=torch.float32, device=dev())
        B.tt_emb_fwd_rows(d.shape, d.g, d.idx, d.off, d.n_bags, out, ws, alpha=d.alpha)
        torch.cuda.synchronize()
        outs.append(out)
    assert torch.equal(*outs)
    return outs[0].cpu().numpy()


@pytest.mark.parametrize("n,R", SHAPES)
@pytest.mark.parametrize("kind,L,n_bags,m", [("uniform", 1, 3, (30, 20, 40)), ("second digit", 511, 40, (30, 20, 40)), ("second digit", 513, 1, (30, 20, 40)),
                                             ("uniform", 5000, 700, (30, 20, 40)), ("hot row", 9000, 300, (30, 20, 40)), ("one row", 3000, 17, (30, 20, 40)),
                                             ("uniform", 6001, 900, (3, 1024, 5)), ("uniform", 4100, 2000, (900, 1, 700))])
def test_forward_over_distinct_rows(n, R, kind, L, n_bags, m):
    d = _table(kind, n, R, L, n_bags, m)
    b = d.batch
    ref = ora.fwd(d.oshape, d.cores, b.indices, b.offsets, alpha=b.alpha)
    assert_close(_run(d), ref, kind)


def _captured(call):
    """A graph of one call, recorded on a stream of its own."""
    side, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(g, stream=side):
        call()
    return g


# either side of every limit, bags of one position and of several, and of the counting pass's tiles (131,072)
@pytest.mark.parametrize("n,R,L,n_bags", [((4, 4, 4), 32, 40_960, 40_960), ((4, 4, 4), 64, 40_960, 40_960), ((2, 2, 4), 32, 131_072, 9000),
                                          ((4, 4, 4), 32, 28_672, 9000), ((4, 4, 4), 64, 12_288, 3000), ((2, 2, 4), 64, 14_336, 14_336)])
def test_the_binding_takes_it_by_the_rule(n, R, L, n_bags):
    for L, n_bags, pays in ((L - 1, min(n_bags, L - 1), False), (L, n_bags, True)):
        d = _table("hot row", n, R, L, n_bags, m=(200, 200, 50), alpha=False)
        assert B.fwd_rows_pays(d.shape, L, n_bags) == pays and not B.fwd_rows_pays(d.shape, L, n_bags, 10)
        out = d.fwd()
        assert_close(out, ora.fwd(d.oshape, d.cores, d.batch.indices, d.batch.offsets), str((n, R, L)))
        old = B.set_fast_path(2)
        wave = d.fwd()
        B.set_fast_path(old)
        assert np.array_equal(out, _run(d) if pays else wave)
        got = torch.full((n_bags, d.t.dim), float("nan"), dtype=torch.float32, device=dev())
        g = _captured(lambda: B.tt_emb_fwd(d.shape, d.g, d.idx, d.off, d.n_bags, got))
        for _ in range(3):
            got.fill_(float("nan"))
            g.replay()
            torch.cuda.synchronize()
            assert np.array_equal(got.cpu().numpy(), wave)


def test_without_room_for_scratch_memory_the_wave_per_bag_runs():
    d = _table("hot row", (4, 4, 4), 32, 60_000, 9000, m=(200, 200, 50))
    assert B.fwd_rows_pays(d.shape, d.L, d.n_bags)
    old = B.set_fast_path(2)
    wave = d.fwd()
    B.set_fast_path(old)
    out = torch.full((d.n_bags, d.t.dim), float("nan"), dtype=torch.float32, device=dev())
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    try:                                                     # (room for a call's own tensors and no more)
        torch.cuda.set_per_process_memory_fraction(torch.cuda.memory_reserved() / torch.cuda.get_device_properties(0).total_memory)
        B.tt_emb_fwd(d.shape, d.g, d.idx, d.off, d.n_bags, out, alpha=d.alpha)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert np.array_equal(out.cpu().numpy(), wave) and not np.array_equal(_run(d), wave)


def test_recorded_and_on_two_streams():
    # every call with scratch memory of its own: replayed three times with eager work between, and side by side
    d = _table("hot row", (2, 2, 4), 64, 20_000, 3000)
    ref = _run(d)
    ws = [torch.full((B.fwd_rows_workspace_bytes(d.shape, d.L, d.n_bags),), 0x7F, dtype=torch.uint8, device=dev()) for _ in range(2)]
    out = [torch.full((d.n_bags, d.t.dim), float("nan"), dtype=torch.float32, device=dev()) for _ in range(2)]

    def call(j):
        B.tt_emb_fwd_rows(d.shape, d.g, d.idx, d.off, d.n_bags, out[j], ws[j], alpha=d.alpha)

    g = _captured(lambda: call(0))
    for _ in range(3):
        out[0].fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out[0].cpu().numpy(), ref) and np.array_equal(d.fwd(), ref)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for _ in range(20):
        for j, s in enumerate(streams):
            with torch.cuda.stream(s):
                call(j)
    torch.cuda.synchronize()
    for o in out:
        assert np.array_equal(o.cpu().numpy(), ref)


def test_scratch_memory_that_is_too_small_is_refused():
    d = _table("uniform", (4, 4, 4), 32, 1000, 10)
    need = B.fwd_rows_workspace_bytes(d.shape, d.L, d.n_bags)
    out = torch.zeros((d.n_bags, d.t.dim), dtype=torch.float32, device=dev())
    for bytes_ in (need - 1, 0):
        with pytest.raises(B.TTError) as e:
            B.tt_emb_fwd_rows(d.shape, d.g, d.idx, d.off, d.n_bags, out, torch.empty(bytes_, dtype=torch.uint8, device=dev()), alpha=d.alpha)
        assert e.value.code == -4
    torch.cuda.synchronize()
    assert float(out.abs().max()) == 0.0


def test_scratch_for_a_longer_batch_is_enough():
    # 131,071 positions have shorter tiles, and so more counters, in the counting pass than 131,072
    d = _table("hot row", (2, 2, 4), 32, 131_071, 5000, m=(20, 1000, 40))
    ws = torch.empty(B.fwd_rows_workspace_bytes(d.shape, d.L + 1, d.n_bags), dtype=torch.uint8, device=dev())
    out = torch.full((d.n_bags, d.t.dim), float("nan"), dtype=torch.float32, device=dev())
    B.tt_emb_fwd_rows(d.shape, d.g, d.idx, d.off, d.n_bags, out, ws, alpha=d.alpha)
    assert_close(out.cpu().numpy(), ora.fwd(d.oshape, d.cores, d.batch.indices, d.batch.offsets, alpha=d.batch.alpha), "longer scratch")


def test_scratch_memory_leaves_captures_elsewhere_alone():
    # a batch scored on a stream of its own, from another thread and from the same one, while a graph is recorded
    d = _table("hot row", (4, 4, 4), 32, 60_000, 9000, m=(200, 200, 50), alpha=False)
    assert B.fwd_rows_pays(d.shape, d.L, d.n_bags)
    ref = _run(d)
    got = [torch.full((d.n_bags, d.t.dim), float("nan"), dtype=torch.float32, device=dev()) for _ in range(2)]
    count, errors = torch.zeros(100, device=dev()), []
    own, side, g = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.CUDAGraph()

    def score(out):
        try:
            with torch.cuda.stream(own):
                B.tt_emb_fwd(d.shape, d.g, d.idx, d.off, d.n_bags, out)
        except Exception as e:                               # (reported by the test's thread)
            errors.append(e)

    torch.cuda.synchronize()
    torch.cuda.empty_cache()                                 # the scratch memory has to come from the device
    with torch.cuda.graph(g, stream=side):
        count += 1
        t = threading.Thread(target=score, args=(got[0],))
        t.start()
        t.join()
        score(got[1])
    assert not errors
    torch.cuda.synchronize()
    for out in got:
        assert np.array_equal(out.cpu().numpy(), ref)
    for _ in range(3):
        g.replay()
        torch.cuda.synchronize()
    assert float(count.min()) == float(count.max()) == 3.0   # (recorded, not run, the first time)


# pooling by a part of a wave per bag, up to an average of six positions (exclusive), or by a wave
@pytest.mark.parametrize("n,R", [((2, 2, 4), 32), ((4, 4, 4), 32)])
@pytest.mark.parametrize("L,n_bags", [(1, 1), (5, 1), (6, 1), (101, 17), (102, 17), (599, 100), (600, 100), (40, 4097)])
def test_pooling_of_short_bags(n, R, L, n_bags):
    d = _table("hot row", n, R, L, n_bags)
    b = d.batch
    assert_close(_run(d), ora.fwd(d.oshape, d.cores, b.indices, b.offsets, alpha=b.alpha), "L %d n_bags %d" % (L, n_bags))


# one bag of nearly everything among empty ones and bags of 64 and 65: a whole wave's, a part's, a whole wave's
@pytest.mark.parametrize("n,R", [((2, 2, 4), 32), ((4, 4, 4), 32)])
def test_pooling_of_a_long_bag_among_short_ones(n, R):
    lens = np.zeros(1500, np.int64)
    lens[[3, 4, 5, 700, 1499]] = [64, 65, 1, 5000, 66]
    d = _table("hot row", n, R, int(lens.sum()), lens.size)
    off = np.concatenate([[0], lens.cumsum()])
    d.off, d.batch = torch.from_numpy(off).to(dev()), W.Batch(d.batch.indices, off, d.batch.grad_output, d.batch.alpha)
    assert d.L < 6 * lens.size
    assert_close(_run(d), ora.fwd(d.oshape, d.cores, d.batch.indices, off, alpha=d.batch.alpha), "long bag")


# long bags side by side among bags of one: shared out over waves, whose bags are as many as there are waves apart (the last wave has fewer)
@pytest.mark.parametrize("n,R", [((2, 2, 4), 32), ((4, 4, 4), 32)])
@pytest.mark.parametrize("n_bags,long", [(1001, 40), (1500, 200), (16, 33), (3, 64)])
def test_pooling_of_long_bags_side_by_side(n, R, n_bags, long):
    lens = np.ones(n_bags, np.int64)
    lens[n_bags // 3:n_bags // 3 + 16] = long
    empty = max(0, int(lens.sum()) // 5 - n_bags + 1)        # as many empty ones as make the batch a short one
    lens = np.concatenate([lens, np.zeros(empty, np.int64)])
    d = _table("hot row", n, R, int(lens.sum()), lens.size)
    off = np.concatenate([[0], lens.cumsum()])
    d.off, d.batch = torch.from_numpy(off).to(dev()), W.Batch(d.batch.indices, off, d.batch.grad_output, d.batch.alpha)
    assert d.L < 6 * lens.size
    assert_close(_run(d), ora.fwd(d.oshape, d.cores, d.batch.indices, off, alpha=d.batch.alpha), "%d bags" % n_bags)


# the same bags in a batch of long ones, of short ones and of hardly any: the same bits, whichever kernel pools them
@pytest.mark.parametrize("n,R", [((2, 2, 4), 32), ((4, 4, 4), 32)])
def test_a_bag_does_not_depend_on_the_length_of_the_others(n, R):
    lens = np.array([*range(41), 63, 64, 65, 66, 100, 131])
    d = _table("hot row", n, R, int(lens.sum()), lens.size)
    ref = None
    for empty in (0, 400, 1200):                             # on average 28, 2.9 and 1.05 positions
        at = np.sort(np.random.default_rng(empty).choice(lens.size + empty, lens.size, replace=False))
        every = np.zeros(lens.size + empty, np.int64)
        every[at] = lens
        off = np.concatenate([[0], every.cumsum()])
        d.off, d.n_bags, d.batch = torch.from_numpy(off).to(dev()), every.size, W.Batch(d.batch.indices, off, d.batch.grad_output, d.batch.alpha)
        out = _run(d)
        ref = out if ref is None else ref
        assert np.array_equal(out[at], ref) and not out[every == 0].any()
    assert_close(out, ora.fwd(d.oshape, d.cores, d.batch.indices, off, alpha=d.batch.alpha), str(n))


# rank 64: bags of ten and more, and of eight and more: either side of the limits of their own; rank 32 has none
@pytest.mark.parametrize("n,R,L,mean", [((4, 4, 4), 64, 8192, 10), ((2, 2, 4), 64, 8192, 10), ((4, 4, 4), 64, 10_240, 8), ((2, 2, 4), 64, 10_240, 8),
                                        ((4, 4, 4), 32, 28_672, 8), ((4, 4, 4), 32, 28_672, 32)])
def test_the_rule_for_long_bags(n, R, L, mean):
    for L, n_bags, pays in ((L - 1, L // mean - 1, False), (L, L // mean, True), (L, L // mean + 1, R == 32)):
        d = _table("hot row", n, R, L, n_bags, m=(200, 200, 50), alpha=False)
        assert B.fwd_rows_pays(d.shape, L, n_bags) == pays
        out = d.fwd()
        assert_close(out, ora.fwd(d.oshape, d.cores, d.batch.indices, d.batch.offsets), str((n, R, L)))
        old = B.set_fast_path(2)
        wave = d.fwd()
        B.set_fast_path(old)
        assert np.array_equal(out, _run(d) if pays else wave)
