"""Shapes without a compile-time configuration (tt_flex.h): forward, backward and fused step against the oracle at the
sizes where the kernels change course: ranks and factors off every tile edge, hot rows (lists sorted and merged, runs added
up by a whole workgroup), several tiles and windows per slice, several workgroups per slice, a cache, no workspace."""
import numpy as np
import pytest
import torch

from oracle import tt_oracle as ora
from paper_2101_11714_amd import binding as B
from paper_2101_11714_amd import workloads as W
from gpu_util import DeviceTable, assert_close, dev

pytestmark = pytest.mark.gpu


def _table(m, n, r, bags, longest, seed, hot=0.3):
    """Bags of 0..longest positions; a share of the positions are one hot row, another share one slice of the second core."""
    t = W.TableShape(m[0] * m[1] * m[2] - 1, m, n, (1, r[0], r[1], 1))
    rng = np.random.default_rng(seed)
    lens = rng.integers(0, longest + 1, bags) if longest > 1 else np.ones(bags, dtype=np.int64)
    lens[0] = max(lens[0], 1)
    off = np.zeros(bags + 1, dtype=np.int64)
    np.cumsum(lens, out=off[1:])
    L = int(off[-1])
    idx = rng.integers(0, t.num_rows, L).astype(np.int64)
    if hot:
        idx[rng.random(L) < hot] = idx[0]
        share = rng.random(L) < 0.2
        i1, i3 = rng.integers(0, m[0], L), rng.integers(0, m[2] - 1, L)
        idx[share] = ((i1 * m[1] + m[1] // 2) * m[2] + i3)[share]
    batch = W.Batch(idx, off, rng.standard_normal((bags, t.dim)).astype(np.float32), (0.5 + rng.random(L)).astype(np.float32))
    return DeviceTable(W.Workload("flex", (t,), bags, (0, longest), "uniform", 0.0, "normal0.1", seed), batch=batch)


def _check(d, name, cache=None, keys=None, crow=None):
    b = d.batch
    out = ora.fwd(d.oshape, d.cores, b.indices, b.offsets, alpha=b.alpha, **({"cache_keys": keys, "cache_rows": crow} if cache else {}))
    assert_close(d.fwd(cache=cache), out, name + " forward")
    rg, rc = ora.bwd(d.oshape, d.cores, b.indices, b.offsets, b.grad_output, alpha=b.alpha, **({"cache_keys": keys} if cache else {}))
    start = [torch.full_like(x, 0.25) for x in d.g]
    dg, dc = d.bwd(cache=cache, grad_cores=[x.clone() for x in start])
    new = d.bwd_sgd(0.05, cache=cache)
    for k in range(3):
        assert_close(dg[k].cpu().numpy() - 0.25, rg[k], "%s dG%d" % (name, k + 1))
        assert_close(new[k].cpu().numpy(), ora.sgd(d.cores[k], rg[k], 0.05), "%s core %d" % (name, k + 1))
    if cache:
        assert_close(dc.cpu().numpy()[:cache.K], rc, name + " dCache")
        assert_close(cache.rows.cpu().numpy()[:cache.K], ora.sgd(crow, rc, 0.05), name + " cache lines")
    else:
        again = d.bwd_sgd(0.05)
        assert all(torch.equal(x, y) for x, y in zip(new, again))


@pytest.mark.parametrize("n,r", [((4, 4, 4), (16, 16)), ((4, 4, 4), (8, 8)), ((2, 4, 4), (24, 24)), ((2, 2, 4), (48, 48)),
                                 ((4, 4, 8), (16, 16)), ((3, 2, 5), (4, 7)), ((1, 1, 1), (1, 1)), ((16, 1, 16), (64, 3)),
                                 ((1, 64, 1), (5, 64)), ((2, 4, 8), (64, 64)), ((5, 3, 7), (17, 33)), ((4, 2, 4), (33, 15)),
                                 ((8, 3, 6), (50, 50)), ((2, 4, 1), (33, 33)), ((3, 2, 3), (64, 64))])
def test_shapes_off_the_tile_edges(n, r):
    _check(_table((7, 6, 9), n, r, 300, 5, 41), "n %s r %s" % (n, r))


def test_one_index_per_bag_no_hot_row():
    _check(_table((40, 50, 60), (2, 4, 4), (24, 24), 1500, 1, 42, hot=0), "one index per bag")


@pytest.mark.parametrize("bags,longest", [(2100, 2), (3300, 7)])
def test_windows_and_several_workgroups_per_slice(bags, longest):
    # few slices: lists beyond a window of 1024 - 3072 entries; 2,100 and about 11,500 positions: one and two workgroups per slice
    _check(_table((5, 2, 6), (2, 2, 3), (5, 6), bags, longest, 43, hot=0.2), "%d bags" % bags)


# 60,000 positions of the first shape take one pass in 45 MB and whole segments of 8,192 in less; of the second, 4.3 KB each,
# a segment of 8,192 takes more than 32 MiB and is cut into pieces of 2,048.
@pytest.mark.parametrize("n,r,bags,longest,sizes", [((2, 4, 4), (24, 24), 20_000, 6, (32 << 20, 38 << 20)), ((16, 1, 16), (64, 3), 3500, 12, (18 << 20, 32 << 20, 64 << 20))])
def test_several_passes_add_in_the_same_order(n, r, bags, longest, sizes):
    d = _table((5, 40, 6), n, r, bags, longest, 47, hot=0.1)
    _check(d, "n %s, %d positions" % (n, d.L))
    full = B.bwd_sgd_workspace_bytes(d.shape, d.L, d.n_bags)
    assert full > max(sizes)
    got = []
    for size in (full,) + sizes:
        ws = torch.full((size,), 0x7F, dtype=torch.uint8, device=dev())
        new = [torch.full_like(x, float("nan")) for x in d.g]
        B.tt_emb_bwd_sgd(d.shape, d.g, new, d.idx, d.off, d.n_bags, d.go, 0.05, alpha=d.alpha, workspace=ws)
        dg = [torch.full_like(x, 0.25) for x in d.g]
        B.tt_emb_bwd(d.shape, d.g, d.idx, d.off, d.n_bags, d.go, dg, alpha=d.alpha, workspace=ws)
        torch.cuda.synchronize()
        got.append(new + dg)
    for other in got[1:]:
        assert all(torch.equal(x, y) for x, y in zip(got[0], other))


# positions, and whether the plain kernels take them, on either side of where they stop being ahead
@pytest.mark.parametrize("n,r,L", [((1, 64, 1), (5, 64), 1), ((1, 64, 1), (5, 64), 130), ((1, 64, 1), (5, 64), 140), ((2, 8, 8), (33, 33), 20),
                                   ((2, 8, 8), (33, 33), 30), ((4, 12, 1), (2, 48), 50)])
def test_short_streams_of_many_turns(n, r, L):
    d = _table((7, 6, 9), n, r, L, 1, 48)
    _check(d, "n %s, %d positions" % (n, L))
    # the same bits from the static scratch memory
    full, static = d.bwd_sgd(0.05), [torch.full_like(x, float("nan")) for x in d.g]
    B.tt_emb_bwd_sgd_static(d.shape, d.g, static, d.idx, d.off, d.n_bags, d.go, 0.05, alpha=d.alpha)
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(full, static))


def test_short_stream_without_room_for_the_plain_kernels():
    # one position: 492,544 bytes for the kernels of longer streams, 494,336 for the plain ones, which keep the gradients of the cores
    d = _table((7, 6, 9), (1, 64, 1), (5, 64), 1, 1, 49)
    b = d.batch
    rg, _ = ora.bwd(d.oshape, d.cores, b.indices, b.offsets, b.grad_output, alpha=b.alpha)
    new = [torch.full_like(x, float("nan")) for x in d.g]
    ws = torch.full((493_000,), 0x7F, dtype=torch.uint8, device=dev())
    B.tt_emb_bwd_sgd(d.shape, d.g, new, d.idx, d.off, d.n_bags, d.go, 0.05, alpha=d.alpha, workspace=ws)
    torch.cuda.synchronize()
    for k in range(3):
        assert_close(new[k].cpu().numpy(), ora.sgd(d.cores[k], rg[k], 0.05), "core %d" % (k + 1))


def test_slices_without_positions_are_copied():
    d = _table((5, 400, 6), (2, 4, 4), (12, 12), 60, 3, 44)
    _check(d, "sparse")


@pytest.mark.parametrize("bags", [300, 13_000])
def test_with_cache(bags):
    d = _table((7, 6, 9), (2, 4, 4), (24, 24), bags, 5, 45)     # one pass, two passes
    rows, counts = np.unique(d.batch.indices, return_counts=True)
    cache, _, _ = d.build_cache(20, rows.astype(np.int64), counts.astype(np.int64))
    keys = ora.cache_select(rows, counts, 20)
    crow = cache.rows.cpu().numpy()[:20].copy()
    _check(d, "cache", cache, keys, crow)


def test_no_workspace_takes_the_plain_kernels():
    d = _table((7, 6, 9), (2, 4, 4), (24, 24), 200, 3, 46)
    dg = [torch.zeros_like(x) for x in d.g]
    B.tt_emb_bwd(d.shape, d.g, d.idx, d.off, d.n_bags, d.go, dg, alpha=d.alpha)
    torch.cuda.synchronize()
    rg, _ = ora.bwd(d.oshape, d.cores, d.batch.indices, d.batch.offsets, d.batch.grad_output, alpha=d.batch.alpha)
    for k in range(3):
        assert_close(dg[k].cpu().numpy(), rg[k], "no workspace dG%d" % (k + 1))


# ranks in eights with one turn over j1 and the columns (every load of a position at once): 8 to 32, two and four rows j1, one, two and four
# columns per lane, lanes without columns, outputs beyond a wave and of odd number; next to them the first ranks and columns that are not
@pytest.mark.parametrize("n,r", [((4, 4, 4), (8, 8)), ((2, 4, 4), (16, 16)), ((4, 4, 4), (24, 24)), ((2, 3, 5), (24, 20)), ((2, 2, 4), (32, 64)), ((4, 8, 8), (32, 32)),
                                 ((4, 3, 1), (16, 23)), ((2, 1, 2), (8, 2)), ((2, 4, 4), (40, 24)), ((2, 4, 8), (24, 65)), ((4, 4, 8), (20, 16)), ((3, 4, 4), (16, 16))])
def test_forward_with_ranks_in_eights(n, r):
    d = _table((7, 6, 9), n, r, 200, 70, 47, hot=0.1)
    b = d.batch
    assert_close(d.fwd(), ora.fwd(d.oshape, d.cores, b.indices, b.offsets, alpha=b.alpha), "n %s r %s" % (n, r))
