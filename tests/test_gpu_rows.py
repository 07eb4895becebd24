"""Grouping by distinct row (tt_rows.h, tt_rows_pass.h) where it changes course: a hot row over several windows, slices of the
first and third core with more rows than one workgroup adds up (the last of several finishes them), slices without any row,
every row different, every position the same row, streams on either side of the window sizes, tables at the limits of the
passes.  Forward, gradients and fused
step against the oracle, and the step twice, bit for bit."""
import numpy as np
import pytest
import torch

from oracle import tt_oracle as ora
from paper_2101_11714_amd import binding as B
from paper_2101_11714_amd import workloads as W
from gpu_util import DeviceTable, assert_close, dev

pytestmark = pytest.mark.gpu

SHAPES = [((2, 2, 4), 32), ((2, 2, 4), 64), ((4, 4, 4), 32), ((4, 4, 4), 64)]


@pytest.fixture
def always_rows():
    old = B.set_fast_path(3)                       # groups whatever the number of positions
    yield
    B.set_fast_path(old)


def _rows(kind, t, L, rng):
    m1, m2, m3 = t.m
    i1, i2, i3 = rng.integers(0, m1, L), rng.integers(0, m2, L), rng.integers(0, m3, L)
    if kind == "first digit":                      # all rows in one slice of the first core: more than RW_PIECE of them
        i1[:] = m1 - 1
    elif kind == "third digit":
        i3[:] = 1
    elif kind == "second digit":                   # one slice of the second core: windows and tiles of one slice
        i2[:] = m2 - 1
    elif kind == "one row":
        i1[:], i2[:], i3[:] = 2, 1, 3
    idx = (i1 * m2 + i2) * m3 + i3
    if kind == "hot row":
        idx[rng.random(L) < 0.6] = idx[0]
    return np.minimum(idx, t.num_rows - 1).astype(np.int64)


def _table(kind, n, R, L, n_bags, seed, m=(30, 20, 40)):
    t = W.TableShape(m[0] * m[1] * m[2] - 3, m, n, (1, R, R, 1))
    rng = np.random.default_rng([seed, L])
    idx = _rows(kind, t, L, rng)
    cuts = np.sort(rng.integers(0, L + 1, n_bags - 1))
    off = np.concatenate([[0], cuts, [L]]).astype(np.int64)
    batch = W.Batch(idx, off, rng.standard_normal((n_bags, t.dim)).astype(np.float32), (0.5 + rng.random(L)).astype(np.float32))
    return DeviceTable(W.Workload("rows", (t,), n_bags, (0, 9), "uniform", 0.0, "normal0.1", seed), batch=batch)


def _check(d, name, ws=None, lists=True):
    assert B.fwd_uses_lists(d.shape, d.L, 0, True) == lists
    b = d.batch
    ws = ws if ws is not None else torch.full((B.bwd_sgd_workspace_bytes(d.shape, d.L, d.n_bags, 0),), 0x7F, dtype=torch.uint8, device=dev())
    steps = []
    for _ in range(2):
        out = torch.full((d.n_bags, d.t.dim), float("nan"), dtype=torch.float32, device=dev())
        t0 = torch.full((d.L, B.t0_floats(d.shape)), float("nan"), dtype=torch.float32, device=dev())
        new = [torch.full_like(x, float("nan")) for x in d.g]
        B.tt_emb_bwd_prepare(d.shape, d.idx, d.off, d.n_bags, workspace=ws, kept_t0=True)
        B.tt_emb_fwd_prepared(d.shape, d.g, d.idx, d.off, d.n_bags, out, ws, t0=t0, alpha=d.alpha)
        B.tt_emb_bwd_sgd(d.shape, d.g, new, d.idx, d.off, d.n_bags, d.go, 0.05, alpha=d.alpha, workspace=ws, t0=t0, prepared=True)
        torch.cuda.synchronize()
        steps.append([out, t0] + new)
    assert all(torch.equal(x, y) for x, y in zip(*steps))
    out, t0, new = steps[0][0], steps[0][1], steps[0][2:]
    assert_close(out.cpu().numpy(), ora.fwd(d.oshape, d.cores, b.indices, b.offsets, alpha=b.alpha), name + " forward")
    assert not torch.isnan(t0).any()
    pick = np.random.default_rng(1).choice(d.L, min(d.L, 40), replace=False)
    assert_close(t0.cpu().numpy()[pick], np.stack([ora.t0(d.oshape, d.cores, int(b.indices[k])).reshape(-1) for k in pick]), name + " T0")
    rg, _ = ora.bwd(d.oshape, d.cores, b.indices, b.offsets, b.grad_output, alpha=b.alpha)
    dg, _ = d.bwd(t0=t0, grad_cores=[torch.full_like(x, 0.25) for x in d.g])
    for k in range(3):
        assert_close(new[k].cpu().numpy(), ora.sgd(d.cores[k], rg[k], 0.05), "%s core %d" % (name, k + 1))
        assert_close(dg[k].cpu().numpy() - 0.25, rg[k], "%s dG%d" % (name, k + 1))


@pytest.mark.parametrize("n,R", SHAPES)
@pytest.mark.parametrize("kind,L", [("spread", 1), ("spread", 700), ("hot row", 1500), ("first digit", 1300), ("third digit", 1300),
                                    ("second digit", 900), ("one row", 700)])
def test_small_streams(n, R, kind, L, always_rows):
    _check(_table(kind, n, R, L, max(1, L // 3), 61), "%s %s R %d L %d" % (kind, n, R, L))


# (4,096 slices of the first and third core are all the counters of a window and of its lists; 1,024 of the second the bins of
# the counting pass; one more of either, and the position tiles or the list owners take over)
@pytest.mark.parametrize("n,R", [((2, 2, 4), 32), ((4, 4, 4), 64)])
@pytest.mark.parametrize("m", [(3072, 6, 1024), (1, 4, 4095), (3072, 6, 1025), (30, 1024, 40), (7, 1021, 9), (30, 1025, 40), (5, 1, 6)])
def test_tables_at_the_limits(n, R, m, always_rows):
    _check(_table("hot row", n, R, 2600, 700, 66, m=m), "%s %s R %d" % (m, n, R), lists=m[1] <= 1024)


@pytest.mark.parametrize("kind", ["hot row", "first digit"])
def test_long_streams_with_long_windows(kind):
    # 70,000 positions: windows of 1,024, by the library's own choice
    _check(_table(kind, (2, 2, 4), 32, 70_000, 9_000, 62), "%s long" % kind)


def test_more_pieces_of_the_final_sums_than_workgroups():
    # some 340,000 distinct rows on 70 slices of the first and third core: about 1,300 pieces of 512 beyond the first ones
    _check(_table("spread", (2, 2, 4), 32, 400_000, 50_000, 64, m=(30, 1000, 40)), "many pieces")


@pytest.mark.parametrize("n,L", [((4, 4, 4), 6144), ((4, 4, 4), 10_240), ((2, 2, 4), 12_288), ((2, 2, 4), 17_001)])
def test_rank_64_by_choice(n, L):
    # the lengths from which the library groups by itself, and the same pair where the workspace has no room for it
    d = _table("spread", n, 64, L, L // 4, 63)
    assert B.bwd_has_prepass(d.shape, L, 0, True) and B.bwd_has_prepass(d.shape, (6143 if n[0] == 4 else 12_287), 0, True) is False
    b = d.batch
    rg, _ = ora.bwd(d.oshape, d.cores, b.indices, b.offsets, b.grad_output, alpha=b.alpha)
    want = [ora.sgd(d.cores[k], rg[k], 0.05) for k in range(3)]
    out_want = ora.fwd(d.oshape, d.cores, b.indices, b.offsets, alpha=b.alpha)
    full = B.bwd_sgd_workspace_bytes(d.shape, L, d.n_bags, 0)
    # (half of the full size is enough for the scanning owners, 2.8 / 1.4 MB for these tables, and too little for the rows, which
    # take more than 15 MB)
    for size in ([full, full // 2] if L < (8192 if n[0] == 4 else 16_384) else [full]):
        ws = torch.full((size,), 0x7F, dtype=torch.uint8, device=dev())
        out = torch.full((d.n_bags, d.t.dim), float("nan"), dtype=torch.float32, device=dev())
        t0 = torch.full((L, B.t0_floats(d.shape)), float("nan"), dtype=torch.float32, device=dev())
        new = [torch.full_like(x, float("nan")) for x in d.g]
        B.tt_emb_bwd_prepare(d.shape, d.idx, d.off, d.n_bags, workspace=ws, kept_t0=True)
        B.tt_emb_fwd_prepared(d.shape, d.g, d.idx, d.off, d.n_bags, out, ws, t0=t0, alpha=d.alpha)
        B.tt_emb_bwd_sgd(d.shape, d.g, new, d.idx, d.off, d.n_bags, d.go, 0.05, alpha=d.alpha, workspace=ws, t0=t0, prepared=True)
        assert_close(out.cpu().numpy(), out_want, "forward, workspace %d" % size)
        for k in range(3):
            assert_close(new[k].cpu().numpy(), want[k], "core %d, workspace %d" % (k + 1, size))


def test_one_workspace_on_either_side_of_the_longer_windows():
    # 65,536 positions on: windows of 1,024 instead of 256, and fewer counters; a workspace for the longer batch does for the shorter
    a, b = _table("hot row", (2, 2, 4), 32, 65_536, 9_000, 64), _table("hot row", (2, 2, 4), 32, 65_535, 9_000, 65)
    ws = torch.full((B.bwd_sgd_workspace_bytes(a.shape, a.L, a.n_bags, 0),), 0x7F, dtype=torch.uint8, device=dev())
    for d in (a, b):
        _check(d, "%d positions" % d.L, ws=ws)


def test_one_workspace_on_either_side_of_the_longest_windows():
    # 262,144 positions on: windows of 2,048 instead of 1,024
    a, b = _table("hot row", (2, 2, 4), 32, 262_144, 30_000, 67), _table("hot row", (2, 2, 4), 32, 262_143, 30_000, 68)
    ws = torch.full((B.bwd_sgd_workspace_bytes(a.shape, a.L, a.n_bags, 0),), 0x7F, dtype=torch.uint8, device=dev())
    for d in (a, b):
        _check(d, "%d positions" % d.L, ws=ws)


# With a cache: slots in one bin of 128 and several, the last bin's slots missing, as many as the passes take and one more (the list owners);
# no position cached, all of them, a hot slot over many windows; streams on either side of the window sizes; long ones, where groups of lanes
# share a hot slot's windows, with one slot and with eight in a bin; so long that the tiles are for more workgroups than run at once.
@pytest.mark.parametrize("n,R,L,K,share", [((4, 4, 4), 32, 4095, 50, 0.7), ((4, 4, 4), 32, 4096, 1, 0.7), ((4, 4, 4), 32, 20_001, 129, 0.8), ((2, 2, 4), 32, 66_000, 300, 0.9),
                                           ((2, 2, 4), 64, 17_000, 1000, 0.0), ((4, 4, 4), 64, 16_500, 128, 1.0), ((2, 2, 4), 32, 16_400, 8192, 0.5),
                                           ((2, 2, 4), 32, 16_400, 8193, 0.5), ((4, 4, 4), 32, 262_144, 129, 0.99), ((2, 2, 4), 64, 300_001, 1000, 0.99), ((4, 4, 4), 32, 1_050_000, 300, 0.995)])
def test_with_a_cache(n, R, L, K, share):
    _with_a_cache(n, R, L, K, share, (30, 20, 40))


# as many slices of the second core as leave room for the bins of cached rows, and one more (the list owners); more than 512 windows;
# the longer windows beside those of cached rows, at rank 64
@pytest.mark.parametrize("n,R,L,K,share,m", [((4, 4, 4), 32, 17_000, 300, 0.6, (9, 896, 11)), ((4, 4, 4), 32, 17_000, 300, 0.6, (9, 897, 11)),
                                             ((2, 2, 4), 64, 5_000, 2000, 0.6, (9, 896, 11)), ((4, 4, 4), 32, 66_000, 500, 0.8, (30, 400, 40)),
                                             ((4, 4, 4), 64, 65_535, 700, 0.9, (30, 20, 40)), ((4, 4, 4), 64, 65_536, 700, 0.9, (30, 20, 40))])
def test_with_a_cache_in_tables_of_many_slices(n, R, L, K, share, m):
    _with_a_cache(n, R, L, K, share, m)


def _with_a_cache(n, R, L, K, share, m):
    rng = np.random.default_rng([L, K])
    t = W.TableShape(m[0] * m[1] * m[2] - 3, m, n, (1, R, R, 1))
    keys = np.sort(rng.choice(t.num_rows, K, replace=False)).astype(np.int64)
    other = np.setdiff1d(np.arange(t.num_rows), keys)
    idx = np.where(rng.random(L) < share, rng.choice(keys, L), rng.choice(other, L)).astype(np.int64)
    if share > 0:
        idx[rng.random(L) < 0.3 * share] = keys[K // 2]
    n_bags = 900
    off = np.concatenate([[0], np.sort(rng.integers(0, L + 1, n_bags - 1)), [L]]).astype(np.int64)
    batch = W.Batch(idx, off, rng.standard_normal((n_bags, t.dim)).astype(np.float32), (0.5 + rng.random(L)).astype(np.float32))
    d = DeviceTable(W.Workload("rows", (t,), n_bags, (0, 9), "uniform", 0.0, "normal0.1", 3), batch=batch)
    counts = np.arange(K, 0, -1).astype(np.int64)
    cache, _, _ = d.build_cache(K, keys, counts)
    sel = ora.cache_select(keys, counts, K)
    lines = cache.rows.clone()
    crow = lines.cpu().numpy()[:K].copy()
    ref = ora.fwd(d.oshape, d.cores, idx, off, alpha=batch.alpha, cache_keys=sel, cache_rows=crow)
    rg, rc = ora.bwd(d.oshape, d.cores, idx, off, batch.grad_output, alpha=batch.alpha, cache_keys=sel)
    need = B.bwd_sgd_workspace_bytes(d.shape, L, n_bags, K)
    got = []
    for two_calls in (True, True, False):
        cache.rows.copy_(lines)
        ws = torch.full((need,), 0x7F, dtype=torch.uint8, device=dev())
        out = torch.full((n_bags, t.dim), float("nan"), dtype=torch.float32, device=dev())
        t0 = torch.full((L, B.t0_floats(d.shape)), float("nan"), dtype=torch.float32, device=dev())
        new = [torch.full_like(x, float("nan")) for x in d.g]
        B.tt_emb_bwd_prepare(d.shape, d.idx, d.off, n_bags, cache=cache, workspace=ws, kept_t0=True)
        B.tt_emb_fwd_prepared(d.shape, d.g, d.idx, d.off, n_bags, out, ws, t0=t0, alpha=d.alpha, cache=cache)
        B.tt_emb_bwd_sgd(d.shape, d.g, new, d.idx, d.off, n_bags, d.go, 0.05, alpha=d.alpha, cache=cache, workspace=ws, t0=t0, prepared=two_calls)
        torch.cuda.synchronize()
        got.append([out] + new + [cache.rows.clone()])
    assert all(torch.equal(x, y) for other_run in got[1:] for x, y in zip(got[0], other_run))
    assert_close(got[0][0].cpu().numpy(), ref, "forward")
    for k in range(3):
        assert_close(got[0][1 + k].cpu().numpy(), ora.sgd(d.cores[k], rg[k], 0.05), "core %d" % (k + 1))
    assert_close(got[0][4].cpu().numpy()[:K], ora.sgd(crow, rc, 0.05), "cache lines")
    # gradients on their own are added to what is there
    cache.rows.copy_(lines)
    gc = torch.full_like(cache.rows, 0.5)
    dg, dc = d.bwd(cache=cache, grad_cores=[torch.full_like(x, 0.25) for x in d.g], grad_cache=gc, t0=t0)
    for k in range(3):
        assert_close(dg[k].cpu().numpy() - 0.25, rg[k], "dG%d" % (k + 1))
    assert_close(dc.cpu().numpy()[:K] - 0.5, rc, "dCache")


@pytest.mark.parametrize("L,R", [(5000, 32), (16_384, 32), (5000, 64), (16_384, 64)])       # the scanning owners, the list owners
def test_with_a_cache_and_little_room_the_owners_run(L, R):
    d = _table("hot row", (2, 2, 4), R, L, 500, 9)
    rows, counts = np.unique(d.batch.indices, return_counts=True)
    cache, _, _ = d.build_cache(100, rows.astype(np.int64), counts.astype(np.int64))
    lines = cache.rows.clone()
    full = B.bwd_sgd_workspace_bytes(d.shape, d.L, d.n_bags, 100)
    out = []
    for size in (full, full // 2):                 # distinct rows take more than half of what the query says
        cache.rows.copy_(lines)
        ws = torch.full((size,), 0x7F, dtype=torch.uint8, device=dev())
        o, t0 = d.fwd_keep_t0(cache=cache)
        o2 = torch.full((d.n_bags, d.t.dim), float("nan"), dtype=torch.float32, device=dev())
        new = [torch.full_like(x, float("nan")) for x in d.g]
        B.tt_emb_bwd_prepare(d.shape, d.idx, d.off, d.n_bags, cache=cache, workspace=ws, kept_t0=True)
        B.tt_emb_fwd_prepared(d.shape, d.g, d.idx, d.off, d.n_bags, o2, ws, t0=t0, alpha=d.alpha, cache=cache)
        B.tt_emb_bwd_sgd(d.shape, d.g, new, d.idx, d.off, d.n_bags, d.go, 0.05, alpha=d.alpha, cache=cache, workspace=ws, t0=t0, prepared=True)
        torch.cuda.synchronize()
        assert_close(o2.cpu().numpy(), o, "forward")
        out.append([x.cpu().numpy() for x in new] + [cache.rows.cpu().numpy()])
    for x, y in zip(*out):
        assert np.isfinite(x).all()
        assert_close(x, y, "rows against list owners")


@pytest.mark.parametrize("n,R,L", [((4, 4, 4), 64, 10_300), ((2, 2, 4), 64, 12_400), ((4, 4, 4), 32, 32_801), ((2, 2, 4), 32, 32_801)])
@pytest.mark.parametrize("mean", [4, 1.5])
def test_short_bags_are_pooled_from_rows_and_from_the_caches_lines(n, R, L, mean):
    # hits and misses in the same bags, bags of 0 to 9 and of 33 to 300 among them, two long ones side by side
    t = W.TableShape(30 * 20 * 40 - 3, (30, 20, 40), n, (1, R, R, 1))
    rng = np.random.default_rng([L, R])
    K = 300
    keys = np.sort(rng.choice(t.num_rows, K, replace=False)).astype(np.int64)
    idx = np.where(rng.random(L) < 0.4, rng.choice(keys, L), rng.integers(0, t.num_rows, L)).astype(np.int64)
    n_bags = int(L / mean)
    lens = rng.multinomial(L - 700, np.full(n_bags, 1 / n_bags)).astype(np.int64)
    lens[[7, n_bags // 2, n_bags // 2 + 1, n_bags - 1]] += (33, 300, 300, 67)
    off = np.concatenate([[0], lens.cumsum()])
    batch = W.Batch(idx, off, np.zeros((n_bags, t.dim), np.float32), (0.5 + rng.random(L)).astype(np.float32))
    d = DeviceTable(W.Workload("rows", (t,), n_bags, (0, 9), "uniform", 0.0, "normal0.1", 4), batch=batch)
    counts = np.arange(K, 0, -1).astype(np.int64)
    cache, _, _ = d.build_cache(K, keys, counts)
    cache.rows += 0.01                                       # (what the lines have learned; a row of the cores is another)
    assert B.fwd_uses_lists(d.shape, L, K, True)
    ws = torch.full((B.bwd_sgd_workspace_bytes(d.shape, L, n_bags, K),), 0x7F, dtype=torch.uint8, device=dev())
    out = torch.full((n_bags, t.dim), float("nan"), dtype=torch.float32, device=dev())
    t0 = torch.empty((L, B.t0_floats(d.shape)), dtype=torch.float32, device=dev())
    B.tt_emb_bwd_prepare(d.shape, d.idx, d.off, n_bags, cache=cache, workspace=ws, kept_t0=True)
    B.tt_emb_fwd_prepared(d.shape, d.g, d.idx, d.off, n_bags, out, ws, t0=t0, alpha=d.alpha, cache=cache)
    ref = ora.fwd(d.oshape, d.cores, idx, off, alpha=batch.alpha, cache_keys=ora.cache_select(keys, counts, K), cache_rows=cache.rows.cpu().numpy()[:K])
    assert_close(out.cpu().numpy(), ref, "forward")
