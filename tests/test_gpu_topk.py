"""The selection behind tt_cache_build / tt_cache_refill (tt_topk.h) at the borders of its three forms: all candidates
ranked, the class of the K-th count and the keys up to it ranked (narrowed down first where ties fill the class), a full
sort (more rows than are ranked, or more candidates than are narrowed down); with ties everywhere, all counts
equal, counts on class borders, and the largest counts."""
import numpy as np
import pytest
import torch

from oracle import tt_oracle as ora
from paper_2101_11714_amd import binding as B
from paper_2101_11714_amd import workloads as W
from gpu_util import dev

pytestmark = pytest.mark.gpu

T = W.TableShape(149_999, (50, 50, 60), (2, 2, 4), (1, 8, 8, 1))
LARGE = W.TableShape(299_999, (100, 50, 60), (2, 2, 4), (1, 8, 8, 1))


@pytest.mark.parametrize("counts", ["ties", "equal", "borders", "wide"])
@pytest.mark.parametrize("n,K", [(1, 1), (100, 10), (8192, 8192), (8192, 5), (8193, 1), (8193, 8192), (20_000, 8193), (30_000, 30_000),
                                 (60_000, 3_000)])
def test_selected_rows_in_order(n, K, counts):
    _select(T, n, K, counts)


# the most candidates that are selected from, and one more: the full sort
@pytest.mark.parametrize("counts", ["ties", "equal", "borders", "wide"])
@pytest.mark.parametrize("n", [1 << 18, (1 << 18) + 1])
def test_many_candidates(n, counts):
    _select(LARGE, n, 3_000, counts)


def _select(T, n, K, counts):
    rng = np.random.default_rng([n, K])
    rows = rng.permutation(T.num_rows)[:n].astype(np.int64)
    rows[0] = T.num_rows - 1 if T.num_rows - 1 not in rows[1:] else rows[0]
    cnt = {"ties": lambda: rng.integers(0, 20, n), "equal": lambda: np.full(n, 7), "borders": lambda: (1 << rng.integers(0, 32, n)) - rng.integers(0, 2, n),
           "wide": lambda: rng.integers(0, 1 << 32, n)}[counts]().astype(np.int64)
    cores = [torch.from_numpy(x).to(dev()) for x in W.make_cores(T, "normal0.1", 1)]
    cache = B.Cache(K, T.dim, dev())
    B.tt_cache_build(B.shape_of(T), cores, torch.from_numpy(rows).to(dev()), torch.from_numpy(cnt).to(dev()), cache)
    torch.cuda.synchronize()
    assert np.array_equal(cache.keys.cpu().numpy()[:K], ora.cache_select(rows, cnt, K))


# the refill's row -> slot map: the largest that is built in LDS (16,384 places), one larger, one with more places than are needed
@pytest.mark.parametrize("K,places", [(1, 16), (5, 16), (4097, 16_384), (8192, 16_384), (8193, 32_768), (100, 32_768), (100, 16_384)])
def test_refilled_map(K, places):
    rng = np.random.default_rng(K + places)
    cores = [torch.from_numpy(x).to(dev()) for x in W.make_cores(T, "normal0.1", 1)]
    shape, n = B.shape_of(T), 3 * K
    rows = rng.permutation(T.num_rows)[:n].astype(np.int64)
    first, second = rng.permutation(n) + 1, rng.permutation(n) + 1
    cache = B.Cache(K, T.dim, dev())
    cache.table = torch.zeros(places, dtype=torch.int64, device=dev())
    cache.c.table, cache.c.capacity = cache.table.data_ptr(), places
    on = lambda x: torch.from_numpy(np.ascontiguousarray(x, dtype=np.int64)).to(dev())
    B.tt_cache_build(shape, cores, on(rows), on(first), cache)
    B.tt_cache_refill(shape, cores, on(rows), on(second), cache)
    torch.cuda.synchronize()
    keys = ora.cache_select(rows, second.astype(np.int64), K)
    assert np.array_equal(cache.keys.cpu().numpy()[:K], keys)
    asked = np.concatenate([rows, rng.integers(0, T.num_rows, 1000)])
    slot = torch.empty(asked.size, dtype=torch.int32, device=dev())
    B.tt_cache_lookup(cache, on(asked), slot)
    assert np.array_equal(slot.cpu().numpy(), ora.cache_lookup(ora.Shape.of(T), keys, asked))
    table = cache.table.cpu().numpy().view(np.uint64)
    used = table[table != np.uint64(0xFFFFFFFFFFFFFFFF)]
    assert np.array_equal(np.sort(used & np.uint64(0xFFFFFFFF)), np.arange(K)) and np.array_equal(np.sort(used >> np.uint64(32)), np.sort(keys.view(np.uint64)))
