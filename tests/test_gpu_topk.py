"""The selection behind tt_cache_build / tt_cache_refill (tt_topk.h) at the borders of its three forms: all candidates
ranked, the class of the K-th count and the keys up to it ranked (narrowed down first where ties fill the class), a full
sort (more rows than are ranked, or more candidates than one workgroup narrows down); with ties everywhere, all counts
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
