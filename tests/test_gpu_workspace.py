"""What the calls take as a workspace: device memory (or pinned host memory) in one piece, counted in bytes whatever its type."""
import numpy as np
import pytest
import torch

from paper_2101_11714_amd import binding as B
from gpu_util import dev
from test_gpu_flex import _table

pytestmark = pytest.mark.gpu


def _calls(d, ws):
    """Every entry point that takes a workspace through the compiled extension, on a run-time shape."""
    new, dg = [torch.full_like(x, float("nan")) for x in d.g], [torch.zeros_like(x) for x in d.g]
    out = torch.empty((d.n_bags, d.t.dim), dtype=torch.float32, device=dev())
    rows, counts = np.unique(d.batch.indices, return_counts=True)
    cand = [torch.from_numpy(x.astype(np.int64)).to(dev()) for x in (rows, counts)]
    cache = d.build_cache(20, rows.astype(np.int64), counts.astype(np.int64))[0]
    return {"fwd": lambda: B.tt_emb_fwd(d.shape, d.g, d.idx, d.off, d.n_bags, out, alpha=d.alpha, workspace=ws),
            "bwd": lambda: B.tt_emb_bwd(d.shape, d.g, d.idx, d.off, d.n_bags, d.go, dg, alpha=d.alpha, workspace=ws),
            "prepare": lambda: B.tt_emb_bwd_prepare(d.shape, d.idx, d.off, d.n_bags, workspace=ws),
            "step": lambda: B.tt_emb_bwd_sgd(d.shape, d.g, new, d.idx, d.off, d.n_bags, d.go, 0.05, alpha=d.alpha, workspace=ws),
            "build": lambda: B.tt_cache_build(d.shape, d.g, cand[0], cand[1], cache, workspace=ws),
            "refill": lambda: B.tt_cache_refill(d.shape, d.g, cand[0], cand[1], cache, workspace=ws)}, new


@pytest.mark.parametrize("kind", ["host", "strided", "expanded"])
def test_other_memory_is_refused(kind):
    d = _table((7, 6, 9), (2, 4, 4), (24, 24), 200, 3, 71)
    n = B.bwd_sgd_workspace_bytes(d.shape, d.L, d.n_bags)
    ws = {"host": lambda: torch.empty(n, dtype=torch.uint8), "strided": lambda: torch.empty(2 * n, dtype=torch.uint8, device=dev())[::2],
          "expanded": lambda: torch.empty(1, dtype=torch.uint8, device=dev()).expand(n)}[kind]()
    for f in _calls(d, ws)[0].values():
        with pytest.raises(AssertionError):
            f()


@pytest.mark.parametrize("kind", ["float32", "int64", "pinned"])
def test_every_type_counts_in_bytes(kind):
    d = _table((7, 6, 9), (2, 4, 4), (24, 24), 200, 3, 72)
    n = B.bwd_sgd_workspace_bytes(d.shape, d.L, d.n_bags)
    want = d.bwd_sgd(0.05)
    ws = {"float32": lambda: torch.empty(n // 4 + 1, dtype=torch.float32, device=dev()), "int64": lambda: torch.empty(n // 8 + 1, dtype=torch.int64, device=dev()),
          "pinned": lambda: torch.empty(n, dtype=torch.uint8, pin_memory=True)}[kind]()
    calls, new = _calls(d, ws)
    for f in calls.values():
        f()
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(new, want))
