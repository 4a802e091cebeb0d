"""GPU parity of the sampler's forms for wide frontiers: the lane groups of every
fanout, tiles of every size and tickets, hubs counted through the window."""
import numpy as np
import pytest
import torch

from oracle import model as omodel
from oracle import sampling
from tests import gpu_common as gc
from tests import helpers
from workloads import configs, graphs

pytestmark = pytest.mark.gpu


def _run(g, seeds, fanouts, key, scan_order=0):
    from paper_2403_17092_amd import gnnhip
    gc.announce("wide sample", len(seeds), fanouts, "n", len(g[0]) - 1, "scan_order", scan_order)
    csr = gc.csr_to_device(g[0], g[1], scan_order=scan_order)
    ws = torch.zeros(gnnhip.sample_workspace_bytes(len(seeds), fanouts, len(g[0]) - 1), dtype=torch.uint8,
                     device="cuda")
    # the second call runs on the words and ids the first one left
    for k in (key, key + 1):
        blocks = gnnhip.sample_blocks(csr, gc.seeds_to_device(seeds), fanouts, k, ws=ws)
        torch.cuda.synchronize()
        assert gnnhip.check_errors() == 0
        ref = sampling.sample_blocks(g[0], g[1], seeds, fanouts, k)
        for h, (gb, ob) in enumerate(zip(blocks, ref)):
            gc.compare_block(gb.host(), ob, f"hop {h + 1}")
    return ref


def _chunglu(n=40_000, d=14.0):
    g = graphs.chunglu_graph(n, d, 2.1, seed=17)
    return g.rowptr, g.col


def _hubs(n, hubs, extra, seed=1):
    """Every node joined to all of `hubs` hub nodes and to a few others."""
    rng = np.random.default_rng(seed)
    ids = rng.permutation(n)
    u = np.concatenate([np.repeat(ids[:hubs], n), rng.integers(0, n, extra)])
    v = np.concatenate([np.tile(np.arange(n), hubs), rng.integers(0, n, extra)])
    ok = u != v
    key = np.unique(np.concatenate([u[ok] * n + v[ok], v[ok] * n + u[ok]]))
    rowptr = np.searchsorted(key, np.arange(n + 1) * n)
    return rowptr.astype(np.int64), (key % n).astype(np.int32)


# more than 8,192 dst nodes: 1, 2, 4, 8 and 16 lanes of four draws, at both ends of each
@pytest.mark.parametrize("f", [1, 3, 4, 5, 8, 9, 16, 17, 32, 33, 64])
def test_lane_groups(f):
    seeds = configs.make_seeds(40_000, 9001, 3, f)
    _run(_chunglu(), seeds, [f], 5 + f)


def test_wide_lane_groups_without_idle_lanes():
    # 270K dst nodes at the capacity: groups as small as the fanout allows
    _run(_chunglu(300_000, 8.0), configs.make_seeds(300_000, 270_001, 3, 0), [2], 8)


@pytest.mark.parametrize("scan_order", [0, 1])
@pytest.mark.parametrize("B,fanouts", [
    (9000, [3]),           # tiles of two items
    (60_001, [8]),         # four
    (120_003, [12]),       # eight
    (150_007, [20]),       # more than a grid of the largest: tickets
])
def test_scan_tiles(B, fanouts, scan_order):
    _run(_chunglu(200_000, 25.0), configs.make_seeds(200_000, B, 3, 1), fanouts, 2, scan_order)


@pytest.mark.parametrize("B", [1500, 9000])
def test_hub_window(B):
    # 12,000 nodes, most picks hubs: counts through the window from id 0 and past the seeds
    g = _hubs(12_000, 5, 30_000)
    seeds = configs.make_seeds(12_000, B, 3, 2)
    _run(g, seeds, [6, 9], 4)


def test_hub_window_transpose():
    # the places the window hands out build the transpose the backward gathers over
    from paper_2403_17092_amd import gnnhip
    gc.announce("hub transpose")
    n, B, dims, fan = 12_000, 9000, (8, 12, 5), [9, 4]
    rowptr, col = _hubs(n, 5, 30_000)
    rng = np.random.default_rng(4)
    X = rng.normal(size=(n, dims[0])).astype(np.float32)
    labels = rng.integers(0, dims[-1], n).astype(np.int32)
    seeds = configs.make_seeds(n, B, 3, 2)
    W = configs.make_weights("sage_mean", dims, 9)
    tr = gnnhip.Trainer("sage_mean", dims, W, B, fan, n)
    tr.step(gc.csr_to_device(rowptr, col), torch.as_tensor(X).cuda(), torch.as_tensor(labels).cuda(),
            gc.seeds_to_device(seeds), 7, 0.01)
    got = tr.inspect()
    assert gnnhip.check_errors() == 0
    ref = omodel.train_step(rowptr, col, X, labels, seeds, fan, 7, "sage_mean", W, 0.01)
    for h, ob in enumerate(ref["blocks"]):
        gc.compare_block(got["blocks"][h], ob, f"hop {h + 1}")
    dW = np.concatenate([x.ravel() for x in ref["dW"]])
    helpers.assert_close(got["dweights"], dW, gc.TOL_GRAD, "dW")
