"""GAT steps against the oracle at the widths where the column sums' lane groups
change (a row of 1 to 64 chunks, whole and ragged), one and two jobs per launch."""
import numpy as np
import pytest
import torch

from oracle import model as omodel
from tests import gpu_common as gc
from tests import helpers
from workloads import configs, graphs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,B", [
    ((4, 1), 3), ((4, 4, 2), 1), ((8, 36, 5), 70), ((256, 20, 3), 33), ((100, 256, 47), 64),
    ((12, 64, 12, 9), 40)])
def test_gat_widths(dims, B):
    from paper_2403_17092_amd import gnnhip
    gc.announce("gat widths", dims, B)
    g = graphs.chunglu_graph(3000, 9.0, 2.1, seed=5)
    L, rng = len(dims) - 1, np.random.default_rng(B)
    X = rng.normal(size=(3000, dims[0])).astype(np.float32)
    labels = rng.integers(0, dims[-1], 3000).astype(np.int32)
    seeds = configs.make_seeds(3000, B, 3, 2)
    W = configs.make_weights("gat", dims, 9)
    fan = [5] * L
    tr = gnnhip.Trainer("gat", dims, W, B, fan, 3000)
    tr.step(gc.csr_to_device(g.rowptr, g.col), torch.as_tensor(X).cuda(), torch.as_tensor(labels).cuda(),
            gc.seeds_to_device(seeds), 7, 0.01)
    got = tr.inspect()
    assert gnnhip.check_errors() == 0
    ref = omodel.train_step(g.rowptr, g.col, X, labels, seeds, fan, 7, "gat", W, 0.01)
    if dims[-1] > 1:  # (one class: every gradient is zero)
        dW = np.concatenate([x.ravel() for x in ref["dW"]])
        helpers.assert_close(got["dweights"], dW, gc.TOL_GRAD, "dW")
    else:
        assert np.abs(got["dweights"]).max() < 1e-6
