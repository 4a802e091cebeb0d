"""The feature cache where the lookup's workgroups take many passes: lists of
touched sets that fill up several times, every lane-group width, invalid ids."""
import numpy as np
import pytest
import torch

from tests import gpu_common as gc
from tests.test_gpu_feature_cache import _run

pytestmark = pytest.mark.gpu


# rows of 4, 20, 36 and 64 chunks: groups of 16, 32 and 64 lanes, 16 to 4 rows a
# pass and 1,024 workgroups; sets of one way, so nearly every miss is a set's
# first.  The first case lists some 320 sets a workgroup, past the list's 256
@pytest.mark.parametrize("F,n_rows,n_ids,S", [
    (16, 420_000, 400_000, 1_000_003),
    (80, 60_000, 40_001, 30_011),
    (144, 60_000, 20_000, 30_011),
    (256, 60_000, 16_385, 30_011),
])
def test_many_passes(F, n_rows, n_ids, S):
    g = np.random.Generator(np.random.PCG64(F))
    X = g.normal(size=(n_rows, F)).astype(np.float32)
    gc.announce("feature cache: many passes", F, n_ids)
    _run(X, [g.choice(n_rows, size=n_ids, replace=False) for _ in range(2)], S, 1, device_table=True)


def test_invalid_ids_count_as_misses():
    from paper_2403_17092_amd import gnnhip
    gc.announce("feature cache: invalid ids")
    X = torch.arange(4000 * 16, dtype=torch.float32, device="cuda").reshape(4000, 16)
    cache = gnnhip.FeatureCache(500, 4, 16, gnnhip.F32, "cuda")
    ids = torch.randperm(4000, device="cuda")[:3000].int()
    bad = ids.clone()
    bad[::7] = -3
    bad[5] = 4000
    stats = torch.zeros(2, dtype=torch.int64, device="cuda")
    n = torch.tensor([3000], dtype=torch.int32, device="cuda")
    out = cache.gather(X, bad, n, 3000, stats)
    torch.cuda.synchronize()
    assert gnnhip.check_errors() == gnnhip.DEVERR_SEED_RANGE
    assert stats.cpu().tolist() == [0, 3000]
    ok = (bad >= 0) & (bad < 4000)
    assert torch.equal(out[:3000][ok], X[bad[ok].long()]) and not out[:3000][~ok].any()
