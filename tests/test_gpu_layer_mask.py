"""The masked input gradient of the single-layer backward against a plain torch
reference, at the widths where the scatter's lane groups and the product's
output parts change shape."""
import numpy as np
import pytest
import torch

from paper_2403_17092_amd import gnnhip

pytestmark = pytest.mark.gpu

# fp32 sums of at most ~40 terms of magnitude one: 40 * 2^-24 of the result's
# scale, and the products' sums of up to 256 terms
TOL = 2e-5


def _block(rng, nd, ns, fmax):
    cnt = rng.integers(0, fmax + 1, nd)
    cnt[0] = 0  # a row with no edges
    indptr = np.concatenate([[0], np.cumsum(cnt)]).astype(np.int32)
    idx = (rng.random(indptr[-1]) ** 3 * ns).astype(np.int32)
    occ = np.bincount(idx, minlength=ns).astype(np.int32)
    occ[:nd] += 1
    t = lambda x: torch.as_tensor(x).cuda()  # noqa: E731
    counts = torch.tensor([nd, ns, len(idx), 0], dtype=torch.int32, device="cuda")
    return gnnhip.Block(t(indptr), t(idx if len(idx) else np.zeros(1, np.int32)), t(np.arange(ns, dtype=np.int32)), t(np.maximum(occ, 1)), counts,
                        nd, ns, len(idx)), cnt, idx, np.maximum(occ, 1)


@pytest.mark.parametrize("kind", ["sage_mean", "gcn", "gin"])
@pytest.mark.parametrize("F_in,F_out,nd,ns,fmax", [
    (4, 3, 1, 1, 3), (12, 16, 65, 130, 7), (36, 47, 129, 500, 70), (64, 64, 64, 64, 5),
    (100, 33, 200, 777, 12), (256, 172, 77, 300, 130)])
def test_masked_input_gradient(kind, F_in, F_out, nd, ns, fmax):
    rng = np.random.default_rng(F_in * 1000 + nd)
    blk, cnt, idx, occ = _block(rng, nd, ns, fmax)
    k = gnnhip.KIND[kind]
    g = torch.Generator().manual_seed(F_in)
    H = torch.relu(torch.randn((ns, F_in), generator=g))
    H[:, 0] = 0.0
    W = torch.randn((gnnhip.w_rows(k, F_in, F_out), F_out), generator=g) / F_in ** 0.5
    dZ = torch.randn((nd, F_out), generator=g)
    X, _ = gnnhip.layer_fwd(blk, k, H.cuda(), W.cuda(), True)
    got = {}
    for mask in (False, True):
        _, dH = gnnhip.layer_bwd(blk, k, F_in, X, H.cuda(), W.cuda(), dZ.cuda(), True, mask)
        got[mask] = dH[:ns].cpu().double()
    rows = torch.as_tensor(np.repeat(np.arange(nd), cnt))
    src = torch.as_tensor(idx.astype(np.int64))
    d, w64 = dZ.double(), W.double()
    c = torch.as_tensor(cnt).double()
    ref = torch.zeros((ns, F_in), dtype=torch.float64)
    if kind == "sage_mean":
        ref[:nd] += d @ w64[:F_in].T
        dagg = d @ w64[F_in:].T
        ref.index_add_(0, src, dagg[rows] / c[rows][:, None])
    elif kind == "gcn":
        dagg, o = d @ w64.T, torch.as_tensor(occ).double()
        ref.index_add_(0, src, dagg[rows] * ((c[rows] + 1) * o[src]).rsqrt()[:, None])
        ref[:nd] += dagg * ((c + 1) * o[:nd]).rsqrt()[:, None]
    else:
        # the hidden rows' mask is the forward's own
        M = X[:nd, F_in:F_in + F_out].cpu()
        dagg = ((d @ w64[F_in:].T) * (M > 0)) @ w64[:F_in].T
        ref.index_add_(0, src, dagg[rows])
        ref[:nd] += dagg
    assert gnnhip.check_errors() == 0
    for mask in (False, True):
        want = ref * (H > 0) if mask else ref
        assert (got[mask] - want).abs().max() <= TOL * max(1.0, float(ref.abs().max()))
    # masked entries are exactly zero, the others what the unmasked call gives up to its sums' order
    assert torch.equal(got[True] == 0, (got[False] * (H > 0)) == 0)
