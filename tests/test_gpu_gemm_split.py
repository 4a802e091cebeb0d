"""The products that run as split bf16 products (98,304 rows and more at the
capacity), through the single-layer entry points, against 64 bits.  The live
counts are small and ragged: the form is chosen by the capacity."""
import numpy as np
import pytest
import torch

from paper_2403_17092_amd import gnnhip
from tests import gpu_common as gc

pytestmark = pytest.mark.gpu

CAP = 98_304
# fp32 sums of up to 512 products: measured 4e-7 of the norm (fp32 MFMAs 4.1e-7),
# and a mean aggregation before it
TOL = 2e-6


def _case(kind, F_in, F_out, nd, seed=0):
    rng = np.random.default_rng(seed + nd)
    ns = nd + 50
    cnt = rng.integers(0, 4, nd)
    indptr = np.zeros(CAP + 1, np.int32)
    indptr[1:nd + 1] = np.cumsum(cnt)
    idx = rng.integers(0, ns, max(1, cnt.sum())).astype(np.int32)
    t = lambda x: torch.as_tensor(x).cuda()  # noqa: E731
    blk = gnnhip.Block(t(indptr), t(idx), torch.zeros(CAP + 50, dtype=torch.int32, device="cuda"),
                       torch.ones(CAP + 50, dtype=torch.int32, device="cuda"),
                       torch.tensor([nd, ns, int(cnt.sum()), 0], dtype=torch.int32, device="cuda"),
                       CAP, CAP + 50, max(1, len(idx)))
    g = torch.Generator().manual_seed(seed)
    H = torch.randn((CAP + 50, F_in), generator=g)
    W = torch.randn((gnnhip.w_rows(kind, F_in, F_out), F_out), generator=g) / F_in ** 0.5
    dZ = torch.randn((CAP, F_out), generator=g)
    return blk, np.repeat(np.arange(nd), cnt), idx[:cnt.sum()], cnt, H, W, dZ


def _close(got, ref, what):
    err = (got.cpu().double() - ref).norm() / ref.norm()
    assert err <= TOL, (what, float(err))


# one row, tile edges, remainders; widths whole, ragged and past a tile; rows of
# 4 and of 1 element alignment (F_out 255, 70); weight gradients of 4 and more tiles
@pytest.mark.parametrize("F_in,F_out,nd", [
    (100, 256, 1), (100, 256, 129), (32, 48, 300), (128, 172, 1025), (256, 255, 200), (36, 70, 640),
    (88, 132, 4099), (256, 256, 8200)])
def test_layer_products(F_in, F_out, nd):
    gc.announce("split products", F_in, F_out, nd)
    kind = gnnhip.SAGE_MEAN
    blk, rows, idx, cnt, H, W, dZ = _case(kind, F_in, F_out, nd)
    X, Hout = gnnhip.layer_fwd(blk, kind, H.cuda(), W.cuda(), True)
    dW, dH = gnnhip.layer_bwd(blk, kind, F_in, X, H.cuda(), W.cuda(), dZ.cuda(), True, False)
    h, w, d = H.double(), W.double(), dZ[:nd].double()
    agg = torch.zeros((nd, F_in), dtype=torch.float64).index_add(0, torch.as_tensor(rows), h[torch.as_tensor(idx).long()])
    c = torch.as_tensor(cnt).double().clamp(min=1)[:, None]
    x = torch.cat([h[:nd], agg / c], 1)
    assert gnnhip.check_errors() == 0
    _close(Hout[:nd], torch.relu(x @ w), "H")
    _close(dW, x.T @ d, "dW")
    dx = d @ w.T
    ref = torch.zeros((nd + 50, F_in), dtype=torch.float64)
    ref[:nd] = dx[:, :F_in]
    ref.index_add_(0, torch.as_tensor(idx).long(), (dx[:, F_in:] / c)[torch.as_tensor(rows)])
    _close(dH[:nd + 50], ref, "dH")


@pytest.mark.parametrize("nd", [65, 700])
def test_gin_masked_products(nd):
    # GIN's products read dZ through the hidden rows' mask
    gc.announce("split GIN", nd)
    kind, F_in, F_out = gnnhip.GIN, 140, 160
    blk, rows, idx, cnt, H, W, dZ = _case(kind, F_in, F_out, nd, 3)
    X, Hout = gnnhip.layer_fwd(blk, kind, H.cuda(), W.cuda(), True)
    dW, dH = gnnhip.layer_bwd(blk, kind, F_in, X, H.cuda(), W.cuda(), dZ.cuda(), True, False)
    h, w, d = H.double(), W.double(), dZ[:nd].double()
    r, i = torch.as_tensor(rows), torch.as_tensor(idx).long()
    agg = h[:nd] + torch.zeros((nd, F_in), dtype=torch.float64).index_add(0, r, h[i])
    m = X[:nd, F_in:F_in + F_out].cpu().double()
    _close(m, torch.relu(agg @ w[:F_in]), "M")
    _close(Hout[:nd], torch.relu(m @ w[F_in:]), "H")
    dP = (d @ w[F_in:].T) * (m > 0)
    _close(dW, torch.cat([agg.T @ dP, m.T @ d]), "dW")
    dagg = dP @ w[:F_in].T
    ref = torch.zeros((nd + 50, F_in), dtype=torch.float64)
    ref[:nd] = dagg
    ref.index_add_(0, i, dagg[r])
    _close(dH[:nd + 50], ref, "dH")


def test_values_bf16_cannot_hold():
    # infinities, NaN and finite values that round to infinity in bf16
    gc.announce("split special values")
    kind, F_in, F_out, nd = gnnhip.GCN, 64, 64, 200
    blk, rows, idx, cnt, H, W, dZ = _case(kind, F_in, F_out, nd, 5)
    blk.counts[2] = 0
    blk.indptr.zero_()  # no edges: every row is its own
    H[3, 5], H[70, 1], H[130, 60], H[131, 7] = float("inf"), float("nan"), 3.4e38, -float("inf")
    H[132] = 1e-36
    W[60] *= 0.01
    X, Hout = gnnhip.layer_fwd(blk, kind, H.cuda(), W.cuda(), False)
    want = H[:nd].double() @ W.double()
    want = torch.where(want.abs() > 3.4028235e38, torch.sign(want) * float("inf"), want)
    got = Hout[:nd].cpu().double()
    assert torch.equal(torch.isnan(got), torch.isnan(want))
    assert torch.equal(torch.isinf(got), torch.isinf(want))
    fine = torch.isfinite(want)
    assert torch.equal(torch.sign(got[torch.isinf(want)]), torch.sign(want[torch.isinf(want)]))
    scale = want.where(fine, torch.zeros_like(want)).norm(dim=1, keepdim=True).expand_as(want)
    assert ((got - want).abs()[fine] <= 1e-6 * scale[fine] + 1e-40).all()
