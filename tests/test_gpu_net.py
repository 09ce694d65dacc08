"""The fused network kernels against the FP64 oracle at the edges of their
tiles: row counts around the 64-row tile, around one pass of the persistent
grid (256 blocks) and one row, the fewest and the most frames, an output buffer
off 16-byte alignment.  Tolerances are those of test_gpu_proposal (the
first-order error of the split products, and normwise gradients).
"""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU-only hosts
    pytest.skip("no HIP device", allow_module_level=True)

import paper_2603_14859_amd as V  # noqa: E402
import oracle.proposal as prop  # noqa: E402
from test_gpu_proposal import BLOCKS, DEV, _params, _tacs, forward_sigma, pack, unpack  # noqa: E402


@pytest.mark.parametrize("n,frames,offset", [(1, 30, 0), (63, 30, 0), (64, 1, 0), (65, 30, 1), (130, 30, 3),
                                             (64 * 256 - 1, 30, 0), (64 * 256 + 65, 30, 0)])
def test_forward_edges(n, frames, offset):
    p = _params(21)
    y = _tacs(min(n, 200), 5)[3][:, :frames]
    y = np.ascontiguousarray(np.tile(y, (n // y.shape[0] + 1, 1))[:n])
    y[:: 7] *= np.float32(1e-12)  # log1p far below the FP64 spacing at 1
    buf = torch.full((n * 96 + 8,), -7.0, device=DEV)
    out = buf[offset:offset + n * 96].view(n, 96)
    V.proposal_forward(torch.from_numpy(pack(p)).to(DEV), torch.from_numpy(y).to(DEV), out=out)
    torch.cuda.synchronize()
    assert bool((buf[:offset] == -7.0).all()) and bool((buf[offset + n * 96:] == -7.0).all())
    rows = np.unique(np.concatenate([np.arange(min(n, 70)), np.arange(max(0, n - 140), n)]))
    g = out[torch.from_numpy(rows).to(DEV)].cpu().numpy().astype(np.float64)
    x = prop.features(y[rows])
    o, _ = prop.forward(p, x)
    assert np.all(np.abs(g[:, :prop.NOUT] - o) <= 6.0 * forward_sigma(p, x) + 1e-6 * (1.0 + np.abs(o)))


@pytest.mark.parametrize("m,frames,dims", [(1, 30, 4), (63, 1, 5), (65, 30, 4), (511, 32, 4), (513, 30, 5),
                                           (64 * 128 + 33, 30, 4)])
def test_gradient_edges(m, frames, dims):
    """The gradient of 2 m rows is the mean of the gradients of its two halves:
    a row's share is the same number but for an exact factor of two, whatever
    its place in a tile, so that only the FP32 sums over the rows differ.  m is
    around the 64-row tile, around 512 rows (where the weight gradients are
    split) and around one pass of the persistent grid.  Bound: each sum is a
    chain of at most 3 max(n / 256, 32) matrix instructions of 16 terms each and
    16 partials, each addition within 2^-23 of T, the sum of the terms'
    magnitudes (from the oracle, whose gradients are within 10 %).  Also the
    same bits from run to run, and the halves' mean loss."""
    n = 2 * m
    p = _params(23, sd=0.2, dims=dims)
    y = _tacs(min(n, 200), 5, model=W.M_2TCM_IRR if dims == 4 else W.M_2TCM_REV)[3]
    y = np.concatenate([y, y[:, :2]], axis=1)[:, :frames]
    y = np.ascontiguousarray(np.tile(y, (n // y.shape[0] + 1, 1))[:n])
    y *= np.random.default_rng(25).uniform(0.5, 1.5, y.shape).astype(np.float32)
    x = prop.features(y)
    o, (_, a1, h1, a2, h2) = prop.forward(p, x)
    logpi, mu, logsd = prop.mixture(o, dims=dims)
    c = logpi.argmax(axis=1)
    rng = np.random.default_rng(24)
    zz = mu[np.arange(n), c] + 0.7 * np.exp(logsd[np.arange(n), c]) * rng.standard_normal((n, dims))
    th = np.zeros((n, V.PSTRIDE), dtype=np.float32)
    th[:, list(prop.head_slots(dims))] = np.exp(zz).astype(np.float32)
    dev = [torch.from_numpy(a).to(DEV) for a in (pack(p), y, th)]

    def run(lo, hi):
        loss, grad = V.proposal_loss_grad(dev[0], dev[1][lo:hi].contiguous(), dev[2][lo:hi].contiguous(), dims=dims)
        return float(loss.item()), grad.cpu().numpy()

    (lw, gw), (la, ga), (lb, gb) = run(0, n), run(0, m), run(m, n)
    assert np.array_equal(gw, run(0, n)[1])
    assert abs(lw - 0.5 * (la + lb)) <= 1e-6 * (abs(lw) + abs(la) + abs(lb))
    # the terms' magnitudes from the oracle's gradients of the single rows
    z = prop.targets(th, dims)
    t = (z[:, None, :] - mu) * np.exp(-logsd)
    comp = logpi + (-0.5 * t * t - logsd - 0.5 * np.log(2.0 * np.pi)).sum(axis=2)
    r = np.exp(comp - np.logaddexp.reduce(comp, axis=1, keepdims=True))
    do = np.zeros_like(o)
    q = prop.C * dims
    do[:, :prop.C] = np.exp(logpi) - r
    do[:, prop.C:prop.C + q] = (-r[:, :, None] * t * np.exp(-logsd)).reshape(n, -1)
    s = (logsd - prop.LS0) / (prop.LS1 - prop.LS0)
    do[:, prop.C + q:prop.C + 2 * q] = (r[:, :, None] * (1.0 - t * t) * (prop.LS1 - prop.LS0) * s * (1.0 - s)).reshape(n, -1)
    dh2 = (do @ p["W3"].T) * (a2 > 0.0)
    dh1 = (dh2 @ p["W2"].T) * (a1 > 0.0)
    T = {}
    for i, (act, d) in enumerate(((x, dh1), (h1, dh2), (h2, do)), 1):
        T[f"W{i}"], T[f"b{i}"] = np.abs(act).T @ np.abs(d) * 1.1 / n, np.abs(d).sum(axis=0) * 1.1 / n
    bound = 2.0 * (3 * max(n / 256, 32) + 16 + 16) * 2.0 ** -23
    gw, gh = unpack(gw, dims), unpack((ga.astype(np.float64) + gb) * 0.5, dims)
    for k, _ in BLOCKS:
        w = T[k].shape[-1]
        assert np.all(np.abs(gw[k] - gh[k])[..., :w] <= bound * T[k] + 1e-30), k
