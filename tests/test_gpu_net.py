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
from test_gpu_proposal import DEV, _params, _tacs, forward_sigma, pack  # noqa: E402


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
