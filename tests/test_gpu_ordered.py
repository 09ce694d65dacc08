"""The ordered scan of the shared-bank form (many voxels against a large bank:
tiles that no voxel of a block needs are skipped) against the FP64 scan of
every row, whose accepted sets it must return exactly: ragged voxel and row
counts, both numbers of blocks per 256 voxels, one and several segments of
tiles, frames that do not fill the padding, caller weights, curves unlike any
bank row, invalid voxels, banks without spread.  The FP64 scan itself is held to
the oracle in test_gpu_bank.
"""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU-only hosts
    pytest.skip("no HIP device", allow_module_level=True)

import paper_2603_14859_amd as V  # noqa: E402

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("models,frames,voxels,draws,n,case", [
    ((W.M_2TCM_IRR,), 30, 40_001, 80_003, 100, "plain"),
    ((W.M_2TCM_IRR, W.M_2TCM_REV), 27, 10_000, 170_000, 60, "plain"),   # three segments of tiles
    ((W.M_MRTM, W.M_LPNTPET), 37, 20_003, 80_001, 400, "plain"),
    ((W.M_1TCM,), 22, 262_400, 16_384, 30, "plain"),                    # two blocks per 256 voxels
    ((W.M_2TCM_IRR,), 30, 40_001, 80_003, 100, "weights"),
    ((W.M_2TCM_IRR,), 30, 40_001, 80_003, 100, "odd"),
    ((W.M_2TCM_IRR,), 8, 40_001, 80_003, 50, "narrow")])
def test_same_sets_as_every_row(models, frames, voxels, draws, n, case):
    ref = models[0] == W.M_MRTM
    sched = W.SCHED_40x90 if ref else W.SCHED_30x50
    ft = W.frame_times(sched)[:frames + 1]
    nodes, cp = W.grid(0.2, float(ft[-1]), reference=ref)
    lam = W.LAMBDA_C11 if ref else W.LAMBDA_F18
    boxes = W.box_array(list(models))
    if case == "narrow":
        boxes[0, 0] = (0.3, 0.3001)
        boxes[0, 1] = (0.2, 0.2001)
    th_b, x_b = V.bank_build(list(models), boxes, draws, 7, cp, ft, 0.2)
    g = torch.Generator(device=DEV).manual_seed(5)
    src = torch.randint(0, x_b.shape[0], (voxels,), generator=g, device=DEV)
    clean = x_b[src, :frames]
    if case == "odd":  # curves unlike any row: reversed, scaled far beyond the bank, negative frames
        clean = clean.clone()
        clean[::5] = clean[::5].flip(1)
        clean[1::5] *= 30.0
        clean[2::5, ::3] *= -0.5
    dt = torch.from_numpy(np.diff(ft.astype(np.float64))).to(DEV)
    y = (clean + torch.sqrt(0.05 * clean.abs() / dt)
         * torch.randn(clean.shape, generator=g, device=DEV, dtype=torch.float64)).float().contiguous()
    y[17] = float("nan")
    y[18] = -1.0
    w = None
    if case == "weights":
        w = torch.rand(y.shape, generator=g, device=DEV) / (y.abs() + 0.5)
        w[:, 3] = 0.0
        w[100, 4] = -1.0
        w[101] = 0.0
    kw = dict(decay_lambda=lam, weights=w, debug=True)
    frac = (n + 0.5) / (draws * len(models))
    a = V.infer_bank(y, ft, 0.2, nodes, list(models), draws, frac, th_b, x_b, bank_scan="bf16", **kw)
    b = V.infer_bank(y, ft, 0.2, nodes, list(models), draws, frac, th_b, x_b, bank_scan="f64", **kw)
    assert a["n"] == n
    for k in ("accept_idx", "accept_dist", "threshold", "moments", "model_prob"):
        assert torch.equal(torch.nan_to_num(a[k].double(), nan=-7.0), torch.nan_to_num(b[k].double(), nan=-7.0)), k
    if case == "plain":
        assert a["fallback_voxels"] <= voxels // 50


@pytest.mark.parametrize("models,frames,voxels,draws,n", [
    ((W.M_1TCM,), 22, 524_301, 16_384, 30),               # one block per 256 voxels
    ((W.M_MRTM, W.M_LPNTPET), 37, 131_900, 20_003, 400)])  # a second, smaller voxel chunk in the first one's buffers
def test_one_block_and_two_chunks(models, frames, voxels, draws, n):
    test_same_sets_as_every_row(models, frames, voxels, draws, n, "plain")


@pytest.mark.parametrize("models,voxels,draws,n", [((W.M_1TCM,), 40_000, 80_000, 30), ((W.M_2TCM_IRR,), 20_000, 150_000, 30),
                                                   ((W.M_1TCM,), 270_000, 20_000, 16)])
def test_narrow_posteriors_fit_their_lists(models, voxels, draws, n):
    """Few accepted rows of a large bank: a voxel's candidates lie in few tiles, and
    every piece of its list holds as many as half an undivided one."""
    test_same_sets_as_every_row(models, 30, voxels, draws, n, "plain")


@pytest.mark.parametrize("frames,voxels,draws,n", [(48, 301, 20_003, 40), (41, 301, 20_003, 400), (48, 20_001, 150_001, 100),
                                                   (43, 20_001, 150_001, 512)])
def test_most_frames(frames, voxels, draws, n):
    """41 to 48 frames, unordered and ordered: the sets of the FP64 scan."""
    ft = W.frame_times([0.2] * 10 + [1.0] * (frames - 10))
    nodes, cp = W.grid(0.2, float(ft[-1]))
    th_b, x_b = V.bank_build([W.M_2TCM_IRR], W.box_array([W.M_2TCM_IRR]), draws, 7, cp, ft, 0.2)
    g = torch.Generator(device=DEV).manual_seed(6)
    clean = x_b[torch.randint(0, draws, (voxels,), generator=g, device=DEV), :frames]
    dt = torch.from_numpy(np.diff(ft.astype(np.float64))).to(DEV)
    y = (clean + torch.sqrt(0.05 * clean.abs() / dt)
         * torch.randn(clean.shape, generator=g, device=DEV, dtype=torch.float64)).float().contiguous()
    a, b = (V.infer_bank(y, ft, 0.2, nodes, [W.M_2TCM_IRR], draws, (n + 0.5) / draws, th_b, x_b, bank_scan=s, debug=True)
            for s in ("bf16", "f64"))
    for k in ("accept_idx", "accept_dist", "threshold", "moments", "model_prob"):
        assert torch.equal(torch.nan_to_num(a[k].double(), nan=-7.0), torch.nan_to_num(b[k].double(), nan=-7.0)), k
