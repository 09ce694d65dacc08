"""Screened draws of the per-voxel path against the FP64 oracle, at the sizes
and inputs where the screen can go wrong: the ends of its range of draw counts,
tile and list edges, one and several wavefronts per voxel, rates at zero and
beyond the short series, signed input functions, ties everywhere and curves
outside the fp32 range (both take the unscreened path).  Tolerances are those
of test_gpu_parity: accepted sets equal up to draws within 1e-5 of the
threshold, means within 1e-5.
"""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU-only hosts
    pytest.skip("no HIP device", allow_module_level=True)

from test_gpu_parity import _check_infer, _inputs  # noqa: E402

T1, IRR, REV = W.M_1TCM, W.M_2TCM_IRR, W.M_2TCM_REV


@pytest.mark.parametrize("models,n_draws,n,wpv", [
    ((IRR,), 2599, 20, 0), ((IRR,), 2600, 20, 1), ((IRR,), 2601, 1, 4), ((IRR,), 5000, 64, 2), ((IRR,), 5000, 65, 4),
    ((IRR,), 5003, 500, 1), ((IRR,), 3000, 3000, 1), ((T1,), 4097, 100, 1), ((T1,), 3072, 63, 4),
    ((T1, IRR), 2500, 100, 2), ((T1, IRR, REV), 3001, 200, 4), ((IRR, REV), 1500, 30, 1), ((REV,), 3001, 129, 2),
    ((REV,), 2600, 40, 4)])
def test_counts(models, n_draws, n, wpv):
    import oracle as ora
    ft, cp, y = _inputs(n_vox=9, model=models[-1], sched=W.SCHED_30x50)
    total = n_draws * len(models)
    _check_infer(ora, y, ft, cp, list(models), W.box_array(list(models)), n_draws, (n + 0.5) / total if n < total else 1.0,
                 11, wpv=wpv, voxel_offset=5)


@pytest.mark.parametrize("case", ["zero_rate", "fast", "signed", "offset", "ties", "tiny_weights", "huge_weights",
                                  "low_counts", "one_frame", "fixed_rate", "rev_fast", "rev_close", "rev_no_k4"])
def test_inputs(case):
    import oracle as ora
    model = T1 if case in ("zero_rate", "one_frame") else (REV if case.startswith("rev") else IRR)
    sched = W.SCHED_30x50
    ft, cp, y = _inputs(n_vox=12, model=model, sched=sched)
    boxes = W.box_array([model])
    weights, n_draws, p = None, 4000, 0.02
    if case == "zero_rate":
        boxes[0, 1] = (0.0, 0.2)
    elif case == "fast":  # beta h up to 1: beyond the short series
        boxes[0, 1] = (0.5, 4.0)
        boxes[0, 2] = (0.2, 1.0)
    elif case == "signed":
        cp = (cp * np.cos(0.7 * np.arange(cp.size))).astype(np.float32)
    elif case == "offset":
        ft = (ft + np.float32(1.4)).astype(np.float32)[:20]
        y = np.ascontiguousarray(y[:, :19])
        cp = np.concatenate([cp, cp[-1:] * np.ones(10, np.float32)])
    elif case == "ties":
        boxes[0, :, 1] = boxes[0, :, 0]
        boxes[0, 0] = boxes[0, 1] = (0.3, 0.3)
        boxes[0, 2] = (0.1, 0.1)
    elif case in ("tiny_weights", "huge_weights"):
        weights = np.full(y.shape, 1e-18 if case == "tiny_weights" else 1e18, np.float32)
        weights[::2] *= np.float32(1e-9 if case == "tiny_weights" else 1e9)
    elif case == "low_counts":
        y = (y * 1e-4).astype(np.float32)
    elif case == "one_frame":
        ft, y = ft[[0, 24]], np.ascontiguousarray(y[:, 20:21])
    elif case == "fixed_rate":
        boxes[0, 1] = (0.2, 0.2)
        boxes[0, 2] = (0.05, 0.05)
    elif case == "rev_fast":
        boxes[0, 1] = (0.5, 4.0)
        boxes[0, 3] = (0.0, 2.0)
    elif case == "rev_close":  # nearly equal eigenvalues
        boxes[0, 1] = (0.05, 0.06)
        boxes[0, 2] = (0.0005, 0.001)
        boxes[0, 3] = (0.05, 0.06)
    elif case == "rev_no_k4":
        boxes[0, 3] = (0.0, 0.0)
    _check_infer(ora, y, ft, cp, [model], boxes, n_draws, p, 3, weights=weights)


@pytest.mark.parametrize("models,n_draws,n,voxels,ties", [
    ((IRR,), 8000, 1, 1, False), ((IRR,), 8001, 100, 3, False), ((T1, IRR, REV), 9001, 300, 2, False),
    ((REV,), 16_000, 64, 1, False), ((T1,), 50_001, 65, 128, False), ((IRR,), 20_000, 2000, 2, False),
    ((IRR,), 9000, 50, 2, True)])
def test_few_voxels(models, n_draws, n, voxels, ties):
    """A voxel's draws over several blocks (a count of upper bounds, then the
    parts' candidates); ties leave every part to the unscreened path."""
    import oracle as ora
    ft, cp, y = _inputs(n_vox=voxels, model=models[-1], sched=W.SCHED_30x50)
    boxes = W.box_array(list(models))
    if ties:
        for s, v in ((0, 0.3), (1, 0.3), (2, 0.1), (4, 0.05)):
            boxes[0, s] = (v, v)
    _check_infer(ora, y, ft, cp, list(models), boxes, n_draws, (n + 0.5) / (n_draws * len(models)), 13, voxel_offset=2)


@pytest.mark.parametrize("n_draws,n,share,scale,spread,sd", [
    (2599, 20, 0.1, 1.0, 0.2, 0.3), (2600, 64, 0.0, 1.0, 0.2, 0.3), (2601, 65, 0.1, 1.5, 0.2, 0.3),
    (5003, 300, 0.5, 1.0, 0.2, 0.3), (4000, 1000, 0.1, 1.0, 0.2, 0.3),
    (6000, 50, 0.0, 1.0, 2.0, 3.0),    # most draws outside the box
    (6000, 50, 0.1, 1.0, 0.05, 0.01),  # a sharp mixture: every draw close
    (3000, 2000, 0.0, 1.0, 3.0, 5.0)])  # fewer valid draws than accepted ones
def test_proposal_draws(n_draws, n, share, scale, spread, sd):
    from test_gpu_proposal import _check_is, _synthetic_outputs, _tacs
    rng = np.random.default_rng(31)
    ft, cp, th, y = _tacs(10, 9)
    o = _synthetic_outputs(th, rng, spread=spread, sd=sd)
    o[2, 3] = np.nan   # a mixture the screen does not take
    o[3, 9] = 300.0
    y[4, 2] = np.nan
    keep = [v for v in range(10) if v not in (2, 3)]
    _check_is(y, ft, cp, o, n_draws, (n + 0.5) / n_draws, 5, share=share, scale=scale, sample=keep, v_off=3)


@pytest.mark.parametrize("n_draws,n,share,sd", [(6000, 100, 0.1, 0.02), (20_000, 30, 0.0, 0.005), (5003, 300, 0.0, 0.003)])
def test_proposal_full_lists(n_draws, n, share, sd):
    """Proposals far narrower than the noise: more draws within their bounds of
    the threshold than a candidate list holds."""
    from test_gpu_proposal import _check_is, _synthetic_outputs, _tacs
    ft, cp, th, y = _tacs(9, 14)
    o = _synthetic_outputs(th, np.random.default_rng(32), spread=0.0, sd=sd)
    _check_is(y, ft, cp, o, n_draws, (n + 0.5) / n_draws, 5, share=share, scale=1.0, sample=list(range(9)), v_off=3)


@pytest.mark.parametrize("models,n_draws,n,wpv,durations", [
    ((IRR,), 3000, 65, 4, W.SCHED_30x50), ((IRR,), 6000, 400, 4, [0.2] * 8), ((T1, REV), 4000, 400, 4, [0.2] * 8),
    ((IRR,), 6000, 700, 2, [0.4] * 3), ((REV,), 5000, 300, 4, [0.2] * 4)])
def test_one_list_for_the_block(models, n_draws, n, wpv, durations):
    """Several wavefronts, n > 64: the block's merged list is read by every
    wavefront before any of them scores its part of it (short grids make the
    exact pass short beside the reading of a long list)."""
    import oracle as ora
    ft, cp, y = _inputs(n_vox=9, model=models[-1], sched=durations)
    total = n_draws * len(models)
    _check_infer(ora, y, ft, cp, list(models), W.box_array(list(models)), n_draws, (n + 0.5) / total, 23, wpv=wpv)


def test_few_voxels_some_parts_full():
    """A voxel's draws over four blocks of which only some have more candidates
    than their lists hold (3072 nearly equal draws of the second model fill the
    lists of the first three and leave the fourth none): the blocks that go on
    without the screen take the same draws as their screened lists did."""
    import oracle as ora
    models = [T1, IRR, REV]
    boxes = W.box_array(models)
    boxes[0, 0] = boxes[2, 0] = (0.9, 1.0)  # far from the observed curves
    boxes[0, 1] = boxes[2, 1] = (0.01, 0.05)
    boxes[2, 2] = (0.001, 0.05)
    boxes[2, 3] = (0.0, 0.01)
    for s, lo, hi in ((0, 0.3, 0.30006), (1, 0.3, 0.3), (2, 0.1, 0.1), (4, 0.05, 0.05)):
        boxes[1, s] = (lo, hi)
    ft = W.frame_times(W.SCHED_30x50)
    _, cp = W.grid(0.2, 50.0)
    rng = np.random.default_rng(41)
    th = W.true_params(rng, 2, IRR, boxes[1])
    clean = ora.simulate(IRR, th, cp, 0.2, ft)
    y = W.add_noise(clean, ft, rng.standard_normal(clean.shape))
    _check_infer(ora, y, ft, cp, models, boxes, 3072, 50.5 / 9216, 17, voxel_offset=4)


def _voxel_scale(y, ft, cp, k1, vb):
    """Largest norm of an observed curve's and a model curve's sum under unit weights."""
    import oracle as ora
    th = np.zeros((2, 8), np.float32)
    th[0, 0] = 1.0           # the input's running integral
    th[1, [0, 1, 4]] = 1.0   # the input itself
    q, p = ora.simulate(T1, th, cp, 0.2, ft).astype(np.float64)
    return np.linalg.norm(y.astype(np.float64), axis=1) + k1 * np.linalg.norm(q) + vb * np.linalg.norm(p)


@pytest.mark.parametrize("models,square,wpv", [((REV,), 1e10, 1), ((REV,), 9.9e11, 1), ((REV,), 9.9e11, 4),
                                               ((T1, REV), 3e11, 1), ((T1, REV), 9.9e11, 2), ((IRR,), 9.9e11, 1),
                                               ((IRR,), 1e-6, 1), ((REV,), 1e-9, 1)])
def test_scale(models, square, wpv):
    """Weights that put the largest squared norm at either end of what the screen takes."""
    import oracle as ora
    ft, cp, y = _inputs(n_vox=9, model=models[-1], sched=W.SCHED_30x50)
    weights = np.repeat(square / _voxel_scale(y, ft, cp, 1.0, 0.1)[:, None] ** 2, y.shape[1], axis=1).astype(np.float32)
    _check_infer(ora, y, ft, cp, list(models), W.box_array(list(models)), 4000, (60 + 0.5) / (4000 * len(models)), 19,
                 weights=weights, wpv=wpv)


def test_wide_proposal_intervals():
    """Wide mixtures and large weights: intervals of 4e8 on distances of 9e11, whose
    widths differ from draw to draw by more than 2^24.  Sets are equal up to draws
    whose fp32 distances may round together (2^-24 relative on either side)."""
    import oracle as ora
    import oracle.proposal as prop
    import paper_2603_14859_amd as V
    nv, n_draws, n, share, scale = 60, 5000, 50, 0.99, 90.0
    ft = W.frame_times(W.SCHED_30x50)
    _, cp = W.grid(0.2, 50.0)
    box = W.box_array([IRR])[0]
    box[0], box[1], box[2], box[4] = (0.98, 1.0), (1e-7, 1e-6), (1e-7, 1e-6), (0.0, 1e-6)
    th = np.zeros((1, 8), np.float32)
    th[0, 0] = 1.0
    q = ora.simulate(T1, th, cp, 0.2, ft)[0].astype(np.float64)
    rng = np.random.default_rng(31)
    y = (0.01 * q * (1.0 + 0.1 * rng.standard_normal((nv, 30)))).astype(np.float32)
    weights = np.repeat(0.95e12 / _voxel_scale(y, ft, cp, 1.0, 0.0)[:, None] ** 2, 30, axis=1).astype(np.float32)
    o = np.zeros((nv, 96), np.float32)
    dev = torch.device("cuda:0")
    g = V.infer(torch.from_numpy(y).to(dev), ft, cp, 0.2, [IRR], box[None], n_draws, (n + 0.5) / n_draws, 5, debug=True,
                proposal=torch.from_numpy(o).to(dev), prior_share=share, sd_scale=scale, waves_per_voxel=1,
                weights=torch.from_numpy(weights).to(dev))
    got = g["accept_idx"].cpu().numpy()
    for v in range(nv):
        order, _, _, d = prop.infer_is(y[v], ft, cp, 0.2, box, o[v].astype(np.float64), n_draws, (n + 0.5) / n_draws, 5, v,
                                       prior_share=share, sd_scale=scale, weights_v=weights[v])
        h = d[order[n - 1]]
        for k in set(got[v].tolist()) ^ set(order.tolist()):
            assert abs(d[k] - h) <= 2.0 ** -22 * h, f"voxel {v}: draw {k}, {abs(d[k] - h) / h:.1e} from the threshold"


@pytest.mark.parametrize("part,voxels", [(0.98, 60), (1.02, 5)])
def test_wide_proposal_gate(part, voxels):
    """The same mixtures (standard deviations of 12) on either side of the largest
    norm whose intervals an error class holds, 2.35e8 / (1.54e-5 + 33 kappa)."""
    import oracle as ora
    import oracle.proposal as prop
    import paper_2603_14859_amd as V
    n_draws, n, share, scale = 5000, 50, 0.99, 90.0
    ft = W.frame_times(W.SCHED_30x50)
    _, cp = W.grid(0.2, 50.0)
    box = W.box_array([IRR])[0]
    box[0], box[1], box[2], box[4] = (0.98, 1.0), (1e-7, 1e-6), (1e-7, 1e-6), (0.0, 1e-6)
    th = np.zeros((1, 8), np.float32)
    th[0, 0] = 1.0
    q = ora.simulate(T1, th, cp, 0.2, ft)[0].astype(np.float64)
    rng = np.random.default_rng(37)
    y = (0.01 * q * (1.0 + 0.1 * rng.standard_normal((voxels, 30)))).astype(np.float32)
    o = np.zeros((voxels, 96), np.float32)
    sd = float(np.exp(np.max(prop.mixture(o[:1].astype(np.float64), scale)[2])))
    square = part * 1.75 * 2.0 ** 27 / (1.54e-5 + 33.0 * (2.3e-6 * sd + 2.1e-7))
    weights = np.repeat(square / _voxel_scale(y, ft, cp, 1.0, 0.0)[:, None] ** 2, 30, axis=1).astype(np.float32)
    dev = torch.device("cuda:0")
    g = V.infer(torch.from_numpy(y).to(dev), ft, cp, 0.2, [IRR], box[None], n_draws, (n + 0.5) / n_draws, 5, debug=True,
                proposal=torch.from_numpy(o).to(dev), prior_share=share, sd_scale=scale, waves_per_voxel=1,
                weights=torch.from_numpy(weights).to(dev))
    got = g["accept_idx"].cpu().numpy()
    for v in range(voxels):
        order, _, _, d = prop.infer_is(y[v], ft, cp, 0.2, box, o[v].astype(np.float64), n_draws, (n + 0.5) / n_draws, 5, v,
                                       prior_share=share, sd_scale=scale, weights_v=weights[v])
        h = d[order[n - 1]]
        for k in set(got[v].tolist()) ^ set(order.tolist()):
            assert abs(d[k] - h) <= 2.0 ** -22 * h, f"voxel {v}: draw {k}, {abs(d[k] - h) / h:.1e} from the threshold"


@pytest.mark.parametrize("models,n_draws,n,voxels", [((IRR,), 130_000, 65, 1), ((T1,), 40_000, 70, 2),
                                                     ((IRR, REV), 60_000, 66, 1)])
def test_few_voxels_nearly_empty_parts(models, n_draws, n, voxels):
    """n a little above 64, over up to 64 blocks: many of them have no candidate
    or one."""
    import oracle as ora
    ft, cp, y = _inputs(n_vox=voxels, model=models[-1], sched=W.SCHED_30x50)
    _check_infer(ora, y, ft, cp, list(models), W.box_array(list(models)), n_draws, (n + 0.5) / (n_draws * len(models)), 29)


@pytest.mark.parametrize("models,n_draws,n,voxels", [((T1, IRR, REV), 667, 80, 9000), ((REV,), 1024, 85, 30_000),
                                                     ((T1, IRR), 4000, 320, 1000), ((IRR, REV), 4000, 320, 9000)])
def test_screened_where_it_pays(models, n_draws, n, voxels):
    """A call with too many accepted draws for its draws (or too few draws) is not
    slower than the same call under L1, which runs the unscreened kernel and costs
    as much there; screened, these took 1.4 to 1.8 times that."""
    ft, cp, y = _inputs(n_vox=200, model=models[-1], sched=W.SCHED_30x50)
    y = torch.from_numpy(np.tile(y, (voxels // 200, 1))).to("cuda:0")
    import paper_2603_14859_amd as V
    times = {}
    for k in ("l1", "l2"):
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(6)]
        for i in range(6):
            V.infer(y, ft, cp, 0.2, list(models), W.box_array(list(models)), n_draws,
                    (n + 0.5) / (n_draws * len(models)), 3, distance=k)
            ev[i].record()
        torch.cuda.synchronize()
        times[k] = min(a.elapsed_time(b) for a, b in zip(ev[1:], ev[2:]))
    print(times)
    assert times["l2"] <= 1.2 * times["l1"]


@pytest.mark.parametrize("models,n_draws,n,voxels", [
    ((REV,), 30_000, 716, 3), ((REV,), 30_000, 718, 3), ((REV,), 20_000, 1500, 600), ((IRR,), 9000, 896, 2),
    ((IRR,), 5000, 720, 600), ((T1, IRR, REV), 20_000, 1000, 2), ((REV,), 20_000, 3000, 3)])
def test_lists_of_fewer_wavefronts(models, n_draws, n, voxels):
    """On both sides of where four wavefronts' lists fill the LDS (n = 717)."""
    import oracle as ora
    ft, cp, y = _inputs(n_vox=min(voxels, 9), model=models[-1], sched=W.SCHED_30x50)
    total = n_draws * len(models)
    p = (n + 0.5) / total
    if voxels <= 9:
        _check_infer(ora, y, ft, cp, list(models), W.box_array(list(models)), n_draws, p, 31)
        return
    # (many voxels: the first ones against the same call of them alone)
    from test_gpu_parity import _gpu_infer
    big = _gpu_infer(np.tile(y, (voxels // 9 + 1, 1))[:voxels], ft, cp, list(models), W.box_array(list(models)), n_draws, p, 31)
    g, _ = _check_infer(ora, y, ft, cp, list(models), W.box_array(list(models)), n_draws, p, 31)
    assert np.array_equal(big["accept_idx"][:9], g["accept_idx"])
    assert np.array_equal(big["moments"][:9], g["moments"], equal_nan=True)


@pytest.mark.parametrize("scale", [1e-6, 3e5])
def test_few_voxels_scale(scale):
    """Few voxels' draws over several blocks with small and large caller weights:
    the sets, and (the threshold of the whole voxel being found at any scale) about
    the time of unit weights (1.9 times that under the large ones without it)."""
    import oracle as ora
    import paper_2603_14859_amd as V
    models = [T1, IRR, REV]
    ft, cp, y = _inputs(n_vox=3, model=IRR, sched=W.SCHED_30x50)
    boxes, p = W.box_array(models), 300.5 / 60_000
    one = np.ones(y.shape, np.float32)
    _check_infer(ora, y, ft, cp, models, boxes, 20_000, p, 37, weights=one * np.float32(scale))
    t = {}
    yd = torch.from_numpy(np.tile(y, (4, 1))).to("cuda:0")
    for w in (1.0, scale):
        wd = torch.full_like(yd, w)
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(12)]
        for e in ev:
            V.infer(yd, ft, cp, 0.2, models, boxes, 20_000, p, 37, weights=wd)
            e.record()
        torch.cuda.synchronize()
        t[w] = min(a.elapsed_time(b) for a, b in zip(ev[1:], ev[2:]))
    print(t)
    assert t[scale] <= 1.4 * t[1.0]
