"""Traversals of shallow forests at the edges of their launch shapes: lanes of
four events, the few-events kernel and its limit, chunks of trees, one to
255 features, and outputs that start at any element."""
import numpy as np
import pytest
import torch

import paper_1609_06119_amd as fb
from oracle import fbdt_oracle as O
from synth import random_forest

pytestmark = pytest.mark.gpu


def _model(f, d, B, bounds=None):
    return fb.Model.from_arrays(f["cut_feature"], f["cut_bin"], f["leaf"], f["f0"], d, B,
                                boundaries=bounds)


@pytest.mark.parametrize("n,d,B,D,T", [
    (1, 1, 2, 1, 1), (3, 40, 256, 3, 3), (255, 7, 256, 2, 5), (256, 7, 17, 3, 66),
    (257, 255, 256, 3, 9), (1021, 40, 256, 3, 700), (5, 255, 256, 1, 2500),
    (393_216, 5, 256, 3, 5), (393_217, 5, 256, 3, 5), (500_003, 40, 256, 2, 7),
    (400_001, 255, 64, 3, 6), (410_003, 3, 256, 3, 600), (420_001, 11, 256, 1, 13),
    (1_000_001, 36, 256, 3, 300),
])
def test_shallow_apply(n, d, B, D, T):
    rng = np.random.default_rng([n, d, T])
    f = random_forest(T, D, d, B, n + T)
    xb = rng.integers(0, B, (d, n)).astype(np.uint8)
    om = O.Model(D, B, d, f["f0"], f["cut_feature"], f["cut_bin"], np.zeros_like(f["leaf"]),
                 f["leaf"])
    p, F = O.apply(om, xb)
    out = torch.empty(n + 3, device="cuda")
    score = torch.empty(n, dtype=torch.float64, device="cuda")
    # values whose codes are xb: boundary k at k + 1, value = code + 1/2
    bounds = np.repeat(np.arange(1, B, dtype=np.float32)[None], d, axis=0)
    m = _model(f, d, B, bounds)
    got = fb.apply(m, fb.Codes.from_numpy(xb), prob=out[3:], score=score)
    assert np.array_equal(score.cpu().numpy(), F)
    assert np.allclose(got.cpu().numpy(), p, rtol=0, atol=6e-8)
    x = torch.zeros(d, n + 5, device="cuda")[:, 1:n + 1]   # rows of an odd start and stride
    x.copy_(torch.from_numpy(xb).float() + 0.5)
    score.zero_()
    got = fb.apply_float(m, x, prob=out[1:n + 1], score=score)
    assert np.array_equal(score.cpu().numpy(), F)
    assert np.allclose(got.cpu().numpy(), p, rtol=0, atol=6e-8)


@pytest.mark.parametrize("n,d,B,D,T,missing", [
    (1, 1, 2, 4, 1, False), (259, 40, 256, 6, 17, False), (1000, 255, 256, 7, 40, False),
    (393_217, 9, 256, 4, 5, False), (400_003, 40, 64, 7, 60, False), (450_001, 255, 256, 5, 3, False),
    (1, 1, 2, 1, 1, True), (257, 12, 255, 3, 9, True), (1023, 40, 100, 7, 33, True),
    (393_219, 7, 255, 2, 4, True), (400_001, 60, 200, 6, 30, True),
])
def test_deep_and_missing_apply(n, d, B, D, T, missing):
    rng = np.random.default_rng([n, d, T])
    f = random_forest(T, D, d, B, n + T)
    xb = rng.integers(0, B, (d, n)).astype(np.uint8)
    inner = None
    if missing:
        inner = rng.normal(0.0, 0.05, f["cut_bin"].shape)
        xb[rng.random((d, n)) < 0.2] = 255
    om = O.Model(D, B, d, f["f0"], f["cut_feature"], f["cut_bin"], np.zeros_like(f["leaf"]),
                 f["leaf"], inner)
    p, F = O.apply(om, xb)
    bounds = np.repeat(np.arange(1, B, dtype=np.float32)[None], d, axis=0)
    m = fb.Model.from_arrays(f["cut_feature"], f["cut_bin"], f["leaf"], f["f0"], d, B,
                             boundaries=bounds, inner=inner)
    score = torch.empty(n, dtype=torch.float64, device="cuda")
    got = fb.apply(m, fb.Codes.from_numpy(xb), score=score)
    assert np.array_equal(score.cpu().numpy(), F)
    assert np.allclose(got.cpu().numpy(), p, rtol=0, atol=6e-8)
    x = xb.astype(np.float32) + 0.5
    if missing:
        x[xb == 255] = np.nan
    wide = torch.zeros(d, n + 5, device="cuda")[:, 1:n + 1]
    wide.copy_(torch.from_numpy(x))
    score.zero_()
    fb.apply_float(m, wide, score=score)
    assert np.array_equal(score.cpu().numpy(), F)


def test_calls_of_few_and_many_events_interleave():
    """Both kernels' node records stay in place for launches still queued."""
    d, B, D, T = 40, 256, 3, 400
    f = random_forest(T, D, d, B, 3)
    m = _model(f, d, B)
    xb = torch.randint(0, B, (d, 1_000_000), dtype=torch.uint8, device="cuda")
    big = fb.Codes(xb, 1_000_000)
    few = fb.Codes(xb[:, :512].contiguous(), 500)
    p_big, p_few = fb.apply(m, big), fb.apply(m, few)
    torch.cuda.synchronize()
    runs = [(fb.apply(m, big), fb.apply(m, few)) for _ in range(4)]
    torch.cuda.synchronize()
    for a, b in runs:
        assert torch.equal(a, p_big) and torch.equal(b, p_few)
    assert torch.equal(p_few, p_big[:500])


@pytest.mark.parametrize("d,D,T,missing,floats", [
    (40, 3, 400, False, False), (8, 3, 100, False, True), (30, 6, 40, False, False),
    (20, 4, 30, True, True),
])
def test_sizes_share_a_model(d, D, T, missing, floats):
    """One warm-up call readies a model for captures of every size (other
    sizes take other launch shapes and node records), and a captured call
    replays after calls of other sizes."""
    B = 200
    f = random_forest(T, D, d, B, 11)
    inner = np.random.default_rng(5).normal(0.0, 0.05, f["cut_bin"].shape) if missing else None
    bounds = np.repeat(np.arange(1, B, dtype=np.float32)[None], d, axis=0)
    m = fb.Model.from_arrays(f["cut_feature"], f["cut_bin"], f["leaf"], f["f0"], d, B,
                             boundaries=bounds, inner=inner)
    sizes = [500, 400_000, 700_000, 1_100_000, 1_700_000, 2_500_000]
    xb = torch.randint(0, B, (d, sizes[-1]), dtype=torch.uint8, device="cuda")
    x = xb.float() + 0.5
    if missing:
        x[:, ::7] = float("nan")

    def call(n, prob):
        if floats:
            return fb.apply_float(m, x[:, :n], prob=prob)
        return fb.apply(m, fb.Codes(xb, n), prob=prob)

    call(500, torch.empty(500, device="cuda"))
    torch.cuda.synchronize()
    outs = [torch.zeros(n, device="cuda") for n in sizes]
    graphs = []
    for n, out in zip(sizes, outs):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            call(n, out)
        graphs.append(g)
    whole = call(sizes[-1], torch.empty(sizes[-1], device="cuda"))
    for _ in range(2):
        for g in graphs:
            g.replay()
        torch.cuda.synchronize()
        for n, out in zip(sizes, outs):
            assert torch.equal(out, whole[:n]), n
            out.zero_()


@pytest.mark.parametrize("n,d,B,D,T,missing", [
    (1000, 255, 256, 3, 3000, False), (393_217, 160, 256, 3, 3000, False),
    (259, 255, 256, 6, 300, False), (394_001, 100, 256, 6, 300, False),
    (77, 255, 255, 7, 200, True), (393_219, 110, 255, 2, 4000, True),
    # fits beside a few trees only: kept in memory for the chunks it would add
    (500, 126, 256, 3, 12_000, False), (513, 110, 256, 6, 1000, False), (255, 118, 200, 7, 400, True),
])
def test_threshold_tables_beyond_the_lds(n, d, B, D, T, missing):
    """Float values of forests whose thresholds do not fit the LDS beside a
    tile score as their codes do."""
    f = random_forest(T, D, d, B, n + T)
    rng = np.random.default_rng([n, d, T, 2])
    inner = rng.normal(0.0, 0.05, f["cut_bin"].shape) if missing else None
    bounds = np.repeat(np.arange(1, B, dtype=np.float32)[None], d, axis=0)
    m = fb.Model.from_arrays(f["cut_feature"], f["cut_bin"], f["leaf"], f["f0"], d, B,
                             boundaries=bounds, inner=inner)
    codes = fb.Codes.empty(d, n)
    codes.data[:, :n] = torch.randint(0, B, (d, n), dtype=torch.uint8, device="cuda")
    x = codes.data[:, :n].float() + 0.5
    if missing:
        codes.data[::3, :n:5] = 255
        x[::3, ::5] = float("nan")
    want = torch.empty(n, dtype=torch.float64, device="cuda")
    score = torch.zeros_like(want)
    fb.apply(m, codes, score=want)
    fb.apply_float(m, x, score=score)
    assert torch.equal(score, want)


@pytest.mark.parametrize("n,d,B,D,T,missing", [
    (1, 1, 2, 1, 1, False), (65, 40, 256, 3, 7, False), (100_001, 40, 256, 3, 230, False),
    (5_003, 255, 256, 5, 40, False), (20_011, 9, 200, 7, 33, True), (70_001, 3, 255, 2, 9, True),
])
def test_event_importance(n, d, B, D, T, missing):
    rng = np.random.default_rng([n, d, T, 1])
    f = random_forest(T, D, d, B, n + T)
    gain = rng.exponential(1.0, f["cut_bin"].shape)
    xb = rng.integers(0, B, (d, n)).astype(np.uint8)
    inner = None
    if missing:
        inner = rng.normal(0.0, 0.05, f["cut_bin"].shape)
        xb[rng.random((d, n)) < 0.2] = 255
    om = O.Model(D, B, d, f["f0"], f["cut_feature"], f["cut_bin"], gain, f["leaf"], inner)
    m = fb.Model.from_arrays(f["cut_feature"], f["cut_bin"], f["leaf"], f["f0"], d, B, gain=gain,
                             inner=inner)
    got = fb.event_importance(m, fb.Codes.from_numpy(xb)).cpu().numpy()
    assert np.array_equal(got, O.event_importance(om, xb))


@pytest.mark.parametrize("threads", [64, 192, 1024])
@pytest.mark.parametrize("n,d,B,D,T", [(70_001, 160, 256, 3, 300), (5_003, 255, 256, 6, 40)])
def test_requested_workgroup_sizes(n, d, B, D, T, threads):
    """A workgroup size that is asked for scores as the planner's does, also
    where the tile has to shrink to leave room for trees."""
    f = random_forest(T, D, d, B, n + T)
    bounds = np.repeat(np.arange(1, B, dtype=np.float32)[None], d, axis=0)
    m = _model(f, d, B, bounds)
    codes = fb.Codes.empty(d, n)
    codes.data[:, :n] = torch.randint(0, B, (d, n), dtype=torch.uint8, device="cuda")
    x = codes.data[:, :n].float() + 0.5
    want = fb.apply(m, codes)
    fb.set_option("apply_threads", threads)
    try:
        assert torch.equal(fb.apply(m, codes), want)
        assert torch.equal(fb.apply_float(m, x), want)
    finally:
        fb.set_option("apply_threads", 0)


@pytest.mark.parametrize("T,D", [(1000, 7), (3000, 3)])
def test_first_float_call_of_a_model_is_no_sort(T, D):
    """A model's first apply_float makes its threshold table and ranks in time
    linear in its nodes, like the records of its first apply: medians over
    nine models, with a sort and a search per node 12 and 6 times the binned
    call's (0.8 and 9.6 ms at 1,000 trees of depth 7)."""
    import time
    d, B = 40, 200
    codes = fb.Codes.empty(d, 64)
    x = torch.rand(d, 64, device="cuda") * B
    bounds = np.repeat(np.arange(1, B, dtype=np.float32)[None], d, axis=0)
    took = {"codes": [], "values": []}
    for seed in range(10):
        f = random_forest(T, D, d, B, seed)
        for name in took:
            m = _model(f, d, B, bounds)
            torch.cuda.synchronize()
            t = time.perf_counter()
            fb.apply(m, codes) if name == "codes" else fb.apply_float(m, x)
            torch.cuda.synchronize()
            if seed:
                took[name].append(time.perf_counter() - t)
    a, b = (float(np.median(took[k])) for k in took)
    print(f"first calls: codes {a * 1e6:.0f} us, values {b * 1e6:.0f} us", flush=True)
    assert b <= 4 * a
