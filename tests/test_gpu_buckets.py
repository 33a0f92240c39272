"""The d = 2 bucketed cell search against the full scan and the oracle.

Each bucket of a layer's reachable box lists every grid point that can be
the FP32 argmin of the half-norm key anywhere in it (the key's rounding
slack included), so the cell must be the brute-force search's cell (Sec. 2:
the nearest-neighbour projection; Sec. 4: the brute-force search) bit for
bit: on the time-layer samples themselves, on the grid points, on midpoints
of neighbouring points (near-ties), on points placed exactly on bucket
edges and one ulp either side, on duplicated grid points (exact ties), and
outside the box (the full-scan fallback); counts with the tables on and off
equal the oracle's."""
import numpy as np
import pytest

import oracle as O
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1101_3228_amd as qt  # noqa: E402


def _case(name):
    print(f"[gpu-case] {name}", flush=True)


def _omodel(spec):
    return O.Model(spec["d"], spec["n"], spec["A"], spec["b"], spec["T"], spec["mu"], spec["L"],
                   spec["x0"])


def _edge_points(plan, k, g, rng, count=3000):
    """Points on bucket edges of layer k (and one ulp either side) along
    both axes, the other coordinate drawn inside the box."""
    lo, sc, B = plan.buckets(k)
    if B[0] == 0:
        return np.zeros((0, 2), np.float32)
    f32 = np.float32
    pts = []
    for axis in (0, 1):
        i = rng.integers(0, B[axis] + 1, count)
        # the FP32 edge lo + i / scale and its neighbours
        e = (lo[axis] + (i.astype(np.float32) / sc[axis]).astype(f32)).astype(f32)
        other = 1 - axis
        span = (B[other] / sc[other]).astype(f32)
        o = (lo[other] + rng.random(count).astype(f32) * span).astype(f32)
        for v in (e, np.nextafter(e, f32(-np.inf)), np.nextafter(e, f32(np.inf))):
            p = np.empty((count, 2), f32)
            p[:, axis] = v
            p[:, other] = o
            pts.append(p)
    return np.concatenate(pts)


GRIDS = {
    "product": lambda spec: synth.layer_grids(spec, [1] + [(40, 50)] * spec["n"],
                                              base=qt.gauss_quantizer),
    "quantile": lambda spec: synth.layer_grids(spec, [1] + [700] * spec["n"]),
    "jitter_ties": lambda spec: synth.layer_grids(spec, [1] + [300] * spec["n"],
                                                  rng=np.random.default_rng(3), jitter=0.3),
}


@pytest.mark.parametrize("model,grid", [("bm2", "product"), ("ou2", "quantile"),
                                        ("bm2", "jitter_ties")])
def test_bucketed_cells_equal_full_scan_and_oracle(model, grid):
    _case(f"bucketed cells {model} {grid}")
    spec = (synth.bm_model(2, 4, T=1.0, rho=0.3) if model == "bm2"
            else synth.ou_model(4, alpha=(0.5, 8.0), sig=(0.7, 1.3), rho=-0.6))
    g_all, N = GRIDS[grid](spec)
    if grid == "jitter_ties":
        # exact ties: every layer repeats some of its points
        off = np.concatenate([[0], np.cumsum(N)])
        for k in range(1, spec["n"] + 1):
            blk = g_all[off[k]:off[k + 1]]
            blk[1::7] = blk[0::7][:len(blk[1::7])]
    plan = qt.Plan(spec, g_all, N)
    off = np.concatenate([[0], np.cumsum(N)])
    rng = np.random.default_rng(17)
    for k in range(spec["n"] + 1):
        g = g_all[off[k]:off[k + 1]].reshape(-1, 2)
        lo, sc, B = plan.buckets(k)
        if N[k] > 1:
            assert B[0] == B[1] and B[0] * B[0] >= 8 * N[k]
        else:
            assert B[0] == 0
        pts = [g.astype(np.float32), ((g[:-1] + g[1:]) * 0.5).astype(np.float32),
               _edge_points(plan, k, g, rng),
               (rng.standard_normal((20_000, 2)) * 8.0).astype(np.float32)]   # also far out
        kk = min(k, spec["n"] - 1)
        xs, ys = qt.layer_samples(plan, kk, 0, 200_000, seed=0x5EED0050)
        pts.append((xs if k == kk else ys).cpu().numpy())
        x = np.concatenate(pts).astype(np.float32)
        xd = torch.from_numpy(x).cuda()
        got = qt.cells(plan, k, xd).cpu().numpy()
        plan.tune(buckets=0)
        full = qt.cells(plan, k, xd).cpu().numpy()
        plan.tune(buckets=1)
        ref = O.cells_bulk(g, 2, x)
        assert np.array_equal(full, ref), k
        assert np.array_equal(got, ref), (k, int(np.sum(got != ref)))


def test_bucketed_counts_equal_full_scan_and_oracle():
    """The 2-D workload's grids (40 x 50 products mapped by sqrt(t_k)
    chol(R)) on 8 layers, M = 400 001 pairs per layer: counts with and
    without the tables equal the oracle's."""
    _case("bucketed counts, 2-D workload grids, n=8, M=400001")
    spec = synth.bm_model(2, 8, T=1.0, rho=0.3)
    grid, N = synth.layer_grids(spec, [1] + [(40, 50)] * 8, base=qt.gauss_quantizer)
    plan = qt.Plan(spec, grid, N)
    assert plan.tuning()["nd_samples"] == 4  # the default with bucket tables
    M, seed = 400_001, 0x5EED0051
    ref = O.transitions(_omodel(spec), grid, N, M, seed=seed, contract=3, nthreads=16)
    # both samples-per-lane settings, with and without the tables
    for s in (4, 8):
        plan.tune(nd_samples=s, buckets=1)
        on = plan.transitions(M, seed, contract=3).cpu().numpy()
        plan.tune(buckets=0)
        off_ = plan.transitions(M, seed, contract=3).cpu().numpy()
        assert np.array_equal(off_, ref), s
        assert np.array_equal(on, ref), s
    plan.tune(nd_samples=4, buckets=1)


@pytest.mark.parametrize("case", ["ring", "piles", "line", "huge"])
def test_lists_of_many_candidates(case):
    """Rows past the four candidates of the straight-line search, past the
    seven of a row (pool rows), past the 31 of a pool row (the full scan): a
    ring of points whose cells all meet in its centre, piles of 1 to 40 equal
    points, points on a line, and a layer at the point limit (byte offsets up
    to 8 x 4096)."""
    _case(f"bucket lists {case}")
    rng = np.random.default_rng(5)
    if case == "ring":
        t = np.linspace(0.0, 2.0 * np.pi, 24, endpoint=False)
        g = np.concatenate([np.stack([np.cos(t), np.sin(t)], 1) * r for r in (1.0, 1.0 + 1e-7)])
    elif case == "piles":
        c = rng.standard_normal((12, 2))
        g = np.repeat(c, [1, 2, 3, 4, 5, 6, 7, 8, 9, 31, 32, 40], axis=0)
        g = g[rng.permutation(len(g))]
    elif case == "line":
        g = np.stack([np.linspace(-3, 3, 200), np.zeros(200)], 1)
    else:
        g = rng.standard_normal((4096, 2))
    spec = synth.bm_model(2, 2, T=1.0)
    g = g.astype(np.float32)
    grid = np.concatenate([np.zeros((1, 2), np.float32), g, g])
    N = np.array([1, len(g), len(g)], np.int32)
    plan = qt.Plan(spec, grid, N)
    c = plan.bucket_counts(1)
    if case == "ring":
        assert ((c > 7) & (c != 0xFFFF)).any()
    if case == "piles":
        assert (c == 0xFFFF).any() and ((c > 7) & (c < 32)).any() and ((c > 4) & (c < 8)).any()
    x = np.concatenate([rng.standard_normal((30_000, 2)), 1e-3 * rng.standard_normal((30_000, 2)),
                        g]).astype(np.float32)
    got = qt.cells(plan, 1, torch.from_numpy(x).cuda()).cpu().numpy()
    assert np.array_equal(got, O.cells_bulk(g, 2, x))
    ref = O.transitions(_omodel(spec), grid, N, 30_001, seed=9, nthreads=8)
    assert np.array_equal(plan.transitions(30_001, 9).cpu().numpy(), ref)
    ref = O.transitions(_omodel(spec), grid, N, 30_001, seed=9, mode=1, nthreads=8)
    assert np.array_equal(plan.transitions(30_001, 9, mode=qt.PATHWISE).cpu().numpy(), ref)


def _grid_3d(case, rng):
    if case == "product":  # eight cells meet at a corner
        a, b, c = qt.gauss_quantizer(7), qt.gauss_quantizer(8), qt.gauss_quantizer(9)
        return np.stack(np.meshgrid(a, b, c, indexing="ij"), -1).reshape(-1, 3)
    if case == "sphere":  # more than fifteen cells meet in the centre: the full scan
        g = rng.standard_normal((40, 3))
        return g / np.linalg.norm(g, axis=1, keepdims=True)
    if case == "piles":  # exact ties, lists up to the row's fifteen and beyond
        c = rng.standard_normal((10, 3))
        g = np.repeat(c, [1, 2, 3, 4, 5, 8, 14, 15, 16, 70], axis=0)
        return g[rng.permutation(len(g))]
    if case == "plane":
        g = rng.standard_normal((150, 3))
        g[:, 2] = 0.25
        return g
    return rng.standard_normal((int(case), 3))


@pytest.mark.parametrize("case", ["product", "sphere", "piles", "plane", "2", "17", "1100"])
def test_3d_tables_equal_full_scan_and_oracle(case):
    """d = 3 counts, layerwise and pathwise, with the tables on and off."""
    _case(f"3-D tables {case}")
    g = _grid_3d(case, np.random.default_rng(5)).astype(np.float32)
    spec = synth.bm_model(3, 3, T=1.0, rho=0.3)
    grid = np.concatenate([np.zeros((1, 3), np.float32), g, 2.0 * g, g[: len(g) // 2 + 1]])
    N = np.array([1, len(g), len(g), len(g) // 2 + 1], np.int32)
    plan = qt.Plan(spec, grid, N)
    M = 30_011
    for mode in (0, qt.PATHWISE):
        ref = O.transitions(_omodel(spec), grid, N, M, seed=9, mode=mode, nthreads=8)
        for on in (1, 0):
            plan.tune(buckets=on)
            got = plan.transitions(M, 9, mode=mode).cpu().numpy()
            assert np.array_equal(got, ref), (mode, on)
    plan.tune(buckets=1)


def test_3d_plan_in_a_workspace_without_room_for_tables(monkeypatch):
    """The layers' records and one chunk per layer alone (no tables, no
    pathwise scratch) still give the same counts."""
    _case("3-D workspace without tables")
    rng = np.random.default_rng(6)
    g = rng.standard_normal((60, 3)).astype(np.float32)
    spec = synth.bm_model(3, 2, T=1.0)
    grid = np.concatenate([np.zeros((1, 3), np.float32), g, g])
    N = np.array([1, 60, 60], np.int32)
    M = 20_001
    ref = O.transitions(_omodel(spec), grid, N, M, seed=4, nthreads=8)
    full = qt.Plan(spec, grid, N)
    assert np.array_equal(full.transitions(M, 4).cpu().numpy(), ref)
    monkeypatch.setattr(qt, "workspace_size", lambda *args: 64 * 1024)
    small = qt.Plan(spec, grid, N)
    assert small.batch_samples > 0
    assert np.array_equal(small.transitions(M, 4).cpu().numpy(), ref)
    assert np.array_equal(small.transitions(M, 4, mode=qt.PATHWISE).cpu().numpy(),
                          full.transitions(M, 4, mode=qt.PATHWISE).cpu().numpy())


@pytest.mark.parametrize("d", [2, 3])
def test_boxes_beyond_the_type_have_no_tables(d):
    """Coefficients whose box passes FP32's range (the samples drawn here stay
    within it): no tables, and the full scan's counts."""
    _case(f"box beyond FP32 {d}-D")
    rng = np.random.default_rng(11)
    scale = np.float32(8.5e37)
    spec = synth.bm_model(d, 2, T=2.0)
    spec["A"][1] = 0.0
    for k in range(2):
        spec["T"][k] = scale * np.eye(d, dtype=np.float32)
        spec["L"][k + 1] = scale * np.eye(d, dtype=np.float32)
    g = (0.1 * rng.standard_normal((60, d))).astype(np.float32)
    grid = np.concatenate([np.zeros((1, d), np.float32), g, g[::-1]])
    N = np.array([1, len(g), len(g)], np.int32)
    plan = qt.Plan(spec, grid, N)
    M = 501
    for k in (1, 2):
        lo, sc, B = plan.buckets(k)
        assert (B == 0).all()
    x, y = qt.layer_samples(plan, 1, 0, M, 3)
    assert torch.isfinite(x).all() and torch.isfinite(y).all()
    for mode in (0, qt.PATHWISE):
        ref = O.transitions(_omodel(spec), grid, N, M, seed=3, mode=mode, nthreads=8)
        assert np.array_equal(plan.transitions(M, 3, mode=mode).cpu().numpy(), ref), mode


def _forward_ms(plan, M, counts):
    best = np.inf
    for _ in range(8):
        e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        e0.record()
        plan.transitions(M, 9, counts=counts)
        e1.record()
        torch.cuda.synchronize()
        best = min(best, e0.elapsed_time(e1))
    return best


@pytest.mark.parametrize("rho,M", [(0.0, 300_001), (0.95, 30_011), (0.95, 1_000_001),
                                   (0.99, 300_001)])
def test_3d_grids_that_lists_do_not_answer_are_scanned(rho, M):
    """Thin clouds crowd the buckets: with the tables on, a layerwise call takes
    no longer than the full scan, and the counts are the same."""
    _case(f"3-D thin clouds {rho} {M}")
    spec = synth.bm_model(3, 4, rho=rho)
    grid, N = synth.layer_grids(spec, [1] + [1000] * 4)
    plan = qt.Plan(spec, grid, N, batch_samples=M)
    times, counts = [], [plan.new_counts() for _ in range(2)]
    for on in (1, 0):
        plan.tune(buckets=on)
        times.append(_forward_ms(plan, M, counts[on]))
    assert torch.equal(counts[0], counts[1])
    if M < 100_000:
        ref = O.transitions(_omodel(spec), grid, N, M, seed=9, nthreads=8)
        assert np.array_equal(counts[0][:plan.entries].cpu().numpy(), ref)
    assert times[0] < 1.25 * times[1], times
    if rho == 0.0:
        assert times[0] < 0.7 * times[1], times


@pytest.mark.parametrize("sizes", [[23, 24, 8, 40], [4, 23, 2, 12], [24, 25, 3, 24]], ids=str)
@pytest.mark.parametrize("mode", [0, 1])
def test_3d_layers_on_either_side_of_the_tables(sizes, mode):
    """Layers of fewer than 24 points have no tables; beside others that have
    them, and alone."""
    _case(f"3-D small layers {sizes} {mode}")
    rng = np.random.default_rng(13)
    spec = synth.bm_model(3, len(sizes), T=1.0, rho=0.2)
    grid = np.concatenate([np.zeros((1, 3))] + [rng.standard_normal((s, 3)) for s in sizes])
    grid = grid.astype(np.float32)
    N = np.array([1] + sizes, np.int32)
    plan = qt.Plan(spec, grid, N)
    ref = O.transitions(_omodel(spec), grid, N, 30_011, seed=4, mode=mode, nthreads=8)
    assert np.array_equal(plan.transitions(30_011, 4, mode=mode).cpu().numpy(), ref)


def test_3d_small_layers_take_no_longer_than_the_scan():
    _case("3-D small layers' time")
    spec = synth.bm_model(3, 50, T=1.0, rho=0.2)
    grid, N = synth.layer_grids(spec, [1] + [(2, 2, 2)] * 50)
    plan = qt.Plan(spec, grid, N, batch_samples=1_000_000)
    counts, times = plan.new_counts(), []
    for on in (1, 0):
        plan.tune(buckets=on)
        times.append(_forward_ms(plan, 1_000_000, counts))
    assert times[0] < 1.08 * times[1], times


@pytest.mark.parametrize("large", [64, 100])
def test_3d_plans_of_many_buckets(large):
    """64 layers of 4096 points take 16 buckets a point instead of 32, 100 of
    them none (all layers alike)."""
    _case(f"3-D many buckets {large}")
    rng = np.random.default_rng(14)
    n = 2 * large
    spec = synth.bm_model(3, n, T=1.0, rho=0.2)
    g = rng.standard_normal((4096, 3))
    parts, N = [np.zeros((1, 3))], [1]
    for k in range(1, n + 1):
        parts.append(g * np.sqrt(k / n) if k % 2 else np.zeros((1, 3)))
        N.append(len(parts[-1]))
    grid, N = np.concatenate(parts).astype(np.float32), np.array(N, np.int32)
    plan = qt.Plan(spec, grid, N, batch_samples=1)
    rows = qt.workspace_size(3, n, N, 1) / 32
    assert (rows > 5_000_000) == (large == 64)
    for mode in (0, 1):
        ref = O.transitions(_omodel(spec), grid, N, 300, seed=4, mode=mode, nthreads=8)
        assert np.array_equal(plan.transitions(300, 4, mode=mode).cpu().numpy(), ref), mode


@pytest.mark.parametrize("shape", [(2, 3, 20), (2, 3, 32), (3, 3, 24), (2, 3, 50)], ids=str)
@pytest.mark.parametrize("mode", [0, 1])
def test_3d_small_grids_of_uneven_sides(shape, mode):
    """Grids with one long side leave 0.05 to 0.12 of the samples without a
    list: counts equal the scan's and the oracle's, and a call takes no longer
    than by the scan (100 layers of 192 points took 1.5 times as long)."""
    _case(f"3-D uneven sides {shape} {mode}")
    spec = synth.bm_model(3, 50, T=1.0)
    grid, N = synth.layer_grids(spec, [1] + [shape] * 50)
    plan = qt.Plan(spec, grid, N, batch_samples=200_000)
    for M in (2_003, 20_011, 100_003):
        counts, times = [], []
        for on in (1, 0):
            plan.tune(buckets=on)
            best = float("inf")
            for _ in range(6):
                a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
                a.record()
                c = plan.transitions(M, 3, mode=mode)
                b.record()
                torch.cuda.synchronize()
                best = min(best, a.elapsed_time(b))
            counts.append(c)
            times.append(best)
        assert torch.equal(counts[0], counts[1])
        assert times[0] < 1.3 * times[1], (M, times)
    ref = O.transitions(_omodel(spec), grid, N, 2_003, seed=3, mode=mode, nthreads=8)
    assert np.array_equal(plan.transitions(2_003, 3, mode=mode).cpu().numpy(), ref)


def _cells_ms(plan, x):
    best = np.inf
    for _ in range(8):
        e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        e0.record()
        qt.cells(plan, 1, x)
        e1.record()
        torch.cuda.synchronize()
        best = min(best, e0.elapsed_time(e1))
    return best


@pytest.mark.parametrize("m", [100, 1 << 17, (1 << 17) + 1, 300_001])
@pytest.mark.parametrize("out", [1, 16, 17, 64])
def test_points_without_a_list_among_others(out, m):
    """`out` of every 64 points outside the box (scanned for by the wave up to
    16 of them, by each lane beyond), with repeated grid points, in calls of one
    point a lane and of eight, and as layers of the forward."""
    _case(f"bucketed cells {out} of 64 outside, {m} points")
    rng = np.random.default_rng(8)
    g = rng.standard_normal((301, 2))
    g[200:240] = g[100:140]
    spec = synth.bm_model(2, 2, T=1.0)
    g = g.astype(np.float32)
    grid = np.concatenate([np.zeros((1, 2), np.float32), g, g])
    plan = qt.Plan(spec, grid, np.array([1, 301, 301], np.int32))
    x = rng.standard_normal((m, 2)) * 0.7
    far = np.arange(m) % 64 >= 64 - out
    x[far] = 40.0 * x[far] / np.linalg.norm(x[far], axis=1, keepdims=True)
    x = x.astype(np.float32)
    got = qt.cells(plan, 1, torch.from_numpy(x).cuda()).cpu().numpy()
    assert np.array_equal(got, O.cells_bulk(g, 2, x))


@pytest.mark.parametrize("N,m", [(1024, (1 << 19) + 1), (1025, 1 << 19), (1025, (1 << 19) + 1),
                                 (60, 1 << 21), (60, (1 << 21) + 1)])
def test_cells_with_one_and_eight_points_a_lane(N, m):
    _case(f"bucketed cells N={N} m={m}")
    rng = np.random.default_rng(4)
    g = rng.standard_normal((N, 2)).astype(np.float32)
    spec = synth.bm_model(2, 2, T=1.0)
    grid = np.concatenate([np.zeros((1, 2), np.float32), g, g])
    plan = qt.Plan(spec, grid, np.array([1, N, N], np.int32))
    x = rng.standard_normal((m, 2)).astype(np.float32)
    x[::5000] *= 30.0
    got = qt.cells(plan, 1, torch.from_numpy(x).cuda()).cpu().numpy()
    assert np.array_equal(got, O.cells_bulk(g, 2, x))


@pytest.mark.parametrize("shape", ["circle", "line", "five rows"])
def test_2d_grids_with_scans(shape):
    """Grids whose lists hold too many points in a part of the box or in all of
    it: both modes, the tables on and off, against the oracle."""
    _case(f"2-D grids with scans: {shape}")
    if shape == "circle":
        t = np.arange(400) * 2 * np.pi / 400
        g = 1.5 * np.stack([np.cos(t), np.sin(t)], 1)
    elif shape == "line":
        g = np.stack([np.zeros(999), np.sort(np.random.default_rng(2).standard_normal(999))], 1)
    else:
        a, b = synth.quantile_grid_1d(5), synth.quantile_grid_1d(400)
        g = np.stack([m.ravel() for m in np.meshgrid(a, b, indexing="ij")], 1)
    g = g.astype(np.float32)
    spec = synth.bm_model(2, 3, T=1.0, rho=0.3)
    grid = np.concatenate([np.zeros((1, 2), np.float32), g, g, g])
    N = np.array([1] + [len(g)] * 3, np.int32)
    plan = qt.Plan(spec, grid, N)
    for mode in (qt.LAYERWISE, qt.PATHWISE):
        ref = O.transitions(_omodel(spec), grid, N, 20_011, seed=9, mode=mode, nthreads=8)
        for on in (1, 0):
            plan.tune(buckets=on)
            assert np.array_equal(plan.transitions(20_011, 9, mode=mode).cpu().numpy(), ref)


def test_a_point_without_a_list_does_not_hold_up_its_wave():
    _case("bucketed cells, time with one point of 64 outside")
    spec = synth.bm_model(2, 2, T=1.0)
    grid, N = synth.layer_grids(spec, [1] + [(50, 50)] * 2)
    plan = qt.Plan(spec, grid, N)
    x = 0.5 * np.random.default_rng(1).standard_normal((100_000, 2)).astype(np.float32)
    inside = _cells_ms(plan, torch.from_numpy(x).cuda())
    x[::64] = 40.0
    assert _cells_ms(plan, torch.from_numpy(x).cuda()) < 3.0 * inside + 0.02
