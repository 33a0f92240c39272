"""GPU checks of the pathwise counts where their kernels change form, bit for
bit against the oracle: layers in groups of four (d = 1) and a remainder, one
super tile and several, the bucket tables and the full scan (d = 2), d = 3,
layers too large for the staged search (or, d = 2, for several layers' points
in LDS beside small neighbours), more paths than one pass of the cell
scratch holds, added counts, a workspace without the scratch or shared with
layerwise calls, other streams and threads, and captured calls."""
import numpy as np
import pytest

import oracle as O
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1101_3228_amd as qt  # noqa: E402

SEED = 0x5EED0007


def _case(name):
    print(f"[gpu-case] {name}", flush=True)


def _model(spec):
    return O.Model(spec["d"], spec["n"], spec["A"], spec["b"], spec["T"], spec["mu"], spec["L"],
                   spec["x0"])


def _ref(spec, grid, N, M, **kw):
    return O.transitions(_model(spec), grid, N, M, seed=SEED, mode=1, nthreads=8, **kw)


@pytest.mark.parametrize("sizes", [[1, 5], [1, 2, 1, 300], [1, 100, 99, 257, 128, 64],
                                   [1, 10, 4100, 12, 700, 3, 1, 2, 9]], ids=str)
@pytest.mark.parametrize("M", [1, 257, 20_001])
def test_paths_1d(sizes, M):
    _case(f"paths 1-D {sizes} {M}")
    spec = synth.bm_model(1, len(sizes) - 1)
    grid, N = synth.layer_grids(spec, sizes)
    plan = qt.Plan(spec, grid, N, batch_samples=1)
    got = plan.transitions(M, SEED, mode=qt.PATHWISE, m0=3).cpu().numpy()
    assert np.array_equal(got, _ref(spec, grid, N, M, m0=3))


@pytest.mark.parametrize("sizes", [[1, 1024, 7], [1, 1025, 3, 1024, 5, 2048], [1, 2, 513, 12]],
                         ids=str)
def test_paths_1d_staged_and_not(sizes):
    """Midpoints through LDS up to 1024 points a layer, from memory beyond;
    through the cells and on the spot."""
    _case(f"paths 1-D staged or not {sizes}")
    spec = synth.bm_model(1, len(sizes) - 1)
    grid, N = synth.layer_grids(spec, sizes)
    plan = qt.Plan(spec, grid, N, batch_samples=1)
    ref = _ref(spec, grid, N, 30_001)
    for p in (plan, _without_cells(plan)):
        assert np.array_equal(p.transitions(30_001, SEED, mode=qt.PATHWISE).cpu().numpy(), ref)


@pytest.mark.parametrize("d,side", [(2, (1, 1)), (2, (5, 6)), (2, (33, 34)), (2, (16, 16)),
                                    (3, (4, 5, 6))], ids=str)
@pytest.mark.parametrize("buckets", [1, 0])
def test_paths_nd(d, side, buckets):
    _case(f"paths {d}-D {side} {buckets}")
    spec = synth.bm_model(d, 5, rho=0.3)
    grid, N = synth.layer_grids(spec, [1, side, side, tuple([2] * d), side, side])
    plan = qt.Plan(spec, grid, N, batch_samples=1).tune(buckets=buckets)
    got = plan.transitions(10_001, SEED, mode=qt.PATHWISE).cpu().numpy()
    assert np.array_equal(got, _ref(spec, grid, N, 10_001))


@pytest.mark.parametrize("sizes", [[1, (1, 2411), (3, 3)], [1, (36, 67), (2, 2), (5, 4)],
                                   [1, (50, 60)], [1, (4, 5), (64, 64), (3, 4), (64, 64)],
                                   [1, (20, 20), (50, 80), (20, 20)]], ids=str)
@pytest.mark.parametrize("buckets", [1, 0])
def test_paths_2d_one_large_layer(sizes, buckets):
    """2411 points are the most whose staged layers fit in LDS; larger ones
    beside small neighbours still have the cell scratch."""
    _case(f"paths 2-D {sizes} {buckets}")
    spec = synth.bm_model(2, len(sizes) - 1, rho=0.3)
    grid, N = synth.layer_grids(spec, sizes)
    plan = qt.Plan(spec, grid, N, batch_samples=1).tune(buckets=buckets)
    counts = plan.transitions(20_001, SEED, mode=qt.PATHWISE)
    assert np.array_equal(counts.cpu().numpy(), _ref(spec, grid, N, 20_001))
    plan.transitions_add(counts, 130, SEED, mode=qt.PATHWISE, m0=20_001)
    assert np.array_equal(counts.cpu().numpy(), _ref(spec, grid, N, 20_131))


def _tree():
    spec = synth.bm_model(1, 6)
    grid, N = synth.layer_grids(spec, [1, 20, 150, 130, 7, 40, 33])
    return spec, grid, N


def test_more_paths_than_a_pass_and_added_counts():
    _case("paths in several passes")
    spec, grid, N = _tree()
    plan = qt.Plan(spec, grid, N, batch_samples=1)
    M = 2 * (1 << 17) + 4097
    ref = _ref(spec, grid, N, M)
    counts = plan.transitions(M, SEED, mode=qt.PATHWISE)
    assert np.array_equal(counts.cpu().numpy(), ref)
    plan.transitions_add(counts, 1000, SEED, mode=qt.PATHWISE, m0=M)
    assert np.array_equal(counts.cpu().numpy(), _ref(spec, grid, N, M + 1000))


def test_workspace_without_the_cell_scratch():
    """A workspace of the tables alone is still accepted and counts directly."""
    _case("paths without scratch")
    import ctypes
    spec, grid, N = _tree()
    plan = qt.Plan(spec, grid, N, batch_samples=1)
    ref = plan.transitions(30_000, SEED, mode=qt.PATHWISE).cpu().numpy()
    model = qt._Model(plan.d, plan.n, *(plan._keep[k].ctypes.data
                                        for k in ("A", "b", "T", "mu", "L", "x0")))
    size = plan.workspace.numel() - 6 * 2 * (1 << 17)   # less than the cells need
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    h = ctypes.c_void_p()
    qt._check(qt.lib().qtree_plan_create(ctypes.byref(model), qt._np_ptr(plan.grid),
                                         qt._np_ptr(plan.N), ws.data_ptr(), size,
                                         ctypes.byref(h)))
    out = plan.new_counts()
    qt._check(qt.lib().qtree_transitions(h, 0, 30_000, SEED, 0, qt.PATHWISE, out.data_ptr(),
                                         qt._stream_handle()))
    torch.cuda.synchronize()
    assert np.array_equal(out[:plan.entries].cpu().numpy(), ref)
    qt.lib().qtree_plan_destroy(h)


def test_paths_on_two_streams_share_the_plan():
    _case("paths on two streams")
    spec, grid, N = _tree()
    plan = qt.Plan(spec, grid, N, batch_samples=1)
    streams = [torch.cuda.Stream() for _ in range(2)]
    outs = [plan.new_counts() for _ in range(6)]
    torch.cuda.synchronize()
    for i, out in enumerate(outs):
        plan.transitions(50_000, SEED, contract=i, mode=qt.PATHWISE, counts=out,
                         stream=streams[i % 2])
    torch.cuda.synchronize()
    for i, out in enumerate(outs):
        ref = O.transitions(_model(spec), grid, N, 50_000, seed=SEED, contract=i, mode=1,
                            nthreads=8)
        assert np.array_equal(out[:plan.entries].cpu().numpy(), ref), i


def test_paths_of_threads_on_their_own_default_streams():
    """One handle (hipStreamPerThread) names a stream of each host thread;
    their calls share the plan's scratch."""
    _case("paths on per-thread streams")
    import threading
    per_thread = 2                      # the value of the hipStreamPerThread handle
    spec, grid, N = _tree()
    plan = qt.Plan(spec, grid, N, batch_samples=1)
    threads, calls, M = 4, 12, 50_000
    outs = [[plan.new_counts() for _ in range(calls)] for _ in range(threads)]
    torch.cuda.synchronize()
    go, failed = threading.Barrier(threads), []

    def work(t):
        torch.cuda.set_device(0)
        go.wait()
        for c in range(calls):
            status = qt.lib().qtree_transitions(plan.handle, 0, M, SEED, calls * t + c,
                                                qt.PATHWISE, outs[t][c].data_ptr(), per_thread)
            if status:
                failed.append((t, c, status))
        torch.cuda.ExternalStream(per_thread).synchronize()

    pool = [threading.Thread(target=work, args=(t,)) for t in range(threads)]
    for th in pool:
        th.start()
    for th in pool:
        th.join()
    torch.cuda.synchronize()
    assert not failed
    for t in range(threads):
        for c in range(calls):
            ref = O.transitions(_model(spec), grid, N, M, seed=SEED, contract=calls * t + c,
                                mode=1, nthreads=8)
            assert np.array_equal(outs[t][c][:plan.entries].cpu().numpy(), ref), (t, c)


def test_captured_paths_replay():
    _case("paths captured")
    spec, grid, N = _tree()
    plan = qt.Plan(spec, grid, N, batch_samples=1)
    ref = _ref(spec, grid, N, 20_000)
    other = plan.transitions(20_000, SEED + 1, mode=qt.PATHWISE).cpu().numpy()
    out = plan.new_counts()
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=s):
        plan.transitions(20_000, SEED, mode=qt.PATHWISE, counts=out, stream=s)
    for _ in range(3):
        out.zero_()
        eager = plan.transitions(20_000, SEED + 1, mode=qt.PATHWISE)
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out[:plan.entries].cpu().numpy(), ref)
        assert np.array_equal(eager.cpu().numpy(), other)


def _plan_in(plan, size):
    """The same model and grids in a workspace of `size` bytes."""
    import ctypes
    model = qt._Model(plan.d, plan.n, *(plan._keep[k].ctypes.data
                                        for k in ("A", "b", "T", "mu", "L", "x0")))
    other = qt.Plan.__new__(qt.Plan)
    other.__dict__.update({k: v for k, v in plan.__dict__.items() if k != "_h"})
    other.workspace = torch.empty(size, dtype=torch.uint8, device="cuda")
    h = ctypes.c_void_p()
    qt._check(qt.lib().qtree_plan_create(ctypes.byref(model), qt._np_ptr(plan.grid),
                                         qt._np_ptr(plan.N), other.workspace.data_ptr(), size,
                                         ctypes.byref(h)))
    other._h = h
    other.batch_samples = int(qt.lib().qtree_plan_batch_samples(h))
    return other


def _best_ms(call, runs=7):
    times = []
    for _ in range(runs):
        e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        e0.record()
        call()
        e1.record()
        torch.cuda.synchronize()
        times.append(e0.elapsed_time(e1))
    return min(times)


def test_layerwise_calls_use_the_room_of_the_cells():
    """A workspace with one chunk per layer behind the path cells: a layerwise
    call that fits the room of both takes one pass, not 25 (whose counts are
    read and written once more each)."""
    _case("layerwise in the cells' room")
    spec = synth.bm_model(1, 50)
    grid, N = synth.layer_grids(spec, [1] + [100] * 50)
    M = 100_000
    own, small = (qt.Plan(spec, grid, N, batch_samples=b) for b in (M, 1))
    assert small.batch_samples < 5000
    counts = [own.new_counts() for _ in range(2)]
    t_own, t_small = (_best_ms(lambda p=p, c=c: p.transitions(M, SEED, counts=c))
                      for p, c in zip((own, small), counts))
    assert torch.equal(counts[0], counts[1])
    assert t_small < 3.0 * t_own, (t_small, t_own)


@pytest.mark.parametrize("d,sizes", [(1, [1, 20, 150, 130, 7, 40, 33]),
                                     (2, [1, (9, 9), (10, 11), (5, 5)]),
                                     (3, [1, (3, 4, 5), (5, 5, 5), (2, 3, 4)])], ids=str)
def test_both_modes_share_a_workspace_of_any_size(d, sizes):
    """From the smallest workspace to the full one, both modes on two streams at
    once and in passes of both views, bit for bit."""
    _case(f"both modes in one workspace {d}-D")
    spec = synth.bm_model(d, len(sizes) - 1, rho=0.2 if d > 1 else 0.0)
    grid, N = synth.layer_grids(spec, sizes)
    full = qt.Plan(spec, grid, N, batch_samples=1)
    M, m0 = 301_111, 1
    refs = [O.transitions(_model(spec), grid, N, M, seed=SEED, m0=m0, mode=mode, nthreads=8)
            for mode in (0, 1)]
    top = full.workspace.numel()
    fits = 0
    for size in sorted({int(top * f) // 16 * 16 for f in
                        (0.02, 0.05, 0.1, 0.2, 0.4, 0.6, 0.8, 0.95, 0.99, 1.0, 1.5)}):
        try:
            plan = _plan_in(full, size)
        except qt.QtreeError as err:
            assert err.status == 2 and not fits       # below the layer tables
            continue
        fits += 1
        streams = [torch.cuda.Stream() for _ in range(2)]
        outs = [[plan.new_counts() for _ in range(3)] for _ in range(2)]
        torch.cuda.synchronize()
        for c in range(3):
            for mode in (0, 1):
                plan.transitions(M, SEED, mode=mode, m0=m0, counts=outs[mode][c],
                                 stream=streams[mode])
        torch.cuda.synchronize()
        for mode in (0, 1):
            for c in range(3):
                assert np.array_equal(outs[mode][c][:plan.entries].cpu().numpy(),
                                      refs[mode]), (size, mode, c)
    assert fits >= 5


def test_captured_layerwise_call_beside_paths():
    """A captured layerwise call keeps to its own scratch, so that its replays
    may run beside pathwise calls of another stream."""
    _case("captured layerwise call beside paths")
    spec, grid, N = _tree()
    plan = qt.Plan(spec, grid, N, batch_samples=1)
    M = 30_000
    layer = O.transitions(_model(spec), grid, N, M, seed=SEED, mode=0, nthreads=8)
    path = _ref(spec, grid, N, 100_000)
    assert plan.batch_samples < M
    assert np.array_equal(plan.transitions(M, SEED).cpu().numpy(), layer)
    out, s, other = plan.new_counts(), torch.cuda.Stream(), torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=s):
        plan.transitions(M, SEED, counts=out, stream=s)
    for _ in range(3):
        out.zero_()
        torch.cuda.synchronize()
        eager = [plan.new_counts() for _ in range(3)]
        for c in eager:
            plan.transitions(100_000, SEED, mode=qt.PATHWISE, counts=c, stream=other)
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out[:plan.entries].cpu().numpy(), layer)
        for c in eager:
            assert np.array_equal(c[:plan.entries].cpu().numpy(), path)


def _without_cells(plan):
    """The same model in a workspace of its tables (within 2 %), which holds no
    path cells: every call counts on the spot."""
    size = 4096
    while True:
        try:
            return _plan_in(plan, size)
        except qt.QtreeError as err:
            assert err.status == 2
            size = int(1.02 * size) // 16 * 16


def test_few_paths_added_to_a_large_tree():
    """Adding a few paths does not read and write every count (their time is that
    of counting on the spot), and counts the same on either side of the line
    12 M n < entries."""
    _case("few paths added")
    spec = synth.bm_model(1, 6)
    grid, N = synth.layer_grids(spec, [1] + [90] * 6)
    plan = qt.Plan(spec, grid, N, batch_samples=1)
    line = plan.entries // (12 * 6)
    counts = plan.transitions(5000, SEED, mode=qt.PATHWISE)
    m0 = 5000
    for M in (1, line, line + 1, 20_000):
        plan.transitions_add(counts, M, SEED, mode=qt.PATHWISE, m0=m0)
        m0 += M
    assert np.array_equal(counts.cpu().numpy(), _ref(spec, grid, N, m0))
    spec = synth.bm_model(1, 100)
    grid, N = synth.layer_grids(spec, [1] + [1000] * 100)
    plan = qt.Plan(spec, grid, N, batch_samples=1)
    counts = plan.transitions(1000, SEED, mode=qt.PATHWISE)
    own, spot = (_best_ms(lambda p=p: p.transitions_add(counts, 100, SEED, mode=qt.PATHWISE))
                 for p in (plan, _without_cells(plan)))
    assert own < 1.5 * spot, (own, spot)


@pytest.mark.parametrize("d,N1", [(2, 1024), (3, 1000)])
def test_scanned_walks_of_many_paths(d, N1):
    """Without tables the walk scans its layers: more paths than a pass of the
    cells take what counting on the spot takes, and count the same."""
    _case(f"scanned walks {d}-D {N1}")
    spec = synth.bm_model(d, 10, rho=0.3)
    grid, N = synth.layer_grids(spec, [1] + [N1] * 10)
    plan = qt.Plan(spec, grid, N, batch_samples=1)
    M = 300_001
    want = plan.transitions(M, SEED, mode=qt.PATHWISE).clone()
    plan.tune(buckets=0)
    other = _without_cells(plan).tune(buckets=0)
    counts = plan.new_counts()
    own, spot = (_best_ms(lambda p=p: p.transitions(M, SEED, mode=qt.PATHWISE, counts=counts))
                 for p in (plan, other))
    plan.transitions(M, SEED, mode=qt.PATHWISE, counts=counts)
    assert torch.equal(counts[:plan.entries], want)
    assert own < 1.25 * spot, (own, spot)


@pytest.mark.parametrize("d,n,N1,M", [(1, 20, 1400, 300_001), (1, 20, 1200, 120_001),
                                      (2, 10, 1369, 300_001)])
def test_paths_through_large_count_blocks(d, n, N1, M):
    """Where a count block has so many super tiles that reading the cells once in
    each costs more than the atomics, the paths are counted on the spot."""
    _case(f"large count blocks {d}-D {N1} {M}")
    spec = synth.bm_model(d, n, rho=0.3 if d > 1 else 0.0)
    grid, N = synth.layer_grids(spec, [1] + [N1] * n)
    plan = qt.Plan(spec, grid, N, batch_samples=1)
    counts = [plan.new_counts() for _ in range(2)]
    own, spot = (_best_ms(lambda p=p, c=c: p.transitions(M, SEED, mode=qt.PATHWISE, counts=c))
                 for p, c in zip((plan, _without_cells(plan)), counts))
    assert torch.equal(counts[0], counts[1])
    assert own < 1.2 * spot, (own, spot)


@pytest.mark.parametrize("d,sizes", [(1, [1, 9]), (1, [1, 4, 5, 3, 7]), (2, [1, 12]), (2, [1, 12, 6]),
                                     (3, [1, 30, 12])], ids=str)
@pytest.mark.parametrize("steps", [1, 512, 513, 2000])
def test_few_steps_added(d, sizes, steps):
    """Few steps added in few layers (d > 1: in one) are counted on the spot,
    more through the cells; both onto counts that are there."""
    _case(f"paths added {d} {sizes} {steps}")
    n = len(sizes) - 1
    spec = synth.bm_model(d, n)
    grid, N = synth.layer_grids(spec, sizes)
    plan = qt.Plan(spec, grid, N, batch_samples=1)
    M = -(-steps // n)
    counts = plan.transitions(1000, SEED, mode=qt.PATHWISE)
    plan.transitions_add(counts, M, SEED, mode=qt.PATHWISE, m0=1000)
    assert np.array_equal(counts[:plan.entries].cpu().numpy(), _ref(spec, grid, N, 1000 + M))
