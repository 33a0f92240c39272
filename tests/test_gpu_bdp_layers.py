"""GPU checks of the backward recursion's kernels (matrix-core tiles of 16
rows and payoffs, the one- and two-payoff path, the batch's steps) at the
sizes where they change form: rows below, at and past a load of four columns,
a tile, a round of loads; the last partial tile of rows; 1, 2, 3, 16 and 17
payoffs.

Tolerance: both sides sum the same products of exact integer counts in FP64
in another order; a row of m terms differs by at most 2 m 2^-53 of its largest
term, and the layers' errors add up: 2 n m 2^-53 <= 1e-11 of the largest value
for the sizes here (n = 4, m <= 2100).
"""
import threading

import numpy as np
import pytest

import oracle as O
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1101_3228_amd as qt  # noqa: E402

SIZES = [[1, 2, 3, 4, 5], [1, 15, 16, 17, 33], [1, 100, 250, 257, 64], [1, 513, 500, 512, 3],
         [1, 1025, 1000, 1024, 7], [1, 300, 2049, 31, 2048], [1, 1, 1, 5, 1]]


def _tree(sizes, M=20_000, seed=3):
    spec = synth.bm_model(1, len(sizes) - 1)
    grid, N = synth.layer_grids(spec, sizes)
    plan = qt.Plan(spec, grid, N)
    return plan, N, plan.transitions(M, seed)


def _close(V, ref):
    fin = np.isfinite(ref)
    assert np.array_equal(V[~fin], ref[~fin], equal_nan=True)
    scale = np.abs(ref[fin]).max()
    assert np.abs(V[fin] - ref[fin]).max() <= 1e-11 * scale


@pytest.mark.parametrize("pays", [1, 2, 3, 16, 17])
@pytest.mark.parametrize("sizes", SIZES, ids=str)
def test_bdp_layers(sizes, pays):
    print(f"[gpu-case] bdp layers {sizes} {pays}", flush=True)
    plan, N, counts = _tree(sizes)
    phi = np.random.default_rng(pays).uniform(0.0, 2.0, (pays, plan.points))
    phi[0, :-int(N[-1])] = -np.inf                      # European
    V0, V = plan.bdp(counts, torch.from_numpy(phi).cuda())
    rV0, rV, _ = O.bdp(counts.cpu().numpy(), N, phi, want_all=True)
    _close(V.cpu().numpy(), rV)
    assert np.allclose(V0, rV0, rtol=1e-11, atol=0)


@pytest.mark.parametrize("pays", [1, 2, 5])
def test_zero_counts_ignore_values_that_are_not_finite(pays):
    """An infinite terminal value reaches the rows with a sample in its cell
    and no others (a zero count times infinity would be NaN)."""
    print(f"[gpu-case] bdp infinite values {pays}", flush=True)
    plan, N, counts = _tree([1, 40, 50, 70], M=3000)
    phi = np.random.default_rng(1).uniform(0.0, 2.0, (pays, plan.points))
    phi[0, -3] = np.inf
    phi[-1, -60] = np.inf
    _, V = plan.bdp(counts, torch.from_numpy(phi).cuda())
    c, off, pt = counts.cpu().numpy(), plan.count_offsets(), plan.point_offsets()
    rV = phi.copy()
    for k in range(len(N) - 2, -1, -1):
        C = c[off[k]:off[k + 1]].reshape(N[k], N[k + 1])
        tot = C.sum(1)
        for q in range(pays):
            nxt = np.broadcast_to(rV[q, pt[k + 1]:pt[k + 2]], C.shape)
            s = np.multiply(C, nxt, out=np.zeros(C.shape), where=C != 0).sum(1)
            cont = np.divide(s, tot, out=np.zeros(len(s)), where=tot > 0)
            rV[q, pt[k]:pt[k + 1]] = np.maximum(phi[q, pt[k]:pt[k + 1]], cont)
    assert np.isinf(rV[:, 1:41]).any() and np.isfinite(rV[:, 1:41]).any()
    _close(V.cpu().numpy(), rV)


@pytest.mark.parametrize("pays", [(2, 1), (2, 5), (17, 2)])
@pytest.mark.parametrize("small", [3, 4])
def test_batch_steps(pays, small):
    print(f"[gpu-case] batch steps {pays} {small}", flush=True)
    items = []
    for i, (p, sizes) in enumerate(zip(pays, ([1, small, 18, 300], [1, 33, 260, 17, 1030]))):
        plan, N, _ = _tree(sizes, M=1000)
        phi = np.random.default_rng(p).uniform(0.0, 2.0, (p, plan.points))
        ph = torch.from_numpy(phi).cuda()
        items.append(dict(plan=plan, M=5000, seed=i, counts=plan.new_counts(), phi=ph,
                          V=torch.empty_like(ph)))
    qt.Batch(items).run()
    for it in items:
        c = it["counts"][:it["plan"].entries].cpu().numpy()
        _close(it["V"].cpu().numpy(), O.bdp(c, it["plan"].N, it["phi"].cpu().numpy(),
                                            want_all=True)[1])


@pytest.mark.parametrize("n_pay,threads", [(1, 1), (17, 1), (2048, 1), (2049, 1), (3, 24)])
def test_v0_on_the_host_is_the_first_value(n_pay, threads):
    """V_0 to the host through a slot of 2048 results, one more than it holds,
    and more callers at a time than there are slots."""
    print(f"[gpu-case] V0 n_pay={n_pay} threads={threads}", flush=True)
    plan, _, counts = _tree([1, 7, 9], M=2000)
    torch.cuda.synchronize()
    out = [None] * threads

    def call(t):
        rng = np.random.default_rng(100 + t)
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            phi = torch.from_numpy(rng.random((n_pay, plan.points))).cuda()
            got = []
            for _ in range(5):
                V0, V = plan.bdp(counts, phi, stream=stream)
                got.append((V0, V[:, 0].cpu().numpy()))
            out[t] = got

    ts = [threading.Thread(target=call, args=(t,)) for t in range(threads)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for got in out:
        for V0, first in got:
            assert V0.shape == (n_pay,) and np.array_equal(V0, first)


def test_a_blocking_call_under_capture_is_refused_and_nothing_else():
    """V_0 on the host cannot be waited for under capture: the call returns an
    error, the capture goes on, and later calls (more refused ones before them
    than there are slots) still get their results."""
    print("[gpu-case] V0 under capture", flush=True)
    plan, _, counts = _tree([1, 7, 9], M=2000)
    phi = torch.from_numpy(np.random.default_rng(3).random((12, plan.points))).cuda()
    V, V1 = torch.empty_like(phi), torch.empty_like(phi)
    batch = qt.Batch([dict(plan=plan, M=2000, seed=1, counts=plan.new_counts(), phi=phi, V=V1)])
    want, _ = plan.bdp(counts, phi, V=V)
    stream, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=stream):
        for _ in range(20):
            with pytest.raises(qt.QtreeError) as err:
                plan.bdp(counts, phi, V=V, stream=stream)
            assert err.value.status == 4
            with pytest.raises(qt.QtreeError) as err:
                batch.run(stream=stream)
            assert err.value.status == 4
    for _ in range(3):
        V.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(V[:, 0].cpu().numpy(), want)
    for _ in range(20):
        assert np.array_equal(plan.bdp(counts, phi, V=V)[0], want)
        assert np.array_equal(batch.run(), V1[:, 0].cpu().numpy())


@pytest.mark.parametrize("pays", [1, 2, 3, 17])
@pytest.mark.parametrize("noise", [1.0, 0.05, 0.002])
@pytest.mark.parametrize("sizes", SIZES, ids=str)
def test_banded_layers(sizes, noise, pays):
    """Bands from all columns down to one or two (rows of fewer than four
    entries, four at a time, several turns of a wave; bands that begin and end
    anywhere), with an infinite terminal value that only some bands hold."""
    print(f"[gpu-case] banded layers {sizes} {noise} {pays}", flush=True)
    spec = synth.bm_model(1, len(sizes) - 1)
    spec["T"] *= np.float32(noise)
    grid, N = synth.layer_grids(spec, sizes)
    plan = qt.Plan(spec, grid, N)
    counts = plan.transitions_stratified(300, 11)
    band, overflow = plan.transitions_stratified_banded(300, 11)
    assert int(overflow.item()) == 0
    phi = np.random.default_rng(pays).uniform(0.0, 2.0, (pays, plan.points))
    phi[0, :-int(N[-1])] = -np.inf                      # European
    if N[-1] > 2:
        phi[-1, -2] = np.inf
    ph = torch.from_numpy(phi).cuda()
    V0, V = plan.bdp_banded(band, ph)
    _, dense = plan.bdp(counts, ph)
    _close(V.cpu().numpy(), dense.cpu().numpy())
    assert np.array_equal(V0, V[:, 0].cpu().numpy())
    phi[-1, -2] = 1.0
    _, V = plan.bdp_banded(band, torch.from_numpy(phi).cuda())
    _close(V.cpu().numpy(), O.bdp(counts.cpu().numpy(), N, phi, want_all=True)[1])
