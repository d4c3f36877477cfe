"""Calls under the caller's own graph captures: what is refused leaves the context and the capture
as they were; what is captured replays with its own inputs and results whatever the context did
in between."""
import numpy as np
import pytest
import torch

import paper_1511_01157_amd as M
from tests.helpers import note

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def test_refused_finite_source_call_leaves_no_trace():
    """The critical curve kept in a context is that of the last call that ran, not of a captured
    call that was refused; the capture that refused it goes on."""
    s = torch.cuda.Stream(device=DEV)
    z = torch.from_numpy(np.random.default_rng(0).normal(0, 0.05, (200, 2))).to(DEV)
    x = torch.zeros(8, device=DEV)
    lens_a, lens_b = (1.0, 0.1), (0.7, 0.4)
    note("graphs: refused finite-source call")
    with torch.cuda.stream(s):
        c, fresh = M.Context.bound(s), M.Context.bound(s)
        want = M.fs_magnification(*lens_b, z, 0.01, ctx=fresh)[0].clone()
        M.fs_magnification(*lens_a, z, 0.01, ctx=c)
        s.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            x += 1
            with pytest.raises(M.MorseError):
                M.fs_magnification(*lens_b, z, 0.01, ctx=c)
        got = M.fs_magnification(*lens_b, z, 0.01, ctx=c)[0]
        assert torch.equal(got, want)
        for rep in range(3):
            g.replay()
            s.synchronize()
            assert torch.equal(x, torch.full_like(x, rep + 1.0))


def chain(seed, npix, n_events, npts, n_u0):
    """A map, a search of it, candidates from the top-k and their gradients, on one context."""
    rng = np.random.default_rng(seed)
    win = (0.0, 0.0, 2.0, 2.0, npix, npix)
    evs = [dict(tt=np.sort(rng.uniform(-30, 30, npts)).astype(np.float32), F=2 + rng.standard_normal(npts),
                w=rng.uniform(50, 150, npts), t_ref=0.1 * e) for e in range(n_events)]
    lcs = M.LightCurveBatch.from_events(evs, DEV)
    grid = M.grid_trajectories(np.linspace(0, 0.8, n_u0), [0.3, 2.0], [0.5], [15.0, 30.0])
    out = torch.empty((npix, npix), dtype=torch.float32, device=DEV)

    def calls(ctx):
        M.build_map(1.0, 0.1, (0.0, 0.0, 4.0, 4.0, 4 * npix, 4 * npix), win, 3.0 * 2.0 / npix, out=out, ctx=ctx)
        r = M.search([(out, win)], lcs, grid, "batched", best=True, top_k=9, ctx=ctx)
        p, e, m = M.candidates_from_topk(grid, r["topk_idx"], 1, ctx=ctx)
        return [out, r["chi2"], r["best_idx"], r["topk_idx"], p, *M.chi2_grad([(out, win)], lcs, p, e, m, ctx=ctx)]

    return calls


def test_graph_replays_after_the_context_has_grown():
    s = torch.cuda.Stream(device=DEV)
    small, large = chain(1, 64, 2, 80, 20), chain(2, 640, 300, 400, 9000)
    note("graphs: replay after growth")
    with torch.cuda.stream(s):
        c = M.Context.bound(s)
        want = [x.clone() for x in small(c)]
        s.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            got = small(c)
        wide = [x.clone() for x in large(c)]  # every buffer of the context grows
        # what a freed buffer would be handed out as
        other = [torch.full((n,), 7, dtype=torch.int32, device=DEV) for n in (1 << 8, 1 << 12, 1 << 14, 1 << 18, 1 << 19, 1 << 20) for _ in range(4)]
        for rep in range(3):
            for x in got:
                x.zero_()
            g.replay()
            s.synchronize()
            for a, b in zip(got, want):
                assert torch.equal(a, b), rep
            assert all(bool((x == 7).all()) for x in other)
            for a, b in zip(large(c), wide):
                assert torch.equal(a, b), rep


def test_capture_that_would_allocate_is_refused():
    s = torch.cuda.Stream(device=DEV)
    small, large = chain(1, 64, 2, 80, 20), chain(2, 640, 300, 400, 9000)
    x = torch.zeros(8, device=DEV)
    note("graphs: refused growth")
    with torch.cuda.stream(s):
        c, fresh = M.Context.bound(s), M.Context.bound(s)
        want = [t.clone() for t in large(fresh)]
        small(c)
        s.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            x += 1
            with pytest.raises(M.MorseError, match="capture"):
                large(c)
        g.replay()
        for a, b in zip(large(c), want):
            assert torch.equal(a, b)
        assert torch.equal(x, torch.ones_like(x))


# direct radii alone, FFT radii alone, both
@pytest.mark.parametrize("rhos,others", [((0.02, 0.05), (0.06,)), ((0.2,), (0.3, 0.25)), ((0.05, 0.3, 0.4), (0.03, 0.35, 0.2))])
def test_captured_stack_keeps_its_profiles(rhos, others):
    """A captured stack replays with its own radii after eager calls with other ones, on the same
    map and on a larger one."""
    s = torch.cuda.Stream(device=DEV)
    rng = np.random.default_rng(5)
    counts = torch.from_numpy(rng.integers(0, 4000, (100, 128)).astype(np.int32)).to(DEV)
    wide = torch.from_numpy(rng.integers(0, 4000, (300, 200)).astype(np.int32)).to(DEV)
    rays, win, win2 = (0, 0, 4, 4, 512, 512), (0.0, 0.0, 2.0, 2.0, 128, 100), (0.0, 0.0, 2.0, 2.0, 200, 300)
    out = torch.empty((len(rhos), 100, 128), dtype=torch.float32, device=DEV)
    note(f"graphs: stack {rhos}")
    with torch.cuda.stream(s):
        c, fresh = M.Context.bound(s), M.Context.bound(s)
        want = M.convolve_stack(counts, rays, win, rhos, out=out, ctx=c).clone()
        want_other = M.convolve_stack(counts, rays, win, others, ctx=fresh).clone()
        s.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            M.convolve_stack(counts, rays, win, rhos, out=out, ctx=c)
            with pytest.raises(M.MorseError, match="capture"):
                M.convolve_stack(counts, rays, win, others, ctx=c)
        for rep in range(3):
            assert torch.equal(M.convolve_stack(counts, rays, win, others, ctx=c), want_other)
            M.convolve_stack(wide, rays, win2, others, ctx=c)
            out.zero_()
            g.replay()
            s.synchronize()
            assert torch.equal(out, want), rep
            assert torch.equal(M.convolve_stack(counts, rays, win, rhos, ctx=c), want), rep


def test_ordinary_calls_after_a_capture_do_not_wait():
    """What an ordinary call put stays for the next one, also when captured calls put theirs: with
    work ahead of it on the stream, a repeated call returns before that work is done."""
    s = torch.cuda.Stream(device=DEV)
    rng = np.random.default_rng(9)
    win = (0.0, 0.0, 2.0, 2.0, 64, 64)
    amap = torch.from_numpy((1 + rng.random((64, 64))).astype(np.float32)).to(DEV)
    n = 2000  # events, and values of an axis: more metadata than goes by value
    lcs = M.LightCurveBatch(torch.from_numpy(np.tile(np.arange(4, dtype=np.float32), n)).to(DEV),
                            torch.from_numpy(rng.random(4 * n)).to(DEV), torch.ones(4 * n, dtype=torch.float64, device=DEV),
                            np.arange(0, 4 * n + 1, 4), np.zeros(n))
    one = M.LightCurveBatch(lcs.t[:8], lcs.flux[:8], lcs.weight[:8], np.array([0, 8]), np.zeros(1))
    grid = M.grid_trajectories(np.linspace(0, 0.8, n), [0.3], [0.5], [15.0])
    P = torch.from_numpy(np.tile(np.array([[0.1, 0.2, 20.0, 0.4]]), (8, 1))).to(DEV)
    z = torch.zeros(8, dtype=torch.int32, device=DEV)
    out = torch.empty((64, 64), dtype=torch.float32, device=DEV)
    big = torch.randn(8192, 8192, device=DEV)
    tmp = torch.empty_like(big)
    note("graphs: ordinary calls after a capture")
    with torch.cuda.stream(s):
        c = M.Context.bound(s)

        def calls():
            M.build_map(1.0, 0.1, (0.0, 0.0, 4.0, 4.0, 256, 256), win, 0.1, out=out, ctx=c)
            r = M.search([(amap, win)], one, grid, "batched", best=True, ctx=c)
            return [out, r["chi2"], r["best_idx"], *M.chi2_grad([(amap, win)], lcs, P, z, z, ctx=c)]

        want = [x.clone() for x in calls()]
        s.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            got = calls()
        calls()
        g.replay()
        s.synchronize()
        behind = torch.cuda.Event()
        for _ in range(20):
            torch.mm(big, big, out=tmp)
        behind.record(s)
        again = calls()
        assert not behind.query()
        s.synchronize()
        for a, b, w in zip(got, again, want):
            assert torch.equal(a, w) and torch.equal(b, w)


def test_captured_ray_statistics_beside_ordinary_calls():
    """A captured ray shooting replayed on one stream while the context shoots other rays on
    another: each call's statistics are its own."""
    s, r = torch.cuda.Stream(device=DEV), torch.cuda.Stream(device=DEV)
    win = (0.0, 0.0, 2.0, 2.0, 256, 256)
    a, b = (1.0, 0.1, (0.0, 0.0, 4.0, 4.0, 8192, 8192), win), (0.8, 0.3, (0.1, 0.05, 6.0, 5.0, 8000, 7000), win)
    bufs = [(torch.zeros((256, 256), dtype=torch.int32, device=DEV), torch.zeros(3, dtype=torch.int64, device=DEV)) for _ in range(2)]
    note("graphs: ray statistics on two streams")
    with torch.cuda.stream(s):
        c = M.Context.bound(s)
        want = []
        for call, (n, st) in zip((a, b), bufs):
            M.rayshoot(*call, n, stats=st, ctx=c)
            want.append((n.clone(), st.clone()))
        s.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            M.rayshoot(*a, *bufs[0][:1], stats=bufs[0][1], ctx=c)
    big = torch.randn(4096, 4096, device=DEV)
    tmp = torch.empty_like(big)
    for rep in range(10):
        for _, st in bufs:
            st.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(r):  # both streams' calls are queued before either runs
            for _ in range(5):
                torch.mm(big, big, out=tmp)
            s.wait_event(r.record_event())
            for _ in range(4):
                g.replay()
        for _ in range(4):
            M.rayshoot(*b, bufs[1][0], stats=bufs[1][1], ctx=c)
        torch.cuda.synchronize()
        for (n, st), (wn, wst) in zip(bufs, want):
            assert torch.equal(n, wn) and torch.equal(st, 4 * wst), rep
