"""Bit-exact parity with the CPU oracle where a kernel changes its form: the edges of the blocks a
vote or lookup works in, and both sides of each rule that picks a variant.  Every output is an
integer, so the bar is equality."""
import numpy as np
import pytest

from paper_2607_04067_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_04067_amd import hough
    hough.load()
    return hough


def _t(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _events(sizes, seed, r_lo=150.0, invalid=0.0):
    """CSR events of the given sizes: random hits, a third of them on a few circles through the
    origin so that there are peaks, and a share `invalid` of hits no kernel may vote."""
    rng = np.random.default_rng(seed)
    xs, ys = [], []
    for n in sizes:
        x, y = synth.random_hits(n, seed + n, r_lo=r_lo)
        m = n // 3
        if m:
            cx, cy = synth.circle_points(rng.uniform(0, 2 * np.pi), 600.0, rng.uniform(max(r_lo, 1.0), 900.0, m))
            x[:m], y[:m] = cx.astype(np.float32), cy.astype(np.float32)
        bad = rng.random(n) < invalid
        x[bad] = rng.choice(np.array([0.0, np.nan, np.inf, 3e38], np.float32), int(bad.sum()))
        y[bad & (x == 0.0)] = 0.0
        p = rng.permutation(n)
        xs.append(x[p]); ys.append(y[p])
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    return np.concatenate(xs), np.concatenate(ys), off


def _check(H, orc, ctx, g, T, W, cap, x, y, off, periodic=False, frac=None, call=None):
    import torch
    xt, yt, ot = _t(x), _t(y), _t(off.astype(np.int32))
    pk, npk, keep, st = call(xt, yt, ot) if call else ctx.run_batch(xt, yt, ot, frac=frac)
    torch.cuda.synchronize()
    ref, n_ref, keep_ref = orc.run_batch(g, x, y, off, threshold=T, rho_window=W, cap=cap, n_threads=8,
                                         periodic=periodic, frac=frac)
    E = off.size - 1
    assert np.array_equal(npk.cpu().numpy()[:E].astype(np.int64), n_ref)
    assert np.array_equal(keep.cpu().numpy()[:x.size], keep_ref)
    p = pk.cpu().numpy()
    for e in range(E):
        m = int(min(n_ref[e], cap))
        assert np.array_equal(H.decode_peaks(p[e], m), ref[e, :m].astype(np.int64)), e
    return st.cpu().numpy()[:E], n_ref


# rho ranges: every vote in range; a few hits of a chunk outside (voted one at a time); most
# outside (clamped chunks); rho = 0 outside the grid (no hit is provably in range); B = -0
VOTE_GRIDS = [(125, 96, -0.02, 0.02, 150.0), (125, 96, -1 / 160, 1 / 160, 150.0), (125, 96, -0.0015, 0.0015, 150.0),
              (70, 64, 0.001, 0.006, 150.0), (70, 64, 0.0, 0.007, 150.0), (33, 128, -0.02, 0.02, 30.0)]


@pytest.mark.parametrize("grid", VOTE_GRIDS)
@pytest.mark.parametrize("invalid", [0.0, 0.05])
def test_matrix_vote_edges(H, orc, grid, invalid):
    """The vote's blocks of 8, 32 and 64 hits per wave, at event sizes around their edges, with
    every mix of hits that vote in the matrix form, one at a time, clamped, or not at all."""
    n_theta, n_rho, lo, hi, r_lo = grid
    sizes = [1, 2, 7, 8, 9, 31, 33, 63, 64, 65, 71, 127, 129, 500, 511, 512, 513, 520, 1025, 2600]
    x, y, off = _events(sizes, 17, r_lo, invalid)
    g = orc.Grid(n_theta, n_rho, lo, hi)
    for T in (1, 4):
        ctx = H.Context(n_theta, n_rho, lo, hi, "i32", T, 1, 4096)
        st, _ = _check(H, orc, ctx, g, T, 1, 4096, x, y, off)
        ctx.close()
        for e in (0, 8, 19):                                  # the per-event vote uses the same loop
            a, b = int(off[e]), int(off[e + 1])
            with_acc = H.Context(n_theta, n_rho, lo, hi, "i32", T, 1, 16)
            acc = with_acc.vote(_t(x[a:b]), _t(y[a:b])).cpu().numpy()
            with_acc.close()
            assert np.array_equal(acc, orc.vote(g, x[a:b], y[a:b])), e
    if lo == -hi:
        ctx = H.Context(n_theta, n_rho, lo, hi, "i32", 3, 1, 4096, periodic=True)
        _check(H, orc, ctx, g, 3, 1, 4096, x, y, off, periodic=True)
        _check(H, orc, ctx, g, 3, 1, 4096, x, y, off, periodic=True, frac=(1, 2))
        ctx.close()


@pytest.mark.parametrize("T,W", [(3, 1), (4, 0), (6, 1), (9, 2), (14, 1), (6, 40)])
@pytest.mark.parametrize("groups", [1, 2])
def test_retention_by_columns(H, orc, T, W, groups):
    """Tiles with many peaks test a hit in rounds of a few columns before the rest, tiles with few
    do not, and hits outside the grid in some column take the literal test: thresholds and windows
    on both sides of the rule, events that leave none, a few and many hits unkept."""
    n_theta, n_rho, lo, hi = 200, 128, -1 / 170, 1 / 170
    x, y, off = _events([90, 700, 1500, 2600, 5000], 5, 160.0, 0.01)
    g = orc.Grid(n_theta, n_rho, lo, hi)
    ctx = H.Context(n_theta, n_rho, lo, hi, "i32", T, W, 8192)
    ctx.set_batch_plan(8, groups)
    _check(H, orc, ctx, g, T, W, 8192, x, y, off)
    ctx.close()



# grids whose columns hold whole quads of rows and not, 32-column groups with remainders, one slab
# and several; a 16-bit accumulator; an accumulator that is not 16-byte aligned
@pytest.mark.parametrize("n_theta,n_rho,acc_type,shift", [(1, 3, "i32", 0), (33, 100, "i32", 0), (64, 97, "i32", 0),
                                                          (65, 96, "u16", 0), (95, 50, "u16", 0), (40, 64, "i32", 1),
                                                          (40, 64, "u16", 1), (31, 1400, "i32", 0),
                                                          (31, 1401, "u16", 0), (20, 8192, "i32", 0)])
def test_event_vote_tiles(H, orc, n_theta, n_rho, acc_type, shift):
    import torch
    for lo, hi in ((-0.008, 0.008), (-0.0015, 0.002)):
        g = orc.Grid(n_theta, n_rho, lo, hi)
        ctx = H.Context(n_theta, n_rho, lo, hi, acc_type, 3, 1, 64)
        for n in (0, 1, 65, 1500):
            x, y, _ = _events([n], 3 + n, 160.0, 0.03) if n else (np.zeros(0, np.float32),) * 2 + (None,)
            dt = torch.int16 if acc_type == "u16" else torch.int32
            buf = torch.full((n_theta * n_rho + 8,), 7, dtype=dt, device="cuda")
            acc = buf[shift:shift + n_theta * n_rho].view(n_theta, n_rho)
            ctx.vote(_t(x), _t(y), acc)
            got = acc.cpu().numpy()
            got = got.view(np.uint16).astype(np.int32) if acc_type == "u16" else got
            assert np.array_equal(got, orc.vote(g, x, y)), (lo, n)
            assert int(buf[shift + n_theta * n_rho].item()) == 7           # nothing past the last cell
        ctx.close()


@pytest.mark.parametrize("n_theta,n_rho,W", [(70, 40, 1), (300, 300, 1), (300, 300, 40), (700, 1000, 2), (37, 2000, 1)])
@pytest.mark.parametrize("n_hits", [1, 63, 64, 65, 1500])
def test_event_retain_forms(H, orc, n_theta, n_rho, W, n_hits):
    """hough_retain against a peak list (up to 1,024 peaks) and against dilated bits (more, in one
    and several blocks of columns), with peaks on the rho edges and cells outside the grid."""
    lo, hi = -1 / 170, 1 / 170
    g = orc.Grid(n_theta, n_rho, lo, hi)
    x, y, _ = _events([n_hits], 9, 160.0, 0.02)
    ctx = H.Context(n_theta, n_rho, lo, hi, "i32", 3, W, 64)
    rng = np.random.default_rng(n_hits)
    for n in (0, 1, 17, 1022, 1023, 6000):
        n = min(n, n_theta * n_rho)
        cell = rng.choice(n_theta * n_rho, n, replace=False)
        pj, pk = cell // n_rho, cell % n_rho
        pk[: n // 5] = rng.choice([0, n_rho - 1], n // 5)           # some on the rho edges
        rec = np.zeros((n + 2, 2), np.uint32)
        rec[:n, 0] = pj | (pk << 16)
        rec[n:, 0] = n_theta, n_rho << 16                          # two cells outside the grid
        keep = ctx.retain(_t(x), _t(y), _t(rec.view(np.int32)), _t(np.array([n + 2], np.int32)), n + 2)
        assert np.array_equal(keep.cpu().numpy(), orc.retain(g, x, y, pj, pk, W)), n
    ctx.close()


@pytest.mark.parametrize("n_theta,n_rho", [(1, 1), (2, 5), (37, 129), (129, 300), (500, 700)])
@pytest.mark.parametrize("frac", [(0, 1), (1, 2), (1, 1)])
def test_event_finder_listed_candidates(H, orc, n_theta, n_rho, frac):
    """The iterative finder on candidates listed by the whole chip: none, a few, one per thread, more
    than one key buffer and more than the list, on accumulators of equal and of random counts."""
    rng = np.random.default_rng(n_theta)
    ctx = H.Context(n_theta, n_rho, -0.005, 0.005, "i32", 4, 1, 64)
    cap = 600
    for kind in range(5):
        acc = np.zeros((n_theta, n_rho), np.int32)
        if kind == 1:
            acc[:] = 5                                             # one flat plateau
        elif kind == 2:
            acc[:] = rng.integers(0, 5, acc.shape)
            acc.flat[rng.integers(0, acc.size, 9)] = 40
        elif kind == 3:
            acc[:] = rng.integers(0, 60, acc.shape)
        elif kind == 4:
            acc[:] = rng.integers(3, 9, acc.shape)
            acc.flat[-1] = 9
        pk, n, st = ctx.peaks_iterative(_t(acc), cap, frac, 3, 4)
        pj, pkk, pc, m = orc.peaks_iterative(acc, 4, frac, 3, 4, cap=cap, sorted_form=True)
        assert int(n.item()) == m, kind
        k = min(m, cap)
        assert np.array_equal(H.decode_peaks(pk, k), np.stack([pj[:k], pkk[:k], pc[:k]], 1).astype(np.int64)), kind
        assert int(st.item()) == (H.EV_PEAKS_TRUNCATED if m > cap else 0)
    ctx.close()


@pytest.mark.parametrize("n_theta,n_rho", [(2, 4096), (64, 128), (3, 2731), (90, 100)])
@pytest.mark.parametrize("acc_type", ["i32", "u16"])
def test_event_finder_on_either_side_of_the_list(H, orc, n_theta, n_rho, acc_type):
    """The iterative finder on accumulators it reads by itself and on ones listed for it, one context after the
    other use, from no candidate to more than its key buffer holds."""
    rng = np.random.default_rng(n_rho)
    ctx = H.Context(n_theta, n_rho, -0.005, 0.005, acc_type, 4, 1, 64)
    cap = 400
    for top, frac in ((4, (1, 2)), (200, (9, 10)), (60, (1, 2)), (60, (0, 1)), (5, (1, 1))):
        acc = rng.integers(0, top, (n_theta, n_rho)).astype(np.int32 if acc_type == "i32" else np.int16)
        acc.flat[-1] = top - 1
        pk, n, st = ctx.peaks_iterative(_t(acc), cap, frac, 3, 4)
        pj, pkk, pc, m = orc.peaks_iterative(acc.astype(np.int32), 4, frac, 3, 4, cap=cap, sorted_form=True)
        k = min(m, cap)
        assert int(n.item()) == m, (top, frac)
        assert np.array_equal(H.decode_peaks(pk, k), np.stack([pj[:k], pkk[:k], pc[:k]], 1).astype(np.int64)), (top, frac)
        assert int(st.item()) == (H.EV_PEAKS_TRUNCATED if m > cap else 0)
    ctx.close()


@pytest.mark.parametrize("n_theta,n_rho", [(2, 2), (3, 70), (5, 64), (8, 100), (130, 257), (4100, 12)])
def test_event_peaks_blocks(H, orc, n_theta, n_rho):
    """hough_peaks' blocks of 4 (many columns: 16) rows, their edges and the periodic border."""
    rng = np.random.default_rng(n_theta * n_rho)
    for periodic in (False, True):
        ctx = H.Context(n_theta, n_rho, -0.005, 0.005, "i32", 3, 1, 64, periodic=periodic)
        for top in (4, 30):
            acc = rng.integers(0, top, (n_theta, n_rho)).astype(np.int32)
            pk, n = ctx.peaks(_t(acc), n_theta * n_rho)
            pj, pkk, pc, m = orc.peaks(acc, 3, periodic=periodic)
            assert int(n.item()) == m
            assert np.array_equal(H.decode_peaks(pk, m), np.stack([pj, pkk, pc], 1).astype(np.int64))
        ctx.close()


@pytest.mark.parametrize("n_theta,n_rho", [(1, 40), (62, 64), (63, 33), (125, 256), (200, 1000), (4000, 24)])
@pytest.mark.parametrize("flags", ["plain", "periodic", "dedup"])
def test_small_batches_by_tile(H, orc, n_theta, n_rho, flags):
    """Batches of few events run one workgroup per (event, tile): 1 to 65 tiles, one batch on each
    side of the rule's event count, empty and oversized events between ordinary ones, peaks that
    overflow the buffer, the gather form and the latency form, each called twice (the slots and the
    counter are left at zero)."""
    import torch
    periodic, dedup = flags == "periodic" and n_theta > 1, flags == "dedup"
    lo, hi = (-1 / 180, 1 / 180)
    g = orc.Grid(n_theta, n_rho, lo, hi)
    half = torch.cuda.get_device_properties(0).multi_processor_count // 2
    x, y, off = _events([700, 0, 1500, 3, 64, 33000, 900], 23, 170.0, 0.01)
    x[100:200], y[100:200] = x[:100], y[:100]                      # copies in the first event
    T, cap = 4, 700
    ctx = H.Context(n_theta, n_rho, lo, hi, "i32", T, 1, cap, periodic=periodic, dedup=dedup)
    ref, n_ref, keep_ref = orc.run_batch(g, x, y, off, threshold=T, rho_window=1, cap=cap, n_threads=8,
                                         periodic=periodic)
    if dedup:                                                      # the event above the limit votes every hit
        d, nd, kd = orc.run_batch(g, x, y, off, threshold=T, rho_window=1, cap=cap, n_threads=8, dedup=True)
        small = np.diff(off) <= 8192
        ref[small], n_ref[small] = d[small], nd[small]
        for e in np.nonzero(small)[0]:
            keep_ref[off[e]:off[e + 1]] = kd[off[e]:off[e + 1]]
    xt, yt, ot = _t(x), _t(y), _t(off.astype(np.int32))
    E = off.size - 1
    ws = ctx.split_workspace(E)

    def same(out, ids):
        pk, npk, keep, st = out
        torch.cuda.synchronize()
        npk, p = npk.cpu().numpy(), pk.cpu().numpy()
        for i, e in enumerate(ids):
            m = int(min(n_ref[e], cap))
            assert npk[i] == n_ref[e], (i, e)
            assert np.array_equal(H.decode_peaks(p[i], m), ref[e, :m].astype(np.int64)), (i, e)
        return keep.cpu().numpy()

    for _ in range(2):
        assert np.array_equal(same(ctx.run_batch(xt, yt, ot), range(E))[:x.size], keep_ref)
        assert np.array_equal(same(ctx.run_batch_split(xt, yt, ot, ws), range(E))[:x.size], keep_ref)
        assert int(ws.count_nonzero()) == 0
    for n in (1, half, half + 1, 3 * half // 2, 3 * half // 2 + 1):   # by tile, by tile or by event
        ids = (np.arange(n) * 3) % E
        ids = ids[ids != 5] if n > 1 else ids
        ids = np.resize(ids, n)
        sizes = np.diff(off)[ids]
        starts = np.concatenate([[0], np.cumsum(sizes)])
        keep = same(ctx.run_batch_gather(xt, yt, ot, _t(ids.astype(np.int32)), _t(starts[:-1].astype(np.int32)),
                                         keep_size=int(starts[-1])), ids)
        want = np.concatenate([keep_ref[off[e]:off[e + 1]] for e in ids])
        assert np.array_equal(keep[:want.size], want), n
    ctx.close()


@pytest.mark.parametrize("n_theta,n_rho,plan", [(130, 1000, None), (130, 1000, (8, 1, 2)), (64, 700, None),
                                                (130, 1500, None), (70, 2000, None)])
@pytest.mark.parametrize("flags", ["plain", "periodic", "dedup"])
def test_windows_over_many_events(H, orc, n_theta, n_rho, plan, flags):
    """Batches large enough for the fused kernel on grids whose column fills a CU or does not fit it:
    events whose hits reach few rows run on a window of them, those that reach beyond it (here every
    seventh) on whole columns or through the spill path, empty and invalid ones between; absolute and
    relative thresholds, windows on both sides of rho = 0's row, twice in a row, and gathered."""
    import torch
    periodic, dedup = flags == "periodic", flags == "dedup"
    lo, hi = (-0.01, 0.01) if periodic else (-0.012, 0.009)
    if plan and periodic:
        pytest.skip("a window is not the caller's to choose on a periodic grid")
    g = orc.Grid(n_theta, n_rho, lo, hi)
    rng = np.random.default_rng(n_rho)
    sizes = rng.integers(0, 260, 2 * torch.cuda.get_device_properties(0).multi_processor_count + 8)
    sizes[::31] = 0
    parts = [_events([int(n)], 40 + i, 60.0 if i % 7 == 3 else 210.0, 0.01)[:2] for i, n in enumerate(sizes)]
    x, y = (np.concatenate([p[i] for p in parts]) for i in (0, 1))
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    x[off[9]:off[9] + 20], y[off[9]:off[9] + 20] = x[off[9] + 20:off[9] + 40], y[off[9] + 20:off[9] + 40]
    T, cap = 3, 1500
    ctx = H.Context(n_theta, n_rho, lo, hi, "i32", T, 1, cap, periodic=periodic, dedup=dedup)
    if plan:
        ctx.set_batch_plan(*plan)
    xt, yt, ot = _t(x), _t(y), _t(off.astype(np.int32))
    E = off.size - 1
    for frac in (None, (1, 2), None):
        pk, npk, keep, st = ctx.run_batch(xt, yt, ot, frac=frac)
        torch.cuda.synchronize()
        ref, n_ref, keep_ref = orc.run_batch(g, x, y, off, threshold=T, rho_window=1, cap=cap, n_threads=8,
                                             periodic=periodic, dedup=dedup, frac=frac)
        assert np.array_equal(npk.cpu().numpy()[:E].astype(np.int64), n_ref), frac
        assert np.array_equal(keep.cpu().numpy()[:x.size], keep_ref), frac
        p = pk.cpu().numpy()
        for e in range(E):
            m = int(min(n_ref[e], cap))
            assert np.array_equal(H.decode_peaks(p[e], m), ref[e, :m].astype(np.int64)), (frac, e)
    ids = np.arange(E)[::-1].copy()
    starts = np.concatenate([[0], np.cumsum(sizes[ids])])
    gk = ctx.run_batch_gather(xt, yt, ot, _t(ids.astype(np.int32)), _t(starts[:-1].astype(np.int32)),
                              keep_size=int(starts[-1]))
    torch.cuda.synchronize()
    assert np.array_equal(gk[1].cpu().numpy()[:E], npk.cpu().numpy()[:E][ids])
    assert np.array_equal(gk[2].cpu().numpy()[:int(starts[-1])],
                          np.concatenate([keep_ref[off[e]:off[e + 1]] for e in ids]))
    ctx.close()


@pytest.mark.parametrize("n_theta,n_rho", [(248, 700), (249, 700), (251, 1000)])
@pytest.mark.parametrize("flags", ["plain", "periodic", "dedup"])
def test_windows_over_many_events_of_wide_grids(H, orc, n_theta, n_rho, flags):
    """The same on both sides of the width from which such batches run on windows."""
    test_windows_over_many_events(H, orc, n_theta, n_rho, None, flags)


@pytest.mark.parametrize("n_theta,n_rho", [(2, 1500), (62, 1217), (63, 1500), (130, 2000), (1000, 1300)])
@pytest.mark.parametrize("periodic", [False, True])
@pytest.mark.parametrize("W", [1, 40])
def test_small_batches_on_windows(H, orc, n_theta, n_rho, periodic, W):
    """Few events on grids taller than a tile: one workgroup per (event, tile), each on the event's
    window of rows.  Events that fit, events that reach beyond the window (60 mm), empty and
    oversized ones, peaks that overflow the buffer, windows on both sides of rho = 0's row, one batch
    on each side of the rule's event count, and gathered; every form called twice."""
    import torch
    lo, hi = (-0.01, 0.01) if periodic else (-0.012, 0.009)
    g = orc.Grid(n_theta, n_rho, lo, hi)
    half = torch.cuda.get_device_properties(0).multi_processor_count // 2
    sizes = [900, 0, 1300, 3, 64, 33000, 700, 257]
    parts = [_events([n], 60 + i, 60.0 if i in (3, 6) else 215.0, 0.01)[:2] for i, n in enumerate(sizes)]
    x, y = (np.concatenate([p[i] for p in parts]) for i in (0, 1))
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    T, cap = 3, 500
    ctx = H.Context(n_theta, n_rho, lo, hi, "i32", T, W, cap, periodic=periodic)
    for _ in range(2):
        _, n_ref = _check(H, orc, ctx, g, T, W, cap, x, y, off, periodic)
    xt, yt, ot = _t(x), _t(y), _t(off.astype(np.int32))
    keep_ref = ctx.run_batch(xt, yt, ot)[2].cpu().numpy()
    for n in (1, half, half + 1):                                  # by tile, by tile, by event
        ids = np.resize([0, 2, 6, 1, 3, 4, 7], n)
        starts = np.concatenate([[0], np.cumsum(np.array(sizes)[ids])])
        for _ in range(2):
            out = ctx.run_batch_gather(xt, yt, ot, _t(ids.astype(np.int32)), _t(starts[:-1].astype(np.int32)),
                                       keep_size=int(starts[-1]))
            torch.cuda.synchronize()
            assert np.array_equal(out[1].cpu().numpy()[:n], n_ref[ids])
            assert np.array_equal(out[2].cpu().numpy()[:int(starts[-1])],
                                  np.concatenate([keep_ref[off[e]:off[e + 1]] for e in ids]))
    ctx.close()


@pytest.mark.parametrize("n_theta,n_rho,rng_lo,rng_hi", [(1, 1, -0.01, 0.01), (3, 5, -0.01, 0.01), (65, 33, -0.006, 0.006),
                                                         (64, 600, -0.006, 0.006), (127, 601, -0.006, 0.006),
                                                         (129, 1000, -0.01, 0.01), (70, 1301, -0.004, 0.006),
                                                         (1000, 1200, -0.01, 0.01)])
@pytest.mark.parametrize("dedup", [False, True])
def test_batch_finder_tiles(H, orc, n_theta, n_rho, rng_lo, rng_hi, dedup):
    """The iterative finder over a batch with tiles that list their candidates and tiles that write
    every cell (small fractions and floors), one slab of rows and several, keys that start on odd
    accumulator boundaries, an empty event and one too large, twice on one workspace."""
    import torch
    g = orc.Grid(n_theta, n_rho, rng_lo, rng_hi)
    x, y, off = _events([400, 0, 1300, 33000, 90], 31, 120.0, 0.01)
    x[50:90], y[50:90] = x[:40], y[:40]
    cap = 300
    xt, yt, ot = _t(x), _t(y), _t(off.astype(np.int32))
    E = off.size - 1
    for floor, frac in ((2, (1, 2)), (6, (3, 4)), (1, (0, 1))):
        if frac[0] == 0 and n_theta * n_rho > 100000:
            continue                                               # every voted cell is a candidate: minutes in the oracle
        ctx = H.Context(n_theta, n_rho, rng_lo, rng_hi, "i32", floor, 1, cap, dedup=dedup)
        ws = ctx.iterative_workspace(E)
        small = np.diff(off) <= 32767
        keep_ids = np.nonzero(small)[0]
        xs = np.concatenate([x[off[e]:off[e + 1]] for e in keep_ids])
        ys = np.concatenate([y[off[e]:off[e + 1]] for e in keep_ids])
        so = np.concatenate([[0], np.cumsum(np.diff(off)[keep_ids])])
        ref, n_ref, keep_ref = orc.run_batch_iterative_fast(g, xs, ys, so, floor, frac, 2, 3, 1, cap, dedup=dedup,
                                                            n_threads=8)
        for _ in range(2):
            pk, npk, keep, st = ctx.run_batch_iterative(xt, yt, ot, frac, 2, 3, ws)
            torch.cuda.synchronize()
            npk, p, kp, st = npk.cpu().numpy(), pk.cpu().numpy(), keep.cpu().numpy(), st.cpu().numpy()
            for i, e in enumerate(keep_ids):
                m = int(min(n_ref[i], cap))
                assert npk[e] == n_ref[i], (floor, e)
                assert np.array_equal(H.decode_peaks(p[e], m), ref[i, :m].astype(np.int64)), (floor, e)
                assert np.array_equal(kp[off[e]:off[e + 1]], keep_ref[so[i]:so[i + 1]]), (floor, e)
                assert bool(st[e] & H.EV_PEAKS_TRUNCATED) == (n_ref[i] > cap)
            assert npk[3] == 0 and st[3] == H.EV_TOO_MANY_HITS and not kp[off[3]:off[4]].any()
        ctx.close()


@pytest.mark.parametrize("n_theta,n_rho,E", [(60, 1216, 3), (60, 1217, 3), (3, 2500, 2), (130, 1300, 85), (130, 1300, 86)])
def test_batch_finder_slabs(H, orc, n_theta, n_rho, E):
    """The iterative finder over batches whose tiles have a CU each and over ones that do not, on columns at
    the edges of the rows a tile then holds at a time, of events that reach every row and ones that reach few."""
    import torch
    g = orc.Grid(n_theta, n_rho, -0.01, 0.01)
    parts = [_events([60 + 11 * (i % 7)], 70 + i, 110.0 if i % 3 else 400.0, 0.01)[:2] for i in range(E)]
    x, y = (np.concatenate([p[i] for p in parts]) for i in (0, 1))
    off = np.concatenate([[0], np.cumsum([p[0].size for p in parts])])
    floor, cap = 3, 200
    ctx = H.Context(n_theta, n_rho, -0.01, 0.01, "i32", floor, 1, cap)
    for frac in ((1, 2), (1, 8)):
        ref, n_ref, keep_ref = orc.run_batch_iterative_fast(g, x, y, off, floor, frac, 2, 3, 1, cap, n_threads=8)
        pk, npk, keep, st = ctx.run_batch_iterative(_t(x), _t(y), _t(off.astype(np.int32)), frac, 2, 3,
                                                    ctx.iterative_workspace(E))
        torch.cuda.synchronize()
        npk, p = npk.cpu().numpy(), pk.cpu().numpy()
        assert np.array_equal(npk.astype(np.int64), n_ref)
        assert np.array_equal(keep.cpu().numpy()[:x.size], keep_ref)
        for e in range(E):
            m = int(min(n_ref[e], cap))
            assert np.array_equal(H.decode_peaks(p[e], m), ref[e, :m].astype(np.int64)), (frac, e)
    ctx.close()


PLANS = [(w, g, 0) for w in (4, 6, 8, 12, 16) for g in (1, 2)] + [(8, 1, 2), (4, 1, 3)]


@pytest.mark.parametrize("grid", VOTE_GRIDS + [(200, 530, -1 / 170, 1 / 170, 160.0),
                                               (130, 1000, -0.01, 0.01, 210.0)])
@pytest.mark.parametrize("flags", ["plain", "periodic", "dedup"])
def test_every_fused_shape_equals_the_oracle(H, orc, grid, flags):
    """A set shape runs the fused kernel whatever the number of events: every count of waves and column
    groups, whole columns and windows of them, with events at the edges of its blocks of hits, an empty one
    and the largest it takes, narrow and wide retention windows, and rho ranges of every mix of votes in
    and out of the grid."""
    n_theta, n_rho, lo, hi, r_lo = grid
    periodic, dedup = flags == "periodic", flags == "dedup"
    if periodic and lo != -hi:
        pytest.skip("a periodic grid is symmetric")
    sizes = [1, 7, 9, 64, 65, 513, 520, 0, 2600, 8192 if dedup else 32767]
    x, y, off = _events(sizes, 41, r_lo, 0.02)
    a = int(off[8])
    x[a + 300:a + 700], y[a + 300:a + 700] = x[a:a + 400], y[a:a + 400]           # copies
    g = orc.Grid(n_theta, n_rho, lo, hi)
    xt, yt, ot = _t(x), _t(y), _t(off.astype(np.int32))
    for T, W in ((1, 1), (4, 40), (9, 300), (12, 0)):
        cap = 6000
        ref, n_ref, keep_ref = orc.run_batch(g, x, y, off, threshold=T, rho_window=W, cap=cap, n_threads=8,
                                             periodic=periodic, dedup=dedup)
        ctx = H.Context(n_theta, n_rho, lo, hi, "i32", T, W, cap, periodic=periodic, dedup=dedup)
        tried = 0
        for plan in PLANS:
            try:
                ctx.set_batch_plan(*plan)
            except H.HoughError:
                continue
            tried += 1
            pk, npk, keep, st = ctx.run_batch(xt, yt, ot)
            p = pk.cpu().numpy()
            assert np.array_equal(npk.cpu().numpy()[:len(sizes)].astype(np.int64), n_ref), (plan, T, W)
            assert np.array_equal(keep.cpu().numpy()[:x.size], keep_ref), (plan, T, W)
            for e in range(len(sizes)):
                m = int(min(n_ref[e], cap))
                assert np.array_equal(H.decode_peaks(p[e], m), ref[e, :m].astype(np.int64)), (plan, T, W, e)
        assert tried >= (11 if n_rho < 531 else 5)             # (two groups: up to some 550 rows)
        ctx.close()


@pytest.mark.parametrize("flags", ["plain", "periodic", "dedup"])
@pytest.mark.parametrize("frac", [None, (1, 2)])
def test_events_around_the_room_for_mapped_hits(H, orc, flags, frac):
    """A launch of 1,024 workgroups leaves each room for 4,096 mapped hits: in a larger event the first
    waves read theirs back on the later tiles while the others map the hits again.  Events on both sides
    of the room, up to the largest the kernel takes, among many small ones."""
    import torch
    periodic, dedup = flags == "periodic", flags == "dedup"
    n_theta, n_rho, lo, hi = 190, 96, -1 / 180, 1 / 180
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    large = [4095, 4096, 4097, 4103, 4104, 4600, 5000, 7000, 8191, 8192] + ([] if dedup else [8193, 10000, 20000, 32767])
    rng = np.random.default_rng(3)
    sizes = np.concatenate([large * 3, rng.integers(0, 40, 4 * cu + 30 - 3 * len(large))])
    sizes = sizes[rng.permutation(sizes.size)]
    x, y, off = _events([int(n) for n in sizes], 71, 170.0, 0.01)
    for e in np.nonzero(sizes > 4000)[0]:                      # copies, and a run of hits no kernel votes
        a = int(off[e])
        x[a + 3000:a + 3200], y[a + 3000:a + 3200] = x[a:a + 200], y[a:a + 200]
        x[a + 3900:a + 4000] = np.nan
    T, cap = 12, 2000
    ctx = H.Context(n_theta, n_rho, lo, hi, "i32", T, 1, cap, periodic=periodic, dedup=dedup)
    ctx.set_batch_plan(8, 1, 4)
    xt, yt, ot = _t(x), _t(y), _t(off.astype(np.int32))
    ref, n_ref, keep_ref = orc.run_batch(orc.Grid(n_theta, n_rho, lo, hi), x, y, off, threshold=T, rho_window=1, cap=cap,
                                         n_threads=8, periodic=periodic, dedup=dedup, frac=frac)
    for _ in range(2):
        pk, npk, keep, st = ctx.run_batch(xt, yt, ot, frac=frac)
        p = pk.cpu().numpy()
        assert np.array_equal(npk.cpu().numpy()[:sizes.size].astype(np.int64), n_ref)
        assert np.array_equal(keep.cpu().numpy()[:x.size], keep_ref)
        for e in range(sizes.size):
            m = int(min(n_ref[e], cap))
            assert np.array_equal(H.decode_peaks(p[e], m), ref[e, :m].astype(np.int64)), e
    ctx.close()


@pytest.mark.parametrize("dedup", [False, True])
def test_batch_finder_over_several_passes(H, orc, dedup):
    """A grid of 65,535 columns takes 64 events at a time: 130 events are three passes, each on its own
    part of the offsets, the workspace and the outputs, over the same heads."""
    import torch
    n_theta, n_rho, lo, hi = 65535, 3, -1 / 170, 1 / 170
    g = orc.Grid(n_theta, n_rho, lo, hi)
    E = 130
    sizes = [(37 * e) % 90 for e in range(E)]
    x, y, off = _events(sizes, 19, 160.0, 0.02)
    a = int(off[2])
    x[a:a + 30], y[a:a + 30] = x[a + 30:a + 60], y[a + 30:a + 60]
    cap, floor, frac = 16, 20, (9, 10)
    ctx = H.Context(n_theta, n_rho, lo, hi, "i32", floor, 0, cap, dedup=dedup)
    ref, n_ref, keep_ref = orc.run_batch_iterative_fast(g, x, y, off, floor, frac, 4000, 1, 0, cap, dedup=dedup, n_threads=8)
    assert (n_ref[64:] > 0).any() and (n_ref[128:] >= 0).all()
    pk, npk, keep, st = ctx.run_batch_iterative(_t(x), _t(y), _t(off.astype(np.int32)), frac, 4000, 1,
                                                ctx.iterative_workspace(E))
    torch.cuda.synchronize()
    p = pk.cpu().numpy()
    assert np.array_equal(npk.cpu().numpy()[:E].astype(np.int64), n_ref)
    assert np.array_equal(keep.cpu().numpy()[:x.size], keep_ref)
    for e in range(E):
        m = int(min(n_ref[e], cap))
        assert np.array_equal(H.decode_peaks(p[e], m), ref[e, :m].astype(np.int64)), e
    ctx.close()


@pytest.mark.parametrize("n_theta,n_rho,W", [(90, 64, 1), (300, 300, 2), (37, 2000, 1)])
@pytest.mark.parametrize("chunks_per_cu", [1, 2, 4, 8, 20])
def test_event_retain_large(H, orc, n_theta, n_rho, W, chunks_per_cu):
    """hough_retain by the number of waves that share 64 hits (16 down to one, by the hits per CU): events
    on both sides of each line, few peaks (listed) and many, most hits kept and few of them."""
    import torch
    lo, hi = -1 / 170, 1 / 170
    g = orc.Grid(n_theta, n_rho, lo, hi)
    edge = 64 * chunks_per_cu * torch.cuda.get_device_properties(0).multi_processor_count
    x, y, _ = _events([edge + 65], 12, 160.0, 0.01)
    xt, yt = _t(x), _t(y)
    ctx = H.Context(n_theta, n_rho, lo, hi, "i32", 3, W, 64)
    rng = np.random.default_rng(chunks_per_cu)
    for n in (3, 900, 1500, min(20000, n_theta * n_rho // 3)):
        cell = rng.choice(n_theta * n_rho, n, replace=False)
        pj, pk = cell // n_rho, cell % n_rho
        if n == 1500:
            pk[:] = rng.choice([0, 1, n_rho - 1], n)               # few hits near the rho edges
        rec = np.zeros((n, 2), np.uint32)
        rec[:, 0] = pj | (pk << 16)
        recs, npk = _t(rec.view(np.int32)), _t(np.array([n], np.int32))
        ref = orc.retain(g, x, y, pj, pk, W)
        for m in (edge - 64, edge, edge + 1, edge + 65):
            buf = torch.full((m + 1,), 7, dtype=torch.uint8, device="cuda")
            keep = ctx.retain(xt[:m], yt[:m], recs, npk, n, buf[:m])
            assert np.array_equal(keep.cpu().numpy(), ref[:m]), (n, m)
            assert int(buf[m].item()) == 7
    ctx.close()


# blocks of 4, 8 and 16 rows (up to 512, up to 2,048 and more columns; fewer where the rows are long), and
# rows on both sides of what one, two and four loads per thread cover
@pytest.mark.parametrize("n_theta,n_rhos", [(5, (42, 43, 85, 86, 170, 171)), (512, (9,)), (513, (9, 51, 52, 102, 103)),
                                            (521, (204, 205)), (2048, (20,)), (2049, (20, 56, 57, 113, 114)),
                                            (2063, (227, 228)), (600, (3000,)), (2050, (1900,)), (65535, (8,))])
@pytest.mark.parametrize("acc_type", ["i32", "u16"])
def test_event_peaks_staging(H, orc, n_theta, n_rhos, acc_type):
    rng = np.random.default_rng(n_theta)
    for n_rho in n_rhos:
        acc = rng.integers(0, 9, (n_theta, n_rho)).astype(np.int32)
        acc[0, :], acc[-1, :] = rng.integers(5, 12, n_rho), rng.integers(5, 12, n_rho)      # the wrapped border
        for periodic in (False, True):
            ctx = H.Context(n_theta, n_rho, -0.005, 0.005, acc_type, 5, 1, 64, periodic=periodic)
            pj, pk, pc, m = orc.peaks(acc, 5, periodic=periodic)
            cap = m + 3
            got, n = ctx.peaks(_t(acc.astype(np.uint16).view(np.int16) if acc_type == "u16" else acc), cap)
            assert int(n.item()) == m, (n_rho, periodic)
            assert np.array_equal(H.decode_peaks(got, m), np.stack([pj, pk, pc], 1).astype(np.int64)), (n_rho, periodic)
            ctx.close()


def _graph_calls(H, form):
    """(context, outputs of a call on one input set, the same on another) for a form of call."""
    import torch
    kw = dict(periodic="periodic" in form, dedup="dedup" in form)
    n_theta, n_rho, rho, E = {"tile": (200, 128, 0.005, 64), "fused": (200, 128, 0.005, 300), "windows": (250, 1000, 0.01, 560),
                              "tall": (130, 1500, 0.01, 24), "tallmany": (70, 1500, 0.01, 200)}.get(
                                  form.split()[0], (200, 128, 0.005, 24))
    ctx = H.Context(n_theta, n_rho, -rho, rho, "i32", 4, 1, 300, **kw)
    call = form.split()[1]
    rng = np.random.default_rng(E)
    sets = []
    for seed in (1, 2):
        if call in ("event", "finder"):
            x, y, off = _events([1100 + 60 * seed], seed, 170.0, 0.01)
        else:
            sizes = rng.integers(0, 200, E)
            sizes[3], sizes[5] = 0, (33000 if E < 100 else 700)
            parts = [_events([int(n)], seed * 1000 + i, 60.0 if rho == 0.01 and i % 9 == 4 else 215.0, 0.01)[:2]
                     for i, n in enumerate(sizes)]
            x, y = (np.concatenate([p[i] for p in parts]) for i in (0, 1))
            off = np.concatenate([[0], np.cumsum(sizes)])
        sets.append((_t(x), _t(y), _t(off.astype(np.int32))))
    n = max(s[0].numel() for s in sets)
    z = lambda shape, dt=torch.int32: torch.zeros(shape, dtype=dt, device="cuda")
    outs = (z((E, 300, 2)), z(E), z(n, torch.uint8), z(E))
    ws = ctx.split_workspace(E) if call == "split" else ctx.iterative_workspace(E) if call == "iterative" else None
    acc, pk, one, st, tr = z((n_theta, n_rho)), z((4000, 2)), z(1), z(1), z((50, 6), torch.float64)

    def run(i, stream=None):
        x, y, o = sets[i]
        if call == "batch":
            ctx.run_batch(x, y, o, *outs, stream=stream)
        elif call == "relative":
            ctx.run_batch(x, y, o, *outs, stream=stream, frac=(1, 2))
        elif call == "split":
            ctx.run_batch_split(x, y, o, ws, *outs, stream=stream)
        elif call == "static":
            ctx.run_batch_split_static(x, y, o, *outs, stream=stream)
        elif call == "iterative":
            ctx.run_batch_iterative(x, y, o, (1, 2), 3, 3, ws, *outs, stream=stream)
        else:
            ctx.vote(x, y, acc, stream=stream)
            if call == "event":
                ctx.peaks(acc, 4000, pk, one, stream=stream)
            else:
                ctx.peaks_iterative(acc, 4000, (1, 2), 3, 3, pk, one, st, stream=stream)
                ctx.track_params(x, y, pk, one, 50, 1.0, tr, stream=stream)
            ctx.retain(x, y, pk, one, 4000, outs[2][:x.numel()], stream=stream)

    def results(i):
        m = sets[i][0].numel()
        if call in ("event", "finder"):
            k = int(one.item())
            return [acc.clone(), one.clone(), pk[:k].clone(), outs[2][:m].clone()] + ([tr[:min(k, 50)].clone()] if call == "finder" else [])
        npk = outs[1].cpu().numpy()
        return [outs[1].clone(), outs[2][:m].clone(), outs[3].clone()] + \
            [outs[0][e, :min(int(npk[e]), 300)].clone() for e in range(E)]

    return ctx, run, results, [*outs, acc, pk, one, st, tr]


@pytest.mark.parametrize("form", ["tile batch", "tile batch dedup", "tile batch periodic", "fused batch", "fused relative dedup",
                                  "windows batch", "windows relative periodic", "tall batch", "tall batch periodic",
                                  "tallmany batch dedup", "tallmany batch periodic", "few split", "tall split", "few static",
                                  "few iterative", "few event", "few finder"])
def test_calls_in_hip_graphs(H, form):
    """Every route of a call captured once and replayed, with eager calls of the same context on other
    data between the replays: each replay gives what the eager call gave."""
    import torch
    ctx, run, results, buffers = _graph_calls(H, form)
    run(1)                                                     # other data first
    run(0)
    torch.cuda.synchronize()
    ref = results(0)
    assert any(int(t.count_nonzero()) for t in ref)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run(0, torch.cuda.current_stream())
    for r in range(4):
        run(1)
        for b in buffers:
            b.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        got = results(0)
        assert len(got) == len(ref) and all(torch.equal(a, b) for a, b in zip(ref, got)), r
    ctx.close()


@pytest.mark.parametrize("n_theta,n_rho,periodic", [(20, 1300, True), (20, 1300, False), (40, 64, False)])
def test_spill_blocks_of_small_batches(H, orc, n_theta, n_rho, periodic):
    """Events left to the spill kernel (beyond the window of a tall grid, or above the fused kernel's
    hits), in batches on both sides of one, two and four events per workgroup: blocks of one to four
    events, all of them left, none, and every third."""
    import torch
    tall = n_rho > 1200
    wgs = torch.cuda.get_device_properties(0).multi_processor_count if tall else 4
    lo, hi = -0.01, 0.01
    g = orc.Grid(n_theta, n_rho, lo, hi)
    T, cap = 2, 200
    ctx = H.Context(n_theta, n_rho, lo, hi, "i32", T, 1, cap, periodic=periodic)
    rng = np.random.default_rng(n_theta)
    for n in (1, 3, wgs - 1, wgs, wgs + 1, 2 * wgs - 1, 2 * wgs, 4 * wgs, 4 * wgs + 3):
        for every in (1, 3):
            left = np.arange(n) % every == 0
            sizes = np.where(left, rng.integers(20, 60, n) if tall else 32768 + rng.integers(0, 9, n), rng.integers(0, 50, n))
            parts = [_events([int(m)], 500 + i, 60.0 if tall and left[i] else 215.0, 0.01)[:2] for i, m in enumerate(sizes)]
            x, y = (np.concatenate([p[i] for p in parts]) for i in (0, 1))
            off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
            for _ in range(2):
                _check(H, orc, ctx, g, T, 1, cap, x, y, off, periodic)
    ctx.close()


@pytest.mark.parametrize("n", [1, 4, 5, 9, 33, 64, 65, 128])
def test_duplicate_marks_leave_small_batches(H, orc, n):
    """After a batch by tile the marks of later copies are dropped by one wave to a workgroup per event,
    four bytes per lane at a time: counts of events and sizes on both sides of those."""
    n_theta, n_rho, lo, hi = 70, 48, -0.005, 0.005
    sizes = np.resize([255, 0, 257, 1023, 1025, 63, 4097, 1, 65, 8192 if n < 40 else 513], n)
    x, y, off = _events([int(m) for m in sizes], 90 + n, 205.0, 0.02)
    for e in range(n):
        a, k = int(off[e]), int(sizes[e]) // 3
        x[a + k:a + 2 * k], y[a + k:a + 2 * k] = x[a:a + k], y[a:a + k]
    g = orc.Grid(n_theta, n_rho, lo, hi)
    T, cap = 9, 600
    ctx = H.Context(n_theta, n_rho, lo, hi, "i32", T, 0, cap, dedup=True)
    ref, n_ref, keep_ref = orc.run_batch(g, x, y, off, threshold=T, rho_window=0, cap=cap, n_threads=8, dedup=True)
    for _ in range(2):
        pk, npk, keep, st = ctx.run_batch(_t(x), _t(y), _t(off.astype(np.int32)))
        assert np.array_equal(npk.cpu().numpy()[:n].astype(np.int64), n_ref)
        assert np.array_equal(keep.cpu().numpy()[:x.size], keep_ref)
    ctx.close()
