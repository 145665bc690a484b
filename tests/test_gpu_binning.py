"""The binning and order forms (one launch for small pairs, three for larger
ones, with and without a layout launch, fused and separate scans) against the
oracle's tile lists and against the advection in index order."""

import numpy as np
import pytest

pytest.importorskip("torch")
import torch  # noqa: E402

import gpu_util as gu  # noqa: E402
import paper_2512_09664_amd as sp  # noqa: E402
from oracle import bins as obins  # noqa: E402

pytestmark = pytest.mark.gpu


def _particles(sizes, counts, seed):
    rng = np.random.default_rng(seed)
    out = {k: [] for k in ("x", "y", "x2", "y2", "z", "d", "I0")}
    for (H, W), n in zip(sizes, counts):
        x, y = rng.uniform(-4, W + 4, n), rng.uniform(-4, H + 4, n)
        out["x"].append(x)
        out["y"].append(y)
        out["x2"].append(x + rng.uniform(-3, 3, n))
        out["y2"].append(y + rng.uniform(-3, 3, n))
        out["z"].append(rng.uniform(-1, 1, n))
        out["d"].append(rng.uniform(1.0, 5.0, n))
        out["I0"].append(np.where(rng.random(n) < 0.1, 0.0, 0.01))
    return {k: np.concatenate(v).astype(np.float32) for k, v in out.items()}


# pairs of one launch (at most 8192 particles), of three, a wave of pairs and one more
BATCHES = [([(96, 128)], [8192]), ([(96, 128)], [8193]), ([(40, 24)] * 63 + [(96, 128)], [3] * 63 + [9000]),
           ([(40, 24)] * 64 + [(96, 128)], [3, 0] * 32 + [9000]), ([(40, 24)] * 65, [7, 0, 30, 1, 0] * 13)]


@pytest.mark.parametrize("batch", range(len(BATCHES)))
@pytest.mark.parametrize("tile", [(64, 32, 2048, 64), (8, 8, 256, 64)])
def test_lists_match_oracle(batch, tile):
    sizes, counts = BATCHES[batch]
    q = _particles(sizes, counts, batch)
    b = gu.batch_for(sizes, [(4, 4)] * len(sizes), counts)
    rp = sp.render_params(0.5, 5.0, 1, 0.7, 0.0, 12)
    t = {k: gu.to_dev(v) for k, v in q.items()}
    tl = sp.tiling(*tile)
    ws = sp.alloc_workspace(b, rp, tl)
    sp.render_pair(b, t["x"], t["y"], t["x2"], t["y2"], t["z"], t["d"], t["I0"], rp, tl, workspace=ws)
    torch.cuda.synchronize()
    assert sp.read_status(ws) == 0
    count, offset, entries = (gu.to_np(v) for v in sp.bin_views(b, rp, tl, ws))
    base = o = 0
    for (H, W), n in zip(sizes, counts):
        sl = slice(o, o + n)
        o += n
        nt = int(np.prod(obins.tile_grid(H, W, tile[1], tile[0])))
        for f, (xk, yk) in enumerate((("x", "y"), ("x2", "y2"))):
            if not (q["I0"][sl] > 0).any():          # the oracle takes at least one particle
                assert not count[f, base:base + nt].any()
                continue
            c, off, ent = obins.bin_frame(q[xk][sl], q[yk][sl], q["d"][sl], q["I0"][sl], H, W, tile[1], tile[0], 1)
            assert np.array_equal(count[f, base:base + nt], c)
            go = offset[f, base:base + nt]
            assert np.array_equal(go - go[0], off[:-1])
            for k in range(nt):
                assert np.array_equal(np.sort(entries[go[k]:go[k] + c[k]]), ent[off[k]:off[k + 1]])
        base += nt


@pytest.mark.parametrize("batch", range(len(BATCHES)))
def test_flags_are_raised_and_cleared(batch):
    """A diameter above d_max in either frame's lists raises its bit in every
    form; the next call on the same workspace clears it."""
    sizes, counts = BATCHES[batch]
    q = _particles(sizes, counts, batch)
    b = gu.batch_for(sizes, [(4, 4)] * len(sizes), counts)
    rp = sp.render_params(0.5, 5.0, 0, 0.7, 0.0, 0)
    t = {k: gu.to_dev(v) for k, v in q.items()}
    ws = sp.alloc_workspace(b, rp)
    for d, want in ((6.0, sp._lib.SP_STATUS_D_ABOVE_MAX), (2.0, 0)):
        t["d"][-1], t["I0"][-1] = d, 0.01
        sp.render_pair(b, t["x"], t["y"], t["x2"], t["y2"], t["z"], t["d"], t["I0"], rp, workspace=ws)
        torch.cuda.synchronize()
        assert sp.read_status(ws) == want


@pytest.mark.parametrize("batch", range(len(BATCHES)))
def test_order_does_not_change_positions(batch):
    """Enough substeps that the home-block order is built: the same bits as in
    index order."""
    sizes, counts = BATCHES[batch]
    q = _particles(sizes, counts, batch)
    b = gu.batch_for(sizes, [(12, 10)] * len(sizes), counts)
    flow = gu.to_dev(np.random.default_rng(batch).normal(0, 1, b.n_flow).astype(np.float32))
    ap = sp.advect_params(1.0, 1024, "rk4")
    x, y = gu.to_dev(q["x"]), gu.to_dev(q["y"])
    ordered = sp.advect(b, flow, ap, x, y)
    plain = sp.advect(b, flow, ap, x, y, ordered=False)
    for u, v in zip(ordered, plain):
        assert torch.equal(u, v)


@pytest.mark.parametrize("integrator", ["euler", "rk4"])
@pytest.mark.parametrize("batch", range(len(BATCHES)))
def test_order_does_not_change_positions_out_of_plane(batch, integrator):
    """Motion out of the plane: planar results and z as in index order, with
    waves and windows that straddle pairs, and particles that leave the window;
    a workspace too small for the order is passed over."""
    sizes, counts = BATCHES[batch]
    q = _particles(sizes, counts, batch)
    b = gu.batch_for(sizes, [(12, 10)] * len(sizes), counts)
    rng = np.random.default_rng(batch)
    flow = gu.to_dev(rng.normal(0, 6, b.n_flow).astype(np.float32))
    w = gu.to_dev(rng.normal(0, 1, b.n_flow // 2).astype(np.float32))
    ap = sp.advect_params(1.0, 1024, integrator)
    x, y, z = (gu.to_dev(q[k]) for k in ("x", "y", "z"))
    ordered = sp.advect(b, flow, ap, x, y, wflow=w, z1=z)
    plain = sp.advect(b, flow, ap, x, y, wflow=w, z1=z, ordered=False)
    small = sp.advect(b, flow, ap, x, y, wflow=w, z1=z, workspace=torch.empty(256, dtype=torch.uint8, device=gu.DEV))
    planar = sp.advect(b, flow, ap, x, y)
    for u, v, s in zip(ordered, plain, small):
        assert torch.equal(u, v) and torch.equal(u, s)
    assert torch.equal(planar[0], ordered[0]) and torch.equal(planar[1], ordered[1])


@pytest.mark.parametrize("out_of_plane", [False, True])
def test_index_order_allocates_nothing(out_of_plane):
    """Without a workspace, a call that runs in index order takes no memory."""
    b = gu.batch_for([(96, 128)], [(12, 10)], [8192])
    flow = torch.zeros(b.n_flow, device=gu.DEV)
    x, y, z, x2, y2, z2 = (torch.ones(8192, device=gu.DEV) for _ in range(6))
    ap = sp.advect_params(1.0, 4, "rk4")
    kw = dict(wflow=torch.zeros(b.n_flow // 2, device=gu.DEV), z1=z, z2=z2) if out_of_plane else {}
    before = torch.cuda.memory_stats()["allocation.all.allocated"]
    sp.advect(b, flow, ap, x, y, x2, y2, **kw)
    assert torch.cuda.memory_stats()["allocation.all.allocated"] == before
    assert torch.equal(x2, x) and torch.equal(y2, y)


def test_out_of_plane_runs_without_memory_for_the_order(monkeypatch):
    """Motion out of the plane falls back to index order where the order's temporary
    cannot be had, as it never needed one."""
    n = 200_000
    b = gu.batch_for([(512, 512)] * 16, [(128, 128)] * 16, [n // 16] * 16)
    rng = np.random.default_rng(4)
    flow, w = (gu.to_dev(rng.normal(0, 2, k).astype(np.float32)) for k in (b.n_flow, b.n_flow // 2))
    x, y, z = (gu.to_dev(rng.uniform(0, 512, n).astype(np.float32)) for _ in range(3))
    ap = sp.advect_params(1.0, 16, "rk4")
    want = sp.advect(b, flow, ap, x, y, wflow=w, z1=z)
    assert sp.advect_workspace_needed(b, ap, True) > 0

    def refuse(*a, **k):
        raise torch.OutOfMemoryError("no memory")

    monkeypatch.setattr(torch, "empty", refuse)
    got = sp.advect(b, flow, ap, x, y, wflow=w, z1=z)
    monkeypatch.undo()
    for u, v in zip(got, want):
        assert torch.equal(u, v)


def _tiny(counts, grid=(4, 4), side=32, seed=6):
    rng = np.random.default_rng(seed)
    b = gu.batch_for([(side, side)] * len(counts), [grid] * len(counts), counts)
    x, y, z = (gu.to_dev(rng.uniform(-2, side + 2, b.n_particles).astype(np.float32)) for _ in range(3))
    flow, w = (gu.to_dev(rng.normal(0, 2, k).astype(np.float32)) for k in (b.n_flow, b.n_flow // 2))
    return b, x, y, z, flow, w


@pytest.mark.parametrize("integrator", ["euler", "rk4"])
@pytest.mark.parametrize("out_of_plane", [False, True])
def test_waves_of_many_pairs(integrator, out_of_plane):
    """Pairs of a few particles each, so that a wave holds one, two or many of them,
    against each pair by itself."""
    counts = [1, 70, 0, 3, 64, 2, 2, 0, 0, 5, 130, 1, 1, 1, 40, 17, 9, 60, 4]
    b, x, y, z, flow, w = _tiny(counts)
    ap = sp.advect_params(1.0, 3, integrator)
    got = sp.advect(b, flow, ap, x, y, **(dict(wflow=w, z1=z) if out_of_plane else {}))
    one_flow = flow.reshape(len(counts), -1)
    one_w = w.reshape(len(counts), -1)
    for p, n in enumerate(counts):
        if not n:
            continue
        o = b.host[p].particle_offset
        one = gu.batch_for([(32, 32)], [(4, 4)], [n])
        xs, ys, zs = (t[o:o + n].clone() for t in (x, y, z))
        kw = dict(wflow=one_w[p].clone(), z1=zs) if out_of_plane else {}
        for u, v in zip(sp.advect(one, one_flow[p].clone(), ap, xs, ys, **kw), got):
            assert torch.equal(u, v[o:o + n]), p


def test_waves_of_many_pairs_cost():
    """The same particles in eight times as many pairs take at most twice as long (a
    wave's pairs are moved together)."""
    ap = sp.advect_params(1.0, 256, "rk4")
    best = []
    for pairs in (8, 64):
        b, x, y, _, flow, _ = _tiny([512 // pairs] * pairs)
        t = 1e9
        for _ in range(6):
            sp.timing_read(None)
            sp.timing_enable(True)
            sp.advect(b, flow, ap, x, y, ordered=False)
            torch.cuda.synchronize()
            sp.timing_enable(False)
            t = min(t, sp.timing_read("advect")[0])
        best.append(t)
    sp.timing_read(None)
    assert best[1] <= 2.0 * best[0], best


MANY = [3, 0, 300, 1, 1100] * 120       # more pairs than the chip holds workgroups of 1024


@pytest.mark.parametrize("tile", [(64, 32, 2048, 64), (8, 8, 256, 64)])
def test_many_small_pairs_lists_and_flags(tile):
    """Pairs enough for the smaller workgroups: tile lists against the oracle for every
    seventh pair, counts of all pairs, and status bits of the last one."""
    sizes = [(40, 24)] * len(MANY)
    q = _particles(sizes, MANY, 17)
    b = gu.batch_for(sizes, [(4, 4)] * len(sizes), MANY)
    rp = sp.render_params(0.5, 5.0, 1, 0.7, 0.0, 12)
    t = {k: gu.to_dev(v) for k, v in q.items()}
    tl = sp.tiling(*tile)
    ws = sp.alloc_workspace(b, rp, tl)
    args = [t[k] for k in ("x", "y", "x2", "y2", "z", "d", "I0")]
    sp.render_pair(b, *args, rp, tl, workspace=ws)
    assert sp.read_status(ws) == 0
    count, offset, entries = (gu.to_np(v) for v in sp.bin_views(b, rp, tl, ws))
    nt = int(np.prod(obins.tile_grid(40, 24, tile[1], tile[0])))
    for p, n in enumerate(MANY):
        o = b.host[p].particle_offset
        sl = slice(o, o + n)
        for f, (xk, yk) in enumerate((("x", "y"), ("x2", "y2"))):
            got = count[f, p * nt:(p + 1) * nt]
            if not (q["I0"][sl] > 0).any():
                assert not got.any()
                continue
            if p % 7 and n > 3:
                continue
            c, off, ent = obins.bin_frame(q[xk][sl], q[yk][sl], q["d"][sl], q["I0"][sl], 40, 24, tile[1], tile[0], 1)
            assert np.array_equal(got, c), (p, f)
            go = offset[f, p * nt:(p + 1) * nt]
            for k in range(nt):
                assert np.array_equal(np.sort(entries[go[k]:go[k] + c[k]]), ent[off[k]:off[k + 1]]), (p, f, k)
    t["d"][-1], t["I0"][-1] = 6.0, 0.01
    sp.render_pair(b, *args, rp, tl, workspace=ws)
    assert sp.read_status(ws) == sp._lib.SP_STATUS_D_ABOVE_MAX


ORDERED = {     # sizes, particles, grid, substeps: batches whose order is built in both forms
    "one launch, 600 pairs": ([(40, 24)] * 600, MANY, (12, 10), 1024),
    "one launch, 70 pairs": ([(96, 128)] * 70, [4000, 0, 700, 1, 8192] * 14, (24, 32), 64),
    "chunks, a wave of pairs": ([(256, 256)] * 64, [9000] * 64, (64, 64), 16),
    "chunks, more pairs": ([(256, 256)] * 66, [9000, 0, 3] * 22, (64, 64), 64),
    "64-pixel blocks": ([(4160, 4160), (300, 200)], [300_000, 5000], (64, 64), 32),
    "64-pixel blocks, the most": ([(8192, 8192)], [400_000], (64, 64), 32),
    "128-pixel blocks": ([(16384, 16384), (64, 64)], [400_000, 100], (64, 64), 32),
    "separate scans": ([(2048, 2048)], [300_000], (512, 512), 16)}


@pytest.mark.parametrize("integrator", ["euler", "rk4"])
@pytest.mark.parametrize("name", list(ORDERED))
def test_ordered_advection(name, integrator):
    """The home-block order in every form that it is built in (asserted), planar and out
    of the plane, with particles outside the image and outside the windows: the same bits
    as in index order."""
    sizes, counts, grid, substeps = ORDERED[name]
    substeps = min(substeps * (4 if integrator == "euler" else 1), 1024)
    b = gu.batch_for(sizes, [grid] * len(sizes), counts)
    gen = torch.Generator(device=gu.DEV).manual_seed(len(name))
    side = torch.tensor([[w, h] for h, w in sizes], dtype=torch.float32, device=gu.DEV)
    side = side.repeat_interleave(torch.tensor(counts, device=gu.DEV), 0)
    xy = torch.rand(b.n_particles, 2, generator=gen, device=gu.DEV) * (side + 8.0) - 4.0
    x, y = xy[:, 0].contiguous(), xy[:, 1].contiguous()
    x[::501], y[::777] = float("nan"), 3.0e7
    z = torch.rand(b.n_particles, generator=gen, device=gu.DEV)
    flow, w = (3.0 * torch.randn(k, generator=gen, device=gu.DEV) for k in (b.n_flow, b.n_flow // 2))
    ap = sp.advect_params(1.0, substeps, integrator)
    for kw in ({}, dict(wflow=w, z1=z)):
        assert sp.advect_workspace_needed(b, ap, bool(kw)) > 0
        got = sp.advect(b, flow, ap, x, y, **kw)
        want = sp.advect(b, flow, ap, x, y, ordered=False, **kw)
        for u, v in zip(got, want):
            assert torch.equal(u.view(torch.int32), v.view(torch.int32))


@pytest.mark.parametrize("tile", [(64, 32, 256, 64), (32, 32, 256, 64)])
@pytest.mark.parametrize("n", [16384, 16385, 17000])
def test_separate_scans(n, tile):
    """A pair on either side of the chunk count from which its scans are launches of
    their own: tile lists against the oracle."""
    size = (96, 128)
    q = _particles([size], [n], n)
    b = gu.batch_for([size], [(4, 4)], [n])
    rp = sp.render_params(0.5, 5.0, 1, 0.7, 0.0, 12)
    tl = sp.tiling(*tile)
    ws = sp.alloc_workspace(b, rp, tl)
    sp.render_pair(b, *[gu.to_dev(q[k]) for k in ("x", "y", "x2", "y2", "z", "d", "I0")], rp, tl, workspace=ws)
    count, offset, entries = (gu.to_np(v) for v in sp.bin_views(b, rp, tl, ws))
    for f, (xk, yk) in enumerate((("x", "y"), ("x2", "y2"))):
        c, off, ent = obins.bin_frame(q[xk], q[yk], q["d"], q["I0"], *size, tile[1], tile[0], 1)
        assert np.array_equal(count[f], c)
        assert np.array_equal(offset[f] - offset[f][0], off[:-1])
        for k in range(len(c)):
            o = offset[f][k]
            assert np.array_equal(np.sort(entries[o:o + c[k]]), ent[off[k]:off[k + 1]]), (f, k)
