"""The pair table (host logic, no GPU): its columns and the checks on its inputs."""

import time

import numpy as np
import pytest

pytest.importorskip("torch")
import torch  # noqa: E402

import paper_2512_09664_amd as sp  # noqa: E402
from paper_2512_09664_amd import _lib as L  # noqa: E402

N = (1, 3, 40)


def _args(n):
    return dict(sizes=[(24 + p, 40) for p in range(n)], grids=[(6, 10 + p % 2) for p in range(n)],
                n_max=[5 + p for p in range(n)], device="cpu")


@pytest.mark.parametrize("short", [0, 1, -1])
@pytest.mark.parametrize("name", ["grids", "n_max", "pair_ids", "flow_index"])
@pytest.mark.parametrize("n", N[1:])
def test_short_sequences_are_refused(n, name, short):
    """A sequence with fewer entries than pairs (none, one, all but one) raises."""
    kw = _args(n)
    kw.update(pair_ids=list(range(7, 7 + n)), flow_index=[0] * n)
    kw[name] = list(kw[name])[:short % n]
    with pytest.raises(IndexError):
        sp.PairBatch.build(**kw)


@pytest.mark.parametrize("ids", [[5], [1, 2], [1, 2, 3, 4], []])
def test_other_ids_need_one_per_pair(ids):
    b = sp.PairBatch.build(**_args(3))
    with pytest.raises(ValueError):
        b.with_pair_ids(ids)


def _plain(sizes, grids, n_max, pair_ids=None, gaps=(0, 0, 0), flow_index=None, **_):
    """The table by its definition: one ctypes record per pair, and the arrays' sizes."""
    arr = (L.Pair * len(sizes))()
    po = io = fo = 0
    for p, ((H, W), (Gh, Gw)) in enumerate(zip(sizes, grids)):
        po, io, fo = po + gaps[0], io + gaps[1], fo + gaps[2]
        arr[p].H, arr[p].W, arr[p].Gh, arr[p].Gw, arr[p].n_max = H, W, Gh, Gw, n_max[p]
        arr[p].particle_offset, arr[p].image_offset, arr[p].flow_offset = po, io, fo
        arr[p].pair_id = pair_ids[p] if pair_ids is not None else p
        po, io, fo = po + n_max[p], io + 2 * H * W, fo + 2 * Gh * Gw
    if flow_index is not None:
        ends = []
        for p, (Gh, Gw) in enumerate(grids):
            arr[p].flow_offset = 2 * Gh * Gw * flow_index[p]
            ends.append(arr[p].flow_offset + 2 * Gh * Gw)
        fo = max([0] + ends)
    return arr, po, io, fo


@pytest.mark.parametrize("gaps", [(0, 0, 0), (3, 5, 8)])
@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("ids", [False, True])
@pytest.mark.parametrize("n", [0, 1, 2, 23, 24, 25, 70])
def test_table(n, ids, shared, gaps):
    """Both builders around the size where they change over."""
    kw = dict(_args(n), gaps=gaps)
    if ids:
        kw["pair_ids"] = [(1 << 64) - 1 - 3 * p for p in range(n)]
    if shared:
        kw["flow_index"] = [p // 3 for p in range(n)]
    b = sp.PairBatch.build(**kw)
    arr, po, io, fo = _plain(**kw)
    assert bytes(b.host) == bytes(arr) == bytes(b.dev.numpy())
    assert (b.n_pairs, b.n_particles, b.n_pixels, b.n_flow) == (n, po, io, fo)
    assert b.n_max == tuple(kw["n_max"]) and b.grids == tuple(kw["grids"]) and b.sizes == tuple(kw["sizes"])


def test_small_tables_are_cheap():
    """One pair's table costs little more than the plain record and its upload (the
    best of many runs of both in turn; half as much again is allowed)."""
    kw = _args(1)

    def plain():
        arr, po, io, fo = _plain(**kw)
        t = torch.from_numpy(np.frombuffer(bytes(arr), dtype=np.uint8).copy()).to("cpu")
        return sp.PairBatch(arr, t, 1, po, io, fo, tuple(map(tuple, kw["sizes"])), tuple(map(tuple, kw["grids"])),
                            tuple(int(v) for v in kw["n_max"]))

    best = [1e9, 1e9]
    for _ in range(60):
        for k, f in enumerate((plain, lambda: sp.PairBatch.build(**kw))):
            t = time.perf_counter()
            for _ in range(20):
                f()
            best[k] = min(best[k], time.perf_counter() - t)
    assert best[1] <= 1.5 * best[0], best
