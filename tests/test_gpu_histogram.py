"""Histogram adjustment on the GPU against the oracle: every frame's codes
mapped onto a target histogram, bit for bit equal to ``oracle.histogram``."""

import numpy as np
import pytest
import torch

from oracle import histogram as oh
from workloads import get_workload

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2512_09664_amd as sp
    from gpu_util import DEV, run_pipeline, to_dev, to_np


def _frames(batch, img):
    a = to_np(img)
    for p in range(batch.n_pairs):
        H, W = batch.host[p].H, batch.host[p].W
        o = batch.host[p].image_offset
        for f in range(2):
            yield p, f, a[o + f * H * W:o + (f + 1) * H * W].reshape(H, W)


def _render(bits, sizes=((160, 224), (97, 131), (256, 256)), noise=0.02):
    wl = get_workload("uneven_256").with_(sizes=sizes, bits=bits, noise_sigma=noise, blur_radius=1,
                                          integrator="rk4", substeps=2, flow="lamb_oseen", seed=3)
    batch, flows, P, x2, y2, img = run_pipeline(wl)
    return batch, img


@pytest.mark.parametrize("bits", [3, 8, 12, 14])
def test_histogram_match_equals_oracle(bits):
    batch, img = _render(bits)
    before = [f.copy() for _, _, f in _frames(batch, img)]
    rng = np.random.default_rng(bits)
    target = rng.integers(0, 1000, 1 << bits).astype(np.uint32)
    target[rng.integers(0, 1 << bits)] += 1
    ws = sp.histogram_match(batch, img, to_dev(target), bits)
    torch.cuda.synchronize()
    assert sp.read_status(ws) == 0
    for (p, f, got), src in zip(_frames(batch, img), before):
        ref = oh.match(src, target, bits)
        assert np.array_equal(got, ref), f"pair {p} frame {f}: {(got != ref).sum()} codes differ"


def test_own_histogram_is_identity_and_bad_target_is_flagged():
    bits = 12
    batch, img = _render(bits, sizes=((128, 192),))
    frames = list(_frames(batch, img))
    own = np.bincount(frames[0][2].reshape(-1), minlength=1 << bits).astype(np.uint32)
    keep = to_np(img).copy()
    ws = sp.histogram_match(batch, img, to_dev(own), bits)
    torch.cuda.synchronize()
    assert sp.read_status(ws) == 0
    got = to_np(img)
    H, W = 128, 192
    assert np.array_equal(got[:H * W], keep[:H * W])           # frame 1: its own histogram
    ref2 = oh.match(keep[H * W:2 * H * W].reshape(H, W), own, bits)
    assert np.array_equal(got[H * W:2 * H * W].reshape(H, W), ref2)
    # an all-zero target leaves the images as they are and raises the flag
    keep = to_np(img).copy()
    ws = sp.histogram_match(batch, img, torch.zeros(1 << bits, dtype=torch.int32, device=DEV), bits)
    torch.cuda.synchronize()
    assert sp.read_status(ws) == 8
    assert np.array_equal(to_np(img), keep)


def test_histogram_match_full_size():
    # four 1024x1024 pairs of the scale workload, 12-bit codes, a flat target
    wl = get_workload("scale_1024").with_(sizes=((1024, 1024),) * 4)
    batch, flows, P, x2, y2, img = run_pipeline(wl)
    before = [f.copy() for _, _, f in _frames(batch, img)]
    target = np.ones(4096, dtype=np.uint32)
    ws = sp.histogram_match(batch, img, to_dev(target), 12)
    torch.cuda.synchronize()
    assert sp.read_status(ws) == 0
    for (p, f, got), src in zip(_frames(batch, img), before):
        assert np.array_equal(got, oh.match(src, target, 12))


@pytest.mark.parametrize("size", [(1, 1), (1, 7), (1, 8), (1, 9), (3, 5), (1, 23), (255, 257), (256, 128), (181, 181),
                                  (256, 256), (257, 256)])
@pytest.mark.parametrize("gap", range(8))
def test_unaligned_and_ragged_images(size, gap):
    """Images at every 2-byte alignment, shorter than one vector and a pixel
    around the workgroups' chunks; codes above the range count as the largest."""
    H, W = size
    bits, n = 6, 2 * H * W
    b = sp.PairBatch.build([size] * 2, [(2, 2)] * 2, [0] * 2, device=DEV, gaps=(0, gap, 0))
    rng = np.random.default_rng([H, W, gap])
    im = np.where(rng.random(b.n_pixels) < 0.5, 0, rng.integers(0, (1 << bits) + 3, b.n_pixels)).astype(np.uint16)
    target = rng.integers(0, 9, 1 << bits).astype(np.uint32)
    target[0] += 1
    dev = to_dev(im.view(np.int16)).view(sp.api.U16)
    sp.histogram_match(b, dev, to_dev(target), bits)
    got, want = to_np(dev), im.copy()
    for p in range(2):
        for f in range(2):
            o = (p + 1) * gap + p * n + f * H * W
            src = np.minimum(im[o:o + H * W], (1 << bits) - 1).reshape(H, W)
            want[o:o + H * W] = oh.match(src, target, bits).reshape(-1)
    assert np.array_equal(got, want)


@pytest.mark.parametrize("pairs,size", [(1, (64, 128)), (1, (1, 8193)), (1, (129, 64)), (9, (257, 257)), (20, (257, 257)),
                                        (33, (257, 257)), (140, (257, 257)), (16, (512, 512))])
def test_chunks_of_every_length(pairs, size):
    """Batches whose counting workgroups take the shortest to the longest chunks, with a
    pixel or more past the last whole one, and images of mostly one code."""
    rng = np.random.default_rng(pairs)
    b = sp.PairBatch.build([size] * pairs, [(2, 2)] * pairs, [1] * pairs, device=DEV)
    two = np.where(rng.random((2, *size)) < 0.9, 7, rng.integers(0, 256, (2, *size))).astype(np.uint16)
    img = to_dev(np.tile(two.reshape(-1), pairs))
    target = rng.integers(1, 1000, 256).astype(np.uint32)
    ws = sp.histogram_match(b, img, to_dev(target), 8)
    torch.cuda.synchronize()
    assert sp.read_status(ws) == 0
    want = np.concatenate([oh.match(f, target, 8).reshape(-1) for f in two])
    assert np.array_equal(to_np(img).reshape(pairs, -1), np.tile(want, (pairs, 1)))


def test_one_code_costs_little_more():
    """One pair of 256^2 whose pixels share one code (each an addition to one counter) takes
    at most 2.25 times as long as one of 32^2, whose count is next to nothing."""
    best = []
    for side in (32, 256):
        b = sp.PairBatch.build([(side, side)], [(2, 2)], [1], device=DEV)
        img = to_dev(np.full(b.n_pixels, 9, np.uint16))
        target = to_dev(np.ones(4096, np.uint32))
        ws = sp.histogram_match(b, img, target, 12)
        t = 1e9
        for _ in range(10):
            sp.timing_read(None)
            sp.timing_enable(True)
            sp.histogram_match(b, img, target, 12, ws)
            torch.cuda.synchronize()
            sp.timing_enable(False)
            t = min(t, sp.timing_read("histogram_match")[0])
        best.append(t)
    sp.timing_read(None)
    assert best[1] <= 2.25 * best[0], best
