"""The ground-truth flow kernel's pixel runs and pair groups against its
binary32 mirror bit for bit."""

import numpy as np
import pytest

pytest.importorskip("torch")

import gpu_util as gu  # noqa: E402
import paper_2512_09664_amd as sp  # noqa: E402
from oracle import ra32 as ra  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("n_pairs", [1, 7, 8, 9, 17])
@pytest.mark.parametrize("size", [(1, 1), (3, 5), (2, 1), (33, 15), (64, 48)])
def test_flow_fields(size, n_pairs, shared):
    H, W = size
    sizes = [(H, W)] * n_pairs
    if not shared:
        sizes[n_pairs // 2] = (H + 1, W)
    grids = [(4, 6)] * n_pairs
    index = [p // 3 for p in range(n_pairs)] if shared else None
    b = sp.PairBatch.build(sizes, grids, [0] * n_pairs, device=gu.DEV, flow_index=index)
    flow = np.random.default_rng(n_pairs).normal(0, 3, b.n_flow).astype(np.float32)
    out = gu.to_np(sp.flow_field(b, gu.to_dev(flow)))
    for p in range(n_pairs):
        h, w = sizes[p]
        o, fo = b.host[p].image_offset, b.host[p].flow_offset
        ref = ra.flow_field(flow[fo:fo + 48].reshape(4, 6, 2), h, w)
        assert np.array_equal(out[o:o + 2 * h * w].reshape(h, w, 2), ref), p
