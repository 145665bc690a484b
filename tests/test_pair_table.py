"""The pair table (host logic, no GPU): its columns and the checks on its inputs."""

import pytest

pytest.importorskip("torch")

import paper_2512_09664_amd as sp  # noqa: E402

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
