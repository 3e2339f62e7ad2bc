"""The autotuner times every launch of the level sums once."""
import pytest

pytest.importorskip("torch")


@pytest.mark.parametrize("batch,n", [(1, 4), (2, 4), (4, 8), (5, 5), (8, 7), (64, 7)])
def test_distinct_tiles(batch, n):
    from paper_2606_28865_amd import autotune
    got, every = autotune.distinct_tiles(batch), autotune.tile_candidates(batch)
    assert len(got) == len(set(got)) == n
    # in the candidates' order, the persistent launches all there, and below
    # five densities everything
    assert got == [t for t in every if t in got]
    assert [t for t in got if t[2]] == [t for t in every if t[2]]
    assert batch >= 5 or got == every
    assert any(not t[2] for t in got)
