"""Which query's row the evaluation's per-query kernel reads for each place of a block's known answers laid end to end
(32 queries per block, 32 places per matrix-core tile, the last of either partly filled).  Host arithmetic, no GPU."""
import numpy as np
import pytest


@pytest.fixture(scope="module")
def kb():
    import os
    from paper_2201_02791_amd import build, binding
    if not os.path.exists(binding.LIB_PATH):
        build.build(verbose=False)
    binding.load()
    return binding


@pytest.mark.parametrize("n_known", [[1], [0, 3], [5, 0, 0], [0] * 19 + [40], [33] + [0] * 30, [2] * 31, [0] * 31 + [1], [7] * 32])
def test_every_place_of_a_tile_names_a_query_of_the_block(kb, n_known):
    owner = np.repeat(np.arange(len(n_known)), n_known)
    for at in range((len(owner) + 31) // 32 * 32):
        i, n = kb.pair_query_for_tests(n_known, at)
        assert n == len(owner)
        if at < len(owner):
            assert i == owner[at]
        else:                                   # no pair: its score is dropped, but the row is read
            assert 0 <= i < len(n_known), at


@pytest.mark.parametrize("n_known", [[70_000_000] * 32, [2**31 - 1, 5], [3, 2**31 - 1, 0, 2**31 - 1]])
def test_more_places_than_32_bits_count(kb, n_known):
    starts = np.concatenate([[0], np.cumsum(n_known)])
    for i, n in enumerate(n_known):
        for at in (starts[i], starts[i] + n - 1) if n else ():
            assert kb.pair_query_for_tests(n_known, int(at)) == (i, starts[-1])
