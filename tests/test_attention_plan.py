"""The rule that takes attention's chunks beyond 64 tiles: over random lengths the list schedule with them never ends later than without."""
import numpy as np
import pytest

import attention_plan_model as model


@pytest.mark.parametrize("spread", [0.0, 0.05, 0.2, 0.8])
def test_longer_chunks_never_end_later(spread):
    rng = np.random.default_rng(3)
    switched = 0
    for _ in range(1500):
        B, ctx, heads = int(np.exp(rng.uniform(0.7, 4.5))), np.exp(rng.uniform(7, 10.4)), int(rng.choice([1, 2, 4, 8, 12, 16, 32]))
        lens = np.clip(ctx * np.exp(rng.normal(0, spread, B)), 1, 32768).astype(int)
        if B > 2 and rng.random() < 0.2:
            lens[rng.integers(B)] = rng.integers(0, 64)
        tiles = model.tiles_of(lens, 1)
        size, short = model.chunk_size(tiles, heads), model.short_size(tiles, heads)[0]
        if size != short:
            switched += 1
            for cost in (3, 4, 6):   # what an item costs besides its tiles, with one to three row tiles per wave
                assert model.span(tiles, size, heads, cost) <= model.span(tiles, short, heads, cost), (lens.tolist(), heads, cost)
    assert switched


def test_counts_by_reciprocal():
    """The planner's chunk counts, ceil((tiles - 1/2) * (1 / size)) in fp32, are exact: all small counts, and next to multiples of the sizes up to 2^21 tiles."""
    for size in list(range(4, 65)) + list(range(67, 257, 3)):
        inv = np.float32(1) / np.float32(size)
        multiples = np.arange(size, 1 << 21, size, dtype=np.int64)
        for tiles in (np.arange(5000), multiples - 1, multiples, np.minimum(multiples + 1, (1 << 21) - 1)):
            got = np.ceil((tiles.astype(np.float32) - np.float32(0.5)) * inv)
            assert got.dtype == np.float32 and (got.astype(np.int64) == model.counts(tiles, size)).all(), size
