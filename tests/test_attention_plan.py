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
