"""The attention planner's choice of chunk lengths in plain Python, and a list schedule of the work items: 256 workgroups at a time, longest first.
Lengths are in tiles of 64 keys."""
import heapq

import numpy as np

ROUND = 4   # what an item costs besides its tiles


def counts(tiles, size):
    return -(-tiles // size)


def rounds(n, heads):
    return -(-int(n) * heads // 256)


def short_size(tiles, heads):
    """The shortest chunks, of 4 to 64 tiles, with no more rounds than chunks of 64 need."""
    r = max(rounds(counts(tiles, 64).sum(), heads), -(-int(tiles.sum()) * heads // (256 * 64)), 1)
    return next(t for t in range(4, 65) if rounds(counts(tiles, t).sum(), heads) <= r), r


def chunk_size(tiles, heads):
    size, r = short_size(tiles, heads)
    if r == 1:
        return size
    n = int(counts(tiles, size).sum())
    long = [c for c in chunks(tiles, size) if 2 * c >= size]
    least = max((int(tiles.sum()) + n * ROUND) * heads / 256, rounds(len(long), heads) * (min(long, default=0) + ROUND))
    most, longer = min((rounds(counts(tiles, s).sum(), heads) * (s + ROUND), s) for s in range(67, 257, 3))
    return longer if most < least else size


def chunks(tiles, size):
    out = []
    for t in tiles[tiles > 0]:
        k = -(-int(t) // size)
        per = -(-int(t) // k)
        out += [max(min(per, int(t) - i * per), 0) for i in range(k)]
    return sorted(out, reverse=True)


def span(tiles, size, heads, cost=ROUND):
    """When the last item ends."""
    free = [0] * 256
    for c in chunks(tiles, size):
        for _ in range(heads):
            heapq.heapreplace(free, free[0] + (c + cost if c else 0))
    return max(free)


def tiles_of(lens, n):
    return (np.asarray(lens, dtype=np.int64) + n + 63) // 64
