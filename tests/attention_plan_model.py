"""The attention planner's choice of the chunk length in plain Python.  Lengths are in tiles of 64 keys."""
import numpy as np


def tiles_of(lens, n):
    return (np.asarray(lens, dtype=np.int64) + n + 63) // 64


def counts(tiles, size):
    return -(-tiles // size)


def rounds(n, heads):
    return -(-int(n) * heads // 256)


def chunk_size(tiles, heads):
    """The shortest chunks, of 4 to 64 tiles, with no more rounds of 256 workgroups than chunks of 64 need."""
    r = max(rounds(counts(tiles, 64).sum(), heads), -(-int(tiles.sum()) * heads // (256 * 64)), 1)
    return next(t for t in range(4, 65) if rounds(counts(tiles, t).sum(), heads) <= r)
