"""Shapes of the expert-product tests and the kernel that each is meant for: the GPU tests run them, a host test asks the library's rule.

A shape is (E, d, F, rows per slot, expert per slot, rows behind the last slot); dtype bf16, slot schedule."""
import numpy as np


def _many(rows, experts, more, seed, low, high):
    """rows and experts, and `more` further experts of one slot each, of low .. high rows."""
    n = max(experts) + 1
    return rows + [int(v) for v in np.random.default_rng(seed).integers(low, high + 1, more)], experts + list(range(n, n + more))


def _dense_tiles():
    rows = [1500, 129, 0, 256, 257, 1, 385, 2000, 128, 513, 384, 64, 65, 96, 289, 320, 321, 32, 160, 224, 97]
    experts = [0, 0, 1, 1, 2, 2, 3, 3, 3, 4, 4, 4, 5, 5, 5, 5, 6, 6, 6, 6, 6]
    rows, experts = _many(rows, experts, 145, 31, 1, 60)             # one column tile: a tile per slot has to fill the chip
    return max(experts) + 1, 256, 512, rows, experts, 3


def _many_short():
    rows = [1500, 129, 0, 256, 257, 1, 385, 2000, 128, 513, 384, 64, 65, 96, 289, 320, 321, 32, 160, 224, 97, 127, 33]
    experts = [0, 0, 1, 1, 2, 2, 3, 3, 3, 4, 4, 4, 5, 5, 5, 5, 6, 6, 6, 6, 6, 7, 7]
    rows, experts = _many(rows, experts, 60, 7, 1, 128)              # many single-slot experts with short rows
    return max(experts) + 1, 512, 768, rows, experts, 5


def _short_tiles(E, d, F, second):
    rng = np.random.default_rng(11)
    rows, experts = [], []
    for e in range(E):
        for _ in range(1 + second(e)):
            rows.append(int(rng.integers(64, 129)))
            experts.append(e)
    return E, d, F, rows, experts, 2


FFN_SHAPES = {
    # first product's h, element by element
    "ragged": (5, 128, 256, [3, 0, 64, 65, 1, 130, 40, 0, 17], [0, 0, 1, 2, 2, 3, 3, 3, 4], 9),
    "long": (3, 256, 512, [300, 129, 0, 128, 1, 700], [0, 0, 1, 1, 2, 2], 9),
    "listed": (64, 1024, 1024, [300, 129, 0, 128, 1, 70], [0, 0, 1, 1, 2, 2], 9),
    "dense": (164, 256, 512, *_many([1500, 129, 0, 256, 257, 1, 385, 2000, 63], [0, 0, 1, 1, 2, 2, 3, 3, 3], 160, 5, 20, 64), 9),
    # whole products
    "dense tiles": _dense_tiles(),
    "many short slots": _many_short(),
    "short tiles": _short_tiles(60, 512, 2048, lambda e: e % 3 != 0),
    "short tiles, listed": _short_tiles(128, 768, 1536, lambda e: e % 17 == 3),
    "persistent": (4, 256, 512, [30000, 20000, 130, 15000, 257, 15001], [0, 1, 1, 2, 3, 3], 0),
}
# the kernel each takes: 128-column tiles (reading the slot tables, or a work list), 128-row tiles through LDS, 256 x 256 tiles
FFN_KERNEL = {
    "ragged": "columns", "long": "lds", "listed": "columns listed", "dense": "dense", "dense tiles": "dense", "many short slots": "dense",
    "short tiles": "dense", "short tiles, listed": "columns listed", "persistent": "dense",
}

# Shapes of the tests on bad tables: kernel, dtype, d, F, factor on the rows per slot, empty slots behind, experts at least.  BAD_ROWS: the
# rows per slot of the two tests before the factor.
BAD_ROWS = ([5, 3, 4, 0, 33, 6, 2, 9, 4], [7, 40, 1, 18])
BAD_TABLES = [
    ("f32 short", 64, 320, 1, 0, 0),
    ("f32 64 rows", 320, 448, 12, 0, 0),
    ("f32 staged", 512, 1536, 20, 0, 0),
    ("f32 narrow", 256, 384, 1, 0, 0),
    ("few rows", 128, 1024, 1, 200, 0),
    ("columns", 128, 256, 3, 0, 0),
    ("columns listed", 1024, 1024, 11, 2, 64),
    ("lds", 256, 512, 10, 0, 0),
    ("dense", 256, 512, 165, 160, 0),
]
