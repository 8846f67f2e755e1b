"""Host checks of the arithmetic the permutation kernels sort and multiply with: the 64-bit angle key against the
exact comparator, the digits of a value by one addition, and the order in which digits are stored."""
import functools

import numpy as np

from oracle.permutation import angle_precedes
from tests.test_mfma_arithmetic import balanced_digits


def angle_key(x: int, y: int) -> int:
    """Upper 52 bits of the kernels' sort key: the angle class, then 50 bits of +-x / (|x| + |y|) in the half-planes
    (one correctly rounded division, as Python's)."""
    c = 0 if y < 0 else 2 if y > 0 else (1 if x >= 0 else 3)
    u = 0
    if c in (0, 2):
        q = float(x if c == 0 else -x) / float(abs(x) + abs(y)) + 0.0
        b = int(np.float64(q).view(np.uint64))
        u = (~b & (2**64 - 1)) if b >> 63 else b | (1 << 63)
    return (c << 50) | (u >> 14)


def test_angle_key_never_contradicts_the_exact_order():
    rng = np.random.default_rng(1)
    lim = (1 << 30) + 1
    pts = [tuple(int(v) for v in p) for p in rng.integers(-lim, lim + 1, size=(400, 2))]
    pts += [(0, 0), (5, 0), (-5, 0), (0, 7), (0, -7), (lim, lim), (lim, -lim), (-lim, lim), (-lim, -lim)]
    for k in range(60):  # directions closer than 50 bits resolve, in every quadrant
        a, b = lim - 2 * k, lim - 2 * k - 1
        pts += [(s * a, t * b) for s in (1, -1) for t in (1, -1)] + [(s * b, t * (b - 1)) for s in (1, -1) for t in (1, -1)]
    pts += [(x * 3, y * 3) for x, y in pts[:20] if max(abs(x), abs(y)) * 3 <= lim]  # equal angles
    pts = [(x, y, i) for i, (x, y) in enumerate(pts)]
    exact = sorted(pts, key=functools.cmp_to_key(lambda p, q: -1 if angle_precedes(p, q) else 1))
    keys = [angle_key(x, y) for x, y, _ in exact]
    assert keys == sorted(keys)
    # keys that agree are one run: the pass over neighbours that puts a run in the exact order needs no more
    assert len(set(keys)) < len({(x, y) for x, y, _ in pts})


def test_digits_by_one_addition():
    rng = np.random.default_rng(2)
    lim = (1 << 30) + 1
    v = np.concatenate([rng.integers(-lim, lim + 1, 100000), [0, 1, -1, 127, 128, -128, -129, lim, -lim]]).astype(np.int64)
    w = ((v + 0x80808080) & 0xFFFFFFFF) ^ 0x80808080
    got = np.stack([((w >> (8 * b)) & 0xFF).astype(np.uint8).view(np.int8) for b in range(4)], axis=-1)
    assert np.array_equal(got, balanced_digits(v))


def test_stored_digit_order_matches_the_mask_bytes():
    """Operand slot 4 d + i of MFMA j holds bit 32 (j / 2) + 4 (j mod 2) + d + 8 i of a word; the digit of that row is
    stored at byte 16 j + 4 d + i of the word's 64."""
    stored = np.empty(64, dtype=int)
    for row in range(64):  # dword 8 (row / 32) + row mod 8, byte (row / 8) mod 4
        stored[4 * (8 * (row // 32) + row % 8) + (row // 8) % 4] = row
    for j in range(4):
        for d in range(4):
            for i in range(4):
                assert stored[16 * j + 4 * d + i] == 32 * (j // 2) + 4 * (j % 2) + d + 8 * i
