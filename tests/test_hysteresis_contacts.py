"""The rule by which the device joins edge components across the 32-pixel tiles of the pre-pass (each contact of
two runs along a border once, by its first pair; csrc/hysteresis.h, union_border), on the CPU: components joined
inside tiles plus those contacts must be the image's 8-connected components, for any mask of candidates."""
import numpy as np
import pytest
from scipy.ndimage import label

T = 32


def _components(m):
    h, w = m.shape
    parent = {(y, x): (y, x) for y, x in np.argwhere(m).tolist()}

    def find(a):
        while parent[a] != a:
            a = parent[a]
        return a

    def join(a, b):
        a, b = find(a), find(b)
        parent[max(a, b)] = min(a, b)

    for y, x in list(parent):                                   # inside a tile
        for n in ((y, x + 1), (y + 1, x - 1), (y + 1, x), (y + 1, x + 1)):
            if n in parent and n[0] // T == y // T and n[1] // T == x // T:
                join((y, x), n)
    for row in (True, False):                                   # across a border
        across_len, along_len = (h, w) if row else (w, h)
        for k in range((across_len - 1) // T):
            for at in range(along_len):
                def pos(side, j):
                    a, b = T * k + T - 1 + side, at + j
                    return (a, b) if row else (b, a)
                c = [[pos(side, j) in parent for j in (-1, 0, 1)] for side in (0, 1)]
                if not c[0][1]:
                    continue
                if c[1][1]:
                    if not (at % T != 0 and c[0][0] and c[1][0]):
                        join(pos(0, 0), pos(1, 0))
                    continue
                for j in (-1, 1):
                    if c[1][1 + j] and not c[0][1 + j]:
                        join(pos(0, 0), pos(1, j))
    return len({find(p) for p in parent})


@pytest.mark.parametrize("seed", range(8))
def test_contacts_across_tiles_give_the_image_components(seed):
    rng = np.random.default_rng(seed)
    for _ in range(12):
        h, w = rng.integers(33, 70, 2)
        m = rng.random((h, w)) < rng.uniform(0.2, 0.95)
        corner = np.zeros_like(m)
        corner[28:36, 28:36] = m[28:36, 28:36]                  # all that happens round one corner of four tiles
        for mask in (m, corner):
            assert _components(mask) == label(mask, np.ones((3, 3)))[1]
