"""GPU: the distance transform's form for tiles of few candidates, around the
number of rows or planes with a site up to which it is taken (7/16 of the
line's length, 88 at most), against the definition; and the nearest site
itself where several are equally near: of the candidates along a line the last
one, whichever form finds it."""
import numpy as np
import pytest

from oracle import edt as O
from tests.test_gpu_edt import _check, _run

pytestmark = pytest.mark.gpu


def _limit(n):
    return min(n * 7 // 16, 88)


def _lines(n, count, rng):
    """count of n positions, the ends among them where count allows."""
    ends = [0, n - 1][:count]
    rest = rng.permutation(np.arange(1, n - 1))[:max(count - len(ends), 0)]
    return np.sort(np.concatenate([ends, rest]).astype(int))


@pytest.mark.parametrize("n", [3, 16, 17, 64, 129, 256, 257, 513, 1023])
@pytest.mark.parametrize("axis", [1, 0])
@pytest.mark.parametrize("over", [-1, 0, 1])
def test_around_the_limit(n, axis, over):
    rng = np.random.default_rng(n * 10 + axis * 3 + over)
    count = min(max(_limit(n) + over, 0), n)
    shape = (2, n, 37) if axis == 1 else (n, 2, 37)
    m = np.zeros(shape, np.uint8)
    for p in _lines(n, count, rng):
        x = rng.integers(0, 37, rng.integers(1, 3))
        if axis == 1:
            m[0, p, x] = 1   # the other plane stays empty
        else:
            m[p, rng.integers(0, 2), x] = 1
    near, dist = _run(m)
    _check(m, near, dist, O.d2_grid(m).reshape(-1), 0.02)


@pytest.mark.parametrize("n", [40, 256])
@pytest.mark.parametrize("step", [2, 6])   # half the rows: by search; a sixth: few candidates
def test_the_last_of_equals(n, step):
    m = np.zeros((1, n, 5), np.uint8)
    m[0, ::step, 2] = 1
    near, _ = _run(m)
    y = np.arange(n)
    rows = np.arange(0, n, step)
    d = np.abs(y[:, None] - rows[None, :])
    last = rows[len(rows) - 1 - np.argmin(d[:, ::-1], 1)]
    for x in range(5):
        np.testing.assert_array_equal(near[0, :, x], 2 | (last << 10))
