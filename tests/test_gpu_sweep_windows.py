"""The sweep's choices, from tile to tile, and its selection: spaces with radices
of one and ragged windows against predictions of every configuration (the same
operations, so the same values), ties to the lower index."""
import numpy as np
import pytest

from paper_2306_14011_amd import fv

pytestmark = pytest.mark.gpu


def space(radix, n_in, seed):
    rng = np.random.default_rng(seed)
    sp = fv.fv_tune_space()
    for s, r in enumerate(radix):
        sp.radix[s] = r
        for c in range(r):
            # few distinct values: many configurations tie
            sp.f1[s][c], sp.f2[s][c] = float(rng.integers(-2, 3)), float(rng.integers(-1, 2)) * 0.5
    sp.n_extra = n_in - 14
    for j in range(sp.n_extra):
        sp.extra[j] = 0.3 - 0.8 * j
    return sp


def rows(sp, radix, n_in, begin, count):
    rem = np.arange(begin, begin + count)
    X = np.zeros((count, n_in), dtype=np.float32)
    for s, r in enumerate(radix):
        d = rem % r
        rem = rem // r
        X[:, 2 * s] = np.array([sp.f1[s][c] for c in range(r)], dtype=np.float32)[d]
        X[:, 2 * s + 1] = np.array([sp.f2[s][c] for c in range(r)], dtype=np.float32)[d]
    for j in range(sp.n_extra):
        X[:, 14 + j] = sp.extra[j]
    return X


@pytest.mark.parametrize("n_in", [14, 16])
@pytest.mark.parametrize("radix", [(1, 1, 1, 1, 1, 1, 1), (1, 5, 3, 1, 7, 2, 11), (32, 3, 1, 9, 5, 4, 13)], ids=str)
def test_windows_of_a_space(radix, n_in):
    from paper_2306_14011_amd.autotune import Network
    N = Network(sum(radix) + n_in, n_in=n_in)
    sp = space(radix, n_in, 5)
    total = int(np.prod(radix))
    windows = {(0, total), (total - 1, 1), (max(total - 33, 0), min(33, total)), (min(17, total - 1), min(129, total - min(17, total - 1))),
               (total // 3, total - total // 3)}
    for begin, count in sorted(windows):
        out = N.predict(rows(sp, radix, n_in, begin, count))
        order = np.lexsort((np.arange(count), out))
        for k in (1, 3, 8):
            ti, tv = N.sweep(sp, begin, count, k)
            m = min(k, count)
            assert ti[:m] == [int(begin + i) for i in order[:m]], (begin, count, k)
            assert np.array_equal(np.asarray(tv[:m], dtype=np.float32), out[order[:m]])
