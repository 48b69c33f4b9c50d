"""Set-up on the GPU against the oracle: candidate and 2-opt lists and the
nearest-neighbour tour, at the sizes and on the matrices where their kernels
change their way."""
import numpy as np
import pytest

from paper_2003_11902_amd import instances as I
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def check(d, cl, ls_nn, pher="dense"):
    from oracle import oracle as O
    from paper_2003_11902_amd import mmas as M
    n = d.shape[0]
    g = M.Colony(d, 2, cand_len=cl, ls_nn=ls_nn, pher=pher)
    if cl:
        assert np.array_equal(g.cand(), O.nearest(d, min(cl, n - 1)))
    if ls_nn:
        assert np.array_equal(g.read(M.MMAS_BUF_LSNN).reshape(n, -1), O.nearest(d, ls_nn))
    t, length = O.nn_tour(d)
    assert np.array_equal(g.read(M.MMAS_BUF_NN_TOUR), t)
    assert g.state().nn_len == length


@pytest.mark.parametrize("n", [3, 4, 63, 64, 65, 66, 128, 129, 257, 1023, 1024, 2049, 5001])
@pytest.mark.parametrize("cl,ls_nn", [(0, 1), (1, 2), (32, 8), (64, 32)])
def test_lists_and_tour(gpu, n, cl, ls_nn):
    _, d = I.make_instance("clustered" if n % 2 else "uniform", n, seed=n)
    say(f"set-up n={n} cl={cl} ls_nn={ls_nn}")
    check(d, cl, min(ls_nn, n - 1))


@pytest.mark.parametrize("n", [1025, 1088, 2048, 2049, 4032, 4096, 4097])
def test_lists_at_register_limits(gpu, n):
    """Rows that fill a wave's registers, one city less than a piece of 64 or
    one more than fits."""
    _, d = I.make_instance("uniform", n, seed=n, side=1e6)
    say(f"register limits n={n}")
    check(d, 16, 8, pher="candidates")


@pytest.mark.parametrize("n", [300, 1500])
def test_equal_distances(gpu, n):
    """Runs of equal distances: more entries up to the k-th smallest than are
    sorted at once, and every tie to the lowest index."""
    rng = np.random.default_rng(n)
    for top in (1, 2, 40):
        d = rng.integers(1, top + 1, (n, n)).astype(np.int32)
        d = np.triu(d, 1)
        d = d + d.T
        say(f"equal distances n={n} up to {top}")
        check(d, 32, 8)
        check(d, 64, 0, pher="candidates")


@pytest.mark.parametrize("n", [1024, 1025, 2049, 4097])
def test_bounds_among_equal_distances(gpu, n):
    """Runs of equal distances with rows in registers and read again: a run at
    the k-th smallest with entries before it, distances far apart, and runs
    short enough to be sorted whole."""
    rng = np.random.default_rng(n)
    for values, p in (([5, 2000000000], None), ([1, 2, 3000, 2147483647], [0.004, 0.004, 0.5, 0.492]),
                      (np.arange(1, 2 + n // 290) * 123457, None)):
        d = rng.choice(np.asarray(values, np.int32), (n, n), p=p)
        d = np.triu(d, 1)
        d = d + d.T
        say(f"bounds among equal distances n={n} {len(values)} values")
        check(d, 16, 0, pher="candidates")
        check(d, 64, 32, pher="candidates")


def test_refused_matrices_stay_refused(gpu):
    """Matrices with negative or zero distances are refused (and leave the
    lists of later set-up steps in bounds)."""
    from paper_2003_11902_amd import mmas as M
    _, d = I.make_instance("uniform", 90, seed=5)
    for value in (-1, 0, -7):
        bad = d.copy()
        bad[3, :] = value
        bad[:, 3] = value
        bad[3, 3] = 0
        say(f"refused: distances {value}")
        for cl, pher in ((32, "dense"), (64, "candidates")):
            with pytest.raises(M.MmasError) as e:
                M.Colony(bad, 4, cand_len=cl, ls_nn=8, pher=pher)
            assert e.value.status == M.MMAS_EINVAL
