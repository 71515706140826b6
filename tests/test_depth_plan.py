"""CPU checks of the sample sort's sizes (csrc/depth_plan.h): the regions hold
their buckets over every scene size that takes the sort.

A bucket runs from one splitter to the next, a fixed number of samples on; it
overflows its region when fewer samples than that lie among ``cap`` Gaussians
in depth order.  For depths that know nothing of the order of the scene, all
visible, their number is Poisson with mean cap / stride.
"""
import math

import numpy as np
import pytest

from tests.parity_util import depth_buckets, depth_plans, depth_samples

TOP = 1 << 23


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    return lambda pairs: depth_plans(d, pairs)


def _sizes():
    edges = [e + d for e in (256 * 6144, 512 * 6144, 1024 * 6144, 1 << 20, 1 << 22) for d in (-1, 0, 1)]
    spread = np.unique(np.exp(np.linspace(0.0, math.log(TOP - 1), 400)).astype(int)).tolist()
    return sorted(set(spread + edges + [1, 2, 15, 16, 17, 4096, 4097, TOP - 1]))


def test_regions_hold_their_buckets(plan):
    worst = 0.0
    for n, (ok, stride, ns, nb, log_nb, cap) in zip(_sizes(), plan([(n, 1) for n in _sizes()])):
        assert ok and stride >= 1 and ns == -(-n // stride) <= 16384 and cap <= 16384, n
        assert (1 << log_nb) >= nb >= 1 and nb <= 2048, n
        per = ns // nb                       # samples of a bucket, at least
        lam = cap / stride
        if n > cap:                          # else one bucket's region holds the scene
            few = sum(math.exp(-lam + k * math.log(lam) - math.lgamma(k + 1)) for k in range(per))
            worst = max(worst, nb * few)
            assert nb * few < 1e-3, (n, nb * few)
            assert cap * nb >= 2.6 * n, n
    print(f"largest chance of an overflow in a frame {worst:.1e}")


def test_sizes_that_take_other_sorts(plan):
    got = plan([(0, 1), (TOP, 1), (TOP - 1, 1 << 17), (TOP - 1, (1 << 17) + 1), (TOP - 1, 1 << 20)])
    assert [g[0] for g in got] == [0, 0, 1, 0, 0]


@pytest.mark.parametrize("n", [1024 * 6144, 8_000_000, TOP - 1])
def test_random_depths_fill_no_region(plan, n):
    """The buckets of scenes of random depths, all visible: places of the
    sampled Gaussians in depth order, and the splitters among them."""
    (p,) = plan([(n, 1)])
    _, stride, ns, _, _, cap = p
    assert np.array_equal(depth_samples(n, stride, ns) // stride, np.arange(ns))   # one per stratum
    for seed in range(4):
        fill = np.diff(depth_buckets(p, np.random.default_rng(seed).permutation(n), n))
        assert fill.max() <= cap, (n, seed, int(fill.max()))
