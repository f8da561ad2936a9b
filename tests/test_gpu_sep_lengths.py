"""Separable filter: every window length on the forms that large frames run, on rows of whole 16-byte vectors and others,
against the oracle.  (test_sepfilter_every_window_length has the form of small frames.)
Tolerance: 2k fp32 multiply-adds of at most |kx| |ky| max|x|."""
import numpy as np
import pytest
import torch

import oracle
from paper_1911_03458_amd import binding as mb


def _plan(N, W, k, rows=0):
    plan = mb.merit_plan_sepfilter(N, 65, W, k)
    return plan.set_tile((0, rows)) if rows else plan


def _check(plan, W, k, N):
    rng = np.random.default_rng(100 * W + k)
    x = rng.uniform(0, 255, (N, 65, W)).astype(np.float32)
    kx, ky = (rng.standard_normal(k).astype(np.float32) for _ in range(2))
    y = mb.merit_sepfilter(plan, *(torch.from_numpy(a).cuda() for a in (x, kx, ky))).cpu().numpy()
    ref = oracle.sepfilter(x, kx, ky).astype(np.float64)
    assert np.all(np.abs(y - ref) <= 1e-5 * np.abs(kx).sum() * np.abs(ky).sum() * x.max())


@pytest.mark.parametrize("W", [1030, 1032])
def test_the_forms(W):
    for k in range(1, 33):
        if k <= 28:      # one tile a workgroup of 256 threads, and (17 taps and more) 96 staged rows on request
            li = _plan(27, W, k).launch_info()
            assert li["block"][0] == 256 and li["tile"][1] == (65 - k) // 4 * 4 and li["grid"][0] == 27 * 2 * 17, (k, li)
        if k >= 17:      # more tiles than the workgroups that walk them
            li = _plan(70, W, k, 96).launch_info()
            assert li["block"][0] == 256 and li["tile"][1] == (97 - k) // 4 * 4 and li["grid"][0] == 1024, (k, li)
            assert 70 * -(-65 // li["tile"][1]) * 17 > 1024
    assert _plan(70, W, 30).launch_info() == _plan(70, W, 30, 96).launch_info()


@pytest.mark.gpu
@pytest.mark.parametrize("W", [1030, 1032])
@pytest.mark.parametrize("k", range(1, 29))
def test_one_tile_a_workgroup(k, W):
    _check(_plan(27, W, k), W, k, 27)


@pytest.mark.gpu
@pytest.mark.parametrize("W", [1030, 1032])
@pytest.mark.parametrize("k", range(17, 33))
def test_workgroups_that_walk_the_tiles(k, W):
    _check(_plan(70, W, k, 96), W, k, 70)
