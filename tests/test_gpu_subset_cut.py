"""Whole strips go through a form of the generator that keeps the wave's common words scalar, and the list's cut changes at
eight strips a wave (20 waves a compute unit): seeds and steps whose every word has high bits, a threshold of 1 and
of 2^32, sizes on both sides of the line.  Whole numbers: equal to the oracle's list."""
import numpy as np
import pytest
import torch

from oracle import oracle as O

pytestmark = pytest.mark.gpu

CUT = 8 * 20 * 256 * 2048                                  # coordinates of eight strips a wave on 256 compute units


@pytest.mark.parametrize("n,p,seed,t", [
    (100_003, 1.0, 0xFFFFFFFF_FFFFFFFF, (1 << 63) + 5), (100_003, 0.31, 0x80000001_FFFFFFFE, 0xFFFFFFFF_FFFFFFFF),
    (700_001, 2.0**-32, 0xDEADBEEF, 3), (700_001, 0.02, 1 << 32, 1 << 32),
    (CUT - 1, 0.001, 5, 2), (CUT + 1, 0.001, 5, 2),
])
def test_strips_by_the_scalar_form(amlib, n, p, seed, t):
    am = amlib
    st = am.init_state(am.make_config(n, 1, fraction=p, seed=seed, optimizer=am.OPT_SGD, beta1=0.0, correction=am.CORR_NONE), torch.zeros(n))
    idx, k = st.subset_indices(t, capacity=min(n, int(n * p * 1.1) + 10_000))
    want = O.subset(seed, t, n, p)
    assert k == want.size and np.array_equal(idx.cpu().numpy().astype(np.uint64), want)


@pytest.mark.parametrize("n,p,kw", [(2 * 20 * 256 * 2048 + d, p, kw) for d in (0, 1) for p, kw in
                                    [(0.01, dict(granule=32)), (0.01, dict(stratified=True)), (0.25, dict())]])
def test_cuts_of_the_other_draws(amlib, n, p, kw):
    """Both sides of two strips a wave, from where whole lines and stratified subsets are cut for more waves."""
    am = amlib
    cfg = am.make_config(n, 1, fraction=p, seed=5, optimizer=am.OPT_SGD, beta1=0.0, correction=am.CORR_NONE, subset_granule=kw.get("granule", 1), subset_kind=int("stratified" in kw))
    idx, k = am.init_state(cfg, torch.zeros(n)).subset_indices(2, capacity=min(n, int(n * p * 1.1) + 10_000))
    want = O.subset(5, 2, n, p, **kw)
    assert k == want.size and np.array_equal(idx.cpu().numpy().astype(np.uint64), want)
