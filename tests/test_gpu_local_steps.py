"""Steps between two averaging rounds: a kernel of their own for blocks of eight replicas beyond 2^20 parameters x replicas with a round every
fourth step or more seldom, beyond 2.5 or 6 times 2^20 with one every second or third.  Every optimizer, forward copy and gradient type, sizes at the edges of a tile and of
four, absent replicas and several blocks, idle replicas, gradient factors, and both sides of the line from where the resident
workgroups are limited."""
import numpy as np
import pytest
import torch
from test_gpu_parity import TOL_F32, compare, grads_for, make_pair, rel_err, run_steps

from oracle import oracle as O

pytestmark = pytest.mark.gpu

SGD = dict(optimizer=O.OPT_SGD, beta1=0.9)
PLAIN = dict(optimizer=O.OPT_SGD, beta1=0.0)


@pytest.mark.parametrize("n,R", [(257, 3), (1025, 8), (131_072, 8), (131_073, 8), (210_175, 5), (90_881, 12), (40_193, 32)])
@pytest.mark.parametrize("kw", [dict(lookahead=True, gamma=0.9), dict(optimizer=O.OPT_NADAMW, beta1=0.99), SGD, PLAIN,
                                dict(grad_bf16=True, fwd_bf16=True), dict(SGD, grad_bf16=True, lookahead=True, gamma=0.5)])
@pytest.mark.parametrize("K", [3, 4])
def test_between_rounds(amlib, n, R, kw, K):
    run_steps(amlib, n, R, 2 * K + 1, delay=1, avg_interval=K, fraction=0.2, seed=9, check_every=2 * K + 1, **kw)


@pytest.mark.parametrize("n,R,K", [((6 << 20) // 8, 8, 2), ((6 << 20) // 8 + 1, 8, 2), ((5 << 19) // 5, 5, 3), ((5 << 19) // 5 + 1, 5, 3)])
def test_frequent_rounds_on_both_sides_of_the_line(amlib, n, R, K):
    run_steps(amlib, n, R, 2 * K + 1, delay=1, avg_interval=K, fraction=0.2, seed=9, check_every=2 * K + 1, grad_bf16=True)


@pytest.mark.parametrize("n,R", [((5 << 20) // 8, 8), ((5 << 20) // 8 + 1, 8), (900_001, 6)])
@pytest.mark.parametrize("kw", [dict(lookahead=True, gamma=0.9), SGD, PLAIN])
def test_residency(amlib, n, R, kw):
    run_steps(amlib, n, R, 4, delay=0, avg_interval=4, fraction=0.05, seed=2, check_every=4, **kw)


def test_idle_replicas_and_factors(amlib):
    n, R = 250_003, 5
    st, orc = make_pair(amlib, n, R, delay=1, avg_interval=4, fraction=0.2, seed=3)
    for t in range(1, 9):
        g, gd = grads_for(n, R, t, 3, False)
        active = 0b10110 if t % 2 else 0b11111
        st.step_masked(t, gd, 1e-3, 0.5, active)
        orc.step_masked(t, g, 1e-3, 0.5, active)
    compare(st, orc, "masked")
    st, orc = make_pair(amlib, n, R, delay=1, avg_interval=4, fraction=0.2, seed=3)
    scale = np.array([1.0, 0.5, 0.25, 2.0, 0.125], np.float32)                       # powers of two: the scaled gradients are exact
    for t in range(1, 7):
        g, gd = grads_for(n, R, t, 3, False)
        st.step_scaled(t, gd, 1e-3, 0.5, 1.0, torch.from_numpy(scale).cuda())
        orc.step(t, [x * f for x, f in zip(g, scale)], 1e-3, 0.5)
    for i in range(R):
        for name in ("w", "m", "v"):
            assert rel_err(getattr(st, name)[i].cpu().numpy(), getattr(orc, name)(i)) < TOL_F32
