"""The local step over the range of fp32 gradients (second moments from denormal to 1e30, zeros between them), the write-back of
d by halves of a line, and sizes on both sides of the line from where the stores go through to memory and the resident workgroups are
limited (5 * 2^20 parameters x replicas)."""
import numpy as np
import pytest
import torch
from test_gpu_parity import TOL_F32, both_layouts, compare, make_pair, rel_err, run_steps

from oracle import oracle as O

pytestmark = pytest.mark.gpu

LINE = 5 << 20


@pytest.mark.parametrize("opt", [O.OPT_ADAMW, O.OPT_NADAMW])
def test_gradients_of_any_size(amlib, opt):
    n, R = 4099, 2
    rng = np.random.default_rng(3)
    st, orc = make_pair(amlib, n, R, delay=1, fraction=0.2, seed=4, optimizer=opt, lookahead=True, gamma=0.9)
    for t in range(1, 5):
        g = [(np.exp(rng.uniform(np.log(1e-24), np.log(1e15), n)) * rng.choice([-1, 0, 1], n)).astype(np.float32) for _ in range(R)]
        st.step(t, [torch.from_numpy(x).cuda() for x in g], 1e-3, 0.5)
        orc.step(t, g, 1e-3, 0.5)
        for i in range(R):
            # moments span forty decades: each against its own size (one rounding to fp32 a step, denormals to their own spacing)
            for name in ("m", "v"):
                got, ref = getattr(st, name)[i].cpu().numpy().astype(np.float64), getattr(orc, name)(i).astype(np.float64)
                assert np.all(np.abs(got - ref) <= 5e-7 * np.abs(ref) + 3e-45), (t, i, name)
            assert rel_err(st.w[i].cpu().numpy(), orc.w(i)) < TOL_F32 and rel_err(st.fwd[i].cpu().numpy(), orc.fwd(i)) < TOL_F32, (t, i)


@pytest.mark.parametrize("R", [1, 2, 3, 4, 5, 8, 12])
@pytest.mark.parametrize("tau,p", [(1, 0.02), (1, 0.3), (0, 0.02), (0, 0.3)])
@both_layouts
def test_halves_of_a_line(amlib, R, tau, p, d_layout):
    run_steps(amlib, 10_007, R, 5, delay=tau, fraction=p, seed=13, d_layout=d_layout)


@pytest.mark.parametrize("R", [1, 2, 4, 8])
@pytest.mark.parametrize("bf16", [False, True])
def test_both_sides_of_the_caches(amlib, R, bf16):
    for n in (LINE // R, LINE // R + 5):
        run_steps(amlib, n, R, 3, delay=1, fraction=0.05, seed=6, d_layout=amlib.D_INTERLEAVED, grad_bf16=bf16, fwd_bf16=bf16, check_every=3)
