"""The fused step without delay: a wave per replica up to 16 replicas, the walking form beyond.  Blocks of
every size, absent replicas, a ragged last tile, an EMA vector that is not zero (the delay was lowered to
nothing at run time), quantised messages and a slot that is too small; against the oracle, fp32 bar."""
import numpy as np
import pytest
import torch
from test_gpu_parity import EMPTY_P, TOL_F32, both_layouts, compare, grads_for, make_pair, rel_err, run_steps

import synth_inputs as si
from oracle import oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R", [1, 2, 3, 4, 7, 8, 9, 15, 16, 17])
@both_layouts
def test_every_number_of_replicas(amlib, R, d_layout):
    run_steps(amlib, 6 * 256 + 130, R, 3, delay=0, fraction=0.3, seed=R, lookahead=True, gamma=0.9, d_layout=d_layout)


@pytest.mark.parametrize("kw", [dict(fraction=1.0), dict(fraction=EMPTY_P), dict(fraction=0.2, correction=O.CORR_NONE, optimizer=O.OPT_SGD, beta1=0.0),
                                dict(fraction=0.2, msg_dtype=O.MSG_E4M3), dict(fraction=0.2, avg_interval=2, optimizer=O.OPT_SGD, beta1=0.9)])
@both_layouts
def test_options(amlib, kw, d_layout):
    run_steps(amlib, 30_011, 11, 4, delay=0, seed=2, d_layout=d_layout, **kw)


@pytest.mark.parametrize("R", [4, 12])
@both_layouts
def test_delay_lowered_to_nothing(amlib, R, d_layout):
    st, orc = make_pair(amlib, 20_003, R, delay=2, fraction=0.3, seed=6, d_layout=d_layout)
    for t in range(1, 10):
        if t == 5:
            st.set_delay(0); orc.set_delay(0)
        g, gd = grads_for(20_003, R, t, 6, False)
        st.step(t, gd, 1e-2, 0.25); orc.step(t, g, 1e-2, 0.25)
        compare(st, orc, f"t={t}")
    assert float(st.d[0].abs().max()) > 0


@pytest.mark.parametrize("n", [60_003, 600_003])           # the step adds up the sizes itself / after an offsets pass
@both_layouts
def test_overflow(amlib, n, d_layout):
    am = amlib
    R, p, seed, cap = 4, 0.2, 19, n // 200
    w0 = np.stack([si.stage_weights(n, 100 + i) for i in range(R)])
    kw = dict(delay=0, fraction=p, seed=seed, optimizer=O.OPT_SGD, beta1=0.0)
    st = am.init_state(am.make_config(n, R, ring_cap_lines=cap, d_layout=d_layout, **kw), torch.from_numpy(w0).cuda())
    full, never = O.Oracle(n, R, **kw), O.Oracle(n, R, **dict(kw, fraction=EMPTY_P))
    full.set_w(w0); never.set_w(w0)
    dropped = []
    for t in range(1, 4):
        g, gd = grads_for(n, R, t, seed, False)
        st.step(t, gd, 0.5, 0.5); full.step(t, g, 0.5, 0.5); never.step(t, g, 0.5, 0.5)
        counts = np.bincount((O.subset(seed, t, n, p) // 256).astype(np.int64), minlength=-(-n // 256))
        dropped.append(int(np.argmax(np.cumsum(-(-counts * 4 // 32)) > cap)))
    lo, hi = min(dropped) * 256, (max(dropped) + 1) * 256
    assert 0 < lo <= hi < n
    for i in range(R):
        got = st.w[i].cpu().numpy()
        assert rel_err(got[:lo], full.w(i)[:lo]) < TOL_F32 and rel_err(got[hi:], never.w(i)[hi:]) < TOL_F32
    assert st.read_flags() & 1
