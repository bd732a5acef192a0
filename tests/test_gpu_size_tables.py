"""The tiles' sizes as bytes: the numbers of tiles at which a call adds them up itself (16 a lane, 1024 a wave and load, 4096 a
wave, 8192 for a step, 16384 for a call that only averages), the one-launch pass on both sides of its limit, and a
checkpoint record whose words an older build left."""
import numpy as np
import pytest
import torch
from test_gpu_parity import both_layouts, compare, grads_for, make_pair, run_average, run_steps

from oracle import oracle as O

pytestmark = pytest.mark.gpu

T = 256
OFF_RECORD_WORDS = 256 + 32 * 1024 * 8                      # of the workspace: after the flags and the reductions' partials


@pytest.mark.parametrize("tiles,R,tau", [(15, 1, 1), (16, 1, 1), (17, 2, 1), (1023, 1, 1), (1025, 1, 1), (2049, 2, 2), (4096, 1, 1), (4097, 1, 1),
                                         (4111, 2, 0), (8193, 2, 1), (12 * 1024 + 5, 3, 0), (4100, 20, 0)])
@both_layouts
def test_steps_around_the_loads(amlib, tiles, R, tau, d_layout):
    run_steps(amlib, tiles * T - 3, R, 4, delay=tau, fraction=0.15, seed=7, check_every=4, d_layout=d_layout)


@pytest.mark.parametrize("tiles,R", [(8192, 4), (8193, 4)])
def test_steps_around_the_limit(amlib, tiles, R):
    run_steps(amlib, tiles * T - 100, R, 4, delay=1, fraction=0.02, seed=3, optimizer=O.OPT_SGD, beta1=0.0, check_every=4)


@pytest.mark.parametrize("tiles,R,tau", [(6144, 4, 1), (6145, 3, 1), (2048, 20, 1), (2049, 17, 1), (768, 32, 1), (769, 25, 1), (1024, 12, 0), (1025, 9, 0)])
def test_steps_around_the_limits_by_blocks(amlib, tiles, R, tau):
    run_steps(amlib, tiles * T - 100, R, 4, delay=tau, fraction=0.05, seed=3, optimizer=O.OPT_SGD, beta1=0.0, check_every=4, d_layout=amlib.D_INTERLEAVED)


@pytest.mark.parametrize("tiles", [15, 17, 4097, 16383, 16384, 16385])
@pytest.mark.parametrize("tau", [0, 1])
def test_averages_around_the_loads(amlib, tiles, tau):
    run_average(amlib, tiles * T - 200, 1, 4, delay=tau, fraction=0.05)


def test_one_launch_pass_around_its_limit(amlib):
    for sb in (511, 512, 513):
        run_steps(amlib, (sb << 17) - 5, 1, 3, delay=1, fraction=0.01, seed=3, optimizer=O.OPT_SGD, beta1=0.0, check_every=3)


@pytest.mark.parametrize("n", [70_001, 700_001])
def test_record_that_names_words(amlib, n):
    """A record of a build that left the sizes as words: the resumed state uses them once, and says so again when it is exported
    before its first step; a record of this build names none."""
    am = amlib
    R, p, seed, steps = 2, 0.1, 8, 3
    st, orc = make_pair(am, n, R, delay=1, fraction=p, seed=seed)
    for t in range(1, steps + 1):
        g, gd = grads_for(n, R, t, seed, False)
        st.step(t, gd, 1e-3, 0.5); orc.step(t, g, 1e-3, 0.5)
    torch.cuda.synchronize()
    snap = st.export_state()
    assert snap.next_lines_step == 0
    ntiles = -(-n // T)
    counts = np.bincount((O.subset(seed, steps + 1, n, p) // T).astype(np.int64), minlength=ntiles)
    ws = st.workspace.clone()
    ws[OFF_RECORD_WORDS:OFF_RECORD_WORDS + 4 * ntiles] = torch.from_numpy((-(-counts * R // 32)).astype(np.int32).view(np.uint8)).cuda()
    snap.next_lines_step = steps + 1
    st2 = am.Stage.resume(st.cfg, snap, *[[x.clone() for x in getattr(st, k)] for k in ("w", "m", "v", "d_storage")], None, ws)
    assert st2.export_state().next_lines_step == steps + 1
    for t in range(steps + 1, steps + 4):
        g, gd = grads_for(n, R, t, seed, False)
        for s in (st, st2):
            s.step(t, gd, 1e-3, 0.5)
        orc.step(t, g, 1e-3, 0.5)
    assert st2.export_state().next_lines_step == 0
    compare(st2, orc, "resumed")
    for k in ("w", "m", "v", "d"):
        assert all(torch.equal(x, y) for x, y in zip(getattr(st, k), getattr(st2, k)))
