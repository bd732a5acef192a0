"""Where a tile's ring lines start, by each of the ways that find it: added up by the step kernel itself (at
most 2048 tiles and 1024 per wave), by the averaging-only kernel (at most 4096 tiles), by the one-launch pass (at
most 128 superblocks), by the two-launch pass.  Sizes on both sides of every line; mixed calls; index lists,
norms and diagnostics between the steps (they share the workspace); an overflowing slot; a resumed record."""
import numpy as np
import pytest
import torch
from test_gpu_parity import TOL_F32, EMPTY_P, both_layouts, compare, grads_for, make_pair, rel_err, run_average, run_steps

import synth_inputs as si
from oracle import oracle as O

pytestmark = pytest.mark.gpu

T = 256


@pytest.mark.parametrize("tiles,R", [(1, 1), (2, 3), (511, 4), (513, 8), (1024, 1), (1025, 1), (2047, 2), (2048, 2), (2049, 2), (2048, 5), (2049, 12)])
@both_layouts
def test_steps_around_the_lines(amlib, tiles, R, d_layout):
    run_steps(amlib, tiles * T - 3, R, 4, delay=1, fraction=0.15, seed=7, lookahead=True, gamma=0.9, check_every=2, d_layout=d_layout)


@pytest.mark.parametrize("tiles,R", [(1, 2), (5, 1), (4095, 2), (4096, 1), (4097, 2), (1027, 12)])
@pytest.mark.parametrize("tau", [0, 2])
def test_averages_around_the_lines(amlib, tiles, R, tau):
    run_average(amlib, tiles * T - 200, R, 4, delay=tau, fraction=0.1)


def test_one_launch_and_two_launch_passes(amlib):
    for sb in (127, 128, 129):                             # 131,072 coordinates each
        run_steps(amlib, (sb << 17) - 5, 1, 3, delay=1, fraction=0.02, seed=3, optimizer=O.OPT_SGD, beta1=0.0, check_every=3)


@pytest.mark.parametrize("n", [70_001, 700_001])           # 274 and 2735 tiles: in-kernel sums for both calls, for one
def test_mixed_calls_share_the_size_tables(amlib, n):
    """Steps and averaging-only calls in turn, an averaging interval of one and of two, with calls in between
    that use other parts of the workspace."""
    am = amlib
    for K in (1, 2):
        R = 3
        st, orc = make_pair(am, n, R, delay=2, avg_interval=K, fraction=0.1, seed=5)
        for t in range(1, 11):
            if t % 3 == 0:
                st.sparse_average(t, 0.5); orc.sparse_average(t, 0.5)
            else:
                g, gd = grads_for(n, R, t, 5, False)
                st.grad_sqnorm(gd)
                st.step(t, gd, 1e-3, 0.5); orc.step(t, g, 1e-3, 0.5)
            idx, k = st.subset_indices(t + 1)
            assert np.array_equal(idx.cpu().numpy().astype(np.uint64), O.subset(5, t + 1, n, 0.1))
            st.diagnostics()
        for i in range(R):
            for name in ("w", "m", "v", "d"):
                assert rel_err(getattr(st, name)[i].cpu().numpy(), getattr(orc, name)(i)) < TOL_F32, (K, i, name)
        assert st.read_flags() == 0


@pytest.mark.parametrize("steps", [3, 4])                   # either size table holds the pending sizes
@pytest.mark.parametrize("n", [70_001, 700_001])
def test_resumed_record_from_either_size_table(amlib, steps, n):
    am = amlib
    R, kw = 2, dict(delay=1, fraction=0.1, seed=8)
    st, orc = make_pair(am, n, R, **kw)
    for t in range(1, steps + 1):
        g, gd = grads_for(n, R, t, 8, False)
        st.step(t, gd, 1e-3, 0.5); orc.step(t, g, 1e-3, 0.5)
    torch.cuda.synchronize()
    st2 = am.Stage.resume(st.cfg, st.export_state(), *[[x.clone() for x in getattr(st, k)] for k in ("w", "m", "v", "d_storage")], None, st.workspace.clone())
    for t in range(steps + 1, steps + 4):
        g, gd = grads_for(n, R, t, 8, False)
        for s in (st, st2):
            s.step(t, gd, 1e-3, 0.5)
        orc.step(t, g, 1e-3, 0.5)
    compare(st2, orc, "resumed")
    for k in ("w", "m", "v", "d"):
        assert all(torch.equal(x, y) for x, y in zip(getattr(st, k), getattr(st2, k)))


@pytest.mark.parametrize("reserved", [0, 1, 1 << 31])
@pytest.mark.parametrize("steps", [3, 4])
@pytest.mark.parametrize("n", [70_001, 700_001])
def test_record_of_any_build(amlib, n, steps, reserved):
    """A record leaves `reserved` at zero and names sizes only where every build looks for them; records that
    hold something else there (bit 0 has named the second table) resume as well."""
    am = amlib
    R = 2
    st, _ = make_pair(am, n, R, delay=1, fraction=0.1, seed=8)
    for t in range(1, steps + 1):
        st.step(t, grads_for(n, R, t, 8, False)[1], 1e-3, 0.5)
    torch.cuda.synchronize()
    snap = st.export_state()
    assert snap.reserved == 0
    if reserved:
        snap.reserved, snap.next_lines_step = reserved, steps + 1
    st2 = am.Stage.resume(st.cfg, snap, *[[x.clone() for x in getattr(st, k)] for k in ("w", "m", "v", "d_storage")], None, st.workspace.clone())
    for t in range(steps + 1, steps + 4):
        for s in (st, st2):
            s.step(t, grads_for(n, R, t, 8, False)[1], 1e-3, 0.5)
    for k in ("w", "m", "v", "d"):
        assert all(torch.equal(x, y) for x, y in zip(getattr(st, k), getattr(st2, k)))


def test_overflow_found_by_the_step_itself(amlib):
    """A slot that is too small, found by the workgroups that add up the sizes: the flag is raised, tiles
    before the capacity follow the method."""
    am = amlib
    n, R, p, seed, cap = 60_003, 4, 0.2, 19, 300
    w0 = si.stage_weights(n, 1)
    kw = dict(delay=1, fraction=p, seed=seed, optimizer=O.OPT_SGD, beta1=0.0)
    st = am.init_state(am.make_config(n, R, ring_cap_lines=cap, **kw), torch.from_numpy(w0).cuda())
    full, never = O.Oracle(n, R, **kw), O.Oracle(n, R, **dict(kw, fraction=EMPTY_P))
    full.set_w(w0); never.set_w(w0)
    dropped = []
    for t in range(1, 6):
        g, gd = grads_for(n, R, t, seed, False)
        st.step(t, gd, 0.5, 0.5); full.step(t, g, 0.5, 0.5); never.step(t, g, 0.5, 0.5)
        counts = np.bincount((O.subset(seed, t, n, p) // T).astype(np.int64), minlength=-(-n // T))
        lines = -(-counts * 4 // 32)
        dropped.append(int(np.argmax(np.cumsum(lines) > cap)))
    lo, hi = min(dropped) * T, (max(dropped) + 1) * T
    for i in range(R):
        got = st.w[i].cpu().numpy()
        assert rel_err(got[:lo], full.w(i)[:lo]) < TOL_F32 and rel_err(got[hi:], never.w(i)[hi:]) < TOL_F32
    assert st.read_flags() & 1
