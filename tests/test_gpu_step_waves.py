"""Large stages of blocks of eight replicas through one-wave workgroups (a delay, at most 10 % of the coordinates; interleaved EMA vectors 6 % and an even number of at most 24
replicas, where not many slots are absent): from 3 * 2^22 weights on where many slots of a block are absent, from 5 * 2^23 with and 2^26 without a correction.  One and two replicas a wave, several blocks, absent
slots, ragged tiles, more received coordinates than a turn holds, every optimizer and type, rounds and steps between them, a slot that is too small, idle replicas."""
import numpy as np
import pytest
import torch
from test_gpu_parity import EMPTY_P, TOL_F32, _free_hbm, _full_size_case, compare, grads_for, make_pair, rel_err, run_steps

import synth_inputs as si
from oracle import oracle as O

pytestmark = pytest.mark.gpu

FEW, MANY = 3 << 22, 5 << 23
PER_REPLICA, INTERLEAVED = dict(d_layout=0), dict(d_layout=1)
LOOK = dict(lookahead=True, gamma=0.9)
NONE = dict(correction=O.CORR_NONE)
BF16 = dict(grad_bf16=True, fwd_bf16=True)


@pytest.mark.parametrize("n,R,p,kw", [
    (2_600_001, 5, 0.1, LOOK), (2_700_800, 5, 0.003, dict(NONE, **BF16)), (2_100_483, 9, 0.1, BF16), (2_098_177, 9, 0.05, dict(NONE, optimizer=O.OPT_NADAMW, beta1=0.99)),
    (2_098_690, 10, 0.1, dict(optimizer=O.OPT_SGD, beta1=0.9)), (2_097_411, 11, 0.02, dict(NONE, optimizer=O.OPT_SGD, beta1=0.0, **LOOK)),
    (MANY // 8 + 1, 8, 0.1, LOOK), (MANY // 12 + 2, 12, 0.05, dict(optimizer=O.OPT_SGD, beta1=0.0, grad_bf16=True)), (MANY // 32 + 3, 32, 0.1, dict(BF16, **LOOK)),
    ((1 << 26) // 8 + 7, 8, 0.05, dict(NONE, **LOOK)), ((1 << 26) // 16 + 5, 16, 0.01, dict(NONE, **BF16))])
def test_parity(amlib, n, R, p, kw):
    run_steps(amlib, n, R, 4, delay=2, fraction=p, seed=5, check_every=4, **PER_REPLICA, **kw)


@pytest.mark.parametrize("n,R,p,kw", [
    (2_600_001, 5, 0.1, LOOK), (2_100_483, 9, 0.1, BF16), (2_098_690, 10, 0.1, dict(optimizer=O.OPT_SGD, beta1=0.9)), (2_097_411, 11, 0.02, dict(optimizer=O.OPT_SGD, beta1=0.0, **LOOK)),
    (MANY // 8 + 1, 8, 0.06, LOOK), (MANY // 12 + 2, 12, 0.05, dict(optimizer=O.OPT_NADAMW, beta1=0.99, grad_bf16=True)), (MANY // 24 + 3, 24, 0.06, dict(BF16, **LOOK)),
    (MANY // 8 + 254, 8, 0.003, dict(correction=O.CORR_EAGER))])
def test_interleaved(amlib, n, R, p, kw):
    run_steps(amlib, n, R, 4, delay=2, fraction=p, seed=5, check_every=4, **INTERLEAVED, **kw)


@pytest.mark.parametrize("n,R,p,kw", [((1 << 26) // 24 + 3, 24, 0.05, dict(BF16, **LOOK)), (MANY // 18 + 5, 18, 0.06, {})])
def test_interleaved_three_blocks(amlib, n, R, p, kw):
    run_steps(amlib, n, R, 4, delay=2, fraction=p, seed=5, check_every=4, **INTERLEAVED, **kw)


@pytest.mark.parametrize("kw", [dict(avg_interval=2), dict(subset_granule=32), dict(subset_kind=O.SUBSET_STRATIFIED), dict(msg_dtype=O.MSG_E4M3)])
def test_options_interleaved(amlib, kw):
    run_steps(amlib, 2_098_433, 9, 4, delay=1, fraction=0.1, seed=7, check_every=4, **INTERLEAVED, **kw)


@pytest.mark.parametrize("kw", [dict(avg_interval=2), dict(subset_granule=32), dict(subset_kind=O.SUBSET_STRATIFIED), dict(correction=O.CORR_EAGER), dict(msg_dtype=O.MSG_E4M3)])
def test_options(amlib, kw):
    run_steps(amlib, 2_098_433, 9, 4, delay=1, fraction=0.1, seed=7, check_every=4, **PER_REPLICA, **kw)


@pytest.mark.parametrize("R,layout,kw", [(9, PER_REPLICA, {}), (10, PER_REPLICA, {}), (9, INTERLEAVED, {}), (10, INTERLEAVED, {}), (9, PER_REPLICA, NONE), (10, PER_REPLICA, NONE)])
def test_several_turns(amlib, R, layout, kw):
    """Whole lines of 32 coordinates are drawn, as many as a turn holds: a tile with two or more takes as many turns, each of which
    overwrites in LDS what the one before has read."""
    run_steps(amlib, 2_100_001, R, 4, delay=1, fraction=0.1, subset_granule=32, seed=11, check_every=2, **layout, **kw)


@pytest.mark.parametrize("n", [FEW // 5, FEW // 5 + 1])
def test_both_sides_of_the_line(amlib, n):
    run_steps(amlib, n, 5, 3, delay=1, fraction=0.05, seed=6, check_every=3, **PER_REPLICA)


def test_idle_replicas_and_factors(amlib):
    n, R = 2_600_003, 5
    st, orc = make_pair(amlib, n, R, delay=1, fraction=0.05, seed=3, **PER_REPLICA)
    scale = np.array([1.0, 0.5, 0.25, 2.0, 0.125], np.float32)                       # powers of two: the scaled gradients are exact
    for t in range(1, 4):
        g, gd = grads_for(n, R, t, 3, False)
        if t == 2:
            st.step_masked(t, gd, 1e-3, 0.5, 0b10110)
            orc.step_masked(t, g, 1e-3, 0.5, 0b10110)
        else:
            st.step_masked(t, gd, 1e-3, 0.5, 0b11111, 1.0, torch.from_numpy(scale).cuda())
            orc.step_masked(t, [x * f for x, f in zip(g, scale)], 1e-3, 0.5, 0b11111)
    compare(st, orc, "masked")
    for i in range(R):
        assert rel_err(st.m[i].cpu().numpy(), orc.m(i)) < TOL_F32


@pytest.mark.parametrize("layout,kw", [(PER_REPLICA, LOOK), (INTERLEAVED, LOOK), (PER_REPLICA, dict(NONE, optimizer=O.OPT_SGD, beta1=0.9))])
def test_idle_replicas_and_factors_of_a_pair(amlib, layout, kw):
    """Two replicas a wave: factors that differ inside a pair, one idle replica of a pair, the other one of the next."""
    n, R = 2_100_003, 10
    st, orc = make_pair(amlib, n, R, delay=1, fraction=0.05, seed=3, **layout, **kw)
    scale = np.array([1.0, 0.5, 0.25, 2.0, 0.125, 4.0, 0.5, 1.0, 2.0, 0.25], np.float32)      # powers of two: the scaled gradients are exact
    for t in range(1, 5):
        g, gd = grads_for(n, R, t, 3, False)
        mask = 0b10_0110_1101 if t % 2 == 0 else 0b11_1111_1111
        st.step_masked(t, gd, 1e-3, 0.5, mask, 1.0, torch.from_numpy(scale).cuda())
        orc.step_masked(t, [x * f for x, f in zip(g, scale)], 1e-3, 0.5, mask)
    compare(st, orc, "masked pairs")


@pytest.mark.parametrize("R,layout", [(10, PER_REPLICA), (10, INTERLEAVED), (9, PER_REPLICA), (9, INTERLEAVED)])
def test_a_slot_that_is_too_small(amlib, R, layout):
    """The tiles past the slot's capacity evolve as if never averaged, those before it follow the method, and the flag is raised."""
    n, p, seed, steps, cap, rb = 2_100_003, 0.1, 19, 4, 40_000, 8
    kw = dict(delay=1, seed=seed, **LOOK)
    w0 = si.stage_weights(n, seed)
    st = amlib.init_state(amlib.make_config(n, R, fraction=p, ring_cap_lines=cap, **layout, **kw), torch.from_numpy(w0).cuda())
    full, never = O.Oracle(n, R, fraction=p, **kw), O.Oracle(n, R, fraction=EMPTY_P, **kw)
    full.set_w(w0); never.set_w(w0)
    first_dropped = []
    for t in range(1, steps + 1):
        g, gd = grads_for(n, R, t, seed, False)
        st.step(t, gd, 1e-3, 0.5); full.step(t, g, 1e-3, 0.5); never.step(t, g, 1e-3, 0.5)
        counts = np.bincount((O.subset(seed, t, n, p) // 256).astype(np.int64), minlength=-(-n // 256))
        lines = -(-counts * rb // 32)
        start = np.cumsum(lines) - lines
        assert (start + lines > cap).any()
        first_dropped.append(int(np.argmax(start + lines > cap)))
    lo, hi = min(first_dropped) * 256, (max(first_dropped) + 1) * 256
    assert 0 < lo <= hi < n - 100_000
    for i in range(R):
        for name in ("w", "m", "v", "d", "fwd"):
            got = getattr(st, name)[i].cpu().numpy()
            assert rel_err(got[:lo], getattr(full, name)(i)[:lo]) < TOL_F32, (name, i, "kept tiles")
            assert rel_err(got[hi:], getattr(never, name)(i)[hi:]) < TOL_F32, (name, i, "dropped tiles")
    assert not np.any(st.d[0].cpu().numpy()[hi:]) and np.any(st.d[0].cpu().numpy()[:lo])
    assert st.read_flags() & 1


def test_more_chunks_than_one_dimension_of_a_grid_holds(amlib):
    """128 tiles a chunk, 65535 chunks and one tile: windows at both ends and about 2^30, where the grid's next layer begins."""
    n = 65_535 * 128 * 256 + 1
    if _free_hbm() < 160e9:
        pytest.skip("not enough free HBM")
    _full_size_case(amlib, n, 5, 1, 0.002, 3, [(0, 30_000), ((1 << 30) - 15_000, 30_000), (n - 30_001, 30_001)], lookahead=False, optimizer=O.OPT_SGD, beta1=0.0, **PER_REPLICA)


@pytest.mark.parametrize("n,R,layout", [(1_500_003, 9, PER_REPLICA), (1_500_003, 9, INTERLEAVED), (1_300_001, 10, INTERLEAVED), (1_200_002, 11, PER_REPLICA)])
def test_first_step_and_the_one_after_a_resume_of_a_smaller_stage(amlib, n, R, layout):
    """Up to 8192 tiles these two, whose subsets are not sized yet, go by waves and all others through the kernel that adds up the sizes itself: what
    one leaves in the ring, the slots of absent replicas with it, the other reads."""
    st, orc = make_pair(amlib, n, R, delay=2, fraction=0.05, seed=13, **layout, **LOOK)
    for t in range(1, 10):
        if t == 6:
            arrays = [[x.clone() for x in getattr(st, k)] for k in ("w", "m", "v", "d_storage", "fwd")]
            st = amlib.Stage.resume(st.cfg, st.export_state(), *arrays, st.workspace.clone())
        g, gd = grads_for(n, R, t, 13, False)
        st.step(t, gd, 1e-3, 0.5); orc.step(t, g, 1e-3, 0.5)
        if t in (1, 4, 6, 9):
            compare(st, orc, f"step {t}")
