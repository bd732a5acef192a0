"""The averaging-only kernel where what a tile receives fills the kilobyte it stages: just below and above,
several turns of it (large stages only: smaller ones read in place), tiles whose members come in whole lines, both
sides of the rule that picks the unstaged form, and more than one block of replicas.  Against the oracle, fp32 bar."""
import pytest
from test_gpu_parity import both_layouts, run_average

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,p", [(8, 0.0625), (8, 0.0626), (8, 0.12), (8, 0.13), (4, 0.125), (4, 0.24), (4, 0.26), (2, 0.25), (2, 0.49),
                                 (2, 0.51), (1, 0.5), (1, 0.99), (1, 1.0), (12, 0.06), (12, 0.3), (20, 0.0625), (8, 1.0)])
@both_layouts
def test_staged_kilobyte(amlib, R, p, d_layout):
    run_average(amlib, 5 * 256 * 4 + 77, R, 5, delay=2, fraction=p, d_layout=d_layout)


@pytest.mark.parametrize("R", [1, 2, 4, 8, 11])
@both_layouts
def test_members_in_whole_lines(amlib, R, d_layout):
    """Blocks of 32 coordinates drawn as a whole: most tiles receive nothing, some several turns' worth."""
    run_average(amlib, 40_003, R, 6, delay=1, fraction=0.06, subset_granule=32, d_layout=d_layout)


@pytest.mark.parametrize("n,R,kw", [(3_200_003, 8, dict(fraction=0.3)), (3_100_000, 8, dict(fraction=0.3)),       # several turns / read in place
                                    (800_001, 5, dict(fraction=1.0)), (500_001, 12, dict(fraction=1.0)),           # eight turns
                                    (3_200_003, 4, dict(fraction=0.7)), (3_200_003, 2, dict(fraction=0.6)), (3_200_003, 1, dict(fraction=1.0))])
def test_turns_on_both_sides_of_the_line(amlib, n, R, kw):
    run_average(amlib, n, R, 4, delay=1, d_layout=amlib.D_INTERLEAVED, **kw)


@pytest.mark.parametrize("n,R,p,granule", [(1_600_003, 11, 0.12, 1), (1_600_003, 11, 0.2, 1), (30_003, 8, 0.3, 1), (30_003, 4, 0.2, 32),
                                           (30_003, 4, 0.8, 32), (30_003, 12, 0.05, 32)])
def test_quantised_messages_in_both_forms(amlib, n, R, p, granule):
    run_average(amlib, n, R, 4, delay=1, fraction=p, subset_granule=granule, msg_dtype=amlib.MSG_E4M3, d_layout=amlib.D_INTERLEAVED)


@pytest.mark.parametrize("n", [24576 * 256, 24576 * 256 + 1])
@pytest.mark.parametrize("R,kw", [(3, dict(fraction=1.0)), (4, dict(fraction=0.5, correction=0)), (1, dict(fraction=0.7))])
def test_per_replica_turns_of_a_large_stage(amlib, n, R, kw):
    """Up to four replicas take several turns beyond 24576 tiles and read in place up to there."""
    run_average(amlib, n, R, 3, delay=1, d_layout=amlib.D_PER_REPLICA, **kw)


@pytest.mark.parametrize("n,R,p", [(30_003, 12, 0.1), (30_003, 12, 0.14), (30_003, 20, 0.12)])
def test_several_blocks_of_a_small_stage(amlib, n, R, p):
    for msg in (amlib.MSG_F32, amlib.MSG_BF16):
        run_average(amlib, n, R, 4, delay=1, fraction=p, msg_dtype=msg, d_layout=amlib.D_INTERLEAVED)


@pytest.mark.parametrize("n,R,p,kw", [(662_500, 8, 0.5, {}), (662_501, 8, 0.5, {}), (30_003, 8, 0.25, {}), (218_751, 12, 0.3, {}), (300_000, 12, 0.9, dict(msg_dtype=2)), (30_003, 20, 0.35, {}), (110_000, 32, 0.5, {}),
                                      (500_000, 4, 0.45, {}), (750_001, 3, 0.5, {}), (700_000, 8, 0.1, dict(subset_granule=32)), (300_000, 12, 0.6, dict(subset_granule=32, msg_dtype=1)), (850_001, 5, 0.5, {}),
                                      (1_060_000, 8, 0.2, dict(subset_granule=32)), (1_050_001, 4, 0.5, dict(correction=0)), (375_001, 9, 0.3, dict(subset_kind=1)), (1_375_000, 8, 1.0, dict(correction=0)), (1_375_001, 8, 1.0, dict(correction=0)),
                                      (230_000, 20, 0.5, dict(correction=0)), (1_063_000, 7, 0.1, dict(correction=0, subset_granule=32))])
@both_layouts
def test_forms_around_the_lines(amlib, n, R, p, kw, d_layout):
    """Several turns of blocks of four and eight on both sides of where the caches hold the stage, whose values change hands through LDS."""
    run_average(amlib, n, R, 3, delay=1, fraction=p, d_layout=d_layout, **kw)


@pytest.mark.parametrize("n,R", [((5 << 20) // 8, 8), ((5 << 20) // 8 + 1, 8), ((5 << 20) // 11, 11), ((5 << 20) // 11 + 1, 11), ((5 << 20) // 4 + 3, 3), ((23 << 19) // 8, 8), ((23 << 19) // 8 + 1, 8), ((20 << 20) // 5 + 1, 5)])
@pytest.mark.parametrize("tau,p", [(0, 0.05), (1, 0.05), (1, 0.9)])
def test_where_the_weights_are_named(amlib, n, R, tau, p):
    """Both sides of the lines between which, for blocks of eight, the kernel takes the weights' pointers from the replicas' records."""
    run_average(amlib, n, R, 3, delay=tau, fraction=p, d_layout=amlib.D_INTERLEAVED)
