"""The averaging-only kernel where what a tile receives fills the kilobyte it stages: just below and above,
several turns of it, tiles whose members come in whole lines, both sides of the rule that picks the
unstaged form for per-replica EMA vectors, and more than one block of replicas.  Against the oracle, fp32 bar."""
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
