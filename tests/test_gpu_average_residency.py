"""Beyond 2^26 weights the averaging-only call limits how many of its workgroups a compute unit holds, by the lines that a
wave reads: two, three, four and more of them, both layouts of the EMA vectors, absent replicas, several turns a tile."""
import pytest
from test_gpu_parity import both_layouts, run_average

pytestmark = pytest.mark.gpu

N = (1 << 26) // 8


@pytest.mark.parametrize("n,R,p", [(N, 8, 0.05), (N + 1, 8, 0.05), (N + 1, 8, 0.3), (2 * N + 3, 4, 0.02), (N // 2 + 77, 21, 0.05)])
@both_layouts
def test_residency_lines(amlib, n, R, p, d_layout):
    run_average(amlib, n, R, 2, delay=1, fraction=p, d_layout=d_layout)
