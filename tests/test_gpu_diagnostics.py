"""Consensus error and EMA variance where the reduction's cut can go wrong: around one pass of the grid
(2048 workgroups of 256 threads, 4096 on large interleaved stages of 5 to 16 replicas, with U groups of four coordinates each, U = 4, 2, 1 by the number of
replicas) and at ragged ends, for both layouts.  Reference: the same sums in fp64.  Sums of fewer than
2^26 non-negative fp64 terms differ by at most 2^26 * 2^-53 < 1e-8 between two orders; block-wise sums by far less."""
import pytest
import torch

pytestmark = pytest.mark.gpu

PASS = 2048 * 256 * 4


def check(am, n, R, interleaved):
    st = am.init_state(am.make_config(n, R, delay=0, fraction=0.5, seed=1, optimizer=am.OPT_SGD, beta1=0.0,
                                      d_layout=am.D_INTERLEAVED if interleaved else am.D_PER_REPLICA))
    g = torch.Generator(device="cuda").manual_seed(n + R)
    for i in range(R):
        st.w[i].copy_(torch.randn(n, generator=g, device="cuda"))
        st.d[i].copy_(torch.randn(n, generator=g, device="cuda"))

    def squares(xs):
        mean = sum(x.double() for x in xs) / R
        return sum((x.double() - mean) ** 2 for x in xs)

    cons, vmean, vmax = st.diagnostics()
    want_c, want_v = squares(st.w), squares(st.d) / R
    for got, want in ((cons, want_c.sum()), (vmean, want_v.mean()), (vmax, want_v.max())):
        want = float(want)
        assert abs(got - want) <= 1e-10 * want, (got, want)
    assert st.diagnostics() == (cons, vmean, vmax)


@pytest.mark.parametrize("n,R", [(4 * PASS + 3, 1), (4 * PASS - 1, 2), (4 * PASS + 257, 2), (2 * PASS + 1, 3), (2 * PASS + 2049, 4),
                                 (PASS + 1, 8), (PASS // 2 + 63, 5), (PASS // 4 + 5, 12), (1025, 32), (2, 7),
                                 # ends of a grid that loads whole waves (768 workgroups up to 16 replicas, 256 beyond) and of 256 partials
                                 (768 * 1024, 9), (768 * 1024 + 1, 16), (384 * 1024, 16), (384 * 1024 + 1, 12), (256 * 1024, 17), (256 * 1024 + 1, 32),
                                 (128 * 1024, 32), (128 * 1024 + 3, 20), (256 * 1024, 2), (256 * 1024 + 1, 2), (131, 16)])
@pytest.mark.parametrize("interleaved", [False, True])
def test_diagnostics_over_grid_edges(amlib, n, R, interleaved):
    check(amlib, n, R, interleaved)


@pytest.mark.parametrize("n", [7499 * 1024, 7499 * 1024 + 1, 4 * PASS + 4096 + 3])
@pytest.mark.parametrize("R", [8, 12, 16, 20])
def test_large_interleaved_stages(amlib, n, R):
    """On both sides of where stages of one and two blocks take 4096 workgroups, and a ragged end of their passes; three blocks never do."""
    check(amlib, n, R, True)
