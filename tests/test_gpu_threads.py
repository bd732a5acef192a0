"""The calls that share a state's scratch (gradient norms, diagnostics, index list) from several threads at once: each
enqueues several kernels that hand results on through it, so none may find another's in between."""
import threading

import numpy as np
import pytest
import torch

from oracle import oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [100_003, 1_000_001])
def test_read_only_calls_from_several_threads(amlib, n):
    am, R, p = amlib, 3, 0.05
    st = am.init_state(am.make_config(n, R, delay=1, fraction=p, seed=31))
    g = torch.Generator(device="cuda").manual_seed(n)
    for i in range(R):
        st.w[i].copy_(torch.randn(n, generator=g, device="cuda"))
    grads = [torch.randn(n, generator=g, device="cuda") for _ in range(R)]
    diagnostics, norms = st.diagnostics(), st.grad_sqnorm(grads).tolist()
    lists = [O.subset(31, t, n, p).astype(np.int64) for t in range(4)]
    wrong, start = [], threading.Barrier(3)

    def repeat(same):
        start.wait()
        for k in range(100):
            if not same(k):
                wrong.append((same.__name__, k))
                return

    def diagnostics_again(k):
        return st.diagnostics() == diagnostics

    def norms_again(k):
        return st.grad_sqnorm(grads).tolist() == norms

    def list_again(k):
        out, count = st.subset_indices(k % 4)
        return count == lists[k % 4].size and np.array_equal(out.cpu().numpy(), lists[k % 4])

    threads = [threading.Thread(target=repeat, args=(f,)) for f in (diagnostics_again, norms_again, list_again)]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    assert not wrong
