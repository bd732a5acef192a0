"""The index list of a subset (am_subset_indices) where its cut into parts can go wrong: the ends of a
lane's 32 coordinates, of a strip, of a part, one strip a wave and several, all three sampling rules, and
capacities around the count.  Whole numbers: equal to the oracle's list."""
import ctypes as C

import numpy as np
import pytest
import torch

from oracle import oracle as O

pytestmark = pytest.mark.gpu


def _stage(am, n, p, seed, **kw):
    return am.init_state(am.make_config(n, 1, fraction=p, seed=seed, optimizer=am.OPT_SGD, beta1=0.0,
                                        correction=am.CORR_NONE, **kw), torch.zeros(n))


@pytest.mark.parametrize("n,p", [
    (31, 1.0), (32, 1.0), (33, 0.5), (2047, 0.3), (2048, 1.0), (2049, 1.0), (8191, 0.05), (8192, 1.0), (8193, 0.9),
    (8192 * 64 + 2047, 0.02),
    (1 << 24, 0.01), ((1 << 24) + 1, 0.01),           # one strip a wave, two strips a wave on 256 compute units
    ((1 << 25) + 8193, 0.003),                        # three strips a wave, the last part cut
])
def test_parts_of_the_list(amlib, n, p):
    st = _stage(amlib, n, p, 17)
    for t in (1, (1 << 32) + 9):
        idx, k = st.subset_indices(t)
        want = O.subset(17, t, n, p)
        assert k == want.size and np.array_equal(idx.cpu().numpy().astype(np.uint64), want), (n, p, t)


@pytest.mark.parametrize("kw,okw", [(dict(subset_granule=32), dict(granule=32)),
                                    (dict(subset_kind=1), dict(stratified=True))])
@pytest.mark.parametrize("n", [2049, 100_003])
def test_other_sampling_rules(amlib, kw, okw, n):
    st = _stage(amlib, n, 0.07, 3, **kw)
    idx, k = st.subset_indices(5)
    want = O.subset(3, 5, n, 0.07, **okw)
    assert k == want.size and np.array_equal(idx.cpu().numpy().astype(np.uint64), want)


def test_capacity_around_the_count(amlib):
    st = _stage(amlib, 70_001, 0.1, 4)
    want = O.subset(4, 2, 70_001, 0.1).astype(np.int64)
    for cap in (0, 1, want.size - 1, want.size, want.size + 1):
        out = torch.full((max(cap, 1) + 8,), -1, dtype=torch.int64, device="cuda")
        count = torch.full((1,), -1, dtype=torch.int64, device="cuda")
        st.subset_indices_static(2, out[:cap], count)
        assert int(count.item()) == want.size
        got = out.cpu().numpy()
        kept = min(cap, want.size)
        assert np.array_equal(got[:kept], want[:kept]) and (got[kept:] == -1).all()


@pytest.mark.parametrize("n", [2049, 100_003, 1024 * 2048, 1024 * 2048 + 1, (1 << 24) + 4097])
@pytest.mark.parametrize("p,kw,okw", [(0.219, {}, {}), (0.22, {}, {}), (0.449, {}, {}), (0.45, {}, {}), (0.97, {}, {}),
                                      (0.45, dict(subset_granule=32), dict(granule=32)), (0.5, dict(subset_kind=1), dict(stratified=True))])
def test_both_sides_of_the_line_to_rows(amlib, n, p, kw, okw):
    """From p = 0.22 (0.45 on stages of up to 1024 strips) a strip is written row by row: below, at and above that, for
    all three sampling rules, with capacities that cut the list short."""
    st = _stage(amlib, n, p, 23, **kw)
    want = O.subset(23, 3, n, p, **okw).astype(np.int64)
    for cap in (want.size // 2, want.size - 1, want.size + 1):
        out = torch.full((cap + 8,), -1, dtype=torch.int64, device="cuda")
        count = torch.full((1,), -1, dtype=torch.int64, device="cuda")
        st.subset_indices_static(3, out[:cap], count)
        got, kept = out.cpu().numpy(), min(cap, want.size)
        assert int(count.item()) == want.size
        assert np.array_equal(got[:kept], want[:kept]) and (got[kept:] == -1).all()


@pytest.fixture(scope="module")
def list_kernel():
    """The kernels under a patience and a cut that the entry points never use (tests/list_kernel_driver.hip)."""
    from paper_2601_22442_amd.build import TEST_LIB, build_test_kernels, source_hash
    if not TEST_LIB.exists():
        build_test_kernels()
    lib = C.CDLL(str(TEST_LIB))
    lib.tk_source_hash.restype = C.c_char_p
    assert lib.tk_source_hash().decode() == source_hash(), "tests/liblist_kernel.so is stale: build again"
    lib.tk_subset_list.argtypes = [C.c_uint64] * 4 + [C.c_uint32, C.c_int, C.c_uint32] + [C.c_void_p, C.c_uint32, C.c_void_p, C.c_uint64, C.c_void_p, C.c_void_p]
    return lib.tk_subset_list


@pytest.mark.parametrize("patience", [0, 1])              # every workgroup counts what is before it itself; only those that had to wait
@pytest.mark.parametrize("rows", [0, 1])
@pytest.mark.parametrize("n,p,strips", [(2049, 0.5, 1), (100_003, 0.05, 1), (100_003, 1.0, 3), (700_001, 0.3, 2), (1_500_001, 0.02, 5)])
def test_a_wait_that_gives_up(list_kernel, n, p, strips, rows, patience):
    """A workgroup that has not seen the counts before it after `patience` looks hashes those coordinates itself: the
    same list and count, for one and several strips a wave, a cut last part and either way of writing."""
    want = O.subset(29, 6, n, p).astype(np.int64)
    words = -(-n // (8192 * strips))
    parts = torch.zeros(words, dtype=torch.int32, device="cuda")
    out = torch.full((want.size + 8,), -1, dtype=torch.int64, device="cuda")
    count = torch.full((1,), -1, dtype=torch.int64, device="cuda")
    assert list_kernel(n, 29, 6, int(p * 2**32), strips, rows, patience, parts.data_ptr(), words, out.data_ptr(), want.size, count.data_ptr(),
                       torch.cuda.current_stream().cuda_stream) == 0
    got = out.cpu().numpy()
    assert int(count.item()) == want.size
    assert np.array_equal(got[:want.size], want) and (got[want.size:] == -1).all()
