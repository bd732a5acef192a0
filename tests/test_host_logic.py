"""The library's host-side arithmetic (ring slot capacity, workspace layout, which slot a step writes
and reads, replica blocks) driven directly on the CPU: csrc/am_host_logic.h holds no HIP, so a plain
g++ build of a small driver exposes it to ctypes."""
import ctypes as C
import math
import random
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parent.parent


@pytest.fixture(scope="module")
def hl(tmp_path_factory):
    so = tmp_path_factory.mktemp("hostlogic") / "libhostlogic.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-fPIC", "-shared", "-o", str(so),
                    str(ROOT / "tests" / "host_logic_driver.cpp")], check=True)
    L = C.CDLL(str(so))
    L.hl_threshold.argtypes = [C.c_double]; L.hl_threshold.restype = C.c_uint64
    L.hl_stratified_block.argtypes = [C.c_double]; L.hl_stratified_block.restype = C.c_uint64
    L.hl_blocks.argtypes = [C.c_uint32] + [C.POINTER(C.c_uint32)] * 3
    L.hl_capacity.argtypes = [C.c_uint64, C.c_double, C.c_uint32, C.c_int, C.c_uint64]; L.hl_capacity.restype = C.c_uint64
    L.hl_layout.argtypes = [C.c_void_p, C.POINTER(C.c_uint64)]
    L.hl_plan_round.argtypes = [C.c_uint64] * 4 + [C.POINTER(C.c_uint64)]
    return L


def _config(**kw):
    """am_config as the binding lays it out (the ABI test checks that layout against the C compiler's)."""
    from paper_2601_22442_amd.binding import Config
    base = dict(n=1000, replicas=2, delay=0, avg_interval=1, optimizer=1, fraction=0.05, seed=0, beta1=0.9, beta2=0.999,
                eps=1e-8, weight_decay=0.01, gamma=0.0, lookahead=0, correction=1, fwd_dtype=0, grad_dtype=0,
                momentum_decay=0.004, subset_granule=1, msg_dtype=0, subset_kind=0, d_layout=0, ring_cap_lines=0)
    base.update(kw)
    return Config(**base)


def test_threshold_and_blocks(hl, amlib):
    assert hl.hl_threshold(0.0) == 0 and hl.hl_threshold(1.0) == 1 << 32 and hl.hl_threshold(0.5) == 1 << 31
    assert hl.hl_threshold(0.05) == math.floor(0.05 * 2 ** 32)
    assert hl.hl_stratified_block(0.05) == 20 and hl.hl_stratified_block(1.0) == 1 and hl.hl_stratified_block(0.3) == 3
    for R in range(1, 33):
        rb, sh, nb = C.c_uint32(), C.c_uint32(), C.c_uint32()
        hl.hl_blocks(R, C.byref(rb), C.byref(sh), C.byref(nb))
        want_rb = min(8, 1 << (R - 1).bit_length())
        assert (rb.value, 1 << sh.value, nb.value) == (want_rb, want_rb, -(-R // want_rb)), R
        assert nb.value * rb.value >= R > (nb.value - 1) * rb.value


@pytest.mark.parametrize("p,rb", [(0.05, 8), (0.05, 1), (0.01, 8), (0.10, 8), (0.3, 4), (0.001, 2), (0.9, 8)])
def test_slot_capacity_is_mean_plus_twelve_sigma_of_the_exact_line_count(hl, p, rb):
    """A tile of 256 coordinates owns ceil(X rb / 32) lines, X ~ Binomial(256, p): exact moments by summation."""
    ntiles = 491_520
    pmf = [math.comb(256, k) * p ** k * (1 - p) ** (256 - k) for k in range(257)]
    lines = [-(-k * rb // 32) for k in range(257)]
    mean = sum(a * b for a, b in zip(pmf, lines))
    var = sum(a * b * b for a, b in zip(pmf, lines)) - mean ** 2
    want = math.ceil(ntiles * mean + 12 * math.sqrt(ntiles * var)) + 64
    got = hl.hl_capacity(ntiles, p, rb, 0, 0)
    assert abs(got - min(want, ntiles * 8 * rb)) <= 1
    # the margin is real: at least ten standard deviations above the mean, never more than every line
    assert got <= ntiles * 8 * rb
    if got < ntiles * 8 * rb:
        assert got >= ntiles * mean + 10 * math.sqrt(ntiles * var)


def test_slot_capacity_special_cases(hl):
    assert hl.hl_capacity(100, 1.0, 8, 0, 0) == 100 * 64                # everything selected: 256 * 8 / 32 lines a tile
    assert hl.hl_capacity(100, 1.0, 1, 0, 0) == 100 * 8
    assert hl.hl_capacity(1000, 0.05, 8, 0, 20) == 1000 * 4              # stratified, B = 20: at most 14 members -> 4 lines
    assert hl.hl_capacity(1000, 1 / 256, 8, 0, 256) == 1000              # B = 256: at most 2 members -> one line
    assert hl.hl_capacity(1000, 1.0, 4, 0, 1) == 1000 * 32               # B = 1: every coordinate
    # whole lines of 32 coordinates drawn: Binomial(8, p) x rb lines a tile
    ntiles, p, rb = 100_000, 0.07, 8
    want = math.ceil(ntiles * 8 * p * rb + 12 * math.sqrt(ntiles * 8 * p * (1 - p)) * rb) + 64
    assert abs(hl.hl_capacity(ntiles, p, rb, 1, 0) - want) <= 1
    assert hl.hl_capacity(1, 0.5, 8, 0, 0) == 64                         # tiny stage: the margin saturates at every line


def test_workspace_regions_do_not_overlap_and_match_the_library(hl, amlib):
    am = amlib
    rng = random.Random(5)
    for _ in range(60):
        n = rng.choice([1, 255, 256, 257, 131_072, 131_073, rng.randrange(1, 50_000_000)])
        R = rng.randrange(1, 33)
        cfg = _config(n=n, replicas=R, delay=rng.randrange(0, 9), fraction=rng.choice([1e-6, 0.01, 0.05, 0.5, 1.0]),
                      subset_kind=rng.randrange(0, 2), ring_cap_lines=rng.choice([0, 0, 17, 10 ** 12]))
        out = (C.c_uint64 * 13)()
        hl.hl_layout(C.byref(cfg), out)
        ntiles, nsb, slots, cap, off_flags, off_reduce, off_next, off_meta, meta_stride, off_ring, ring_stride, total, sb_off = out
        assert ntiles == -(-n // 256) and nsb == -(-ntiles // 512) and slots == cfg.delay + 1
        rb = min(8, 1 << (R - 1).bit_length()); nblocks = -(-R // rb)
        if cfg.ring_cap_lines:
            assert cap == min(cfg.ring_cap_lines, ntiles * 8 * rb)
        regions = [(off_flags, 256), (off_reduce, 32 * 1024 * 8), (off_next, ntiles * 4)]
        for s in range(slots + 1):
            base = off_meta + s * meta_stride
            regions += [(base, ntiles * 4), (base + sb_off, (nsb + 1) * 4)]
        for s in range(slots):
            regions.append((off_ring + s * ring_stride, cap * 128 * nblocks))
        regions.sort()
        for (a, la), (b, _) in zip(regions, regions[1:]):
            assert a + la <= b, (a, la, b)
        assert regions[-1][0] + regions[-1][1] <= total
        assert all(a % 256 == 0 for a, _ in regions)
        assert am.workspace_bytes(cfg) == total                           # the library uses this very arithmetic


def test_ring_slots_hold_what_a_step_expects_under_any_delay_sequence(hl):
    """Model: a slot holds the round that last wrote it.  Whatever the interval, the ring depth and
    the delays in force from step to step (am_set_delay), a receive must find, in the slot it reads,
    exactly the round sent tau rounds earlier, and nothing is received before anything was sent."""
    rng = random.Random(11)
    for _ in range(200):
        K, delay = rng.randrange(1, 6), rng.randrange(0, 7)
        depth = delay + 1
        held = {}
        out = (C.c_uint64 * 6)()
        for t in range(1, 12 * K * depth + 3):
            tau = rng.randrange(0, depth)
            hl.hl_plan_round(K, depth, tau, t, out)
            send, recv, same, slot_s, slot_r, step_r = out
            if t % K:
                assert not send and not recv
                continue
            assert send and slot_s == (t // K) % depth
            if recv:
                assert step_r == t - tau * K and step_r >= 1 and bool(same) == (tau == 0)
                if same:
                    assert slot_r == slot_s
                else:
                    assert held[slot_r] == step_r, (K, delay, tau, t)      # still there: not yet overwritten
            else:
                assert t - tau * K < 1
            held[slot_s] = t                                              # the send of this step lands after the receive


def test_static_scratch_limit_is_stated_consistently():
    """The header, and the entry point's refusal, speak of 2^27 coordinates."""
    text = (ROOT / "include" / "asyncmesh.h").read_text()
    assert "n <= 2^27 = 134,217,728" in text
    src = (ROOT / "paper_2601_22442_amd" / "csrc" / "asyncmesh.hip").read_text()
    assert "kStaticMaxN = 1ull << 27" in src


@pytest.mark.parametrize("compute_units", [1, 64, 256, 304])
def test_list_parts_cover_the_stage_and_fit_their_scratch(hl, compute_units):
    """Every strip belongs to exactly one part; the parts' counts fit the reductions' partials, whose size does not
    grow with the stage, and, up to 2^27 coordinates, the static scratch (a word per four strips)."""
    layout, out = (C.c_uint64 * 13)(), (C.c_uint32 * 4)()
    for n in (1, 255, 2048, 2049, 8192, 8193, 1 << 24, (1 << 24) + 1, 125_829_120, 1 << 27, 1 << 30, (1 << 32) - (1 << 20) - 1):
        hl.hl_layout(C.byref(_config(n=n, replicas=1)), layout)
        partials_words = (layout[6] - layout[5]) // 4
        assert partials_words == 32 * 1024 * 2
        hl.hl_list_shape(C.c_uint64(n), C.c_double(0.05), compute_units, out)
        nstrips, strips, parts = list(out)[:3]
        assert nstrips == -(-n // 2048) and 1 <= strips <= 32
        assert (parts - 1) * 4 * strips < nstrips <= parts * 4 * strips
        assert parts <= partials_words
        if n <= 1 << 27:
            assert parts <= (1 << 27) // 8192


def test_a_record_names_sizes_that_every_build_finds(hl):
    """A record passes on the sized step it was resumed with as long as that step is still to come, and names none of its own; a record whose
    reserved field is not zero may mean another table, so nothing in it counts as sized."""
    hl.hl_record_sized_step.argtypes, hl.hl_record_sized_step.restype = [C.c_uint64, C.c_uint64], C.c_uint64
    hl.hl_resumed_sized_step.argtypes, hl.hl_resumed_sized_step.restype = [C.c_uint64, C.c_uint32], C.c_uint64
    assert hl.hl_record_sized_step(9, 8) == 9 and hl.hl_record_sized_step(9, 9) == 0 and hl.hl_record_sized_step(9, 1 << 40) == 0
    assert hl.hl_record_sized_step(1 << 40, 8) == 1 << 40 and hl.hl_record_sized_step(0, 0) == 0
    assert hl.hl_resumed_sized_step(9, 0) == 9
    assert all(hl.hl_resumed_sized_step(9, r) == 0 for r in (1, 2, 3, 1 << 31))


@pytest.mark.parametrize("n,R,kw,staged", [
    # blocks of eight: up to 22 % of the coordinates always, more beyond what the caches hold (slots of absent replicas count)
    (20_000_000, 8, dict(fraction=0.0625, d_layout=0), True), (20_000_000, 8, dict(fraction=0.5, d_layout=0), True), (100_000, 8, dict(fraction=0.21), True), (100_000, 8, dict(fraction=0.23), False),
    (850_000, 8, dict(fraction=0.5, d_layout=0), False), (850_001, 8, dict(fraction=0.5, d_layout=0), True), (850_001, 5, dict(fraction=0.5, d_layout=0), True),
    (662_500, 8, dict(fraction=0.5), False), (662_501, 8, dict(fraction=0.5), True), (437_500, 8, dict(fraction=1.0), False), (437_501, 8, dict(fraction=1.0), True),
    # several blocks; E4M3
    (218_750, 12, dict(fraction=0.3), False), (218_751, 12, dict(fraction=0.3), True), (300_000, 12, dict(fraction=0.3, msg_dtype=2), False), (300_000, 12, dict(fraction=0.9, msg_dtype=2), True),
    (375_000, 12, dict(fraction=0.3, d_layout=0), False), (375_001, 12, dict(fraction=0.3, d_layout=0), True), (100_000, 20, dict(fraction=0.35), True), (100_000, 20, dict(fraction=0.36), False),
    (216_000, 20, dict(fraction=0.5, d_layout=0), False), (217_000, 20, dict(fraction=0.5, d_layout=0), True), (150_000, 20, dict(fraction=1.0, d_layout=0), True), (150_000, 20, dict(fraction=1.0, d_layout=0, msg_dtype=2), False),
    (110_000, 32, dict(fraction=0.5, d_layout=0), True), (109_000, 32, dict(fraction=0.5, d_layout=0), False),
    # blocks of four, also where the caches hold one form and not the other
    (1_175_000, 4, dict(fraction=0.25, d_layout=0), True), (1_180_000, 4, dict(fraction=0.25, d_layout=0), False), (2_120_000, 3, dict(fraction=0.04, d_layout=0), False), (2_130_000, 3, dict(fraction=0.04, d_layout=0), True),
    (1_500_000, 4, dict(fraction=0.03, d_layout=0), True), (1_500_000, 4, dict(fraction=0.08), True), (1_500_000, 4, dict(fraction=0.1), False), (1_500_000, 4, dict(fraction=0.1, subset_granule=32), True),
    (2_400_000, 4, dict(fraction=0.2, correction=0), False), (2_510_000, 4, dict(fraction=0.2, correction=0), True), (2_000_000, 4, dict(fraction=0.15, correction=0), True),
    (500_000, 4, dict(fraction=0.45), True), (750_000, 4, dict(fraction=0.5), False), (750_001, 3, dict(fraction=0.5), True), (1_050_000, 4, dict(fraction=0.5, d_layout=0), False), (1_050_001, 4, dict(fraction=0.5, d_layout=0), True),
    # members in whole lines
    (500_000, 8, dict(fraction=0.09, subset_granule=32), True), (500_000, 8, dict(fraction=0.1, subset_granule=32), False), (700_000, 8, dict(fraction=0.1, subset_granule=32), True), (300_000, 12, dict(fraction=0.5, subset_granule=32), False),
    (300_000, 12, dict(fraction=0.6, subset_granule=32), True), (387_000, 12, dict(fraction=0.25, subset_granule=32), False), (388_000, 12, dict(fraction=0.25, subset_granule=32), True), (1_050_000, 8, dict(fraction=0.2, subset_granule=32, d_layout=0), False), (1_060_000, 8, dict(fraction=0.2, subset_granule=32, d_layout=0), True),
    (830_000, 8, dict(fraction=0.6, subset_granule=32, d_layout=0), True), (1_200_000, 4, dict(fraction=0.3, subset_granule=32, d_layout=0), False), (1_200_000, 4, dict(fraction=0.6, subset_granule=32, d_layout=0), True),
    # blocks of one and two: per replica up to half a turn or a large stage, interleaved one turn, a large stage or nearly whole tiles
    (500_000, 2, dict(fraction=0.25, d_layout=0), True), (500_000, 2, dict(fraction=0.26, d_layout=0), False), (6_300_000, 2, dict(fraction=1.0, d_layout=0), True), (6_200_000, 2, dict(fraction=1.0, d_layout=0), False),
    (500_000, 2, dict(fraction=0.4), True), (500_000, 2, dict(fraction=0.5), False), (3_200_000, 2, dict(fraction=0.5), True), (800_000, 2, dict(fraction=0.9), True), (800_000, 1, dict(fraction=1.0), True),
    # no correction
    (1_000_000, 8, dict(fraction=0.17, correction=0), True), (3_250_000, 8, dict(fraction=0.18, correction=0), False), (3_250_001, 8, dict(fraction=0.18, correction=0), True), (1_375_000, 8, dict(fraction=1.0, correction=0), False),
    (1_375_001, 8, dict(fraction=1.0, correction=0), True), (5_600_000, 5, dict(fraction=0.5, correction=0), False), (5_700_000, 5, dict(fraction=0.5, correction=0), True), (13_700_000, 5, dict(fraction=1.0, correction=0), True), (13_800_000, 5, dict(fraction=1.0, correction=0), False), (1_000_000, 12, dict(fraction=0.5, correction=0), False), (1_070_000, 12, dict(fraction=0.5, correction=0), True), (700_000, 12, dict(fraction=0.7, correction=0), True),
    (357_000, 12, dict(fraction=1.0, correction=0), True), (230_000, 20, dict(fraction=0.5, correction=0), False), (240_000, 20, dict(fraction=0.5, correction=0), True), (1_050_001, 4, dict(fraction=0.5, correction=0), True),
    (1_062_000, 8, dict(fraction=0.1, correction=0, subset_granule=32), False), (1_063_000, 8, dict(fraction=0.1, correction=0, subset_granule=32), True), (3_250_000, 8, dict(fraction=0.5, correction=0, subset_granule=32), False),
    (2_125_000, 4, dict(fraction=0.4, correction=0, subset_granule=32), False), (1_430_000, 4, dict(fraction=0.5, correction=0, subset_granule=32), True), (500_000, 12, dict(fraction=0.1, correction=0, subset_granule=32), False),
    # the measured cases
    (125_829_120, 8, dict(fraction=0.05), True), (1_048_576, 4, dict(fraction=0.01, d_layout=0), True),
])
def test_averaging_stages_where_that_is_the_faster_form(hl, n, R, kw, staged):
    kw = dict(dict(d_layout=1), **kw)
    assert bool(hl.hl_average_staged(C.byref(_config(n=n, replicas=R, delay=1, **kw)), kw["d_layout"] and kw.get("correction", 1) != 0)) == staged


@pytest.mark.parametrize("n,R,kw,fwd,receives,workgroups", [
    # by what the step moves of a replica's part of a tile, more easily with a dense d
    (16_000_000, 4, dict(d_layout=0), True, True, 5), (16_000_000, 4, dict(d_layout=0), False, True, 5), (16_000_000, 4, dict(d_layout=1), False, True, 6),
    (16_000_000, 4, dict(d_layout=1, grad_dtype=1), False, True, 0), (16_000_000, 4, dict(d_layout=0, grad_dtype=1), False, True, 5), (16_000_000, 4, dict(d_layout=0), False, False, 0),
    (16_000_000, 4, dict(optimizer=0), False, True, 5), (16_000_000, 4, dict(optimizer=0, d_layout=1), True, True, 0), (16_000_000, 4, dict(correction=0), True, True, 6), (16_000_000, 4, dict(optimizer=0, beta1=0.0), True, True, 0),
    (30_000_000, 2, dict(d_layout=0), True, True, 11), (30_000_000, 2, dict(correction=0), True, True, 11), (30_000_000, 2, dict(correction=0), False, True, 0),
    (30_000_000, 2, dict(d_layout=1), False, True, 0), (30_000_000, 2, dict(d_layout=1, grad_dtype=1), True, True, 0), (30_000_000, 2, dict(d_layout=0, grad_dtype=1), False, True, 11), (3_000_017, 2, dict(optimizer=0, fraction=0.1), False, True, 0),
    # absent replicas, one replica, eight; a stage that the caches hold
    (20_000_000, 3, dict(d_layout=0), True, True, 0), (60_000_000, 1, dict(d_layout=0), True, True, 0), (20_000_000, 8, dict(d_layout=0), True, True, 0), (1_300_000, 4, dict(d_layout=0), True, True, 0),
])
def test_step_residency_follows_what_a_wave_moves(hl, n, R, kw, fwd, receives, workgroups):
    assert hl.hl_step_workgroups(C.byref(_config(n=n, replicas=R, delay=1, **kw)), fwd, receives) == workgroups


@pytest.mark.parametrize("n,R,kw,fwd,waves", [
    # interleaved EMA vectors: even numbers of replicas up to 24 and small fractions, or many absent slots
    (125_829_120, 8, dict(d_layout=1), True, 10), (5_242_880, 8, dict(d_layout=1), True, 0), (5_242_881, 8, dict(d_layout=1), True, 11), (31_457_281, 8, dict(d_layout=1, fraction=0.07), True, 0),
    (31_457_281, 7, dict(d_layout=1), True, 0), (10_000_000, 32, dict(d_layout=1), True, 0), (10_000_000, 24, dict(d_layout=1), True, 10), (2_600_000, 5, dict(d_layout=1, fraction=0.1), True, 21),
    # per replica and without a correction
    (31_457_281, 8, dict(d_layout=0, fraction=0.1), True, 9), (31_457_281, 7, dict(d_layout=0), False, 20), (31_457_281, 8, dict(d_layout=0, fraction=0.11), True, 0), (8_388_608, 8, dict(correction=0), True, 0),
    (8_388_609, 8, dict(correction=0), True, 11), (125_829_120, 16, dict(correction=0, grad_dtype=1, fwd_dtype=1, fraction=0.01), True, 11), (31_457_281, 4, dict(d_layout=0), True, 0),
])
def test_large_steps_go_by_waves(hl, n, R, kw, fwd, waves):
    hl.hl_step_by_waves.restype = C.c_uint32
    assert hl.hl_step_by_waves(C.byref(_config(n=n, replicas=R, delay=1, **kw)), fwd) == waves


@pytest.mark.parametrize("n,R,kw,waves", [
    # interleaved EMA vectors, few absent slots: neither the shortest nor the longest steps, small fractions, no momentum alone
    (50_331_648 // 16, 16, {}, False), (50_331_648 // 16 + 1, 16, {}, True), (1 << 25, 16, {}, True), ((1 << 25) + 1, 16, {}, False), (10_000_000, 16, dict(fraction=0.06), False),
    (10_000_000, 16, dict(optimizer=0), False), (10_000_000, 16, dict(optimizer=0, beta1=0.0), True), (60_000_000 // 22, 22, {}, False), (90_000_000 // 22, 22, {}, True), (45_000_000 // 18, 18, dict(fraction=0.06), True),
    (125_829_120, 8, {}, True), (31_457_281, 8, dict(optimizer=0, fraction=0.06), True), (10_000_000, 14, {}, True),
    # many: five and eleven replicas, one a wave, up to smaller fractions than nine and ten
    (9_000_003, 5, dict(fraction=0.05), True), (9_000_003, 5, dict(fraction=0.06), False), (26_000_003, 5, dict(fraction=0.03), True), (26_000_003, 5, dict(fraction=0.05), False), (2_600_000, 5, {}, True),
    (4_090_912, 11, dict(fraction=0.06), True), (4_090_912, 11, dict(fraction=0.07), False), (6_666_669, 9, dict(fraction=0.1), True), (6_666_669, 10, dict(fraction=0.1), True),
    # every other layout: odd numbers, too, but the largest
    (10_000_000, 25, dict(d_layout=0), True), (10_000_000, 31, dict(d_layout=0), False), (10_000_000, 27, dict(correction=0), False), (10_000_000, 32, dict(d_layout=0, fraction=0.1), True),
    (26_000_003, 5, dict(d_layout=0, fraction=0.1), True), (4_090_912, 11, dict(correction=0, fraction=0.1), True),
])
def test_large_steps_go_by_waves_where_that_is_faster(hl, n, R, kw, waves):
    hl.hl_step_by_waves.restype = C.c_uint32
    assert bool(hl.hl_step_by_waves(C.byref(_config(n=n, replicas=R, delay=1, **dict(dict(d_layout=1), **kw))), True)) == waves


@pytest.mark.parametrize("n", [2_097_153, 32_768 * 128 * 256, 32_768 * 128 * 256 + 1, 65_535 * 128 * 256 + 1, (1 << 31) + 1, (1 << 32) - (1 << 20) - 1])
@pytest.mark.parametrize("waves", [4, 5, 16, 31])
def test_the_grid_of_a_step_by_waves_covers_every_stage(hl, n, waves):
    """128 tiles a chunk: a grid may have 65535 workgroups in y and in z, and 2^32 work-items in x."""
    ntiles, g = (n + 255) // 256, (C.c_uint32 * 3)()
    hl.hl_wave_step_grid(ntiles, waves, g)
    assert g[0] == 128 * waves and g[1] <= 65_535 and g[2] <= 65_535
    assert g[1] * g[2] * 128 >= ntiles and g[1] * (g[2] - 1) * 128 < ntiles          # no tile is left out, no layer of the grid is idle


@pytest.mark.parametrize("bound", range(1, 33))
def test_every_number_that_a_rule_can_name_is_held_to(hl, bound):
    """160 KB in granules of 1280 bytes: a compute unit holds as many as named, or the next smaller number that equal shares allow."""
    attainable = {128 // g for g in range(1, 129)}
    share = -(-hl.hl_lds_for_residency(1, bound, 0) // 1280)
    assert 128 // share == hl.hl_workgroups_held(bound) == max(k for k in attainable if k <= bound)


@pytest.mark.parametrize("workgroups", [2, 3, 4, 5, 6, 7, 11])
@pytest.mark.parametrize("fixed", [0, 16])
def test_lds_holds_as_many_workgroups_as_a_rule_names(hl, workgroups, fixed):
    """160 KB of LDS in granules of 1280 bytes: that many fit, one more does not; a larger need is kept, and 0 limits nothing."""
    granules = -(-(hl.hl_lds_for_residency(100, workgroups, fixed) + fixed) // 1280)
    assert workgroups * granules <= 128 < (workgroups + 1) * granules
    assert hl.hl_lds_for_residency(70_000, workgroups, fixed) >= 70_000 and hl.hl_lds_for_residency(100, 0, fixed) == 100


def test_steps_add_up_offsets_on_fewer_tiles_with_more_blocks(hl):
    tiles = {(R, sync): hl.hl_step_sum_tiles(C.byref(_config(replicas=R, delay=0 if sync else 1)), sync) for R in range(1, 33) for sync in (0, 1)}
    assert all(tiles[R, 0] == (8192 if R <= 2 else 6144 if R <= 4 else 8192 if R <= 16 else 2048 if R <= 24 else 768) for R in range(1, 33))
    assert all(tiles[R, 1] == (8192 if R <= 8 or R > 16 else 1024 if R in (13, 14) else 2560) for R in range(1, 33))
    assert all(hl.hl_step_sum_tiles(C.byref(_config(replicas=R, delay=0, optimizer=0, beta1=0.0)), 1) == (4608 if 5 <= R <= 7 else tiles[R, 1]) for R in range(1, 33))


@pytest.mark.parametrize("kw", [dict(subset_granule=32), dict(subset_kind=1), dict(subset_kind=1, fraction=0.01), dict(fraction=0.3), dict(fraction=0.3, subset_granule=32), {}])
def test_list_cut_follows_how_the_subset_is_drawn_and_written(hl, kw):
    """Waves of a compute unit (strips a wave): 20 for coordinates drawn one by one and written lane by lane (40 beyond eight strips); 32 for the others,
    where 20 would leave more than two strips a wave, the strips are written row by row or a stratified subset is small.  The parts fit their scratch."""
    out, cus, short = (C.c_uint32 * 4)(), 256, kw.get("fraction", 0.05) >= 0.03
    rows, one_by_one = kw.get("fraction", 0.05) >= 0.22, "subset_granule" not in kw and "subset_kind" not in kw
    for n in (3_000_000, 12_000_000, 20_971_520, 20_971_521, 48_000_000, 83_886_080, 83_886_081, 1 << 27, 1 << 30):
        hl.hl_list_shape_of(C.byref(_config(n=n, **kw)), cus, out)
        nstrips, strips, parts = list(out)[:3]
        waves = cus * ((20 if nstrips <= 8 * 20 * cus else 40) if one_by_one and not rows else 20 if not rows and short and nstrips <= 2 * 20 * cus else 32)
        assert strips == min(32, -(-nstrips // waves)) and bool(out[3]) == rows
        assert (parts - 1) * 4 * strips < nstrips <= parts * 4 * strips and parts <= (1 << 27) // 8192 or n > 1 << 27


@pytest.mark.parametrize("weights,R,kw", [
    (1 << 20, 8, dict(avg_interval=4)), (1 << 20, 5, dict(avg_interval=5)), (6 << 20, 8, dict(avg_interval=2)), (6 << 20, 16, dict(avg_interval=3)), (6 << 20, 8, dict(avg_interval=2, optimizer=0)),
    (5 << 19, 8, dict(avg_interval=2, optimizer=0, beta1=0.0)), (5 << 19, 5, dict(avg_interval=2)),
])
def test_steps_between_rounds_have_a_kernel_of_their_own_where_it_pays(hl, weights, R, kw):
    """Beyond this many weights, by how often a round comes and by what a wave moves; blocks of four and fewer never."""
    assert not hl.hl_local_step_alone(C.byref(_config(n=weights // R, replicas=R, delay=1, **kw)))
    assert hl.hl_local_step_alone(C.byref(_config(n=weights // R + 1, replicas=R, delay=1, **kw)))
    assert not hl.hl_local_step_alone(C.byref(_config(n=10 * weights, replicas=4, delay=1, **kw)))


@pytest.mark.parametrize("weights,R,kw,workgroups", [
    # some 114 KB of lines on their way a compute unit: the measured cases and their neighbours
    (1_006_632_960, 8, dict(d_layout=1), 3), (1_006_632_960, 8, dict(d_layout=1, fraction=0.01), 0), (250_000_000, 8, dict(d_layout=0), 2), (250_000_000, 8, dict(d_layout=1, fraction=0.1), 2),
    (250_000_000, 4, dict(d_layout=0), 4), (250_000_000, 4, dict(d_layout=1), 5), (250_000_000, 8, dict(correction=0), 4),
    # the caches still help; several turns a tile; absent replicas; three blocks
    (1 << 26, 8, dict(d_layout=0), 0), (80_000_000, 8, dict(d_layout=0), 3), (80_000_000, 8, dict(d_layout=1, fraction=0.1), 3), (250_000_000, 8, dict(d_layout=1, fraction=0.6), 3),
    (250_000_000, 8, dict(d_layout=1, fraction=1.0), 4), (250_000_000, 4, dict(d_layout=0, fraction=1.0), 4), (250_000_000, 16, dict(d_layout=1, fraction=1.0), 3),
    (250_000_000, 5, dict(d_layout=1, fraction=0.1), 3), (250_000_000, 5, dict(d_layout=1), 4), (250_000_000, 5, dict(d_layout=1, fraction=0.02), 0), (250_000_000, 5, dict(d_layout=0), 3), (250_000_000, 3, dict(d_layout=0, fraction=0.5), 4), (130_000_000, 20, dict(d_layout=1, fraction=0.2), 3),
    # tiles of eight replicas that take several turns, without interleaved EMA entries; R = 2 and 3
    (120_000_000, 8, dict(d_layout=0, fraction=0.1), 2), (120_000_000, 8, dict(d_layout=0, fraction=0.25), 0), (120_000_000, 12, dict(d_layout=0, fraction=0.5), 0), (220_000_000, 12, dict(d_layout=0, fraction=0.5), 3),
    (220_000_000, 5, dict(d_layout=0, fraction=0.25), 4), (220_000_000, 8, dict(d_layout=0, fraction=1.0), 4), (220_000_000, 8, dict(d_layout=0, fraction=0.25, msg_dtype=1), 0),
    (220_000_000, 8, dict(correction=0, fraction=0.25), 0), (120_000_000, 5, dict(d_layout=0, fraction=0.25, msg_dtype=2), 0), (120_000_000, 2, dict(d_layout=1, fraction=0.4), 6), (120_000_000, 2, dict(d_layout=1, fraction=0.5), 7), (120_000_000, 2, dict(d_layout=1, fraction=1.0), 7),
    (90_000_000, 3, dict(d_layout=0, fraction=0.2), 4), (126_000_000, 5, dict(d_layout=1, fraction=0.5), 3),
    # rounded messages; no correction where most are drawn; members in whole lines
    (250_000_000, 8, dict(d_layout=1, fraction=0.2, msg_dtype=1), 3), (250_000_000, 8, dict(d_layout=1, fraction=0.2, msg_dtype=2), 4), (250_000_000, 20, dict(d_layout=1, msg_dtype=2), 0),
    (250_000_000, 4, dict(correction=0, fraction=0.4), 5), (250_000_000, 4, dict(correction=0, fraction=0.8), 0), (250_000_000, 8, dict(d_layout=1, fraction=0.4, subset_granule=32), 0),
])
def test_averaging_residency_follows_the_lines_and_the_turns(hl, weights, R, kw, workgroups):
    assert hl.hl_average_workgroups(C.byref(_config(n=weights // R + (weights % R > 0), replicas=R, delay=1, **kw))) == workgroups


@pytest.mark.parametrize("R,kw,low,high", [
    # in the records above `low` and up to `high` weights
    (8, {}, 5 << 20, 23 << 19), (5, dict(fraction=1.0), 5 << 20, 23 << 19), (32, dict(fraction=0.03, d_layout=1), 5 << 20, 23 << 19), (8, dict(fraction=0.02), 0, 0), (8, dict(subset_granule=32), 0, 0), (4, {}, 0, 0),
    (8, dict(delay=0, fraction=0.5), 5 << 20, 20 << 20), (8, dict(delay=0, fraction=0.4), 0, 0), (12, dict(delay=0, fraction=1.0), 0, 0), (6, dict(correction=0, fraction=0.5), 5 << 20, 20 << 20), (8, dict(correction=0, fraction=0.25), 0, 0),
])
def test_weights_of_blocks_of_eight_are_named_in_a_table_but_for_a_few(hl, R, kw, low, high):
    kw = dict(dict(delay=1), **kw)
    for weights in (1 << 20, 5 << 20, 23 << 19, 20 << 20):
        for n in (weights // R, weights // R + 1, 50_000_000):
            assert bool(hl.hl_average_weights_table(C.byref(_config(n=n, replicas=R, **kw)))) == (not low < n * R <= high)
