// C entry points over the library's host-side arithmetic (am_host_logic.h: no HIP inside), so that a
// test on a machine without a GPU can drive it directly.  Built by tests/test_host_logic.py with g++.
#include "../paper_2601_22442_amd/csrc/am_host_logic.h"

extern "C" {

uint64_t hl_threshold(double p) { return am_host::subset_threshold(p); }
uint64_t hl_stratified_block(double p) { return am_host::stratified_block(p); }

void hl_blocks(uint32_t replicas, uint32_t *rb, uint32_t *rb_shift, uint32_t *nblocks)
{
    const am_host::Blocks b = am_host::block_geometry(replicas);
    *rb = b.rb; *rb_shift = b.rb_shift; *nblocks = b.nblocks;
}

uint64_t hl_capacity(uint64_t ntiles, double p, uint32_t rb, int by_line, uint64_t strat_block)
{
    return am_host::slot_capacity_lines(ntiles, p, rb, by_line != 0, strat_block);
}

// out[0..11]: ntiles, nsb, slots, cap_lines, off_flags, off_reduce, off_next, off_meta, meta_stride, off_ring, ring_stride, total
// out[12]: meta_sb_off
void hl_layout(const am_config *c, uint64_t *out)
{
    const am_host::Layout L = am_host::make_layout(*c);
    const uint64_t v[] = { L.ntiles, L.nsb, L.slots, L.cap_lines, L.off_flags, L.off_reduce, L.off_next, L.off_meta,
                           L.meta_stride, L.off_ring, L.ring_stride, L.total, L.meta_sb_off };
    for (unsigned k = 0; k < sizeof v / sizeof v[0]; ++k) out[k] = v[k];
}

// out: send, recv, same_slot, slot_send, slot_recv, step_recv
void hl_plan_round(uint64_t K, uint64_t depth, uint64_t tau, uint64_t t, uint64_t *out)
{
    const am_host::Round r = am_host::plan_round(K, depth, tau, t);
    out[0] = r.send; out[1] = r.recv; out[2] = r.same_slot; out[3] = r.slot_send; out[4] = r.slot_recv; out[5] = r.step_recv;
}

// out: nstrips, strips, parts, rows
void hl_list_shape_of(const am_config *c, uint32_t compute_units, uint32_t *out)
{
    const am_host::ListShape s = am_host::list_shape(*c, compute_units);
    out[0] = s.nstrips; out[1] = s.strips; out[2] = s.parts; out[3] = s.rows;
}

// the same for coordinates drawn one by one
void hl_list_shape(uint64_t n, double fraction, uint32_t compute_units, uint32_t *out)
{
    am_config c = {};
    c.n = n; c.fraction = fraction;
    hl_list_shape_of(&c, compute_units, out);
}

void hl_d_shape(const am_config *c, uint32_t *rb, uint32_t *arrays, uint64_t *floats) { am_host::d_layout_shape(*c, rb, arrays, floats); }

int hl_average_staged(const am_config *c, int interleaved_d)
{
    const am_host::Layout L = am_host::make_layout(*c);
    return am_host::average_staged(*c, L.ntiles, L.blocks, interleaved_d != 0);
}

uint32_t hl_step_workgroups(const am_config *c, int forward_copy, int receives)
{
    return am_host::step_workgroups(*c, am_host::block_geometry(c->replicas), forward_copy != 0, receives != 0);
}

uint32_t hl_step_sum_tiles(const am_config *c, int sync) { return am_host::step_sum_tiles(*c, am_host::block_geometry(c->replicas), sync != 0); }

// waves of a compute unit in the step by one-wave workgroups; 0: the fused kernel's workgroups
uint32_t hl_step_by_waves(const am_config *c, int forward_copy)
{
    const am_host::Blocks b = am_host::block_geometry(c->replicas);
    return am_host::step_by_waves(*c, b) ? am_host::wave_step_workgroups(*c, b, am_host::wave_step_replicas(*c), forward_copy != 0, true) : 0u;
}

// how many of them the launch's LDS lets be resident
uint32_t hl_workgroups_held(uint32_t workgroups) { return am_host::workgroups_held(workgroups); }

// its grid, x, y and z
void hl_wave_step_grid(uint32_t ntiles, uint32_t waves_of_a_tile, uint32_t *out)
{
    const am_host::Grid g = am_host::wave_step_grid(ntiles, waves_of_a_tile);
    out[0] = g.x; out[1] = g.y; out[2] = g.z;
}

int hl_local_step_alone(const am_config *c) { return am_host::local_step_alone(*c, am_host::block_geometry(c->replicas)); }
uint32_t hl_average_workgroups(const am_config *c)
{
    return am_host::average_workgroups(*c, am_host::block_geometry(c->replicas), c->d_layout == AM_D_INTERLEAVED && c->correction != AM_CORR_NONE);
}

int hl_average_weights_table(const am_config *c) { return am_host::average_weights_table(*c, am_host::block_geometry(c->replicas)); }

uint32_t hl_lds_for_residency(uint32_t need, uint32_t workgroups, uint32_t fixed) { return am_host::lds_for_residency(need, workgroups, fixed); }

uint64_t hl_record_sized_step(uint64_t record_step, uint64_t last_t) { return am_host::record_sized_step(record_step, last_t); }

uint64_t hl_resumed_sized_step(uint64_t next_lines_step, uint32_t reserved)
{
    am_snapshot s = {};
    s.next_lines_step = next_lines_step;
    s.reserved = reserved;
    return am_host::resumed_sized_step(s);
}

}  // extern "C"
