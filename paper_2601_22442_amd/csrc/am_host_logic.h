// Host-side arithmetic of the AsyncMesh stage update that involves no device: subset threshold,
// replica blocks, ring slot capacity, workspace layout, and which ring slots a step sends to and
// receives from.  Plain C++ (no HIP), so that it can be compiled and tested on a machine without a GPU.
#pragma once
#include <stdint.h>

#include <algorithm>
#include <cmath>

#include "../../include/asyncmesh.h"
#include "am_geometry.h"

namespace am_host {

inline uint64_t round_up(uint64_t x, uint64_t a) { return (x + a - 1) / a * a; }

// floor(p 2^32); 2^32 selects every coordinate (sampling model of the sparse-averaging lemma)
inline uint64_t subset_threshold(double p)
{
    if (!(p > 0.0)) return 0;
    if (p >= 1.0) return 1ull << 32;
    return (uint64_t)std::floor(p * 4294967296.0);
}

// B = round(1/p) of the stratified sampling variant
inline uint64_t stratified_block(double p)
{
    const long long B = std::llround(1.0 / p);
    return B < 1 ? 1 : (uint64_t)B;
}

// Replicas are cut into blocks of rb = min(8, R rounded up to a power of two) consecutive replicas;
// the sparse values of a block's replicas sit side by side in memory.
struct Blocks {
    uint32_t rb, rb_shift, nblocks;
};

inline Blocks block_geometry(uint32_t replicas)
{
    Blocks b{1, 0, 1};
    while (b.rb < replicas && b.rb < am::kMaxBlockReplicas) { b.rb <<= 1; ++b.rb_shift; }
    b.nblocks = (replicas + b.rb - 1) / b.rb;
    return b;
}

// Lines (of 32 floats) one block's part of a ring slot must hold.  Every tile of 256 coordinates
// owns ceil(X rb / 32) whole lines, X ~ Binomial(256, p) its number of selected coordinates; the
// slot has room for the expected total plus twelve standard deviations (and 64 lines).
//   by_line: aligned blocks of 32 coordinates are drawn as a whole (X = 32 Binomial(8, p))
//   strat_block != 0: stratified sampling with that block length (no chance involved)
inline uint64_t slot_capacity_lines(uint64_t ntiles, double p, uint32_t rb, bool by_line, uint64_t strat_block)
{
    const uint64_t lines_per_tile = am::kTileCoords * rb / am::kLineFloats;     // every coordinate selected
    const uint64_t all = ntiles * lines_per_tile;
    if (p >= 1.0) return all;
    if (strat_block) {     // a tile meets at most floor(255 / B) + 2 blocks, one member each
        const uint64_t members = std::min<uint64_t>(am::kTileCoords, (am::kTileCoords - 1) / strat_block + 2);
        return std::min(all, ntiles * ((members * rb + am::kLineFloats - 1) / am::kLineFloats));
    }
    double mean = 0.0, sq = 0.0;
    if (by_line) {         // Binomial(8, p) drawn lines of 32 coordinates, rb lines of values each
        const double per = am::kTileCoords / am::kLineFloats;
        mean = per * p * rb;
        sq = per * p * (1.0 - p) * rb * rb + mean * mean;
    } else {
        const double lp = std::log(p), lq = std::log1p(-p), T = am::kTileCoords;
        for (int k = 0; k <= (int)am::kTileCoords; ++k) {
            const double pmf = std::exp(std::lgamma(T + 1.0) - std::lgamma(k + 1.0) - std::lgamma(T - k + 1.0) + k * lp + (T - k) * lq);
            const double lines = (double)(((uint64_t)k * rb + am::kLineFloats - 1) / am::kLineFloats);
            mean += pmf * lines;
            sq += pmf * lines * lines;
        }
    }
    const double var = sq - mean * mean > 0.0 ? sq - mean * mean : 0.0;
    const double cap = std::ceil((double)ntiles * mean + 12.0 * std::sqrt((double)ntiles * var)) + 64.0;
    return cap >= (double)all ? all : (uint64_t)cap;
}

// workspace = [flags 256 B][reduction partials 32 x 1024 doubles][sizes of a record u32[ntiles]][meta x (slots + 1)][ring values x slots]
//   meta = tile words u32[ntiles] | sb_base u32[nsb + 1]      (tile words of the extra block: two tables of the tiles' sizes, a byte each; its
//   sb_base is unused).  The sizes of a record: words that builds before the byte tables left for a resumed step; only read.
//   ring slot = nblocks * cap_lines * 32 fp32: [block][line][32], a line = [coordinate][replica in block]
constexpr uint64_t kReduceBytes = (uint64_t)AM_MAX_REPLICAS * 1024 * 8;
struct Layout {
    uint32_t ntiles, nsb, slots;
    Blocks blocks;
    uint64_t cap_lines;
    uint64_t off_flags, off_reduce, off_next, off_meta, meta_stride, meta_sb_off, off_ring, ring_stride, total;
};

inline Layout make_layout(const am_config &c)
{
    Layout L{};
    L.ntiles = (uint32_t)((c.n + am::kTileCoords - 1) / am::kTileCoords);
    L.nsb = (L.ntiles + am::kTilesPerSuperblock - 1) / am::kTilesPerSuperblock;
    L.slots = c.delay + 1;
    L.blocks = block_geometry(c.replicas);
    const uint64_t all = (uint64_t)L.ntiles * (am::kTileCoords * L.blocks.rb / am::kLineFloats);
    L.cap_lines = c.ring_cap_lines ? std::min<uint64_t>(c.ring_cap_lines, all)
                                   : slot_capacity_lines(L.ntiles, c.fraction, L.blocks.rb, c.subset_granule == 32,
                                                         c.subset_kind == AM_SUBSET_STRATIFIED ? stratified_block(c.fraction) : 0);
    L.off_flags = 0;
    L.off_reduce = 256;
    L.off_next = L.off_reduce + kReduceBytes;
    L.off_meta = L.off_next + round_up((uint64_t)L.ntiles * 4, 256);
    L.meta_sb_off = round_up((uint64_t)L.ntiles * 4, 256);
    L.meta_stride = L.meta_sb_off + round_up(((uint64_t)L.nsb + 1) * 4, 256);
    L.off_ring = L.off_meta + L.meta_stride * (L.slots + 1);
    L.ring_stride = round_up(L.cap_lines * am::kLineFloats * L.blocks.nblocks * 4, 256);
    L.total = L.off_ring + L.ring_stride * L.slots;
    return L;
}

// How a subset's index list is cut: a part = one workgroup of four waves with `strips` strips each; waves: of a compute unit, of which the
// kernel's registers keep 20 resident.  Coordinates drawn one by one and written lane by lane: 20 waves, one round, up to eight strips a wave (20 / 40 waves,
// p = 5 %: 16M 14.2 / 17.1 us, 31.5M, p = 10 % 24.5 / 25.3, 60M 35.3 / 35.6); beyond, two rounds let the second's hashing run beside the
// first's stores (125.8M 62.7 / 60.5).  Whole lines and stratified subsets (the general form of the generator) and strips written row by row have more
// to hide behind each other: 32 waves, but 20 where at most two strips a wave are left to cut (not the smallest stratified subsets).  us, 20 / 32 waves: whole
// lines, p = 5 % 12M 17.7 / 20.3, 16M 21.1 / 22.4, 32M 33.5 / 32.8, 48M 45.7 / 42.7, 63M 57.3 / 52.2; stratified, p = 1 % 14M 24.8 / 23.8, 5 % 16M 25.9 / 26.6, 32M 44.9 / 43.0, 63M 85.9 / 76.5, 100M 119 / 109;
// row by row, whole lines, p = 25 % 12M 19.5 / 17.7, 24M 26.7 / 25.0, p = 100 % 24M 40.1 / 38.5, 48M 89.0 / 83.8, one by one, p = 25 % 32M 37.2 / 36.8, 60M 61.3 / 61.3, p = 100 % 24M
// 42.0 / 37.9, 60M 105 / 98.2.  A part waits only for earlier ones.  At most 32 strips (a kilobyte of masks in LDS each), from where on the
// parts grow in number.
// rows: a strip is written row by row.  Lane by lane / row by row, us: 130M 15 % 106 / 143, 20 % 132 / 144, 25 % 167 / 147,
// 50 % 313 / 155, 100 % 589 / 219; 17M 20 % 28.6 / 30.4, 25 % 33.6 / 31.0; 4M 20 % 13.9 / 13.8, 100 % 70 / 15.5; up to 2M,
// where little is written, 1M 30 % 11.2 / 11.8, 50 % 13.0 / 11.9, 100,003 40 % 9.4 / 9.8, 50 % 9.9 / 9.8.
struct ListShape {
    uint32_t nstrips, strips, parts;
    bool rows;
};

inline ListShape list_shape(const am_config &c, uint32_t compute_units)
{
    ListShape s;
    s.nstrips = (uint32_t)((c.n + am::kStripCoords - 1) / am::kStripCoords);
    s.rows = c.fraction >= (s.nstrips <= 1024u ? 0.45 : 0.22);
    const uint32_t cus = std::max(compute_units, 1u), resident = 20u * cus;
    const bool one_by_one = c.subset_kind != AM_SUBSET_STRATIFIED && c.subset_granule != 32;
    const uint32_t waves = one_by_one && !s.rows ? (s.nstrips > 8u * resident ? 2u * resident : resident)
                         : !s.rows && s.nstrips <= 2u * resident && (c.subset_granule == 32 || c.fraction >= 0.03) ? resident : 32u * cus;
    s.strips = std::min((s.nstrips + waves - 1u) / waves, 32u);
    s.parts = (s.nstrips + 4u * s.strips - 1u) / (4u * s.strips);
    return s;
}

// Whether the averaging-only call (with a delay) takes its ring values and interleaved EMA entries through LDS, am::kStageFloats of a block at a
// time (a turn), or reads them where they are used.  Staging hides the latency of scattered reads, but every turn after a tile's first
// waits once more.  Time staged / time direct on the same arrays, no limit of resident workgroups.
//
// Blocks of four and eight replicas, whose members' values change hands through LDS, are faster staged, except where a tile takes several turns
// and everything the call touches lies in the caches; sizes here in weights including the slots of absent replicas.
//   interleaved, R = 8, 20 % 0.2M 1.00, 3M 0.97, 8M 1.00, 16M 0.82; R = 5 25 % 5M 1.07; 30 % 2M 1.11, 5M 1.08, 6.5M 0.86, 16M 0.77; 50 % 2M 1.28, 5M 1.06, 6.5M 0.73; 100 % 2M 1.44, 3M 1.21, 4M 0.94, 5M 0.79;
//     R = 12 30 % 3M 1.01, 50 % 3M 1.19, 4M 1.02, 5M 1.00, 100 % 3M 1.20, 4M 0.67; R = 20 50 % 2M 1.06, 3M 1.00; R = 4 40 % 2M 1.01, 50 % 2M 1.11, 3M 1.03, 4M 0.97; 10 % 4M 0.84, 7M 1.05, 9.5M 0.95, 25 % 4M 0.95, 5.5M 1.11, 7M 1.07, 9.5M 0.91.
//   per replica, R = 8, 20 % 2M 1.01, 30 % 5M 1.14, 6.5M 0.99, 100 % 5M 1.12, 8M 0.83; R = 5 50 % 6.4M 1.10, 13M 1.04; R = 12 40 % 5M 1.17, 6.5M 1.10, 10M 0.85; R = 32 40 % 3M 1.06, 4M 0.94; R = 4 50 %
//     4M 1.08, 5M 1.02, 6.5M 0.92; 5 % 4M 0.85, 5.5M 1.08, 7M 1.15, 9.5M 1.00, 25 % 4M 0.99, 5.5M 1.16, 7M 1.14, 9.5M 0.96.
//   E4M3, interleaved R = 12 50 % 4M 1.15, 5M 1.11, 6.5M 0.98, 100 % 4M 0.91; R = 8 70 % 5M 1.15, 6.5M 0.77.
//   members in whole lines, interleaved R = 8 8 % 2M 0.99, 10 % 1.05, 30 % 5M 1.27, 6.5M 1.00, 16M 0.54; R = 12 15 % 2M 1.04, 30 % 5M 1.17, R = 16 25 % 6M 1.11, R = 12 70 % 3M 1.32, 4M 0.98; R = 4 15 % 2M 1.03, 40 % 5M 1.04;
//     per replica R = 8 8 % 2M 1.02, 20 % 8M 1.13, 10M 0.89, 70 % 6.5M 1.06, 8M 0.95; R = 20 20 % 8M 1.07, 10M 0.80; R = 4 30 % 6.5M 1.06, 50 % 5M 1.13, 70 % 0.99.
//   no correction, R = 8 10 % 8M 0.96, 25 % 3M 1.11, 8M 1.14, 24M 1.02, 40M 0.92, 50 % 8M 1.27, 24M 1.04, 40M 0.99, 100 % 8M 1.11, 11M 1.01, 13M 0.97; R = 5 50 % 24M 1.12, 37M 1.05, 120M 0.95, 100 % 64M 0.96, 128M 1.02, 200M 1.06; R = 12 25 % 4M 1.01, 7M 1.16, 9.5M 0.82, 13M 0.96, 50 % 13M 1.02, 24M
//     0.98, 100 % 5.5M 1.21, 7M 0.67; R = 20 35 % 5.5M 1.14, 8M 0.99, 100 % 3M 1.16, 4M 0.71; R = 4 25 % 4M 0.99, 7M 1.13, 9.5M 1.04, 18M 0.91, 35 % 4M 1.06, 5.5M 1.01, 50 % 4M 1.15, 5.5M 0.98; whole lines R = 8 10 % 8M 1.14, 11M 0.91, 50 % 16M 1.14,
//     24M 1.04, R = 5 1.09, 100 % 11M 1.01, 13M 0.98.
// Blocks of one and two replicas have nothing to hand over: per-replica EMA vectors are dense reads in both forms, and the staged one gains with half a
// turn at most, or at every fraction where the weights come from memory (11M R = 1 and 2 25 % 0.86 to 0.95, 100 % 0.80 to 0.91); interleaved
// ones with one turn, where the weights come from memory, and for nearly whole tiles.
inline bool average_staged(const am_config &c, uint32_t ntiles, const Blocks &b, bool interleaved_d)
{
    const bool by_line = c.subset_granule == 32, e4m3 = c.msg_dtype == AM_MSG_E4M3;
    if (b.rb >= 4u) {
        const bool wide = b.rb == 8u, one = wide && b.nblocks == 1u;
        double few, small;                                 // staged up to this fraction; beyond, from this many millions of weights (with absent slots) on
        if (c.correction == AM_CORR_NONE) {                // half of what the caches would have to hold, and less to wait for
            few = by_line ? (!wide ? 0.12 : b.nblocks <= 2u ? 0.09 : 0.2) : !wide || b.nblocks > 2u ? 0.3 : one ? 0.17 : 0.2;
            if (one) small = c.fraction > 0.8 ? 11.0 : by_line && c.fraction <= 0.2 ? 8.5 : !by_line && c.replicas <= 6u && c.fraction <= 0.6 ? 45.0 : 26.0;
            else if (wide && b.nblocks == 2u) small = c.fraction > 0.8 ? 5.7 : c.fraction > 0.6 ? (by_line ? 6.0 : 11.0) : c.fraction <= (by_line ? 0.2 : 0.4) ? 8.5 : 17.0;
            else if (wide) small = c.fraction > 0.8 ? 3.5 : 5.7;
            else small = !by_line ? 4.2 : c.fraction <= 0.4 ? 8.5 : c.fraction <= 0.6 ? 5.7 : 4.2;
        } else {
            few = by_line ? (one ? 0.09 : b.nblocks > 2u ? 0.2 : wide ? 0.12 : 0.15) : !wide ? 0.45 : b.nblocks <= 2u ? 0.22 : 0.35;
            if (interleaved_d) {
                small = by_line && b.nblocks == 2u ? 6.2 : by_line || (wide && (one || e4m3)) ? 5.3 : wide ? 3.5 : 3.0;
                if (c.fraction > (by_line && !one ? 0.55 : 0.8)) small = std::min(small, 3.5);
            } else {
                small = by_line ? (wide && b.nblocks <= 3u ? 8.4 : 5.2) : one ? 6.8 : !wide ? 4.2 : b.nblocks <= 2u || e4m3 ? 6.0 : b.nblocks == 3u ? 5.2 : 3.5;
                if (by_line && c.fraction > 0.5) small = one ? 6.6 : wide && b.nblocks <= 3u ? 5.4 : 4.2;
                if (c.fraction > 0.8 && b.nblocks >= 3u && !e4m3) small = 3.5;
            }
        }
        const double slots = (double)c.n * b.rb * b.nblocks / 1e6;
        // blocks of four with most of a tile's values in one turn: in place where the caches hold what is in place, but not what is staged besides
        if (!wide && !by_line && c.fraction <= few && c.fraction > (c.correction == AM_CORR_NONE ? 0.15 : interleaved_d ? 0.08 : 0.03))
            return slots <= 4.7 || slots > (c.correction == AM_CORR_NONE ? 10.0 : 8.5);
        if (c.correction == AM_CORR_NONE && one && c.replicas <= 6u && c.fraction > 0.85 && slots > 110.0) return false;   // (absent slots' values pass through LDS, too)
        return c.fraction <= few || slots > small;
    }
    const double drawn = c.fraction * am::kTileCoords, turn = (double)am::kStageFloats / b.rb;     // members of a tile, and those a turn holds
    if (!interleaved_d) return drawn <= 0.5 * turn || (!by_line && c.msg_dtype == AM_MSG_F32 && ntiles > 24576u);
    const double members = by_line ? std::max(drawn, (double)am::kLineFloats) : drawn;             // of a tile that receives
    if (members + 1.5 * std::sqrt(members * (1.0 - c.fraction)) <= turn) return true;
    if (ntiles > 12288u || c.n * c.replicas > 1ull << 25) return true;
    return c.fraction > (c.msg_dtype != AM_MSG_F32 ? 0.75 : 0.5) && (ntiles > 3072u || c.n * c.replicas >= 6000000u);
}

// Whether a step's arrays come from memory each time (20 to 36 bytes a parameter and replica; half of the 256 MB that the caches hold
// survives to the next call).  Stores through to memory / with the non-temporal hint alone, us a step: R = 8 125.8M 5834 / 5882, 31.5M 1799 / 1816,
// R = 4 7.1M 171.7 / 174.5, R = 2 30M SGD 287.7 / 295.4, 3M SGD 23.2 / 23.9; R = 4 1M 31.7 / 31.4, 500k 17.8 / 17.0.
inline bool beyond_caches(const am_config &c) { return c.n * c.replicas > 5ull << 20; }

// Kilobytes that a step reads and writes of one replica's part of a tile: weights, gradient, moments, forward copy and, where it receives, the EMA
// entries (whole lines are read, halves written) and the ring.
inline double step_kilobytes(const am_config &c, const Blocks &b, bool forward_copy, bool receives)
{
    const double moments = c.optimizer != AM_OPT_SGD ? 2.0 : c.beta1 != 0.f ? 1.0 : 0.0;
    double kb = 2.0 + (c.grad_dtype == AM_BF16 ? 0.5 : 1.0) + 2.0 * moments + (forward_copy ? (c.fwd_dtype == AM_BF16 ? 0.5 : 1.0) : 0.0);
    if (!receives) return kb;
    kb += 2.0 * c.fraction;
    if (c.correction != AM_CORR_NONE) {
        const double line = c.d_layout == AM_D_INTERLEAVED ? (double)am::kLineFloats / b.rb : am::kLineFloats;      // coordinates of one
        kb += 2.0 - std::pow(1.0 - c.fraction, line) - std::pow(1.0 - c.fraction, line / 2.0);
    }
    return kb;
}

// Workgroups (a wave per replica of a block) of the fused step that a compute unit may hold at a time; 0: as many as fit.  The stream mix moves
// fastest with few requests on their way (without arithmetic, 125.8M x 8: 16 waves a compute unit 6.05 to 6.3 TB/s, 24 5.5 to 6.1); fewer leave the
// step's chain of waits visible, and a wave that moves less has less on its way.  So the limit follows what the step moves, and is there only for
// whole blocks of two and four replicas.  Time with the limit / without, same arrays, 16M, 28M, 64M and 160M parameters x replicas, p = 5 %:
//   R = 4, 5: per replica, AdamW with forward copy (9.5 KB) 0.96 0.96 0.98 1.02, without (8.5) 0.98 0.96 0.98 0.97, bf16 gradient (8.0) 0.98 0.97 0.98 0.98, SGD with
//     momentum (6.5) 16M 0.98, 31M 0.98, 80M 0.98, without (4.5) 1.15, 1.18; interleaved, AdamW with forward copy (8.6) 0.99 0.99 1.00 1.02, without (7.6) 1.02 1.01
//     1.02 0.99, there 6: 1.01 1.01 1.00 0.99, bf16 gradient (7.1) 6: 1.02 1.02 1.01 0.99, SGD 5: 1.03 to 1.17; no correction (8.1) 6: 0.99 0.99 0.99 1.00.
//   R = 2, 11: per replica with forward copy 0.96 0.96 0.95 0.99, without 0.95 0.96 0.97 0.97, bf16 gradient 0.96 0.98 0.99 0.97; interleaved with forward copy 0.98
//     0.99 1.00 0.97, without 1.02 1.02 1.05 0.98, bf16 gradient 1.00 1.02 1.03 0.97; no correction with 0.97 0.98 0.97 0.99, without 1.00 1.01 1.01 1.00.
//   R = 3, 5: AdamW 16M 1.02 to 1.08, SGD 1.21; 6: 1.00 to 1.03, 1.09.  R = 1, 25 (one wave each): AdamW 0.97 to 1.03, SGD 1.05.  R = 8, 2: 1.02 to 1.15.
// (Small stages that add up their offsets themselves take no limit: R = 4 6M, 5: AdamW 1.00 to 1.03, SGD 1.10 to 1.22.)
inline uint32_t step_workgroups(const am_config &c, const Blocks &b, bool forward_copy, bool receives)
{
    if (!beyond_caches(c)) return 0;
    const double kb = step_kilobytes(c, b, forward_copy, receives);
    const bool dense_d = receives && c.correction != AM_CORR_NONE && c.d_layout != AM_D_INTERLEAVED;
    if (c.replicas == 4u) return kb >= (dense_d ? 6.4 : 8.2) ? 5u : kb >= 7.2 ? 6u : 0u;
    if (c.replicas == 2u) return (dense_d ? kb >= 7.4 : forward_copy && c.grad_dtype != AM_BF16 && kb >= 8.0) ? 11u : 0u;
    return 0;
}

// The fused step adds up its tiles' places itself on stages of at most this many tiles (and what its waves can add up), and no launch precedes
// it; sync: no delay.  Every workgroup does it, so with more blocks, or more waves a tile (no delay), it pays on fewer tiles.  Time added up / offsets launched:
// R = 4 AdamW interleaved 100,003 0.77, 480k 0.85, 1M 0.94, 1.6M 1.00, SGD 1.3M 0.97, 1.6M 1.08; R = 3 1.6M 0.97, 2M 1.08; R = 2 2M 0.94; R = 8 1M 0.96, 2M 0.98; R = 12 1M 0.98,
// 2M 1.00.  R = 20 250k AdamW 1.02, SGD 0.91, 480k 1.03, 0.94, 1.5M 1.13, p = 100 % 700k 1.10, 1.4M 1.14; R = 24 480k 0.99, 0.96; R = 32 150k 0.98, 0.99, 250k 1.01,
// 1.04, 740k 1.13.  No delay: R = 8 2M 0.98; R = 5 plain SGD 1M 0.99, 1.3M 1.02, 1.6M 1.05, 2M 1.07, AdamW 2M 0.99; SGD and AdamW R = 9 250k 0.90, 400k 0.96, 480k 1.00, 650k 0.97 to 1.00, 1M 1.05; R = 12 250k 0.91, 300k 0.95, 600k 0.96 to 1.02, 2M 1.07; R = 16 250k 0.93, 300k 0.95, 400k to
// 650k 0.97, 1M 0.97 to 1.02, 1.3M 1.07; R = 13 and 14 300k 1.05, 450k 1.03 and 1.06, 650k 1.03 and 1.05; R = 20 and more 0.96 to 1.00.
inline uint32_t step_sum_tiles(const am_config &c, const Blocks &b, bool sync)
{
    if (sync && c.replicas > 8u && c.replicas <= 16u) return c.replicas == 13u || c.replicas == 14u ? 1024u : 2560u;
    if (sync) return c.replicas >= 5u && c.replicas <= 7u && c.optimizer == AM_OPT_SGD && c.beta1 == 0.f ? 4608u : 8192u;
    return b.nblocks == 4u ? 768u : b.nblocks == 3u ? 2048u : b.rb == 4u ? 6144u : 8192u;
}

// Whether a step with a delay goes through the kernel of one-wave workgroups instead of the fused kernel's workgroup per tile and block.  Time by
// waves / by the fused kernel, same arrays, median of three to eight placements of the arrays on one to three cards, AdamW with look-ahead and 5 % where not said (a single placement is off the median by up to 5 %; most of these arrays were freed
// and allocated again in one process: where a process allocates them once, R = 8 gains 2.5 % interleaved, 6.5 % per replica, 4.5 % in bf16 without correction, R = 12 4 %):
//   weights (n R)                                45M   60M   90M   130M  200M  300M  400M  500M  1000M
//   interleaved EMA vectors   R = 6              0.97  0.98  0.97  1.00  0.98        0.98
//                             8                  0.97  0.97  0.97  0.97  0.96  0.97  0.96  0.96  0.96
//                             12                 0.97  0.95  0.97  0.97  0.98  0.97  0.96  0.97  0.98
//                             14                 0.97  0.97  0.99  0.99  0.98        0.97
//                             18                 0.92  0.91  0.90  0.91  0.91        0.91
//     few absent slots        16                 1.02  0.95  0.98  0.99  0.99  1.00  0.98  0.99  1.02
//                             20                 1.01  0.98  0.95  0.97  0.97        0.98
//                             22                 1.02  1.01  0.95  0.98  0.99        0.99
//                             24                 0.97  0.99  0.97  0.99  0.99  0.99  0.99  0.99  1.00
//     SGD with momentum, R = 8 0.98, but 16 1.00; 6 % 8 0.98, 12 0.96 to 0.97, but 20 0.98 to 0.99, 22 1.00 to 1.01, 24 0.99 to 1.02; 10 % 1.00 to 1.04; 1 and 2 % 8 and 12 0.94 to 0.97, 16 0.94 to 0.96, 20 0.95 to 0.97.
//     R = 32 0.93 to 1.04, R = 7 0.99 to 1.03 (one placement).
//   per replica               7                  0.94  0.94  0.94  0.96  0.94  0.94
//                             8                  0.95  0.95  0.96  0.98  0.97  0.97
//                             13, 15             0.96  0.94  0.97  0.96  0.95  0.95
//                             12, 16             0.93  0.93  0.94  0.95  0.94  0.94
//                             23                 0.96  0.99  0.94  0.96  0.98  0.95
//                             32                 0.96  0.93  0.96  0.92  0.95  0.95
//                             31                 0.99              0.95        0.99
//   no correction (70M first) 7, 8                     0.95        0.95  0.95  0.95        0.95
//                             15                       0.96        0.98  0.95  0.97        0.98
//                             16, 32                   0.95        0.94  0.95  0.95        0.97
//                             13, 23                   0.97        0.98        0.97
//                             31                       0.98        1.00        1.03
//     17, 19, 25 0.87 to 0.95; 10 % (60M, 250M) per replica 7, 8, 16 0.92 to 0.98, 31 1.03, no correction 0.95 to 0.99, 31 1.06; one placement: 15 % 1.09, 20 % 1.08, 30 % 1.23.
//   three tenths or more of the fused kernel's waves absent: R = 9 0.78 to 0.84 (10 % 0.79 to 0.93), 10 0.82 to 0.87 (0.85 to 0.93), 11 per replica 0.90 (0.90 to 0.94), interleaved 0.94 to 0.97, 6 % 0.96, 7 % 0.99, 8 % 1.01, 10 % 1.06;
//     5 per replica 0.92 to 0.96 (0.95 to 0.99), interleaved 15M 0.97, 45M 0.98, 130M 1.00, 300M 0.99, 2 % 0.95, 6 % 1.00, 8 % 1.03, 10 % 1.06 (13M to 18M 1.06, too).
//   types and kinds, R = 8 and 12 (60M, 250M): bf16 0.90 to 0.98, without a forward copy 0.89 to 0.98, SGD with momentum 0.88 to 0.99, plain 0.72 to 0.91, members in whole lines 0.95 to 0.99, stratified 0.93 to 0.98, messages in bf16
//     0.91 to 0.98, E4M3 0.90 to 0.97.
//   fewer weights (one placement): interleaved 15M 0.99 to 1.05, 25M 0.98 to 1.05, per replica 20M and 30M 0.99 to 1.03, no correction 30M 1.04.
inline bool step_by_waves(const am_config &c, const Blocks &b)
{
    if (b.rb != 8u || c.fraction > 0.1) return false;
    const uint64_t weights = c.n * c.replicas;
    const uint32_t slots = 8u * b.nblocks, absent = slots - c.replicas;
    const bool idle = 10u * absent >= 3u * slots, odd = c.replicas % 2u != 0u;             // (R = 5, 9, 10 and 11)
    if (odd && c.replicas > 25u) return false;
    if (c.correction == AM_CORR_NONE || c.d_layout != AM_D_INTERLEAVED)
        return weights > (idle ? 3ull << 22 : c.correction != AM_CORR_NONE ? 5ull << 23 : 1ull << 26);
    if (c.replicas == 5u && weights > 1ull << 24) return c.fraction <= (weights > 1ull << 26 ? 0.03 : 0.05);
    if (c.replicas == 11u && c.fraction > 0.06) return false;
    if (idle) return weights > 3ull << 22;
    if (odd || c.replicas > 24u || c.fraction > 0.06) return false;
    if (c.replicas >= 16u && 5u * absent < slots)
        return weights > (c.replicas == 16u ? 3ull << 24 : 1ull << 26) && weights <= 1ull << 29 && c.fraction <= 0.05 && !(c.optimizer == AM_OPT_SGD && c.beta1 != 0.f);
    return weights > 5ull << 23;
}

// Replicas that a wave of that kernel takes: two share the hashing and send pairs of values (R = 12 10M 0.96 either way, R = 32 4M 0.98 / 0.965; four, interleaved 125.8M x 8, 1.005
// of the fused kernel's time, one 1.01, two 0.98).
inline uint32_t wave_step_replicas(const am_config &c) { return c.replicas % 2u ? 1u : 2u; }

// Its grid: the tiles of a chunk and the tile's waves in x, the chunks in y, and past 32768 chunks (2^30 coordinates) in z, too: neither of those may pass 65535, and
// a stage has up to 131,040 chunks.
struct Grid { uint32_t x, y, z; };
inline Grid wave_step_grid(uint32_t ntiles, uint32_t waves_of_a_tile)
{
    const uint32_t chunks = (ntiles + am::kWaveChunk - 1u) / am::kWaveChunk, y = std::min(chunks, 32768u);
    return {am::kWaveChunk * waves_of_a_tile, y, (chunks + y - 1u) / y};
}

// Waves of it that a compute unit may hold at most: the less a wave moves the more of them, and one more where the step is short.  (LDS comes in shares, by which 8 to 12, 14, 16, 18, 21, 25 and 32 can
// be held to: a bound of 13 holds 12, of 15 14, of 17 16, of 19 and 20 18, of 22 to 24 21.)  Time over the fused kernel's by the number resident, median of three placements of the arrays,
// * what the bound holds; two replicas a wave: AdamW interleaved 250M weights (8.4 KB a replica) 8: 0.969, 9: 0.964, 10: 0.967*, 11: 0.974, 14: 0.992, 60M 9: 0.966, 10: 0.964, 11: 0.967*, 14: 0.980; per
// replica (9.5 KB) 250M 8: 0.929, 9: 0.933*, 10: 0.942, 14: 0.977, 60M 8: 0.925, 10: 0.936*; interleaved without a forward copy (7.4 KB) 250M 8: 1.000, 10: 0.974, 11: 0.980*; bf16 without correction (7.0 KB) 250M
// 8: 0.973, 10: 0.940, 11: 0.943*, 14: 0.956; SGD with momentum, interleaved (5.4 KB) 60M 8: 1.135, 10: 1.024, 12: 0.991, 14: 0.981*, 250M 10: 0.996, 11: 0.989, 12: 0.994*, 14: 1.008; plain SGD, interleaved
// (3.4 KB) 250M 8: 1.412, 12: 1.037, 16: 0.887, 18: 0.884*, 21: 0.889, without correction (3.1 KB) 16: 0.939, 18: 0.905, 21: 0.875*.  One replica a wave: AdamW R = 7 250M 8: 1.178, 12: 0.939, 14: 0.935, 18: 0.955*, 21: 0.964,
// R = 5 interleaved 60M 12: 1.013, 16: 0.969, 21: 0.981*.
inline uint32_t wave_step_workgroups(const am_config &c, const Blocks &b, uint32_t v, bool forward_copy, bool receives)
{
    const double pairs = (c.n * c.replicas > 1ull << 27 ? 4.0 : 5.0) + 50.0 / step_kilobytes(c, b, forward_copy, receives);
    return (uint32_t)std::floor(pairs * 2.0 / v + 0.5);
}

// Whether a step between two averaging rounds (which neither sends nor receives) goes through the kernel of its own.  It pays for blocks of
// eight waves; the kernel change costs the round's step some microseconds of cold instructions, which every second or third step feels on larger
// stages than every fourth, and full blocks more than those whose absent slots idle.  Time by its own / by the fused kernel on average over rounds, by weights (n R):
//   K = 2 R = 8 AdamW 1.1M 1.19, 1.6M 1.04, 3M 1.04, 6M 1.03, 10M 0.97, momentum 2.2M to 4M 1.08, 8M 1.02, 10M 0.97, bf16 gradients 1.1M 1.24; R = 12 and 16 2M to 4M 1.07 to 1.10, 10M 0.99;
//     R = 5 1.1M 1.10, 2.6M and more 0.99, plain SGD 0.90;  K = 3 R = 8 2M to 4M 1.03 to 1.07, 8M 0.99;  K = 4 and 5 0.80 to 1.00 from 1.1M on.
// us a step: AdamW R = 8 K = 2 15M 575.7 / 571.7 (fused / its own), but R = 4 K = 4 6M 111.5 / 114.3, SGD R = 4 15M K = 2 203.0 / 205.7, R = 2 15M K = 4 100.2 / 102.7.
inline bool local_step_alone(const am_config &c, const Blocks &b)
{
    if (b.rb != 8u) return false;
    const bool light = c.replicas <= 6u || (c.optimizer == AM_OPT_SGD && c.beta1 == 0.f);
    return c.n * c.replicas > (c.avg_interval >= 4u ? 1ull << 20 : light ? 5ull << 19 : 6ull << 20);
}

// The workgroups (four tiles of one replica) of that kernel that a compute unit may hold at a time: some 60 KB of requested operands a compute
// unit.  us a step by their number: AdamW 30M R = 8 as many as fit 1346, 3: 1285, 4: 1215, 5: 1260, 3M R = 8 135.8, 136.3, 126.8, 131.2; SGD with
// momentum 30M R = 2 199.3, 211.5, 192.2, 190.7.  Plain SGD, which reads two streams: as many as fit.
inline uint32_t local_step_workgroups(const am_config &c)
{
    if (!beyond_caches(c) || (c.optimizer == AM_OPT_SGD && c.beta1 == 0.f)) return 0;
    return c.optimizer == AM_OPT_SGD ? 5u : 4u;
}

// Whether the averaging-only kernel finds the replicas' weights in a table, a block's pointers in one line of the kernel's arguments, or in the
// replicas' records, a line each.  The lines are cold at every launch, which calls below 10M weights feel (0.82 to 0.95 of the time with a table), and it makes no difference
// on large stages; but with a table the requests of a wave's eight replicas leave closer together, which stages at the edge of the caches do not like where they
// ask for much at a time.  Time table / records, by weights (n R): staged EMA entries, R = 8 5 % 4M 0.92, 7M 1.07, 9.5M 1.06, 13M 0.99, R = 16 5 % 4M 0.91, 7M 1.12, 9.5M 1.14, 13M 0.98;
// 0.2 % 4M 0.88, 7M 0.97, 9.5M 1.01.  No delay, R = 8 interleaved 100 % 4M 0.99, 7M 1.11, 13M 1.13, 18M 1.10, 26M 1.04, 50 % 7M 1.25, 9.5M 1.04; 25 % 7M 1.01; but R = 16 50 % 4M 0.89, 7M 0.93,
// 13M 1.02.  No correction R = 8 50 % 7M 1.20, 13M 1.11, 25 % 0.98; R = 12 50 % 7M 0.97, 13M 0.96; R = 16 50 % 1.11, 1.03, 100 % 0.88, 0.96.  Members in whole lines 0.90 to 1.00.  Blocks of four: 1M 0.90 / 0.91
// of the code before both, the table always.
inline bool average_weights_table(const am_config &c, const Blocks &b)
{
    const uint64_t weights = c.n * c.replicas;
    if (b.rb != 8u || c.subset_granule == 32 || weights <= 5ull << 20 || weights > 20ull << 20 || c.fraction <= 0.02) return true;
    if (c.delay == 0 || c.correction == AM_CORR_NONE) return b.nblocks > 1u || c.fraction <= 0.4;
    return weights > 23ull << 19;
}

// Workgroups (of four tiles, a wave each) of the staged averaging-only call that a compute unit may hold at a time; 0: as many as
// fit.  Where the weights come from memory (more than the 256 MB cache holds) it is fastest with some 114 KB of lines a compute
// unit on their way; with more the streams get in each other's way, as in the fused step, with fewer latency shows.  So the number
// follows from the lines that a wave reads.  But where a tile takes several turns, messages are rounded or the caches still help, latency is the
// cost: then not fewer than three or four (R = 2 interleaved seven; three with absent replicas); without a correction a wave has less to wait for (130 KB, none where most coordinates are drawn), and members
// in whole lines are not limited (interleaved, 80M, p = 40 % R = 8 3: 1.24, R = 4 4: 1.16, R = 12 3: 1.19).  Blocks of eight without interleaved EMA entries
// that take several turns: none either, but for EMA vectors of more than 200M weights.
// us a call by workgroups a compute unit, * the one chosen: interleaved, R = 8, 125.8M 5 % 2: 1711, 3: 1574*, 4: 1631, 8: 1675; 1 % 3: 1030, 5: 717, 6: 655, as many as
// fit 636*.  Time over as many as fit, 250M weights (80M in brackets): interleaved R = 8 2 % 4: 0.96*, 3: 1.12; 5 % 3: 0.93*, 2: 0.99; 10 % 2: 0.94* (1.13, 3: 1.00*);
// 40 % 2: 0.97*; 80 % 4: 0.99*, 2: 1.14; 100 % 4: 0.95*, 2: 1.31; R = 5 5 % 4: 0.91*, 5: 0.99; 10 % 3: 0.92*, 4: 0.98 (2: 1.18); 40 % 3: 0.96*, 2: 1.05; R = 12 10 % 3: 0.96*, 20 % 2: 0.96* (3: 0.98*);
// R = 4 5 % 4: 0.92, 5: 0.96*; 40 % 3: 0.93*; 100 % 4: 0.93*, 2: 1.33; R = 20 20 % 2: 0.89* (160M 0.93, 3: 0.98*).  Per replica R = 8 5 % 2: 0.90* (3: 0.98*), 2 % 3: 0.95*; R = 5 5 % 3: 0.87*;
// R = 4 5 % 4: 0.93*, 10 % 3: 0.93*, 100 % 4: 0.89*, 2: 1.29; R = 3 5 % 4: 0.92*, 100 % 4: 0.97*, 2: 1.56.  No correction R = 8 5 % 4: 0.92*, R = 12 5: 1.01*, 4: 1.04;
// R = 4 40 % 5: 0.91*, R = 3 80 % 5: 1.20.  E4M3 interleaved R = 8 10 % 5: 1.00 (2: 1.26), R = 5 20 % 4: 0.99* (2: 1.10), R = 12 5 % 4: 0.94, 3: 1.01 (1.16); R = 20 and 32 5 % 4: 0.93 to 1.07, 3: 1.03 to 1.22.
// R = 2 interleaved, 103M 40 % 6: 0.95*, 5: 0.95, 50 % 7: 1.01*, 6: 1.05, 5: 1.12, 70 % 7: 0.99*, 6: 1.02, 100 % 7: 0.98*, 6: 0.98, 5: 1.04, R = 3 per replica 20 % 3: 1.05, 4: 0.98*.  Several turns of eight, per replica, 120M, R = 12 25 % 3: 1.03, 50 % 1.04, R = 5 25 % 1.00,
// 50 % 1.18; 220M R = 12 25 % 3: 0.95*, 50 % 0.97*, R = 5 25 % 0.91*, 50 % 4: 0.98*, R = 16 50 % 3: 0.92*, R = 8 100 % 4: 0.98*; no correction, 120M R = 8 25 % 4: 1.03, 3: 1.20, 50 % 1.08, 1.27, R = 12 25 % 1.05, 1.21.
inline uint32_t average_workgroups(const am_config &c, const Blocks &b, bool interleaved_d)
{
    const uint64_t weights = c.n * c.replicas;
    const bool ema = c.correction != AM_CORR_NONE, e4m3 = c.msg_dtype == AM_MSG_E4M3, wide = b.rb == 8u;
    if (weights <= 1ull << 26 || c.subset_granule == 32 || (!ema && c.fraction > 0.5) || (e4m3 && b.nblocks > 2u)) return 0;
    const bool turns = wide && !interleaved_d && c.fraction > 0.125;               // (more than one a tile)
    if (turns) return ema && c.msg_dtype == AM_MSG_F32 && weights > 3ull << 26 ? (c.replicas <= 6u || c.fraction > 0.7 ? 4u : 3u) : 0u;
    auto touched = [&](double coordinates) { return 1.0 - std::pow(1.0 - c.fraction, coordinates); };
    double kb = touched(2.0 * am::kLineFloats) + c.fraction * b.nblocks;           // of each replica: weights sent or received, ring values
    if (ema) kb += touched(interleaved_d ? (double)am::kLineFloats / b.rb : am::kLineFloats);
    const double replicas = wide ? (double)c.replicas / b.nblocks : b.rb;          // of a wave
    const bool absent = wide && c.replicas <= 6u;                                  // (slots of the block that ask for nothing)
    const double on_the_way = !wide ? 114.0 : !ema ? 130.0 : e4m3 ? 150.0 : absent ? 100.0 : 114.0;
    const double workgroups = std::floor(on_the_way / 4.0 / (kb * replicas) + 0.5);
    if (workgroups >= (absent ? 6.0 : 7.0)) return 0;
    uint32_t least = 2;
    if (c.msg_dtype != AM_MSG_F32 || c.fraction > 0.5 || weights <= 3ull << 25 || (b.nblocks > 2u && weights <= 3ull << 26)) least = 3;
    if (e4m3 || (b.nblocks == 1u && c.fraction > 0.7) || (c.replicas == 3u && !interleaved_d)) least = 4;
    if (absent) least = std::max(least, 3u);
    if (c.replicas == 2u && interleaved_d && c.fraction > 0.45) least = 7;
    return std::max(least, (uint32_t)workgroups);
}

// Dynamic LDS of a workgroup that needs `need` bytes besides `fixed` bytes of static LDS, with which a compute unit holds at most `workgroups` of them (0: no limit):
// the smallest allocation of which one more does not fit.  (1 to 12, 14, 16, 18, 21, 25 and 32 fit exactly.)
constexpr uint32_t kLdsGranules = am::kLdsBytes / am::kLdsGranule;
constexpr uint32_t lds_for_residency(uint32_t need, uint32_t workgroups, uint32_t fixed = 0)
{
    if (workgroups == 0u) return need;
    const uint32_t share = (kLdsGranules / (workgroups + 1u) + 1u) * am::kLdsGranule - fixed;
    return need > share ? need : share;
}
constexpr bool residency_is_exact(uint32_t workgroups)
{
    const uint32_t granules = (lds_for_residency(1, workgroups) + am::kLdsGranule - 1u) / am::kLdsGranule;
    return workgroups * granules <= kLdsGranules && (workgroups + 1u) * granules > kLdsGranules;
}
// How many it holds: the largest number that is exact and not above `workgroups`.
constexpr uint32_t workgroups_held(uint32_t workgroups)
{
    while (workgroups > 1u && !residency_is_exact(workgroups)) --workgroups;
    return workgroups;
}
constexpr bool residency_holds(uint32_t workgroups)
{
    return kLdsGranules / ((lds_for_residency(1, workgroups) + am::kLdsGranule - 1u) / am::kLdsGranule) == workgroups_held(workgroups);
}
constexpr bool every_residency_holds()
{
    for (uint32_t w = 1; w <= 32u; ++w)
        if (!residency_holds(w)) return false;
    return true;
}
static_assert(every_residency_holds() && workgroups_held(7) == 7u && workgroups_held(11) == 11u && workgroups_held(13) == 12u && workgroups_held(20) == 18u,
              "as many as a rule names fit, or the next number below that shares of the LDS allow, and not one more");

// Floats of one array of the EMA vectors and how many arrays there are, per layout.
inline void d_layout_shape(const am_config &c, uint32_t *rb, uint32_t *arrays, uint64_t *floats)
{
    if (c.d_layout == AM_D_INTERLEAVED) {
        const Blocks b = block_geometry(c.replicas);
        *rb = b.rb; *arrays = b.nblocks;
        *floats = round_up(c.n, am::kTileCoords) * b.rb;
    } else {
        *rb = 1; *arrays = c.replicas; *floats = c.n;
    }
}

// What step t does to the ring: averaging happens at steps t with t mod K == 0 (round t / K); the
// round's values go to slot round mod (depth), depth = configured delay + 1; what was sent tau rounds
// ago (tau = the delay in force, <= the configured one) is received once t - tau K >= 1.
struct Round {
    bool send, recv, same_slot;
    uint32_t slot_send, slot_recv;
    uint64_t step_recv;
};

inline Round plan_round(uint64_t K, uint64_t depth, uint64_t tau, uint64_t t)
{
    Round r{};
    if (t % K != 0) return r;
    const uint64_t round = t / K;
    r.send = true;
    r.slot_send = (uint32_t)(round % depth);
    if (t >= tau * K + 1) {                       // s = t - tau K >= 1: something was sent that long ago
        r.recv = true;
        r.step_recv = t - tau * K;
        r.slot_recv = (uint32_t)((round - tau) % depth);
        r.same_slot = tau == 0;
    }
    return r;
}

// What a checkpoint record says about subsets that are already sized, and what a record is taken to say.
// A record names sizes only where every build has looked for them, in the words at off_next, which this one does not write: a
// record says that nothing is sized, unless it was resumed from one that names words (of step record_step) not yet used at the last step made, and the step
// after the resume hashes its subset once more and finds the same sizes.  Records whose reserved field is not zero (some named
// another table in its bit 0) count as not sized, too.
inline uint64_t record_sized_step(uint64_t record_step, uint64_t last_t) { return record_step > last_t ? record_step : 0; }
inline uint64_t resumed_sized_step(const am_snapshot &s) { return s.reserved ? 0 : s.next_lines_step; }

}  // namespace am_host
