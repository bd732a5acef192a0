// Kernels of the AsyncMesh stage update (gfx950).  All of them are bound by HBM bandwidth; none is a
// contraction, so none uses the matrix cores.
#pragma once
#include "am_device.h"

namespace am {

// =============================================================================================
// Where the tiles' lines start in a ring slot:  k_subset_count (sizes not known yet)  ->  k_subset_scan, or from
// known sizes  k_subset_offsets_at_once,  or  k_subset_offsets  ->  k_subset_scan,  or lines_before in the kernel itself
// =============================================================================================
// cnt[512] (LDS) holds the lines of the tiles of superblock blockIdx.x: write their exclusive
// prefix, with the tile's own lines in the high 8 bits (a tile owns at most 64 lines and a superblock
// at most 2^15), to local_off and their sum to *total.
// Called by all threads of the workgroup (256 or more) after a barrier.
__device__ __forceinline__ void scan_superblock(const uint32_t *cnt, uint32_t *wave_tot, uint32_t ntiles,
                                                uint32_t *__restrict__ local_off, uint32_t *__restrict__ total)
{
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const uint32_t tile0 = blockIdx.x * kTilesPerSuperblock;
    uint32_t a = 0, b = 0, incl = 0;
    if (wave < 4u) {                             // thread j owns entries 2j, 2j+1
        a = cnt[2 * threadIdx.x]; b = cnt[2 * threadIdx.x + 1];
        incl = a + b;                            // inclusive scan across the wave, by shuffles
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t up = __shfl_up(incl, off);
            if ((int)lane >= off) incl += up;
        }
        if (lane == 63) wave_tot[wave] = incl;
    }
    __syncthreads();
    if (wave >= 4u) return;
    uint32_t base = 0;
    for (uint32_t w = 0; w < wave; ++w) base += wave_tot[w];
    const uint32_t excl = base + incl - (a + b);
    const uint32_t t_a = tile0 + 2 * threadIdx.x;
    if (t_a < ntiles) local_off[t_a] = excl | (a << 24);
    if (t_a + 1 < ntiles) local_off[t_a + 1] = (excl + a) | (b << 24);
    if (threadIdx.x == 255) *total = base + incl;
}

// Which of the 32 consecutive coordinates of a lane (2048 strip + 32 lane + bit) are in the subset.
__device__ __forceinline__ uint32_t strip_mask(const SubsetKey &key, uint64_t n, uint32_t strip, uint32_t lane)
{
    const uint64_t mu0 = (uint64_t)strip * kStripCoords + lane * 32u;
    const bool whole = (uint64_t)(strip + 1u) * kStripCoords <= n;             // same for the whole wave
    uint32_t m = 0;
    if (whole && key.mode == kDrawCoordinate && key.threshold != 0u) {
        const uint32_t group = strip * (kStripCoords / 4u) + lane * 8u, last = (uint32_t)(key.threshold - 1u);
#pragma unroll
        for (uint32_t q = 0; q < 8u; ++q) {
            const U4 x = philox4x32_10_group(group + q, key.step_lo, key.step_hi, key.seed_lo, key.seed_hi);
            m |= (x.x0 <= last ? 1u : 0u) << (4u * q) | (x.x1 <= last ? 2u : 0u) << (4u * q)
               | (x.x2 <= last ? 4u : 0u) << (4u * q) | (x.x3 <= last ? 8u : 0u) << (4u * q);
        }
        return m;
    }
#pragma unroll 2
    for (uint32_t q = 0; q < 8u; ++q) {
        const uint64_t mu = mu0 + 4u * q;
        const int nvalid = whole ? 4 : (mu >= n ? 0 : (n - mu >= 4u ? 4 : (int)(n - mu)));
        m |= member_mask(key, mu >> 2, nvalid) << (4u * q);
    }
    return m;
}

// One workgroup (16 waves) per superblock of 512 tiles.  Pure integer hashing, no array reads.
// A tile owns ceil(count * mul / 32) whole 128-byte lines of [coordinate][replica] values in a ring slot,
// count its number of selected coordinates and mul the replicas per block.  Writes, per tile, the lines
// of the tiles of the same superblock before it (local_off) and, per superblock, its total (sb_sum).
// A small stage has few superblocks, so the time is what one workgroup needs for its 64 strips: sixteen
// waves of four strips each.
__global__ void __launch_bounds__(1024)
k_subset_count(SubsetKey key, uint64_t n, uint32_t ntiles, uint32_t mul,
               uint32_t *__restrict__ local_off, uint32_t *__restrict__ sb_sum)
{
    __shared__ uint32_t cnt[kTilesPerSuperblock];
    __shared__ uint32_t wave_tot[4];
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    for (uint32_t k = wave; k < kStripsPerSuperblock; k += 16u) {
        const uint32_t strip = blockIdx.x * kStripsPerSuperblock + k;
        uint32_t count = (uint64_t)strip * kStripCoords < n ? (uint32_t)__popc(strip_mask(key, n, strip, lane)) : 0u;
#pragma unroll
        for (int off = 1; off < 8; off <<= 1) count += __shfl_xor(count, off);       // the eight lanes of a tile
        if ((lane & 7u) == 0u) cnt[k * 8u + (lane >> 3)] = (count * mul + kLineFloats - 1u) / kLineFloats;
    }
    __syncthreads();
    scan_superblock(cnt, wave_tot, ntiles, local_off, sb_sum + blockIdx.x);
}

// Same, from tile sizes that are already in memory (the step and averaging kernels leave the line counts of
// the next step's subset there, a byte a tile, so that step needs no hashing pass of its own; T = uint32_t: the words of a
// checkpoint record of builds that kept words).
template <typename T>
__global__ void __launch_bounds__(256)
k_subset_offsets(const T *__restrict__ tile_size, uint32_t ntiles,
                 uint32_t *__restrict__ local_off, uint32_t *__restrict__ sb_sum)
{
    __shared__ uint32_t cnt[kTilesPerSuperblock];
    __shared__ uint32_t wave_tot[4];
    const uint32_t tile0 = blockIdx.x * kTilesPerSuperblock;
    for (uint32_t k = threadIdx.x; k < kTilesPerSuperblock; k += 256u)
        cnt[k] = tile0 + k < ntiles ? tile_size[tile0 + k] : 0u;
    __syncthreads();
    scan_superblock(cnt, wave_tot, ntiles, local_off, sb_sum + blockIdx.x);
}

// Sum of the sixteen bytes of x and acc.
__device__ __forceinline__ uint32_t sum_bytes(const v4u &x, uint32_t acc)
{
    acc = __builtin_amdgcn_sad_u8(x.x, 0u, acc);
    acc = __builtin_amdgcn_sad_u8(x.y, 0u, acc);
    acc = __builtin_amdgcn_sad_u8(x.z, 0u, acc);
    return __builtin_amdgcn_sad_u8(x.w, 0u, acc);
}

// The same with the superblocks' bases, in one launch instead of k_subset_offsets and k_subset_scan (9 to 10 us
// with the gap between them): every workgroup adds up the sizes of all tiles before its own.  4.7 us for 123 superblocks, 5.1 for
// 237, 7.7 for 504 (a word a tile: 12 us for 240), so it serves stages of at most kOffsetsAtOnce superblocks (67M coordinates).
constexpr uint32_t kOffsetsAtOnce = 512;
__global__ void __launch_bounds__(1024)
k_subset_offsets_at_once(const uint8_t *__restrict__ tile_size, uint32_t ntiles, uint32_t nsb, uint32_t capacity,
                         uint32_t *__restrict__ local_off, uint32_t *__restrict__ sb_base, uint32_t *__restrict__ flags)
{
    __shared__ uint32_t cnt[kTilesPerSuperblock];
    __shared__ uint32_t wave_tot[4], before[16], total;
    const uint32_t tile0 = blockIdx.x * kTilesPerSuperblock;
    if (threadIdx.x < kTilesPerSuperblock) cnt[threadIdx.x] = tile0 + threadIdx.x < ntiles ? tile_size[tile0 + threadIdx.x] : 0u;
    uint32_t sum = 0;
    for (uint32_t q = threadIdx.x; q < tile0 / 16u; q += 1024u) sum = sum_bytes(reinterpret_cast<const v4u *>(tile_size)[q], sum);
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) sum += __shfl_xor(sum, off);
    if ((threadIdx.x & 63u) == 0u) before[threadIdx.x >> 6] = sum;
    __syncthreads();
    scan_superblock(cnt, wave_tot, ntiles, local_off, &total);
    if (threadIdx.x == 255u) {                       // the thread that wrote the superblock's total
        uint32_t base = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) base += before[w];
        sb_base[blockIdx.x] = base;
        if (blockIdx.x == nsb - 1u) {
            sb_base[nsb] = base + total;
            if (base + total > capacity) atomicOr(flags, 1u);
        }
    }
}

// Lines that tile `tile` sends (lines: a byte a tile), as a scalar.
__device__ __forceinline__ uint32_t lines_of_tile(const uint8_t *lines, uint32_t tile)
{
    return (uniform_load(reinterpret_cast<const uint32_t *>(lines), tile / 4u) >> (8u * (tile % 4u))) & 0xFFu;
}

// Lines of the tiles before `tile`, this wave's share: of `waves` waves, wave w adds up the tiles 1024 w .. 1024 w + 1023, sixteen
// a lane, then the stretch 1024 waves further on, and so on for kSumLoads loads.  The shares of all waves add up to
// all of them when tile <= kSumTiles * waves.  All loads leave together: what lies past the tile's sixteen reads as zero, because the
// buffer descriptor ends there; those sixteen are added by the last wave.  lines: padded to whole 128 bytes.
constexpr uint32_t kSumLoads = 4, kSumTiles = 1024 * kSumLoads;
__device__ __forceinline__ uint32_t lines_before(const uint8_t *lines, uint32_t tile, uint32_t wave, uint32_t waves, uint32_t lane)
{
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(lines), 0, tile & ~15u, 0x00020000);
    v4u x[kSumLoads];
#pragma unroll
    for (uint32_t q = 0; q < kSumLoads; ++q) x[q] = v4u{0u, 0u, 0u, 0u};
    x[0] = __builtin_amdgcn_raw_buffer_load_b128(r, (int)(wave * 1024u + lane * 16u), 0, 0);
    if (tile > 1024u * waves) {
#pragma unroll
        for (uint32_t q = 1; q < kSumLoads; ++q)
            x[q] = __builtin_amdgcn_raw_buffer_load_b128(r, (int)((wave + q * waves) * 1024u + lane * 16u), 0, 0);
    }
    uint32_t sum = 0;
    if (wave + 1u == waves && lane < 4u) {               // the tiles of the tile's own sixteen that come before it
        const uint32_t first = (tile & ~15u) + 4u * lane, count = tile > first ? (tile - first < 4u ? tile - first : 4u) : 0u;
        if (count) sum = __builtin_amdgcn_sad_u8(reinterpret_cast<const uint32_t *>(lines)[first / 4u] & (0xFFFFFFFFu >> (32u - 8u * count)), 0u, 0u);
    }
#pragma unroll
    for (uint32_t q = 0; q < kSumLoads; ++q) sum = sum_bytes(x[q], sum);
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) sum += __shfl_xor(sum, off);
    return sum;
}
// The fused step adds up its tiles' places itself on the stages that am_host::step_sum_tiles names, and no launch precedes it.
// The averaging-only kernel (four waves, and little else to read) does so for as many as four waves can add up, 16384
// tiles (4.2M coordinates): R = 8 2M 31.8 / 29.8, 4.1M 53.5 / 51.4, R = 4 p = 2 % 34.6 / 32.3, R = 1 21.8 / 20.0; 1M R = 4 p = 1 %, whose four serial loads of
// words became one of bytes, 10.9 / 10.4.

// Single workgroup: exclusive scan of the superblock totals, in place (sb[i] <- sum of sb[<i]),
// grand total to sb[nsb]; raises flag bit 0 when the total exceeds the ring slot capacity.
__global__ void __launch_bounds__(256)
k_subset_scan(uint32_t *__restrict__ sb, uint32_t nsb, uint32_t capacity, uint32_t *__restrict__ flags)
{
    __shared__ uint64_t part[256];
    const uint32_t per = (nsb + 255u) / 256u;
    const uint32_t lo = threadIdx.x * per;
    const uint32_t hi = lo + per < nsb ? lo + per : nsb;
    uint64_t s = 0;
    for (uint32_t i = lo; i < hi; ++i) s += sb[i];
    part[threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t run = 0;
        for (int i = 0; i < 256; ++i) { const uint64_t x = part[i]; part[i] = run; run += x; }
        sb[nsb] = run > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)run;
        if (run > capacity) atomicOr(flags, 1u);
    }
    __syncthreads();
    uint64_t run = part[threadIdx.x];
    for (uint32_t i = lo; i < hi; ++i) { const uint32_t x = sb[i]; sb[i] = (uint32_t)run; run += x; }
}

// =============================================================================================
// Ascending index list of a subset (am_subset_indices):   k_list_clear  ->  k_subset_list
// =============================================================================================
// The cost is the generator (40 us for the words of 125.8M coordinates; the list itself is 50 MB at
// p = 5 %), so every coordinate is hashed once: a workgroup (four waves of `strips` strips each) keeps its
// masks in LDS, publishes how many coordinates it holds, adds up what all the workgroups before it
// hold and writes its indices there.  A lane holds 32 consecutive coordinates, so a strip of 2048 needs one
// scan over the lanes, and as many stores as the fullest lane has members.  Those stores scatter over as many lines as
// there are lanes, so where many coordinates are members (am_host::list_shape) a strip is written row by row instead
// (ROWS): 64 consecutive coordinates, one a lane, whose members go next to each other, 32 stores a strip.
// No workgroup waits before it has published, and each only for lower-numbered ones, which start before it; so
// every wait ends without all of them being resident (at 82 registers 20 waves a compute unit are).  None waits for good: one that has not seen a count after kListPatience looks
// (well over 10 ms) counts the members before its own part itself, so the kernel ends whatever else happens to the scratch.
// A thread looks at one count at a time: the counts sit in few lines, and eight looks in flight a thread make them the
// bottleneck (16M 14.2 -> 18.7 us, 31.5M 24.5 -> 29.0).
// Measured, p = 5 %: 125.8M coordinates 60.5 us (85.4 with the general form of the generator), 16M 14.2 (19.4), 1M 8.4 (9.9).
// part_count: word p = the count of part p, bit 31 set once it is known; k_list_clear zeroes them first.
constexpr uint32_t kListPatience = 1u << 15;

__global__ void __launch_bounds__(256)
k_list_clear(uint32_t *__restrict__ part_count, uint32_t parts)
{
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    if (i < parts) part_count[i] = 0u;
}

template <bool ROWS>
__global__ void __launch_bounds__(256)
k_subset_list(SubsetKey key, uint64_t n, uint32_t nstrips, uint32_t strips, uint32_t patience, uint32_t *part_count,
              uint64_t *__restrict__ out, uint64_t capacity, uint64_t *__restrict__ count_out)
{
    extern __shared__ uint32_t masks[];                       // [strips][256]
    __shared__ uint32_t wave_count[4];
    __shared__ uint64_t before[4];
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t part = blockIdx.x;
    const uint32_t strip0 = (part * 4u + wave) * strips;

    uint32_t mine = 0;                                        // members among the lane's coordinates of all its strips
    for (uint32_t k = 0; k < strips; ++k) {
        const uint32_t mask = strip0 + k < nstrips ? strip_mask(key, n, strip0 + k, lane) : 0u;
        masks[k * 256u + threadIdx.x] = mask;
        mine += (uint32_t)__popc(mask);
    }
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) mine += __shfl_xor(mine, off);
    if (lane == 0) wave_count[wave] = mine;
    __syncthreads();
    const uint32_t total = wave_count[0] + wave_count[1] + wave_count[2] + wave_count[3];
    if (threadIdx.x == 0)
        __hip_atomic_store(&part_count[part], total | 0x80000000u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

    uint64_t sum = 0;                                         // members of the parts before mine
    uint32_t looks = 0;
    for (uint32_t p = threadIdx.x; p < part; p += 256u) {
        uint32_t x;
        while (!((x = __hip_atomic_load(&part_count[p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) & 0x80000000u) && looks < patience) {
            ++looks;
            __builtin_amdgcn_s_sleep(1);
        }
        sum += x & 0x7FFFFFFFu;
        if (looks >= patience) break;
    }
    if (__syncthreads_or(looks >= patience)) {
        sum = 0;
        for (uint32_t k = wave; k < part * 4u * strips; k += 4u) sum += (uint32_t)__popc(strip_mask(key, n, k, lane));
    }
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) sum += __shfl_xor(sum, off);
    if (lane == 0) before[wave] = sum;
    __syncthreads();
    uint64_t pos = before[0] + before[1] + before[2] + before[3];
    if (part == gridDim.x - 1u && threadIdx.x == 0) *count_out = pos + total;
    if (capacity == 0u) return;
    for (uint32_t w = 0; w < wave; ++w) pos += wave_count[w];

    for (uint32_t k = 0; k < strips; ++k) {
        uint32_t mask = masks[k * 256u + threadIdx.x];
        const uint64_t strip_mu = (uint64_t)(strip0 + k) * kStripCoords;
        if constexpr (ROWS) {
#pragma unroll 4
            for (uint32_t q = 0; q < 32u; ++q) {              // coordinates 64 q .. 64 q + 63 of the strip, one a lane
                const uint64_t row = (uint32_t)__builtin_amdgcn_readlane((int)mask, (int)(2u * q))
                                     | (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)mask, (int)(2u * q + 1u)) << 32;
                const uint64_t at = pos + lanes_below(row);
                if (((row >> lane) & 1ull) && at < capacity) out[at] = strip_mu + q * 64u + lane;
                pos += (uint32_t)__popcll(row);
            }
        } else {
            const uint32_t members = (uint32_t)__popc(mask);
            uint32_t incl = members;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const uint32_t up = __shfl_up(incl, off);
                if ((int)lane >= off) incl += up;
            }
            uint64_t at = pos + (incl - members);
            const uint64_t mu0 = strip_mu + lane * 32u;
            while (mask) {
                if (at < capacity) out[at] = mu0 + (uint32_t)__builtin_ctz(mask);
                ++at;
                mask &= mask - 1u;
            }
            pos += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        }
    }
}

// =============================================================================================
// Fused step kernel
// =============================================================================================
enum : int { kOptSgdPlain = 0, kOptSgdMomentum = 1, kOptAdam = 2 };
enum : int { kFwdNone = 0, kFwdF32 = 1, kFwdBf16 = 2 };

// What one replica's wave needs to know about its replica: 64 bytes, one scalar load.  The record
// of replica b rb + k sits in slot 8 b + k of StepArgs::rep, whatever rb is, so that a wave finds its
// record from its block and wave numbers alone, in the same breath as the kernel's other arguments.
// Slots of absent replicas (R not a multiple of rb) repeat the record of the block's first replica:
// their waves may load through it, and store nothing.
struct ReplicaArgs {
    float *w, *m, *v;
    void *fwd;
    const void *g;              // NULL: the replica makes no local step in this launch (w^ = w; m, v kept)
    // bias corrections of the optimizer, per replica: replicas of unequal speed have made unequal
    // numbers of optimizer steps
    double c_g, c_m, c_v;
};

struct StepArgs {
    uint64_t n;
    uint32_t ntiles;
    uint32_t replicas;
    // blocks: replicas b rb .. b rb + rb - 1 form block b; one wave of a workgroup per replica of a block
    uint32_t rb, rb_shift;                         // replicas per block (1, 2, 4 or 8) and its log2
    uint32_t nblocks;                              // ceil(replicas / rb)
    uint32_t blocks_per_wg;                        // k_step: 1 (grid = tiles x blocks), or nblocks when tau = 0 (grid = tiles)
    uint32_t lookahead;
    // averaging
    uint32_t do_send, do_recv, ema, same_slot;     // ema: a correction vector d is kept; same_slot: tau = 0,
                                                   // the average is of this step's w^
    uint32_t through;                              // more than the caches hold: stores go through to memory
    uint32_t do_next;                              // also count the lines each tile will send next step
    uint32_t sum_lines;                            // small stage: the kernel itself adds up where the tile's lines start in the
                                                   // send slot (from send_lines) and writes the tile's word for the receive
    uint32_t msg_dtype;                            // precision of the exchanged values: 0 fp32, 1 bf16, 2 E4M3
    uint32_t cap_lines;                            // lines (of 32 floats) per block in a ring slot
    const uint8_t *send_lines;                     // [ntiles] lines each tile sends now (sum_lines)
    uint32_t *send_meta_out, *send_sb_out, *flags; // where its words go (sum_lines)
    const uint32_t *send_meta, *send_sb_base;      // tile's word: lines << 24 | offset in its superblock; first line = sb_base[tile >> 9] + offset
    const uint32_t *recv_meta, *recv_sb_base;
    float *ring_send;                              // slot written now: [block][line][32], a line = [coordinate][rb]
    const float *ring_recv;                        // slot sent tau rounds ago
    uint8_t *next_lines;                           // [ntiles], written when do_next (a tile owns at most 64 lines)
    const float *replica_scale;                    // NULL, or one more gradient factor per replica (DEVICE)
    SubsetKey key;                                 // seed, threshold and sampling rule; the step words are filled per job
    uint32_t step_lo[3], step_hi[3];               // the steps whose subsets are hashed: [0] received now, [1] sent now, [2] sent next step
    double coef_d, coef_s;                         // d <- coef_d d + coef_s (w^ - sent): EMA (1-lambda, lambda), eager (0, 1/R)
    // optimizer, every coefficient a per-step scalar evaluated once on the host in double:
    //   g  = grad_scale * g_raw                        (folded into b_m, b_v, c_g on the host)
    //   m' = a_m m + b_m g ;  v' = a_v v + b_v g^2
    //   w^ = w - (c_wd w + (c_g g + c_m m') / (c_v sqrt(v') + eps))           (Adam family)
    //   w^ = w - (c_wd w + c_m m')     resp.     w - (c_wd w + c_g g)          (SGD with / without momentum)
    double a_m, b_m, a_v, b_v, c_wd, eps;
    double gamma, inv_replicas;
    float *d[kMaxReplicas];          // one array per replica, or (interleaved) one per block: [tiles * 256][rb]
    union {
        ReplicaArgs rep[kMaxReplicas];
        float *w[kMaxReplicas];      // averaging alone (am_host::average_weights_table): every replica's weights.  In the records' place: a kernel's
                                     // arguments are copied at every launch (256 bytes more: SGD 6181 R = 1 6.75 us a step, 6.53 without)
    };
};

// Replica i's weights in the averaging-only kernel.
template <bool TABLE>
__device__ __forceinline__ float *weights_of(const StepArgs &a, uint32_t i) { return TABLE ? a.w[i] : a.rep[i].w; }

// Precision.  State is fp32 in memory (the method's precision).  The accumulating expressions
// (moments, weight update, EMA, look-ahead) are evaluated in fp64 from the stored fp32 values
// and rounded once on store, so that rounding noise does not random-walk over hundreds of steps;
// on this chip an fp64 FMA issues at the rate of an unpacked fp32 FMA, and the kernel is bound by
// memory.  The square root and the quotient start from the hardware's fp64 approximations of the reciprocal
// root and the reciprocal (some 24 bits, at a quarter of the rate) and take one Newton step each: 7 and 4 instructions, where the correctly
// rounded fp32 root with its scaling and an fp32 reciprocal with the conversions took 28 and 10 (a local step of four
// coordinates 250 -> 125 vector instructions).

// sqrt(x) of an fp32 value x >= 0, to (nearly) double accuracy
__device__ __forceinline__ double sqrt_refined(float x)
{
    const double xd = (double)x, y = __builtin_amdgcn_rsq(xd);
    const double s = xd * y;
    return x == 0.0f ? 0.0 : fma(fma(-s, s, xd), 0.5 * y, s);             // (the reciprocal root of zero is infinite)
}

// num / den for den > 0, to (nearly) double accuracy
__device__ __forceinline__ double quotient_refined(double num, double den)
{
    const double y = __builtin_amdgcn_rcp(den);
    const double q = num * y;
    return fma(fma(-q, den, num), y, q);
}

// What one replica's update of one group reads from memory.
struct GroupIn {
    F4 w, g, m, v;          // weights, gradients (widened), moments
    F4 d;                   // EMA entries of the group (per-replica layout: loaded when its line receives)
};

// A small stage's tile word and superblock base as the offsets pass would leave them for the receive; the
// word holds the first line in the slot itself, so every base is zero.  Called by one lane of one
// workgroup per tile; first + lines is the slot's total for the last tile.
__device__ __forceinline__ void write_send_word(const StepArgs &a, uint32_t tile, uint32_t first, uint32_t lines)
{
    a.send_meta_out[tile] = first | (lines << 24);
    if (tile % kTilesPerSuperblock == 0u) a.send_sb_out[tile / kTilesPerSuperblock] = 0u;
    if (first + lines > a.cap_lines) atomicOr(a.flags, 1u);
    if (tile + 1u == a.ntiles) a.send_sb_out[tile / kTilesPerSuperblock + 1u] = first + lines;
}

// Local optimizer step on one group of replica i, from loaded operands.  SCALAR: the replica's gradient factor is a scalar load; a vector load waits for everything
// that is on its way before it, but the kernels of small stages and those without delay have no scalar registers to spare (the former spill some already).  Either way it is read where it is
// used: requested beside the operands it takes registers in every step, without factors, too.  us a step, vector load / requested early / scalar load here: 3M AdamW, with factors R = 2 43.8 / 42.1 / 41.9,
// R = 8 150.8 / 148.7 / 148.4, without R = 1 24.5 / 25.0 / 24.5, R = 2 41.6 / 42.1 / 41.6; SGD with momentum R = 1 18.4 / 19.0 / 18.4, R = 6 4M with 94.9 / 90.2 / 89.6.  No delay, early: k_step_sync (65
// registers for 61: two workgroups of 16 waves no longer fit a compute unit) R = 13 3M 1.10 of the time, R = 15 300k 1.17, R = 16 no correction 3M 1.17; the walking form (40 bytes of scratch a lane for none) R = 20 1.5M 1.10, R = 32 1.09.
template <int OPT, bool SCALAR>
__device__ __forceinline__ void local_step(const StepArgs &a, const ReplicaArgs &r, uint32_t i, const GroupIn &in,
                                           F4 &w_hat, F4 &m_new, F4 &v_new)
{
    // A replica that is idle in this tick keeps its weights and moments; its gradient was not loaded.
    if (r.g == nullptr) {
        w_hat = in.w;
        if (OPT == kOptSgdMomentum || OPT == kOptAdam) m_new = in.m;
        if (OPT == kOptAdam) v_new = in.v;
        return;
    }
    double g[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) g[j] = (double)in.g.v[j];      // grad_scale is folded into b_m, b_v, c_g
    if (a.replica_scale) {
        const double rs = (double)(SCALAR ? __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)uniform_load(reinterpret_cast<const uint32_t *>(a.replica_scale), i))) : a.replica_scale[i]);
#pragma unroll
        for (int j = 0; j < 4; ++j) g[j] *= rs;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const double wo = (double)in.w.v[j];
        double step;                                           // what is subtracted besides the decay
        if (OPT == kOptSgdPlain) {
            step = r.c_g * g[j];
        } else if (OPT == kOptSgdMomentum) {
            m_new.v[j] = (float)fma(a.a_m, (double)in.m.v[j], a.b_m * g[j]);
            step = r.c_m * (double)m_new.v[j];
        } else {
            m_new.v[j] = (float)fma(a.a_m, (double)in.m.v[j], a.b_m * g[j]);
            v_new.v[j] = (float)fma(a.a_v, (double)in.v.v[j], a.b_v * g[j] * g[j]);
            const double den = fma(r.c_v, sqrt_refined(v_new.v[j]), a.eps);
            const double num = fma(r.c_g, g[j], r.c_m * (double)m_new.v[j]);
            step = quotient_refined(num, den);
        }
        w_hat.v[j] = (float)(wo - fma(a.c_wd, wo, step));
    }
}

// LDS written by some lanes of a wave is about to be read by other lanes of the same wave.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A touched line of the tile's interleaved EMA entries in the list: its index in the tile, and in bits 8 and 9 whether its 64-byte halves hold a
// received coordinate.  Called by the line's first lane.  mask: the lane's coordinates that are received; any: the lanes that have one; sh: log2
// of the replicas per block.
__device__ __forceinline__ uint32_t touched_line(uint32_t lane, uint32_t mask, uint64_t any, uint32_t sh)
{
    uint32_t lo = mask & 3u, hi = mask & 12u;              // eight replicas: a line is one group, a half two of its coordinates
    if (sh != 3u) {
        const uint32_t lanes = 4u >> sh, group_bits = (1u << lanes) - 1u;
        lo = (uint32_t)(any >> lane) & group_bits;
        hi = (uint32_t)(any >> (lane + lanes)) & group_bits;
    }
    return lane >> (3u - sh) | (lo ? 0x100u : 0u) | (hi ? 0x200u : 0u);
}
__device__ __forceinline__ uint32_t line_index(uint32_t entry) { return entry & 0xFFu; }
__device__ __forceinline__ bool half_received(uint32_t entry, uint32_t half) { return ((entry >> 8) >> half) & 1u; }

// Where the coordinates of one group (= one lane) sit in the subsets of this step.
struct GroupSubsets {
    uint32_t mask_send, mask_recv;      // bit j: coordinate 4*group + j is sent / received now
    uint32_t rank_send, rank_recv;      // rank of the first such coordinate among those of the tile
    bool half_recv;                     // the 64 bytes of a per-replica array (4 lanes) holding the group receive something
    uint32_t d_slot;                    // interleaved d: float offset, in the LDS staging area, of the group's first entry
};

// LDS of one workgroup (floats): what the replicas sent tau rounds ago, the touched lines of d, the
// lines about to be sent, and the list of touched lines.
struct TileLds {
    float *recv;        // [nblocks][256 coordinates in rank order][rb]
    float *d;           // [touched line][32]         (interleaved d only)
    float *send;        // [256 coordinates in rank order][rb]
    uint32_t *list;     // [64] tile-local index of the q-th touched line of d
    uint8_t *masks;     // [0..63] the lanes' masks of the sent subset, [64..127] of the received one
    uint32_t *part;     // [8] the waves' shares of the lines before the tile (sum_lines)
    float *abar;        // [256] mean over the replicas of what they sent, per received coordinate in rank order
};

// Issues the loads of replica i's dense operands for one group.
template <int OPT, bool GRAD_BF16>
__device__ __forceinline__ void load_group(const ReplicaArgs &r, uint64_t tbase, uint32_t loff, int nvalid, GroupIn &in)
{
    in.w = load_f32x4(r.w + tbase, loff, nvalid);
    // An idle replica has no gradient: its wave reads its weights in their place (memory that is
    // surely there; the optimizer step drops the value), without a branch, so that no load waits
    // for another.
    const void *gp = r.g == nullptr ? static_cast<const void *>(r.w) : r.g;
    in.g = GRAD_BF16 ? load_bf16x4(static_cast<const uint16_t *>(gp) + tbase, loff, nvalid)
                     : load_f32x4(static_cast<const float *>(gp) + tbase, loff, nvalid);
    if (OPT != kOptSgdPlain) in.m = load_f32x4(r.m + tbase, loff, nvalid);
    if (OPT == kOptAdam) in.v = load_f32x4(r.v + tbase, loff, nvalid);
}

// What the averaging touches in the per-replica arrays besides the dense operands: the EMA entries of
// a line that receives (per-replica layout of d).
template <bool DIL>
__device__ __forceinline__ void load_group_sparse(const StepArgs &a, uint32_t i, uint64_t tbase, uint32_t loff, int nvalid,
                                                  const GroupSubsets &s, GroupIn &in)
{
    if (!DIL && a.ema && s.half_recv) in.d = load_f32x4(a.d[i] + tbase, loff, nvalid);
}

// The new weights of one group and their forward copy.  SHORT: a bf16 copy without look-ahead is one conversion of the stored weight (the same bits); not in the
// walking form, which has no registers for a second way through (us a step with it / without: R = 20 1.5M 231 / 222, R = 32 408 / 389).
template <int FWD, bool SHORT = true>
__device__ __forceinline__ void store_weights(const StepArgs &a, const ReplicaArgs &r, uint64_t tbase, uint32_t loff, int nvalid, const GroupIn &in,
                                              const F4 &w_hat, const F4 &w_new)
{
    store_tile_f32x4(r.w + tbase, loff, nvalid, w_new, a.through != 0u);
    if (SHORT && FWD == kFwdBf16 && !a.lookahead) {
        store_bf16x4_from_f32(static_cast<uint16_t *>(r.fwd) + tbase, loff, nvalid, w_new, a.through != 0u);
    } else if (FWD != kFwdNone) {
        // fwd = w + gamma (w^ - w_before): product and sum rounded separately in fp64, then ONE
        // rounding to the stored type
        double f[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            f[j] = a.lookahead ? __dadd_rn((double)w_new.v[j], __dmul_rn(a.gamma, (double)w_hat.v[j] - (double)in.w.v[j]))
                               : (double)w_new.v[j];
        if (FWD == kFwdF32) {
            F4 o;
#pragma unroll
            for (int j = 0; j < 4; ++j) o.v[j] = (float)f[j];
            store_tile_f32x4(static_cast<float *>(r.fwd) + tbase, loff, nvalid, o, a.through != 0u);
        } else {
            store_bf16x4_from_f64(static_cast<uint16_t *>(r.fwd) + tbase, loff, nvalid, f, a.through != 0u);
        }
    }
}

// Replica i (slot `slot` of its block) of one group, from its stepped weights to stored results: the
// receive, the new weights and the forward copy.  WALKS: the workgroup walks the blocks of its tile.
// recv_block: what the replicas of i's block sent tau rounds ago, [rank][rb] (TAU0: unused, the sent value is w^ itself).
template <int FWD, bool DIL, bool TAU0, bool WALKS>
__device__ __forceinline__ void finish_replica(const StepArgs &a, const ReplicaArgs &r, uint32_t i, uint32_t slot, uint64_t tbase, uint32_t loff, int nvalid,
                                               const GroupSubsets &s, const bool tile_receives, const float (&abar)[4], GroupIn &in,
                                               const F4 &w_hat, const float *recv_block, const TileLds &L)
{
    const uint32_t rb = a.rb;
    F4 w_new;
#pragma unroll
    for (int j = 0; j < 4; ++j) w_new.v[j] = w_hat.v[j];
    if (tile_receives) {                                   // receive: old average (+ EMA of staleness)
        // Same for the whole workgroup, and free of branches inside: every lane reads (a lane without
        // a received coordinate reads entry 0 and drops the result), so that the LDS reads of the four
        // coordinates are in flight together instead of one dependent round trip per coordinate.
        uint32_t cj[4], c = s.rank_recv;
#pragma unroll
        for (int j = 0; j < 4; ++j) { const uint32_t bit = (s.mask_recv >> j) & 1u; cj[j] = bit ? c : 0u; c += bit; }
        if (a.ema) {
            float sent[4], d_old[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t bit = (s.mask_recv >> j) & 1u;
                sent[j] = TAU0 ? w_hat.v[j] : recv_block[cj[j] * rb + slot];
                d_old[j] = DIL ? L.d[bit ? s.d_slot + (uint32_t)j * rb + slot : 0u] : in.d.v[j];
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float d_new = (float)fma(a.coef_d, (double)d_old[j], a.coef_s * ((double)w_hat.v[j] - (double)sent[j]));
                if ((s.mask_recv >> j) & 1u) {
                    if (DIL) L.d[s.d_slot + (uint32_t)j * rb + slot] = d_new;
                    else in.d.v[j] = d_new;
                    w_new.v[j] = (float)((double)abar[j] + (double)d_new);
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if ((s.mask_recv >> j) & 1u) w_new.v[j] = abar[j];
        }
    }
    if (!DIL && a.ema && s.half_recv) store_tile_f32x4(a.d[i] + tbase, loff, nvalid, in.d, a.through != 0u);

    store_weights<FWD, !WALKS>(a, r, tbase, loff, nvalid, in, w_hat, w_new);
}

// The same from loaded operands: local step (unless the caller has done it while it waited), send, receive.
template <int OPT, int FWD, bool DIL, bool TAU0>
__device__ __forceinline__ void step_replica(const StepArgs &a, const ReplicaArgs &r, uint32_t i, uint32_t slot, uint64_t tbase, uint32_t loff, int nvalid,
                                             const GroupSubsets &s, const bool tile_receives, const float (&abar)[4], GroupIn &in,
                                             F4 &w_hat, F4 &m_new, F4 &v_new, const float *recv_block, const TileLds &L)
{
    const uint32_t rb = a.rb;
    if (TAU0) {
        local_step<OPT, false>(a, r, i, in, w_hat, m_new, v_new);
        // the moments are final: out they go, before the averaging needs registers
        if (OPT == kOptSgdMomentum || OPT == kOptAdam) store_tile_f32x4(r.m + tbase, loff, nvalid, m_new, a.through != 0u);
        if (OPT == kOptAdam) store_tile_f32x4(r.v + tbase, loff, nvalid, v_new, a.through != 0u);
    }

    if (s.mask_send) {                                     // send: into the staging lines, [rank][rb]
        uint32_t c = s.rank_send;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if ((s.mask_send >> j) & 1u) L.send[(c++) * rb + slot] = w_hat.v[j];
    }
    finish_replica<FWD, DIL, TAU0, TAU0>(a, r, i, slot, tbase, loff, nvalid, s, tile_receives, abar, in, w_hat, recv_block, L);
}

template <int RB>
__device__ __forceinline__ void load_block_values(const float *p, float (&x)[RB])
{
    if constexpr (RB == 8) {
        const v4f lo = *reinterpret_cast<const v4f *>(p), hi = *reinterpret_cast<const v4f *>(p + 4);
        x[0] = lo.x; x[1] = lo.y; x[2] = lo.z; x[3] = lo.w; x[4] = hi.x; x[5] = hi.y; x[6] = hi.z; x[7] = hi.w;
    } else if constexpr (RB == 4) {
        const v4f lo = *reinterpret_cast<const v4f *>(p);
        x[0] = lo.x; x[1] = lo.y; x[2] = lo.z; x[3] = lo.w;
    } else if constexpr (RB == 2) {
        const v2f lo = *reinterpret_cast<const v2f *>(p);
        x[0] = lo.x; x[1] = lo.y;
    } else {
        x[0] = p[0];
    }
}

// Mean over the replicas, in replica order and in fp64, of what they sent for the coordinate of
// rank c of the tile (recv: [block][rank][RB], `stride` floats a block): the RB values of a block come with one or two wide
// LDS reads.  ABSENT: the slots of absent replicas may hold anything; else they hold zeros, which add nothing.
template <int RB, bool ABSENT>
__device__ __forceinline__ float replica_mean(const StepArgs &a, const float *recv, uint32_t c, uint32_t stride = kTileCoords * RB)
{
    double sum = 0.;
    for (uint32_t b = 0; b < a.nblocks; ++b) {
        const float *p = recv + b * stride + c * RB;
        float x[RB];
        load_block_values<RB>(p, x);
        if (a.msg_dtype != 0u) {
#pragma unroll
            for (int k = 0; k < RB; ++k) x[k] = quantize_message(x[k], a.msg_dtype);
        }
        const uint32_t nrep = a.replicas - b * RB;         // replicas present in this block (>= RB: all)
#pragma unroll
        for (int k = 0; k < RB; ++k)
            if (!ABSENT || (uint32_t)k < nrep) sum += (double)x[k];
    }
    return (float)(sum * a.inv_replicas);
}

// The means of the received coordinates of ranks first, first + stride, ... below count, into L.abar.
template <bool ABSENT>
__device__ __forceinline__ void tile_means(const StepArgs &a, const TileLds &L, uint32_t first, uint32_t stride, uint32_t count)
{
    if (a.rb == 8u) for (uint32_t c = first; c < count; c += stride) L.abar[c] = replica_mean<8, ABSENT>(a, L.recv, c);
    else if (a.rb == 4u) for (uint32_t c = first; c < count; c += stride) L.abar[c] = replica_mean<4, ABSENT>(a, L.recv, c);
    else if (a.rb == 2u) for (uint32_t c = first; c < count; c += stride) L.abar[c] = replica_mean<2, ABSENT>(a, L.recv, c);
    else for (uint32_t c = first; c < count; c += stride) L.abar[c] = replica_mean<1, ABSENT>(a, L.recv, c);
}

// One workgroup per (tile of 256 coordinates, block of rb <= 8 replicas); its rb waves are the
// replicas of the block, one lane per group of 4 coordinates.  Each wave streams its replica's 1 KB
// of every per-replica array once, with non-temporal accesses (measured on MI355X: the fastest way
// through the 4-read / 4-write stream mix of this update).
//
// This memory system reads 128-byte lines and writes their 64-byte halves; a write of part of a half costs several whole ones.  S^t is
// the same for every replica, so the sparse structures keep the replicas of a block side by side,
// [coordinate][replica]: a line holds 32 / rb coordinates of all rb replicas and is written as a whole.
//  * Ring slot: per block, every tile owns ceil(count rb / 32) whole lines ([block][line][32]); the
//    selected values sit in ascending coordinate order, the rest of the last line is zero.  The
//    tile's word in the slot's offset table (a scalar load) says where its lines start and how
//    many there are, so the lines sent tau rounds ago are requested without any hashing, straight
//    into LDS; the waves gather this step's values in LDS and the lines leave with 16 bytes per thread.
//  * EMA vector d, interleaved layout: [coordinate][replica] per block.  Lines that hold a received
//    coordinate are copied to LDS (16 bytes per lane) and updated there; of each, the halves that hold one are
//    written back.  Per-replica layout: dense per replica; the 8 lanes that share a line of d load their
//    groups together whenever any of them holds a received coordinate, and the 4 that share a half store theirs.
// Hashing a subset costs ten rounds of two 32 x 32 -> 64 multiplies per lane; the subsets are the
// same for every wave of the workgroup, so (fused step) one wave hashes the received subset, one
// the sent one, one the next step's, and the others read the 4-bit masks from LDS after the barrier
// they have to pass anyway.  (Where the masks steer loads of per-replica arrays -- a correction vector in
// the per-replica layout -- every wave still hashes the received subset itself, so that those loads go out
// before the barrier.)
//
// What the write-back of d costs is halved by halves: only the 64-byte halves of a line that hold a received coordinate are
// written (interleaved, R = 8, p = 5 %: 9.8 % of them instead of 18.5 % of the lines; per replica 56 % instead of 81 %); with fewer vector instructions
// in the local step and the mean, stores that go through to memory (store_through) and the residency of
// am_host::step_workgroups, us a step before / after: R = 8 125.8M interleaved 5940 / 5834 (34.0 GB: 5.8 TB/s), 31.5M per replica 1840 / 1799,
// R = 4 31.5M 757 / 722, 7.1M 178.5 / 171.7, R = 2 31.5M 373 / 363, R = 1 200 / 193, R = 16 125.8M bf16 9931 / 9845, R = 2 3M SGD with K = 5 24.5 / 23.2,
// 1M R = 4 32.5 / 31.1 and 500k 17.7 / 17.0 (ordinary non-temporal stores).
//
// FULL = every coordinate of the tile exists (all but possibly the last tile of the stage): all
// dense accesses are unconditional 128-bit ones.
// SUM = small stage: the workgroup adds up where its tile's lines start in the send slot itself (as a run-time
// switch it costs every stage 0.5 %: 5990 against 5962 us on the headline one).
// TAU0 = the average is of this very step's values (tau = 0) and there are more than kSyncWaves replicas: the
// workgroup walks all the blocks of its tile, because it needs every replica's new weights (fewer
// replicas: step_tile_sync).
template <int OPT, bool GRAD_BF16, int FWD, bool DIL, bool TAU0, bool SUM, bool FULL>
__device__ __forceinline__ void step_tile(const StepArgs &a, const uint32_t tile, const uint32_t b0, const uint32_t wave,
                                          const uint32_t lane, const TileLds &L)
{
    // One wave hashes the sent subset for all; so it is with the received subset, unless its masks steer
    // loads of per-replica arrays that should leave before the barrier (per-replica layout of d).
    const bool kShareRecv = DIL || !a.ema;
    const bool sum_lines = TAU0 ? a.sum_lines != 0u : SUM;
    const uint32_t R = a.replicas, rb = a.rb, sh = a.rb_shift;
    const uint32_t flat = wave * 64u + lane;                               // 64 rb threads; thread f owns 16-byte chunk f
    const uint64_t group = (uint64_t)tile * 64u + lane;
    const uint64_t mu = group * 4u;
    const int nvalid = FULL ? 4 : (mu >= a.n ? 0 : (a.n - mu >= 4u ? 4 : (int)(a.n - mu)));
    // addresses in the per-replica arrays: a pointer that is the same for the whole wave plus a 32-bit lane offset
    const uint64_t tbase = (uint64_t)tile * kTileCoords;
    const uint32_t loff = lane * 4u;
    const uint64_t block_floats = (uint64_t)a.cap_lines * kLineFloats;     // one block's part of a ring slot
    const uint32_t tile_floats = kTileCoords * rb;                         // one tile's part of an interleaved array
    constexpr bool recv_is_send = TAU0;                                    // the host launches TAU0 iff do_recv && same_slot

    // ---- dense operands of my replica of the first block: nothing else is requested before them
    uint32_t i = b0 * rb + wave;
    ReplicaArgs rep = a.rep[8u * b0 + wave];               // my replica's pointers and coefficients, one scalar load
    GroupIn in;
    // (no condition on i < R: the record of an absent replica names the arrays of the block's first
    // replica, whose values its wave loads and never uses -- with a condition the compiler parks
    // the conversions of the loaded values, and with them a wait for memory, right behind the loads)
    load_group<OPT, GRAD_BF16>(rep, tbase, i < R ? loff : 0u, nvalid, in);      // (an absent replica's wave: one group for all lanes)
    __builtin_amdgcn_sched_barrier(0);

    // ---- subsets: bit j of a lane's mask = coordinate 4 group + j is received / sent now.
    //      Jobs: 0 = the received subset, 1 = the sent one, 2 = the size of what the next step sends.
    //      A shared job is done by wave (job mod rb), the others by every wave for itself.
    GroupSubsets s;
    s.mask_send = s.mask_recv = s.rank_send = s.rank_recv = s.d_slot = 0;
    s.half_recv = false;
    const uint32_t lpl = 8u >> sh;                                         // lanes (groups) per 128-byte line of d
    const uint32_t leader = lane & ~(lpl - 1u);
    // interleaved d: the lines of the tile that hold a received coordinate go straight into LDS, requested
    // by the wave that hashes the received subset as soon as it knows them.  (Noting the touched lines
    // in memory when a subset is sent and reading them back before hashing was measured slower: the
    // scalar load of the note holds the hashing wave up for longer than the hashing takes.)
    auto request_d_lines = [&](const uint64_t leaders, const uint32_t mask) {
        const uint32_t nlines = (uint32_t)__popcll(leaders);
        if (nlines) {
            const uint64_t any = __ballot(mask != 0u);
            if ((leaders >> lane) & 1ull) L.list[__popcll(leaders & ((1ull << lane) - 1ull))] = touched_line(lane, mask, any, sh);
            wave_lds_sync();
            const float *src = a.d[b0] + (uint64_t)tile * tile_floats + (lane & 7u) * 4u;
            for (uint32_t q0 = 0; q0 < nlines; q0 += 8u) {
                const uint32_t q = q0 + (lane >> 3);
                if (q < nlines) lds_dma_16(src + line_index(L.list[q]) * kLineFloats, L.d + q0 * kLineFloats);
            }
        }
    };
    auto lines_of = [&](const uint32_t mask) {              // bit = first lane of a line of d that holds a coordinate of the mask
        const uint64_t any = __ballot(mask != 0u);
        const bool touched = ((any >> leader) & ((1ull << lpl) - 1ull)) != 0ull;
        return (uint64_t)__ballot(touched && lane == leader);
    };
#pragma unroll
    for (uint32_t job = 0; job < 3u; ++job) {
        const bool shared = job == 0u ? kShareRecv : true;
        if (shared && wave != (job & (rb - 1u))) continue;
        if (job == 0u && !a.do_recv) continue;
        if (job == 1u && (!a.do_send || recv_is_send)) continue;
        if (job == 2u && !(a.do_next && b0 == 0u)) continue;
        SubsetKey key = a.key;
        const uint32_t which = (job == 0u && recv_is_send) ? 1u : job;
        key.step_lo = a.step_lo[which]; key.step_hi = a.step_hi[which];
        const uint32_t mask = member_mask(key, group, nvalid);
        if (job == 0u) {
            s.mask_recv = mask;
            if (kShareRecv) L.masks[64u + lane] = (uint8_t)mask;
            if (DIL && a.ema && wave == 0u) request_d_lines(lines_of(mask), mask);
        } else if (job == 1u) {
            s.mask_send = mask;
            L.masks[lane] = (uint8_t)mask;
        } else {
            uint32_t count;
            (void)wave_prefix_mask4(mask, count);
            if (lane == 0) a.next_lines[tile] = (uint8_t)((count * rb + kLineFloats - 1u) / kLineFloats);
        }
    }
    // ---- the tile's words in the offset tables of the two slots (scalar loads)
    uint32_t word_s = 0, base_s = 0, word_r = 0, base_r = 0;
    if (sum_lines) word_s = lines_of_tile(a.send_lines, tile) << 24;
    else if (a.do_send) { word_s = uniform_load(a.send_meta, tile); base_s = uniform_load(a.send_sb_base, tile / kTilesPerSuperblock); }
    if (a.do_recv && !TAU0) { word_r = uniform_load(a.recv_meta, tile); base_r = uniform_load(a.recv_sb_base, tile / kTilesPerSuperblock); }

    // ---- where the tile's lines sit in the two slots.  A tile whose lines would pass the slot
    //      capacity is left out, at send and at receive alike.  (sum_lines: where it sends to is known after
    //      the barrier.)
    uint32_t first_s = base_s + (word_s & 0xFFFFFFu), lines_s = word_s >> 24;
    uint32_t first_r = base_r + (word_r & 0xFFFFFFu), lines_r = word_r >> 24;
    bool keep_s = a.do_send != 0u, keep_r = a.do_recv != 0u;
    auto find_send = [&]() {                                // every wave's share is in LDS
        first_s = 0;
        for (uint32_t w = 0; w < rb; ++w) first_s += L.part[w];
        first_s = (uint32_t)__builtin_amdgcn_readfirstlane((int)first_s);
        if (b0 == 0u && flat == 0u) write_send_word(a, tile, first_s, lines_s);
        if (first_s + lines_s > a.cap_lines) { keep_s = false; lines_s = 0; s.mask_send = 0u; }
    };
    if (sum_lines) {
        const uint32_t share = lines_before(a.send_lines, tile, wave, rb, lane);
        if (lane == 0) L.part[wave] = share;
        if (TAU0) { __syncthreads(); find_send(); }
    } else if ((uint64_t)first_s + lines_s > a.cap_lines) { keep_s = false; lines_s = 0; }
    if (recv_is_send) { first_r = first_s; lines_r = lines_s; keep_r = keep_s; }
    else if ((uint64_t)first_r + lines_r > a.cap_lines) { keep_r = false; lines_r = 0; }

    // ---- what every replica sent tau rounds ago: straight into LDS.  The chunks are dealt out from
    //      the last wave down: the first waves are busy hashing.
    const uint32_t wave_r = rb - 1u - wave;
    if (a.do_recv && !TAU0 && wave_r * 64u + lane < lines_r * 8u) {
        const float *src = a.ring_recv + (uint64_t)first_r * kLineFloats + (wave_r * 64u + lane) * 4u;
        for (uint32_t b = 0; b < a.nblocks; ++b)
            lds_dma_16(src + b * block_floats, L.recv + b * tile_floats + wave_r * 256u);
    }
    if (!keep_r) s.mask_recv = 0u;                          // (masks a wave hashed for itself)
    if (!keep_s) s.mask_send = 0u;

    // the masks of the hashing waves, ranks inside the tile, and where the group's d entries sit in LDS
    uint32_t count_recv = 0, d_lines = 0;
    auto finish_subsets = [&]() {
        if (kShareRecv) s.mask_recv = keep_r ? (uint32_t)L.masks[64u + lane] : 0u;
        s.mask_send = recv_is_send ? s.mask_recv : (keep_s ? (uint32_t)L.masks[lane] : 0u);
        uint32_t count_send;
        s.rank_send = wave_prefix_mask4(s.mask_send, count_send);
        if (recv_is_send) { s.rank_recv = s.rank_send; count_recv = count_send; }
        else s.rank_recv = wave_prefix_mask4(s.mask_recv, count_recv);
        const uint64_t any_recv = __ballot(s.mask_recv != 0u);
        s.half_recv = ((any_recv >> (lane & ~3u)) & 0xFull) != 0ull;
        if (DIL && a.ema) {
            const bool touched = ((any_recv >> leader) & ((1ull << lpl) - 1ull)) != 0ull;
            const uint64_t leaders = __ballot(touched && lane == leader);
            d_lines = (uint32_t)__popcll(leaders);
            s.d_slot = (uint32_t)__popcll(leaders & ((1ull << leader) - 1ull)) * kLineFloats + (lane & (lpl - 1u)) * 4u * rb;
        }
    };

    if (!DIL && a.ema) {                                   // loads of per-replica arrays that the masks steer
        const uint64_t any_recv = __ballot(s.mask_recv != 0u);
        s.half_recv = ((any_recv >> (lane & ~3u)) & 0xFull) != 0ull;
        if (i < R) load_group_sparse<DIL>(a, i, tbase, loff, nvalid, s, in);
    }

    // ---- staging lines of the send start at zero: line tails and the slots of absent replicas stay zero
    if (flat < lines_s * 8u) *reinterpret_cast<v4f *>(L.send + flat * 4u) = v4f{0.f, 0.f, 0.f, 0.f};

    // ---- tau = 0: the average is of this step's w^ : every wave puts those of its replicas in place
    if (recv_is_send) {
        if (kShareRecv) __syncthreads();                   // the masks are in LDS
        finish_subsets();
        if (count_recv) {
            for (uint32_t b = 0; b < a.nblocks; ++b) {
                const uint32_t ib = b * rb + wave;
                if (ib >= R) continue;
                GroupIn pre;
                F4 w_hat, m_new, v_new;
                if (b == b0) {
                    pre = in;
                } else {
                    load_group<OPT, GRAD_BF16>(a.rep[8u * b + wave], tbase, loff, nvalid, pre);
                    load_group_sparse<DIL>(a, ib, tbase, loff, nvalid, s, pre);
                }
                local_step<OPT, false>(a, a.rep[8u * b + wave], ib, pre, w_hat, m_new, v_new);
                uint32_t c = s.rank_recv;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if ((s.mask_recv >> j) & 1u) L.recv[b * tile_floats + (c++) * rb + wave] = w_hat.v[j];
            }
        }
    }
    // the local optimizer step needs nothing but the wave's own operands: it runs while the lines
    // for LDS and the other waves' operands are still on their way.  The branch (the same for the whole wave)
    // keeps absent replicas' waves idle and the conversions of the operands behind the hashing: 54
    // registers instead of 66 to 72.  Measured with that, in us a step, before / after: no correction, bf16, R = 16, 125.8M
    // 10107 / 9924, R = 8, 31.5M 1195 / 1162; per-replica d, 31.5M, R = 2 369 / 363; absent replicas: R = 12, 10M, bf16 772 /
    // 751 (per replica), 713 / 692 (interleaved), R = 6 386 / 364; no change beyond noise on the headline step.
    F4 w_hat, m_new, v_new;
    if (!TAU0 && i < R) local_step<OPT, !SUM>(a, rep, i, in, w_hat, m_new, v_new);
    lds_dma_wait();
    __syncthreads();
    if (!TAU0 && i < R) {                                  // the moments are final: out they go at once
        if (OPT == kOptSgdMomentum || OPT == kOptAdam) store_tile_f32x4(rep.m + tbase, loff, nvalid, m_new, a.through != 0u);
        if (OPT == kOptAdam) store_tile_f32x4(rep.v + tbase, loff, nvalid, v_new, a.through != 0u);
    }
    if (!TAU0 && sum_lines) find_send();
    if (!recv_is_send) finish_subsets();

    // ---- old average of the coordinates received now: thread c forms the mean of the coordinate of
    //      rank c once for the whole workgroup (in fp64, in replica order); after one more barrier every
    //      lane picks up the means of its own coordinates (a lane with fewer than four reads entry 0 and
    //      drops it, so that the four reads are in flight together)
    float abar[4] = {0.f, 0.f, 0.f, 0.f};
    if (count_recv) {                                      // same for the whole workgroup
        tile_means<TAU0>(a, L, flat, 64u * rb, count_recv);
        __syncthreads();
        uint32_t c = s.rank_recv;
#pragma unroll
        for (int j = 0; j < 4; ++j) { const uint32_t bit = (s.mask_recv >> j) & 1u; abar[j] = L.abar[bit ? c : 0u]; c += bit; }
    }

    // my chunk of the touched lines of d: float offset inside the tile's part of the array
    const uint32_t d_line = (DIL && flat < d_lines * 8u) ? L.list[flat >> 3] : 0u;     // (0: no half received)
    const uint32_t d_chunk_off = line_index(d_line) * kLineFloats + (flat & 7u) * 4u;
    const bool d_chunk_changes = DIL && half_received(d_line, (flat >> 2) & 1u);

    // ---- my replica of each block of this workgroup (one block, except when tau = 0 and R > 8)
    for (uint32_t bb = 0; bb < (TAU0 ? a.blocks_per_wg : 1u); ++bb) {
        const uint32_t b = b0 + bb;
        i = b * rb + wave;
        if (TAU0 && bb != 0u) {
            __syncthreads();                               // the staging areas are free again
            if (flat < lines_s * 8u) *reinterpret_cast<v4f *>(L.send + flat * 4u) = v4f{0.f, 0.f, 0.f, 0.f};
            if (DIL && flat < d_lines * 8u)
                lds_dma_16(a.d[b] + (uint64_t)tile * tile_floats + d_chunk_off, L.d + wave * 256u);
            if (i < R) {
                rep = a.rep[8u * b + wave];
                load_group<OPT, GRAD_BF16>(rep, tbase, loff, nvalid, in);
                load_group_sparse<DIL>(a, i, tbase, loff, nvalid, s, in);
            }
            lds_dma_wait();
            __syncthreads();
        }
        if (i < R) step_replica<OPT, FWD, DIL, TAU0>(a, rep, i, wave, tbase, loff, nvalid, s, count_recv != 0u, abar, in, w_hat, m_new, v_new, L.recv + b * tile_floats, L);
        __syncthreads();
        // whole lines leave with 16 bytes per thread
        if (flat < lines_s * 8u) {
            float *dst = a.ring_send + b * block_floats + (uint64_t)first_s * kLineFloats + flat * 4u;
            __builtin_nontemporal_store(*reinterpret_cast<const v4f *>(L.send + flat * 4u), reinterpret_cast<v4f *>(dst));
        }
        if (d_chunk_changes) {
            float *dst = a.d[b] + (uint64_t)tile * tile_floats + d_chunk_off;
            __builtin_nontemporal_store(*reinterpret_cast<const v4f *>(L.d + flat * 4u), reinterpret_cast<v4f *>(dst));
        }
    }
}

// Floats of dynamic LDS a workgroup needs.
__host__ __device__ inline uint32_t step_lds_floats(uint32_t rb, uint32_t nblocks, bool d_interleaved)
{
    return nblocks * kTileCoords * rb + (d_interleaved ? kTileCoords * rb : 0u) + kTileCoords * rb + 64u + 32u + 8u + kTileCoords;
}

// grid = (tiles, blocks) (tau = 0: (tiles, 1)); blockDim = 64 rb; dynamic LDS = step_lds_floats() floats
// (at most 80 registers, so that three workgroups of eight waves fit a compute unit)
template <bool DIL>
__device__ __forceinline__ TileLds step_lds(const StepArgs &a)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];
    const uint32_t tile_floats = kTileCoords * a.rb;
    TileLds L;
    L.recv = lds;
    L.d = L.recv + a.nblocks * tile_floats;
    L.send = L.d + (DIL ? tile_floats : 0u);
    L.list = reinterpret_cast<uint32_t *>(L.send + tile_floats);
    L.masks = reinterpret_cast<uint8_t *>(L.list + 64);
    L.part = L.list + 96;
    L.abar = reinterpret_cast<float *>(L.list + 104);
    return L;
}

template <int OPT, bool GRAD_BF16, int FWD, bool DIL, bool TAU0>
__global__ void __launch_bounds__(512, 6)
k_step(const StepArgs a)
{
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t tile = blockIdx.x, b0 = TAU0 ? 0u : blockIdx.y;
    const TileLds L = step_lds<DIL>(a);
    if ((uint64_t)(tile + 1u) * kTileCoords <= a.n)
        step_tile<OPT, GRAD_BF16, FWD, DIL, TAU0, false, true>(a, tile, b0, wave, lane, L);
    else
        step_tile<OPT, GRAD_BF16, FWD, DIL, TAU0, false, false>(a, tile, b0, wave, lane, L);
}

// The same for small stages, which add up their tiles' places themselves (a delay).  Few tiles, whose chains of waits are the time: with at
// most 80 scalar registers eight waves a SIMD are resident, not seven.  us a step, without / with that: R = 4 500k 16.5 / 15.2, 1M 29.0 / 28.6,
// R = 8 2M 99.8 / 99.3.
template <int OPT, bool GRAD_BF16, int FWD, bool DIL>
__global__ void __launch_bounds__(512, 6) __attribute__((amdgpu_num_sgpr(80)))
k_step_small(const StepArgs a)
{
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t tile = blockIdx.x, b0 = blockIdx.y;
    const TileLds L = step_lds<DIL>(a);
    if ((uint64_t)(tile + 1u) * kTileCoords <= a.n)
        step_tile<OPT, GRAD_BF16, FWD, DIL, false, true, true>(a, tile, b0, wave, lane, L);
    else
        step_tile<OPT, GRAD_BF16, FWD, DIL, false, true, false>(a, tile, b0, wave, lane, L);
}

// A step that neither sends nor receives (between two averaging rounds, interval > 1; am_host::local_step_alone): the local step alone,
// a wave per tile of one replica, replica after replica, so that few streams are on their way at a time, without LDS and barriers.  us a
// step, by k_step / by this: AdamW with look-ahead, R = 8 30M 1324 / 1215 (6.3 TB/s), 3M 136.2 / 126.8.
// grid = (ceil(tiles / 4), replicas); blockDim = 256
template <int OPT, bool GRAD_BF16, int FWD>
__global__ void __launch_bounds__(256)
k_step_local(const StepArgs a)
{
    const uint32_t lane = threadIdx.x & 63u, loff = lane * 4u;
    const uint32_t tile = blockIdx.x * 4u + (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), i = blockIdx.y;
    if (tile >= a.ntiles) return;
    const uint64_t tbase = (uint64_t)tile * kTileCoords, mu = tbase + loff;
    const int nvalid = tbase + kTileCoords <= a.n ? 4 : (mu >= a.n ? 0 : (a.n - mu >= 4u ? 4 : (int)(a.n - mu)));
    const ReplicaArgs rep = a.rep[8u * (i >> a.rb_shift) + (i & (a.rb - 1u))];
    GroupIn in;
    load_group<OPT, GRAD_BF16>(rep, tbase, loff, nvalid, in);
    __builtin_amdgcn_sched_barrier(0);
    if (a.do_next && i == 0u) {                              // how many lines the tile sends next step
        SubsetKey key = a.key;
        key.step_lo = a.step_lo[2]; key.step_hi = a.step_hi[2];
        uint32_t count;
        (void)wave_prefix_mask4(member_mask(key, (uint64_t)tile * 64u + lane, nvalid), count);
        if (lane == 0) a.next_lines[tile] = (uint8_t)((count * a.rb + kLineFloats - 1u) / kLineFloats);
    }
    F4 w_hat, m_new, v_new;
    local_step<OPT, true>(a, rep, i, in, w_hat, m_new, v_new);
    if (OPT == kOptSgdMomentum || OPT == kOptAdam) store_tile_f32x4(rep.m + tbase, loff, nvalid, m_new, a.through != 0u);
    if (OPT == kOptAdam) store_tile_f32x4(rep.v + tbase, loff, nvalid, v_new, a.through != 0u);
    store_weights<FWD>(a, rep, tbase, loff, nvalid, in, w_hat, w_hat);
}

// V floats at byte `byte` of a resource; past its end nothing moves.
template <int V> struct Entry { float v[V]; };
template <int V>
__device__ __forceinline__ void store_entry(__amdgpu_buffer_rsrc_t r, uint32_t byte, const Entry<V> &x)
{
    if constexpr (V == 2) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2u, x), r, (int)byte, 0, 0);
    else __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, x), r, (int)byte, 0, 0);
}
template <int V>
__device__ __forceinline__ Entry<V> load_entry(const float *p)
{
    if constexpr (V == 2) return __builtin_bit_cast(Entry<V>, *reinterpret_cast<const v2f *>(p));
    else return __builtin_bit_cast(Entry<V>, *p);
}
template <int V>
__device__ __forceinline__ void store_entry(float *p, const Entry<V> &x)
{
    if constexpr (V == 2) *reinterpret_cast<v2f *>(p) = __builtin_bit_cast(v2f, x);
    else *p = x.v[0];
}

constexpr uint32_t kWaveBlockShift = 3;                      // log2 of a block's replicas, in the kernel below
constexpr uint32_t kWaveTurn = kStageFloats >> kWaveBlockShift;         // received coordinates of a turn

// The step of large stages of blocks of eight replicas with a delay, in rounds that send (am_host::step_by_waves; steps between rounds go through k_step_local): a workgroup is ONE wave, which takes V
// neighbouring replicas of a block through one tile; no barrier, and what the replicas of a tile share meets in the L2.
// What it buys is order.  The stream mix moves faster the fewer streams are on their way at a time and the finer the grain in which waves come and go
// (without arithmetic, 125.8M x 8: a workgroup of eight waves a tile 5.7 TB/s with three of them a compute unit and 6.2 with two; one-wave workgroups, 16 a
// compute unit, 6.1 with a tile's replicas side by side and 6.6 with the replicas of a chunk of 512 tiles one after the other).  So the grid
// runs over the tiles of a chunk, then its replicas, then the chunks: the waves of one tile are on the same XCD (consecutive workgroups go round the eight) and
// near enough in time that its ring lines and interleaved EMA entries are fetched from memory once and that the parts of the lines they write merge in the
// L2 (GB read + written a launch by the counters, k_step / this: interleaved 125.8M x 8 17.14 + 16.73 / 17.15 + 16.54, per replica 19.64 + 18.59 either way; this alone:
// bf16 without correction 125.8M x 16 28.38 + 28.32).  The price is in requests: every wave asks for the ring lines, and sends V values of a coordinate at a time, so it pays up to a fraction of 10 %.  Interleaved EMA entries cost little where the lane of rank c takes those of the received
// coordinate c, one load and one store a wave, and the weights change hands through LDS (every lane taking its own four coordinates' entries, eight scattered accesses: 5814 / 5846 us,
// no gain); narrower blocks have too little to gain.
// us a step, k_step / this, median of ten processes that allocate their arrays once, on two cards (one process differs from the next by less than 2 % in either): interleaved, R = 8 125.8M 5 % 5897 / 5746
// (33.69 GB: 5.86 TB/s), 31.5M 1460 / 1415, R = 12 30M 2195 / 2103; per replica, R = 8 with factors 31.5M 1688 / 1576, 125.8M 6850 / 6400; bf16 without correction R = 16 125.8M 1 % 9914 / 9480.  On arrays that a
// process frees and allocates again many times both get faster, k_step the more: 125.8M x 8 interleaved 5456 / 5525, per replica 6165 / 6165.
// Bound by memory: with a generator of a few instructions in the place of the hashing it takes as long.
template <int OPT, bool GRAD_BF16, int FWD, bool DIL, int V, bool FULL>
__device__ __forceinline__ void step_wave(const StepArgs &a, const uint32_t tile, const uint32_t i0, const uint32_t lane, float *lds)
{
    constexpr uint32_t sh = kWaveBlockShift, turn = kWaveTurn;
    const uint32_t b = i0 >> sh, slot = i0 & ((1u << sh) - 1u);
    const uint64_t group = (uint64_t)tile * 64u + lane;
    const uint64_t mu = group * 4u;
    const int nvalid = FULL ? 4 : (mu >= a.n ? 0 : (a.n - mu >= 4u ? 4 : (int)(a.n - mu)));
    const uint64_t tbase = (uint64_t)tile * kTileCoords;
    const uint32_t loff = lane * 4u;
    const uint64_t block_floats = (uint64_t)a.cap_lines * kLineFloats;
    constexpr uint32_t kNone = 0x40000000u;                  // past the end of every resource
    float *const ring = lds, *const mean = ring + a.nblocks * kStageFloats;
    float *const x_lds = mean;                               // (DIL) [V][turn] my replicas' weights of the received coordinates of a turn, by rank
    uint8_t *const list = reinterpret_cast<uint8_t *>(x_lds + V * turn);     // (DIL) those coordinates

    // ---- dense operands: nothing else is requested before them.  (Until everything is requested the wave goes before the
    //      older ones of its SIMD, which have arithmetic to do: us a step without / with that, per replica 31.5M x 8 1648 / 1632, interleaved 1447 / 1425.)
    __builtin_amdgcn_s_setprio(3);
    const ReplicaArgs *const rep = a.rep + 8u * b + slot;
    GroupIn in[V];
#pragma unroll
    for (int v = 0; v < V; ++v) load_group<OPT, GRAD_BF16>(rep[v], tbase, loff, nvalid, in[v]);
    __builtin_amdgcn_sched_barrier(0);

    const uint32_t word_s = uniform_load(a.send_meta, tile), base_s = uniform_load(a.send_sb_base, tile / kTilesPerSuperblock);
    uint32_t word_r = 0, base_r = 0;
    if (a.do_recv) { word_r = uniform_load(a.recv_meta, tile); base_r = uniform_load(a.recv_sb_base, tile / kTilesPerSuperblock); }
    // a tile whose lines would pass the slot capacity is left out, at send and at receive alike
    const uint32_t first_s = base_s + (word_s & 0xFFFFFFu), first_r = base_r + (word_r & 0xFFFFFFu);
    uint32_t lines_s = word_s >> 24, lines_r = word_r >> 24;
    if ((uint64_t)first_s + lines_s > a.cap_lines) lines_s = 0;
    if ((uint64_t)first_r + lines_r > a.cap_lines) lines_r = 0;

    // ---- what every replica sent tau rounds ago goes straight into LDS, a kilobyte of every block (a turn) at a time
    auto request_ring = [&](const uint32_t c0) {             // from rank c0 on
        const uint32_t at = (c0 << sh) + loff;
        if (at < lines_r * kLineFloats) {
            const float *src = a.ring_recv + (uint64_t)first_r * kLineFloats + at;
            for (uint32_t q = 0; q < a.nblocks; ++q) lds_dma_16(src + q * block_floats, ring + q * kStageFloats);
        }
    };
    SubsetKey key = a.key;
    uint32_t mask_recv = 0, rank_recv = 0, count_recv = 0;
    bool half_recv = false;                                  // the 64 bytes of a per-replica array (4 lanes) holding the group receive something
    // the rank in the turn from c0 on of the lane's coordinates that are received, one after the other
    auto each = [&](const uint32_t c0, auto use) {
        uint32_t c = rank_recv - c0;                         // (wraps below the turn's first: not this turn's)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t bit = (mask_recv >> j) & 1u;
            if (bit && c < turn) use(j, c);
            c += bit;
        }
    };
    // interleaved EMA entries: the lane of rank c takes those of its coordinate, one request a wave
    Entry<V> entry = {};
    auto request_entries = [&](const uint32_t c0) {
        each(c0, [&](int j, uint32_t c) { list[c] = (uint8_t)(loff + (uint32_t)j); });
        wave_lds_sync();
        if (lane < turn && c0 + lane < count_recv) entry = load_entry<V>(a.d[b] + ((tbase + list[lane]) << sh) + slot);
    };
    auto mean_of = [&]() {                                   // of the coordinate of the lane's rank
        return replica_mean<1 << sh, true>(a, ring, lane, kStageFloats);
    };
    if (lines_r) {
        request_ring(0u);
        key.step_lo = a.step_lo[0]; key.step_hi = a.step_hi[0];
        mask_recv = member_mask(key, group, nvalid);
        half_recv = ((__ballot(mask_recv != 0u) >> (lane & ~3u)) & 0xFull) != 0ull;
        if (!DIL && a.ema && half_recv) {
#pragma unroll
            for (int v = 0; v < V; ++v) in[v].d = load_f32x4(a.d[i0 + v] + tbase, loff, nvalid);
        }
        rank_recv = wave_prefix_mask4(mask_recv, count_recv);
        if (DIL) request_entries(0u);
    }
    uint32_t mask_send = 0, rank_send = 0, count_send = 0;
    if (lines_s) {
        key.step_lo = a.step_lo[1]; key.step_hi = a.step_hi[1];
        mask_send = member_mask(key, group, nvalid);
        rank_send = wave_prefix_mask4(mask_send, count_send);
    }
    if (a.do_next && i0 == 0u) {                             // how many lines the tile sends next step
        key.step_lo = a.step_lo[2]; key.step_hi = a.step_hi[2];
        uint32_t count;
        (void)wave_prefix_mask4(member_mask(key, group, nvalid), count);
        if (lane == 0) a.next_lines[tile] = (uint8_t)(((count << sh) + kLineFloats - 1u) / kLineFloats);
    }
    __builtin_amdgcn_sched_barrier(0);                       // (the operands' conversions stay behind the hashing)
    __builtin_amdgcn_s_setprio(0);

    F4 w_hat[V], w_new[V], m_new[V], v_new[V];
#pragma unroll
    for (int v = 0; v < V; ++v) local_step<OPT, true>(a, rep[v], i0 + v, in[v], w_hat[v], m_new[v], v_new[v]);
    lds_dma_wait();                                          // (before the first store: the wait counts stores, too)
    wave_lds_sync();
#pragma unroll
    for (int v = 0; v < V; ++v) {
        if (OPT == kOptSgdMomentum || OPT == kOptAdam) store_tile_f32x4(rep[v].m + tbase, loff, nvalid, m_new[v], a.through != 0u);
        if (OPT == kOptAdam) store_tile_f32x4(rep[v].v + tbase, loff, nvalid, v_new[v], a.through != 0u);
        w_new[v] = w_hat[v];
    }

    // ---- send: my replicas' values of every coordinate at its rank, zeros in the rest of the tile's last line.  (The slots of absent replicas are
    //      not written: they stay zero, as am_init_state leaves them, and other kernels of the same stage add them up.)
    if (lines_s) {
        const __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc(a.ring_send + b * block_floats + (uint64_t)first_s * kLineFloats, 0, lines_s * kLineFloats * 4u, 0x00020000);
        uint32_t c = rank_send;
        Entry<V> x;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t bit = (mask_send >> j) & 1u;
#pragma unroll
            for (int v = 0; v < V; ++v) x.v[v] = w_hat[v].v[j];
            store_entry<V>(out, bit ? ((c << sh) + slot) * 4u : kNone, x);
            c += bit;
        }
#pragma unroll
        for (int v = 0; v < V; ++v) x.v[v] = 0.f;
        store_entry<V>(out, (((count_send + lane) << sh) + slot) * 4u, x);
    }

    // ---- receive: the lane of rank c forms the mean (in fp64, in replica order)
    auto next_turn = [&](const uint32_t c0) {                // nearly always there is none
        wave_lds_sync();
        lds_access_wait();                                   // what the last turn read from the ring's stretch has been read
        request_ring(c0);
        if (DIL) request_entries(c0);
        lds_dma_wait();
        wave_lds_sync();
    };
    if (DIL) {                                               // and the new entries and weights of its coordinate, which change hands through LDS
        for (uint32_t c0 = 0; c0 < count_recv; c0 += turn) {
            if (c0) next_turn(c0);
            each(c0, [&](int j, uint32_t c) {
#pragma unroll
                for (int v = 0; v < V; ++v) x_lds[v * turn + c] = w_hat[v].v[j];
            });
            wave_lds_sync();
            if (lane < turn && c0 + lane < count_recv) {
                const float abar = mean_of();
                const Entry<V> sent = *reinterpret_cast<const Entry<V> *>(ring + b * kStageFloats + (lane << sh) + slot);
                Entry<V> d_new;
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    d_new.v[v] = (float)fma(a.coef_d, (double)entry.v[v], a.coef_s * ((double)x_lds[v * turn + lane] - (double)sent.v[v]));
                    x_lds[v * turn + lane] = (float)((double)abar + (double)d_new.v[v]);
                }
                store_entry<V>(a.d[b] + ((tbase + list[lane]) << sh) + slot, d_new);
            }
            wave_lds_sync();
            each(c0, [&](int j, uint32_t c) {
#pragma unroll
                for (int v = 0; v < V; ++v) w_new[v].v[j] = x_lds[v * turn + c];
            });
        }
    } else if (count_recv) {                                 // every lane picks up those of its own coordinates (a lane with
                                                             // fewer than four reads entry 0 and drops it, so that the reads are in flight together)
        for (uint32_t c0 = 0; c0 < count_recv; c0 += turn) {
            if (c0) next_turn(c0);
            if (lane < turn && c0 + lane < count_recv) mean[lane] = mean_of();
            wave_lds_sync();
            uint32_t c = rank_recv - c0;                     // (wraps below the turn's first: not this turn's)
            bool mine[4];
            float abar[4];
            Entry<V> sent[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t bit = (mask_recv >> j) & 1u;
                mine[j] = bit && c < turn;
                const uint32_t at = mine[j] ? c : 0u;
                abar[j] = mean[at];
                sent[j] = *reinterpret_cast<const Entry<V> *>(ring + b * kStageFloats + (at << sh) + slot);
                c += bit;
            }
#pragma unroll
            for (int v = 0; v < V; ++v)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (a.ema) {
                        const float d_new = (float)fma(a.coef_d, (double)in[v].d.v[j], a.coef_s * ((double)w_hat[v].v[j] - (double)sent[j].v[v]));
                        if (mine[j]) { in[v].d.v[j] = d_new; w_new[v].v[j] = (float)((double)abar[j] + (double)d_new); }
                    } else if (mine[j]) {
                        w_new[v].v[j] = abar[j];
                    }
                }
        }
        if (a.ema && half_recv) {
#pragma unroll
            for (int v = 0; v < V; ++v) store_tile_f32x4(a.d[i0 + v] + tbase, loff, nvalid, in[v].d, a.through != 0u);
        }
    }
#pragma unroll
    for (int v = 0; v < V; ++v) store_weights<FWD>(a, rep[v], tbase, loff, nvalid, in[v], w_hat[v], w_new[v]);
}

// Floats of dynamic LDS that it needs.
__host__ __device__ inline uint32_t step_wave_lds_floats(uint32_t nblocks, bool d_interleaved, uint32_t v)
{
    return nblocks * kStageFloats + (d_interleaved ? kWaveTurn * v + kWaveTurn / 4u : kWaveTurn);
}

// grid = am_host::wave_step_grid(); blockDim = 64; dynamic LDS = step_wave_lds_floats() floats, or more where fewer are to be resident
template <int OPT, bool GRAD_BF16, int FWD, bool DIL, int V>
__global__ void __launch_bounds__(64, 4)
k_step_wave(const StepArgs a)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];
    const uint32_t tile = (blockIdx.z * gridDim.y + blockIdx.y) * kWaveChunk + blockIdx.x % kWaveChunk, i0 = V * (blockIdx.x / kWaveChunk);
    if (tile >= a.ntiles) return;
    if ((uint64_t)(tile + 1u) * kTileCoords <= a.n) step_wave<OPT, GRAD_BF16, FWD, DIL, V, true>(a, tile, i0, threadIdx.x, lds);
    else step_wave<OPT, GRAD_BF16, FWD, DIL, V, false>(a, tile, i0, threadIdx.x, lds);
}

// tau = 0 with at most kSyncWaves replicas: the average is of this step's values, so a tile needs all its
// replicas at once.  One workgroup per tile, one wave per replica whatever its block: every operand is read once
// and every local step made once, the stepped weights of the sampled coordinates meet in LDS (they are also
// the lines that are sent), and from there on it is the delayed kernel.  (A workgroup of one block's waves
// walking the blocks reads the operands of all blocks but its first twice and steps every replica twice.
// Measured, us a step before / after: R = 12, 7.1M, AdamW, no correction 529 / 417 (5.7 TB/s), R = 16, 10M, bf16 1149 /
// 796, R = 8, 10M, EMA 500 / 460 (interleaved) and 531 / 488 (per replica), R = 3 213 / 193.)
constexpr uint32_t kSyncWaves = 16;

template <int OPT, bool GRAD_BF16, int FWD, bool DIL, bool FULL>
__device__ __forceinline__ void step_tile_sync(const StepArgs &a, const uint32_t tile, const uint32_t wave, const uint32_t lane, const TileLds &L)
{
    const uint32_t R = a.replicas, rb = a.rb, sh = a.rb_shift;
    const uint32_t b = wave >> sh, slot = wave & (rb - 1u), flat = wave * 64u + lane, threads = R * 64u;
    const uint64_t group = (uint64_t)tile * 64u + lane;
    const uint64_t mu = group * 4u;
    const int nvalid = FULL ? 4 : (mu >= a.n ? 0 : (a.n - mu >= 4u ? 4 : (int)(a.n - mu)));
    const uint64_t tbase = (uint64_t)tile * kTileCoords;
    const uint32_t loff = lane * 4u, tile_floats = kTileCoords * rb;
    const uint64_t block_floats = (uint64_t)a.cap_lines * kLineFloats;

    const ReplicaArgs rep = a.rep[8u * b + slot];
    GroupIn in;
    load_group<OPT, GRAD_BF16>(rep, tbase, loff, nvalid, in);
    __builtin_amdgcn_sched_barrier(0);

    // ---- the subset: hashed by the first wave of every block (which requests its block's lines of an
    //      interleaved d), and by every wave where it steers the loads of a per-replica d
    GroupSubsets s;
    s.mask_send = s.mask_recv = s.rank_send = s.rank_recv = s.d_slot = 0;
    s.half_recv = false;
    const uint32_t lpl = 8u >> sh, leader = lane & ~(lpl - 1u);            // lanes (groups) per 128-byte line of an interleaved d
    auto leaders_of = [&](const uint32_t mask) {                           // bit = first lane of a touched line of d
        const uint64_t any = __ballot(mask != 0u);
        return (uint64_t)__ballot(((any >> leader) & ((1ull << lpl) - 1ull)) != 0ull && lane == leader);
    };
    SubsetKey key = a.key;
    if (slot == 0u || (!DIL && a.ema)) {
        key.step_lo = a.step_lo[1]; key.step_hi = a.step_hi[1];
        const uint32_t mask = member_mask(key, group, nvalid);
        if (wave == 0u) L.masks[lane] = (uint8_t)mask;
        if (DIL && a.ema) {
            const uint64_t leaders = leaders_of(mask);
            const uint32_t nlines = (uint32_t)__popcll(leaders);
            const uint64_t any = __ballot(mask != 0u);
            if ((leaders >> lane) & 1ull) L.list[__popcll(leaders & ((1ull << lane) - 1ull))] = touched_line(lane, mask, any, sh);    // (the same from every block)
            wave_lds_sync();
            const float *src = a.d[b] + (uint64_t)tile * tile_floats + (lane & 7u) * 4u;
            for (uint32_t q0 = 0; q0 < nlines; q0 += 8u) {
                const uint32_t q = q0 + (lane >> 3);
                if (q < nlines) lds_dma_16(src + line_index(L.list[q]) * kLineFloats, L.d + b * tile_floats + q0 * kLineFloats);
            }
        }
        if (!DIL && a.ema) {
            const uint64_t any = __ballot(mask != 0u);
            s.half_recv = ((any >> (lane & ~3u)) & 0xFull) != 0ull;
            load_group_sparse<DIL>(a, wave, tbase, loff, nvalid, s, in);
        }
    }
    if (a.do_next && wave == (R > 1u ? 1u : 0u)) {
        key.step_lo = a.step_lo[2]; key.step_hi = a.step_hi[2];
        uint32_t count;
        (void)wave_prefix_mask4(member_mask(key, group, nvalid), count);
        if (lane == 0) a.next_lines[tile] = (uint8_t)((count * rb + kLineFloats - 1u) / kLineFloats);
    }

    // ---- where the tile's lines sit in the slot
    uint32_t first = 0, lines;
    if (a.sum_lines) {
        lines = lines_of_tile(a.send_lines, tile);
        const uint32_t share = lines_before(a.send_lines, tile, wave, R, lane);
        if (lane == 0) L.part[wave] = share;
    } else {
        const uint32_t word = uniform_load(a.send_meta, tile);
        first = uniform_load(a.send_sb_base, tile / kTilesPerSuperblock) + (word & 0xFFFFFFu);
        lines = word >> 24;
    }
    for (uint32_t q = 0; q < a.nblocks; ++q)               // line tails and the slots of absent replicas are zero
        for (uint32_t f = flat; f < lines * 8u; f += threads)
            *reinterpret_cast<v4f *>(L.recv + q * tile_floats + f * 4u) = v4f{0.f, 0.f, 0.f, 0.f};

    F4 w_hat, m_new, v_new;
    local_step<OPT, false>(a, rep, wave, in, w_hat, m_new, v_new);
    lds_dma_wait();
    __syncthreads();
    if (OPT == kOptSgdMomentum || OPT == kOptAdam) store_tile_f32x4(rep.m + tbase, loff, nvalid, m_new, a.through != 0u);
    if (OPT == kOptAdam) store_tile_f32x4(rep.v + tbase, loff, nvalid, v_new, a.through != 0u);

    if (a.sum_lines) {
        for (uint32_t w = 0; w < R; ++w) first += L.part[w];
        first = (uint32_t)__builtin_amdgcn_readfirstlane((int)first);
        if (flat == 0u) write_send_word(a, tile, first, lines);
    }
    if ((uint64_t)first + lines > a.cap_lines) lines = 0;  // a tile whose lines would pass the slot capacity is left out
    s.mask_send = s.mask_recv = lines ? (uint32_t)L.masks[lane] : 0u;
    uint32_t count, d_lines = 0;
    s.rank_send = s.rank_recv = wave_prefix_mask4(s.mask_recv, count);
    const uint64_t any = __ballot(s.mask_recv != 0u);
    s.half_recv = ((any >> (lane & ~3u)) & 0xFull) != 0ull;
    if (DIL && a.ema) {
        const uint64_t leaders = leaders_of(s.mask_recv);
        d_lines = (uint32_t)__popcll(leaders);
        s.d_slot = (uint32_t)__popcll(leaders & ((1ull << leader) - 1ull)) * kLineFloats + (lane & (lpl - 1u)) * 4u * rb;
    }

    float abar[4] = {0.f, 0.f, 0.f, 0.f};
    if (count) {                                           // same for the whole workgroup
        uint32_t c = s.rank_send;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if ((s.mask_send >> j) & 1u) L.recv[b * tile_floats + (c++) * rb + slot] = w_hat.v[j];
        __syncthreads();
        for (uint32_t q = 0; q < a.nblocks; ++q)           // whole lines leave with 16 bytes per thread
            for (uint32_t f = flat; f < lines * 8u; f += threads) {
                float *dst = a.ring_send + q * block_floats + (uint64_t)first * kLineFloats + f * 4u;
                __builtin_nontemporal_store(*reinterpret_cast<const v4f *>(L.recv + q * tile_floats + f * 4u), reinterpret_cast<v4f *>(dst));
            }
        tile_means<false>(a, L, flat, threads, count);
        __syncthreads();
        c = s.rank_recv;
#pragma unroll
        for (int j = 0; j < 4; ++j) { const uint32_t bit = (s.mask_recv >> j) & 1u; abar[j] = L.abar[bit ? c : 0u]; c += bit; }
    }
    TileLds mine = L;
    if (DIL) mine.d = L.d + b * tile_floats;
    finish_replica<FWD, DIL, true, false>(a, rep, wave, slot, tbase, loff, nvalid, s, count != 0u, abar, in, w_hat, nullptr, mine);
    if (DIL && a.ema && d_lines) {
        __syncthreads();
        for (uint32_t q = 0; q < a.nblocks; ++q)
            for (uint32_t f = flat; f < d_lines * 8u; f += threads) {
                const uint32_t line = L.list[f >> 3];
                if (!half_received(line, (f >> 2) & 1u)) continue;
                float *dst = a.d[q] + (uint64_t)tile * tile_floats + line_index(line) * kLineFloats + (f & 7u) * 4u;
                __builtin_nontemporal_store(*reinterpret_cast<const v4f *>(L.d + q * tile_floats + f * 4u), reinterpret_cast<v4f *>(dst));
            }
    }
}

__host__ __device__ inline uint32_t step_sync_lds_floats(uint32_t rb, uint32_t nblocks, bool d_interleaved)
{
    return nblocks * kTileCoords * rb * (d_interleaved ? 2u : 1u) + 64u + 32u + kSyncWaves + kTileCoords;
}

// grid = tiles; blockDim = 64 replicas; dynamic LDS = step_sync_lds_floats() floats
// At most 80 scalar registers: with the trap handler's reserve more leave seven waves a SIMD, and two workgroups of 13
// to 16 waves a compute unit need eight on one of them.  With interleaved EMA vectors AdamW had 83: us a step relative to
// the walking form at p = 50 %, 13 replicas of 1.5M 1.15, 16 of 1.5M 1.08; with 80, 13 of 1M 0.95, 16 of 1M 0.77.
template <int OPT, bool GRAD_BF16, int FWD, bool DIL>
__global__ void __launch_bounds__(64 * kSyncWaves, 6) __attribute__((amdgpu_num_sgpr(80)))
k_step_sync(const StepArgs a)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t tile = blockIdx.x, all_floats = a.nblocks * kTileCoords * a.rb;
    TileLds L;
    L.recv = L.send = lds;
    L.d = L.recv + all_floats;
    L.list = reinterpret_cast<uint32_t *>(L.d + (DIL ? all_floats : 0u));
    L.masks = reinterpret_cast<uint8_t *>(L.list + 64);
    L.part = L.list + 96;
    L.abar = reinterpret_cast<float *>(L.list + 96 + kSyncWaves);
    if ((uint64_t)(tile + 1u) * kTileCoords <= a.n) step_tile_sync<OPT, GRAD_BF16, FWD, DIL, true>(a, tile, wave, lane, L);
    else step_tile_sync<OPT, GRAD_BF16, FWD, DIL, false>(a, tile, wave, lane, L);
}

// =============================================================================================
// Averaging alone (am_sparse_average): subset, send, replica mean, EMA correction and scatter
// (asynchronous sparse averaging equations) on weights the caller has already stepped.
//
// Only lines that hold a selected coordinate move, so the call lives on how many of those lines are
// in flight, not on bytes.  The fused kernel's shape (a wave per replica, staging in LDS, four
// barriers a tile) keeps four tiles per compute unit in flight; here ONE wave owns one (tile, block
// of replicas) and keeps the block's RB replicas side by side in registers: lane l holds the four
// coordinates of its group for every replica of the block.  The RB values of a coordinate are one
// aligned stretch of 4 RB bytes in the ring slot and in the interleaved EMA vector ([coordinate][RB]),
// so the lane reads and writes them with one or two 128-bit accesses: no barrier, two dozen
// tiles per compute unit in flight.  (Several lanes write parts of one line within a few
// instructions of each other; these are ordinary cached stores, which the L2 merges.)
// What bounds it is the chain of waits a wave goes through, so everything a tile reads is requested at
// once: the first kilobyte of its ring lines (256 / RB received coordinates: nearly always all of them)
// and their EMA entries go straight into the wave's own stretch of LDS beside the loads of the weights
// (read where they are used, they are up to eight waits in a row); more coordinates come a kilobyte at a
// time.  The staging does not pay everywhere (am_host::average_staged); where it does not, the ring and the EMA
// entries are read in place.
// Few of a lane's coordinates are members (one in twenty at p = 5 %), so with blocks of four and eight replicas the lanes do not
// work on their own coordinates one bit position after the other, with a few lanes busy each time: the members' values change
// hands through LDS and a lane takes four replicas of one member, for the send as for the receive (937 -> about 500
// vector instructions a tile; the sent lines leave with 16 bytes a lane side by side).  And memory writes whole 64-byte halves of a line at
// half a line's cost (reads move the line whatever part of it is asked for), so only halves that hold a received
// coordinate are written: 56 % at p = 5 %, 81 % of the lines.  How many workgroups are resident: am_host::average_workgroups.
// us a call before / after the three: interleaved, R = 8, 125.8M 5 % 1693 / 1567 (7.7 GB: 4.9 TB/s), 1 % 804 / 640, 31.5M 0.5 % 184 / 148,
// 2 % 262 / 257, 10 % 550 / 519, 40 % 972 / 937, 7M 5 % 94 / 83.5, 2M 37.3 / 31.6, 500k 13.0 / 11.3; R = 12, 31.5M 5 % 688 / 659;
// R = 4 240 / 228; no correction 325 / 304; per replica, 125.8M 5 % 2681 / 2413, 31.5M 1 % 287 / 266.
// Arithmetic and its order are those of the fused kernel: mean in fp64 in replica order, rounded to
// fp32; d <- coef_d d + coef_s (w^ - sent) and w = mean + d in fp64, rounded once each.
// =============================================================================================
template <int RB>
__device__ __forceinline__ void store_block_values(float *p, const float (&x)[RB])
{
    if constexpr (RB == 8) {
        *reinterpret_cast<v4f *>(p) = v4f{x[0], x[1], x[2], x[3]};
        *reinterpret_cast<v4f *>(p + 4) = v4f{x[4], x[5], x[6], x[7]};
    } else if constexpr (RB == 4) {
        *reinterpret_cast<v4f *>(p) = v4f{x[0], x[1], x[2], x[3]};
    } else if constexpr (RB == 2) {
        *reinterpret_cast<v2f *>(p) = v2f{x[0], x[1]};
    } else {
        p[0] = x[0];
    }
}

// The values block `b` of the replicas sends for the tile: the RB values of a selected coordinate side
// by side at the coordinate's rank; the rest of the tile's last line is zero.
template <int RB>
__device__ __forceinline__ void average_send_block(float *slot, const F4 (&w)[RB], uint32_t mask_send, uint32_t rank_send,
                                                   uint32_t count_send, uint32_t room, uint32_t lane)
{
    uint32_t c = rank_send;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (((mask_send >> j) & 1u) && c < room) {             // (the rank is below that by construction of the table)
            float x[RB];
#pragma unroll
            for (int k = 0; k < RB; ++k) x[k] = w[k].v[j];
            store_block_values<RB>(slot + (uint64_t)c * RB, x);
            ++c;
        }
    }
    if (count_send + lane < room) {                            // fewer than 32 / RB <= 32 lanes
        float x[RB];
#pragma unroll
        for (int k = 0; k < RB; ++k) x[k] = 0.f;
        store_block_values<RB>(slot + (uint64_t)(count_send + lane) * RB, x);
    }
}

// Coordinate j of the group receives the old average abar: EMA of the staleness of each replica of the
// block (own[k] = what replica k itself sent), corrected weight.  dp: the coordinate's RB entries of the
// interleaved EMA vector (DIL; in memory or their copy in LDS), else the entries are in dv.  HALVES: the
// replicas' fp64 values are formed four at a time, not eight (76 registers instead of 84).
template <bool DIL, int RB, bool HALVES>
__device__ __forceinline__ void average_receive(const StepArgs &a, int j, float abar, const float (&own)[RB], float *dp, F4 (&w)[RB], F4 (&dv)[RB])
{
    if (a.ema) {
        float d_new[RB];
        if (DIL) {
            load_block_values<RB>(dp, d_new);
        } else {
#pragma unroll
            for (int k = 0; k < RB; ++k) d_new[k] = dv[k].v[j];
        }
#pragma unroll
        for (int k = 0; k < RB; ++k) {
            if (HALVES && k == 4) __builtin_amdgcn_sched_barrier(0);
            d_new[k] = (float)fma(a.coef_d, (double)d_new[k], a.coef_s * ((double)w[k].v[j] - (double)own[k]));
            w[k].v[j] = (float)((double)abar + (double)d_new[k]);
            if (!DIL) dv[k].v[j] = d_new[k];
        }
        if (DIL) store_block_values<RB>(dp, d_new);
    } else {
#pragma unroll
        for (int k = 0; k < RB; ++k) w[k].v[j] = abar;
    }
}

// Blocks of four and eight replicas: a coordinate's values change hands through LDS, and lanes work on four of them each
// (blocks of fewer have stretches shorter than 16 bytes).
template <int RB, bool STAGED>
constexpr bool kAverageItems = STAGED && RB >= 4;
// Bytes of dynamic LDS of a workgroup: per wave a kilobyte of ring values per block, and (items) one of weights, one of EMA
// entries and the list of received coordinates.
template <bool DIL, int RB>
__host__ __device__ constexpr uint32_t average_wave_bytes(uint32_t nblocks)
{
    return (nblocks * kStageFloats + (kAverageItems<RB, true> ? 2u * kStageFloats + (DIL ? 64u : 0u) : 0u)) * (uint32_t)sizeof(float);
}

// grid = (ceil(tiles / 4), blocks) (TAU0: (ceil(tiles / 4), 1)); blockDim = 256: four waves, each with
// a tile and (STAGED) average_wave_bytes() of LDS of its own, or more where fewer are to be resident.
// DIL: the EMA vectors are interleaved ([coordinate][RB] per block); else one flat array per replica.
// TAU0: the average is of this very call's values (tau = 0): the wave walks all blocks of its tile,
// once for the sums and the send, once more for the update (another wave must not rewrite a block's
// weights while this one still needs them for the mean).
// STAGED: a kilobyte at a time through LDS; else (where am_host::average_staged says so) the ring and the
// interleaved EMA entries are read where their values are used.
// At most 128 registers (the staged form with interleaved EMA entries and items takes 72); in place with
// interleaved EMA entries, where latency is the cost, at most 80 and 24 tiles: 20 replicas, us a call relative to
// the form before the staging, 500k p = 0.2 0.85, p = 0.3 0.89, 900k p = 0.2 0.94 (slower than that form at 84 registers).
// TABLE: where the weights' pointers are (am_host::average_weights_table).
template <bool DIL, int RB, bool TAU0, bool STAGED, bool TABLE>
__global__ void __launch_bounds__(256, (DIL && !TAU0 && !STAGED) ? 6 : 4)
k_average(const StepArgs a)
{
    constexpr uint32_t kPerLine = kLineFloats / RB;                        // coordinates a ring line holds
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t tile = blockIdx.x * 4u + wave, b0 = TAU0 ? 0u : blockIdx.y;
    // small stage: the lines before the workgroup's first tile, a share a wave, and those of its own tiles before mine
    uint32_t first_sum = 0, lines_sum = 0;
    if (a.sum_lines) {
        __shared__ uint32_t part[4];
        const uint32_t share = lines_before(a.send_lines, blockIdx.x * 4u, wave, 4u, lane);
        if (lane == 0) part[wave] = share;
        __syncthreads();
        first_sum = part[0] + part[1] + part[2] + part[3];
        for (uint32_t w = 0; w < wave; ++w) first_sum += tile < a.ntiles ? lines_of_tile(a.send_lines, blockIdx.x * 4u + w) : 0u;
        first_sum = (uint32_t)__builtin_amdgcn_readfirstlane((int)first_sum);
    }
    if (tile >= a.ntiles) return;
    if (a.sum_lines) {
        lines_sum = lines_of_tile(a.send_lines, tile);
        if (b0 == 0u && lane == 0) write_send_word(a, tile, first_sum, lines_sum);
    }
    const uint32_t R = a.replicas;
    const uint64_t group = (uint64_t)tile * 64u + lane;
    const uint64_t mu = group * 4u;
    const int nvalid = mu >= a.n ? 0 : (a.n - mu >= 4u ? 4 : (int)(a.n - mu));
    const uint64_t tbase = (uint64_t)tile * kTileCoords;
    const uint32_t loff = lane * 4u;
    const uint64_t block_floats = (uint64_t)a.cap_lines * kLineFloats;     // one block's part of a ring slot

    // ---- where the tile's lines sit in the two slots (scalar loads, on their way while the subsets are hashed)
    uint32_t word_s = 0, base_s = 0, word_r = 0, base_r = 0;
    if (a.sum_lines) { word_s = lines_sum << 24; base_s = first_sum; }
    else if (a.do_send) { word_s = uniform_load(a.send_meta, tile); base_s = uniform_load(a.send_sb_base, tile / kTilesPerSuperblock); }
    if (a.do_recv && !TAU0) { word_r = uniform_load(a.recv_meta, tile); base_r = uniform_load(a.recv_sb_base, tile / kTilesPerSuperblock); }

    // ---- the subsets: bit j of a lane's mask = coordinate 4 group + j is received / sent now
    uint32_t mask_recv = 0, mask_send = 0;
    SubsetKey key = a.key;
    if (a.do_recv && !TAU0) {
        key.step_lo = a.step_lo[0]; key.step_hi = a.step_hi[0];
        mask_recv = member_mask(key, group, nvalid);
    }
    if (a.do_send) {
        key.step_lo = a.step_lo[1]; key.step_hi = a.step_hi[1];
        mask_send = member_mask(key, group, nvalid);
    }
    if (a.do_next && b0 == 0u) {                                           // how many lines the tile sends next step
        key.step_lo = a.step_lo[2]; key.step_hi = a.step_hi[2];
        uint32_t count;
        (void)wave_prefix_mask4(member_mask(key, group, nvalid), count);
        if (lane == 0) a.next_lines[tile] = (uint8_t)((count * RB + kLineFloats - 1u) / kLineFloats);
    }

    // a tile whose lines would pass the slot capacity is left out, at send and at receive alike
    const uint32_t first_s = base_s + (word_s & 0xFFFFFFu), first_r = base_r + (word_r & 0xFFFFFFu);
    uint32_t lines_s = word_s >> 24, lines_r = word_r >> 24;
    if ((uint64_t)first_s + lines_s > a.cap_lines) { lines_s = 0; mask_send = 0u; }
    if ((uint64_t)first_r + lines_r > a.cap_lines) { lines_r = 0; mask_recv = 0u; }
    if (TAU0) mask_recv = mask_send;                                       // what is sent now is received now

    uint32_t count_send, count_recv;
    const uint32_t rank_send = wave_prefix_mask4(mask_send, count_send);
    const uint32_t rank_recv = TAU0 ? rank_send : wave_prefix_mask4(mask_recv, count_recv);
    if (TAU0) count_recv = count_send;
    const uint64_t any_recv = __ballot(mask_recv != 0u);
    const bool half_recv = ((any_recv >> (lane & ~3u)) & 0xFull) != 0ull;     // my 64 bytes of a per-replica array receive
    const bool need_w = mask_send != 0u || half_recv;
    const double inv_replicas = a.inv_replicas;

    F4 w[RB], dv[RB];
    // the weights (and, per-replica layout, the EMA entries) of block b's replicas; an absent replica counts as zeros
    auto load_block = [&](const uint32_t b, const bool with_w, const bool with_d) {
#pragma unroll
        for (int k = 0; k < RB; ++k) {
            const uint32_t i = b * RB + k;
            if (with_w) {
#pragma unroll
                for (int j = 0; j < 4; ++j) w[k].v[j] = 0.f;
                if (i < R && need_w) w[k] = load_f32x4(weights_of<TABLE>(a, i) + tbase, loff, nvalid);
            }
            if (with_d) {
#pragma unroll
                for (int j = 0; j < 4; ++j) dv[k].v[j] = 0.f;
                if (!DIL && a.ema && i < R && half_recv) dv[k] = load_f32x4(a.d[i] + tbase, loff, nvalid);
            }
        }
    };
    // only half lines that received are rewritten
    auto store_block = [&](const uint32_t b) {
        if (!half_recv) return;
#pragma unroll
        for (int k = 0; k < RB; ++k) {
            const uint32_t i = b * RB + k;
            if (i >= R) continue;
            store_f32x4(weights_of<TABLE>(a, i) + tbase, loff, nvalid, w[k]);
            if (!DIL && a.ema) store_f32x4(a.d[i] + tbase, loff, nvalid, dv[k]);
        }
    };

    if constexpr (!TAU0) {
        constexpr uint32_t kStaged = kStageFloats / RB;                    // received coordinates whose values are staged
        constexpr bool kItems = kAverageItems<RB, STAGED>;
        extern __shared__ __attribute__((aligned(16))) float lds[];
        float *const ring_lds = lds + wave * (average_wave_bytes<DIL, RB>(a.nblocks) / sizeof(float));
        float *const x_lds = ring_lds + a.nblocks * kStageFloats;          // [RB][kStaged] weights of the received coordinates
        float *const d_lds = x_lds + kStageFloats;                         // their EMA entries: interleaved [kStaged][RB], else [RB][kStaged]
        uint8_t *const list = reinterpret_cast<uint8_t *>(d_lds + kStageFloats);
        // the rank in this turn of the lane's coordinates that are in `mask`, one after the other; `rank`: of the first
        auto each = [&](const uint32_t mask, const uint32_t rank, auto use) {
            uint32_t c = rank;                                             // (wraps below the turn's first: not this turn's)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if ((mask >> j) & 1u) {
                    if (c < kStaged) use(j, c);
                    ++c;
                }
        };
        // requests what the received coordinates of rank c0 .. c0 + kStaged - 1 need
        auto stage = [&](const uint32_t c0) {
            const uint32_t at = c0 * RB + lane * 4u;                       // a lane takes 16 bytes
            if (at < lines_r * kLineFloats) {
                const float *src = a.ring_recv + (uint64_t)first_r * kLineFloats + at;
                for (uint32_t b = 0; b < a.nblocks; ++b) lds_dma_16(src + b * block_floats, ring_lds + b * kStageFloats);
            }
            if (kItems && DIL && a.ema) {
                each(mask_recv, rank_recv - c0, [&](int j, uint32_t c) { list[c] = (uint8_t)(loff + (uint32_t)j); });
                wave_lds_sync();
                const uint32_t rank = lane * 4u / RB;                      // all or half of a coordinate's entries
                if (c0 + rank < count_recv) lds_dma_16(a.d[b0] + (tbase + list[rank]) * RB + (lane * 4u) % RB, d_lds);
            }
        };
        if (STAGED && count_recv != 0u) stage(0u);
        load_block(b0, true, true);
        if (STAGED) {                                                      // (before the first store: the wait counts stores, too)
            lds_dma_wait();
            wave_lds_sync();
        }
        if constexpr (kItems) {
            // A coordinate's values change hands through LDS: the lane that holds its group puts them there, and lane l takes
            // item l, replicas 4 l mod RB .. + 3 of the coordinate of rank 4 l / RB: sixteen bytes of [coordinate][RB].
            const uint32_t ci = lane * 4u / RB, k0 = (lane * 4u) % RB;
            if (a.do_send) {
                for (uint32_t c0 = 0; c0 * RB < lines_s * kLineFloats; c0 += kStaged) {
                    each(mask_send, rank_send - c0, [&](int j, uint32_t c) {
#pragma unroll
                        for (int k = 0; k < RB; ++k) x_lds[k * kStaged + c] = w[k].v[j];
                    });
                    wave_lds_sync();
                    const uint32_t at = c0 * RB + lane * 4u;
                    v4f x = {0.f, 0.f, 0.f, 0.f};                          // the rest of the tile's last line is zero
                    if (c0 + ci < count_send) {
                        const float *p = x_lds + k0 * kStaged + ci;
                        x = v4f{p[0], p[kStaged], p[2 * kStaged], p[3 * kStaged]};
                    }
                    if (at < lines_s * kLineFloats)
                        *reinterpret_cast<v4f *>(a.ring_send + b0 * block_floats + (uint64_t)first_s * kLineFloats + at) = x;
                    wave_lds_sync();
                }
            }
            for (uint32_t c0 = 0; c0 < count_recv; c0 += kStaged) {        // nearly always one turn
                if (c0 != 0u) {
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup"); // what the last turn read from LDS has been read
                    stage(c0);
                    lds_dma_wait();
                }
                each(mask_recv, rank_recv - c0, [&](int j, uint32_t c) {
#pragma unroll
                    for (int k = 0; k < RB; ++k) {
                        x_lds[k * kStaged + c] = w[k].v[j];
                        if (!DIL) d_lds[k * kStaged + c] = dv[k].v[j];
                    }
                });
                wave_lds_sync();
                if (c0 + ci < count_recv && c0 + ci < lines_r * kPerLine) {        // (the rank is below that by construction of the table)
                    double sum = 0.;
                    for (uint32_t b = 0; b < a.nblocks; ++b) {
                        float x[RB];
                        load_block_values<RB>(ring_lds + b * kStageFloats + ci * RB, x);
                        if (a.msg_dtype != 0u) {
#pragma unroll
                            for (int k = 0; k < RB; ++k) x[k] = quantize_message(x[k], a.msg_dtype);
                        }
                        const uint32_t nrep = R - b * RB;                  // replicas present in this block (>= RB: all)
#pragma unroll
                        for (int k = 0; k < RB; ++k)
                            if ((uint32_t)k < nrep) sum += (double)x[k];
                    }
                    const float abar = (float)(sum * inv_replicas);
                    float *const xp = x_lds + k0 * kStaged + ci, *const dp = DIL ? d_lds + lane * 4u : d_lds + k0 * kStaged + ci;
                    constexpr uint32_t ds = DIL ? 1u : kStaged;
                    if (a.ema) {
                        const v4f own = *reinterpret_cast<const v4f *>(ring_lds + b0 * kStageFloats + lane * 4u);     // my own staleness term takes the exact value
                        v4f d_new;
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            d_new[q] = (float)fma(a.coef_d, (double)dp[q * ds], a.coef_s * ((double)xp[q * kStaged] - (double)own[q]));
                            xp[q * kStaged] = (float)((double)abar + (double)d_new[q]);
                            if (!DIL) dp[q * ds] = d_new[q];
                        }
                        if (DIL) *reinterpret_cast<v4f *>(a.d[b0] + (tbase + list[ci]) * RB + k0) = d_new;
                    } else {
#pragma unroll
                        for (int q = 0; q < 4; ++q) xp[q * kStaged] = abar;
                    }
                }
                wave_lds_sync();
                each(mask_recv, rank_recv - c0, [&](int j, uint32_t c) {
#pragma unroll
                    for (int k = 0; k < RB; ++k) {
                        w[k].v[j] = x_lds[k * kStaged + c];
                        if (!DIL) dv[k].v[j] = d_lds[k * kStaged + c];
                    }
                });
            }
        } else {
            if (a.do_send && lines_s != 0u)
                average_send_block<RB>(a.ring_send + b0 * block_floats + (uint64_t)first_s * kLineFloats, w, mask_send, rank_send,
                                       count_send, lines_s * kPerLine, lane);
            // ---- receive: old average of what every replica sent (+ EMA of staleness)
            // the received coordinates of rank c0 .. c0 + most - 1; values(b, c, x): what block b's replicas sent for rank c0 + c
            auto receive = [&](const uint32_t c0, const uint32_t most, auto values) {
                uint32_t c = rank_recv - c0;                                   // (wraps below c0: not this turn's)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (!((mask_recv >> j) & 1u)) continue;
                    if (c < most && c0 + c < lines_r * kPerLine) {             // (as at the send)
                        double sum = 0.;
                        float own[RB];
                        for (uint32_t b = 0; b < a.nblocks; ++b) {
                            float x[RB];
                            values(b, c, x);
                            const uint32_t nrep = R - b * RB;                  // replicas present in this block (>= RB: all)
#pragma unroll
                            for (int k = 0; k < RB; ++k) {
                                if (b == b0) own[k] = x[k];                    // my own staleness term takes the exact value
                                const float q = a.msg_dtype != 0u ? quantize_message(x[k], a.msg_dtype) : x[k];
                                if ((uint32_t)k < nrep) sum += (double)q;
                            }
                        }
                        float *const dp = DIL ? a.d[b0] + (tbase + loff + (uint32_t)j) * RB : nullptr;
                        average_receive<DIL, RB, DIL && !STAGED>(a, j, (float)(sum * inv_replicas), own, dp, w, dv);
                    }
                    ++c;
                }
            };
            if constexpr (!STAGED) {
                receive(0u, kTileCoords, [&](const uint32_t b, const uint32_t c, float (&x)[RB]) {
                    load_block_values<RB>(a.ring_recv + (uint64_t)first_r * kLineFloats + b * block_floats + (uint64_t)c * RB, x);
                });
            } else {
                for (uint32_t c0 = 0; c0 < count_recv; c0 += kStaged) {        // nearly always one turn
                    if (c0 != 0u) {
                        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup"); // what the last turn read from LDS has been read
                        stage(c0);
                        lds_dma_wait();
                        wave_lds_sync();
                    }
                    receive(c0, kStaged, [&](const uint32_t b, const uint32_t c, float (&x)[RB]) {
                        load_block_values<RB>(ring_lds + b * kStageFloats + c * RB, x);
                    });
                }
            }
        }
        store_block(b0);
    } else {
        // ---- first walk: every block sends, and the sums over all replicas (in replica order) build up
        double sum[4] = {0., 0., 0., 0.};
        for (uint32_t b = 0; b < a.nblocks; ++b) {
            load_block(b, true, false);
            if (lines_s != 0u)
                average_send_block<RB>(a.ring_send + b * block_floats + (uint64_t)first_s * kLineFloats, w, mask_send, rank_send,
                                       count_send, lines_s * kPerLine, lane);
            const uint32_t nrep = R - b * RB;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (!((mask_recv >> j) & 1u)) continue;
#pragma unroll
                for (int k = 0; k < RB; ++k) {
                    const float q = a.msg_dtype != 0u ? quantize_message(w[k].v[j], a.msg_dtype) : w[k].v[j];
                    if ((uint32_t)k < nrep) sum[j] += (double)q;
                }
            }
        }
        // ---- second walk: the update of every block (one block: its weights are still in registers)
        if (count_recv != 0u) {
            for (uint32_t b = 0; b < a.nblocks; ++b) {
                if (a.nblocks > 1u) load_block(b, true, false);
                load_block(b, false, true);
                uint32_t c = rank_recv;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (((mask_recv >> j) & 1u) && c < lines_s * kPerLine) {
                        float own[RB];
#pragma unroll
                        for (int k = 0; k < RB; ++k) own[k] = w[k].v[j];   // no delay: what was sent is this very value
                        float *const dp = DIL ? a.d[b] + (tbase + loff + (uint32_t)j) * RB : nullptr;
                        average_receive<DIL, RB, false>(a, j, (float)(sum[j] * inv_replicas), own, dp, w, dv);
                        ++c;
                    }
                }
                store_block(b);
            }
        }
    }
}

// =============================================================================================
// Stateless look-ahead: out = w + gamma (w - w_prev)
// =============================================================================================
template <bool OUT_BF16>
__global__ void __launch_bounds__(256)
k_lookahead(void *__restrict__ out, const float *__restrict__ w, const float *__restrict__ w_prev,
            uint64_t n, double gamma)
{
    const uint64_t ngroups = (n + 3u) / 4u;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t group = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; group < ngroups; group += stride) {
        const uint64_t mu = group * 4u;
        const int nvalid = n - mu >= 4u ? 4 : (int)(n - mu);
        const F4 a = load_f32x4(w, mu, nvalid), b = load_f32x4(w_prev, mu, nvalid);
        double f[4];                                   // product and sum rounded separately in fp64, then one rounding
#pragma unroll
        for (int j = 0; j < 4; ++j) f[j] = __dadd_rn((double)a.v[j], __dmul_rn(gamma, (double)a.v[j] - (double)b.v[j]));
        if (OUT_BF16) {
            store_bf16x4_from_f64(static_cast<uint16_t *>(out), mu, nvalid, f);
        } else {
            F4 o;
#pragma unroll
            for (int j = 0; j < 4; ++j) o.v[j] = (float)f[j];
            store_f32x4(static_cast<float *>(out), mu, nvalid, o);
        }
    }
}

// =============================================================================================
// Diagnostics: consensus error and variance of the EMA estimates over the replicas
// =============================================================================================
struct DiagArgs {
    const float *w[kMaxReplicas];
    const float *d[kMaxReplicas];      // d_stride == 1: one array per replica; else one per block of d_stride replicas,
                                       // [coordinate][d_stride] (padded to whole tiles); all NULL when there is no correction vector
    uint64_t n;
    uint32_t replicas;
    uint32_t d_stride;                 // 1 (one array per replica) or the replicas per block (interleaved)
};

// Squared distance of the replicas' values x[0 .. R) of one coordinate from their mean, in fp64: the sum over
// the coordinates and the largest one.
struct Spread {
    double sum = 0., max = 0.;
    __device__ __forceinline__ void add(double e) { sum += e; max = e > max ? e : max; }
};

// One array per replica.  A thread takes groups of 4 coordinates and holds a group's values of all
// replicas in registers (RMAX >= replicas of them).  A wave's U groups of 64 follow each other in
// memory, and all their loads are requested before the first is used (few replicas: U > 1, so that as many
// bytes are in flight as with many).  WHOLE: a wave whose coordinates all exist loads without a lane's branch
// between the loads.  That takes 148 registers instead of 117 (RMAX = 16), 254 instead of 216 (32), so it serves grids
// that leave the chip idle (the host's rule), where what a call costs is one wave's chain of loads.
template <int RMAX, int U, bool WHOLE>
__device__ __forceinline__ void diag_flat(const float *const *arrays, uint32_t R, uint64_t n, Spread &out)
{
    const uint64_t ngroups = (n + 3u) / 4u;
    const double inv_r = 1.0 / (double)R;
    for (uint64_t g0 = ((uint64_t)blockIdx.x * 256u + (threadIdx.x & 192u)) * U + (threadIdx.x & 63u); g0 < ngroups;
         g0 += (uint64_t)gridDim.x * (256u * U)) {
        F4 x[U][RMAX];
        if (WHOLE && __ballot((g0 + 64u * (U - 1) + 1u) * 4u > n) == 0ull) {
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int i = 0; i < RMAX; ++i)
                    if ((uint32_t)i < R) x[u][i] = load_f32x4(arrays[i], (g0 + 64u * u) * 4u, 4);
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint64_t mu = (g0 + 64u * u) * 4u;
                const int nvalid = mu >= n ? 0 : n - mu >= 4u ? 4 : (int)(n - mu);
#pragma unroll
                for (int i = 0; i < RMAX; ++i)
                    if ((uint32_t)i < R) x[u][i] = load_f32x4(arrays[i], mu, nvalid);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint64_t mu = (g0 + 64u * u) * 4u;
            const int nvalid = mu >= n ? 0 : n - mu >= 4u ? 4 : (int)(n - mu);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (j >= nvalid) continue;
                double mean = 0., e = 0.;
#pragma unroll
                for (int i = 0; i < RMAX; ++i) if ((uint32_t)i < R) mean += (double)x[u][i].v[j];
                mean *= inv_r;
#pragma unroll
                for (int i = 0; i < RMAX; ++i) if ((uint32_t)i < R) { const double y = (double)x[u][i].v[j] - mean; e += y * y; }
                out.add(e);
            }
        }
    }
}

// One array [coordinate][RB] per block of RB replicas (NB blocks at most).  A thread takes 16-byte chunks, so
// that a wave reads whole lines with every load: a chunk is four replicas of a coordinate (RB = 8: the
// lane beside it has the other four) or (RB = 2) two coordinates.  A thread that took whole coordinates would
// read every line eight times over, 16 bytes of each at a time.  A wave's U runs of 64 chunks follow
// each other in memory.
// Measured (8 x 31.5M, weights and interleaved EMA vectors, whole call): 338 us = 6.0 TB/s, 570 us with a thread
// per four coordinates, 369 us with a wave's runs a grid apart.
template <int RB, int NB, int U>
__device__ __forceinline__ void diag_interleaved(const float *const *arrays, uint32_t R, uint64_t n, Spread &out)
{
    const uint64_t nchunks = (n * RB + 3u) / 4u;
    const double inv_r = 1.0 / (double)R;
    for (uint64_t g0 = ((uint64_t)blockIdx.x * 256u + (threadIdx.x & 192u)) * U + (threadIdx.x & 63u); g0 < nchunks; g0 += (uint64_t)gridDim.x * (256u * U)) {
        v4f x[U][NB];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const uint64_t g = g0 + 64u * u;
                x[u][b] = v4f{0.f, 0.f, 0.f, 0.f};
                if (g < nchunks && (uint32_t)(b * RB) < R) x[u][b] = __builtin_nontemporal_load(reinterpret_cast<const v4f *>(arrays[b]) + g);
            }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint64_t g = g0 + 64u * u;
            if (g >= nchunks) continue;                        // (RB = 8: the same for both lanes of a coordinate)
            if constexpr (RB == 2) {                           // chunk = coordinates 2 g, 2 g + 1
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    if (2u * g + c >= n) continue;
                    const double p = (double)x[u][0][2 * c], q = R > 1u ? (double)x[u][0][2 * c + 1] : 0.;
                    const double mean = (p + q) * inv_r, a = p - mean, b = R > 1u ? q - mean : 0.;
                    out.add(a * a + b * b);
                }
            } else {
                const uint32_t first = RB == 8 ? 4u * (threadIdx.x & 1u) : 0u;        // replica of the chunk's first value
                double mean = 0., e = 0.;
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (b * RB + first + j < R) mean += (double)x[u][b][j];
                if (RB == 8) mean += __shfl_xor(mean, 1);
                mean *= inv_r;
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (b * RB + first + j < R) { const double y = (double)x[u][b][j] - mean; e += y * y; }
                if (RB == 8) e += __shfl_xor(e, 1);
                if (RB == 4 || (threadIdx.x & 1u) == 0u) out.add(e);
            }
        }
    }
}

// grid = (blocks, 2): row 0 the weights, row 1 the EMA vectors (1 row without them); partial[row][block] = (sum, largest).
// A fixed grid and a fixed order make the result reproducible.
template <int RMAX, bool WHOLE>
__global__ void __launch_bounds__(256)
k_diag_partial(const DiagArgs a, double *__restrict__ partial)
{
    __shared__ double red[2][256];
    Spread s;
    const uint32_t R = a.replicas;
    constexpr int NB = RMAX >= 8 ? RMAX / 8 : 1, U = RMAX == 2 ? 4 : RMAX == 4 ? 2 : 1;
    if (blockIdx.y == 0u) diag_flat<RMAX, U, WHOLE>(a.w, R, a.n, s);
    else if (a.d_stride == 1u) diag_flat<RMAX, U, WHOLE>(a.d, R, a.n, s);
    else if constexpr (RMAX == 2) diag_interleaved<2, 1, 4>(a.d, R, a.n, s);
    else if constexpr (RMAX == 4) diag_interleaved<4, 1, 4>(a.d, R, a.n, s);
    else diag_interleaved<8, NB, NB == 1 ? 4 : NB == 2 ? 2 : 1>(a.d, R, a.n, s);
    red[0][threadIdx.x] = s.sum; red[1][threadIdx.x] = s.max;
    __syncthreads();
    for (uint32_t off = 128; off > 0; off >>= 1) {
        if (threadIdx.x < off) {
            red[0][threadIdx.x] += red[0][threadIdx.x + off];
            const double o = red[1][threadIdx.x + off];
            if (o > red[1][threadIdx.x]) red[1][threadIdx.x] = o;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        double *p = partial + 2u * (blockIdx.y * gridDim.x + blockIdx.x);
        p[0] = red[0][0]; p[1] = red[1][0];
    }
}

// T threads: 256 where there are no more partials (0.4 us less of a 7 us call), else 1024
template <int T>
__global__ void __launch_bounds__(T)
k_diag_final(const double *__restrict__ partial, uint32_t nblocks, uint32_t rows, uint32_t replicas, uint64_t n, double *__restrict__ out3)
{
    __shared__ double red[3][T];
    double cons = 0., var_sum = 0., var_max = 0.;
    for (uint32_t b = threadIdx.x; b < nblocks; b += T) {
        cons += partial[2u * b];
        if (rows == 2u) {
            var_sum += partial[2u * (nblocks + b)];
            const double o = partial[2u * (nblocks + b) + 1u];
            var_max = o > var_max ? o : var_max;
        }
    }
    red[0][threadIdx.x] = cons; red[1][threadIdx.x] = var_sum; red[2][threadIdx.x] = var_max;
    __syncthreads();
    for (uint32_t off = T / 2; off > 0; off >>= 1) {
        if (threadIdx.x < off) {
            red[0][threadIdx.x] += red[0][threadIdx.x + off];
            red[1][threadIdx.x] += red[1][threadIdx.x + off];
            const double o = red[2][threadIdx.x + off];
            if (o > red[2][threadIdx.x]) red[2][threadIdx.x] = o;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double inv_r = 1.0 / (double)replicas;
        out3[0] = red[0][0]; out3[1] = red[1][0] * inv_r / (double)n; out3[2] = red[2][0] * inv_r;
    }
}

// =============================================================================================
// Squared gradient norms (the stage's share of each replica's global norm, for clipping)
// =============================================================================================
struct NormArgs {
    const void *g[kMaxReplicas];
    uint64_t n;
    uint32_t replicas;
    uint32_t is_bf16;
};

// grid = (blocks, replicas); block (b, i) sums the squares of groups b, b + blocks, ... of replica i
__global__ void __launch_bounds__(256)
k_sqnorm_partial(const NormArgs a, double *__restrict__ partial)
{
    __shared__ double red[256];
    const uint32_t i = blockIdx.y;
    const uint64_t ngroups = (a.n + 3u) / 4u;
    const uint64_t stride = (uint64_t)gridDim.x * 256u;
    double acc = 0.;
    for (uint64_t group = (uint64_t)blockIdx.x * 256u + threadIdx.x; group < ngroups; group += stride) {
        const uint64_t mu = group * 4u;
        const int nvalid = a.n - mu >= 4u ? 4 : (int)(a.n - mu);
        const F4 g = a.is_bf16 ? load_bf16x4(static_cast<const uint16_t *>(a.g[i]), mu, nvalid)
                               : load_f32x4(static_cast<const float *>(a.g[i]), mu, nvalid);
#pragma unroll
        for (int j = 0; j < 4; ++j) acc += (double)g.v[j] * (double)g.v[j];     // tail entries are 0
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (uint32_t off = 128; off > 0; off >>= 1) {
        if (threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[(uint64_t)i * gridDim.x + blockIdx.x] = red[0];
}

// one block per replica: fixed-order sum of its partials
__global__ void __launch_bounds__(256)
k_sqnorm_final(const double *__restrict__ partial, uint32_t nblocks, double *__restrict__ out)
{
    __shared__ double red[256];
    double acc = 0.;
    for (uint32_t b = threadIdx.x; b < nblocks; b += 256u) acc += partial[(uint64_t)blockIdx.x * nblocks + b];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (uint32_t off = 128; off > 0; off >>= 1) {
        if (threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[blockIdx.x] = red[0];
}

}  // namespace am
