// The index list's kernels with launch parameters that no entry point of the library uses: a patience the caller
// names (0: every workgroup counts what is before it itself), any number of strips a wave, either way of writing.  Built beside the
// library, loaded by tests/test_gpu_subset_list.py.
#include "../paper_2601_22442_amd/csrc/am_kernels.h"

extern "C" {

const char *tk_source_hash(void) { return AM_SOURCE_HASH; }

// part_count: one word per part of 4 strips waves; count: one word.  Returns the HIP error, or -1 for a shape the kernels do not take.
int tk_subset_list(uint64_t n, uint64_t seed, uint64_t step, uint64_t threshold, uint32_t strips, int rows, uint32_t patience,
                   uint32_t *part_count, uint32_t words, uint64_t *out, uint64_t capacity, uint64_t *count, void *stream)
{
    const uint64_t nstrips = (n + am::kStripCoords - 1) / am::kStripCoords;
    if (n == 0 || nstrips > (1u << 21) || strips == 0 || strips > 32u) return -1;
    const uint32_t parts = (uint32_t)((nstrips + 4u * strips - 1u) / (4u * strips));
    if (parts > words) return -1;
    const am::SubsetKey key = {(uint32_t)seed, (uint32_t)(seed >> 32), (uint32_t)step, (uint32_t)(step >> 32), threshold, am::kDrawCoordinate, 1u};
    hipStream_t s = static_cast<hipStream_t>(stream);
    am::k_list_clear<<<(parts + 255u) / 256u, 256, 0, s>>>(part_count, parts);
    const auto kernel = rows ? am::k_subset_list<true> : am::k_subset_list<false>;
    kernel<<<parts, 256, strips * 256u * sizeof(uint32_t), s>>>(key, n, (uint32_t)nstrips, strips, patience, part_count, out, capacity, count);
    return (int)hipGetLastError();
}

}  // extern "C"
