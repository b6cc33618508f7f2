// Which rows of a tensor the workgroups of a launch take: index arithmetic without anything of the GPU's, so that it can be checked
// on the CPU at sizes that no test runs (tests/test_work_index.py).
#pragma once

#include <cstdint>

namespace fftconv {

// Rows of a launch of the column kernels (long_fft.hip): row i, i < 65536, is row first + i of the tensor, or, counted in pairs of batch
// rows of H < 2^31 - 65536 channels, channel j % H of batch row 2 (j / H), j = first + i (its partner lies H rows further, if the tensor has so many).
// A row may be a single sample, so that a tensor holds more than 2^32 of them; the division, in every thread, is of 32 bits all the
// same (64 bits cost 2 % of a pass): the host takes the pairs before the launch's first channel out.
struct LongRows {
    int64_t base, rows;                        // row 0 of the launch; rows of the tensor
    uint32_t channel, H;                       // channel of row 0; H = 0: not in pairs
    __host__ __device__ int64_t at(uint32_t i) const { return base + i + (H ? (int64_t)((channel + i) / H) * H : 0); }
    __host__ __device__ bool partner(uint32_t i) const { return at(i) + H < rows; }
};
inline LongRows long_rows(int64_t first) { return LongRows{first, INT64_MAX, 0, 0}; }
inline LongRows long_row_pairs(int64_t first, int64_t H, int64_t rows)
{
    return LongRows{first / H * H + first, rows, (uint32_t)(first % H), (uint32_t)H};
}

// Work items of the streamed-table kernel (fused3_big.hip), pairs of batch rows of a channel: a workgroup takes every step-th of up to
// 2^31 - 9 of them, counted in 32 bits, so that the last one plus a step may lie beyond; batch rows are counted in 32 bits as well, up to the
// number of a pair's second one.
inline bool big_items_fit(int64_t B, int64_t H) { return B < INT32_MAX && H * ((B + 1) / 2) < ((int64_t)1 << 31) - 8; }
// Workgroups, and the dies (8, or 1: all items in turn) they are dealt to, for H channels of `pairs` items on a chip that holds `resident` of them at
// once.  A die's channels one after another, unless that takes more steps of a workgroup than all items in turn on as many workgroups
// as there can be (not only on a multiple of 8 of them: 37 items are one step of 37, but two of 32).
struct BigSplit { int grid, nx; };
inline BigSplit big_split(int64_t H, int64_t pairs, int64_t resident)
{
    const int64_t items = H * pairs, most = items < resident ? items : resident, steps = (items + most - 1) / most;
    const int64_t each = most / 8;                                  // workgroups of a die
    if (each > 0 && ((H + 7) / 8 * pairs + each - 1) / each <= steps) return BigSplit{(int)(8 * each), 8};
    return BigSplit{(int)most, 1};
}
__host__ __device__ inline bool big_item_follows(int v, int step, int items) { return v < items - step; }

}  // namespace fftconv
