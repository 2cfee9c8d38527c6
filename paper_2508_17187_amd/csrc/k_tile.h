// Arguments and helpers the tile gridders share (k_grid.hip: FP64,
// k_tile32.hip: FP32 on the matrix cores).
#pragma once

#include "k_common.h"

namespace lr {

struct TileArgs {
    const GroupMeta *groups;
    const int32_t *tp_group, *chunk_start, *chunk_tile, *chunk_excl, *chunk_order, *tile_state;
    const void *A;
    void *grid;
    CFView cf;
    int32_t nx, ny, ntx, nty;
    int64_t pol_stride;   // nx * ny
    int32_t n_chunks;
    int32_t set;          // GRID_SET: exclusive chunks overwrite their whole tile
    int32_t run;          // chunks in a row per XCD (0: dealt one by one)
    uint32_t mix;         // Mueller pass: bit q * NPOL + p adds pol q's sum into slot p (0: none)
};

// The chunk of workgroup b < n_chunks.  Workgroups are dealt to the eight XCDs
// one by one; with chunks in plane order each XCD takes runs of kChunkRun
// consecutive chunks, which read the same kernel plane through one L2 (A+W
// chunk 10.92 -> 10.58 ms).  Chunks in order of their work are dealt one by
// one: runs would unbalance them (W-projection 138 -> 143 us).
constexpr int kChunkRun = 32;
__device__ __forceinline__ int chunk_of(const TileArgs &a, int b) {
    if (a.run > 0 && b < a.n_chunks / (8 * a.run) * (8 * a.run))
        b = ((b >> 3) / a.run * 8 + (b & 7)) * a.run + (b >> 3) % a.run;
    return a.chunk_order ? a.chunk_order[b] : b;
}

// Thread t of a 256-thread workgroup clears column t % 32 of tile `tile`.
template <typename T, int NPOL>
__device__ __forceinline__ void clear_tile(int tile, int32_t ntx, int32_t nty, int32_t nx,
                                           int32_t ny, int64_t pol_stride, cpx<T> *grid) {
    const int tx = tile % ntx;
    const int rest = tile / ntx;
    const int ty = rest % nty;
    const int P = rest / nty;
    const int x = tx * kTile + (threadIdx.x & 31);
    if (x >= nx) return;
    for (int r = threadIdx.x >> 5; r < kTile; r += blockDim.x >> 5) {
        const int y = ty * kTile + r;
        if (y >= ny) break;
        for (int p = 0; p < NPOL; ++p)
            grid[((int64_t)P * NPOL + p) * pol_stride + (int64_t)y * nx + x] = {(T)0, (T)0};
    }
}

hipError_t launch_grid_tile32(const TileArgs &ta, int64_t n_blocks, int precision, int npol,
                              bool po, bool psf, bool det, hipStream_t s);

}  // namespace lr
