// Arguments, chunk order, clearing and shared-tile flush of the tile gridders
// (k_grid.hip: FP64, k_tile32.hip: FP32 on the matrix cores).
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

// Flush of a tile that several chunks share: rows of 64 values in LDS, added to
// the grid by one wavefront each.  Device-wide atomics leave the L2 as one
// request per 64 bytes and instruction (the L2s of the XCDs are not coherent):
// through LDS a row goes out in one instruction, four full requests in FP32 and
// eight in FP64, where lanes adding their own cells made twice as many
// half-empty ones (FP32 A+W chunk 14.2 -> 11.6 ms).  The PSF adds half of each
// row and half of its conjugate mirror image, whose cells run backwards
// (W-projection PSF 298 -> 202 us in FP32, 507 -> 346 in FP64); row and column 0
// have no image on the grid.
template <typename T, bool PSF>
struct TileFlush {
    T *own, *img;                 // this lane's value of the first row, and its image's
    int64_t row, pol;             // values per row and per pol
    int img_at, y, ny;
    bool in, img_in;

    // grid: pol 0 of the plane; (x0, y0): first cell of the first row
    __device__ __forceinline__ TileFlush(T *grid, int x0, int y0, int nx, int ny_, int64_t pols) {
        const int lane = threadIdx.x & 63, c = kTile - 1 - (lane >> 1);   // the image's cell
        y = y0;
        ny = ny_;
        row = 2 * (int64_t)nx;
        pol = 2 * pols;
        own = grid + y0 * row + 2 * x0 + lane;
        in = x0 + (lane >> 1) < nx;
        if (PSF) {
            img = grid + (ny - y0) * row + 2 * (nx - x0 - c) + (lane & 1);
            img_at = 2 * c + (lane & 1);
            img_in = x0 + c > 0 && x0 + c < nx;
        }
    }

    // values: row dy of pol p
    __device__ __forceinline__ void add(const T *values, int dy, int p) const {
        const int lane = threadIdx.x & 63;
        const T v = values[lane];
        if (v != (T)0 && in && y + dy < ny)
            atomicAdd(own + (dy * row + p * pol), PSF ? (T)0.5 * v : v);
        if (PSF) {
            const T u = values[img_at];
            if (u != (T)0 && img_in && y + dy > 0 && y + dy < ny)
                atomicAdd(img + (p * pol - dy * row), lane & 1 ? -(T)0.5 * u : (T)0.5 * u);
        }
    }
};

hipError_t launch_grid_tile32(const TileArgs &ta, int64_t n_blocks, int precision, int npol,
                              bool po, bool psf, bool det, hipStream_t s);

}  // namespace lr
