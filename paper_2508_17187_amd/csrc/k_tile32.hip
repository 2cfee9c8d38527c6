// Tile gridder of the FP32 forms, on the matrix cores.
//
// A wavefront owns a band of 8 rows of a 32 x 32 tile; in step s (0 .. 3) lane
// l stands for the cell of column l % 32 and row 2 s + l / 32.  Adding a group
// to 64 cells is an outer product, (2 npol components of its sum) x (64 kernel
// values), which is what v_mfma_f32_4x4x1_16b_f32 computes for sixteen blocks
// of four cells: A, the four components of one group, is broadcast from block
// j of a register that holds four groups (cbsz = 4, abid = j), B holds every
// lane's own kernel value and D the lane's own four accumulators.  A complex
// tap is two such products per four components, Re C (Re A, Im A) and
// Im C (-Im A, Re A), each a fused multiply-add of FP32 (bit for bit what
// fmaf gives).  The group's sums then need no broadcast instructions, and a
// conjugated or scaled kernel costs nothing (signs and 2^-e are in A).
//
// What bounds it: the kernel values past the L2.  A chunk of the A+W image
// reads 55 GB of them and flushes 9 GB per launch, at 5.7 of the 6.8 TB/s that
// reads beyond the L2 reach here.  Before (vector FMAs, exec-masked loads, one
// batch in flight, flushes of half-empty requests): 16.0 ms per A+W chunk of
// 12.6 M visibilities, now 10.9 ms; W-projection gridding call 174 -> 140 us.
// Variants: two columns per lane and 16-byte loads (11.6 ms: the edges' masks
// cost more than the loads save), vector FMAs on them (11.6 ms).
//
// Matrix instructions ignore the lane mask, so a lane outside the footprint
// must hold 0: the kernel values are buffer loads whose bounds are the group's
// own S x S sub-kernel, and a lane outside its columns asks past the end
// (reading nothing, returning 0; rows outside fall off either end by
// themselves).  Infinities and NaN would spread through those zeros (0 x inf),
// so groups whose sums or pointing phasors are not finite are added tap by tap
// afterwards.
//
// The loads of the next kBatch groups are in flight while a batch is added; with
// a pointing phasor they are not: the phasor of every tap bounds it then, and
// the registers of a second batch cost the fourth wavefront per SIMD (150
// registers against 104; A+W grid call of 53.9 M visibilities with pointing
// offsets 1160 against 1043 us, of 0.45 M on 1024^2 70 against 69 us).
#include "k_tile.h"

namespace lr {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kBatch = 4;            // groups per batch
constexpr uint32_t kOutside = 0x80000000u;   // a byte offset beyond every sub-kernel

// One (tile, group) pair of a chunk, staged in LDS.
//   x, y   low word of the sub-kernel's address; high 16 bits, half-width << 16,
//          form << 25, not-finite << 28, used << 29
//   z, w   tile origin minus footprint origin, (column, row)
__device__ __forceinline__ int item_h(uint32_t y) { return (int)((y >> 16) & 0x1FF); }
__device__ __forceinline__ int item_form(uint32_t y) { return (int)((y >> 25) & 7); }
constexpr uint32_t kNotFinite = 1u << 28, kUsed = 1u << 29;

// Raw kernel values of one step in flight.
template <int ST, bool RE>
struct TapRaw {
    static constexpr int E = CFRaw<ST>::bytes;
    typedef typename std::conditional<E == 8 && !RE, u32x2, uint32_t>::type R;
    __device__ static R load(__amdgpu_buffer_rsrc_t r, uint32_t off) {
        if constexpr (E == 8 && !RE) return __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
        else return __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
    }
    // unscaled (the plane's 2^-e is in the staged sums)
    __device__ static cpx<float> value(R v) {
        if constexpr (E == 8 && RE) return {__uint_as_float(v), 0.f};
        else if constexpr (E == 8) return {__uint_as_float(v.x), __uint_as_float(v.y)};
        else return CFRaw<ST>::decode(v, 1.0f);
    }
};

template <int ST, int NPOL, bool PO, bool PSF, bool RE, bool DET>
__global__ __launch_bounds__(256, 4) void k_grid_tile32(TileArgs a) {
    constexpr int E = CFRaw<ST>::bytes;
    constexpr int NH = NPOL == 4 ? 2 : 1;             // registers of four components
    constexpr int NA = 4 * NH;                        // components per item, padded to 4
    constexpr int MAXI = kChunkMax;
    typedef TapRaw<ST, RE> Tap;
    typedef typename Tap::R Raw;
    __shared__ u32x4 items[MAXI + 1];                 // the last one is empty
    __shared__ float avs[(MAXI + 1) * NA];
    __shared__ uint16_t lists[4][MAXI + 2 * kBatch];
    __shared__ GroupMeta gms[PO ? MAXI : 1];
    __shared__ cpx<float> rows[4][64];                // two rows of a band, one pol
    const int c0 = (int)blockIdx.x < a.n_chunks ? chunk_of(a, (int)blockIdx.x) : (int)blockIdx.x;
    if (!PSF && c0 >= a.n_chunks) {      // GRID_SET: tiles without pairs
        const int tile = c0 - a.n_chunks;
        if (a.tile_state[tile] == 0)
            clear_tile<float, NPOL>(tile, a.ntx, a.nty, a.nx, a.ny, a.pol_stride,
                                    (cpx<float> *)a.grid);
        return;
    }
    const int32_t key = a.chunk_tile[c0];
    // DET (deterministic order): the workgroup of a tile's first chunk takes
    // all of the tile's chunks in order and owns the tile; the others exit
    if (DET && c0 > 0 && a.chunk_tile[c0 - 1] == key) return;
    const bool excl = !PSF && (DET || a.chunk_excl[c0]);
    const int tx = key % a.ntx;
    const int rest = key / a.ntx;
    const int ty = rest % a.nty;
    const int P = rest / a.nty;
    const int lane = threadIdx.x & 63, wv = uni(threadIdx.x >> 6);
    const int lx = lane & 31, ly = lane >> 5;          // column; row of a step
    const int band = 8 * wv;                           // first row of the wavefront's band
    f32x4 acc[4][NH];
    for (int s = 0; s < 4; ++s)
        for (int q = 0; q < NH; ++q) acc[s][q] = f32x4{0.f, 0.f, 0.f, 0.f};
    const cpx<float> *Av = (const cpx<float> *)a.A;
    if (threadIdx.x == 0) items[MAXI] = u32x4{0u, 0u, 0u, 0u};
    if (threadIdx.x < NA) avs[MAXI * NA + threadIdx.x] = 0.f;
    for (int c = c0;;) {
        const int32_t s0 = a.chunk_start[c];
        const int n = a.chunk_start[c + 1] - s0;
        for (int t = threadIdx.x; t < n; t += blockDim.x) {
            const int32_t g = a.tp_group[s0 + t];
            const GroupMeta gm = a.groups[g];
            const float sc = E == 4 ? a.cf.scale[(int64_t)gm.fg * a.cf.n_w + gm.k] : 1.0f;
            cpx<float> v[NPOL];
            if (a.mix == 0) {
                for (int p = 0; p < NPOL; ++p) v[p] = Av[(int64_t)g * NPOL + p];
            } else {
                // a Mueller pass: slot p takes the sum of the correlations q
                // whose element M[q][p] is the pass's kind
                cpx<float> in[NPOL];
                for (int q = 0; q < NPOL; ++q) in[q] = Av[(int64_t)g * NPOL + q];
                for (int p = 0; p < NPOL; ++p) {
                    v[p] = {0.f, 0.f};
                    for (int q = 0; q < NPOL; ++q)
                        if ((a.mix >> (q * NPOL + p)) & 1u) {
                            v[p].x += in[q].x;
                            v[p].y += in[q].y;
                        }
                    if (negated(a.cf, gm.form)) v[p] = {-v[p].x, -v[p].y};
                }
            }
            // slopes small enough that the phase overflows nowhere in the tile
            // (|t O - o| < 2^15), and a loss factor that is a number
            bool finite = !PO || (fabs(gm.bu) + fabs(gm.bv) < 1e300 && isfinite(gm.f));
            for (int p = 0; p < NPOL; ++p) {
                v[p].x *= sc;
                v[p].y *= sc;
                finite = finite && isfinite(v[p].x) && isfinite(v[p].y);
                avs[t * NA + 2 * p] = v[p].x;
                avs[t * NA + 2 * p + 1] = v[p].y;
            }
            for (int p = 2 * NPOL; p < NA; ++p) avs[t * NA + p] = 0.f;
            const uint64_t at = (uint64_t)((const char *)a.cf.table + gm.cf_off * E);
            items[t] = u32x4{(uint32_t)at,
                             (uint32_t)(at >> 32) | (uint32_t)gm.h << 16 |
                                 (uint32_t)gm.form << 25 | (finite ? 0u : kNotFinite) | kUsed,
                             (uint32_t)(tx * kTile - gm.pu + gm.h),
                             (uint32_t)(ty * kTile - gm.pv + gm.h)};
            if (PO) gms[t] = gm;
        }
        __syncthreads();
        // the items whose footprints meet this wavefront's band, in order
        uint16_t *list = lists[wv];
        int hits = 0;
        bool odd = false;              // this lane saw one that is not finite
        for (int w = 0; w < n; w += 64) {
            const int i = w + lane;
            bool hit = false;
            if (i < n) {
                const u32x4 it = items[i];
                const int S = 2 * item_h(it.y) + 1, r = (int)it.w + band;
                hit = r < S && r + 8 > 0;
                if (hit && (it.y & kNotFinite)) {
                    odd = true;
                    hit = false;
                }
            }
            const uint64_t m = __ballot(hit);
            if (hit) list[hits + __popcll(m & ((1ull << lane) - 1))] = (uint16_t)i;
            hits += __popcll(m);
        }
        if (lane < 2 * kBatch) list[hits + lane] = MAXI;       // empty items
        __builtin_amdgcn_wave_barrier();

        // a batch in flight: its four groups' components and, per group, the
        // kernel values of the four steps
        struct Batch {
            float re[NH], im[NH];        // A of Re C and of Im C: lane 4 b + i holds
                                         // component i of group b % kBatch
            Raw cv[kBatch][4];
            int dx[PO ? kBatch : 1], r[PO ? kBatch : 1];
        };
        auto load = [&](int k, Batch &b) {
            const int ia = list[k + ((lane >> 2) & (kBatch - 1))], ip = list[k + (lane & (kBatch - 1))];
            const u32x4 it = items[ip];
            const uint32_t ya = items[ia].y;
            const int i = lane & 3;
            for (int q = 0; q < NH; ++q) {
                b.re[q] = avs[ia * NA + 4 * q + i];
                if (!RE) {
                    // (-Im A, Re A), times -1 for a conjugated kernel (a
                    // pointing phasor needs the conjugate before it)
                    const float v = avs[ia * NA + 4 * q + (i ^ 1)];
                    const bool neg = ((i & 1) == 0) != (!PO && (item_form(ya) & kConj) != 0);
                    b.im[q] = neg ? -v : v;
                }
            }
            for (int j = 0; j < kBatch; ++j) {
                const uint32_t lo = __builtin_amdgcn_readlane(it.x, j);
                const uint32_t hi = __builtin_amdgcn_readlane(it.y, j);
                const int bx = (int)__builtin_amdgcn_readlane(it.z, j);
                const int by = (int)__builtin_amdgcn_readlane(it.w, j);
                const int S = 2 * item_h(hi) + 1, form = item_form(hi);
                // an unused slot has no bytes
                const int bytes = hi & kUsed ? S * S * E : 0;
                __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                    (void *)(((uint64_t)(hi & 0xFFFF) << 32) | lo), 0, bytes, 0x00020000);
                const int su = form & kFlipU ? -E : E, sv = form & kFlipV ? -S * E : S * E;
                const int k0 = (form & kFlipU ? (S - 1) * E : 0) +
                               (form & kFlipV ? (S - 1) * S * E : 0);
                const int dx = bx + lx, r = by + band + ly;
                int off = __mul24(r, sv) + (__mul24(dx, su) + k0);
                if ((unsigned)dx >= (unsigned)S) off = (int)kOutside;
                for (int s = 0; s < 4; ++s) {
                    b.cv[j][s] = Tap::load(rs, (uint32_t)off);
                    off += 2 * sv;
                }
                if (PO) {
                    b.dx[j] = dx;
                    b.r[j] = r;
                }
            }
        };
        auto add = [&](int k, const Batch &b) {
            auto one = [&](auto jc) {
                constexpr int j = decltype(jc)::value;
                cpx<float> cv[4];
                for (int s = 0; s < 4; ++s) cv[s] = Tap::value(b.cv[j][s]);
                if constexpr (PO) {
                    const int i = uni(list[k + j]);
                    if (i != MAXI) {
                        const uint32_t y = items[i].y;
                        const int h = item_h(y);
                        for (int s = 0; s < 4; ++s) {
                            if (item_form(y) & kConj) cv[s].y = -cv[s].y;
                            cv[s] = cmul(cv[s], phasor<float>(gms[i], b.dx[j] - h,
                                                              b.r[j] + 2 * s - h, a.cf.O));
                        }
                    }
                }
                for (int s = 0; s < 4; ++s)
                    for (int q = 0; q < NH; ++q)
                        acc[s][q] = __builtin_amdgcn_mfma_f32_4x4x1f32(b.re[q], cv[s].x, acc[s][q],
                                                                       4, j, 0);
                if (!RE)
                    for (int s = 0; s < 4; ++s)
                        for (int q = 0; q < NH; ++q)
                            acc[s][q] = __builtin_amdgcn_mfma_f32_4x4x1f32(b.im[q], cv[s].y,
                                                                           acc[s][q], 4, j, 0);
            };
            one(std::integral_constant<int, 0>{});
            one(std::integral_constant<int, 1>{});
            one(std::integral_constant<int, 2>{});
            one(std::integral_constant<int, 3>{});
        };
        static_assert(kBatch == 4, "a batch is unrolled by hand");
        if constexpr (PO) {
            for (int k = 0; k < hits; k += kBatch) {
                Batch b0;
                load(k, b0);
                add(k, b0);
            }
        } else if (hits > 0) {
            Batch b0, b1;
            load(0, b0);
            for (int k = 0;;) {
                load(k + kBatch, b1);
                __builtin_amdgcn_sched_barrier(0);
                add(k, b0);
                k += kBatch;
                if (k >= hits) break;
                load(k + kBatch, b0);
                __builtin_amdgcn_sched_barrier(0);
                add(k, b1);
                k += kBatch;
                if (k >= hits) break;
            }
        }
        if (__builtin_expect(__any(odd), 0)) {
            // tap by tap, only the cells of the footprints
            for (int i = 0; i < n; ++i) {
                const u32x4 it = items[i];
                if (!(it.y & kNotFinite)) continue;
                const int S = 2 * item_h(it.y) + 1, h = item_h(it.y), form = item_form(it.y);
                const char *sub = (const char *)(((uint64_t)(it.y & 0xFFFF) << 32) | it.x);
                const int dx = (int)it.z + lx;
                for (int s = 0; s < 4; ++s) {
                    const int r = (int)it.w + band + 2 * s + ly;
                    if ((unsigned)dx >= (unsigned)S || (unsigned)r >= (unsigned)S) continue;
                    const int e = (form & kFlipV ? S - 1 - r : r) * S + (form & kFlipU ? S - 1 - dx : dx);
                    cpx<float> cv = CFElem<ST>::load(sub, e, 1.0f);
                    if (form & kConj) cv.y = -cv.y;
                    if constexpr (PO) cv = cmul(cv, phasor<float>(gms[i], dx - h, r - h, a.cf.O));
                    for (int p = 0; p < NPOL; ++p) {
                        const cpx<float> av = {avs[i * NA + 2 * p], avs[i * NA + 2 * p + 1]};
                        f32x4 &t = acc[s][p / 2];
                        cpx<float> v = {t[2 * (p & 1)], t[2 * (p & 1) + 1]};
                        if (RE) {
                            v.x = fmaf(cv.x, av.x, v.x);
                            v.y = fmaf(cv.x, av.y, v.y);
                        } else {
                            cmac(v, cv, av);
                        }
                        t[2 * (p & 1)] = v.x;
                        t[2 * (p & 1) + 1] = v.y;
                    }
                }
            }
        }
        if (!DET || ++c >= a.n_chunks || a.chunk_tile[c] != key) break;
        __syncthreads();      // every wavefront is done with this chunk's items
    }
    float *grid = (float *)a.grid;
    const bool set = excl && a.set;
    if (!excl) {
        const TileFlush<float, PSF> flush(grid + 2 * ((int64_t)P * NPOL * a.pol_stride), tx * kTile,
                                          ty * kTile + band, a.nx, a.ny, a.pol_stride);
        for (int s = 0; s < 4; ++s)
            for (int p = 0; p < NPOL; ++p) {
                rows[wv][lane] = {acc[s][p / 2][2 * (p & 1)], acc[s][p / 2][2 * (p & 1) + 1]};
                __builtin_amdgcn_wave_barrier();
                for (int r = 0; r < 2; ++r) flush.add((const float *)rows[wv] + 64 * r, 2 * s + r, p);
                __builtin_amdgcn_wave_barrier();
            }
        return;
    }
    const int x = tx * kTile + lx;
    for (int s = 0; s < 4; ++s) {
        const int y = ty * kTile + band + 2 * s + ly;
        if (x >= a.nx || y >= a.ny) continue;
        if (!set) {
            // cells that received nothing are left alone (adding an exact
            // zero would not change them)
            bool any = false;
            for (int p = 0; p < 2 * NPOL; ++p) any |= acc[s][p / 4][p & 3] != 0.f;
            if (!any) continue;
        }
        for (int p = 0; p < NPOL; ++p) {
            const float vx = acc[s][p / 2][2 * (p & 1)], vy = acc[s][p / 2][2 * (p & 1) + 1];
            const int64_t base = ((int64_t)P * NPOL + p) * a.pol_stride;
            float *q = grid + 2 * (base + (int64_t)y * a.nx + x);
            if (set) {
                q[0] = vx;
                q[1] = vy;
            } else {
                q[0] += vx;
                q[1] += vy;
            }
        }
    }
}

template <int ST, int NPOL>
static hipError_t tile32_t(const TileArgs &ta, int64_t n_blocks, bool po, bool psf, bool det,
                           hipStream_t s) {
    dim3 grd((unsigned)n_blocks), blk(256);
    // the point-spread function's mirror image is always flushed with
    // atomics: it has no deterministic form
    if (po) {
        if (psf) hipLaunchKernelGGL((k_grid_tile32<ST, NPOL, true, true, false, false>), grd, blk, 0, s, ta);
        else if (det) hipLaunchKernelGGL((k_grid_tile32<ST, NPOL, true, false, false, true>), grd, blk, 0, s, ta);
        else hipLaunchKernelGGL((k_grid_tile32<ST, NPOL, true, false, false, false>), grd, blk, 0, s, ta);
    } else if (ta.cf.real) {
        if (psf) hipLaunchKernelGGL((k_grid_tile32<ST, NPOL, false, true, true, false>), grd, blk, 0, s, ta);
        else if (det) hipLaunchKernelGGL((k_grid_tile32<ST, NPOL, false, false, true, true>), grd, blk, 0, s, ta);
        else hipLaunchKernelGGL((k_grid_tile32<ST, NPOL, false, false, true, false>), grd, blk, 0, s, ta);
    } else {
        if (psf) hipLaunchKernelGGL((k_grid_tile32<ST, NPOL, false, true, false, false>), grd, blk, 0, s, ta);
        else if (det) hipLaunchKernelGGL((k_grid_tile32<ST, NPOL, false, false, false, true>), grd, blk, 0, s, ta);
        else hipLaunchKernelGGL((k_grid_tile32<ST, NPOL, false, false, false, false>), grd, blk, 0, s, ta);
    }
    return hipGetLastError();
}

template <int ST>
static hipError_t tile32_np(const TileArgs &ta, int64_t n_blocks, int npol, bool po, bool psf,
                            bool det, hipStream_t s) {
    switch (npol) {
        case 1: return tile32_t<ST, 1>(ta, n_blocks, po, psf, det, s);
        case 2: return tile32_t<ST, 2>(ta, n_blocks, po, psf, det, s);
        default: return tile32_t<ST, 4>(ta, n_blocks, po, psf, det, s);
    }
}

hipError_t launch_grid_tile32(const TileArgs &ta, int64_t n_blocks, int precision, int npol,
                              bool po, bool psf, bool det, hipStream_t s) {
    switch (precision) {
        case LR_F32: return tile32_np<LR_F32>(ta, n_blocks, npol, po, psf, det, s);
        case LR_F32_CF16: return tile32_np<LR_F32_CF16>(ta, n_blocks, npol, po, psf, det, s);
        default: return tile32_np<LR_F32_CFBF16>(ta, n_blocks, npol, po, psf, det, s);
    }
}

}  // namespace lr
