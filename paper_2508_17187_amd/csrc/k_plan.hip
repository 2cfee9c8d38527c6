// Binning of (row, channel) pairs (the PreSolvePrep re-ordering): index map,
// 64-bit sort keys, radix sort, grouping of identical samples and the
// decomposition of the gridder's work into wavefront tasks.
#include <string.h>

#include <cstddef>
#include <cstring>

#include <rocprim/rocprim.hpp>

#include "lr_internal.h"
#include "lr_launch.h"

namespace lr {

// ---------------------------------------------------------------------------
// Small host arrays reach the device through kernel arguments, so no host
// buffer has to outlive an asynchronous copy.
struct ChanUpload {
    ChanConst c[kMaxChanPerUpload];
    int32_t n, base;
};

__global__ void k_upload_chan(ChanUpload up, ChanConst *dst) {
    int i = threadIdx.x;
    if (i < up.n) dst[up.base + i] = up.c[i];
}

struct WordUpload {
    uint32_t w[512];
    int32_t n, base;
};

__global__ void k_upload_words(WordUpload up, uint32_t *dst) {
    for (int i = threadIdx.x; i < up.n; i += blockDim.x) dst[up.base + i] = up.w[i];
}

hipError_t upload_chan(const std::vector<ChanConst> &cc, ChanConst *d, hipStream_t s) {
    for (size_t b = 0; b < cc.size(); b += kMaxChanPerUpload) {
        ChanUpload up;
        up.n = (int32_t)std::min<size_t>(kMaxChanPerUpload, cc.size() - b);
        up.base = (int32_t)b;
        for (int i = 0; i < up.n; ++i) up.c[i] = cc[b + i];
        hipLaunchKernelGGL(k_upload_chan, dim3(1), dim3(64), 0, s, up, d);
    }
    return hipGetLastError();
}

hipError_t upload_words(const void *src, size_t bytes, void *d, hipStream_t s) {
    const uint32_t *w = (const uint32_t *)src;
    size_t n = bytes / 4;
    for (size_t b = 0; b < n; b += 512) {
        WordUpload up;
        up.n = (int32_t)std::min<size_t>(512, n - b);
        up.base = (int32_t)b;
        for (int i = 0; i < up.n; ++i) up.w[i] = w[b + i];
        hipLaunchKernelGGL(k_upload_words, dim3(1), dim3(256), 0, s, up, (uint32_t *)d);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// The channel constants travel by value, `up.n` channels from `up.base`.
__global__ void k_debug_map(int64_t nrow, int32_t nchan, const double *uvw, ChanUpload up,
                            MapGeom g, int32_t *out) {
    int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= nrow * up.n) return;
    int64_t r = j / up.n;
    int32_t cl = (int32_t)(j - r * up.n);
    int32_t c = up.base + cl;
    int64_t i = r * nchan + c;
    ChanConst ch = up.c[cl];
    Map m = map_sample(uvw[3 * r], uvw[3 * r + 1], uvw[3 * r + 2], ch, g);
    int32_t *o = out + 8 * i;
    o[0] = m.pu; o[1] = m.pv; o[2] = m.ou; o[3] = m.ov;
    o[4] = m.k; o[5] = m.conj; o[6] = m.keep; o[7] = ch.fg;
}

hipError_t launch_debug_map(int64_t nrow, int32_t nchan, const double *uvw,
                            const std::vector<ChanConst> &cc, const MapGeom &g, int32_t *out,
                            hipStream_t s) {
    for (int32_t b = 0; b < nchan; b += kMaxChanPerUpload) {
        ChanUpload up;
        up.n = std::min<int32_t>(kMaxChanPerUpload, nchan - b);
        up.base = b;
        for (int i = 0; i < up.n; ++i) up.c[i] = cc[b + i];
        int64_t n = nrow * up.n;
        if (n == 0) continue;
        hipLaunchKernelGGL(k_debug_map, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                           nrow, nchan, uvw, up, g, out);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Sort keys.  Fields from most to least significant: plane, A-term group,
// w-plane, block of pixels (v, u), conj, p_v, p_u in the block, [baseline,
// channel when a pointing phasor is applied], o_v, o_u.  Keys of dropped or
// skipped pairs are all ones, which no kept pair's 63 bits reach.
constexpr uint64_t kDropKey = ~0ull;

__device__ __forceinline__ void put(unsigned __int128 &key, uint32_t v, int bits) {
    if (bits) key = (key << bits) | (unsigned __int128)v;
}

__global__ __launch_bounds__(256) void k_plan_keys(uint32_t n_pairs, uint32_t nchan,
                                                   const double *uvw, const ChanConst *cc,
                                                   MapGeom g, KeyLayout kl, const int32_t *ant1,
                                                   const int32_t *ant2, int32_t nant,
                                                   uint64_t *keys, int32_t *vals) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_pairs) return;
    const uint32_t r = i / nchan, c = i - r * nchan;
    const ChanConst ch = cc[c];
    uint64_t key = kDropKey;
    int32_t val = (int32_t)i;
    if (ch.plane < 0) {
        val |= (1 << 30);
    } else {
        const double *q = uvw + 3 * (int64_t)r;
        Map m = map_sample(q[0], q[1], q[2], ch, g);
        if (m.keep) {
            unsigned __int128 k128 = 0;
            put(k128, (uint32_t)ch.plane, kl.b_plane);
            put(k128, (uint32_t)ch.fg, kl.b_fg);
            put(k128, (uint32_t)m.k, kl.b_k);
            const uint32_t low = (1u << kl.b_blk) - 1;
            put(k128, (uint32_t)m.pv >> kl.b_blk, kl.b_pv - kl.b_blk);
            put(k128, (uint32_t)m.pu >> kl.b_blk, kl.b_pu - kl.b_blk);
            put(k128, (uint32_t)m.conj, kl.b_conj);
            put(k128, (uint32_t)m.pv & low, kl.b_blk);
            put(k128, (uint32_t)m.pu & low, kl.b_blk);
            if (kl.b_bl) put(k128, (uint32_t)(ant1[r] * nant + ant2[r]), kl.b_bl);
            if (kl.b_ch) put(k128, c, kl.b_ch);
            put(k128, (uint32_t)(m.ov + (g.O >> 1)), kl.b_o);
            put(k128, (uint32_t)(m.ou + (g.O >> 1)), kl.b_o);
            key = (uint64_t)(k128 >> kl.shift);
        }
    }
    keys[i] = key;
    vals[i] = val;
}

// Tiles [tx0, tx1] x [ty0, ty1] a footprint overlaps.
__device__ __forceinline__ void tile_span(int pu, int pv, int h, int &tx0, int &tx1, int &ty0,
                                          int &ty1) {
    tx0 = (pu - h) / kTile;
    tx1 = (pu + h) / kTile;
    ty0 = (pv - h) / kTile;
    ty1 = (pv + h) / kTile;
}

// What sorted pair i adds to the running totals: a group in the low word
// and the tiles of its footprint in the high word when the pair begins a
// group (its key differs from the one before it, or every pair is a group
// of its own), else nothing.  The pixel and the w-plane come from the key
// itself (the fields the shift may drop lie below them), so one scan over
// the sorted keys numbers the groups and places their tile pairs.
struct GroupHead {
    const uint64_t *keys;
    const int32_t *h;
    KeyLayout kl;
    int32_t merged;
    __device__ uint64_t operator()(uint32_t i) const {
        const uint64_t key = keys[i];
        if (key == kDropKey || (merged && i > 0 && keys[i - 1] == key)) return 0;
        uint64_t f = key >> (2 * kl.b_o + kl.b_ch + kl.b_bl - kl.shift);
        auto field = [&](int bits) {
            const int v = (int)(f & ((1ull << bits) - 1));
            f >>= bits;
            return v;
        };
        int pu = field(kl.b_blk), pv = field(kl.b_blk);
        f >>= kl.b_conj;
        pu |= field(kl.b_pu - kl.b_blk) << kl.b_blk;
        pv |= field(kl.b_pv - kl.b_blk) << kl.b_blk;
        const int k = field(kl.b_k);
        int tx0, tx1, ty0, ty1;
        tile_span(pu, pv, h[k], tx0, tx1, ty0, ty1);
        return 1ull | ((uint64_t)((tx1 - tx0 + 1) * (ty1 - ty0 + 1)) << 32);
    }
};

__device__ __forceinline__ double airy_power(double x) {
    if (x == 0.0) return 1.0;
    double b = 2.0 * j1(x) / x;
    return b * b;
}

// Sums of a workgroup's threads added to out[0] and out[1], one request per
// workgroup (two lanes of one instruction; requests to one word go one after
// another).
__device__ __forceinline__ void block_add2(unsigned long long u, unsigned long long v,
                                           unsigned long long *out) {
    __shared__ unsigned long long part[4][2];
    for (int off = 32; off > 0; off >>= 1) {
        u += __shfl_xor(u, off);
        v += __shfl_xor(v, off);
    }
    if ((threadIdx.x & 63) == 0) {
        part[threadIdx.x >> 6][0] = u;
        part[threadIdx.x >> 6][1] = v;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        const int i = threadIdx.x;
        const unsigned long long s = part[0][i] + part[1][i] + part[2][i] + part[3][i];
        if (s) atomicAdd(out + i, s);
    }
}

// Groups from the scan over the sorted pairs: the group of every pair, the
// record of each group (written by its first pair) and its (tile, group)
// pairs; the counts.  A bounded number of workgroups walks the pairs, so
// that the totals cost a bounded number of atomic requests.
constexpr int kMetaBlocks = 2048;

__global__ __launch_bounds__(256) void k_group_meta(
    const uint64_t *keys, const uint64_t *scan, const int32_t *vals, uint32_t n_pairs,
    uint32_t nchan, const double *uvw, const ChanConst *cc, MapGeom g, CFView cf,
    const int32_t *ant1, const int32_t *ant2, const double *ant_dlm, double du_dl, double dv_dm,
    int32_t ntx, int32_t nty, int32_t *gidx, int32_t *group_start, GroupMeta *groups,
    int64_t *geo, uint32_t *tile_keys, int32_t *tile_vals, PlanCounts *pc) {
    unsigned long long taps = 0, tiles = 0;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n_pairs;
         i += gridDim.x * blockDim.x) {
        if (keys[i] == kDropKey) continue;
        const uint64_t now = scan[i], before = i > 0 ? scan[i - 1] : 0;
        const int32_t gi = (int32_t)(uint32_t)now - 1;
        gidx[i] = gi;
        if (i + 1 == n_pairs || keys[i + 1] == kDropKey) {      // the last kept pair
            group_start[gi + 1] = (int32_t)(i + 1);
            pc->n_kept = (int32_t)(i + 1);
            pc->n_groups = gi + 1;
        }
        if ((uint32_t)now == (uint32_t)before) continue;
        group_start[gi] = (int32_t)i;
        const uint32_t pair = (uint32_t)vals[i] & ~(1u << 30);
        const uint32_t r = pair / nchan, c = pair - r * nchan;
        const ChanConst ch = cc[c];
        const double *q = uvw + 3 * (int64_t)r;
        Map m = map_sample(q[0], q[1], q[2], ch, g);
        GroupMeta gm;
        const int32_t h = g.h[m.k];
        const int64_t S = 2 * h + 1;
        const int64_t no = g.O + 1;
        gm.cf_off = cf.plane_off[(int64_t)ch.fg * g.n_w + m.k] +
                    ((int64_t)((g.O >> 1) - abs(m.ov)) * no + ((g.O >> 1) - abs(m.ou))) * S * S;
        gm.cell = ((int64_t)ch.plane * g.npol) * (int64_t)g.ny * g.nx + (int64_t)m.pv * g.nx + m.pu;
        gm.pu = m.pu;
        gm.pv = m.pv;
        gm.k = m.k;
        gm.form = (m.conj ? kConj : 0) | (m.ou > 0 ? kFlipU : 0) | (m.ov > 0 ? kFlipV : 0);
        gm.ou = m.ou;
        gm.ov = m.ov;
        gm.plane = ch.plane;
        gm.fg = ch.fg;
        gm.h = h;
        gm.sc = cf.scale[(int64_t)ch.fg * g.n_w + m.k];
        gm.f = 1.0;
        gm.bu = 0.0;
        gm.bv = 0.0;
        if (ant1) {
            int32_t a1 = ant1[r], a2 = ant2[r];
            double l1 = ant_dlm[2 * a1], m1 = ant_dlm[2 * a1 + 1];
            double l2 = ant_dlm[2 * a2], m2 = ant_dlm[2 * a2 + 1];
            double dl = 0.5 * (l1 + l2), dm = 0.5 * (m1 + m2);
            double ddl = l1 - l2, ddm = m1 - m2;
            double dist = sqrt(ddl * ddl + ddm * ddm);
            gm.f = airy_power(ch.fscale * 0.5 * dist);
            gm.bu = (du_dl * dl) / (double)g.O;
            gm.bv = (dv_dm * dm) / (double)g.O;
        }
        groups[gi] = gm;
        geo[gi] = (int64_t)(uint16_t)m.pu | ((int64_t)(uint16_t)m.pv << 16) |
                  ((int64_t)(uint16_t)(int16_t)m.ou << 32) |
                  ((int64_t)(uint16_t)(int16_t)m.ov << 48);
        taps += (unsigned long long)(S * S);
        // the group's (tile, group) pairs
        int tx0, tx1, ty0, ty1;
        tile_span(m.pu, m.pv, h, tx0, tx1, ty0, ty1);
        uint32_t o = (uint32_t)(before >> 32);
        for (int ty = ty0; ty <= ty1; ++ty)
            for (int tx = tx0; tx <= tx1; ++tx) {
                tile_keys[o] = (uint32_t)(((int64_t)ch.plane * nty + ty) * ntx + tx);
                tile_vals[o] = gi;
                ++o;
            }
        tiles += (unsigned long long)((tx1 - tx0 + 1) * (ty1 - ty0 + 1));
    }
    static_assert(offsetof(PlanCounts, n_tile_pairs) == 8, "taps and n_tile_pairs are added as one");
    block_add2(taps, tiles, &pc->taps);
}

// ---- tiles of the gridder ----------------------------------------------------
// The (tile, group) pairs sorted by tile are cut into chunks of at most
// `per` pairs, one workgroup each, and (separable tables) into the parts of
// the separable gridder.  Everything follows from each tile's number of
// pairs, so one scan over the tiles places them.
struct TileSums {
    uint32_t chunks;      // gridder chunks
    uint32_t shared;      // tiles with several chunks
    uint32_t used;        // tiles with pairs
};

struct TileSumsPlus {
    __host__ __device__ TileSums operator()(const TileSums &a, const TileSums &b) const {
        return TileSums{a.chunks + b.chunks, a.shared + b.shared, a.used + b.used};
    }
};

struct TileCounts {
    const int32_t *tile_tp;
    uint32_t per;
    __device__ TileSums operator()(uint32_t t) const {
        const uint32_t n = (uint32_t)(tile_tp[t + 1] - tile_tp[t]);
        const uint32_t c = (n + per - 1) / per;
        return TileSums{c, c > 1 ? 1u : 0u, c > 0 ? 1u : 0u};
    }
};

// Chunks, ownership and shared list of every tile, one wavefront per tile.
// A chunk that holds all of its tile's pairs owns the tile: it may update
// the grid with plain loads and stores instead of atomics.
__global__ __launch_bounds__(256) void k_tile_chunks(const int32_t *tile_tp, const TileSums *sums,
                                                     uint32_t n_tiles, uint32_t per,
                                                     int32_t *chunk_start, int32_t *chunk_tile,
                                                     int32_t *chunk_excl, int32_t *tile_state,
                                                     int32_t *shared, PlanCounts *pc) {
    const uint32_t t = (uint32_t)(((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6);
    const uint32_t lane = threadIdx.x & 63;
    if (t >= n_tiles) return;
    const TileSums end = sums[t], beg = t > 0 ? sums[t - 1] : TileSums{0, 0, 0};
    const uint32_t n = end.chunks - beg.chunks;
    const int32_t p0 = tile_tp[t];
    for (uint32_t c = lane; c < n; c += 64) {
        chunk_start[beg.chunks + c] = p0 + (int32_t)(c * per);
        chunk_tile[beg.chunks + c] = (int32_t)t;
        chunk_excl[beg.chunks + c] = n == 1 ? 1 : 0;
    }
    if (lane != 0) return;
    tile_state[t] = n == 0 ? 0 : n == 1 ? 1 : 2;
    if (n > 1) shared[beg.shared] = (int32_t)t;
    if (t + 1 == n_tiles) {
        chunk_start[end.chunks] = tile_tp[n_tiles];
        pc->n_chunks = (int32_t)end.chunks;
        pc->n_shared = (int32_t)end.shared;
    }
}

// Work estimate of each chunk (one wavefront per chunk): the footprint
// cells of its pairs inside the tile, subtracted from the most it can be,
// so that an ascending sort puts the largest first (in steps of 2 cells:
// two 8-bit digits); the chunk ids ride along.  Slots past the chunks sort
// last.
constexpr int kCostBits = 16;
static_assert(kChunkCells >> 1 < 1 << kCostBits, "chunk cost exceeds its sort digits");

__global__ __launch_bounds__(256) void k_chunk_cost(const int32_t *chunk_start,
                                                    const int32_t *chunk_tile,
                                                    const int32_t *tp_group,
                                                    const GroupMeta *groups, int32_t ntx,
                                                    int32_t nty, uint32_t slots,
                                                    const PlanCounts *pc, uint32_t *key,
                                                    int32_t *id) {
    const uint32_t c = (uint32_t)(((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6);
    const int lane = threadIdx.x & 63;
    if (c >= slots) return;
    uint32_t w = 0;
    if ((int32_t)c < pc->n_chunks) {
        const int32_t s0 = chunk_start[c], n = chunk_start[c + 1] - s0;
        const int tx = chunk_tile[c] % ntx, ty = (chunk_tile[c] / ntx) % nty;
        for (int i = lane; i < n; i += 64) {
            const GroupMeta &gm = groups[tp_group[s0 + i]];
            const int pu = gm.pu, pv = gm.pv, h = gm.h;
            const int cx = min(pu + h + 1, (tx + 1) * kTile) - max(pu - h, tx * kTile);
            const int cy = min(pv + h + 1, (ty + 1) * kTile) - max(pv - h, ty * kTile);
            w += (uint32_t)(max(cx, 0) * max(cy, 0));
        }
    }
    for (int off = 32; off > 0; off >>= 1) w += __shfl_xor(w, off);
    if (lane == 0) {
        key[c] = (uint32_t)(kChunkCells - (int)w) >> 1;
        id[c] = (int32_t)c;
    }
}

// Table plane of each chunk (that of its first pair; a tile's pairs follow
// the group order, whose keys put the frequency group and w-plane first, so
// a chunk rarely spans two planes); the chunk ids ride along.  Slots past
// the chunks get the last plane, behind its chunks (the sort is stable).
__global__ void k_chunk_plane(const int32_t *chunk_start, const int32_t *tp_group,
                              const GroupMeta *groups, int32_t n_w, uint32_t last, uint32_t slots,
                              const PlanCounts *pc, uint32_t *key, int32_t *id) {
    const uint32_t c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= slots) return;
    uint32_t k = last;
    if ((int32_t)c < pc->n_chunks) {
        const GroupMeta &g = groups[tp_group[chunk_start[c]]];
        k = (uint32_t)(g.fg * n_w + g.k);
    }
    key[c] = k;
    id[c] = (int32_t)c;
}

// Single-run groups: with a period L, a group whose pairs are p, p + L,
// p + 2 L, ... (one unbroken stretch of one track) is summed completely by
// the presum lane that walks that track, which may then store the sum
// without an atomic.  single[g] starts at 1 and is cleared by any gap.
__global__ void k_single_init(int32_t *single, int64_t n_groups, int32_t value) {
    int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g < n_groups) single[g] = value;
}

__global__ void k_single_gaps(const int32_t *order, const int32_t *gidx, int64_t n_kept,
                              int64_t period, int32_t *single) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < 1 || i >= n_kept || gidx[i] != gidx[i - 1]) return;
    if ((int64_t)order[i] - order[i - 1] != period) single[gidx[i]] = 0;
}

// One-member groups (bit 1 of single[g]; the presum stores their sums, which
// never need a cleared start) and the list of the other groups, which the
// presum may add to with atomics (any order).  A wavefront takes up to 1024
// groups, so that the list's end moves once per 1024 (the end is one word, and
// requests to it go one after another), and fewer when there are few.
constexpr int kKindRounds = 16;

__global__ __launch_bounds__(256) void k_group_kinds(const int32_t *group_start, int64_t n_groups,
                                                     int32_t rounds, int32_t *single,
                                                     int32_t *multi, PlanCounts *pc) {
    const int lane = threadIdx.x & 63;
    const int64_t g0 = (((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6) * (64 * rounds);
    uint64_t many[kKindRounds];
    int total = 0;
    for (int r = 0; r < kKindRounds; ++r) {
        many[r] = 0;
        if (r >= rounds) continue;
        const int64_t g = g0 + r * 64 + lane;
        const bool in = g < n_groups;
        const bool one = in && group_start[g + 1] - group_start[g] == 1;
        if (one) single[g] |= 2;
        many[r] = __ballot(in && !one);
        total += __popcll(many[r]);
    }
    if (total == 0) return;
    int at = 0;
    if (lane == 0) at = atomicAdd(&pc->n_multi, total);
    at = __shfl(at, 0);
    for (int r = 0; r < kKindRounds; ++r) {
        if ((many[r] >> lane) & 1)
            multi[at + __popcll(many[r] & ((1ull << lane) - 1))] = (int32_t)(g0 + r * 64 + lane);
        at += __popcll(many[r]);
    }
}

// First (tile, group) pair of every tile in the tile-sorted pair list
// (keys), by binary search; tile_tp[n_tiles] = n.
__global__ void k_tile_ranges(const uint32_t *keys, int64_t n, int64_t n_tiles,
                              int32_t *tile_tp) {
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t > n_tiles) return;
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        int64_t mid = (lo + hi) >> 1;
        if ((int64_t)keys[mid] < t) lo = mid + 1; else hi = mid;
    }
    tile_tp[t] = (int32_t)lo;
}

// Parts of the separable gridder: a tile's (tile, group) pairs in pieces of
// at most kSepPart, so that no workgroup is left with a tile many times
// heavier than the rest.  A wavefront takes its pairs one after another
// (about 60 ns each in FP64), so when the data fall on few tiles the longest
// part is the call: the compact 22,464-sample observation on 4 tiles of a
// 256^2 grid took 356 us whole and takes 29 us in parts of 64.  Fewer than
// `few` tiles with pairs are therefore cut so finely that there are about
// kSepFill parts.  The line lies at 1024 tiles for supports up to 7 (4 per
// CU; W-projection tracks on 1024^2, about 500 tiles: 414 -> 177 us; on
// 2048^2, above it, parts would cost more in atomic flushes than they
// balance, 108 -> 118 us) and lower by the number of taps a lane holds, since
// wider supports keep a SIMD busy with fewer wavefronts (support 15: 800 ->
// 585 us on 512^2, but 975 -> 1081 us on 1024^2).  The nearer to the line,
// the fuller the chip is without cuts and the more each cut costs (its tile
// is cleared first and flushed by atomics): a part is the share of one of
// kSepFill with few tiles in use and 1 + kSepEven shares at the line, so that
// only tiles well above the mean are cut there.  Calls with the shares as
// they are and with longer parts, 80,000 groups on 2048^2: about 900 tiles,
// kernel 56 -> 44 us (uncut 44); 100 tiles 111 -> 104 us; 10 tiles 96 -> 95 us
// (uncut 410); on 1024^2, 500 tiles 100 -> 92 us (uncut 261).
// Keys sort the tiles by pair count, most first
// (counts of 65535 and more alike: such tiles are cut into equal parts).
__global__ void k_sep_count(const int32_t *tile_tp, int64_t n_tiles, uint32_t *key,
                            int32_t *tile) {
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n_tiles) return;
    key[t] = 0xFFFFu - (uint32_t)min(tile_tp[t + 1] - tile_tp[t], 0xFFFF);
    tile[t] = (int32_t)t;
}

__global__ void k_sep_nparts(const int32_t *tile_tp, const int32_t *tile, const TileSums *sums,
                             int64_t n_tiles, int32_t few, int32_t *nparts) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_tiles) return;
    int32_t most = kSepPart;
    const int32_t used = (int32_t)sums[n_tiles - 1].used;
    if (used < few) {
        const int64_t per = (tile_tp[n_tiles] + kSepFill - 1) / kSepFill;
        most = (int32_t)max((int64_t)kSepPartMin,
                            min((int64_t)kSepPart, per + kSepEven * per * used / few));
    }
    const int32_t t = tile[i];
    const int32_t n = tile_tp[t + 1] - tile_tp[t];
    nparts[i] = (n + most - 1) / most;
}

__global__ void k_sep_fill(const int32_t *tile_tp, const int32_t *tile, const int32_t *nparts,
                           const int32_t *first, int64_t n_tiles, int4 *part, int32_t *shared,
                           PlanCounts *pc) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_tiles) return;
    const int32_t t = tile[i], np = nparts[i];
    if (i + 1 == n_tiles) pc->n_sep_parts = first[i] + np;
    if (np == 0) return;
    const int32_t b0 = tile_tp[t], b1 = tile_tp[t + 1];
    // equal pieces, the last one shorter by the remainder
    const int32_t len = (b1 - b0 + np - 1) / np;
    for (int q = 0; q < np; ++q)
        part[first[i] + q] = make_int4(t, b0 + q * len, min(b1, b0 + (q + 1) * len), np > 1);
    if (np > 1) shared[atomicAdd(&pc->n_sep_shared, 1)] = t;
}

// Group of every pair in natural (row, channel) order: >= 0 kept (bit
// kSingleRun set for a single-run group, kSingleton for a one-member
// group), -1 dropped, -2 skipped channel.
__global__ void k_pair_group(const int32_t *order, const int32_t *gidx, const int32_t *single,
                             int64_t n_kept, int64_t n_pairs, int32_t *pair_group) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_pairs) return;
    int32_t v = order[i];
    int32_t pair = v & ~(1 << 30);
    int32_t out = ((v >> 30) & 1) ? -2 : -1;
    if (i < n_kept) {
        const int32_t g = gidx[i];
        const int32_t k = single ? single[g] : 0;
        out = g | ((k & 1) ? kSingleRun : 0) | ((k & 2) ? kSingleton : 0);
    }
    pair_group[pair] = out;
}

// Row period: the smallest r for which rows i and i + r have nearly the same
// (u, v, w) for all of the first 64 rows (the next sample of the same
// baseline in time-major data).  Only the work order of the presum and
// expand kernels depends on it, never a result.
__global__ void k_row_period(const double *uvw, int64_t nrow, int32_t rmax, int32_t *best) {
    int32_t r = blockIdx.x * blockDim.x + threadIdx.x + 1;
    if (r > rmax) return;
    const int nchk = (int)(nrow - r < 64 ? nrow - r : 64);
    if (nchk < 4) return;
    // eight rows' loads in flight together: the true period's thread checks all
    // 64, and row by row that was 16 us of every plan
    for (int i0 = 0; i0 < nchk; i0 += 8) {
        bool same = true;
        for (int k = 0; k < 8; ++k) {
            const int64_t i = min(i0 + k, nchk - 1);
            const double a0 = uvw[3 * i], a1 = uvw[3 * i + 1], a2 = uvw[3 * i + 2];
            const double b0 = uvw[3 * (i + r)], b1 = uvw[3 * (i + r) + 1], b2 = uvw[3 * (i + r) + 2];
            const double d = fabs(a0 - b0) + fabs(a1 - b1) + fabs(a2 - b2);
            const double s = fabs(a0) + fabs(a1) + fabs(a2);
            same = same && d <= 1e-2 * s + 1e-3;
        }
        if (!same) return;
    }
    atomicMin(best, r);
}

// Start values of a build: counts, and (without pairs) the tile arrays.
__global__ void k_plan_init(PlanCounts *pc, int32_t *tile_state, int32_t *tile_tp,
                            int64_t n_tiles) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t == 0) {
        PlanCounts z = {};
        z.period = kNoPeriod;
        *pc = z;
    }
    if (t < n_tiles) tile_state[t] = 0;
    if (t <= n_tiles) tile_tp[t] = 0;
}

// ---------------------------------------------------------------------------
static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Radix sorts of the build.  Up to this many items the library's merge sort
// is used, beyond it the one-sweep radix sort, whose passes each cost several
// small launches.  Jobs without a plan, one-sweep from 2^15 / 2^17 / 2^18 items
// on: 5e4 pairs 396 / 315 / 323 us, 1e5 488 / 416 / 409 us, 2e5 604 / 610 / 564
// us; 1.3e6 pairs (4e5 tile pairs) 769 / 772 / 765 us, and more at the library's
// own 2^20 (twenty launches of merges).
constexpr unsigned kMergeSortMost = 1 << 18;
using SortConfig = rocprim::radix_sort_config<rocprim::default_config, rocprim::default_config,
                                              rocprim::default_config, kMergeSortMost>;

static rocprim::transform_iterator<rocprim::counting_iterator<uint32_t>, GroupHead, uint64_t>
group_heads(const GroupHead &f) {
    return rocprim::transform_iterator<rocprim::counting_iterator<uint32_t>, GroupHead, uint64_t>(
        rocprim::counting_iterator<uint32_t>(0), f);
}

static rocprim::transform_iterator<rocprim::counting_iterator<uint32_t>, TileCounts, TileSums>
tile_counts(const TileCounts &f) {
    return rocprim::transform_iterator<rocprim::counting_iterator<uint32_t>, TileCounts, TileSums>(
        rocprim::counting_iterator<uint32_t>(0), f);
}

static size_t sort_temp_bytes(int64_t n, int64_t n_tp, int64_t n_tiles) {
    size_t b[5] = {0, 0, 0, 0, 0};
    rocprim::radix_sort_pairs<SortConfig>((void *)nullptr, b[0], (uint64_t *)nullptr,
                                          (uint64_t *)nullptr, (int32_t *)nullptr,
                                          (int32_t *)nullptr, (size_t)n, 0, 64);
    rocprim::radix_sort_pairs<SortConfig>((void *)nullptr, b[1], (uint32_t *)nullptr,
                                          (uint32_t *)nullptr, (int32_t *)nullptr,
                                          (int32_t *)nullptr, (size_t)std::max(n_tp, n_tiles), 0,
                                          32);
    rocprim::inclusive_scan((void *)nullptr, b[2], group_heads(GroupHead{}), (uint64_t *)nullptr,
                            (size_t)n, rocprim::plus<uint64_t>());
    rocprim::inclusive_scan((void *)nullptr, b[3], tile_counts(TileCounts{}),
                            (TileSums *)nullptr, (size_t)n_tiles, TileSumsPlus());
    rocprim::exclusive_scan((void *)nullptr, b[4], (int32_t *)nullptr, (int32_t *)nullptr,
                            (int32_t)0, (size_t)n_tiles, rocprim::plus<int32_t>());
    // small sorts are not monotonic in scratch: the merge sort's most, too
    size_t small = 0;
    const size_t most = std::min<size_t>(kMergeSortMost, (size_t)std::max(n, n_tp));
    rocprim::radix_sort_pairs<SortConfig>((void *)nullptr, small, (uint64_t *)nullptr,
                                          (uint64_t *)nullptr, (int32_t *)nullptr,
                                          (int32_t *)nullptr, most, 0, 64);
    return std::max(small, *std::max_element(b, b + 5));
}

int64_t max_tiles_per_group(int32_t h_max) {
    int64_t span = (2 * (int64_t)h_max + kTile - 1) / kTile + 1;
    return span * span;
}

int64_t tile_count(int32_t nx, int32_t ny, int32_t nplane) {
    return (int64_t)nplane * ((nx + kTile - 1) / kTile) * ((ny + kTile - 1) / kTile);
}

PlanLayout plan_layout(int64_t n_pairs, int32_t nchan, int32_t h_max, int64_t n_tiles) {
    PlanLayout L;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off += align256(bytes); return o; };
    int64_t n = std::max<int64_t>(n_pairs, 1);
    int64_t ntp = n * max_tiles_per_group(h_max);
    L.chan = take(sizeof(ChanConst) * (nchan > 0 ? nchan : 1));
    L.order = take(sizeof(int32_t) * n);
    L.gidx = take(sizeof(int32_t) * n);
    L.pair_group = take(sizeof(int32_t) * n);
    L.group_start = take(sizeof(int32_t) * (n + 1));
    L.groups = take(sizeof(GroupMeta) * n);
    L.tp_group = take(sizeof(int32_t) * ntp);
    L.chunk_start = take(sizeof(int32_t) * (ntp + 1));
    L.chunk_tile = take(sizeof(int32_t) * ntp);
    L.chunk_excl = take(sizeof(int32_t) * ntp);
    L.chunk_order = take(sizeof(int32_t) * ntp);
    L.tile_state = take(sizeof(int32_t) * std::max<int64_t>(n_tiles, 1));
    L.shared_tiles = take(sizeof(int32_t) * std::max<int64_t>(n_tiles, 1));
    L.geo = take(sizeof(int64_t) * n);
    L.tile_tp = take(sizeof(int32_t) * (std::max<int64_t>(n_tiles, 1) + 1));
    L.multi = take(sizeof(int32_t) * n);
    const int64_t nt = std::max<int64_t>(n_tiles, 1);
    L.sep_part = take(sizeof(int4) * (nt + ntp / kSepPart + kSepFill + 1));
    L.sep_shared = take(sizeof(int32_t) * nt);
    L.persistent = off;
    // transient (the tile sort of the separable gridder's parts needs
    // n_tiles + 1 entries)
    const int64_t nx_ = std::max(std::max(n, ntp), nt + 1);
    L.keys_a = take(std::max(sizeof(uint64_t) * nx_, sizeof(TileSums) * nt));   // keys, then tile sums
    L.keys_b = take(sizeof(uint64_t) * nx_);
    L.vals_a = take(sizeof(int32_t) * nx_);
    L.flags = take(sizeof(int32_t) * nx_);
    L.scan = take(sizeof(int32_t) * nx_);
    L.counter = take(sizeof(PlanCounts));
    L.temp_bytes = sort_temp_bytes(n, ntp, nt);
    L.temp = take(L.temp_bytes);
    L.max_tp = ntp;
    L.total = off;
    return L;
}

static inline unsigned blocks(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

hipError_t build_plan_device(lr_plan *P, char *buf, const PlanLayout &L, const double *uvw,
                             const ChanConst *d_cc, const MapGeom &g, const KeyLayout &kl,
                             const CFView &cf, const int32_t *ant1, const int32_t *ant2,
                             int32_t nant, const double *ant_dlm, double du_dl,
                             double dv_dm, int32_t per, bool lpt, hipStream_t s) {
    hipError_t e;
    const int64_t n = P->n_pairs;
    const int64_t nt = tile_count(g.nx, g.ny, g.nplane);
    uint64_t *keys_a = (uint64_t *)(buf + L.keys_a), *keys_b = (uint64_t *)(buf + L.keys_b);
    int32_t *vals_a = (int32_t *)(buf + L.vals_a);
    int32_t *order = (int32_t *)(buf + L.order);
    int32_t *flags = (int32_t *)(buf + L.flags);
    int32_t *scan = (int32_t *)(buf + L.scan);
    int32_t *gidx = (int32_t *)(buf + L.gidx);
    PlanCounts *pc = (PlanCounts *)(buf + L.counter);
    void *temp = buf + L.temp;
    size_t temp_bytes = L.temp_bytes;
    P->order = order;
    P->gidx = gidx;
    P->pair_group = (int32_t *)(buf + L.pair_group);
    P->period = 0;
    P->group_start = (int32_t *)(buf + L.group_start);
    P->groups = (GroupMeta *)(buf + L.groups);
    P->tp_group = (int32_t *)(buf + L.tp_group);
    P->chunk_start = (int32_t *)(buf + L.chunk_start);
    P->chunk_tile = (int32_t *)(buf + L.chunk_tile);
    P->chunk_excl = (int32_t *)(buf + L.chunk_excl);
    P->chunk_order = nullptr;
    P->by_plane = 0;
    P->tile_state = (int32_t *)(buf + L.tile_state);
    P->n_tiles = nt;
    P->shared_tiles = (int32_t *)(buf + L.shared_tiles);
    P->n_shared = 0;
    P->geo = (int64_t *)(buf + L.geo);
    P->tile_tp = (int32_t *)(buf + L.tile_tp);
    P->multi = (int32_t *)(buf + L.multi);
    P->n_multi = 0;
    P->sep_part = (int4 *)(buf + L.sep_part);
    P->n_sep_parts = 0;
    P->sep_shared = (int32_t *)(buf + L.sep_shared);
    P->n_sep_shared = 0;
    P->cc = d_cc;
    P->n_kept = P->n_groups = P->n_tile_pairs = P->n_chunks = P->taps = 0;
    PlanCounts hc = {};
    auto read_counts = [&]() {
        hipError_t r = hipMemcpyAsync(&hc, pc, sizeof hc, hipMemcpyDeviceToHost, s);
        return r != hipSuccess ? r : hipStreamSynchronize(s);
    };
    // The host waits twice: for the numbers of groups and tile pairs, which
    // size the second half's launches, and at the end for what the calls on
    // the plan launch by.  (One wait per count and a launch per small pass
    // had left the GPU idle for a third of a small build: a degridding job of
    // 1.6e4 pairs without a plan took 808 us, now 238 us, of which the build
    // is about 190; a gridding job of 1.3e6 pairs 2340 us, now 750 us.)  What
    // is left of a small build is the latency of some thirty launches, of a
    // large one the radix sorts' passes.
    hipLaunchKernelGGL(k_plan_init, dim3(blocks(nt + 1, 256)), dim3(256), 0, s, pc,
                       P->tile_state, P->tile_tp, nt);
    if (n == 0) return hipGetLastError();
    const int32_t rmax = (int32_t)std::min<int64_t>(P->nrow - 1, 1 << 16);
    if (rmax >= 1)
        hipLaunchKernelGGL(k_row_period, dim3(blocks(rmax, 64)), dim3(64), 0, s, uvw, P->nrow,
                           rmax, &pc->period);
    hipLaunchKernelGGL(k_plan_keys, dim3(blocks(n, 256)), dim3(256), 0, s, (uint32_t)n,
                       (uint32_t)P->nchan, uvw, d_cc, g, kl, ant1, ant2, nant, keys_a, vals_a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    e = rocprim::radix_sort_pairs<SortConfig>(temp, temp_bytes, keys_a, keys_b, vals_a, order,
                                              (size_t)n, 0, kl.end_bit, s);
    if (e != hipSuccess) return e;
    const int32_t ntx = (g.nx + kTile - 1) / kTile, nty = (g.ny + kTile - 1) / kTile;
    uint64_t *heads = keys_a;                   // the sort is done with its input
    uint32_t *tk_a = (uint32_t *)flags, *tk_b = (uint32_t *)keys_b;
    e = rocprim::inclusive_scan(temp, temp_bytes, group_heads(GroupHead{keys_b, cf.h, kl, P->merged}),
                                heads, (size_t)n, rocprim::plus<uint64_t>(), s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_group_meta, dim3(std::min(blocks(n, 256), (unsigned)kMetaBlocks)),
                       dim3(256), 0, s, keys_b, heads, order, (uint32_t)n, (uint32_t)P->nchan, uvw,
                       d_cc, g, cf, ant1, ant2, ant_dlm, du_dl, dv_dm, ntx, nty, gidx,
                       P->group_start, P->groups, P->geo, tk_a, vals_a, pc);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = read_counts()) != hipSuccess) return e;
    const int64_t nk = hc.n_kept, ng = hc.n_groups, ntp = (int64_t)hc.n_tile_pairs;
    if (ntp > L.max_tp || ntp > 0x7fffffff) return hipErrorInvalidValue;
    P->n_kept = nk;
    P->n_groups = ng;
    P->n_tile_pairs = ntp;
    P->taps = (int64_t)hc.taps;
    if (nk == 0) {
        hipLaunchKernelGGL(k_pair_group, dim3(blocks(n, 256)), dim3(256), 0, s, order, gidx,
                           (const int32_t *)nullptr, (int64_t)0, n, P->pair_group);
        return hipGetLastError();
    }
    if (hc.period != kNoPeriod) P->period = (int64_t)hc.period * P->nchan;

    // (tile, group) pairs by tile, their chunks
    int end_bit = 1;
    while (end_bit < 32 && ((int64_t)1 << end_bit) < nt) ++end_bit;
    e = rocprim::radix_sort_pairs<SortConfig>(temp, temp_bytes, tk_a, tk_b, vals_a, P->tp_group,
                                              (size_t)ntp, 0, end_bit, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_tile_ranges, dim3(blocks(nt + 1, 256)), dim3(256), 0, s, tk_b, ntp, nt,
                       P->tile_tp);
    TileSums *sums = (TileSums *)keys_a;
    e = rocprim::inclusive_scan(temp, temp_bytes, tile_counts(TileCounts{P->tile_tp, (uint32_t)per}),
                                sums, (size_t)nt, TileSumsPlus(), s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_tile_chunks, dim3(blocks(nt * 64, 256)), dim3(256), 0, s, P->tile_tp,
                       sums, (uint32_t)nt, (uint32_t)per, P->chunk_start, P->chunk_tile,
                       P->chunk_excl, P->tile_state, P->shared_tiles, pc);
    if (sep_table(P, cf)) {
        // parts of the separable gridder, tiles with most pairs first
        uint32_t *ck_a = (uint32_t *)flags, *ck_b = (uint32_t *)scan;
        int32_t *tile = (int32_t *)keys_b, *nparts = flags, *first = vals_a;
        const int32_t S = 2 * cf.h0 + 1;
        hipLaunchKernelGGL(k_sep_count, dim3(blocks(nt, 256)), dim3(256), 0, s, P->tile_tp, nt,
                           ck_a, vals_a);
        e = rocprim::radix_sort_pairs<SortConfig>(temp, temp_bytes, ck_a, ck_b, vals_a, tile,
                                                  (size_t)nt, 0, 16, s);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_sep_nparts, dim3(blocks(nt, 256)), dim3(256), 0, s, P->tile_tp,
                           tile, sums, nt, kSepFill / ((S * S + 63) / 64), nparts);
        e = rocprim::exclusive_scan(temp, temp_bytes, nparts, first, (int32_t)0, (size_t)nt,
                                    rocprim::plus<int32_t>(), s);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_sep_fill, dim3(blocks(nt, 256)), dim3(256), 0, s, P->tile_tp, tile,
                           nparts, first, nt, P->sep_part, P->sep_shared, pc);
    } else {
        // with a small kernel table (lpt) the gridder launches chunks largest
        // first (a stable sort: ties keep tile order), so the long ones do not
        // trail the launch; with a larger table it launches them plane by
        // plane (tile order within a plane), so the chunks in flight read one
        // plane of the table, which the caches hold, instead of all of them.
        // Sorted at their most possible number, so that the host need not wait
        // for the count.
        const uint32_t slots = (uint32_t)std::min<int64_t>(ntp, ntp / per + nt);
        int end_bits = kCostBits;
        if (lpt) {
            hipLaunchKernelGGL(k_chunk_cost, dim3(blocks((int64_t)slots * 64, 256)), dim3(256), 0,
                               s, P->chunk_start, P->chunk_tile, P->tp_group, P->groups, ntx, nty,
                               slots, pc, tk_a, vals_a);
        } else {
            const int64_t planes = (int64_t)cf.n_fg * cf.n_w;
            end_bits = 1;
            while (end_bits < 32 && ((int64_t)1 << end_bits) < planes) ++end_bits;
            hipLaunchKernelGGL(k_chunk_plane, dim3(blocks(slots, 256)), dim3(256), 0, s,
                               P->chunk_start, P->tp_group, P->groups, cf.n_w,
                               (uint32_t)planes - 1, slots, pc, tk_a, vals_a);
        }
        P->chunk_order = (int32_t *)(buf + L.chunk_order);
        P->by_plane = lpt ? 0 : 1;
        e = rocprim::radix_sort_pairs<SortConfig>(temp, temp_bytes, tk_a, (uint32_t *)scan, vals_a,
                                                  P->chunk_order, (size_t)slots, 0, end_bits, s);
        if (e != hipSuccess) return e;
    }

    // with a row period: groups that are one unbroken stretch of one track
    // (pairs of another track, or a gap, break the stride L between
    // consecutive members), one-member groups, the list of the others
    int32_t *single = nullptr;
    if (P->period > 0) {
        single = scan;
        hipLaunchKernelGGL(k_single_init, dim3(blocks(ng, 256)), dim3(256), 0, s, single, ng, 1);
        hipLaunchKernelGGL(k_single_gaps, dim3(blocks(nk, 256)), dim3(256), 0, s, order, gidx,
                           nk, P->period, single);
        const int32_t rounds = (int32_t)std::max<int64_t>(1, std::min<int64_t>(kKindRounds, ng >> 16));
        hipLaunchKernelGGL(k_group_kinds, dim3(blocks(ng, 256 * rounds)), dim3(256), 0, s,
                           P->group_start, ng, rounds, single, P->multi, pc);
    }
    hipLaunchKernelGGL(k_pair_group, dim3(blocks(n, 256)), dim3(256), 0, s, order, gidx,
                       (const int32_t *)single, nk, n, P->pair_group);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = read_counts()) != hipSuccess) return e;
    P->n_chunks = hc.n_chunks;
    P->n_shared = hc.n_shared;
    P->n_sep_parts = hc.n_sep_parts;
    P->n_sep_shared = hc.n_sep_shared;
    P->n_multi = hc.n_multi;
    return hipSuccess;
}

}  // namespace lr
