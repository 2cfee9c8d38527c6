// Degridding D (Eq. ME-MOD-GRIDDED): one wavefront (half or a quarter of one
// for supports up to 15) per group gathers sum_t conj(Ct phi) grid over the
// footprint and reduces across lanes.
#include "k_common.h"

namespace lr {

// ---------------------------------------------------------------------------
struct DegridArgs {
    const GroupMeta *groups;
    int64_t n_groups;
    const void *grid;
    void *Vg;
    CFView cf;
    int32_t nx, ny;
    int64_t pol_stride;
    uint32_t mix;     // Mueller pass: bit q * NPOL + p adds grid pol p's gather into q (0: none)
    int32_t accum;    // add to Vg (later Mueller passes) instead of writing it
};

// Workgroups are dealt to the eight XCDs one by one; workgroup b takes the
// place that hands each XCD runs of kDegridRun consecutive workgroups.  The plan
// orders the groups of one kernel plane by blocks of 16 x 16 pixels, so a run's
// footprints share most of their cells and its kernels come from one plane,
// and both stay in that XCD's L2.  Degridding with runs of 1 / 4 / 16 / 32 / 128:
// A+W chunk 14.9 / 13.1 / 12.5 / 12.4 / 12.2 ms, W-projection (FP32) 128 / 107 /
// 104 / 103 / 109 us, a job of 1e4 groups 35.5 / 33.2 / 32.0 / 32.2 / 36.6 us
// (long runs leave XCDs idle at the end).  The launch is padded to whole rounds
// (dealing the last, partial round one by one instead: W-projection 103 -> 105 us).
constexpr int kDegridRun = 32;
__device__ __forceinline__ int64_t xcd_run(unsigned b) {
    return ((b >> 3) / kDegridRun * 8 + (b & 7)) * kDegridRun + (b >> 3) % kDegridRun;
}
static inline unsigned run_blocks(int64_t n_groups, int per) {
    const int64_t round = 8 * kDegridRun;
    return (unsigned)((nblk(n_groups, per) + round - 1) / round * round);
}

// A group's NPOL gathers written to Vg: as they are, or (a Mueller pass)
// correlation q gets the sum of the pols p its mask bits select, added to
// what earlier passes left when accum is set.
template <typename T, int NPOL>
__device__ __forceinline__ void store_group(const DegridArgs &a, int64_t g, int form,
                                            const cpx<T> (&v)[NPOL]) {
    cpx<T> *out = (cpx<T> *)a.Vg + g * NPOL;
    for (int q = 0; q < NPOL; ++q) {
        cpx<T> r;
        if (a.mix == 0) {
            r = v[q];
        } else {
            r = {(T)0, (T)0};
            for (int p = 0; p < NPOL; ++p)
                if ((a.mix >> (q * NPOL + p)) & 1u) {
                    r.x += v[p].x;
                    r.y += v[p].y;
                }
            if (negated(a.cf, form)) r = {-r.x, -r.y};
        }
        if (a.accum) {
            r.x += out[q].x;
            r.y += out[q].y;
        }
        out[q] = r;
    }
}

// Taps per lane whose loads are in flight together in the degridder: 4, or
// 8 with 4-byte (FP16 / BF16) kernel values, whose raw words take half the
// registers.
constexpr int kDegridTaps = 4;

// One wavefront per group: lanes walk the footprint taps in row-major order,
// four or eight taps per lane in flight; the sub-kernel and the footprint's
// corner cell (per pol) are scalar base addresses and a lane carries 32-bit
// offsets, advanced by 64 taps at a time without division.
template <typename T, int ST, int NPOL, bool PO, bool RE>
__global__ __launch_bounds__(256) void k_degrid(DegridArgs a) {
    constexpr int E = CFRaw<ST>::bytes;
    constexpr int NT = E <= 4 ? 2 * kDegridTaps : kDegridTaps;
    typedef typename std::conditional<RE, typename CFReal<ST>::R, typename CFRaw<ST>::R>::type Raw;
    const int lane = threadIdx.x & 63;
    const int64_t g = xcd_run(blockIdx.x) * (blockDim.x >> 6) + uni(threadIdx.x >> 6);
    if (g >= a.n_groups) return;
    const GroupMeta gm = a.groups[g];
    const int h = uni(gm.h);
    const int S = 2 * h + 1;
    const int SS = S * S;
    const float sc = a.cf.scale[(int64_t)gm.fg * a.cf.n_w + gm.k];
    const int form = uni(gm.form);
    const bool cj = (form & kConj) != 0;
    const char *cfb = (const char *)a.cf.table + uni64(gm.cf_off) * E;
    // corner cell (tap (0, 0)) of pol 0
    const int64_t corner = uni64(gm.cell) - (int64_t)h * a.nx - h;
    const int64_t pstride = a.pol_stride * (int64_t)(2 * sizeof(T));
    // one scalar base per pol (its byte offset made opaque, so that a lane's
    // offset is added to it rather than folded into 64-bit vector arithmetic)
    const char *gbp[NPOL];
    for (int p = 0; p < NPOL; ++p)
        gbp[p] = (const char *)a.grid + uni64(corner * (int64_t)(2 * sizeof(T)) + p * pstride);
    const int row = a.nx * (int)(2 * sizeof(T));          // bytes per grid row
    // lane's first tap and the per-step advance of 64 taps
    const int dty = 64 / S, dtx = 64 - dty * S;
    // taps in the order the sub-kernel stores them; on flipped axes the grid
    // (and the tap's coordinate) runs backwards
    const int scol = form & kFlipU ? -(int)(2 * sizeof(T)) : (int)(2 * sizeof(T));
    const int srow = form & kFlipV ? -row : row;
    int ty = lane / S, tx = lane - (lane / S) * S;
    int goff = (form & kFlipV ? (S - 1) * row : 0) +
               (form & kFlipU ? (S - 1) * (int)(2 * sizeof(T)) : 0) + ty * srow + tx * scol;
    cpx<T> sum[NPOL];
    for (int p = 0; p < NPOL; ++p) sum[p] = {(T)0, (T)0};
    for (int t0 = 0; t0 < SS; t0 += 64 * NT) {
        Raw cr[NT];
        cpx<T> gv[NT][NPOL];
        bool ok[NT];
        int txs[NT], tys[NT];
        for (int u = 0; u < NT; ++u) {
            const int tap = t0 + u * 64 + lane;
            ok[u] = tap < SS;
            txs[u] = form & kFlipU ? S - 1 - tx : tx;
            tys[u] = form & kFlipV ? S - 1 - ty : ty;
            // every lane loads (a lane past the footprint reads tap 0, in
            // bounds, and adds nothing): loads outside divergent branches
            // let the waits count down tap by tap
            const uint32_t co = ok[u] ? (uint32_t)tap * (uint32_t)E : 0u;
            const uint32_t go = ok[u] ? (uint32_t)goff : 0u;
            cr[u] = *(const Raw *)(cfb + co);
            for (int p = 0; p < NPOL; ++p) {
                const T *q = (const T *)(gbp[p] + go);
                gv[u][p] = {q[0], q[1]};
            }
            // advance by 64 taps
            tx += dtx;
            ty += dty;
            goff += dty * srow + dtx * scol;
            if (tx >= S) {
                tx -= S;
                ++ty;
                goff += srow - S * scol;
            }
        }
        for (int u = 0; u < NT; ++u) {
            if constexpr (RE) {
                const T c = ok[u] ? CFReal<ST>::decode(cr[u], sc) : (T)0;
                for (int p = 0; p < NPOL; ++p) {
                    sum[p].x = fma(c, gv[u][p].x, sum[p].x);
                    sum[p].y = fma(c, gv[u][p].y, sum[p].y);
                }
            } else {
                cpx<T> cv = CFRaw<ST>::decode(cr[u], sc);
                if (!ok[u]) cv = {(T)0, (T)0};
                if (cj) cv.y = -cv.y;
                if (PO) cv = cmul(cv, phasor<T>(gm, txs[u] - h, tys[u] - h, a.cf.O));
                for (int p = 0; p < NPOL; ++p) cmac_conj(sum[p], cv, gv[u][p]);
            }
        }
    }
    cpx<T> tot[NPOL];
    for (int p = 0; p < NPOL; ++p) tot[p] = {wave_sum(sum[p].x), wave_sum(sum[p].y)};
    if (lane == 0) store_group<T, NPOL>(a, g, form, tot);
}

// FP32 grids without a pointing phasor: lanes over pairs of neighbouring
// taps of a footprint row, so that one 16-byte load brings two grid values
// of a pol and one 16-byte (8-byte with FP16 / BF16 values) load two kernel
// values: half the vector-memory instructions of one tap per load, whose
// address processing bounds the one-tap kernel.  Pairs start at even grid
// columns (the row's first pair may begin one column before the
// footprint); with nx even a pair never crosses a grid row.  A pair's tap
// outside the footprint row reads its neighbour in the table (the row
// before or after, or the blob's padding past the table's end) and adds
// zero.
// With small footprints the instructions per pair and per group count: offsets
// are advanced, not multiplied out, the quotients by the pairs per row come
// from one reciprocal, and a mirrored row's values are swapped by a second copy
// of the sums, not by selects.  With products, divisions and selects: A+W chunk
// 12.99 against 12.37 ms, W-projection 107 against 103 us, narrow A+W with one
// correlation 110 against 102 us.
constexpr int kDegridPairs = 3;      // pairs per lane in flight

template <int ST, int NPOL, bool RE>
__global__ __launch_bounds__(256) void k_degrid_pair(DegridArgs a) {
    constexpr int E = CFRaw<ST>::bytes;                 // 8: f32, 4: f16 / bf16 pair
    typedef typename std::conditional<E == 8, f32x4_a8, u32x2_a4>::type Raw2;
    typedef typename CFRaw<ST>::R Raw;
    constexpr int NT = kDegridPairs;
    const int lane = threadIdx.x & 63;
    const int64_t g = xcd_run(blockIdx.x) * (blockDim.x >> 6) + uni(threadIdx.x >> 6);
    if (g >= a.n_groups) return;
    const GroupMeta gm = a.groups[g];
    const int h = uni(gm.h);
    const int S = 2 * h + 1;
    const float sc = a.cf.scale[(int64_t)gm.fg * a.cf.n_w + gm.k];
    const int form = uni(gm.form);
    const bool cj = (form & kConj) != 0;
    const int lead = (uni(gm.pu) - h) & 1;              // footprint starts at an odd column
    const int W2 = (S + lead + 1) >> 1;                 // pairs per footprint row
    const int NP = S * W2;
    // kernel bytes from one element before the sub-kernel; the pair of row r and
    // columns (2 c - lead, 2 c - lead + 1) starts at byte k0 + r sv + c su, where
    // a flipped row holds the pair's two values in reverse order.
    // grid cell (0, -lead) of pol 0
    const char *cfb = (const char *)a.cf.table + (uni64(gm.cf_off) - 1) * E;
    const bool fu = (form & kFlipU) != 0;
    const int su = fu ? -2 * E : 2 * E, sv = form & kFlipV ? -S * E : S * E;
    const int k0 = E * (1 + (fu ? S - 2 + lead : -lead) + (form & kFlipV ? (S - 1) * S : 0));
    const int64_t corner = uni64(gm.cell) - (int64_t)h * a.nx - h - lead;
    const int64_t pstride = a.pol_stride * 8;
    const char *gbp[NPOL];
    for (int p = 0; p < NPOL; ++p)
        gbp[p] = (const char *)a.grid + uni64(corner * 8 + p * pstride);
    const int row = a.nx * 8;
    // quotients of at most 64 by W2 (halves keep clear of whole numbers)
    const float inv = __builtin_amdgcn_rcpf((float)W2);
    const int dr = uni((int)(64.5f * inv)), dc = 64 - dr * W2;
    // this lane's pair, and its steps to the one 64 pairs on without and with a
    // change of row
    const int r = (int)(((float)lane + 0.5f) * inv);
    int c = lane - r * W2;
    int co = r * sv + c * su + k0, go = r * row + c * 16;
    const int dco = dr * sv + dc * su, dgo = dr * row + dc * 16;
    const int wco = dco + sv - W2 * su, wgo = dgo + row - W2 * 16;
    cpx<float> sum[NPOL];
    for (int p = 0; p < NPOL; ++p) sum[p] = {0.f, 0.f};
    for (int t0 = 0; t0 < NP; t0 += 64 * NT) {
        Raw2 cr[NT];
        f32x4_a8 gv[NT][NPOL];
        bool ok[NT], v0[NT], v1[NT];
        for (int u = 0; u < NT; ++u) {
            const int pp = t0 + u * 64 + lane;
            ok[u] = pp < NP;
            const int tu0 = 2 * c - lead;
            v0[u] = ok[u] && tu0 >= 0;
            v1[u] = ok[u] && tu0 + 1 < S;
            // lanes past the footprint load pair 0 (in bounds) and add nothing
            const uint32_t kat = ok[u] ? (uint32_t)co : 0u, gat = ok[u] ? (uint32_t)go : 0u;
            cr[u] = *(const Raw2 *)(cfb + kat);
            for (int p = 0; p < NPOL; ++p) gv[u][p] = *(const f32x4_a8 *)(gbp[p] + gat);
            c += dc;
            const bool wrap = c >= W2;
            c -= wrap ? W2 : 0;
            co += wrap ? wco : dco;
            go += wrap ? wgo : dgo;
        }
        // one copy of the sums for each order of the pair's values
        auto add = [&](auto flipped) {
            for (int u = 0; u < NT; ++u) {
                // the pair's two kernel values, zero outside the footprint row
                cpx<float> c0, c1;
                if constexpr (E == 8) {
                    c0 = {cr[u].x, cr[u].y};
                    c1 = {cr[u].z, cr[u].w};
                } else {
                    c0 = CFRaw<ST>::decode((Raw)cr[u].x, sc);
                    c1 = CFRaw<ST>::decode((Raw)cr[u].y, sc);
                }
                if constexpr (decltype(flipped)::value) {
                    const cpx<float> t = c0;
                    c0 = c1;
                    c1 = t;
                }
                if (RE) c0.y = c1.y = 0.f;
                if (!v0[u]) c0 = {0.f, 0.f};
                if (!v1[u]) c1 = {0.f, 0.f};
                if (cj) {
                    c0.y = -c0.y;
                    c1.y = -c1.y;
                }
                for (int p = 0; p < NPOL; ++p) {
                    const cpx<float> g0 = {gv[u][p].x, gv[u][p].y}, g1 = {gv[u][p].z, gv[u][p].w};
                    if constexpr (RE) {
                        sum[p].x = fmaf(c0.x, g0.x, sum[p].x);
                        sum[p].y = fmaf(c0.x, g0.y, sum[p].y);
                        sum[p].x = fmaf(c1.x, g1.x, sum[p].x);
                        sum[p].y = fmaf(c1.x, g1.y, sum[p].y);
                    } else {
                        cmac_conj(sum[p], c0, g0);
                        cmac_conj(sum[p], c1, g1);
                    }
                }
            }
        };
        if (fu) add(std::true_type{});
        else add(std::false_type{});
    }
    cpx<float> tot[NPOL];
    for (int p = 0; p < NPOL; ++p) tot[p] = {wave_sum(sum[p].x), wave_sum(sum[p].y)};
    if (lane == 0) store_group<float, NPOL>(a, g, form, tot);
}

// Small supports (S <= 2 kDegridSmallH + 1): a 7 x 7 footprint would leave
// most of a wavefront idle, so 16 lanes take one group (four groups per
// wavefront), four taps per lane in flight, and reduce over their 16 lanes.
constexpr int kDegridSmallH = 7;

template <typename T, int ST, int NPOL, bool PO, bool RE>
__global__ __launch_bounds__(256) void k_degrid_small(DegridArgs a) {
    constexpr int E = CFRaw<ST>::bytes;
    typedef typename std::conditional<RE, typename CFReal<ST>::R, typename CFRaw<ST>::R>::type Raw;
    const int sub = threadIdx.x & 15;
    const int64_t g = xcd_run(blockIdx.x) * (blockDim.x >> 4) + (threadIdx.x >> 4);
    const bool live = g < a.n_groups;
    int form = 0;
    cpx<T> sum[NPOL];
    for (int p = 0; p < NPOL; ++p) sum[p] = {(T)0, (T)0};
    if (live) {
        const GroupMeta gm = a.groups[g];
        const int h = gm.h;
        const int S = 2 * h + 1;
        const int SS = S * S;
        const float invS = 1.0f / (float)S;
        const float sc = a.cf.scale[(int64_t)gm.fg * a.cf.n_w + gm.k];
        const char *cfb = (const char *)a.cf.table + gm.cf_off * E;
        form = gm.form;
        // taps in storage order; on flipped axes the grid runs backwards
        const bool fu = (form & kFlipU) != 0, fv = (form & kFlipV) != 0;
        const int64_t corner = gm.cell - (int64_t)h * a.nx - h;
        const T *grid = (const T *)a.grid;
        for (int t0 = 0; t0 < SS; t0 += 64) {
            Raw cr[4];
            cpx<T> gv[4][NPOL];
            int tys[4], txs[4];
            for (int u = 0; u < 4; ++u) {
                const int tap = t0 + u * 16 + sub;
                int ty, tx;
                divmod_small(tap, S, invS, ty, tx);
                if (fu) tx = S - 1 - tx;
                if (fv) ty = S - 1 - ty;
                tys[u] = ty;
                txs[u] = tx;
                // every lane loads (past the footprint: tap 0, in bounds,
                // adding nothing), outside divergent branches
                const bool in = tap < SS;
                const int64_t cell = in ? corner + (int64_t)ty * a.nx + tx : corner;
                cr[u] = *(const Raw *)(cfb + (in ? (int64_t)tap * E : 0));
                for (int p = 0; p < NPOL; ++p) {
                    const T *q = grid + 2 * (cell + p * a.pol_stride);
                    gv[u][p] = {q[0], q[1]};
                }
            }
            for (int u = 0; u < 4; ++u) {
                const bool in = t0 + u * 16 + sub < SS;
                if constexpr (RE) {
                    const T c = in ? CFReal<ST>::decode(cr[u], sc) : (T)0;
                    for (int p = 0; p < NPOL; ++p) {
                        sum[p].x = fma(c, gv[u][p].x, sum[p].x);
                        sum[p].y = fma(c, gv[u][p].y, sum[p].y);
                    }
                } else {
                    cpx<T> cv = CFRaw<ST>::decode(cr[u], sc);
                    if (!in) cv = {(T)0, (T)0};
                    if (form & kConj) cv.y = -cv.y;
                    if (PO) cv = cmul(cv, phasor<T>(gm, txs[u] - h, tys[u] - h, a.cf.O));
                    for (int p = 0; p < NPOL; ++p) cmac_conj(sum[p], cv, gv[u][p]);
                }
            }
        }
    }
    for (int p = 0; p < NPOL; ++p)
        for (int off = 8; off > 0; off >>= 1) {
            sum[p].x += __shfl_xor(sum[p].x, off);
            sum[p].y += __shfl_xor(sum[p].y, off);
        }
    if (live && sub == 0) store_group<T, NPOL>(a, g, form, sum);
}

// Single-plane real tables of support up to 15 (the Standard kernel), FP32
// grids: 32 lanes per group, lanes over pairs of neighbouring taps (4 pairs x 8
// rows for supports up to 7, else 8 x 4), starting at even grid columns as in
// k_degrid_pair, so one 16-byte load brings two cells of a pol and one the two
// kernel values.  A pair that would reach past the row's end moves one column
// in, so that no cell outside the footprint is read: it may hold anything, and
// 0 times an infinity is not 0.  A vector load costs a quarter clock per lane
// whatever its width, so a 7 x 7 footprint takes 5 loads of 32 lanes where
// k_degrid_small needs 20 of 16.  Two groups per half wavefront are in flight.  A
// group is known from its pixel and offsets alone (geo, one scalar load of four
// groups instead of four 80-byte records through the vector path).
// 6.2 M groups of one sample (8192^2 x 4), degrid call against k_degrid_small:
// 1352 -> 798 us, of which 140 us expand the groups; supports of 11 and 15:
// 2304 -> 1668 and 4004 -> 2379 us.  (With pairs that reach past the row's end
// 846, 1738 and 2322 us.)
constexpr int kSepGroups = 2;            // groups per half wavefront

struct DegridSepArgs {
    const int64_t *geo;
    int64_t n_groups;
    const void *grid, *table;            // table: element 0 of plane (0, 0)
    float *Vg;
    const float *sc;                     // 2^-e of plane (0, 0)
    int32_t O, h, nx;
    int64_t pol_stride;
};

template <int CTRL>
__device__ __forceinline__ float dpp_add(float v) {
    return v + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, true));
}

// Sum over each half wavefront of each of N = 8, 4 or 2 values; lane l of the
// half receives value l / (32 / N).
template <int N>
__device__ __forceinline__ float half_sums(const float (&v)[N]) {
    typedef uint32_t u2 __attribute__((ext_vector_type(2)));
    constexpr int ROR8 = 0x128, MIRROR8 = 0x141, XOR2 = 0x4E, XOR1 = 0xB1;
    // the rows of 16 lanes swap the values the other row keeps
    auto fold = [](float a, float b) {
        const u2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        return __uint_as_float(r.x) + __uint_as_float(r.y);
    };
    float t;
    if constexpr (N == 8) {
        float a[4];
        for (int i = 0; i < 4; ++i) a[i] = dpp_add<ROR8>(fold(v[i], v[i + 4]));
        const bool q = threadIdx.x & 8;
        const float c0 = dpp_add<MIRROR8>(q ? a[2] : a[0]), c1 = dpp_add<MIRROR8>(q ? a[3] : a[1]);
        t = (threadIdx.x & 4) ? c1 : c0;
    } else if constexpr (N == 4) {
        const float a0 = dpp_add<ROR8>(fold(v[0], v[2])), a1 = dpp_add<ROR8>(fold(v[1], v[3]));
        t = dpp_add<MIRROR8>((threadIdx.x & 8) ? a1 : a0);
    } else {
        t = dpp_add<MIRROR8>(dpp_add<ROR8>(fold(v[0], v[1])));
    }
    return dpp_add<XOR1>(dpp_add<XOR2>(t));
}

template <int ST, int NPOL, int PW>
__global__ __launch_bounds__(256) void k_degrid_sep(DegridSepArgs a) {
    constexpr int E = CFRaw<ST>::bytes, NV = 2 * NPOL, NR = 32 / PW, NG = kSepGroups;
    typedef typename std::conditional<E == 8, f32x4_a8, u32x2_a4>::type Raw2;
    const int lane = threadIdx.x & 63, c = lane & (PW - 1), rl = (lane & 31) / PW;
    const bool second = lane >= 32;
    const int64_t gw = (xcd_run(blockIdx.x) * 4 + uni(threadIdx.x >> 6)) * (2 * NG);
    if (gw >= a.n_groups) return;
    const int h = a.h, S = 2 * h + 1, half = a.O >> 1, no = a.O + 1;
    const int row = a.nx * 8;
    const char *gbp[NPOL];
    for (int p = 0; p < NPOL; ++p) gbp[p] = (const char *)a.grid + uni64(p * a.pol_stride * 8);
    // of this lane's half, per group: kernel element and grid byte of this lane's
    // pair in row 0, the kernel's walk, and which cells of the pair count
    uint32_t kb[NG], gb[NG];
    int sv[NG];
    bool fu[NG], in0[NG], in1[NG];
    for (int u = 0; u < NG; ++u) {
        uint32_t kk[2], gg[2];
        int vv[2];
        bool ff[2], ll[2];
        for (int q = 0; q < 2; ++q) {
            const int64_t g = gw + 2 * u + q;
            const int64_t geo = a.geo[g < a.n_groups ? g : a.n_groups - 1];
            const int pu = (int)(geo & 0xFFFF), pv = (int)((geo >> 16) & 0xFFFF);
            const int ou = (int)(int16_t)(geo >> 32), ov = (int)(int16_t)(geo >> 48);
            const bool fv = ov > 0;
            ff[q] = ou > 0;
            ll[q] = ((pu - h) & 1) != 0;
            vv[q] = fv ? -S : S;
            // the first row's pair (0, 1), where a flipped row holds it last
            kk[q] = (uint32_t)(((half - abs(ov)) * no + (half - abs(ou))) * S * S +
                               (ff[q] ? S - 2 : 0) + (fv ? (S - 1) * S : 0));
            gg[q] = (uint32_t)((int64_t)(pv - h) * row + (pu - h) * 8);
        }
        fu[u] = second ? ff[1] : ff[0];
        sv[u] = second ? vv[1] : vv[0];
        // the aligned pair (t, t + 1); one that reaches past the row's end is
        // read one column further in, where its other cell is another lane's
        const int t = 2 * c - ((second ? ll[1] : ll[0]) ? 1 : 0);
        const int at = min(max(t, 0), S - 2);
        in0[u] = t <= S - 2;
        in1[u] = t >= 0 && t < S;
        kb[u] = (second ? kk[1] : kk[0]) + (uint32_t)(fu[u] ? -at : at);
        gb[u] = (second ? gg[1] : gg[0]) + (uint32_t)(at * 8);
    }
    const float sc = E == 4 ? a.sc[0] : 1.0f;
    float sum[NG][NV];
    for (int u = 0; u < NG; ++u)
        for (int i = 0; i < NV; ++i) sum[u][i] = 0.f;
    for (int r0 = 0; r0 < S; r0 += NR) {
        const int r = r0 + rl;
        const bool ok = r < S;
        const int rr = ok ? r : 0;             // lanes past the footprint add nothing
        Raw2 kv[NG];
        f32x4_a8 gv[NG][NPOL];
        for (int u = 0; u < NG; ++u) {
            kv[u] = *(const Raw2 *)((const char *)a.table + (int64_t)(int32_t)(kb[u] + rr * sv[u]) * E);
            const uint32_t at = gb[u] + (uint32_t)(rr * row);
            for (int p = 0; p < NPOL; ++p) gv[u][p] = *(const f32x4_a8 *)(gbp[p] + at);
        }
        for (int u = 0; u < NG; ++u) {
            float c0, c1;
            if constexpr (E == 8) {
                c0 = kv[u].x;
                c1 = kv[u].z;
            } else {
                c0 = CFReal<ST>::decode((uint16_t)(kv[u].x & 0xFFFF), sc);
                c1 = CFReal<ST>::decode((uint16_t)(kv[u].y & 0xFFFF), sc);
            }
            if (fu[u]) {
                const float s = c0;
                c0 = c1;
                c1 = s;
            }
            if (!ok || !in0[u]) c0 = 0.f;
            if (!ok || !in1[u]) c1 = 0.f;
            for (int p = 0; p < NPOL; ++p) {
                sum[u][2 * p] = fmaf(c1, gv[u][p].z, fmaf(c0, gv[u][p].x, sum[u][2 * p]));
                sum[u][2 * p + 1] = fmaf(c1, gv[u][p].w, fmaf(c0, gv[u][p].y, sum[u][2 * p + 1]));
            }
        }
    }
    for (int u = 0; u < NG; ++u) {
        const float t = half_sums<NV>(sum[u]);
        const int64_t g = gw + 2 * u + (second ? 1 : 0);
        if ((lane & (32 / NV - 1)) == 0 && g < a.n_groups)
            a.Vg[g * NV + (lane & 31) / (32 / NV)] = t;
    }
}

template <int ST, int NPOL>
static hipError_t degrid_sep_t(const DegridSepArgs &da, hipStream_t s) {
    dim3 grd(run_blocks(da.n_groups, 8 * kSepGroups)), blk(256);
    if (da.h <= 3) hipLaunchKernelGGL((k_degrid_sep<ST, NPOL, 4>), grd, blk, 0, s, da);
    else hipLaunchKernelGGL((k_degrid_sep<ST, NPOL, 8>), grd, blk, 0, s, da);
    return hipGetLastError();
}

template <int ST>
static hipError_t degrid_sep_np(const DegridSepArgs &da, int npol, hipStream_t s) {
    switch (npol) {
        case 1: return degrid_sep_t<ST, 1>(da, s);
        case 2: return degrid_sep_t<ST, 2>(da, s);
        default: return degrid_sep_t<ST, 4>(da, s);
    }
}

template <typename T, int ST, int NPOL>
static hipError_t degrid_t(const DegridArgs &da, bool po, bool small, hipStream_t s) {
    dim3 blk(256);
    const bool re = !po && da.cf.real;
    if (small) {
        dim3 grd(run_blocks(da.n_groups, 16));
        if (po) hipLaunchKernelGGL((k_degrid_small<T, ST, NPOL, true, false>), grd, blk, 0, s, da);
        else if (re) hipLaunchKernelGGL((k_degrid_small<T, ST, NPOL, false, true>), grd, blk, 0, s, da);
        else hipLaunchKernelGGL((k_degrid_small<T, ST, NPOL, false, false>), grd, blk, 0, s, da);
        return hipGetLastError();
    }
    dim3 grd(run_blocks(da.n_groups, 4));
    if constexpr (sizeof(T) == 4) {
        if (!po) {
            if (re) hipLaunchKernelGGL((k_degrid_pair<ST, NPOL, true>), grd, blk, 0, s, da);
            else hipLaunchKernelGGL((k_degrid_pair<ST, NPOL, false>), grd, blk, 0, s, da);
            return hipGetLastError();
        }
    }
    if (po) hipLaunchKernelGGL((k_degrid<T, ST, NPOL, true, false>), grd, blk, 0, s, da);
    else if (re) hipLaunchKernelGGL((k_degrid<T, ST, NPOL, false, true>), grd, blk, 0, s, da);
    else hipLaunchKernelGGL((k_degrid<T, ST, NPOL, false, false>), grd, blk, 0, s, da);
    return hipGetLastError();
}

template <typename T, int ST>
static hipError_t degrid_np(const DegridArgs &da, int npol, bool po, bool small,
                            hipStream_t s) {
    switch (npol) {
        case 1: return degrid_t<T, ST, 1>(da, po, small, s);
        case 2: return degrid_t<T, ST, 2>(da, po, small, s);
        default: return degrid_t<T, ST, 4>(da, po, small, s);
    }
}

hipError_t launch_degrid(const lr_plan *P, const CFView &cf, const void *grid, void *Vg,
                         int precision, int32_t npol, int32_t nx, int32_t ny, int32_t nplane,
                         int32_t h_max, uint32_t mix, bool accum, hipStream_t s) {
    if (P->n_groups == 0) return hipSuccess;
    DegridArgs da{P->groups, P->n_groups, grid, Vg, cf, nx, ny, (int64_t)nx * ny, mix,
                  accum ? 1 : 0};
    bool po = P->po != 0;
    bool sm = h_max <= kDegridSmallH;
    // geo names a group completely where the table has one plane and the grid
    // one plane; h >= 1: a footprint has a second pair of columns to fall back on
    if (precision != LR_F64 && mix == 0 && !accum && nplane == 1 && cf.h0 >= 1 && sep_table(P, cf)) {
        DegridSepArgs sa{P->geo, P->n_groups, grid, nullptr, (float *)Vg, cf.scale, cf.O, cf.h0,
                         nx, (int64_t)nx * ny};
        const int64_t elem = precision == LR_F32 ? 8 : 4;
        sa.table = (const char *)cf.table + cf.off0 * elem;
        switch (precision) {
            case LR_F32: return degrid_sep_np<LR_F32>(sa, npol, s);
            case LR_F32_CF16: return degrid_sep_np<LR_F32_CF16>(sa, npol, s);
            default: return degrid_sep_np<LR_F32_CFBF16>(sa, npol, s);
        }
    }
    switch (precision) {
        case LR_F64: return degrid_np<double, LR_F64>(da, npol, po, sm, s);
        case LR_F32: return degrid_np<float, LR_F32>(da, npol, po, sm, s);
        case LR_F32_CF16: return degrid_np<float, LR_F32_CF16>(da, npol, po, sm, s);
        default: return degrid_np<float, LR_F32_CFBF16>(da, npol, po, sm, s);
    }
}

}  // namespace lr
