// Hogbom minor cycle (the ModelUpdate step of the imaging section): loop
// gain, threshold exit, one image plane.
//
// One launch per iteration.  Launch k finds the peak from the candidates that
// the workgroups of launch k - 1 left (every workgroup reduces the few hundred
// of them for itself), subtracts gain x peak x PSF (its centre (ny/2, nx/2) on
// the peak) from the residual, adds gain x peak to the model, and leaves its
// own candidates for the next launch in the same pass.  Launch 0 only
// searches.  The launch that meets the exit test records its number, and later
// launches return at once, so a caller may enqueue the whole budget without
// waiting.  (Its own wavefronts may read the number before or after it is
// written, and go the same way either way.)  Ties go to the lowest index.
//
// What bounds it: the image and the PSF read and the image written once per
// iteration, which the XCDs' L2s do not keep from launch to launch.  No
// workgroup waits for, or publishes to, another within a launch: a last
// workgroup that reduced the candidates needed a device-wide fence in each
// workgroup, which writes the XCD's L2 back, and the pixels' coordinates came
// from 64-bit divisions (2048^2 FP32: 35.7 us an iteration, now 14.5 us; the
// 50 MB at the 6.8 TB/s reads reach here take 7.4 us).
#include "lr_internal.h"
#include "lr_launch.h"

namespace lr {

struct HogbomState {
    int32_t iter;         // subtractions done
    int32_t stop;         // the launch that met the exit test (kNoStop: none)
};
constexpr int32_t kNoStop = 0x7fffffff;

// A candidate peak: signed value and pixel, y << 32 | x (-1: none).  An image may
// have more than 2^32 pixels; ordered like the row-major index, and taken apart
// without a division in every thread.
struct Cand {
    double v;
    int64_t i;
};

__device__ __forceinline__ bool better(const Cand &x, const Cand &y) {
    if (x.i < 0) return false;
    const double a = fabs(x.v), b = fabs(y.v);
    return y.i < 0 || a > b || (a == b && x.i < y.i);
}

// Best candidate of the workgroup, returned in every thread.
__device__ Cand block_best(Cand c) {
    __shared__ Cand part[kHogbomThreads / 64];
    for (int off = 32; off > 0; off >>= 1) {
        Cand o;
        o.v = __shfl_xor(c.v, off);
        o.i = (int64_t)__shfl_xor((long long)c.i, off);
        if (better(o, c)) c = o;
    }
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = c;
    __syncthreads();
    c = part[0];
    for (int k = 1; k < kHogbomThreads / 64; ++k)
        if (better(part[k], c)) c = part[k];
    __syncthreads();
    return c;
}

// Four neighbouring pixels, aligned to one (rows and the shifted PSF start
// anywhere).
template <typename T>
struct Quad {
    typedef T V __attribute__((ext_vector_type(4), aligned(sizeof(T))));
};

template <typename T>
__global__ __launch_bounds__(kHogbomThreads) void k_hogbom(T *__restrict__ res,
                                                           const T *__restrict__ psf, T *model,
                                                           int32_t nx, int32_t ny, double gain,
                                                           double threshold, int32_t k,
                                                           HogbomState *st,
                                                           const Cand *in, Cand *out) {
    typedef typename Quad<T>::V V;
    const bool sub = k > 0;
    T c = (T)0;
    int py = 0, px = 0;
    if (sub) {
        if (st->stop < k) return;
        Cand g{0.0, -1};
        for (int b = threadIdx.x; b < (int)gridDim.x; b += kHogbomThreads) {
            const Cand p = in[b];
            if (better(p, g)) g = p;
        }
        g = block_best(g);
        if (g.i < 0 || fabs(g.v) < threshold) {
            if (blockIdx.x == 0 && threadIdx.x == 0) st->stop = k;
            return;
        }
        // the scale is rounded to T before use, in the precision of the image
        c = (T)(gain * g.v);
        py = (int)(g.i >> 32);
        px = (int)(uint32_t)g.i;
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            model[(int64_t)py * nx + px] += c;
            st->iter = k;
        }
    }
    const int cy = ny / 2, cx = nx / 2;
    // this thread's quads of pixels: (y, 4 q), walked without divisions
    const uint32_t nq = ((uint32_t)nx + 3) >> 2, step = gridDim.x * kHogbomThreads;
    const uint32_t dy = step / nq, dq = step - dy * nq;
    const uint32_t first = blockIdx.x * kHogbomThreads + threadIdx.x;
    uint32_t y = first / nq, q = first - y * nq;
    Cand best{0.0, -1};
    T bv = (T)0;
    // pixels come in order along the walk: the first of equal ones wins
    auto see = [&](T r, int64_t i) {
        const T a = r < (T)0 ? -r : r;
        if (a > bv || (best.i < 0 && a == bv)) {
            bv = a;
            best = Cand{(double)r, i};
        }
    };
#pragma unroll 2
    for (; y < (uint32_t)ny; y += dy, q += dq) {
        if (q >= nq) {
            q -= nq;
            if (++y >= (uint32_t)ny) break;
        }
        const int x = (int)(4 * q), sy = (int)y - py + cy, sx = x - px + cx;
        const int64_t i = (int64_t)y * nx + x, at = (int64_t)y << 32 | (uint32_t)x;
        const bool row = sub && (unsigned)sy < (unsigned)ny;
        if (x <= nx - 4 && (!row || (sx >= 0 && sx <= nx - 4) || sx >= nx || sx <= -4)) {
            V r = *(const V *)(res + i);
            if (row && sx >= 0 && sx < nx) {
                const V p = *(const V *)(psf + (int64_t)sy * nx + sx);
                r = r - c * p;
                *(V *)(res + i) = r;
            }
            for (int e = 0; e < 4; ++e) see(r[e], at + e);
        } else {
            for (int e = 0; e < 4 && x + e < nx; ++e) {
                T r = res[i + e];
                if (row && (unsigned)(sx + e) < (unsigned)nx) {
                    r = r - c * psf[(int64_t)sy * nx + sx + e];
                    res[i + e] = r;
                }
                see(r, at + e);
            }
        }
    }
    best = block_best(best);
    if (threadIdx.x == 0) out[blockIdx.x] = best;
}

__global__ void k_hogbom_reset(HogbomState *st) {
    if (threadIdx.x == 0) {
        st->iter = 0;
        st->stop = kNoStop;
    }
}

size_t hogbom_work_bytes(int32_t nx, int32_t ny) {
    (void)nx;
    (void)ny;
    return 256 + 2 * sizeof(Cand) * kHogbomBlocks;
}

template <typename T>
static hipError_t hogbom_t(T *res, const T *psf, T *model, int32_t nx, int32_t ny, double gain,
                           double threshold, int32_t niter, HogbomState *st, Cand *part,
                           hipStream_t s) {
    const int64_t quads = (int64_t)ny * ((nx + 3) / 4);
    const unsigned blocks = (unsigned)std::min<int64_t>(
        kHogbomBlocks, (quads + kHogbomThreads - 1) / kHogbomThreads);
    for (int32_t k = 0; k <= niter; ++k) {
        hipLaunchKernelGGL(k_hogbom<T>, dim3(blocks), dim3(kHogbomThreads), 0, s, res, psf, model,
                           nx, ny, gain, threshold, k, st,
                           part + ((k + 1) & 1) * kHogbomBlocks, part + (k & 1) * kHogbomBlocks);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_hogbom(void *res, const void *psf, void *model, int32_t nx, int32_t ny,
                         int precision, double gain, double threshold, int32_t niter,
                         void *work, int32_t *iters, hipStream_t s) {
    HogbomState *st = (HogbomState *)work;
    Cand *part = (Cand *)((char *)work + 256);
    hipLaunchKernelGGL(k_hogbom_reset, dim3(1), dim3(64), 0, s, st);
    hipError_t e =
        precision == LR_F64
            ? hogbom_t((double *)res, (const double *)psf, (double *)model, nx, ny, gain, threshold,
                       niter, st, part, s)
            : hogbom_t((float *)res, (const float *)psf, (float *)model, nx, ny, gain, threshold,
                       niter, st, part, s);
    if (e != hipSuccess) return e;
    HogbomState h;
    e = hipMemcpyAsync(&h, st, sizeof h, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e == hipSuccess) *iters = h.iter;
    return e;
}

}  // namespace lr
