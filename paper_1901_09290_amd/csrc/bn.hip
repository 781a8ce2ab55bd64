// Feature (batch) normalisation over the N*H*W pixels of an NHWC bf16 tensor, training mode: forward and
// backward (Sec. 2.1 of the paper: the bandwidth-bound layers next to the convolutions; after a
// reconfiguration their cost scales with the compacted channel count).
//
// Both directions are two streaming passes: per-channel sums over all pixels (a column reduction: every
// thread keeps 8 consecutive channels = one 16-byte vector in registers for all the pixel rows it visits,
// workgroups own contiguous pixel ranges, partial sums go to a workspace and are combined in fp64 in a fixed
// order), then an element-wise pass with the per-channel constants in registers.  Sums are taken about a
// per-channel pivot (the first pixel) so that variance = E[d^2] - E[d]^2 does not cancel for channels whose
// mean is large against their spread.  No atomics: results are run-to-run identical.
//
// Algorithmic bytes per element: forward 2+2 read, 2 written; backward 4+4 read, 2 written.
#include "common.h"

namespace pt {

constexpr int kBnThreads = 256;
constexpr int kBnMaxC = 2048;      // 256 lanes x 8 channels
// A workgroup costs these streaming passes its constants, a reduction of its threads' sums and a row of partials, so
// there are few of them, and loads in flight come from unrolling instead: one workgroup a CU with eight rows a thread for
// the sums, two to four a CU with four rows a thread for the element-wise pass.  Forward and backward, against 1024 and
// 2048 workgroups with one row in flight: 200704 x 256 195 -> 147 us (820 MB moved: 5.6 TB/s), 12544 x 1024 115 -> 56 us,
// 12544 x 371 78 -> 36 us, 3136 x 115 26 -> 21 us.
constexpr int kBnMaxBlocks = 256;  // pixel ranges of the reduction passes
constexpr int kBnSumRows = 8;      // rows whose loads a thread of the reduction passes has in flight
constexpr int kBnApplyRows = 4;    // ... of the element-wise passes

struct BnGeom {
    int64_t pixels;
    int C, cv, ty;           // cv: 8-channel vectors per row = lanes across channels; ty rows in flight
    int nblocks, rows_per_block;
};

inline BnGeom bn_geom(int64_t pixels, int C) {
    BnGeom g;
    g.pixels = pixels;
    g.C = C;
    g.cv = (C + 7) / 8;
    g.ty = kBnThreads / g.cv;
    // at least 8 passes of ty rows per workgroup, at most kBnMaxBlocks workgroups
    int64_t rpb = (int64_t)g.ty * 8;
    if (ceil_div(pixels, rpb) > kBnMaxBlocks) rpb = round_up(ceil_div(pixels, kBnMaxBlocks), g.ty);
    g.rows_per_block = (int)rpb;
    g.nblocks = (int)ceil_div(pixels, rpb);
    return g;
}

// Workgroups of the element-wise passes: 512 (two a CU) until every thread has 16 rows, then as many as leave it 16, at most
// 1024.  12544 x 1024 forward and backward: 114 us with 2048 workgroups, 58 with 1024, 56 with 512; 200704 x 256: 157 us
// with 512, 147 with 1024, 173 with 2048.
inline unsigned bn_apply_blocks(const BnGeom& g) {
    const int64_t passes = ceil_div(g.pixels, g.ty);
    int64_t n = passes / 16;
    n = n < 512 ? 512 : n > 1024 ? 1024 : n;
    return (unsigned)(passes < n ? passes : n);
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void unpack8(const uint4& v, float (&f)[8]) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f[2 * i] = __uint_as_float(w[i] << 16);
        f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
}

__device__ __forceinline__ float half_of(const uint4& v, int e) {
    const uint32_t w = e < 2 ? v.x : e < 4 ? v.y : e < 6 ? v.z : v.w;
    return __uint_as_float(e & 1 ? w & 0xffff0000u : w << 16);
}

// MODE 0: a = sum (x - pivot), b = sum (x - pivot)^2.   MODE 1: a = sum dy, b = sum dy * xhat.
// partial layout: [2][nblocks][C].
template <int MODE>
__global__ __launch_bounds__(kBnThreads) void k_bn_sums(const uint16_t* __restrict__ x, int xpitch,
                                                        const uint16_t* __restrict__ dy, int dypitch, BnGeom g,
                                                        const float* __restrict__ mean, const float* __restrict__ invstd,
                                                        float* __restrict__ partial) {
    __shared__ float red[2][kBnThreads * 8];
    const int tid = threadIdx.x;
    const int ty = tid / g.cv, tx = tid - ty * g.cv;
    const bool live = ty < g.ty;
    float c0[8], c1[8];  // MODE 0: pivot, unused.  MODE 1: mean, invstd
#pragma unroll
    for (int e = 0; e < 8; ++e) c0[e] = 0.f, c1[e] = 0.f;
    if (live) {
        if (MODE == 0) {
            unpack8(*reinterpret_cast<const uint4*>(x + tx * 8), c0);  // pixel 0 of every channel
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int c = tx * 8 + e;
                c0[e] = c < g.C ? mean[c] : 0.f;
                c1[e] = c < g.C ? invstd[c] : 0.f;
            }
        }
    }
    // Neither sum is one chain of additions over a thread's rows.  a: a batch is summed by itself, in two chains of four, and then
    // added, which is no instruction more.  b: four running sums, for the rows 0 and 4, 1 and 5, ... of the batches, so that
    // every product stays part of an FMA.  Relative error of invstd for 200704 x 256 (98 rows a thread): 3.0e-7 row by row,
    // 4.0e-8 this way, as with 1024 ranges; forward and backward 137.8 and 138.3 us (3136 x 115: 20.1 and 20.3).
    float a[8], b[4][8];
#pragma unroll
    for (int e = 0; e < 8; ++e) a[e] = b[0][e] = b[1][e] = b[2][e] = b[3][e] = 0.f;
    const int64_t r0 = (int64_t)blockIdx.x * g.rows_per_block;
    const int64_t r1 = min(g.pixels, r0 + g.rows_per_block);
    if (live) {
        // element e of a row: f0 is a term of a, f0 * f1 one of b
        auto factors = [&](const uint4& xq, const uint4& gq, int e, float& f0, float& f1) {
            const float d = half_of(xq, e) - c0[e];
            f0 = MODE == 0 ? d : half_of(gq, e);
            f1 = MODE == 0 ? d : d * c1[e];
        };
        const uint16_t* px = x + (r0 + ty) * xpitch + tx * 8;
        const uint16_t* pg = MODE == 1 ? dy + (r0 + ty) * dypitch + tx * 8 : nullptr;
        const int64_t sx = (int64_t)g.ty * xpitch, sg = (int64_t)g.ty * dypitch;
        int n = (int)((r1 - r0 - ty + g.ty - 1) / g.ty);  // rows of this thread (<= 0: none)
        for (; n >= kBnSumRows; n -= kBnSumRows) {
            uint4 xq[kBnSumRows], gq[kBnSumRows];
#pragma unroll
            for (int u = 0; u < kBnSumRows; ++u) {
                xq[u] = *reinterpret_cast<const uint4*>(px + u * sx);
                if (MODE == 1) gq[u] = *reinterpret_cast<const uint4*>(pg + u * sg);
            }
            px += kBnSumRows * sx;
            if (MODE == 1) pg += kBnSumRows * sg;
            float ta[2][8];
#pragma unroll
            for (int u = 0; u < kBnSumRows; ++u) {  // (row by row: the first ones while the last are still on their way)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    float f0, f1;
                    factors(xq[u], MODE == 1 ? gq[u] : xq[u], e, f0, f1);
                    ta[u / 4][e] = u % 4 ? ta[u / 4][e] + f0 : f0;
                    b[u % 4][e] += f0 * f1;
                }
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) a[e] += ta[0][e] + ta[1][e];
        }
        if (n > 0) {  // the rows left over, summed by themselves as well
            float ra[8], rb[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) ra[e] = 0.f, rb[e] = 0.f;
            for (; n > 0; --n) {
                const uint4 xq = *reinterpret_cast<const uint4*>(px);
                const uint4 gq = MODE == 1 ? *reinterpret_cast<const uint4*>(pg) : xq;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    float f0, f1;
                    factors(xq, gq, e, f0, f1);
                    ra[e] += f0;
                    rb[e] += f0 * f1;
                }
                px += sx;
                if (MODE == 1) pg += sg;
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                a[e] += ra[e];
                b[0][e] += rb[e];
            }
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        red[0][tid * 8 + e] = a[e];
        red[1][tid * 8 + e] = (b[0][e] + b[1][e]) + (b[2][e] + b[3][e]);
    }
    __syncthreads();
    // row groups added in a fixed order (many of them in four chains): thread f owns channel f
    const int row = g.cv * 8;
    for (int f = tid; f < g.C; f += kBnThreads) {
        float s0 = 0.f, s1 = 0.f;
        int y = 0;
        if (g.ty >= 8) {
            float t0[4] = {0.f, 0.f, 0.f, 0.f}, t1[4] = {0.f, 0.f, 0.f, 0.f};
            for (; y + 4 <= g.ty; y += 4) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    t0[u] += red[0][(y + u) * row + f];
                    t1[u] += red[1][(y + u) * row + f];
                }
            }
            s0 = (t0[0] + t0[1]) + (t0[2] + t0[3]);
            s1 = (t1[0] + t1[1]) + (t1[2] + t1[3]);
        }
        for (; y < g.ty; ++y) {
            s0 += red[0][y * row + f];
            s1 += red[1][y * row + f];
        }
        partial[(size_t)blockIdx.x * g.C + f] = s0;
        partial[((size_t)g.nblocks + blockIdx.x) * g.C + f] = s1;
    }
}

// 8 channels per workgroup, kBnSlices threads per channel: each thread adds every kBnSlices-th workgroup partial in fp64
// in ascending order (loads issued 4 at a time), the slices are then added in a fixed order, so results are run-to-run
// identical.  Bound by the latency of the partials: with 32 slices (two rounds of loads, 32 dependent LDS reads) 6.4 us
// for 1024 partials of 256 channels.   MODE 0 -> mean, invstd.  MODE 1 -> dbeta (= a), dgamma (= b).
constexpr int kBnSlices = 128;
template <int MODE>
__global__ __launch_bounds__(8 * kBnSlices) void k_bn_finish(const float* __restrict__ partial, const uint16_t* __restrict__ x,
                                                             BnGeom g, float eps, float* __restrict__ out0,
                                                             float* __restrict__ out1) {
    __shared__ double red[2][kBnSlices / 8][8];
    const int cx = threadIdx.x & 7, sl = threadIdx.x >> 3;
    const int c = blockIdx.x * 8 + cx;
    double s0 = 0.0, s1 = 0.0;
    if (c < g.C) {
        const float* pa = partial + c;
        const float* pb = partial + (size_t)g.nblocks * g.C + c;
        for (int b = sl; b < g.nblocks; b += kBnSlices * 4) {
            float va[4], vb[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                // unconditional loads from a clamped row (so that all 8 are in flight together), masked after
                const size_t row = (size_t)min(b + kBnSlices * u, g.nblocks - 1) * g.C;
                va[u] = pa[row];
                vb[u] = pb[row];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (b + kBnSlices * u >= g.nblocks) va[u] = 0.f, vb[u] = 0.f;
                s0 += (double)va[u];
                s1 += (double)vb[u];
            }
        }
    }
    // the 8 slices of a wave first, lane by lane, then the waves' sums
#pragma unroll
    for (int d = 8; d < 64; d <<= 1) {
        s0 += __shfl_xor(s0, d, 64);
        s1 += __shfl_xor(s1, d, 64);
    }
    if ((sl & 7) == 0) {
        red[0][sl >> 3][cx] = s0;
        red[1][sl >> 3][cx] = s1;
    }
    __syncthreads();
    if (sl != 0 || c >= g.C) return;
    s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int i = 0; i < kBnSlices / 8; ++i) {
        s0 += red[0][i][cx];
        s1 += red[1][i][cx];
    }
    if (MODE == 0) {
        const double pivot = x ? (double)__uint_as_float((uint32_t)x[c] << 16) : 0.0;  // no x: plain sums
        const double m = s0 / (double)g.pixels;           // mean of (x - pivot)
        double var = s1 / (double)g.pixels - m * m;       // biased variance
        if (var < 0.0) var = 0.0;
        out0[c] = (float)(pivot + m);
        out1[c] = (float)(1.0 / sqrt(var + (double)eps));
    } else {
        out0[c] = (float)s0;
        out1[c] = (float)s1;
    }
}

// MODE 0: y = (x - mean) * (gamma * invstd) + beta.
// MODE 1: dx = (gamma * invstd) * (dy - dbeta/M - xhat * dgamma/M).
template <int MODE>
__global__ __launch_bounds__(kBnThreads) void k_bn_apply(const uint16_t* __restrict__ x, int xpitch,
                                                         const uint16_t* __restrict__ dy, int dypitch, BnGeom g,
                                                         const float* __restrict__ mean, const float* __restrict__ invstd,
                                                         const float* __restrict__ p0, const float* __restrict__ p1,
                                                         const float* __restrict__ gamma, uint16_t* __restrict__ out,
                                                         int opitch) {
    const int tid = threadIdx.x;
    const int ty = tid / g.cv, tx = tid - ty * g.cv;
    if (ty >= g.ty) return;
    float mu[8], sc[8], k0[8], k1[8];  // MODE 0: k0 = beta.  MODE 1: k0 = dbeta/M, k1 = invstd * dgamma/M
    const float invM = 1.0f / (float)g.pixels;
    float ga[8], is[8], q0[8], q1[8];
    const int c0 = tx * 8;
    if (c0 + 8 <= g.C) {  // contiguous: wide loads
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            mu[e] = mean[c0 + e], is[e] = invstd[c0 + e], ga[e] = gamma[c0 + e], q0[e] = p0[c0 + e];
            q1[e] = MODE == 1 ? p1[c0 + e] : 0.f;
        }
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int c = min(c0 + e, g.C - 1);
            mu[e] = mean[c], is[e] = invstd[c], ga[e] = gamma[c], q0[e] = p0[c], q1[e] = MODE == 1 ? p1[c] : 0.f;
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        sc[e] = ga[e] * is[e];
        k0[e] = MODE == 0 ? q0[e] : q0[e] * invM;
        k1[e] = MODE == 0 ? 0.f : is[e] * (q1[e] * invM);
    }
    // Padding channels of the last vector go out as zero: whole rows are written, never partial ones (a hole in
    // every row costs the memory system a merge of partial lines and halves the store rate).
    const int nlast = g.C - tx * 8;  // valid channels of this thread's vector (>= 8: all)
    auto halves = [&](int k) { return (k < nlast ? 0xFFFFu : 0u) | (k + 1 < nlast ? 0xFFFF0000u : 0u); };
    const uint32_t m0 = halves(0), m1 = halves(2), m2 = halves(4), m3 = halves(6);
    const int64_t stride = (int64_t)gridDim.x * g.ty;
    // last pixels first: the reduction pass before this one ended there, so they are the likeliest to still sit
    // in the chip's caches
    auto one = [&](const uint4& xq, const uint4& gq, uint16_t* dst) {
        float xv[8], o[8];
        unpack8(xq, xv);
        if (MODE == 0) {
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = (xv[e] - mu[e]) * sc[e] + k0[e];
        } else {
            float gv[8];
            unpack8(gq, gv);
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = sc[e] * (gv[e] - k0[e] - (xv[e] - mu[e]) * k1[e]);
        }
        u32x4 pk;
        pk.x = cvt_pk_bf16(o[0], o[1]) & m0;
        pk.y = cvt_pk_bf16(o[2], o[3]) & m1;
        pk.z = cvt_pk_bf16(o[4], o[5]) & m2;
        pk.w = cvt_pk_bf16(o[6], o[7]) & m3;
        // not kept in the caches: they hold the rows still to be read again (200704 x 256 forward: 82 -> 67 us)
        __builtin_nontemporal_store(pk, reinterpret_cast<u32x4*>(dst));
    };
    int64_t r = g.pixels - 1 - ((int64_t)blockIdx.x * g.ty + ty);
    for (; r - (kBnApplyRows - 1) * stride >= 0; r -= kBnApplyRows * stride) {
        uint4 xq[kBnApplyRows], gq[kBnApplyRows];
#pragma unroll
        for (int u = 0; u < kBnApplyRows; ++u) {
            xq[u] = *reinterpret_cast<const uint4*>(x + (r - u * stride) * xpitch + tx * 8);
            if (MODE == 1) gq[u] = *reinterpret_cast<const uint4*>(dy + (r - u * stride) * dypitch + tx * 8);
        }
#pragma unroll
        for (int u = 0; u < kBnApplyRows; ++u) one(xq[u], MODE == 1 ? gq[u] : xq[u], out + (r - u * stride) * opitch + tx * 8);
    }
    for (; r >= 0; r -= stride) {
        const uint4 xq = *reinterpret_cast<const uint4*>(x + r * xpitch + tx * 8);
        const uint4 gq = MODE == 1 ? *reinterpret_cast<const uint4*>(dy + r * dypitch + tx * 8) : xq;
        one(xq, gq, out + r * opitch + tx * 8);
    }
}

}  // namespace pt

using namespace pt;

static int32_t bn_check(int64_t pixels, int32_t C, int32_t p0, int32_t p1, int32_t p2) {
    if (pixels <= 0 || C <= 0 || p0 < C || p1 < C || p2 < C) return PT_ERR_SHAPE;
    if (C > kBnMaxC || pixels > 0x7fffffff) return PT_ERR_UNSUPPORTED;
    if (p0 % 8 || p1 % 8 || p2 % 8) return PT_ERR_UNSUPPORTED;  // 16-byte rows only
    return PT_OK;
}
static bool al16(const void* p) { return ((uintptr_t)p & 15) == 0; }

extern "C" int32_t pt_bn_workspace_bytes(int64_t pixels, int32_t C, size_t* bytes) {
    if (!bytes) return PT_ERR_NULL;
    const int32_t rc = bn_check(pixels, C, (C + 7) & ~7, (C + 7) & ~7, (C + 7) & ~7);
    if (rc != PT_OK) return rc;
    const BnGeom g = bn_geom(pixels, C);
    *bytes = (size_t)round_up((int64_t)2 * g.nblocks * C * 4, 256);
    return PT_OK;
}

extern "C" int32_t pt_bn_fwd(const uint16_t* x, int64_t pixels, int32_t C, int32_t x_cpitch, const float* gamma,
                             const float* beta, float eps, uint16_t* y, int32_t y_cpitch, float* mean, float* invstd,
                             void* ws, size_t ws_bytes, void* stream) {
    int32_t rc = bn_check(pixels, C, x_cpitch, y_cpitch, x_cpitch);
    if (rc != PT_OK) return rc;
    if (!(eps >= 0.f)) return PT_ERR_SHAPE;
    if (!x || !gamma || !beta || !y || !mean || !invstd || !ws) return PT_ERR_NULL;
    if (!al16(x) || !al16(y) || !al16(ws)) return PT_ERR_UNSUPPORTED;
    const BnGeom g = bn_geom(pixels, C);
    if (ws_bytes < (size_t)2 * g.nblocks * C * 4) return PT_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    float* part = (float*)ws;
    hipLaunchKernelGGL(k_bn_sums<0>, dim3(g.nblocks), dim3(kBnThreads), 0, st, x, x_cpitch, (const uint16_t*)nullptr, 0, g,
                       (const float*)nullptr, (const float*)nullptr, part);
    rc = launch_status();
    if (rc != PT_OK) return rc;
    hipLaunchKernelGGL(k_bn_finish<0>, dim3((unsigned)ceil_div(C, 8)), dim3(8 * kBnSlices), 0, st, part, x, g, eps, mean, invstd);
    rc = launch_status();
    if (rc != PT_OK) return rc;
    const unsigned grid = bn_apply_blocks(g);
    hipLaunchKernelGGL(k_bn_apply<0>, dim3(grid), dim3(kBnThreads), 0, st, x, x_cpitch, (const uint16_t*)nullptr, 0, g, mean,
                       invstd, beta, (const float*)nullptr, gamma, y, y_cpitch);
    return launch_status();
}

extern "C" int32_t pt_bn_bwd(const uint16_t* x, const uint16_t* dy, int64_t pixels, int32_t C, int32_t x_cpitch,
                             int32_t dy_cpitch, const float* gamma, const float* mean, const float* invstd, uint16_t* dx,
                             int32_t dx_cpitch, float* dgamma, float* dbeta, void* ws, size_t ws_bytes, void* stream) {
    int32_t rc = bn_check(pixels, C, x_cpitch, dy_cpitch, dx_cpitch);
    if (rc != PT_OK) return rc;
    if (!x || !dy || !gamma || !mean || !invstd || !dx || !dgamma || !dbeta || !ws) return PT_ERR_NULL;
    if (!al16(x) || !al16(dy) || !al16(dx) || !al16(ws)) return PT_ERR_UNSUPPORTED;
    const BnGeom g = bn_geom(pixels, C);
    if (ws_bytes < (size_t)2 * g.nblocks * C * 4) return PT_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    float* part = (float*)ws;
    hipLaunchKernelGGL(k_bn_sums<1>, dim3(g.nblocks), dim3(kBnThreads), 0, st, x, x_cpitch, dy, dy_cpitch, g, mean, invstd,
                       part);
    rc = launch_status();
    if (rc != PT_OK) return rc;
    hipLaunchKernelGGL(k_bn_finish<1>, dim3((unsigned)ceil_div(C, 8)), dim3(8 * kBnSlices), 0, st, part, x, g, 0.f, dbeta, dgamma);
    rc = launch_status();
    if (rc != PT_OK) return rc;
    const unsigned grid = bn_apply_blocks(g);
    hipLaunchKernelGGL(k_bn_apply<1>, dim3(grid), dim3(kBnThreads), 0, st, x, x_cpitch, dy, dy_cpitch, g, mean, invstd, dbeta,
                       dgamma, gamma, dx, dx_cpitch);
    return launch_status();
}

// Normalisation whose statistics pass was done by the producing convolution (pt_conv_fwd_stats): finish + apply.
extern "C" int32_t pt_bn_fwd_from_sums(const uint16_t* x, int64_t pixels, int32_t C, int32_t x_cpitch, const float* sums,
                                       int32_t n_partial, const float* gamma, const float* beta, float eps, uint16_t* y,
                                       int32_t y_cpitch, float* mean, float* invstd, void* stream) {
    int32_t rc = bn_check(pixels, C, x_cpitch, y_cpitch, x_cpitch);
    if (rc != PT_OK) return rc;
    if (!(eps >= 0.f) || n_partial <= 0) return PT_ERR_SHAPE;
    if (!x || !sums || !gamma || !beta || !y || !mean || !invstd) return PT_ERR_NULL;
    if (!al16(x) || !al16(y)) return PT_ERR_UNSUPPORTED;
    BnGeom g = bn_geom(pixels, C);
    g.nblocks = n_partial;  // rows of `sums` per statistic
    hipStream_t st = (hipStream_t)stream;
    hipLaunchKernelGGL(k_bn_finish<0>, dim3((unsigned)ceil_div(C, 8)), dim3(8 * kBnSlices), 0, st, sums, (const uint16_t*)nullptr, g,
                       eps, mean, invstd);
    rc = launch_status();
    if (rc != PT_OK) return rc;
    const unsigned grid = bn_apply_blocks(g);
    hipLaunchKernelGGL(k_bn_apply<0>, dim3(grid), dim3(kBnThreads), 0, st, x, x_cpitch, (const uint16_t*)nullptr, 0, g, mean,
                       invstd, beta, (const float*)nullptr, gamma, y, y_cpitch);
    return launch_status();
}
