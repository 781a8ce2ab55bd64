// Implicit-GEMM convolution kernels for gfx950: forward, input gradient, weight gradient
// (Sec. 2.1, Alg. 1 ForwardProp/BackProp, Eq. 4).  bf16 operands, fp32 accumulation on the
// 32x32x16 bf16 MFMA, NHWC activations, KRSC weights.
//
// forward / input gradient share one kernel (k_igemm): output pixels x output channels, reduced over
// (filter tap, reduction channel).  Both operands are contiguous along the reduction channel, which
// is what the MFMA wants per lane (8 consecutive k), so 16-byte global loads go to LDS unchanged.
//   forward:        A = x gathered at (p*stride - pad + r, q*stride - pad + s),  B = w[k][r][s][c]
//   input gradient: per stride-parity class of input pixels (dense sub-problem with only the taps
//                   that can reach that class), A = dy gathered at (h' + off - jr, w' + off - js),
//                   B = w transposed to [c][r][s][k] in the workspace.
// The MFMA "row" operand is the weight tile and the "column" operand the pixel tile, so each lane's
// four consecutive accumulator rows are four consecutive output channels of one pixel (one 8-byte
// store of bf16).
//
// weight gradient (k_wgrad): output (tap, c) x k, reduced over output pixels.  Memory is contiguous
// along channels, not along the reduction axis, so tiles are stored pixel-major in LDS exactly as
// loaded and read back with the LDS transpose read (ds_read_b64_tr_b16), which hands every lane four
// consecutive reduction elements of one channel.  The pixel range is split over workgroups; partial
// sums go to an fp32 workspace and are combined in a fixed order by k_wgrad_reduce.
//
// Ragged channel counts: the reduction axis is laid out as taps x (C rounded up to 8), so a ragged C
// costs one partially filled 8-vector per tap; lanes beyond C are masked to zero on load.  32-wide
// accumulator blocks that lie wholly outside the logical output are skipped.
#include <algorithm>
#include <exception>
#include <vector>

#include "conv_kernels.h"
#include "norms.h"

namespace pt {

// w[K][RS][wpitch] -> wt[C][RS][kpitch]  (bf16), for the input-gradient GEMM.  A workgroup takes 64 filters x 64 channels of
// one tap: whole 128-byte lines in and out, 16 bytes a lane, through LDS rows of 33 dwords.  Bound by HBM and by the launch:
// the copies of ResNet-50 (47 MB in, 47 MB out) 46.7 us as 32 x 32 tiles with two bytes a lane, 20.3 so; pruned 22.3 and 13.
constexpr int kTrTile = 64, kTrPitch = 66;
__device__ __forceinline__ void transpose_tile(const uint16_t* __restrict__ w, uint16_t* __restrict__ wt, int K, int RS, int C,
                                               int wpitch, int kpitch, int k0, int c0, int rs, uint16_t* tile) {
    const bool vec_in = wpitch % 8 == 0 && ((uintptr_t)w & 15) == 0, vec_out = ((uintptr_t)wt & 15) == 0;  // uniform
    const int row = threadIdx.x >> 3, at = (threadIdx.x & 7) * 8;
    uint16_t v[2][8];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int k = k0 + row + 32 * i, c = c0 + at;
        uint4 q = make_uint4(0u, 0u, 0u, 0u);
        if (k < K && c < C) {
            const uint16_t* src = w + ((int64_t)k * RS + rs) * wpitch + c;
            if (vec_in && c + 8 <= C) {
                q = *reinterpret_cast<const uint4*>(src);
            } else {
                uint32_t h[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) h[e] = c + e < C ? src[e] : 0u;
                q = make_uint4(h[0] | h[1] << 16, h[2] | h[3] << 16, h[4] | h[5] << 16, h[6] | h[7] << 16);
            }
        }
        const uint32_t d[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) v[i][e] = (uint16_t)(d[e >> 1] >> (16 * (e & 1)));
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) tile[(at + e) * kTrPitch + row + 32 * i] = v[i][e];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int cl = row + 32 * i, c = c0 + cl, k = k0 + at;
        if (c >= C || k >= kpitch) continue;  // (kpitch is a multiple of 8)
        const uint32_t* src = reinterpret_cast<const uint32_t*>(tile + cl * kTrPitch + at);
        const uint4 q = make_uint4(src[0], src[1], src[2], src[3]);
        uint16_t* dst = wt + ((int64_t)c * RS + rs) * kpitch + k;
        if (vec_out) {
            *reinterpret_cast<uint4*>(dst) = q;
        } else {
            const uint32_t d[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) dst[e] = (uint16_t)(d[e >> 1] >> (16 * (e & 1)));
        }
    }
}
__global__ __launch_bounds__(256) void k_transpose_w(const uint16_t* __restrict__ w, int K, int RS, int C, int wpitch,
                                                     uint16_t* __restrict__ wt, int kpitch) {
    __shared__ __attribute__((aligned(16))) uint16_t tile[kTrTile * kTrPitch];
    transpose_tile(w, wt, K, RS, C, wpitch, kpitch, blockIdx.y * kTrTile, blockIdx.x * kTrTile, blockIdx.z, tile);
}

// The same transposition for many layers in one launch (descriptors in the kernel arguments).
constexpr int kMaxTransposeJobs = 64;
struct TransposeJob {
    const uint16_t* w;
    uint16_t* wt;
    int K, RS, C, wpitch, kpitch, nbx, nby, pad;
};
struct TransposeJobs {
    TransposeJob j[kMaxTransposeJobs];
    int first[kMaxTransposeJobs];  // first workgroup of each job
    int n;
};
__global__ __launch_bounds__(256) void k_transpose_w_multi(const TransposeJobs jobs) {
    __shared__ __attribute__((aligned(16))) uint16_t tile[kTrTile * kTrPitch];
    const int ji = job_of_block(jobs.first, blockIdx.x);
    const TransposeJob jb = jobs.j[ji];
    int b = blockIdx.x - jobs.first[ji];
    const int bx = b % jb.nbx;
    b /= jb.nbx;
    const int by = b % jb.nby, rs = b / jb.nby;
    transpose_tile(jb.w, jb.wt, jb.K, jb.RS, jb.C, jb.wpitch, jb.kpitch, by * kTrTile, bx * kTrTile, rs, tile);
}

// Zero the destination pixels of a stride-parity class that no output pixel reaches.  One thread clears
// 8 channels (one 16-byte store when the rows are 16-byte aligned).
__global__ void k_zero_class(uint16_t* __restrict__ D, int64_t pixels, int gH, int gW, int DH, int DW, int d_hmul,
                             int d_hadd, int d_wmul, int d_wadd, int dpitch, int Nout, int vec16) {
    const int cv = (Nout + 7) >> 3;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= pixels * cv) return;
    const int64_t m = t / cv;
    const int ch = (int)(t - m * cv) * 8;
    const int gHW = gH * gW;
    const int64_t n = m / gHW;
    const int rem = (int)(m - n * gHW);
    const int gi = rem / gW, gj = rem - gi * gW;
    uint16_t* dst = D + ((n * DH + gi * d_hmul + d_hadd) * DW + gj * d_wmul + d_wadd) * dpitch + ch;
    if (vec16 && ch + 7 < Nout) {
        *reinterpret_cast<uint4*>(dst) = make_uint4(0u, 0u, 0u, 0u);
    } else {
        for (int e = 0; e < 8; ++e)
            if (ch + e < Nout) dst[e] = 0;
    }
}

// dw[k][tap][c] = sum over splits of partial[split][k][tap*CP + c], in a fixed order, for every split layer of a weight
// gradient launch.  Two forms, chosen per layer:
//   deep: many splits over few outputs.  A workgroup owns 64 consecutive outputs; wavefront v adds the splits v, v+8,
//         v+16, ... (eight loads in flight), and the eight wavefront sums are added in ascending order.
//   wide: few splits over many outputs.  Four consecutive outputs of the slab per thread (16-byte loads); one, two or four
//         wavefronts share 256 outputs and take every first, second or fourth split, at most four loads each and all in
//         flight at once, and their sums are added in ascending order.  CP is a multiple of 8: the four outputs share a
//         filter tap.  Bound by the partial sums' way from memory (14 splits of 256 x 1024 outputs: 14.7 MB in 5.0 us, two of
//         them the launch); against one thread adding all splits the 53 layers of a ResNet-50 gain 1 %.
// Results do not depend on timing.  With `lw` the gradient of the group-lasso penalty (Eq. 1-2) is added on the way out,
// with the arithmetic of k_group_lasso_grad: dw = sum + lambda * (w * (1/out_norm[k] + 1/in_norm[c])), a zero norm
// contributing 0.
constexpr int kReduceWaves = 8;
constexpr int kReduceWideLoads = 4, kReduceWideMaxSplits = 16;
constexpr int64_t kReduceWideMinOutputs = 64 * 1024;
struct ReduceLasso {
    const float* w;         // [K][RS][wpitch], the pitch of dw; nullptr: no regulariser
    const float* out_norm;  // [K], nullptr: output groups not regularised
    const float* in_norm;   // [C], nullptr: input groups not regularised
    float lambda;
};
struct ReduceJob {
    const float* part;
    float* dw;
    ReduceLasso rl;
    int splits, K, RS, C, CP, wpitch, o_vec;
    int wide;  // 0: deep form, else wavefronts per 256 outputs of the wide form (1, 2 or 4)
};
struct ReduceJobs {
    ReduceJob j[kWgMaxProblems];
    int first[64];
};
__device__ __forceinline__ float inv_norm(const float* n, int i) {
    const float v = n ? n[i] : 0.f;
    return v > 0.f ? 1.0f / v : 0.f;
}
// Where output t of the slab goes: filter k, tap tp, channel c.  (A division of 64-bit numbers is some hundred
// instructions: only for slabs that need it.)
struct ReduceIndex {
    int k, tp, c;
};
__device__ __forceinline__ ReduceIndex reduce_index(const ReduceJob& J, int Mtot, int64_t total, int64_t t) {
    ReduceIndex r;
    r.k = total <= 0xffffffffll ? (int)((uint32_t)t / (uint32_t)Mtot) : (int)(t / Mtot);
    const uint32_t mrow = (uint32_t)(t - (int64_t)r.k * Mtot);
    r.tp = J.RS == 1 ? 0 : (int)(mrow / (uint32_t)J.CP);
    r.c = (int)mrow - r.tp * J.CP;
    return r;
}
// Sum of part[i * total] over i = first, first + step, ... < n: kReduceLoads loads in flight, those past the end repeated
// from the last valid slab and left out (a loop of single loads for the remainder costs a round trip to memory each).
constexpr int kReduceLoads = 8;
__device__ __forceinline__ float sum_slabs(const float* __restrict__ part, int64_t total, int first, int step, int n) {
    float s[4] = {0.f, 0.f, 0.f, 0.f};
    for (int i = first; i < n; i += kReduceLoads * step) {
        float v[kReduceLoads];
#pragma unroll
        for (int u = 0; u < kReduceLoads; ++u) v[u] = part[(int64_t)min(i + u * step, n - 1) * total];
#pragma unroll
        for (int u = 0; u < kReduceLoads; ++u) s[u & 3] += i + u * step < n ? v[u] : 0.f;
    }
    return (s[0] + s[1]) + (s[2] + s[3]);
}
__device__ __forceinline__ void wgrad_reduce_deep(const ReduceJob& J, int block, float (*red)[64]) {
    const int Mtot = J.RS * J.CP;
    const int64_t total = (int64_t)J.K * Mtot;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t t = (int64_t)block * 64 + lane;
    red[wave][lane] = t < total ? sum_slabs(J.part + t, total, wave, kReduceWaves, J.splits) : 0.f;
    __syncthreads();
    if (wave == 0 && t < total) {
        float s = 0.f;
#pragma unroll
        for (int v = 0; v < kReduceWaves; ++v) s += red[v][lane];
        const ReduceIndex r = reduce_index(J, Mtot, total, t);
        if (r.c < J.C) {
            const int64_t o = ((int64_t)r.k * J.RS + r.tp) * J.wpitch + r.c;
            if (J.rl.w) s += J.rl.lambda * (J.rl.w[o] * (inv_norm(J.rl.out_norm, r.k) + inv_norm(J.rl.in_norm, r.c)));
            J.dw[o] = s;
        }
    }
}
__device__ __forceinline__ void wgrad_reduce_wide(const ReduceJob& J, int block, float (*red)[256]) {
    const int Mtot = J.RS * J.CP, groups = J.wide;
    const int64_t total = (int64_t)J.K * Mtot;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    const int g = wave & (groups - 1), sub = wave / groups;
    const int64_t t = ((int64_t)block * (waves / groups) + sub) * 256 + lane * 4;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    if (t < total) {
        float4 v[kReduceWideLoads];
#pragma unroll
        for (int u = 0; u < kReduceWideLoads; ++u)
            if (g + u * groups < J.splits) v[u] = *reinterpret_cast<const float4*>(J.part + (int64_t)(g + u * groups) * total + t);
#pragma unroll
        for (int u = 0; u < kReduceWideLoads; ++u)
            if (g + u * groups < J.splits) s.x += v[u].x, s.y += v[u].y, s.z += v[u].z, s.w += v[u].w;
    }
    if (groups > 1) {  // uniform
        float (*mine)[256] = red + sub * (groups - 1) - 1;
        if (g > 0) *reinterpret_cast<float4*>(&mine[g][lane * 4]) = s;
        __syncthreads();
        if (g > 0) return;
        for (int o = 1; o < groups; ++o) {
            const float4 r = *reinterpret_cast<const float4*>(&mine[o][lane * 4]);
            s.x += r.x; s.y += r.y; s.z += r.z; s.w += r.w;
        }
    }
    if (t >= total) return;
    const ReduceIndex ix = reduce_index(J, Mtot, total, t);
    const int k = ix.k, tp = ix.tp, c = ix.c;
    if (c >= J.C) return;
    const int64_t o = ((int64_t)k * J.RS + tp) * J.wpitch + c;
    float v[4] = {s.x, s.y, s.z, s.w};
    if (J.rl.w) {
        const float inv_out = inv_norm(J.rl.out_norm, k);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (c + e < J.C) v[e] += J.rl.lambda * (J.rl.w[o + e] * (inv_out + inv_norm(J.rl.in_norm, c + e)));
    }
    if (J.o_vec && c + 3 < J.C) {
        *reinterpret_cast<float4*>(J.dw + o) = make_float4(v[0], v[1], v[2], v[3]);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (c + e < J.C) J.dw[o + e] = v[e];
    }
}
__global__ __launch_bounds__(64 * kReduceWaves) void k_wgrad_reduce(const ReduceJob J) {
    extern __shared__ __attribute__((aligned(16))) float reduce_lds[];
    if (J.wide) wgrad_reduce_wide(J, blockIdx.x, reinterpret_cast<float (*)[256]>(reduce_lds));
    else wgrad_reduce_deep(J, blockIdx.x, reinterpret_cast<float (*)[64]>(reduce_lds));
}
__global__ __launch_bounds__(64 * kReduceWaves) void k_wgrad_reduce_multi(const ReduceJobs jobs) {
    extern __shared__ __attribute__((aligned(16))) float reduce_lds[];
    const int ji = job_of_block(jobs.first, blockIdx.x);
    const ReduceJob J = jobs.j[ji];
    const int block = blockIdx.x - jobs.first[ji];
    if (J.wide) wgrad_reduce_wide(J, block, reinterpret_cast<float (*)[256]>(reduce_lds));
    else wgrad_reduce_deep(J, block, reinterpret_cast<float (*)[64]>(reduce_lds));
}

// The same for the slabs of k_stem_wgrad, [slab][r][64 output channels][8 taps x 4 channels]: one output per lane, the
// slabs spread over eight wavefronts (eight loads in flight each) and the eight sums added in ascending order.
__global__ __launch_bounds__(64 * kReduceWaves) void k_stem_wgrad_reduce(const float* __restrict__ part, int slabs, int K,
                                                                          int R, int S, int C, int wpitch,
                                                                          float* __restrict__ dw, const ReduceLasso rl) {
    __shared__ float red[kReduceWaves][64];
    const int64_t total = (int64_t)R * kSwSlabRow;  // a multiple of 64
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int t = blockIdx.x * 64 + lane;
    red[wave][lane] = sum_slabs(part + t, total, wave, kReduceWaves, slabs);
    __syncthreads();
    if (wave == 0) {
        float s = 0.f;
#pragma unroll
        for (int v = 0; v < kReduceWaves; ++v) s += red[v][lane];
        const int n = t & 31, k = (t >> 5) & 63, r = t >> 11;
        const int fs = n >> 2, c = n & 3;
        if (k < K && fs < S && c < C) {
            const int64_t o = ((int64_t)(k * R + r) * S + fs) * wpitch + c;
            if (rl.w) s += rl.lambda * (rl.w[o] * (inv_norm(rl.out_norm, k) + inv_norm(rl.in_norm, c)));
            dw[o] = s;
        }
    }
}

}  // namespace pt

#include "conv_host.h"

using namespace pt;

extern "C" int32_t pt_conv_fwd_workspace_bytes(const pt_conv_desc* d, size_t* bytes) {
    if (!bytes) return PT_ERR_NULL;
    int32_t rc = check_desc(d);
    if (rc != PT_OK) return rc;
    *bytes = 0;
    return PT_OK;
}

extern "C" int32_t pt_conv_bwd_data_workspace_bytes(const pt_conv_desc* d, size_t* bytes) {
    if (!bytes) return PT_ERR_NULL;
    int32_t rc = check_desc(d);
    if (rc != PT_OK) return rc;
    *bytes = bwd_data_ws(d);
    return PT_OK;
}

extern "C" int32_t pt_conv_bwd_weight_workspace_bytes(const pt_conv_desc* d, size_t* bytes) {
    if (!bytes) return PT_ERR_NULL;
    int32_t rc = check_desc(d);
    if (rc != PT_OK) return rc;
    *bytes = wgrad_ws(d);
    return PT_OK;
}

static int32_t hip_status(hipError_t e) {
    if (e != hipSuccess) {
        set_hip_error(e);
        return PT_ERR_LAUNCH;
    }
    return launch_status();
}

// image-like first layer (at most 4 channels at a pitch of 8, zero padding vouched for): its own kernel
static bool stem_fwd_ok(const pt_conv_desc* d, const uint16_t* x, const uint16_t* w, const uint16_t* y) {
    return d->C <= 4 && d->x_cpitch == 8 && d->w_cpitch == 8 && (d->flags & PT_CONV_PAD_ZERO) && d->y_cpitch % 8 == 0 &&
           aligned16(x) && aligned16(w) && aligned16(y) && d->stride_h == d->stride_w && d->stride_h <= 2 &&
           d->R <= kStemMaxR && d->S <= 8 && (int64_t)d->H * d->W * 16 <= 0x7fffffff;
}

extern "C" int32_t pt_conv_fwd(const pt_conv_desc* d, const uint16_t* x, const uint16_t* w, uint16_t* y, void* ws,
                               size_t ws_bytes, void* stream) {
    (void)ws;
    (void)ws_bytes;
    int32_t rc = check_desc(d);
    if (rc != PT_OK) return rc;
    if (!x || !w || !y) return PT_ERR_NULL;
    if (stem_fwd_ok(d, x, w, y)) {
        StemArgs s{x, w, y, d->N, d->H, d->W, d->P, d->Q, d->K, d->R, d->S, d->pad_h, d->pad_w, d->y_cpitch, 0, 0, 0, 0};
        return hip_status(launch_stem_fwd(s, d->stride_h, kStemSlots, (hipStream_t)stream));
    }
    if (res3_fwd_ok(d, x, w, y)) {  // early 3 x 3 layer: the filter bank stays in LDS
        const int cinp = (int)round_up(d->C, 8);
        Res3Args r{x, w, y, d->N, d->H, d->W, d->C, cinp, d->x_cpitch, d->K, d->w_cpitch, d->y_cpitch, 0, 0, 0, 0, 0, 0, 0};
        return hip_status(launch_conv3x3_res(r, kRes3Fwd, (hipStream_t)stream));
    }
    IgemmArgs a = make_fwd_args(d, x, w, y);
    const bool vec = d->x_cpitch % 8 == 0 && d->w_cpitch % 8 == 0 && aligned16(x) && aligned16(w);
    return hip_status(launch_igemm(a, vec, (hipStream_t)stream, nullptr, nullptr, fwd_kernel(d, x, w, y)));
}

// Problems of the direct kernel waiting to be sent out together: those that chose the same instantiation share a launch.
struct IgemmPending {
    IgemmArgs a[kIgemmMaxProblems];
    IgemmDlPlan p[kIgemmMaxProblems];
    int n = 0;
    int32_t flush(hipStream_t st) {
        if (n == 0) return PT_OK;
        const int32_t r = hip_status(launch_igemm_dl_planned(a, p, n, st));
        n = 0;
        return r;
    }
    // launches or queues one problem
    int32_t add(IgemmArgs& args, bool vec, hipStream_t st, int kernel = -1, bool alone = false) {
        bool planned = false;
        const int32_t rc = hip_status(launch_igemm(args, vec, st, &p[n], &planned, kernel, alone));
        if (rc != PT_OK || !planned) return rc;
        a[n++] = args;
        return n == kIgemmMaxProblems ? flush(st) : PT_OK;
    }
};

extern "C" int32_t pt_conv_fwd_batched(const pt_conv_desc* descs, const uint16_t* const* x, const uint16_t* const* w,
                                       uint16_t* const* y, int32_t n, void* stream) {
    if (n <= 0) return PT_ERR_SHAPE;
    if (!descs || !x || !w || !y) return PT_ERR_NULL;
    for (int i = 0; i < n; ++i) {
        const int32_t rc = check_desc(&descs[i]);
        if (rc != PT_OK) return rc;
        if (!x[i] || !w[i] || !y[i]) return PT_ERR_NULL;
    }
    hipStream_t st = (hipStream_t)stream;
    IgemmPending pend;
    for (int i = 0; i < n; ++i) {
        const pt_conv_desc* d = &descs[i];
        int32_t rc;
        if (stem_fwd_ok(d, x[i], w[i], y[i]) || res3_fwd_ok(d, x[i], w[i], y[i])) {  // layers with a kernel of their own
            rc = pt_conv_fwd(d, x[i], w[i], y[i], nullptr, 0, stream);
        } else {
            IgemmArgs a = make_fwd_args(d, x[i], w[i], y[i]);
            rc = pend.add(a, d->x_cpitch % 8 == 0 && d->w_cpitch % 8 == 0 && aligned16(x[i]) && aligned16(w[i]), st, fwd_kernel(d, x[i], w[i], y[i]));
        }
        if (rc != PT_OK) return rc;
    }
    return pend.flush(st);
}

// Input gradient from weights already in [C][RS][round_up(K,8)] order: one implicit GEMM per stride-parity class.
// `alone`: nothing else joins the call.
static int32_t bwd_data_classes(const pt_conv_desc* d, const uint16_t* dy, const uint16_t* wt, uint16_t* dx,
                                hipStream_t st, IgemmPending& pend, bool alone = false) {
    int32_t rc = PT_OK;
    bool resident = res3_bwd_ok(d, dy, wt, dx, false);
    if (!resident && alone && res3_bwd_ok(d, dy, wt, dx, true)) {  // (only where a batched call adds in the same order: the same bits)
        IgemmArgs a = make_bwd_data_args(d, bwd_data_class(d, 0, 0), 0, 0, dy, wt, dx);
        igemm_fold(a);
        resident = ceil_div(a.M, 128) >= 256 || !igemm_small_ok(a) || pick_igemm_kernel(&a, 1) == 0;
    }
    if (resident) {  // the same kernel on dy with the k-innermost filter copy and mirrored taps
        const int kp = (int)round_up(d->K, 8);
        Res3Args r{dy, wt, dx, d->N, d->H, d->W, d->K, kp, d->y_cpitch, d->C, kp, d->x_cpitch, 0, 0, 0, 0, 0, 0, 0};
        return hip_status(launch_conv3x3_res(r, kRes3Bwd, st));
    }
    // A filter no larger than the stride reaches only some stride-parity classes of input pixels.  When class
    // (0, 0) is the only one with taps, its launch also clears the other classes (they tile into cells anchored at
    // its pixels), which saves up to stride_h * stride_w - 1 small launches; this needs the vector store path and a
    // channel count whose last 8-chunk may be written whole.
    int with_taps = 0;
    for (int ca = 0; ca < d->stride_h; ++ca)
        for (int cb = 0; cb < d->stride_w; ++cb) {
            const BwdClass c = bwd_data_class(d, ca, cb);
            if (c.gH > 0 && c.gW > 0 && c.TR > 0 && c.TS > 0) ++with_taps;
        }
    const BwdClass c00 = bwd_data_class(d, 0, 0);
    const bool vec_all = d->x_cpitch % 8 == 0 && d->y_cpitch % 8 == 0 && aligned16(dx) && aligned16(dy);
    const bool fuse_zero = with_taps == 1 && c00.TR > 0 && c00.TS > 0 && d->stride_h * d->stride_w > 1 && vec_all &&
                           (d->C % 8 == 0 || (d->flags & PT_CONV_PAD_ZERO)) && c00.TR * c00.TS <= 64;
    // Classes that a direct kernel takes are collected and sent out together (a 3 x 3 filter at stride 2 has four
    // classes of 1, 2, 2 and 4 taps: four short launches one after the other otherwise).
    const bool vec = d->y_cpitch % 8 == 0 && aligned16(dy);
    auto args_of = [&](int ca, int cb) {
        const BwdClass c = bwd_data_class(d, ca, cb);
        IgemmArgs a = make_bwd_data_args(d, c, ca, cb, dy, wt, dx);
        if (fuse_zero) {
            a.zf_h = d->stride_h;
            a.zf_w = d->stride_w;
        }
        return a;
    };
    auto has_taps = [&](int ca, int cb) {
        const BwdClass c = bwd_data_class(d, ca, cb);
        return c.gH > 0 && c.gW > 0 && c.TR > 0 && c.TS > 0;
    };
    // several classes: one choice of kernel for each four of them, which share a launch, by what they are together (each by itself
    // they would not all choose the same and share fewer: 24 x 24 297 <- 5, 4 x 4 at stride 3, batch 24, 15.2 us in four launches)
    auto pick = [&](int first) {  // first class of the four, counted row by row
        IgemmArgs some[kIgemmMaxProblems];
        int n = 0;
        int64_t tiles128 = 0;
        bool small_ok = true;
        for (int i = first; i < d->stride_h * d->stride_w && n < kIgemmMaxProblems; ++i) {
            const int ca = i / d->stride_w, cb = i % d->stride_w;
            if (!has_taps(ca, cb)) continue;
            some[n] = args_of(ca, cb);
            igemm_fold(some[n]);
            tiles128 += ceil_div(some[n].M, 128) * ceil_div(some[n].Nout, 128);
            small_ok = small_ok && igemm_small_ok(some[n]);
            ++n;
        }
        return tiles128 >= 256 ? kIgemmLarge : small_ok ? pick_igemm_kernel(some, n) : 0;
    };
    int kernel = -1, seen = 0;
    for (int ca = 0; ca < d->stride_h; ++ca) {
        for (int cb = 0; cb < d->stride_w; ++cb) {
            BwdClass c = bwd_data_class(d, ca, cb);
            if (c.gH == 0 || c.gW == 0) continue;
            if (fuse_zero && (ca != 0 || cb != 0)) continue;  // cleared by the launch of class (0, 0)
            if (c.TR == 0 || c.TS == 0) {
                const int64_t pixels = (int64_t)d->N * c.gH * c.gW;
                const int64_t nblk = ceil_div(pixels * ceil_div(d->C, 8), 256);
                if (nblk > 0x7fffffff) return PT_ERR_UNSUPPORTED;
                const int vec16 = (d->x_cpitch % 8 == 0) && aligned16(dx);
                hipLaunchKernelGGL(k_zero_class, dim3((unsigned)nblk), dim3(256), 0, st, dx, pixels, c.gH, c.gW, d->H, d->W,
                                   d->stride_h, ca, d->stride_w, cb, d->x_cpitch, d->C, vec16);
                rc = launch_status();
            } else {
                IgemmArgs a = args_of(ca, cb);
                if (vec && with_taps > 1 && seen++ % kIgemmMaxProblems == 0) kernel = pick(ca * d->stride_w + cb);
                rc = pend.add(a, vec, st, kernel, alone && d->stride_h * d->stride_w == 1);
            }
            if (rc != PT_OK) return rc;
        }
    }
    return PT_OK;
}
static int32_t bwd_data_one(const pt_conv_desc* d, const uint16_t* dy, const uint16_t* wt, uint16_t* dx, hipStream_t st) {
    IgemmPending pend;
    const int32_t rc = bwd_data_classes(d, dy, wt, dx, st, pend, true);
    return rc == PT_OK ? pend.flush(st) : rc;
}

// Per-channel sums and sums of squares of 128 output pixels (blockIdx.x) x 64 channels (blockIdx.y), laid out as
// IgemmArgs::stats: 8 channels a lane, four rows a thread, the 32 threads of a channel added as a tree (a chain of 3 + 5
// additions, as short as that of the convolution kernels' epilogue).
__global__ __launch_bounds__(256) void k_tile_stats(const uint16_t* __restrict__ y, int64_t pixels, int K, int ypitch,
                                                    float* __restrict__ stats) {
    __shared__ float red[2][32][65];
    const int v = threadIdx.x & 7, row = threadIdx.x >> 3;
    const int k0 = blockIdx.y * 64 + v * 8;
    float s[8] = {}, q[8] = {};
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int64_t p = (int64_t)blockIdx.x * 128 + u * 32 + row;
        if (p >= pixels || k0 >= K) continue;
        const uint4 w = *reinterpret_cast<const uint4*>(y + p * ypitch + k0);
        const uint32_t words[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float f = __uint_as_float(e & 1 ? words[e / 2] & 0xffff0000u : words[e / 2] << 16);
            s[e] += f;
            q[e] += f * f;
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        red[0][row][v * 8 + e] = s[e];
        red[1][row][v * 8 + e] = q[e];
    }
    __syncthreads();
    if (threadIdx.x >= 128) return;
    const int c = threadIdx.x & 63, which = threadIdx.x >> 6, k = blockIdx.y * 64 + c;
    float t[32];
#pragma unroll
    for (int r = 0; r < 32; ++r) t[r] = red[which][r][c];
#pragma unroll
    for (int n = 16; n > 0; n /= 2)
#pragma unroll
        for (int r = 0; r < n; ++r) t[r] += t[r + n];
    if (k < K) stats[((size_t)which * gridDim.x + blockIdx.x) * K + k] = t[0];
}

// Forward convolution with the statistics epilogue: only the direct kernel has it.
static int32_t fwd_stats_supported(const pt_conv_desc* d, const uint16_t* x, const uint16_t* w, const uint16_t* y) {
    const bool vec = d->x_cpitch % 8 == 0 && d->w_cpitch % 8 == 0 && d->y_cpitch % 8 == 0 && aligned16(x) && aligned16(w) &&
                     aligned16(y);
    if (!vec || d->R * d->S > 64) return PT_ERR_UNSUPPORTED;
    if (d->C % 8 != 0 && !(d->flags & PT_CONV_PAD_ZERO)) return PT_ERR_UNSUPPORTED;
    return PT_OK;
}

extern "C" int32_t pt_conv_fwd_stats_workspace_bytes(const pt_conv_desc* d, size_t* bytes, int32_t* n_partial) {
    const int32_t rc = check_desc(d);
    if (rc != PT_OK) return rc;
    if (!bytes || !n_partial) return PT_ERR_NULL;
    *n_partial = (int32_t)ceil_div((int64_t)d->N * d->P * d->Q, 128);
    *bytes = (size_t)round_up((int64_t)2 * *n_partial * d->K * 4, 256);
    return PT_OK;
}

extern "C" int32_t pt_conv_fwd_stats(const pt_conv_desc* d, const uint16_t* x, const uint16_t* w, uint16_t* y, float* sums,
                                     size_t sums_bytes, void* stream) {
    int32_t rc = check_desc(d);
    if (rc != PT_OK) return rc;
    if (!x || !w || !y || !sums) return PT_ERR_NULL;
    rc = fwd_stats_supported(d, x, w, y);
    if (rc != PT_OK) return rc;
    const int64_t n_partial = ceil_div((int64_t)d->N * d->P * d->Q, 128);
    if (sums_bytes < (size_t)(2 * n_partial * d->K * 4)) return PT_ERR_WORKSPACE;
    IgemmArgs a = make_fwd_args(d, x, w, y);
    // A layer that pt_conv_fwd gives to a small-tile kernel: those have no epilogue of this kind and add in another order,
    // so they are called as they are and the sums are taken from their output.
    IgemmArgs f = a;
    igemm_fold(f);
    if (!stem_fwd_ok(d, x, w, y) && !res3_fwd_takes(d, x, w, y) && ceil_div(f.M, 128) * ceil_div(f.Nout, 128) < 256 &&
        igemm_small_ok(f) && pick_igemm_kernel(&f, 1) != 0) {
        rc = hip_status(launch_igemm(a, true, (hipStream_t)stream));
        if (rc != PT_OK) return rc;
        hipLaunchKernelGGL(k_tile_stats, dim3((unsigned)n_partial, (unsigned)ceil_div(d->K, 64)), dim3(256), 0,
                           (hipStream_t)stream, y, (int64_t)a.M, d->K, d->y_cpitch, sums);
        return launch_status();
    }
    a.stats = sums;
    return hip_status(launch_igemm(a, true, (hipStream_t)stream));
}

extern "C" int32_t pt_conv_bwd_data(const pt_conv_desc* d, const uint16_t* dy, const uint16_t* w, uint16_t* dx,
                                    void* ws, size_t ws_bytes, void* stream) {
    int32_t rc = check_desc(d);
    if (rc != PT_OK) return rc;
    if (!dy || !w || !dx || !ws) return PT_ERR_NULL;
    if (ws_bytes < bwd_data_ws(d)) return PT_ERR_WORKSPACE;
    if (!aligned16(ws)) return PT_ERR_SHAPE;
    hipStream_t st = (hipStream_t)stream;
    const int RS = d->R * d->S;
    const int kpitch = (int)round_up(d->K, 8);
    if (res3_bwd_ok(d, dy, w, dx, false) && d->w_cpitch % 8 == 0 && r3_krsc_bank_ok(d->K, d->C)) {  // transposes the filter bank itself
        Res3Args r{dy, w, dx, d->N, d->H, d->W, d->K, kpitch, d->y_cpitch, d->C, d->w_cpitch, d->x_cpitch, 0, 0, 0, 0, 0, 0, 0};
        return hip_status(launch_conv3x3_res(r, kRes3BwdKrsc, st));
    }
    uint16_t* wt = (uint16_t*)ws;
    hipLaunchKernelGGL(k_transpose_w, dim3((unsigned)ceil_div(d->C, kTrTile), (unsigned)ceil_div(kpitch, kTrTile), RS), dim3(256),
                       0, st, w, d->K, RS, d->C, d->w_cpitch, wt, kpitch);
    rc = launch_status();
    if (rc != PT_OK) return rc;
    return bwd_data_one(d, dy, wt, dx, st);
}

extern "C" int32_t pt_conv_bwd_data_crsk(const pt_conv_desc* d, const uint16_t* dy, const uint16_t* wt, uint16_t* dx,
                                         void* stream) {
    int32_t rc = check_desc(d);
    if (rc != PT_OK) return rc;
    if (!dy || !wt || !dx) return PT_ERR_NULL;
    if (!aligned16(wt)) return PT_ERR_SHAPE;
    return bwd_data_one(d, dy, wt, dx, (hipStream_t)stream);
}

extern "C" int32_t pt_conv_bwd_data_crsk_batched(const pt_conv_desc* descs, const uint16_t* const* dy,
                                                 const uint16_t* const* wt, uint16_t* const* dx, int32_t n, void* stream) {
    if (n <= 0) return PT_ERR_SHAPE;
    if (!descs || !dy || !wt || !dx) return PT_ERR_NULL;
    for (int i = 0; i < n; ++i) {
        const int32_t rc = check_desc(&descs[i]);
        if (rc != PT_OK) return rc;
        if (!dy[i] || !wt[i] || !dx[i]) return PT_ERR_NULL;
        if (!aligned16(wt[i])) return PT_ERR_SHAPE;
    }
    IgemmPending pend;
    for (int i = 0; i < n; ++i) {
        const int32_t rc = bwd_data_classes(&descs[i], dy[i], wt[i], dx[i], (hipStream_t)stream, pend);
        if (rc != PT_OK) return rc;
    }
    return pend.flush((hipStream_t)stream);
}

extern "C" int32_t pt_weights_to_crsk_batched(const pt_layer_crsk* layers, int32_t n, void* stream) {
    if (n < 0) return PT_ERR_SHAPE;
    if (n == 0) return PT_OK;
    if (!layers) return PT_ERR_NULL;
    for (int i = 0; i < n; ++i) {
        const pt_layer_crsk& l = layers[i];
        if (!l.w || !l.wt) return PT_ERR_NULL;
        if (l.K <= 0 || l.RS <= 0 || l.C <= 0 || l.w_cpitch < l.C) return PT_ERR_SHAPE;
        // (tiles of 32 x 32: what one launch held with the kernel's former tiles, kept as the limit of a layer)
        if ((int64_t)ceil_div(l.C, 32) * ceil_div(round_up(l.K, 8), 32) * l.RS > 0x3fffffff) return PT_ERR_UNSUPPORTED;
    }
    TransposeJobs t;
    t.n = 0;
    int64_t blocks = 0;
    auto flush = [&]() -> int32_t {
        if (t.n == 0) return PT_OK;
        end_table(t.first, t.n);
        hipLaunchKernelGGL(k_transpose_w_multi, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, t);
        t.n = 0;
        blocks = 0;
        return launch_status();
    };
    for (int i = 0; i < n; ++i) {
        const pt_layer_crsk& l = layers[i];
        const int kpitch = (int)round_up(l.K, 8);
        const int nbx = (int)ceil_div(l.C, kTrTile), nby = (int)ceil_div(kpitch, kTrTile);
        const int64_t nb = (int64_t)nbx * nby * l.RS;
        if (blocks + nb > 0x3fffffff) {
            const int32_t rc = flush();
            if (rc != PT_OK) return rc;
        }
        t.first[t.n] = (int)blocks;
        t.j[t.n++] = TransposeJob{l.w, l.wt, l.K, l.RS, l.C, l.w_cpitch, kpitch, nbx, nby, 0};
        blocks += nb;
        if (t.n == kMaxTransposeJobs) {
            const int32_t rc = flush();
            if (rc != PT_OK) return rc;
        }
    }
    return flush();
}

// Few slices over many outputs take the four-outputs-per-thread reduction, the rest the one-output-per-lane form.
static bool reduce_is_wide(const pt_conv_desc* d, const WgradPlan& p) {
    const int64_t work = (int64_t)d->K * p.Mtot;
    return p.splits <= kReduceWideMaxSplits && work >= kReduceWideMinOutputs && p.Mtot % 4 == 0;
}

extern "C" int32_t pt_conv_bwd_weight_plan(const pt_conv_desc* d, int32_t aligned, pt_wgrad_plan_info* info) {
    if (!info) return PT_ERR_NULL;
    const int32_t rc = check_desc(d);
    if (rc != PT_OK) return rc;
    const bool vec = aligned != 0 && d->x_cpitch % 8 == 0 && d->y_cpitch % 8 == 0;
    if (vec && stem_wgrad_ok(d)) {  // the first layer's own kernel: one slab per workgroup, always reduced
        StemWgradArgs s = make_stem_wgrad_args(d, nullptr, nullptr, nullptr);
        int slabs = 0;
        plan_stem_wgrad(s, &slabs);
        info->splits = slabs;
        info->tiles = 1;
        info->reduce_kind = PT_WGRAD_REDUCE_DEEP;
        info->tile_m = 32;
        info->tile_n = 64;
        return PT_OK;
    }
    const WgradPlan p = plan_wgrad(d, vec);
    info->splits = p.splits;
    info->tiles = p.tiles_m * p.tiles_n;
    info->reduce_kind = p.splits == 1 ? PT_WGRAD_REDUCE_NONE : (reduce_is_wide(d, p) ? PT_WGRAD_REDUCE_WIDE : PT_WGRAD_REDUCE_DEEP);
    info->tile_m = p.BM;
    info->tile_n = p.BN;
    return PT_OK;
}

// One layer of a weight gradient call.
struct WgradLayer {
    const pt_conv_desc* d;
    const uint16_t* x;
    const uint16_t* dy;
    float* dw;
    ReduceLasso rl;  // rl.w == nullptr: plain weight gradient
    bool vec, stem;
    WgradPlan p;
    size_t ws_off, ws_bytes;
};
static int32_t check_wgrad_layer(WgradLayer& L) {
    const int32_t rc = check_desc(L.d);
    if (rc != PT_OK) return rc;
    if (!L.x || !L.dy || !L.dw) return PT_ERR_NULL;
    // the direct kernel needs 16-byte aligned rows; it keeps one tile row block per filter tap
    L.vec = L.d->x_cpitch % 8 == 0 && L.d->y_cpitch % 8 == 0 && aligned16(L.x) && aligned16(L.dy);
    L.stem = L.vec && stem_wgrad_ok(L.d);
    return PT_OK;
}
// Workspace of a layer whose splits are planned; the regulariser needs a slab where the main kernel cannot add it.
static size_t wgrad_layer_ws(const WgradLayer& L) {
    if (L.stem) return stem_wgrad_ws(L.d);
    return L.rl.w ? wgrad_lasso_ws_of(L.d, L.p) : L.p.ws_bytes;
}

// Image-like first layer: its own kernel, one slab of partial sums per workgroup.
static int32_t launch_wgrad_stem(const WgradLayer& L, char* ws, hipStream_t st) {
    StemWgradArgs s = make_stem_wgrad_args(L.d, L.x, L.dy, (float*)(ws + L.ws_off));
    int slabs = 0;
    plan_stem_wgrad(s, &slabs);
    if (slabs <= 0) return PT_OK;
    const int32_t rc = hip_status(launch_stem_wgrad(s, slabs, L.d->stride_h, st));
    if (rc != PT_OK) return rc;
    hipLaunchKernelGGL(k_stem_wgrad_reduce, dim3((unsigned)(L.d->R * (kSwSlabRow / 64))), dim3(64 * kReduceWaves), 0, st,
                       (const float*)(ws + L.ws_off), slabs, L.d->K, L.d->R, L.d->S, L.d->C, L.d->w_cpitch, L.dw, L.rl);
    return launch_status();
}

// Weight gradients of n checked and planned layers: one launch of the direct kernel and one of the reduction per
// kWgMaxProblems layers (the register-staged kernel and the first layer's go out by themselves).  The regulariser's
// gradient is added where dw is written: in the reduction of a split layer, in the epilogue of an unsplit one of the
// direct kernel, and for an unsplit one of the register-staged kernel in a reduction over one slab of partial sums.
static int32_t launch_wgrad_layers(const WgradLayer* L, int n, bool beside, void* ws, hipStream_t st) {
    int32_t rc = PT_OK;
    WgradJobs main_jobs;
    ReduceJobs red_jobs;
    int nm = 0, nr = 0;
    int64_t red_blocks = 0;
    auto flush = [&]() -> int32_t {
        if (nm > 0) {
            const int32_t r = hip_status(launch_wgrad_dl(main_jobs, nm, beside, st));
            if (r != PT_OK) return r;
        }
        // (no more LDS than the form needs: beside a weight gradient and an input gradient a CU has 16 KB left)
        auto lds_of = [](int wide, int waves) { return (size_t)(wide ? waves / wide * (wide - 1) * 1024 : waves * 256); };
        if (nr == 1) {
            // (wide form: workgroups of 256 find room beside other kernels sooner)
            const int wide = red_jobs.j[0].wide;
            hipLaunchKernelGGL(k_wgrad_reduce, dim3((unsigned)(wide ? 2 * red_blocks : red_blocks)), dim3(wide ? 256 : 64 * kReduceWaves),
                               lds_of(wide, wide ? 4 : kReduceWaves), st, red_jobs.j[0]);
        } else if (nr > 1) {
            end_table(red_jobs.first, nr);
            size_t lds = 0;
            for (int i = 0; i < nr; ++i) lds = lds_of(red_jobs.j[i].wide, kReduceWaves) > lds ? lds_of(red_jobs.j[i].wide, kReduceWaves) : lds;
            hipLaunchKernelGGL(k_wgrad_reduce_multi, dim3((unsigned)red_blocks), dim3(64 * kReduceWaves), lds, st, red_jobs);
        }
        nm = nr = 0;
        red_blocks = 0;
        return launch_status();
    };
    for (int i = 0; i < n; ++i) {
        const pt_conv_desc* d = L[i].d;
        const WgradPlan& p = L[i].p;
        if (L[i].stem) {
            rc = launch_wgrad_stem(L[i], (char*)ws, st);
            if (rc != PT_OK) return rc;
            continue;
        }
        WgradArgs a = make_wgrad_args(d, p, L[i].x, L[i].dy, L[i].dw, (char*)ws + L[i].ws_off);
        if (L[i].rl.w && a.direct && p.dl && aligned16(L[i].rl.w)) {  // the direct kernel's own epilogue adds the term
            a.lw = L[i].rl.w;
            a.l_on = L[i].rl.out_norm;
            a.l_in = L[i].rl.in_norm;
            a.l_lambda = L[i].rl.lambda;
        } else if (L[i].rl.w) {  // the reduction adds it (one slab when the layer is not split)
            a.direct = 0;
            a.OUT = (float*)((char*)ws + L[i].ws_off);
        }
        if (p.dl) {
            main_jobs.a[nm++] = a;
        } else {
            rc = hip_status(L[i].vec ? launch_wgrad_cfg<kWgBM, kWgBN, kWgBK, 2, 2, 2>(a, st)
                                     : launch_wgrad_cfg<kWgBM, kWgBN, kWgBK, 2, 2, 2, false>(a, st));
            if (rc != PT_OK) return rc;
        }
        if (!a.direct) {
            const int64_t work = (int64_t)d->K * p.Mtot;
            const int wide = !reduce_is_wide(d, p) ? 0 : p.splits <= 4 ? 1 : p.splits <= 8 ? 2 : 4;
            red_jobs.first[nr] = (int)red_blocks;
            red_jobs.j[nr++] = ReduceJob{a.OUT, L[i].dw, L[i].rl, p.splits, d->K, a.RS, d->C, p.CP, d->w_cpitch, a.o_vec, wide};
            red_blocks += wide ? ceil_div(work, 256 * (kReduceWaves / wide)) : ceil_div(work, 64);
            if (red_blocks > 0x3fffffff) return PT_ERR_UNSUPPORTED;
        }
        if (nm == kWgMaxProblems || nr == kWgMaxProblems) {
            rc = flush();
            if (rc != PT_OK) return rc;
        }
    }
    return flush();
}

static int32_t bwd_weight_one(const pt_conv_desc* d, const uint16_t* x, const uint16_t* dy, float* dw, void* ws,
                              size_t ws_bytes, void* stream, const ReduceLasso& rl) {
    WgradLayer L{d, x, dy, dw, rl, false, false, {}, 0, 0};
    const int32_t rc = check_wgrad_layer(L);
    if (rc != PT_OK) return rc;
    if (!L.stem) L.p = plan_wgrad(d, L.vec);
    const size_t need = wgrad_layer_ws(L);
    if (need > 0 && !ws) return PT_ERR_NULL;
    if (ws_bytes < need) return PT_ERR_WORKSPACE;
    if (need > 0 && !aligned16(ws)) return PT_ERR_SHAPE;
    return launch_wgrad_layers(&L, 1, false, ws, (hipStream_t)stream);
}

extern "C" int32_t pt_conv_bwd_weight(const pt_conv_desc* d, const uint16_t* x, const uint16_t* dy, float* dw, void* ws,
                                      size_t ws_bytes, void* stream) {
    return bwd_weight_one(d, x, dy, dw, ws, ws_bytes, stream, ReduceLasso{nullptr, nullptr, nullptr, 0.f});
}

extern "C" int32_t pt_conv_bwd_weight_lasso_workspace_bytes(const pt_conv_desc* d, size_t* bytes) {
    if (!bytes) return PT_ERR_NULL;
    int32_t rc = check_desc(d);
    if (rc != PT_OK) return rc;
    const size_t a = wgrad_lasso_ws_of(d, plan_wgrad(d, true)), b = wgrad_lasso_ws_of(d, plan_wgrad(d, false));
    const size_t c = stem_wgrad_ok(d) ? stem_wgrad_ws(d) : 0;
    *bytes = a > b ? (a > c ? a : c) : (b > c ? b : c);
    return PT_OK;
}

extern "C" int32_t pt_conv_bwd_weight_lasso(const pt_conv_desc* d, const uint16_t* x, const uint16_t* dy, const float* w,
                                            const float* out_norm, const float* in_norm, float lambda, uint32_t flags,
                                            float* dw, void* ws, size_t ws_bytes, void* stream) {
    if (!w || !out_norm || !in_norm) return PT_ERR_NULL;
    if (flags & ~(PT_LASSO_OUT | PT_LASSO_IN)) return PT_ERR_UNSUPPORTED;
    const ReduceLasso rl{w, flags & PT_LASSO_OUT ? out_norm : nullptr, flags & PT_LASSO_IN ? in_norm : nullptr, lambda};
    return bwd_weight_one(d, x, dy, dw, ws, ws_bytes, stream, rl);
}

extern "C" int32_t pt_conv_layer_step(const pt_conv_desc* d, const uint16_t* x, const uint16_t* dy, const float* w,
                                      uint16_t* w_bf16, float* out_norm, float* in_norm, float lambda, uint32_t flags,
                                      uint16_t* y, uint16_t* dx, float* dw, void* ws, size_t ws_bytes, void* stream) {
    int32_t rc = check_desc(d);
    if (rc != PT_OK) return rc;
    if (!x || !dy || !w || !w_bf16 || !out_norm || !in_norm || !y || !dw) return PT_ERR_NULL;
    if (flags & ~(PT_LASSO_OUT | PT_LASSO_IN)) return PT_ERR_UNSUPPORTED;
    // everything that any of the calls would refuse, before the first of them enqueues anything
    const int RS = d->R * d->S;
    rc = check_norm_layer(NormLayer{w, out_norm, in_norm, w_bf16, nullptr, nullptr, d->K, RS, d->C, d->w_cpitch});
    if (rc != PT_OK) return rc;
    if (!ws) return PT_ERR_NULL;
    if (ws_bytes < norm_layer_ws_bytes(d->K, RS, d->C) || (dx && ws_bytes < bwd_data_ws(d))) return PT_ERR_WORKSPACE;
    if (!aligned16(ws)) return PT_ERR_SHAPE;
    WgradLayer L{d, x, dy, dw, ReduceLasso{w, flags & PT_LASSO_OUT ? out_norm : nullptr, flags & PT_LASSO_IN ? in_norm : nullptr, lambda},
                 false, false, {}, 0, 0};
    rc = check_wgrad_layer(L);
    if (rc != PT_OK) return rc;
    if (!L.stem) L.p = plan_wgrad(d, L.vec);
    const bool fused = ws_bytes >= wgrad_layer_ws(L);
    if (!fused) L.rl.w = nullptr;
    if (ws_bytes < wgrad_layer_ws(L)) return PT_ERR_WORKSPACE;

    rc = pt_group_norms(w, d->K, RS, d->C, d->w_cpitch, out_norm, in_norm, w_bf16, ws, ws_bytes, stream);
    if (rc == PT_OK) rc = pt_conv_fwd(d, x, w_bf16, y, ws, ws_bytes, stream);
    if (rc == PT_OK && dx) rc = pt_conv_bwd_data(d, dy, w_bf16, dx, ws, ws_bytes, stream);
    if (rc == PT_OK) rc = launch_wgrad_layers(&L, 1, false, ws, (hipStream_t)stream);
    if (rc != PT_OK || fused) return rc;
    return pt_group_lasso_grad(w, out_norm, in_norm, lambda, flags, dw, d->K, RS, d->C, d->w_cpitch, stream);
}

// Plans the layers of a batched call and lays their workspaces out one after the other; returns the bytes needed.
// Splits: every candidate cuts the work of the call into pieces of total / (rounds * CUs); of four, the one with the least
// estimated time, the work spread over the CUs + half of the longest piece (the last round is that uneven) + the partial
// sums.  Layers are put in descending order of the time their workgroups take, so that the short ones fill the end.
static int32_t plan_wgrad_batched(const pt_layer_wgrad* layers, int n, float lambda, int workgroups,
                                  std::vector<WgradLayer>& out, size_t* bytes, bool query) {
    if (workgroups < 0) return PT_ERR_SHAPE;
    const int slots = workgroups ? workgroups : kWgSlots;
    try {
        out.resize((size_t)n);
    } catch (const std::exception&) {  // (no memory for the plan: no exception leaves a C entry point)
        return PT_ERR_UNSUPPORTED;
    }
    float total = 0.f;
    for (int i = 0; i < n; ++i) {
        const pt_layer_wgrad& l = layers[i];
        ReduceLasso rl{nullptr, nullptr, nullptr, lambda};
        if (l.w) {
            if (l.flags & ~(PT_LASSO_OUT | PT_LASSO_IN)) return PT_ERR_UNSUPPORTED;
            if (!query && (!l.out_norm || !l.in_norm)) return PT_ERR_NULL;
            rl.w = l.w;
            rl.out_norm = l.flags & PT_LASSO_OUT ? l.out_norm : nullptr;
            rl.in_norm = l.flags & PT_LASSO_IN ? l.in_norm : nullptr;
        }
        out[i] = WgradLayer{&l.d, l.x, l.dy, l.dw, rl, false, false, {}, 0, 0};
        const int32_t rc = check_wgrad_layer(out[i]);
        if (rc != PT_OK) return rc;
        if (out[i].stem) continue;
        out[i].p = n == 1 && workgroups ? plan_wgrad_beside(&l.d, out[i].vec) : plan_wgrad_tiles(&l.d, out[i].vec);
        total += (float)out[i].p.tiles_m * out[i].p.tiles_n * out[i].p.iters_total * wgrad_step_us(out[i].p);
    }
    const bool alone = n == 1 && !workgroups;  // one layer with the chip to itself: planned as pt_conv_bwd_weight plans it
    if (alone && !out[0].stem) out[0].p = plan_wgrad(out[0].d, out[0].vec);
    float best_us = 1e30f;
    int best = 1;
    for (int rounds = 1; !alone && rounds <= (workgroups ? 1 : 4); ++rounds) {
        const float piece = total / (float)(rounds * slots);
        float longest = 0.f, part = 0.f;
        for (int i = 0; i < n; ++i) {
            if (out[i].stem) continue;
            WgradPlan& p = out[i].p;
            const float step = wgrad_step_us(p);
            set_wgrad_splits(out[i].d, p, (int64_t)(p.iters_total * step / piece + 0.5f));
            if (p.iters_per_split * step > longest) longest = p.iters_per_split * step;
            if (p.splits > 1) part += (float)p.splits * p.tiles_m * p.tiles_n * p.BM * p.BN * 4 * kWgPartialUsPerByte;
        }
        const float us = total / slots + 0.5f * longest + part;
        if (us < best_us) {
            best_us = us;
            best = rounds;
        }
    }
    size_t off = 0;
    for (int i = 0; i < n; ++i) {
        if (!out[i].stem && !alone) {
            WgradPlan& p = out[i].p;
            const float piece = total / (float)(best * slots);
            if (n == 1 && workgroups)  // (two of the smaller workgroups find room on a CU beside others)
                set_wgrad_splits(out[i].d, p, (p.cfg == 0 || p.cfg == kWgRow3 ? slots : slots * 5 / 3) / (p.tiles_m * p.tiles_n));
            else
                set_wgrad_splits(out[i].d, p, (int64_t)(p.iters_total * wgrad_step_us(p) / piece + 0.5f));
        }
        out[i].ws_off = off;
        off += wgrad_layer_ws(out[i]);
    }
    *bytes = off;
    std::stable_sort(out.begin(), out.end(), [](const WgradLayer& a, const WgradLayer& b) {
        if (a.stem || b.stem) return !a.stem && b.stem;
        return a.p.iters_per_split * wgrad_step_us(a.p) > b.p.iters_per_split * wgrad_step_us(b.p);
    });
    return PT_OK;
}

extern "C" int32_t pt_conv_bwd_weight_batched_workspace_bytes(const pt_layer_wgrad* layers, int32_t n, int32_t workgroups,
                                                              size_t* bytes) {
    if (!bytes) return PT_ERR_NULL;
    if (n < 0) return PT_ERR_SHAPE;
    *bytes = 0;
    if (n == 0) return PT_OK;
    if (!layers) return PT_ERR_NULL;
    std::vector<WgradLayer> v;
    return plan_wgrad_batched(layers, n, 0.f, workgroups, v, bytes, true);
}

extern "C" int32_t pt_conv_bwd_weight_batched(const pt_layer_wgrad* layers, int32_t n, float lambda, int32_t workgroups,
                                              void* ws, size_t ws_bytes, void* stream) {
    if (n < 0) return PT_ERR_SHAPE;
    if (n == 0) return PT_OK;
    if (!layers) return PT_ERR_NULL;
    std::vector<WgradLayer> v;
    size_t need = 0;
    const int32_t rc = plan_wgrad_batched(layers, n, lambda, workgroups, v, &need, false);
    if (rc != PT_OK) return rc;
    if (need > 0 && !ws) return PT_ERR_NULL;
    if (ws_bytes < need) return PT_ERR_WORKSPACE;
    if (need > 0 && !aligned16(ws)) return PT_ERR_SHAPE;
    return launch_wgrad_layers(v.data(), n, workgroups > 0, ws, (hipStream_t)stream);
}
