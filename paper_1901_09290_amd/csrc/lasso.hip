// Channel group-lasso kernels (Eq. 1-2): group L2 norms (+ bf16 shadow weights) and the gradient.
//
// Both are HBM-bound: group_norms reads the fp32 master weights once (4 B/param, +2 B/param written
// when the bf16 shadow is emitted); the gradient pass reads w and dw and writes dw (12 B/param).
// A network has tens of layers whose weight tensors are small (KBs to a few MB), so every kernel here
// is multi-tensor: up to kMaxJobs layers ride in the kernel arguments of ONE launch and a workgroup
// finds its (layer, row chunk) from a table of first-workgroup indices.
//
// Thread layout: a workgroup of 256 threads is a TY x TX grid, TX = lanes across the channel axis (a
// power of two <= 64, so a row of TX lanes lives inside one wavefront), TY = 256/TX rows in flight.  A
// thread keeps the same channel columns for every row it visits, so input-channel (column) sums stay
// in registers; output-channel (row) sums are reduced across the TX lanes with wavefront shuffles.
// Two levels, fixed order, no atomics: a workgroup owns whole rows of a chunk and writes one
// sum-of-squares per row and one partial per column; the finish kernel adds the R*S row sums of each
// filter and the per-chunk column partials in ascending order.
#include <exception>
#include <vector>
#include "common.h"
#include "norms.h"

namespace pt {

constexpr int kThreads = 256;
constexpr int kMaxC = 2048;  // 64 lanes x (8 float4 column groups | 32 scalar column groups) per thread
#ifndef PT_NORM_JOBS
#define PT_NORM_JOBS 64  // 64 x 88 bytes + 16 = 5.5 KiB of kernel arguments
#endif
constexpr int kNormBatches = 2, kNormFewBatches = 8, kNormMaxChunkRows = kThreads * 8 * kNormBatches;  // see plan_norm_chunks
constexpr int kMaxJobs = PT_NORM_JOBS;  // layers per launch (the table rides in the kernel arguments)

struct NormJob {
    const float* w;
    uint16_t* shadow;   // nullptr: no bf16 copy
    float* out_norm;
    float* in_norm;
    uint8_t* zero_out;  // nullptr, or [K]: the finish pass also writes (out_norm < thr)
    uint8_t* zero_in;   // nullptr, or [C]
    uint32_t ws_off;    // this job's scratch in the workspace, in floats: [K*RS] row sums, then [n_chunks][C] column partials
    int K, RS, C, cpitch;
    int n_chunks, rows_per_chunk;
};
struct NormJobs {
    NormJob j[kMaxJobs];
    int first[kMaxJobs];  // first workgroup of each job in the partial kernel ...
    int fin[kMaxJobs];    // ... and in the finish kernel
    float* ws;
    float thr;
    int n;
};
static_assert(sizeof(NormJobs) <= 8192, "kernel-argument table");
// One layer by itself: its kernel arguments are one read away instead of two, and the launch copies 96 bytes instead of 6 KB
// (16 x 16 channels 3 x 3: group norms 7.4 us in two launches -> 4.0 in one, gradient 3.8 -> 3.1 us).
struct NormJob1 {
    NormJob j;
    float* ws;
    float thr;
};
__device__ __forceinline__ const NormJob& norm_job(const NormJobs& jobs, const int (&first)[kMaxJobs], int& block) {
    const int ji = job_of_block(first, block);
    block -= first[ji];
    return jobs.j[ji];
}

struct LassoJob {
    const float* w;
    const float* out_norm;
    const float* in_norm;
    float* dw;
    float* mom;  // optimizer step only: momentum buffer; then w is updated in place and dw is read-only
    int K, RS, C, cpitch;
    int rows_per_chunk, txlog2;
    uint32_t flags;
    int pad;
};
constexpr int kMaxLassoJobs = 64;  // 5.6 KiB of kernel arguments: the 53 layers of ResNet-50 are one launch
struct LassoJobs {
    LassoJob j[kMaxLassoJobs];
    int first[kMaxLassoJobs];  // first workgroup of each job
    int n;
};
struct LassoJob1 {
    LassoJob j;
};
__device__ __forceinline__ const LassoJob& lasso_job(const LassoJobs& jobs, int& block) {
    const int ji = job_of_block(jobs.first, block);
    block -= jobs.first[ji];
    return jobs.j[ji];
}
__device__ __forceinline__ const LassoJob& lasso_job(const LassoJob1& jobs, int&) { return jobs.j; }

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
template <int VEC, bool NT = false>  // NT: not to be kept in the caches
__device__ __forceinline__ void load_vec(const float* p, float (&v)[VEC]) {
    if constexpr (VEC == 4) {
        const f32x4* q = reinterpret_cast<const f32x4*>(p);
        f32x4 t;
        if constexpr (NT) t = __builtin_nontemporal_load(q);
        else t = *q;
        v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    } else {
        v[0] = *p;
    }
}
template <int VEC, bool NT>
__device__ __forceinline__ void store_elems(float* p, const float (&v)[VEC], int n) {  // the first n
    if constexpr (VEC == 4) {
        const f32x4 t = {v[0], v[1], v[2], v[3]};
        if (n == 4) {
            if constexpr (NT) __builtin_nontemporal_store(t, reinterpret_cast<f32x4*>(p));
            else *reinterpret_cast<f32x4*>(p) = t;
        } else {
#pragma unroll
            for (int e = 0; e < 3; ++e)
                if (e < n) p[e] = v[e];
        }
    } else {
        *p = v[0];
    }
}

// Channel-axis layout of a layer for the vector kernel: Lv float4 columns, CG = 1 << cglog2 column groups per
// thread (1, 2, 4 or 8), TX = 1 << txlog2 lanes across a row; column of (tx, j) = tx + j * TX.
struct NormLayout {
    int cglog2, txlog2;
};
__host__ __device__ inline NormLayout norm_layout(int C) {
    const int Lv = (C + 3) >> 2;
    NormLayout l;
    l.cglog2 = 0;
    while ((64 << l.cglog2) < Lv) ++l.cglog2;           // <= 3 for C <= 2048
    const int per = (Lv + (1 << l.cglog2) - 1) >> l.cglog2;  // columns per group
    l.txlog2 = 0;
    while ((1 << l.txlog2) < per) ++l.txlog2;            // <= 6
    return l;
}

__device__ __forceinline__ void store_norm(float* norm, uint8_t* zero, int i, float sumsq, float thr) {
    const float n = sqrtf(sumsq);
    norm[i] = n;
    if (zero) zero[i] = n < thr ? 1 : 0;  // the comparison of pt_zero_groups
}

// kThreads threads (tid) = one chunk of whole rows of one layer (vector path: 16-byte aligned rows).  A thread keeps eight
// 16-byte loads in flight: 8 / CG rows at a time, CG column groups each.  Row sums: per thread over its columns,
// then a shuffle tree over the TX lanes of the row.  Column sums: in registers over the rows a thread visits, then
// over the rows of a wavefront by shuffles and over the four wavefronts through LDS, all in a fixed order; put(c, sum)
// takes them.  The row sums are behind the last barrier.
template <int CG, typename PUT>
__device__ __forceinline__ void norms_partial_body(const NormJob& J, float* __restrict__ rowsq, const PUT& put, int chunk,
                                                   int txlog2, float (*colred)[1024], int tid) {
    constexpr int U = 8 / CG;  // rows in flight per thread
    const int lane = tid & 63, wave = tid >> 6;
    const int TX = 1 << txlog2, TY = kThreads >> txlog2;
    const int tx = tid & (TX - 1), ty = tid >> txlog2;
    const int64_t rows = (int64_t)J.K * J.RS;
    const int64_t r0 = (int64_t)chunk * J.rows_per_chunk;
    const int64_t r1 = min(rows, r0 + J.rows_per_chunk);
    const int C = J.C, cpitch = J.cpitch;
    const int Lv = (C + 3) >> 2;
    const float* __restrict__ w = J.w;
    uint16_t* __restrict__ shadow = J.shadow;

    float acc[CG][4];
    bool col_ok[CG];
    int col_n[CG];  // valid elements of this thread's j-th column vector (0: none)
#pragma unroll
    for (int j = 0; j < CG; ++j) {
        const int cg = tx + j * TX;
        col_ok[j] = cg < Lv;
        col_n[j] = col_ok[j] ? min(4, C - cg * 4) : 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[j][e] = 0.f;
    }

    for (int64_t rb = r0 + ty; rb < r1; rb += (int64_t)TY * U) {
        float4 v[U][CG];
        // all loads first (rows past the chunk and columns past the row re-read a valid vector and are masked below)
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t r = min(rb + (int64_t)u * TY, r1 - 1);
#pragma unroll
            for (int j = 0; j < CG; ++j) {
                const int cg = col_ok[j] ? tx + j * TX : 0;
                v[u][j] = *reinterpret_cast<const float4*>(w + (size_t)r * cpitch + (size_t)cg * 4);
            }
        }
        float rs[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t r = rb + (int64_t)u * TY;
            const bool row_ok = r < r1;
            rs[u] = 0.f;
#pragma unroll
            for (int j = 0; j < CG; ++j) {
                float e4[4] = {v[u][j].x, v[u][j].y, v[u][j].z, v[u][j].w};
                const int n = row_ok ? col_n[j] : 0;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float x = e < n ? e4[e] : 0.f;  // pitch padding is not data
                    e4[e] = x;
                    const float q = x * x;
                    acc[j][e] += q;
                    rs[u] += q;
                }
                if (shadow && n > 0) {
                    const size_t off = (size_t)r * cpitch + (size_t)(tx + j * TX) * 4;
                    if (n == 4) {
                        // (past the caches: norms, value and step of the published ResNet-50 131.6 -> 129.8 us, of a
                        // pruned one 81.6 -> 79.9)
                        const u32x2 o = {cvt_pk_bf16(e4[0], e4[1]), cvt_pk_bf16(e4[2], e4[3])};
                        __builtin_nontemporal_store(o, reinterpret_cast<u32x2*>(shadow + off));
                    } else {
                        for (int e = 0; e < n; ++e) shadow[off + e] = f32_to_bf16(e4[e]);
                    }
                }
            }
        }
        for (int off = TX >> 1; off > 0; off >>= 1) {
#pragma unroll
            for (int u = 0; u < U; ++u) rs[u] += __shfl_xor(rs[u], off);
        }
        if (tx == 0) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t r = rb + (int64_t)u * TY;
                if (r < r1) rowsq[r] = rs[u];
            }
        }
    }

    // column partials: rows of one wavefront by shuffles (lanes tx, tx + TX, ... hold the same columns) ...
    for (int off = TX; off < 64; off <<= 1) {
#pragma unroll
        for (int j = 0; j < CG; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[j][e] += __shfl_xor(acc[j][e], off);
    }
    // ... then the four wavefronts through LDS in wavefront order, at most four column groups (1024 floats) per round
    constexpr int ROUNDS = CG > 4 ? CG / 4 : 1, PER = CG > 4 ? 4 : CG;
#pragma unroll
    for (int rnd = 0; rnd < ROUNDS; ++rnd) {
        if (rnd > 0) __syncthreads();
        if (lane < TX) {
#pragma unroll
            for (int jj = 0; jj < PER; ++jj)
#pragma unroll
                for (int e = 0; e < 4; ++e) colred[wave][(jj * TX + lane) * 4 + e] = acc[rnd * PER + jj][e];
        }
        __syncthreads();
        // with fewer than 64 lanes per row every wavefront holds full sums of its own rows; all four are added
        for (int f = tid; f < PER * TX * 4; f += kThreads) {
            const int c = rnd * PER * TX * 4 + f;
            if (c < C) put(c, ((colred[0][f] + colred[1][f]) + colred[2][f]) + colred[3][f]);
        }
    }
}

template <typename PUT>
__device__ __forceinline__ void norms_partial(const NormJob& J, float* rowsq, const PUT& put, int chunk, float (*colred)[1024], int tid) {
    const NormLayout l = norm_layout(J.C);
    switch (l.cglog2) {  // uniform
        case 0: norms_partial_body<1>(J, rowsq, put, chunk, l.txlog2, colred, tid); break;
        case 1: norms_partial_body<2>(J, rowsq, put, chunk, l.txlog2, colred, tid); break;
        case 2: norms_partial_body<4>(J, rowsq, put, chunk, l.txlog2, colred, tid); break;
        default: norms_partial_body<8>(J, rowsq, put, chunk, l.txlog2, colred, tid); break;
    }
}
// The same by a workgroup, with this job's scratch in the workspace.
__device__ __forceinline__ void norms_partial(const NormJob& J, float* ws, int chunk, float (*colred)[1024]) {
    float* rowsq = ws + J.ws_off;
    float* __restrict__ colpart = rowsq + (int64_t)J.K * J.RS + (int64_t)chunk * J.C;
    norms_partial(J, rowsq, [=](int c, float sum) { colpart[c] = sum; }, chunk, colred, threadIdx.x);
}
__global__ __launch_bounds__(kThreads) void k_group_norms_partial_vec(const NormJobs jobs) {
    __shared__ float colred[4][1024];
    int chunk = blockIdx.x;
    const NormJob& J = norm_job(jobs, jobs.first, chunk);
    norms_partial(J, jobs.ws, chunk, colred);
}
__global__ __launch_bounds__(kThreads) void k_group_norms_partial_vec_one(const NormJob1 job) {
    __shared__ float colred[4][1024];
    norms_partial(job.j, job.ws, blockIdx.x, colred);
}
// Element-wise path (rows that are not 16-byte aligned): one element per lane and column group, one row at a time.
__global__ __launch_bounds__(kThreads) void k_group_norms_partial_elem(const NormJobs jobs) {
    constexpr int kColsPerThread = kMaxC / 64;
    __shared__ float colred[kThreads];
    int chunk = blockIdx.x;
    const NormJob& J = norm_job(jobs, jobs.first, chunk);
    const int tid = threadIdx.x;
    int txlog2 = 0;
    while ((1 << txlog2) < J.C && txlog2 < 6) ++txlog2;
    const int TX = 1 << txlog2, TY = kThreads >> txlog2;
    const int tx = tid & (TX - 1), ty = tid >> txlog2;
    const int64_t rows = (int64_t)J.K * J.RS;
    const int64_t r0 = (int64_t)chunk * J.rows_per_chunk;
    const int64_t r1 = min(rows, r0 + J.rows_per_chunk);
    const int C = J.C, cpitch = J.cpitch;
    const float* __restrict__ w = J.w;
    uint16_t* __restrict__ shadow = J.shadow;
    float* __restrict__ rowsq = jobs.ws + J.ws_off;
    float* __restrict__ colpart = rowsq + rows;

    float acc[kColsPerThread];
#pragma unroll
    for (int j = 0; j < kColsPerThread; ++j) acc[j] = 0.f;
    for (int64_t r = r0 + ty; r < r1; r += TY) {
        const size_t roff = (size_t)r * cpitch;
        float rs = 0.f;
#pragma unroll
        for (int j = 0; j < kColsPerThread; ++j) {
            const int c = tx + j * TX;
            if (c < C) {
                const float v = w[roff + c];
                const float q = v * v;
                acc[j] += q;
                rs += q;
                if (shadow) shadow[roff + c] = f32_to_bf16(v);
            }
        }
        for (int off = TX >> 1; off > 0; off >>= 1) rs += __shfl_xor(rs, off);
        if (tx == 0) rowsq[r] = rs;
    }
    // column partials: across the TY row groups of the workgroup, in ty order, one column group at a time
#pragma unroll
    for (int j = 0; j < kColsPerThread; ++j) {
        if (j * TX >= C) break;  // uniform
        __syncthreads();
        colred[ty * TX + tx] = acc[j];
        __syncthreads();
        for (int f = tid; f < TX; f += kThreads) {
            const int c = j * TX + f;
            if (c < C) {
                float s = 0.f;
                for (int y = 0; y < TY; ++y) s += colred[y * TX + f];
                colpart[(size_t)chunk * C + c] = s;
            }
        }
    }
}

// The second level: first the K filters of a job, a thread each (their R*S row sums are contiguous), then its C input
// channels, 32 of them to a workgroup, whose per-chunk partials eight groups of lanes add (chunks g, g + 8, ...) and the
// eight sums in ascending order.  Eight loads in flight: bound by their latency (ResNet-50, 53 layers, 3 MB: 8.2 us with
// sixteen lanes on a group, each reading 16 of a 64-byte segment, 4.8 us so).  The order of additions depends only on
// the shapes, so results are run-to-run identical.  Jobs with mask pointers also get their zero masks here.
constexpr int kFinCols = 32, kFinSlices = kThreads / kFinCols;
__host__ __device__ inline int64_t fin_blocks_of(int K, int C) { return (K + kThreads - 1) / kThreads + (C + kFinCols - 1) / kFinCols; }
// Sum of p[i * stride], i = first, first + step, ... < n; loads past the end repeat the last one and are left out.
__device__ __forceinline__ float sum_strided(const float* __restrict__ p, int64_t stride, int first, int step, int n) {
    float s[4] = {0.f, 0.f, 0.f, 0.f};
    for (int i = first; i < n; i += 8 * step) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = p[(int64_t)min(i + u * step, n - 1) * stride];
#pragma unroll
        for (int u = 0; u < 8; ++u) s[u & 3] += i + u * step < n ? v[u] : 0.f;
    }
    return (s[0] + s[1]) + (s[2] + s[3]);
}
__device__ __forceinline__ void norms_finish(const NormJob& J, const float* __restrict__ ws, float thr, int block, float (*red)[kFinCols]) {
    const float* __restrict__ rowsq = ws + J.ws_off;
    const float* __restrict__ colpart = rowsq + (int64_t)J.K * J.RS;
    const int row_blocks = (J.K + kThreads - 1) / kThreads, tid = threadIdx.x;
    if (block < row_blocks) {  // uniform
        const int k = block * kThreads + tid;
        if (k < J.K) store_norm(J.out_norm, J.zero_out, k, sum_strided(rowsq + (int64_t)k * J.RS, 1, 0, 1, J.RS), thr);
        return;
    }
    const int l = tid % kFinCols, g = tid / kFinCols, c = (block - row_blocks) * kFinCols + l;
    red[g][l] = c < J.C ? sum_strided(colpart + c, J.C, g, kFinSlices, J.n_chunks) : 0.f;
    __syncthreads();
    if (g == 0 && c < J.C) {
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < kFinSlices; ++i) s += red[i][l];
        store_norm(J.in_norm, J.zero_in, c, s, thr);
    }
}
__global__ __launch_bounds__(kThreads) void k_group_norms_finish(const NormJobs jobs) {
    __shared__ float red[kFinSlices][kFinCols];
    int block = blockIdx.x;
    const NormJob& J = norm_job(jobs, jobs.fin, block);
    norms_finish(J, jobs.ws, jobs.thr, block, red);
}
__global__ __launch_bounds__(kThreads) void k_group_norms_finish_one(const NormJob1 job) {
    __shared__ float red[kFinSlices][kFinCols];
    norms_finish(job.j, job.ws, job.thr, blockIdx.x, red);
}
// A layer of up to two chunks (16 K elements): norms, masks and bf16 copy in one launch of one workgroup, with the row sums
// and column partials in LDS and kThreads threads to a chunk, which all reach the same barriers (32 x 32 channels 3 x 3: 9.1 us
// in two launches, 7.0 with one chunk after the other, 4.8 so).  The additions are those of the two launches (a chunk's partial is its slice's only
// one, so the slices in ascending order are the chunks in ascending order), and a layer has the same norms, bit for bit, by
// itself and among others: a group at the threshold of a detection cannot be zero by one route only.
static_assert(kNormBatches <= kFinSlices, "one chunk a slice");
__global__ __launch_bounds__(kThreads * kNormBatches) void k_group_norms_whole(const NormJob1 job) {
    __shared__ float colred[kNormBatches][4][1024];
    __shared__ float rowsq[kNormMaxChunkRows], colpart[kNormBatches * kMaxC];
    const NormJob& J = job.j;
    const int chunk = __builtin_amdgcn_readfirstlane(threadIdx.x / kThreads);  // blockDim.x = n_chunks * kThreads
    auto put = [&](int c, float sum) {
        if (J.n_chunks > 1) colpart[chunk * J.C + c] = sum;
        else store_norm(J.in_norm, J.zero_in, c, sum, job.thr);
    };
    norms_partial(J, rowsq, put, chunk, colred[chunk], threadIdx.x % kThreads);
    for (int k = threadIdx.x; k < J.K; k += blockDim.x) {
        float s[4] = {0.f, 0.f, 0.f, 0.f};  // sum_strided's four sums, without its loads past the end
        for (int t = 0; t < J.RS; ++t) {
            const float v = rowsq[k * J.RS + t];
            s[3] += (t & 3) == 3 ? v : 0.f;
            s[2] += (t & 3) == 2 ? v : 0.f;
            s[1] += (t & 3) == 1 ? v : 0.f;
            s[0] += (t & 3) == 0 ? v : 0.f;
        }
        store_norm(J.out_norm, J.zero_out, k, (s[0] + s[1]) + (s[2] + s[3]), job.thr);
    }
    if (J.n_chunks == 1) return;
    __syncthreads();
    for (int c = threadIdx.x; c < J.C; c += blockDim.x)
        store_norm(J.in_norm, J.zero_in, c, colpart[c] + colpart[J.C + c], job.thr);
}

// UPDATE = false: dw += lambda * d(penalty)/dw.   UPDATE = true: the optimizer step with the regulariser folded in,
//   g = dw + wd*w + lambda*w*(a/out_norm + b/in_norm);  mom = mu*mom + g;  w -= lr*mom   (one pass over w, dw, mom).
struct StepParams {
    float lr, mu, wd;
};
// Bound by HBM and by how many loads are in flight: a thread sends out those of four rows before the first store (which the
// compiler would otherwise not let a later row's loads pass), and walks filters and rows of a filter without divisions.
// HINT: what goes past the caches; the gradient pass 0 = nothing, the optimizer step 1 = the loads of dw and mom, or, when w,
// dw and mom of the call do not fit the chip's last cache anyway, 2 = every access.  Norms, value and step, row by row
// without hints / four rows with 0 / 1 / 2: published ResNet-50 (282 MB) 141 / 133 / 140 / 125 us, pruned ones (113 MB)
// 92.1 / 87.8 / 81.4 / 86.1 and 83.7 / 80.7 / 74.2 / 78.2, pruned ResNet-32 (2 MB) 31.0 / 30.3 / 30.5 / 30.8.  Two and eight
// rows: 1 to 4 and 3 to 8 % slower.
constexpr int kLassoRows = 4;
constexpr int64_t kInfinityCacheBytes = 256ll << 20;
template <int VEC, bool UPDATE, typename JOBS, int HINT = 0>
__global__ __launch_bounds__(kThreads) void k_group_lasso_grad(const JOBS jobs, float lambda, StepParams sp) {
    int chunk = blockIdx.x;
    const LassoJob& J = lasso_job(jobs, chunk);
    const int tid = threadIdx.x;
    const int TX = 1 << J.txlog2, TY = kThreads >> J.txlog2;
    const int tx = tid & (TX - 1), ty = tid >> J.txlog2;
    const int C = J.C, cpitch = J.cpitch, RS = J.RS;
    const int Lv = (C + VEC - 1) / VEC;
    const int64_t rows = (int64_t)J.K * RS;
    const int64_t r0 = (int64_t)chunk * J.rows_per_chunk;
    const int64_t r1 = min(rows, r0 + J.rows_per_chunk);
    const bool reg_out = J.flags & PT_LASSO_OUT, reg_in = J.flags & PT_LASSO_IN;
    float* __restrict__ w = const_cast<float*>(J.w);
    float* __restrict__ dw = J.dw;
    float* __restrict__ mom = J.mom;

    const int tk = TY / RS, trs = TY - tk * RS;  // filters and rows of a filter that TY rows are
    for (int cg = tx; cg < Lv; cg += TX) {
        float inv_in[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            const int c = cg * VEC + e;
            const float nrm = (reg_in && c < C) ? J.in_norm[c] : 0.f;
            inv_in[e] = nrm > 0.f ? 1.0f / nrm : 0.f;
        }
        const int n = min(VEC, C - cg * VEC);  // valid elements of this thread's column vector
        int k = (int)((r0 + ty) / RS), rs = (int)(r0 + ty - (int64_t)k * RS);
        for (int64_t r = r0 + ty; r < r1; r += (int64_t)kLassoRows * TY) {
            float v[kLassoRows][VEC], g[kLassoRows][VEC], m[kLassoRows][VEC], on[kLassoRows];
            // all loads first (rows past the chunk re-read its last one and are not stored)
#pragma unroll
            for (int u = 0; u < kLassoRows; ++u) {
                const size_t off = (size_t)min(r + (int64_t)u * TY, r1 - 1) * cpitch + (size_t)cg * VEC;
                load_vec<VEC, HINT == 2>(w + off, v[u]);
                load_vec<VEC, HINT != 0>(dw + off, g[u]);
                if constexpr (UPDATE) load_vec<VEC, HINT != 0>(mom + off, m[u]);
                on[u] = reg_out ? J.out_norm[min(k, J.K - 1)] : 0.f;
                k += tk;
                rs += trs;
                if (rs >= RS) rs -= RS, ++k;
            }
#pragma unroll
            for (int u = 0; u < kLassoRows; ++u) {
                if (r + (int64_t)u * TY >= r1) break;
                const size_t off = (size_t)(r + (int64_t)u * TY) * cpitch + (size_t)cg * VEC;
                const float inv_out = on[u] > 0.f ? 1.0f / on[u] : 0.f;
                float* dst = dw;
#pragma unroll
                for (int e = 0; e < VEC; ++e) g[u][e] += lambda * (v[u][e] * (inv_out + inv_in[e]));
                if constexpr (UPDATE) {
#pragma unroll
                    for (int e = 0; e < VEC; ++e) {
                        m[u][e] = sp.mu * m[u][e] + (g[u][e] + sp.wd * v[u][e]);
                        g[u][e] = v[u][e] - sp.lr * m[u][e];  // g now holds the new weight
                    }
                    store_elems<VEC, HINT == 2>(mom + off, m[u], n);
                    dst = w;
                }
                store_elems<VEC, HINT == 2>(dst + off, g[u], n);
            }
        }
    }
}

// ---- host-side planning ---------------------------------------------------------------------- //
struct ChunkPlan {
    int txlog2, rows_per_chunk, n_chunks;
};

// Gradient / optimizer pass and the element-wise norms pass: TX lanes across a row, about `elements` per workgroup.
static ChunkPlan plan_chunks(int64_t rows, int C, bool vec, int elements = 16384) {
    const int Lv = vec ? (C + 3) / 4 : C;
    int l = 0;
    while ((1 << l) < Lv && l < 6) ++l;
    const int TY = kThreads >> l;
    int64_t rpc = ceil_div(elements, C);
    rpc = round_up(rpc, TY);
    ChunkPlan p;
    p.txlog2 = l;
    p.rows_per_chunk = (int)rpc;
    p.n_chunks = (int)ceil_div(rows, rpc);
    return p;
}

// Vector norms pass: a workgroup streams whole batches of TY * U rows (256 threads x eight 16-byte loads, 8 K
// elements when every lane has a column), kNormBatches of them per chunk, or one where the whole layer is few: such a
// network's pass is a chain of latencies, and a second batch is one more of them (a pruned ResNet-32, norms, value and step:
// 30.3 -> 26.4 us; ResNet-50 with one batch everywhere 124.9 -> 127.6, with four 125.6, pruned 80.8 -> 80.6 and 83.9).
static ChunkPlan plan_norm_chunks(int64_t rows, int C) {
    const NormLayout l = norm_layout(C);
    const int batch_rows = (kThreads >> l.txlog2) * (8 >> l.cglog2);
    ChunkPlan p;
    p.txlog2 = l.txlog2;
    p.rows_per_chunk = batch_rows * (rows <= (int64_t)batch_rows * kNormFewBatches ? 1 : kNormBatches);
    p.n_chunks = (int)ceil_div(rows, p.rows_per_chunk);
    return p;
}

static bool norms_vec_ok(const NormLayer& L) {
    return (L.cpitch % 4 == 0) && (((uintptr_t)L.w & 15) == 0) && (!L.shadow || ((uintptr_t)L.shadow & 7) == 0) && L.C <= kMaxC;
}

int32_t check_norm_layer(const NormLayer& L) {
    if (!L.w || !L.out_norm || !L.in_norm) return PT_ERR_NULL;
    if (L.K <= 0 || L.RS <= 0 || L.C <= 0 || L.cpitch < L.C) return PT_ERR_SHAPE;
    if (L.C > kMaxC) return PT_ERR_UNSUPPORTED;  // register tile of the column sums
    if ((int64_t)L.K * L.RS >= (1ll << 31)) return PT_ERR_UNSUPPORTED;
    return PT_OK;
}

// Workspace of one layer: row sums + per-chunk column partials, sized for whichever loader is used.
size_t norm_layer_ws_bytes(int32_t K, int32_t RS, int32_t C) {
    const int64_t rows = (int64_t)K * RS;
    const ChunkPlan a = plan_norm_chunks(rows, C), b = plan_chunks(rows, C, false);
    const int n_chunks = a.n_chunks > b.n_chunks ? a.n_chunks : b.n_chunks;
    return (size_t)round_up((rows + (int64_t)n_chunks * C) * 4, 256);
}

// Group norms (and optionally zero masks) of n layers: one partial + one finish launch per kMaxJobs layers of a
// loader kind.  The workspace is split between the layers in array order.
int32_t launch_norms(const NormLayer* layers, int n, void* ws, size_t ws_bytes, float thr, hipStream_t st) {
    size_t need = 0;
    for (int i = 0; i < n; ++i) {
        const int32_t rc = check_norm_layer(layers[i]);
        if (rc != PT_OK) return rc;
        need += norm_layer_ws_bytes(layers[i].K, layers[i].RS, layers[i].C);
    }
    if (!ws) return PT_ERR_NULL;
    if (ws_bytes < need) return PT_ERR_WORKSPACE;
    if (((uintptr_t)ws & 15) != 0) return PT_ERR_SHAPE;
    if (need / 4 >= (1ull << 32)) return PT_ERR_UNSUPPORTED;
    for (int pass = 0; pass < 2; ++pass) {
        const bool want_vec = pass == 0;
        NormJobs jobs;
        jobs.n = 0;
        jobs.ws = (float*)ws;
        jobs.thr = thr;
        int64_t blocks = 0, fin_blocks = 0;
        auto flush = [&]() -> int32_t {
            if (jobs.n == 0) return PT_OK;
            if (jobs.n == 1 && want_vec) {  // a layer by itself
                NormJob1 one{jobs.j[0], jobs.ws, jobs.thr};
                if (one.j.n_chunks <= kNormBatches) {  // a few chunks of one batch
                    hipLaunchKernelGGL(k_group_norms_whole, dim3(1), dim3(kThreads * one.j.n_chunks), 0, st, one);
                } else {
                    hipLaunchKernelGGL(k_group_norms_partial_vec_one, dim3((unsigned)blocks), dim3(kThreads), 0, st, one);
                    const int32_t rc = launch_status();
                    if (rc != PT_OK) return rc;
                    hipLaunchKernelGGL(k_group_norms_finish_one, dim3((unsigned)fin_blocks), dim3(kThreads), 0, st, one);
                }
                jobs.n = 0;
                blocks = 0;
                fin_blocks = 0;
                return launch_status();
            }
            end_table(jobs.first, jobs.n);
            end_table(jobs.fin, jobs.n);
            if (want_vec) hipLaunchKernelGGL(k_group_norms_partial_vec, dim3((unsigned)blocks), dim3(kThreads), 0, st, jobs);
            else hipLaunchKernelGGL(k_group_norms_partial_elem, dim3((unsigned)blocks), dim3(kThreads), 0, st, jobs);
            int32_t rc = launch_status();
            if (rc != PT_OK) return rc;
            hipLaunchKernelGGL(k_group_norms_finish, dim3((unsigned)fin_blocks), dim3(kThreads), 0, st, jobs);
            jobs.n = 0;
            blocks = 0;
            fin_blocks = 0;
            return launch_status();
        };
        size_t off = 0;  // bytes
        for (int i = 0; i < n; ++i) {
            const NormLayer& L = layers[i];
            const size_t bytes = norm_layer_ws_bytes(L.K, L.RS, L.C);
            if (norms_vec_ok(L) == want_vec) {
                const int64_t rows = (int64_t)L.K * L.RS;
                const ChunkPlan cp = want_vec ? plan_norm_chunks(rows, L.C) : plan_chunks(rows, L.C, false);
                if (blocks + cp.n_chunks > 0x3fffffff) {
                    const int32_t rc = flush();
                    if (rc != PT_OK) return rc;
                }
                jobs.first[jobs.n] = (int)blocks;
                jobs.fin[jobs.n] = (int)fin_blocks;
                NormJob& J = jobs.j[jobs.n++];
                J.w = L.w; J.shadow = L.shadow; J.out_norm = L.out_norm; J.in_norm = L.in_norm;
                J.zero_out = L.zero_out; J.zero_in = L.zero_in;
                J.ws_off = (uint32_t)(off / 4);
                J.K = L.K; J.RS = L.RS; J.C = L.C; J.cpitch = L.cpitch;
                J.n_chunks = cp.n_chunks; J.rows_per_chunk = cp.rows_per_chunk;
                blocks += cp.n_chunks;
                fin_blocks += fin_blocks_of(L.K, L.C);
                if (jobs.n == kMaxJobs) {
                    const int32_t rc = flush();
                    if (rc != PT_OK) return rc;
                }
            }
            off += bytes;
        }
        const int32_t rc = flush();
        if (rc != PT_OK) return rc;
    }
    return PT_OK;
}

// Value of the regulariser (GroupLassoReg of Alg. 1): the sum of the enabled group norms of up to
// kMaxPenaltyJobs layers, ONE workgroup, fp64 accumulation in a fixed order (wavefront v adds the vectors v, v+16, ... of
// the table, lane l of it the elements 4l .. 4l+3, 4l+256 .. of a vector; fixed trees add the lanes and the wavefronts),
// so the value is run-to-run identical.  A few 10^4 floats: bound by the latency of the loads, so the wavefronts work on
// different vectors at once and a lane has four 16-byte loads in flight (ResNet-50, 106 vectors: 24 us when all threads
// walked the vectors one after the other with 4-byte loads, 6 us so).
constexpr int kMaxPenaltyJobs = 96;
struct PenaltyJob {
    const float* out_norm;
    const float* in_norm;
    int K, C;  // 0 when that group kind is not regularised
};
struct PenaltyJobs {
    PenaltyJob j[kMaxPenaltyJobs];
    int n, accumulate;
};
__global__ __launch_bounds__(1024) void k_group_lasso_penalty(const PenaltyJobs jobs, double* __restrict__ penalty) {
    __shared__ double red[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    double s = 0.0;
    for (int v = wave; v < 2 * jobs.n; v += 16) {
        const PenaltyJob& J = jobs.j[v >> 1];
        const float* __restrict__ p = (v & 1) == 0 ? J.out_norm : J.in_norm;
        const int n = (v & 1) == 0 ? J.K : J.C;
        const int n4 = ((uintptr_t)p & 15) == 0 ? n >> 2 : 0;  // whole 16-byte groups
#pragma unroll 4
        for (int e = lane; e < n4; e += 64) {
            const float4 q = reinterpret_cast<const float4*>(p)[e];
            s += ((double)q.x + (double)q.y) + ((double)q.z + (double)q.w);
        }
        for (int e = n4 * 4 + lane; e < n; e += 64) s += (double)p[e];
    }
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    if (lane == 0) red[wave] = s;
    __syncthreads();
    if (tid == 0)
        for (int w = 1; w < 16; ++w) s += red[w];
    if (tid == 0) *penalty = (jobs.accumulate ? *penalty : 0.0) + s;
}

}  // namespace pt

using namespace pt;

// A host table of n layers; false where there is no memory for it (no exception leaves a C entry point).
template <typename T>
static bool make_table(std::vector<T>& v, int32_t n) {
    try {
        v.resize((size_t)n);
    } catch (const std::exception&) {
        return false;
    }
    return true;
}

extern "C" int32_t pt_group_norms_batched_workspace_bytes(const pt_layer_weights* layers, int32_t n, size_t* bytes) {
    if (!bytes || (n > 0 && !layers)) return PT_ERR_NULL;
    if (n < 0) return PT_ERR_SHAPE;
    size_t total = 0;
    for (int i = 0; i < n; ++i) {
        if (layers[i].K <= 0 || layers[i].RS <= 0 || layers[i].C <= 0) return PT_ERR_SHAPE;
        total += norm_layer_ws_bytes(layers[i].K, layers[i].RS, layers[i].C);
    }
    *bytes = total;
    return PT_OK;
}

extern "C" int32_t pt_group_norms_batched(const pt_layer_weights* layers, int32_t n, void* ws, size_t ws_bytes,
                                          void* stream) {
    if (n < 0) return PT_ERR_SHAPE;
    if (n == 0) return PT_OK;
    if (!layers || !ws) return PT_ERR_NULL;
    std::vector<NormLayer> v;
    if (!make_table(v, n)) return PT_ERR_UNSUPPORTED;
    for (int i = 0; i < n; ++i) {
        const pt_layer_weights& L = layers[i];
        v[i] = NormLayer{L.w, L.out_norm, L.in_norm, L.w_shadow, nullptr, nullptr, L.K, L.RS, L.C, L.w_cpitch};
    }
    return launch_norms(v.data(), n, ws, ws_bytes, 0.f, (hipStream_t)stream);
}

extern "C" int32_t pt_group_norms_detect_batched_workspace_bytes(const pt_layer_detect* layers, int32_t n, size_t* bytes) {
    if (!bytes || (n > 0 && !layers)) return PT_ERR_NULL;
    if (n < 0) return PT_ERR_SHAPE;
    size_t total = 0;
    for (int i = 0; i < n; ++i) {
        if (layers[i].K <= 0 || layers[i].RS <= 0 || layers[i].C <= 0) return PT_ERR_SHAPE;
        total += norm_layer_ws_bytes(layers[i].K, layers[i].RS, layers[i].C);
    }
    *bytes = total;
    return PT_OK;
}

extern "C" int32_t pt_group_norms_detect_batched(const pt_layer_detect* layers, int32_t n, float thr, void* ws,
                                                 size_t ws_bytes, void* stream) {
    if (n < 0) return PT_ERR_SHAPE;
    if (n == 0) return PT_OK;
    if (!layers || !ws) return PT_ERR_NULL;
    std::vector<NormLayer> v;
    if (!make_table(v, n)) return PT_ERR_UNSUPPORTED;
    for (int i = 0; i < n; ++i) {
        const pt_layer_detect& L = layers[i];
        if (!L.zero_out || !L.zero_in) return PT_ERR_NULL;
        v[i] = NormLayer{L.w, L.out_norm, L.in_norm, nullptr, L.zero_out, L.zero_in, L.K, L.RS, L.C, L.w_cpitch};
    }
    return launch_norms(v.data(), n, ws, ws_bytes, thr, (hipStream_t)stream);
}

// Shared launcher of the gradient pass and of the optimizer step (mom == nullptr in every layer <=> gradient pass).
struct LassoLayer {
    const float* w;
    const float* out_norm;
    const float* in_norm;
    float* dw;
    float* mom;
    int32_t K, RS, C, w_cpitch;
    uint32_t flags;
};
// Elements per workgroup of the gradient / optimizer pass over `total` elements, which plan_chunks rounds up to as many rows as
// a workgroup takes at a time (8 K elements at 2048 channels): the most of 1 to 16 K with which there are 1280 workgroups, or
// 1 K (a small network's pass is a chain of rounds of loads, and at 1 K and 2 K a thread of a narrow layer has one and two
// rows: of the four it loads, the others are its chunk's last one again), or 32 K where everything passes by the caches.
// Norms, value and step with 1 / 2 / 4 / 8 / 16 / 32 K: pruned ResNet-32 (0.15 M elements) 20.5 / 20.7 / 27 / 28 / 31 / 26 us
// (4 K and 16 K also seen at 26), pruned ResNet-50 (9.4 M) 90.1 / 80.4 / 75.4 / 78.1 / 80.9 / 94.5, published (23.5 M) 171 /
// 161 / 141 / 128.5 / 125.5 / 121.6.
static bool past_caches(int64_t elements) { return elements * 12 > kInfinityCacheBytes; }  // w, dw, mom
static int lasso_chunk(int64_t total, bool update) {
    if (update && past_caches(total)) return 32768;
    int chunk = 1024;
    while (chunk < 16384 && total / (2 * chunk) >= 1280) chunk *= 2;
    return chunk;
}
static int32_t launch_lasso(const LassoLayer* layers, int n, bool update, float lambda, StepParams sp, hipStream_t st) {
    int64_t total = 0;
    for (int i = 0; i < n; ++i) total += (int64_t)layers[i].K * layers[i].RS * layers[i].w_cpitch;
    const int chunk = lasso_chunk(total, update);
    for (int pass = 0; pass < 2; ++pass) {
        const bool want_vec = pass == 0;
        LassoJobs jobs;
        jobs.n = 0;
        int blocks = 0;
        auto flush = [&]() -> int32_t {
            if (jobs.n == 0) return PT_OK;
            end_table(jobs.first, jobs.n);
            if (want_vec && jobs.n == 1 && !update)  // a layer by itself
                hipLaunchKernelGGL((k_group_lasso_grad<4, false, LassoJob1>), dim3(blocks), dim3(kThreads), 0, st, LassoJob1{jobs.j[0]}, lambda, sp);
            else if (want_vec && update) {
                const auto kern = past_caches(total) ? k_group_lasso_grad<4, true, LassoJobs, 2> : k_group_lasso_grad<4, true, LassoJobs, 1>;
                hipLaunchKernelGGL(kern, dim3(blocks), dim3(kThreads), 0, st, jobs, lambda, sp);
            }
            else if (want_vec)
                hipLaunchKernelGGL((k_group_lasso_grad<4, false, LassoJobs>), dim3(blocks), dim3(kThreads), 0, st, jobs, lambda, sp);
            else if (update)
                hipLaunchKernelGGL((k_group_lasso_grad<1, true, LassoJobs>), dim3(blocks), dim3(kThreads), 0, st, jobs, lambda, sp);
            else
                hipLaunchKernelGGL((k_group_lasso_grad<1, false, LassoJobs>), dim3(blocks), dim3(kThreads), 0, st, jobs, lambda, sp);
            jobs.n = 0;
            blocks = 0;
            return launch_status();
        };
        for (int i = 0; i < n; ++i) {
            const LassoLayer& L = layers[i];
            const bool vec = (L.w_cpitch % 4 == 0) && (((uintptr_t)L.w & 15) == 0) && (((uintptr_t)L.dw & 15) == 0) &&
                             (!update || ((uintptr_t)L.mom & 15) == 0);
            if (vec != want_vec) continue;
            const ChunkPlan cp = plan_chunks((int64_t)L.K * L.RS, L.C, vec, chunk);
            jobs.first[jobs.n] = blocks;
            LassoJob& J = jobs.j[jobs.n++];
            J.w = L.w; J.out_norm = L.out_norm; J.in_norm = L.in_norm; J.dw = L.dw; J.mom = L.mom;
            J.K = L.K; J.RS = L.RS; J.C = L.C; J.cpitch = L.w_cpitch;
            J.rows_per_chunk = cp.rows_per_chunk; J.txlog2 = cp.txlog2;
            J.flags = L.flags; J.pad = 0;
            blocks += cp.n_chunks;
            if (jobs.n == kMaxLassoJobs) {
                int32_t rc = flush();
                if (rc != PT_OK) return rc;
            }
        }
        int32_t rc = flush();
        if (rc != PT_OK) return rc;
    }
    return PT_OK;
}

extern "C" int32_t pt_group_lasso_grad_batched(const pt_layer_lasso* layers, int32_t n, float lambda, void* stream) {
    if (n < 0) return PT_ERR_SHAPE;
    if (n == 0) return PT_OK;
    if (!layers) return PT_ERR_NULL;
    for (int i = 0; i < n; ++i) {
        const pt_layer_lasso& L = layers[i];
        if (!L.w || !L.out_norm || !L.in_norm || !L.dw) return PT_ERR_NULL;
        if (L.K <= 0 || L.RS <= 0 || L.C <= 0 || L.w_cpitch < L.C) return PT_ERR_SHAPE;
        if (L.flags & ~3u) return PT_ERR_UNSUPPORTED;
    }
    std::vector<LassoLayer> v;
    if (!make_table(v, n)) return PT_ERR_UNSUPPORTED;
    for (int i = 0; i < n; ++i) {
        const pt_layer_lasso& L = layers[i];
        v[i] = LassoLayer{L.w, L.out_norm, L.in_norm, L.dw, nullptr, L.K, L.RS, L.C, L.w_cpitch, L.flags};
    }
    return launch_lasso(v.data(), n, false, lambda, StepParams{0.f, 0.f, 0.f}, (hipStream_t)stream);
}

extern "C" int32_t pt_sgd_momentum_lasso_batched(const pt_layer_update* layers, int32_t n, float lambda, float lr,
                                                 float momentum, float weight_decay, void* stream) {
    if (n < 0) return PT_ERR_SHAPE;
    if (n == 0) return PT_OK;
    if (!layers) return PT_ERR_NULL;
    for (int i = 0; i < n; ++i) {
        const pt_layer_update& L = layers[i];
        if (!L.w || !L.dw || !L.mom || !L.out_norm || !L.in_norm) return PT_ERR_NULL;
        if (L.K <= 0 || L.RS <= 0 || L.C <= 0 || L.w_cpitch < L.C) return PT_ERR_SHAPE;
        if (L.flags & ~3u) return PT_ERR_UNSUPPORTED;
    }
    std::vector<LassoLayer> v;
    if (!make_table(v, n)) return PT_ERR_UNSUPPORTED;
    for (int i = 0; i < n; ++i) {
        const pt_layer_update& L = layers[i];
        v[i] = LassoLayer{L.w, L.out_norm, L.in_norm, const_cast<float*>(L.dw), L.mom, L.K, L.RS, L.C, L.w_cpitch, L.flags};
    }
    return launch_lasso(v.data(), n, true, lambda, StepParams{lr, momentum, weight_decay}, (hipStream_t)stream);
}

// ---- single-layer forms: the batched calls with one entry ------------------------------------- //
extern "C" int32_t pt_group_norms_workspace_bytes(int32_t K, int32_t RS, int32_t C, size_t* bytes) {
    if (!bytes) return PT_ERR_NULL;
    if (K <= 0 || RS <= 0 || C <= 0) return PT_ERR_SHAPE;
    *bytes = norm_layer_ws_bytes(K, RS, C);
    return PT_OK;
}

extern "C" int32_t pt_group_norms(const float* w, int32_t K, int32_t RS, int32_t C, int32_t w_cpitch, float* out_norm,
                                  float* in_norm, uint16_t* w_shadow, void* ws, size_t ws_bytes, void* stream) {
    if (!w || !out_norm || !in_norm || !ws) return PT_ERR_NULL;
    pt_layer_weights L{};
    L.w = w; L.K = K; L.RS = RS; L.C = C; L.w_cpitch = w_cpitch;
    L.out_norm = out_norm; L.in_norm = in_norm; L.w_shadow = w_shadow;
    return pt_group_norms_batched(&L, 1, ws, ws_bytes, stream);
}

extern "C" int32_t pt_group_lasso_grad(const float* w, const float* out_norm, const float* in_norm, float lambda,
                                       uint32_t flags, float* dw, int32_t K, int32_t RS, int32_t C, int32_t w_cpitch,
                                       void* stream) {
    pt_layer_lasso L{};
    L.w = w; L.out_norm = out_norm; L.in_norm = in_norm; L.dw = dw;
    L.K = K; L.RS = RS; L.C = C; L.w_cpitch = w_cpitch; L.flags = flags;
    return pt_group_lasso_grad_batched(&L, 1, lambda, stream);
}

extern "C" int32_t pt_group_lasso_penalty_batched(const pt_layer_penalty* layers, int32_t n, double* penalty_dev,
                                                  void* stream) {
    if (n < 0) return PT_ERR_SHAPE;
    if (!penalty_dev || (n > 0 && !layers)) return PT_ERR_NULL;
    for (int i = 0; i < n; ++i) {
        if (layers[i].K < 0 || layers[i].C < 0) return PT_ERR_SHAPE;
        if (layers[i].flags & ~(PT_LASSO_OUT | PT_LASSO_IN)) return PT_ERR_UNSUPPORTED;
        if (((layers[i].flags & PT_LASSO_OUT) && layers[i].K > 0 && !layers[i].out_norm) ||
            ((layers[i].flags & PT_LASSO_IN) && layers[i].C > 0 && !layers[i].in_norm))
            return PT_ERR_NULL;
    }
    PenaltyJobs jobs;
    jobs.n = 0;
    jobs.accumulate = 0;
    int i = 0;
    do {  // at least one launch, so that n == 0 writes 0
        for (; i < n && jobs.n < kMaxPenaltyJobs; ++i) {
            const pt_layer_penalty& L = layers[i];
            jobs.j[jobs.n++] = PenaltyJob{L.out_norm, L.in_norm, (L.flags & PT_LASSO_OUT) ? L.K : 0,
                                          (L.flags & PT_LASSO_IN) ? L.C : 0};
        }
        hipLaunchKernelGGL(k_group_lasso_penalty, dim3(1), dim3(1024), 0, (hipStream_t)stream, jobs, penalty_dev);
        const int32_t rc = launch_status();
        if (rc != PT_OK) return rc;
        jobs.n = 0;
        jobs.accumulate = 1;
    } while (i < n);
    return PT_OK;
}

extern "C" int32_t pt_lasso_set_coeff(double loss1, double loss2, double ratio, double* lambda) {
    if (!lambda) return PT_ERR_NULL;
    if (!(ratio > 0.0 && ratio < 1.0) || !(loss2 > 0.0) || !(loss1 >= 0.0)) return PT_ERR_SHAPE;
    *lambda = ratio * loss1 / ((1.0 - ratio) * loss2);
    return PT_OK;
}
